"""Staged products (x entries of a row group copied to LDS, shared row
patterns): against the oracle, and bitwise against the unstaged product
(spmv_batch reads the per-slot stream), at the edges of what the staging
rule accepts."""
import numpy as np
import pytest

import paper_1501_00324_amd as fs
from workloads.meshes import CSR
from tests.gpu_util import assert_spmv_close, dev, host, make, note

pytestmark = pytest.mark.gpu


def block_matrix(nodes, dof, per_node, span, seed, n_cols=None, empty=()):
    """Rows in runs of `dof` with equal columns; `per_node` (a range) nodes
    per row within `span` of the diagonal (0: anywhere), unsorted."""
    g = np.random.default_rng(seed)
    n_cols = n_cols or nodes * dof
    rowptr, col = [0], []
    for i in range(nodes):
        k = 0 if i in empty else int(g.integers(*per_node))
        lo, hi = (0, n_cols // dof) if not span else (max(0, i - span), min(n_cols // dof, i + span + 1))
        nb = g.choice(np.arange(lo, hi), min(k, hi - lo), replace=False)
        cols = (nb[:, None] * dof + np.arange(dof)).reshape(-1)
        for _ in range(dof):
            c = g.permutation(cols)
            col.append(c)
            rowptr.append(rowptr[-1] + len(c))
    col = np.concatenate(col).astype(np.int32) if col else np.zeros(0, np.int32)
    return CSR(len(rowptr) - 1, n_cols, np.array(rowptr, np.int32), col,
               g.uniform(-1, 1, len(col)))


CASES = {
    # three unknowns per node, patterns cut by group ends, partial last group
    "three": dict(nodes=347, dof=3, per_node=(3, 16), span=20),
    # six rows of equal columns: more than one pattern of four
    "six": dict(nodes=113, dof=6, per_node=(2, 9), span=9),
    # several lanes per row, patterns shared
    "lanes": dict(nodes=131, dof=3, per_node=(30, 60), span=60),
    # empty rows, and a group without entries
    "empty": dict(nodes=200, dof=3, per_node=(1, 5), span=8, empty=range(60, 130)),
    # one unknown per node, and one row
    "single": dict(nodes=500, dof=1, per_node=(1, 20), span=30),
    "one row": dict(nodes=1, dof=1, per_node=(1, 2), span=0),
    # rectangular
    "wide": dict(nodes=150, dof=2, per_node=(2, 12), span=0, n_cols=80),
    # columns anywhere: too many distinct ones per slot, not staged
    "scattered": dict(nodes=3000, dof=1, per_node=(8, 30), span=0),
    # groups span more than 16-bit offsets, 32-bit lists
    "far": dict(nodes=40000, dof=3, per_node=(2, 3), span=0),
}


@pytest.mark.parametrize("vec", [0, 1, 2])
@pytest.mark.parametrize("name", sorted(CASES))
def test_staged_product(orc, name, vec):
    note("staged product %s vec=%d" % (name, vec))
    A = block_matrix(seed=7, **CASES[name])
    M = make(A, reorder=fs.REORDER_NONE, vec=vec)
    x = np.random.default_rng(8).uniform(-1, 1, A.n_cols)
    y = host(fs.spmv(M, dev(x)))
    assert_spmv_close(y, orc.spmv(A, x), orc.spmv_abs(A, x), name)
    assert np.array_equal(y, host(fs.spmv_batch([M], [dev(x)])[0]))


@pytest.mark.parametrize("bits", [0, 32])
@pytest.mark.parametrize("name", ["three", "lanes", "single"])
def test_staged_keeps_padding_from_x(name, bits):
    """An infinity in x reaches exactly the rows that reference it."""
    note("staged padding %s bits=%d" % (name, bits))
    A = block_matrix(seed=9, **CASES[name])
    M = make(A, index_bits=bits)
    rows = np.repeat(np.arange(A.n_rows), np.diff(A.rowptr))
    for j in (0, A.n_cols // 2, A.n_cols - 1):
        x = np.ones(A.n_cols)
        x[j] = np.inf
        hit = np.zeros(A.n_rows, bool)
        hit[rows[A.col == j]] = True
        assert np.array_equal(~np.isfinite(host(fs.spmv(M, dev(x)))), hit)


@pytest.mark.parametrize("dtype", [fs.DT_F32, fs.DT_BF16])
@pytest.mark.parametrize("name", ["three", "six", "lanes", "single"])
def test_staged_low_precision(orc, name, dtype):
    """Float sums within their rounding bound gamma_m (|A||x|), m = the
    longest row plus the reduction's few steps."""
    note("staged low precision %s dtype=%d" % (name, dtype))
    A = block_matrix(seed=11, **CASES[name])
    M = make(A, dtypes=dtype)
    x = np.random.default_rng(12).uniform(-1, 1, A.n_cols).astype(np.float32)
    perm = fs.csr_get_perm(M)
    y = host(fs.spmv_lowp(M, dtype, dev(x[perm])))
    v = orc.round_f32(A.val) if dtype == fs.DT_F32 else orc.bf16_bits_to_f32(orc.round_bf16(A.val))
    R = CSR(A.n_rows, A.n_cols, A.rowptr, A.col, np.asarray(v, np.float64))
    xd = x.astype(np.float64)
    bound = (np.diff(A.rowptr).max() + 8) * 2.0 ** -24 * orc.spmv_abs(R, xd)
    assert np.all(np.abs(y - orc.spmv(R, xd)[perm]) <= bound[perm])


@pytest.mark.parametrize("k", [2, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("name", ["three", "six", "lanes", "empty", "wide", "far"])
def test_tile_product(orc, name, k):
    """Several columns, matrices whose rows share columns (matrix cores from
    three columns on), row strides over k, both slot widths."""
    note("tile product %s k=%d" % (name, k))
    A = block_matrix(seed=13, **CASES[name])
    for vec in (1, 2):
        M = make(A, vec=vec)
        X = np.random.default_rng(14).uniform(-1, 1, (A.n_cols, k))
        Y = host(fs.spmm(M, dev(X)))
        scale = np.stack([orc.spmv_abs(A, X[:, c]) for c in range(k)], 1)
        assert_spmv_close(Y, orc.spmm(A, X), scale, "%s k=%d" % (name, k))


@pytest.mark.parametrize("k", [4, 7, 16])
def test_tile_padding_and_infinity(k):
    """An infinity in one column of X stays in that column and in the rows
    that reference it."""
    note("tile infinity k=%d" % k)
    A = block_matrix(seed=15, **CASES["three"])
    M = make(A)
    rows = np.repeat(np.arange(A.n_rows), np.diff(A.rowptr))
    for j, c in ((0, 0), (A.n_cols // 2, k - 1), (A.n_cols - 1, 1)):
        X = np.ones((A.n_cols, k))
        X[j, c] = np.inf
        hit = np.zeros((A.n_rows, k), bool)
        hit[rows[A.col == j], c] = True
        assert np.array_equal(~np.isfinite(host(fs.spmm(M, dev(X)))), hit)


@pytest.mark.parametrize("vec", [1, 2])
@pytest.mark.parametrize("lanes", [0, 2, 8, 16, 32])
@pytest.mark.parametrize("name", ["three", "lanes", "empty", "single", "one row", "wide"])
def test_refresh_rows_in_lds(name, lanes, vec):
    """New values land in their slots whatever the lanes per row (over 16 the
    rows are gathered), unsorted rows included: bitwise a fresh handle."""
    note("refresh %s lanes=%d vec=%d" % (name, lanes, vec))
    A = block_matrix(seed=17, **CASES[name])
    opts = dict(vec=vec, lanes_min=lanes, lanes_max=lanes, dtypes=fs.DT_F32 | fs.DT_BF16)
    new = np.random.default_rng(18).uniform(-1, 1, A.nnz)
    M = make(A, **opts)
    fs.csr_update_values(M, dev(new))
    F = make(CSR(A.n_rows, A.n_cols, A.rowptr, A.col, new), **opts)
    assert np.array_equal(host(fs.csr_get_values(M)), new)
    x = dev(np.random.default_rng(19).uniform(-1, 1, A.n_cols))
    assert np.array_equal(host(fs.spmv(M, x)), host(fs.spmv(F, x)))
    if A.n_rows == A.n_cols:
        for d in (fs.DT_F32, fs.DT_BF16):
            assert np.array_equal(host(fs.spmv_lowp(M, d, x.float())),
                                  host(fs.spmv_lowp(F, d, x.float())))
