"""Which form a product takes at the edges of the rules, and the strided forms
of the multi-column products."""
import ctypes as C

import numpy as np
import pytest

import paper_1501_00324_amd as fs
import workloads as W
from workloads.meshes import CSR
from tests.gpu_util import STAGED, STAGED16, STAGED64, TILES, TILES8, TILES16, REFRESH_TILES, assert_spmv_close, dev, forms, host, make, note
from tests.test_gpu_stage import CASES, block_matrix

pytestmark = pytest.mark.gpu

# the forms that the cases of tests/test_gpu_stage.py run in.  "single": rows
# are sorted by length inside windows, so a group references most of its
# window: 0.46 distinct columns per slot, 0.44 with the slots in pairs, whose
# padding counts ("single" is staged then; one unknown per node and staged
# without pairs: tests/test_gpu_stage_widths.py).
EXPECTED = {"three": STAGED | TILES, "six": STAGED | TILES, "lanes": STAGED | TILES8 | TILES16, "empty": STAGED | TILES,
            "single": 0, "one row": 0, "wide": STAGED, "scattered": 0, "far": STAGED | TILES}


@pytest.mark.parametrize("vec", [0, 1, 2])
@pytest.mark.parametrize("name", sorted(EXPECTED))
def test_forms_of_the_stage_cases(name, vec):
    note("forms %s vec=%d" % (name, vec))
    M = make(block_matrix(seed=7, **CASES[name]), reorder=fs.REORDER_NONE, vec=vec)
    want = STAGED if name == "single" and vec == 2 else EXPECTED[name]
    assert forms(M) & ~STAGED16 == want | (STAGED64 if want else 0) | REFRESH_TILES


@pytest.mark.parametrize("permute,bf16", [(False, False), (True, True)])
def test_runs_of_neighbours(orc, permute, bf16):
    """Q1 Laplacian in natural numbering: the lanes of a slot gather runs of
    neighbouring columns, and the BF16 product does so without staging."""
    note("runs permute=%d" % permute)
    A = W.hex_q1(41, "laplace", seed=(93, 0), permute=permute)
    M = make(A, dtypes=fs.DT_F32 | fs.DT_BF16)
    assert fs.csr_info(M)["vec"] == 2
    assert forms(M) & STAGED64 and forms(M) & STAGED and bool(forms(M) & STAGED16) == bf16
    x = np.random.default_rng(3).uniform(-1, 1, A.n_cols).astype(np.float32)
    perm = fs.csr_get_perm(M)
    R = CSR(A.n_rows, A.n_cols, A.rowptr, A.col, np.asarray(orc.bf16_bits_to_f32(orc.round_bf16(A.val)), np.float64))
    xd = x.astype(np.float64)
    bound = (27 + 8) * 2.0 ** -24 * orc.spmv_abs(R, xd)
    y = host(fs.spmv_lowp(M, fs.DT_BF16, dev(x[perm])))
    assert np.all(np.abs(y - orc.spmv(R, xd)[perm]) <= bound[perm])
    b = dev(np.random.default_rng(4).uniform(-1, 1, A.n_rows))
    S = make(CSR(A.n_rows, A.n_cols, A.rowptr, A.col, shifted(A)))
    X, info = fs.cg_solve(S, b, precision=fs.PREC_IR_BF16)
    assert info["relres"] <= 1e-8


@pytest.mark.parametrize("n,f32", [(60, True), (77, False)])
def test_float_runs_of_neighbours(orc, n, f32):
    """The FP32 product of a Q1 Laplacian in natural numbering gathers per
    slot where its slots take 64 to 180 MB."""
    note("float runs n=%d" % n)
    A = W.hex_q1(n, "laplace", seed=(94, 0), permute=False)
    M = make(A, dtypes=fs.DT_F32)
    assert fs.csr_info(M)["vec"] == 2
    assert forms(M) & STAGED64 and bool(forms(M) & STAGED) == f32
    x = np.random.default_rng(5).uniform(-1, 1, A.n_cols).astype(np.float32)
    perm = fs.csr_get_perm(M)
    R = CSR(A.n_rows, A.n_cols, A.rowptr, A.col, A.val.astype(np.float32).astype(np.float64))
    xd = x.astype(np.float64)
    bound = (27 + 8) * 2.0 ** -24 * orc.spmv_abs(R, xd)
    y = host(fs.spmv_lowp(M, fs.DT_F32, dev(x[perm])))
    assert np.all(np.abs(y - orc.spmv(R, xd)[perm]) <= bound[perm])
    b = dev(np.random.default_rng(6).uniform(-1, 1, A.n_rows))
    S = make(CSR(A.n_rows, A.n_cols, A.rowptr, A.col, shifted(A)))
    X, info = fs.cg_solve(S, b, precision=fs.PREC_IR_F32)
    assert info["relres"] <= 1e-8


def shifted(A):
    """The values with twice the diagonal (positive definite)."""
    rows = np.repeat(np.arange(A.n_rows), np.diff(A.rowptr))
    return np.where(A.col == rows, 2.0 * A.val, A.val)


def test_one_row(orc):
    note("one staged row")
    A = CSR(1, 9, np.array([0, 7], np.int32), np.array([8, 0, 3, 5, 4, 2, 7], np.int32), np.arange(1.0, 8.0))
    M = make(A)
    assert forms(M) & STAGED64
    x = np.arange(9.0)
    assert np.array_equal(host(fs.spmv(M, dev(x))), orc.spmv(A, x))


def long_rows(distinct, shared, rows=64):
    """One row group of `rows` rows that reference `distinct` columns
    together, every row three quarters of them, `shared` rows the same."""
    g = np.random.default_rng(distinct)
    each = distinct * 3 // 4
    cols = [np.arange(each), np.arange(distinct - each, distinct)]
    cols += [g.choice(distinct, each, replace=False) for _ in range(rows)]
    cols = [c for c in cols for _ in range(shared)][:rows]
    rowptr = np.arange(rows + 1, dtype=np.int32) * each
    return CSR(rows, 20000, rowptr, np.concatenate(cols).astype(np.int32), g.uniform(-1, 1, rows * each))


@pytest.mark.parametrize("shared", [1, 3])
@pytest.mark.parametrize("distinct", [1023, 1024, 1280, 1281])
def test_widest_group(orc, distinct, shared):
    """A group of 1,280 distinct columns fills the LDS; one more is gathered
    per slot, in FP64 over 1,023 where the rows do not share their columns.
    (Lanes fixed to one: all rows in one group.)"""
    note("widest group %d shared=%d" % (distinct, shared))
    A = long_rows(distinct, shared)
    M = make(A, reorder=fs.REORDER_NONE, lanes_min=1, lanes_max=1)
    assert fs.csr_info(M)["n_groups"] == 1
    assert bool(forms(M) & STAGED) == (distinct <= 1280)
    assert bool(forms(M) & STAGED64) == (distinct <= (1280 if shared == 3 else 1023))
    x = np.random.default_rng(1).uniform(-1, 1, A.n_cols)
    y = host(fs.spmv(M, dev(x)))
    assert np.array_equal(y, host(fs.spmv_batch([M], [dev(x)])[0]))
    assert_spmv_close(y, orc.spmv(A, x), orc.spmv_abs(A, x))


@pytest.mark.parametrize("span,staged", [(327680, True), (327681, False)])
def test_widest_span(orc, span, staged):
    """Columns of a group spread over 327,680 columns (the bitmap that finds
    them), and over one more."""
    note("widest span %d" % span)
    g = np.random.default_rng(2)
    shared = np.sort(g.choice(span - 2, 30, replace=False)) + 1
    cols = np.tile(np.concatenate([[0], shared, [span - 1]]), 64).astype(np.int32)
    A = CSR(64, span, np.arange(65, dtype=np.int32) * 32, cols, g.uniform(-1, 1, len(cols)))
    M = make(A, reorder=fs.REORDER_NONE)
    assert bool(forms(M) & STAGED) == staged
    x = g.uniform(-1, 1, span)
    y = host(fs.spmv(M, dev(x)))
    assert np.array_equal(y, host(fs.spmv_batch([M], [dev(x)])[0]))
    assert_spmv_close(y, orc.spmv(A, x), orc.spmv_abs(A, x))


def strided_spmm(M, X, k, ldx, ldy):
    """fs spmm on rows of ldx and ldy values; the columns past k of Y keep
    the sentinel."""
    import torch
    Xd = torch.full((M.n_cols, ldx), float("nan"), dtype=torch.float64, device="cuda")
    Xd[:, :k] = dev(X)
    Yd = torch.full((M.n_rows, ldy), 7.25, dtype=torch.float64, device="cuda")
    st = fs.load().spmm(C.c_void_p(M._h), k, C.c_void_p(Xd.data_ptr()), ldx, C.c_void_p(Yd.data_ptr()), ldy, None)
    assert st == fs.FS_OK, fs.last_error()
    torch.cuda.synchronize()
    Y = host(Yd)
    assert np.all(Y[:, k:] == 7.25)
    return Y[:, :k]


@pytest.mark.parametrize("k", [2, 3, 4, 5, 7, 8, 9, 15, 16])
@pytest.mark.parametrize("name", ["three", "six", "lanes", "single", "wide"])
def test_rows_longer_than_k(orc, name, k):
    """Row strides of X and Y over k (odd and even: pairs of columns at
    8-byte addresses), the caller's numbering and a permuted one; NaN in the
    unused columns of X reaches nothing."""
    note("spmm strides %s k=%d" % (name, k))
    A = block_matrix(seed=23, **CASES[name])
    X = np.random.default_rng(24).uniform(-1, 1, (A.n_cols, k))
    ref = orc.spmm(A, X)
    scale = np.stack([orc.spmv_abs(A, X[:, c]) for c in range(k)], 1)
    for opts in (dict(reorder=fs.REORDER_NONE, sort_window=1), dict()):
        M = make(A, **opts)
        plain = host(fs.spmm(M, dev(X)))
        for more in (0, 1, 2, 3):
            Y = strided_spmm(M, X, k, k + more, k + 3 - more)
            assert np.array_equal(Y, plain)
            assert_spmv_close(Y, ref, scale, "%s k=%d +%d" % (name, k, more))


@pytest.mark.parametrize("ldx", [131007, 131009])
def test_stride_past_31_bit_offsets(orc, ldx):
    """The widest rows of X that the matrix-core product's 31-bit byte offsets
    reach (2,049 columns of 131,007 values are 2^31 - 128 bytes less a few),
    and rows past them, which take the other form."""
    import torch
    note("spmm ldx=%d" % ldx)
    A = block_matrix(nodes=683, dof=3, per_node=(3, 10), span=20, seed=25)
    M = make(A, reorder=fs.REORDER_NONE, sort_window=1)
    assert forms(M) & TILES8 and A.n_cols == 2049
    k = 5
    X = np.random.default_rng(26).uniform(-1, 1, (A.n_cols, k))
    Xd = torch.zeros(A.n_cols * ldx, dtype=torch.float64, device="cuda").view(A.n_cols, ldx)
    Xd[:, :k] = dev(X)
    Y = torch.empty(A.n_rows, k, dtype=torch.float64, device="cuda")
    assert fs.load().spmm(C.c_void_p(M._h), k, C.c_void_p(Xd.data_ptr()), ldx, C.c_void_p(Y.data_ptr()), k, None) == fs.FS_OK
    scale = np.stack([orc.spmv_abs(A, X[:, c]) for c in range(k)], 1)
    assert_spmv_close(host(Y), orc.spmm(A, X), scale)
