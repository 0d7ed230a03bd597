"""Staged products over every row length: the last batch of a row's slots has
a block of its own for each of its lengths (batches of 8)."""
import numpy as np
import pytest

import paper_1501_00324_amd as fs
from workloads.meshes import CSR
from tests.gpu_util import STAGED, STAGED64, assert_spmv_close, dev, forms, host, make, note

pytestmark = pytest.mark.gpu


def band(n, width, dof=1, seed=31):
    """Rows of exactly `width` * dof entries near the diagonal, in runs of
    `dof` rows with equal columns."""
    g = np.random.default_rng(seed + width)
    m = n // dof
    first = np.clip(np.arange(m) - width // 2, 0, m - width)
    nodes = first[:, None] + np.arange(width)
    cols = (nodes[:, :, None] * dof + np.arange(dof)).reshape(m, -1)
    col = np.repeat(cols, dof, axis=0).astype(np.int32)
    rowptr = np.arange(m * dof + 1, dtype=np.int32) * col.shape[1]
    return CSR(m * dof, m * dof, rowptr, col.reshape(-1), g.uniform(-1, 1, col.size))


@pytest.mark.parametrize("vec", [1, 2])
@pytest.mark.parametrize("dof", [1, 3])
def test_every_row_length(orc, dof, vec):
    """FP64 bitwise the product that gathers per slot (spmv_batch), and within
    1e-12 of the oracle; FP32 and BF16 within the rounding bound of a float
    sum of that many terms."""
    for width in list(range(1, 37)) + [47, 48]:
        if dof == 3 and width > 16:
            break
        note("staged width=%d dof=%d vec=%d" % (width, dof, vec))
        A = band(210, width, dof)
        M = make(A, reorder=fs.REORDER_NONE, vec=vec, dtypes=fs.DT_F32 | fs.DT_BF16)
        slots = -(-dof * width // vec) * vec
        assert bool(forms(M) & STAGED) == bool(forms(M) & STAGED64) == (slots > 4)
        x = np.random.default_rng(width).uniform(-1, 1, A.n_cols)
        y = host(fs.spmv(M, dev(x)))
        assert np.array_equal(y, host(fs.spmv_batch([M], [dev(x)])[0]))
        assert_spmv_close(y, orc.spmv(A, x), orc.spmv_abs(A, x), "width %d" % width)
        perm = fs.csr_get_perm(M)
        x32 = x.astype(np.float32)
        for dtype in (fs.DT_F32, fs.DT_BF16):
            v = orc.round_f32(A.val) if dtype == fs.DT_F32 else orc.bf16_bits_to_f32(orc.round_bf16(A.val))
            R = CSR(A.n_rows, A.n_cols, A.rowptr, A.col, np.asarray(v, np.float64))
            xd = x32.astype(np.float64)
            bound = (width * dof + 8) * 2.0 ** -24 * orc.spmv_abs(R, xd)
            z = host(fs.spmv_lowp(M, dtype, dev(x32[perm])))
            assert np.all(np.abs(z - orc.spmv(R, xd)[perm]) <= bound[perm])
