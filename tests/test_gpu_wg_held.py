"""One-workgroup solves whose slots stay in registers."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_util import dev, host, make, note
from tests.test_gpu_wg import fs, true_relres  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,lo", [(10, 0), (18, 0), (34, 0), (57, 0), (57, 1),
                                  (60, 0)])
def test_wg_slots_in_registers(fs, orc, n, lo):
    """Systems whose slots a workgroup holds in registers (one lane per row,
    at most 8 slots, up to 48 row groups) and the first beyond (3,364 rows,
    53 groups; 57 x 57 nodes without the boundary are 48 groups): bitwise the
    other workgroup sizes, alone and with a wider system in the batch."""
    note("cg wg held n=%d lo=%d" % (n, lo))
    A = W.poisson_2d_p1(n, seed=(78, n), bc="all", permute=bool(lo))
    wide = W.tet_p1(6, "laplace", seed=(78, 1), bc="all")
    M, Mw = make(A), make(wide)
    b = W.random_vector(A.n_rows, 78, W.BVEC, 0)
    bw = W.random_vector(wide.n_rows, 78, W.BVEC, 1)
    for precond in (0, 1):
        for x0 in (None, W.random_vector(A.n_rows, 78, W.XVEC, 2)):
            out = []
            for threads, other in ((256, False), (0, False), (1024, False),
                                   (1024, True)):
                Ms, bs = [M], [dev(b)]
                xs = None if x0 is None else [dev(x0)]
                if other:
                    Ms.append(Mw)
                    bs.append(dev(bw))
                    if xs is not None:
                        xs.append(dev(np.zeros(wide.n_rows)))
                got, inf = fs.cg_solve_batch_wg(Ms, bs, xs, precond=precond,
                                                wg_threads=threads)
                out.append((host(got[0]), inf[0]["iters"]))
            assert true_relres(orc, A, out[0][0], b) <= 1.001e-8
            for x, it in out[1:]:
                assert np.array_equal(x, out[0][0]) and it == out[0][1]
