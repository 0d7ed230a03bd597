"""Kept graphs of a handle over solves of different check_every."""
import numpy as np
import pytest

import paper_1501_00324_amd as fs
import workloads as W
from tests.gpu_util import dev, host, make, note

pytestmark = pytest.mark.gpu


def test_foreign_chunk_lengths_before_the_default():
    """check_every 3, then 5, then the default on one handle, nothing in
    between that drops its graphs: the bits and iterations of a solve without
    graphs."""
    note("check_every 3, 5, default")
    A = W.config0_poisson2d()
    b = dev(np.random.default_rng(21).uniform(-1, 1, A.n_rows))
    ref, info = fs.cg_solve(make(A), b, use_graph=0, check_every=1)
    M = make(A)
    for every in (3, 5, 0, 0, 3, 16, 0, 4, 0):
        x, d = fs.cg_solve(M, b, check_every=every)
        assert np.array_equal(host(x), host(ref)), every
        assert d["iters"] == info["iters"], every


def test_all_iterations_of_an_unreachable_tolerance():
    """A tolerance whose square underflows runs maxit iterations."""
    note("rtol 1e-200")
    A = W.config0_poisson2d()
    b = dev(np.random.default_rng(22).uniform(-1, 1, A.n_rows))
    M = make(A)
    ref, _ = fs.cg_solve(M, b, rtol=1e-200, maxit=50, use_graph=0, check_every=1, check=False)
    x, d = fs.cg_solve(M, b, rtol=1e-200, maxit=50, check=False)
    assert d["status"] == fs.FS_E_NOT_CONVERGED and d["iters"] == 50
    assert np.array_equal(host(x), host(ref))
