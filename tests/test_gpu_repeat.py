"""Repeated solves on one handle: graphs and descriptors kept between solves,
chunk lengths chosen from the rate of convergence.  The results do not
depend on any of it."""
import numpy as np
import pytest

import paper_1501_00324_amd as fs
import workloads as W
from tests.gpu_util import dev, host, make, note

pytestmark = pytest.mark.gpu


def test_repeated_solves_agree():
    note("repeated solves")
    A = W.config0_poisson2d()
    M = make(A)
    b = dev(np.random.default_rng(3).uniform(-1, 1, A.n_rows))
    B = dev(np.random.default_rng(4).uniform(-1, 1, (A.n_rows, 3)))
    ref, info = fs.cg_solve(M, b, use_graph=0, check_every=1)
    refm, infom = fs.cg_solve_multi(M, B, use_graph=0, check_every=1)
    for every in (0, 1, 3, 4, 12, 32, 1000, 32):
        for graph in (1, 0, 1):
            x, d = fs.cg_solve(M, b, use_graph=graph, check_every=every)
            assert np.array_equal(host(x), host(ref))
            assert d["iters"] == info["iters"]
        X, ds = fs.cg_solve_multi(M, B, check_every=every)
        assert np.array_equal(host(X), host(refm))
        assert [d["iters"] for d in ds] == [d["iters"] for d in infom]


def test_solve_after_failures():
    """An iteration limit, a bad diagonal and new values between solves."""
    note("solves around failures")
    A = W.config0_poisson2d()
    M = make(A)
    b = dev(np.random.default_rng(5).uniform(-1, 1, A.n_rows))
    ref, info = fs.cg_solve(M, b)
    for maxit in (1, 5, 33):
        _, d = fs.cg_solve(M, b, maxit=maxit, check=False)
        assert d["status"] == fs.FS_E_NOT_CONVERGED and d["iters"] == maxit
    rows = np.repeat(np.arange(A.n_rows), np.diff(A.rowptr))
    bad = A.val.copy()
    bad[(rows == A.col) & (rows == 17)] = 0.0
    fs.csr_update_values(M, dev(bad))
    with pytest.raises(fs.FsError) as e:
        fs.cg_solve(M, b)
    assert e.value.status == fs.FS_E_ARG and "1 rows" in str(e.value)
    fs.csr_update_values(M, dev(A.val))
    x, d = fs.cg_solve(M, b)
    assert np.array_equal(host(x), host(ref)) and d["iters"] == info["iters"]


@pytest.mark.parametrize("precision", [fs.PREC_IR_F32, fs.PREC_IR_BF16])
@pytest.mark.parametrize("restart", [0, 1])
def test_refinement_pace(precision, restart):
    """Refinement steps take the same inner iterations whatever the chunks
    (check_every = 3 is taken as it is, 12 in chunks of 4)."""
    note("refinement pace precision=%d restart=%d" % (precision, restart))
    A = W.config0_poisson2d()
    M = make(A)
    b = dev(np.random.default_rng(6).uniform(-1, 1, A.n_rows))
    opts = dict(precision=precision, ir_restart=restart, max_outer=3, check=False)
    ref, info = fs.cg_solve(M, b, use_graph=0, check_every=12, **opts)
    for graph in (1, 0, 1):
        x, d = fs.cg_solve(M, b, use_graph=graph, check_every=12, **opts)
        assert np.array_equal(host(x), host(ref))
        assert (d["iters"], d["outer"]) == (info["iters"], info["outer"])


@pytest.mark.parametrize("vec", [1, 2])
@pytest.mark.parametrize("k", [2, 3, 4, 8, 9])
def test_batch_of_both_product_forms(k, vec):
    """Systems whose multi-column products run on the matrix cores (rows that
    share their columns) beside ones whose do not: every result is that of
    the system alone."""
    note("batch of both product forms k=%d vec=%d" % (k, vec))
    mats = [W.tet_p1(7, physics="elastic", bc="x0"), W.tet_p1(11, bc="all")]
    mats = [m for m in mats for _ in range(2)]
    Ms = [make(m, vec=vec) for m in mats]
    g = np.random.default_rng(10)
    Bs = [dev(g.uniform(-1, 1, (m.n_rows, k))) for m in mats]
    alone = [host(fs.cg_solve_multi(M, B)[0]) for M, B in zip(Ms, Bs)]
    Xs, _ = fs.cg_solve_batch(Ms, Bs)
    for X, ref in zip(Xs, alone):
        assert np.array_equal(host(X), ref)
    srv = fs.Server(check_every=4)
    subs = [srv.submit(M, B) for M, B in zip(Ms, Bs)]
    done = srv.drain()
    srv.close()
    assert len(done) == len(subs)
    for (_, X), ref in zip(subs, alone):
        assert np.array_equal(host(X), ref)
