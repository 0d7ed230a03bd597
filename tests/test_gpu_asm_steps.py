"""Assembly over every number of steps of a batch (rows in 0 to 24 elements
each, whole and partial blocks of eight steps), in few and in many row groups:
bitwise the oracle's element loop."""
import itertools

import numpy as np
import pytest

import paper_1501_00324_amd as fs
from workloads.meshes import CSR
from tests.gpu_util import dev, host, make, note

pytestmark = pytest.mark.gpu


def connectivity(kind, n):
    """Nodes of every element of a grid of n nodes per direction."""
    d = 2 if kind == "tri" else 3
    cells = np.stack(np.meshgrid(*[np.arange(n - 1)] * d, indexing="ij"), -1).reshape(-1, d)
    if kind == "tri":
        subs = [[(0, 0), (1, 0), (1, 1)], [(0, 0), (1, 1), (0, 1)]]
    elif kind == "tet":
        subs = []
        for s in itertools.permutations(range(3)):
            t = [np.zeros(3, int)]
            for ax in s:
                t.append(t[-1] + np.eye(3, dtype=int)[ax])
            subs.append(t)
    else:
        subs = [list(itertools.product((0, 1), repeat=3))]
    stride = n ** np.arange(d)[::-1]
    return np.concatenate([(cells[:, None] + np.array(t)[None]) @ stride for t in subs])


def system(kind, n, dof, drop, seed):
    """Pattern of the whole mesh, a random part of its elements in random
    order with random values, some unknowns without a row (-1)."""
    g = np.random.default_rng(seed)
    e = connectivity(kind, n)
    rows = int(e.max()) + 1
    edof = (e[:, :, None] * dof + np.arange(dof)).reshape(len(e), -1).astype(np.int32)
    i, j = np.repeat(edof, edof.shape[1], 1).reshape(-1), np.tile(edof, edof.shape[1]).reshape(-1)
    pair = np.unique(i.astype(np.int64) * (rows * dof) + j)
    r, c = pair // (rows * dof), pair % (rows * dof)
    rowptr = np.zeros(rows * dof + 1, np.int32)
    rowptr[1:] = np.cumsum(np.bincount(r, minlength=rows * dof))
    A = CSR(rows * dof, rows * dof, rowptr, c.astype(np.int32), np.zeros(len(c)))
    edof = edof[g.permutation(len(edof))[:int(len(edof) * (1 - drop))]]
    edof[g.random(edof.shape) < 0.02] = -1
    nde = edof.shape[1]
    return A, edof, g.uniform(-1, 1, (len(edof), nde, nde)), g.uniform(-1, 1, (len(edof), nde))


# up to 512 row groups (32,768 rows of one lane) and more
@pytest.mark.parametrize("kind,n,dof", [("tri", 20, 1), ("tri", 190, 1), ("tri", 12, 3), ("tet", 7, 1), ("tet", 33, 1),
                                        ("tet", 6, 3), ("tet", 23, 3), ("hex", 6, 1), ("hex", 5, 3), ("hex", 23, 3)])
@pytest.mark.parametrize("drop", [0.0, 0.3, 0.8])
def test_steps(orc, kind, n, dof, drop):
    note("asm steps %s n=%d dof=%d drop=%.1f" % (kind, n, dof, drop))
    A, edof, ke, re = system(kind, n, dof, drop, seed=n)
    M = make(A)
    P = fs.asm_create(M, dev(edof), plan=fs.ASM_ROWGROUP)
    want = orc.assemble_matrix(A, edof, ke).view(np.int64)
    r_want = orc.assemble_vector(A.n_rows, edof, re).view(np.int64)

    def values():
        return host(fs.csr_get_values(M)).view(np.int64)
    fs.asm_matrix(P, dev(ke))
    assert np.array_equal(values(), want)
    fs.csr_update_values(M, dev(A.val + 1.0))
    r = host(fs.asm_system(P, dev(ke), dev(re))).view(np.int64)
    assert np.array_equal(values(), want) and np.array_equal(r, r_want)
    pos, rows = fs.asm_element_rows(P)
    ko = np.full((rows, edof.shape[1]), np.nan)
    ko[pos[pos >= 0]] = ke.reshape(-1, edof.shape[1])[pos >= 0]
    fs.csr_update_values(M, dev(A.val + 1.0))
    fs.asm_matrix_ordered(P, dev(ko))
    assert np.array_equal(values(), want)
