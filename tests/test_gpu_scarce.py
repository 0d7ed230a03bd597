"""When device memory is short.  csr_create: an allocation that fails either
fails the creation with FS_E_OOM or, for the arrays of the staged products,
leaves a handle whose products gather per slot.  Solves: a handle whose
workspace could not grow solves on.  Every allocation fails once; a child
process resolves hipMalloc to a counting one."""
import os
import subprocess
import sys
import textwrap

import pytest

from tests.gpu_util import note

pytestmark = pytest.mark.gpu

SHIM = r"""
#include <dlfcn.h>
#include <stddef.h>
static int left = -1, seen = 0;
void arm(int n) { left = n; seen = 0; }
int count(void) { return seen; }
int hipMalloc(void **p, size_t n)
{
    static int (*real)(void **, size_t);
    if (!real) {
        void *h = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
        real = (int (*)(void **, size_t))dlsym(h, "hipMalloc");
    }
    ++seen;
    if (left >= 0 && left-- == 0) { *p = NULL; return 2; }   /* out of memory */
    return real(p, n);
}
"""

CHILD = r"""
import ctypes, sys
import numpy as np, torch
torch.cuda.init()
shim = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
import paper_1501_00324_amd as fs
import workloads as W
from tests.gpu_util import STAGED, forms, make, dev, host
fs.load(build_if_missing=False)
for build, bits in ((fs.BUILD_DEVICE, 0), (fs.BUILD_DEVICE, 32), (fs.BUILD_HOST, 0)):
    A = W.tet_p1(9, "elastic", seed=(91, 0), bc="x0", permute=True)
    t = dev(A.rowptr), dev(A.col), dev(A.val)
    x = dev(np.random.default_rng(0).uniform(-1, 1, A.n_cols))
    new = lambda: fs.csr_create(*t, build=build, index_bits=bits)
    shim.arm(-1)
    M = new()
    total = shim.count()
    assert total > 10 and forms(M) & STAGED
    ref = host(fs.spmv(M, x))
    kinds = ""
    for n in range(total):
        shim.arm(n)
        try:
            B = new()
        except fs.FsError as e:
            assert e.status == fs.FS_E_OOM, e
            kinds += "E"
            continue
        finally:
            shim.arm(-1)
        assert not forms(B) & STAGED
        assert np.array_equal(host(fs.spmv(B, x)), ref)
        fs.csr_update_values(B, t[2] * 2.0)
        assert np.array_equal(host(fs.spmv(B, x)), 2.0 * ref)
        assert fs.cg_solve(B, x, maxit=3, check=False)[1]["iters"] == 3
        kinds += "s"
    print("KINDS", build, bits, kinds, flush=True)
    B = new()
    assert forms(B) & STAGED and np.array_equal(host(fs.spmv(B, x)), ref)
print("DONE")
"""


SOLVES = r"""
import ctypes, sys
import numpy as np, torch
torch.cuda.init()
shim = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
import paper_1501_00324_amd as fs
import workloads as W
from tests.gpu_util import make, dev, host
fs.load(build_if_missing=False)
A = W.tet_p1(8, "elastic", seed=(92, 0), bc="x0")
g = np.random.default_rng(1)
B2, B16 = dev(g.uniform(-1, 1, (A.n_rows, 2))), dev(g.uniform(-1, 1, (A.n_rows, 16)))
ref2, ref16 = (host(fs.cg_solve_multi(make(A), B)[0]) for B in (B2, B16))
kinds = ""
for n in range(40):
    M = make(A)
    X = fs.cg_solve_multi(M, B2)[0]
    assert np.array_equal(host(X), ref2)
    shim.arm(n)
    try:
        X = fs.cg_solve_multi(M, B16)[0]
        done = shim.count() <= n
    except fs.FsError as e:
        assert e.status == fs.FS_E_OOM, e
        done = False
        kinds += "E"
    finally:
        shim.arm(-1)
    # the handle's kept arrays grew, or a part of them: smaller, then larger
    for B, ref in ((B2, ref2), (B2, ref2), (B16, ref16), (B2, ref2)):
        assert np.array_equal(host(fs.cg_solve_multi(M, B)[0]), ref), n
    if done:
        break
assert done and kinds.count("E") >= 8, kinds
print("DONE")
"""


def run_child(tmp_path, code):
    src, lib = tmp_path / "shim.c", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src), "-ldl"], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(code), str(lib)], cwd=root, capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0 and "DONE" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
    return r.stdout


def test_solves_around_a_failed_growth(tmp_path):
    """A handle's kept launch arrays grow for more columns; where one of them
    fails, the next solves find arrays that hold what they need."""
    note("scarce memory: solves")
    run_child(tmp_path, SOLVES)


def test_every_allocation_fails_once(tmp_path):
    note("scarce memory")
    for line in run_child(tmp_path, CHILD).splitlines():
        if line.startswith("KINDS"):
            # list positions, columns, groups, patterns (the host build also counts apart)
            assert line.split()[-1].count("s") >= 4, line
