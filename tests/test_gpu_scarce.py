"""csr_create when device memory is short: an allocation that fails either
fails the creation with FS_E_OOM or, for the arrays of the staged products,
leaves a handle whose products gather per slot.  Every allocation of a build
fails once; a child process resolves hipMalloc to a counting one."""
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


def test_every_allocation_fails_once(tmp_path):
    note("scarce memory")
    src, lib = tmp_path / "shim.c", tmp_path / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src), "-ldl"], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(CHILD), str(lib)], cwd=root, capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0 and "DONE" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
    for line in r.stdout.splitlines():
        if line.startswith("KINDS"):
            # list positions, columns, groups, patterns (the host build also counts apart)
            assert line.split()[-1].count("s") >= 4, line
