"""Calls whose faster form needs a buffer of its own, where that buffer cannot
be had: the form that needs less serves them, with the same results. The
allocator is made to fail from outside, for buffers above a limit: a small
library that defines hipMalloc is loaded in front of the runtime's, in a
process of its own."""
import os
import subprocess
import sys
import textwrap

import pytest

import paper_2509_26222_amd

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(paper_2509_26222_amd.__file__)))

STUB = """
#include <dlfcn.h>
#include <stddef.h>
typedef int (*malloc_fn)(void**, size_t);
size_t limit = (size_t)-1;  /* larger requests fail */
int refused = 0;
int hipMalloc(void** p, size_t n) {
  static malloc_fn real;
  if (!real) real = (malloc_fn)dlsym(dlopen("libamdhip64.so.7", RTLD_NOW), "hipMalloc");
  if (n > limit) { ++refused; *p = 0; return 2; /* hipErrorOutOfMemory */ }
  return real(p, n);
}
"""

CHILD = """
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np, torch
from paper_2509_26222_amd import api, synth, _lib as L
limit = ctypes.c_size_t.in_dll(stub, "limit")
refused = ctypes.c_int.in_dll(stub, "refused")
rng = np.random.default_rng(3)
dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
p = api.Params()
xy = dev(rng.uniform(0.0, 30.0, size=(40000, 2)))
z = dev(rng.normal(size=40000))
gf = dev(rng.normal(size=40000))
warm = [torch.empty(n, device="cuda", dtype=torch.uint8) for n in (1 << 27, 1 << 10)]
del warm  # torch keeps these: its own tensors below need no new memory
got = {}
for short in (0, 1):
    torch.zeros(1, device="cuda")
    ctx = api.Context(0)
    grid = ctx.grid(p, dev(synth.grid_centers(rng, 60, 60, 0.5, jitter=0.0)))
    w = dev(np.cos(np.arange(grid.N)))
    rowptr, colidx = ctx.gram_pattern(p, grid)
    limit.value = 1 << 22 if short else 2 ** 64 - 1
    n0 = refused.value
    c = ctx.select_centers(xy, (0.0, 0.0, 75.0, 75.0), 0.5, 0.5, 2, L.SELECT_RADIUS)
    n1 = refused.value
    vals, b = ctx.assemble_gram(p, grid, xy, z, rowptr, colidx)
    n2 = refused.value
    d_w = torch.zeros_like(w)
    ctx.eval_adjoint(p, grid, w, xy, gbar_f=gf, d_w=d_w)
    n3 = refused.value
    ctx.sync_status()
    limit.value = 2 ** 64 - 1
    assert (n1 > n0, n2 > n1, n3 > n2) == (bool(short),) * 3, (short, n0, n1, n2, n3)
    got[short] = [t.cpu().numpy() for t in (c, vals, b, d_w)]
    ctx.close()
assert np.array_equal(got[0][0], got[1][0])
# sums of up to some thousand terms of one size in another order
for u, v in zip(got[0][1:], got[1][1:]):
    assert np.abs(u - v).max() <= 1e4 * np.finfo(np.float64).eps * np.abs(u).max()
print("SHORT_OK")
"""


def test_forms_that_need_less(tmp_path):
    src, lib = tmp_path / "stub.c", tmp_path / "stub.so"
    src.write_text(STUB)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(lib), str(src), "-ldl"],
                   check=True, timeout=60)
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(CHILD), str(lib), ROOT],
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "SHORT_OK" in r.stdout, r.stderr[-2000:]
