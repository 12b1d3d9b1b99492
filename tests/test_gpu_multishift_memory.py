"""Device memory of the multi-shift solver, with hipMalloc held to a budget.

The shift updates wait in a ring of up to eight residual vectors.  The ring is
a matter of speed only: a call that fits with one residual vector per
right-hand side succeeds, with the same bits, and the refinement has the memory
that the ring took.  A child process puts a hipMalloc with a budget before the
runtime's; a refused allocation returns hipErrorOutOfMemory as the runtime's
would."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
static int (*real_malloc)(void **, size_t);
static int (*real_free)(void *);
static size_t budget = (size_t)-1, used;
static struct { void *p; size_t n; } live[65536];
static int nlive;
int shim_init(const char *path)
{
    void *h = dlopen(path, RTLD_NOW | RTLD_NOLOAD);
    if (!h) return 1;
    real_malloc = (int (*)(void **, size_t))dlsym(h, "hipMalloc");
    real_free = (int (*)(void *))dlsym(h, "hipFree");
    return !real_malloc || !real_free;
}
void shim_budget(size_t n) { budget = n; }
size_t shim_used(void) { return used; }
int hipMalloc(void **p, size_t n)
{
    if (!real_malloc || used + n > budget || nlive == 65536) return 2;
    int e = real_malloc(p, n);
    if (!e) {
        live[nlive].p = *p;
        live[nlive++].n = n;
        used += n;
    }
    return e;
}
int hipFree(void *p)
{
    for (int k = 0; k < nlive; k++)
        if (live[k].p == p) {
            used -= live[k].n;
            live[k] = live[--nlive];
            break;
        }
    return real_free ? real_free(p) : 0;
}
"""

CHILD = r"""
import ctypes, os, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.shim_used.restype = ctypes.c_size_t
sys.path.insert(0, sys.argv[2])
import torch
torch.cuda.init()
hip = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
assert shim.shim_init(hip.encode()) == 0
import numpy as np
from paper_1712_00143_amd import hisq as H, synth
dims, nrhs, slack = (8, 8, 8, 8), 32, 1 << 19
h = 8 ** 4 // 2
v32 = nrhs * h * 24
fat, lng = synth.make_links(dims, 0.3, 91)
b = synth.gaussian_even(dims, 92, nrhs)
def lattice():
    lat = H.Lattice(dims)
    lat.load_links(fat, lng)
    lat.prepare_links(H.HISQ_F32, 18)
    return lat
def budget(n):
    shim.shim_budget(ctypes.c_size_t(n))
ms = lambda l, sh: l.multishift_cg(0.1, sh, b, params=H.hisq_default_params(tol=1e-9, sloppy=H.HISQ_F32, flags=H.HISQ_NO_TUNE))[0]
for shifts in (np.array([0.01]), np.array([0.0, 0.02, 0.5])):
    ns = len(shifts)
    # r, p, Ap, t, and x_k, p_k of every shift in FP32; b and x_k in FP64
    one = (4 + 2 * ns) * v32 + (1 + ns) * 2 * v32 + slack
    print("free", ns, flush=True)
    budget(2 ** 63)
    lat = lattice()
    before = shim.shim_used()
    want = ms(lat, shifts)
    kept = shim.shim_used() - before            # the refinement's set
    assert kept > 7 * v32                       # it alone would not show a ring that stays
    for name, first in (("repeated", False), ("first", True)):
        print(name, ns, flush=True)
        if first:
            budget(2 ** 63)
            lat.close()
            lat = lattice()
            budget(shim.shim_used() + kept + one)
        else:
            budget(shim.shim_used() + one)
        got = ms(lat, shifts)
        assert np.array_equal(got, want), name
    print("too little", ns, flush=True)
    budget(shim.shim_used() + one - v32 - slack)
    try:
        ms(lat, shifts)
        raise SystemExit("no error")
    except H.HisqError as e:
        assert e.status == H.HISQ_ERR_OOM, e
    budget(2 ** 63)
    assert np.array_equal(ms(lat, shifts), want)
    lat.close()
print("OK", flush=True)
"""


def test_a_call_that_fits_with_one_residual_vector_succeeds(tmp_path):
    src, so, child = tmp_path / "shim.c", tmp_path / "shim.so", tmp_path / "child.py"
    src.write_text(SHIM)
    child.write_text(CHILD)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", str(so), "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-u", str(child), str(so), ROOT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout[-1500:] + r.stderr[-3000:]
