"""A call whose k-th device allocation is refused returns out of memory and
leaves its handle fit for the next call, which gives what a fresh handle gives.

A child process puts a hipMalloc before the runtime's that refuses one chosen
allocation."""
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
static long countdown = -1;   /* allocations until the refused one; negative: none is */
static long made;
int shim_init(const char *path)
{
    void *h = dlopen(path, RTLD_NOW | RTLD_NOLOAD);
    if (h) real_malloc = (int (*)(void **, size_t))dlsym(h, "hipMalloc");
    return !real_malloc;
}
void shim_refuse(long k) { countdown = k; made = 0; }
long shim_made(void) { return made; }
int hipMalloc(void **p, size_t n)
{
    made++;
    if (!real_malloc || countdown-- == 0) return 2;
    return real_malloc(p, n);
}
"""

CHILD = r"""
import ctypes, os, sys
os.environ["HISQ_TUNE"] = "0"
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.shim_made.restype = ctypes.c_long
sys.path.insert(0, sys.argv[2])
import torch
torch.cuda.init()
hip = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
assert shim.shim_init(hip.encode()) == 0
import numpy as np
from paper_1712_00143_amd import hisq as H, synth
dims = (4, 4, 4, 6)
h = synth.volume(dims) // 2
fat, lng = synth.make_links(dims, 0.3, 41)
b = synth.gaussian_even(dims, 42, 3)
rng = np.random.default_rng(3)
ws = [0.2 * (rng.standard_normal((q, p, 9)) + 1j * rng.standard_normal((q, p, 9))) for p, q in ((1, 4), (4, 1))]
r = torch.randn(h * 6, device="cuda")
v, g = torch.randn(2 * h * 6, device="cuda"), torch.randn(4 * 2 * h * 6, device="cuda")
torch.cuda.synchronize()

def lattice():
    lat = H.Lattice(dims)
    lat.load_links(fat, lng)
    lat.prepare_links(H.HISQ_F32, 18)
    return lat

def network(lat):
    net = H.PTC(lat, (1, 4, 1))
    net.set_weights(ws)
    net.harvest(lat, 0.1, b[0], every=4, maxpairs=3)
    return net

prm = lambda f=0: H.hisq_default_params(tol=1e-10, sloppy=H.HISQ_F32, flags=f)
def apply(lat, net):
    z = torch.empty_like(r)
    net.apply(r, z)
    torch.cuda.synchronize()
    return z.cpu().numpy()
def train(batch):
    def f(lat, net):
        net.set_weights(ws)
        loss = net.train(2, batch=batch, seed=1)
        return np.concatenate([loss] + [np.concatenate([w.real.ravel(), w.imag.ravel()]) for w in net.get_weights()])
    return f
def both(first, then):
    # a call that has its workspace, one that needs another, the first again
    def f(lat, net):
        return [first(lat, net), then(lat, net), first(lat, net)]
    return f
calls = {
    "cg": lambda lat, net: lat.cg(0.1, b[0], params=prm())[0],
    "cg captured": lambda lat, net: lat.cg(0.1, b[0], params=prm(H.HISQ_USE_GRAPH))[0],
    "batch": lambda lat, net: np.stack(H.hisq_batch_cg([lat] * 3, [0.1, 0.2, 0.3], list(b), params=prm())[0]),
    "learned": lambda lat, net: net.cg_learned(lat, 0.1, b[0], params=prm())[0],
    "apply": apply,
    "layer": lambda lat, net: net.layer_backward(0, v, g),
    "train": both(train(2), train(5)),
}
for name, f in calls.items():
    solver = name in ("cg", "cg captured", "batch")   # on a handle without a work set
    lat = lattice()
    net = None if solver else network(lat)
    shim.shim_refuse(ctypes.c_long(-1))
    want = f(lat, net)
    n = shim.shim_made()
    if net: net.close()
    lat.close()
    assert 0 < n < 60, (name, n)
    refused = 0
    for k in range(n):
        print(name, "allocation", k, "of", n, flush=True)
        lat = lattice()
        net = None if solver else network(lat)
        shim.shim_refuse(ctypes.c_long(k))
        try:
            f(lat, net)
        except H.HisqError as e:
            assert e.status == H.HISQ_ERR_OOM, (name, k, e)
            refused += 1
        shim.shim_refuse(ctypes.c_long(-1))
        got = f(lat, net)
        for x, y in zip(want if isinstance(want, list) else [want], got if isinstance(got, list) else [got]):
            assert np.array_equal(x, y), (name, k)
        if net: net.close()
        lat.close()
    assert refused, name
print("OK", flush=True)
"""


def test_handles_survive_a_refused_allocation(tmp_path):
    src, so, child = tmp_path / "shim.c", tmp_path / "shim.so", tmp_path / "child.py"
    src.write_text(SHIM)
    child.write_text(CHILD)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", str(so), "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-u", str(child), str(so), ROOT], capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout[-1500:] + r.stderr[-3000:]
