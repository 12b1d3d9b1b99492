"""The multi-right-hand-side Dslash in groups of one, two and three at every
block shape, and training batches whose weight gradient shares units."""
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
from paper_1712_00143_amd import synth

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_CHILD = r"""
import os, sys
import numpy as np
import torch
import oracle
from paper_1712_00143_amd import synth, hisq as H

arch = torch.cuda.get_device_properties(0).gcnArchName.replace(" ", "_")
W = int(sys.argv[1])
dims = (6, 4, 6, 4)                          # h = 288, a ragged last tile
h = synth.volume(dims) // 2
t = (h + 63) // 64
lines = [f"mrhs2:{arch}:p{p}:r{r}:t{t}:nr{n} {W} 1 0 1.0" for p, r in ((1, 18), (1, 12), (2, 12)) for n in (1, 2, 3)]
lines += [f"mrhs2:{arch}:p0:r18:t{t}:nr{n} {min(W, 8)} 1 0 1.0" for n in (1, 2, 3)]
path = os.environ["HISQ_TUNE_CACHE"]
with open(path, "w") as f:
    f.write("\n".join(lines) + "\n")
tol = {1: 5e-6, 2: 2e-3}
fat, lng = synth.make_links(dims, 0.3, seed=63)
lat = H.Lattice(dims)
lat.load_links(fat, lng)
for p, r in ((1, 18), (1, 12), (2, 12)):
    lat.prepare_links(p, r)
    for n in (2, 3):                         # PLAIN, FP32 vectors
        psi = synth.gaussian_even(dims, 80 + n, n)
        out = np.zeros_like(psi)
        for par in (0, 1):
            print("dslash", W, p, r, n, par, flush=True)
            lat.dslash(par, p, r, psi, out, nrhs=n)
            for j in range(n):
                ref = oracle.dslash_half(dims, fat, lng, par, psi[j])
                rel = float(np.linalg.norm(out[j] - ref) / np.linalg.norm(ref))
                site = float(np.linalg.norm(out[j] - ref, axis=1).max() / (np.linalg.norm(ref) / np.sqrt(h)))
                assert rel <= tol[p] and site <= 10 * tol[p], (W, p, r, n, par, j, rel, site)
    for n in (1, 2, 3):
        # AX with its tile sums, and in the refinement PLAIN and RES in FP64
        print("multi-shift", W, p, r, n, flush=True)
        b = synth.gaussian_even(dims, 90 + n, n)
        x, infos = lat.multishift_cg(0.1, [0.02], b, params=H.hisq_default_params(tol=1e-10, sloppy=p, recon=r))
        for j in range(n):
            assert oracle.true_residual(dims, fat, lng, 0.1, b[j], x[j, 0], 0.02) <= 1e-10, (W, p, r, n, j)
for n in (2, 3):
    print("batch", W, n, flush=True)
    ms = [0.1, 0.15, 0.25][:n]
    bs = [synth.gaussian_even(dims, 95 + q) for q in range(n)]
    xs, infos = H.hisq_batch_cg([lat] * n, ms, bs, params=H.hisq_default_params(tol=1e-10, sloppy=1))
    for q in range(n):
        assert infos[q]["converged"] == 1 and oracle.true_residual(dims, fat, lng, ms[q], bs[q], xs[q]) <= 1e-10
lat.close()
with open(path) as f:
    extra = [ln for ln in f if ":nr" in ln][len(lines):]
assert not extra, extra
print("OK")
"""


@pytest.mark.parametrize("shape", [2, 4, 8, 16])
def test_groups_below_four_at_every_block_shape(tmp_path, shape):
    """The partial vectors of W waves are exchanged among as many waves as there
    are right-hand sides (four for three): every W and group size of the PLAIN,
    AX and FP64 RES epilogues against the oracle, through a prefilled tuner cache."""
    env = dict(os.environ, HISQ_TUNE_CACHE=str(tmp_path / "tune.txt"))
    env["PYTHONPATH"] = ROOT + os.pathsep + env.get("PYTHONPATH", "")
    r = subprocess.run([sys.executable, "-u", "-c", _CHILD, str(shape)], cwd=ROOT, env=env, capture_output=True,
                       text=True, timeout=110)
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout[-1000:] + r.stderr[-3000:]


@pytest.mark.parametrize("chans", [(1, 4, 4, 1), (1, 8)])
def test_weight_gradient_units_of_several_entries(chans):
    """101 entries on 34 tiles: a unit of the weight gradient takes two entries
    (17 tiles, the even sites alone: one) and the last one; a block of the layers
    takes four and the last one.  Two Adam steps against the oracle: the first
    shows the signs of the gradient, the second its ratio to the first, where an
    entry of at least a twentieth of the largest is known to 1e-5 / 0.05 of
    itself, a few 1e-7 of an update of 1e-3."""
    from paper_1712_00143_amd import hisq as H
    dims, B, lr = (6, 6, 6, 10), 101, 1e-3
    fat, lng = synth.make_links(dims, 0.25, seed=4021)
    lat = H.Lattice(dims)
    lat.load_links(fat, lng)
    net = H.PTC(lat, chans)
    net.set_transport(H.HISQ_F32, 18)
    net.set_loss(H.HISQ_LOSS_EUCLIDEAN)
    rng = np.random.default_rng(9)
    net.set_weights([0.2 * (rng.standard_normal((b, a, 9)) + 1j * rng.standard_normal((b, a, 9)))
                     for a, b in zip(chans[:-1], chans[1:])])
    b = synth.gaussian_even(dims, 4521)
    assert net.harvest(lat, 0.1, b, every=4, maxpairs=2) == 2
    pairs = [net.get_pair(i, b.shape[0]) for i in range(2)]
    w = [u.astype(np.complex128) for u in net.get_weights()]
    state = {}
    for step in (1, 2):
        loss = net.train(1, batch=B, lr=lr, seed=step)[0]
        # which pairs were drawn shows in the loss through their counts only
        z = [oracle.ptc_apply(dims, fat, w, r) for r, _ in pairs]
        ee = [np.vdot(e, e).real for _, e in pairs]
        S = [np.vdot(zi, e) / n for zi, (_, e), n in zip(z, pairs, ee)]
        Q = [np.vdot(zi, zi).real / n for zi, n in zip(z, ee)]
        want = [1 - abs(k * S[0] + (B - k) * S[1]) ** 2 / (B * (k * Q[0] + (B - k) * Q[1])) for k in range(B + 1)]
        k = int(np.argmin(np.abs(np.array(want) - loss)))
        assert abs(want[k] - loss) <= 1e-5 * abs(loss)
        drawn = [pairs[0]] * k + [pairs[1]] * (B - k)
        _, grads = oracle.ptc_loss_and_grad(dims, fat, w, [r for r, _ in drawn], [e for _, e in drawn])
        got = [u.astype(np.complex128) for u in net.get_weights()]
        for l, g in enumerate(grads):
            for part in ("real", "imag"):
                gp, p0 = getattr(g, part), getattr(w[l], part)
                m, v = state.get((l, part), (np.zeros_like(gp), np.zeros_like(gp)))
                p1, m, v = oracle.adam_step(p0, gp, m, v, step, lr=lr)
                state[l, part] = m, v
                big = np.abs(gp) > 0.05 * np.abs(gp).max()
                assert np.allclose(getattr(got[l], part)[big], p1[big], atol=2e-6, rtol=0), (step, l, part)
        w = got
    net.close()
    lat.close()


def test_one_handle_used_by_several_threads():
    """Eight threads apply one lattice's operator, single and in groups, with the
    launch shapes not yet known to the handle."""
    import threading

    import torch
    from paper_1712_00143_amd import hisq as H
    dims = (8, 6, 4, 10)
    h = synth.volume(dims) // 2
    fat, lng = synth.make_links(dims, 0.25, seed=4031)
    psi = [synth.gaussian_even(dims, 4600 + k, 6) for k in range(8)]
    ins = [torch.from_numpy(np.ascontiguousarray(p.astype(np.complex64)).view(np.float32).ravel()).cuda() for p in psi]
    torch.cuda.synchronize()
    lat = H.Lattice(dims)
    lat.load_links(fat, lng)
    lat.prepare_links(H.HISQ_F32, 18)
    want = None
    for _ in range(2):
        outs = [torch.zeros_like(v) for v in ins]
        torch.cuda.synchronize()
        failed = []

        def work(k):
            try:
                n = 6 if k % 2 else 1
                for _ in range(20):
                    lat.dslash(H.HISQ_ODD, H.HISQ_F32, 18, ins[k], outs[k], nrhs=n)
            except Exception as e:  # noqa: BLE001
                failed.append((k, e))

        ts = [threading.Thread(target=work, args=(k,)) for k in range(8)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        torch.cuda.synchronize()
        assert not failed, failed
        for k in range(8):
            got = outs[k].cpu().numpy().view(np.complex64).reshape(6, h, 3)
            for j in range(6 if k % 2 else 1):
                ref = oracle.dslash_half(dims, fat, lng, 1, psi[k][j])
                assert np.linalg.norm(got[j] - ref) <= 5e-6 * np.linalg.norm(ref), (k, j)
    lat.close()
