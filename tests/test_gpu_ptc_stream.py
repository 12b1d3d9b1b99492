"""Layers of the parallel-transport network, one entry at a time, on lattices
whose links stream from memory: above 2^19 sites (FP32 links) and 2^20 sites the
layer and the weight gradient take other forms (plain block order, one wave per
tile, nine-wave blocks).  Against the same sums in plain torch FP64."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# ragged last tiles of 64 sites, extents that are no powers of two
DIMS = [(34, 26, 22, 28), (38, 30, 34, 28)]
# relative norms: FP32 sums of at most 8 channels x 9 paths x 3 colours; links
# stored as FP16 rows (2^-12 of the scale per entry, the third row from products
# of two: three times that against entries of 0.58)
TOL = {1: 2e-6, 2: 2e-3}


class _Ref:
    def __init__(self, dims, fat):
        import torch
        self.dims, self.V = dims, math.prod(dims)
        r = torch.arange(self.V, device="cuda")
        x, q = [], r
        for L in dims:
            x.append(q % L)
            q = q // L
        par = (x[0] + x[1] + x[2] + x[3]) % 2
        # slot of every site: even sites first, each parity in lex / 2 order
        self.slot = par * (self.V // 2) + r // 2
        self.F = fat

    def shift(self, f, mu, k):
        import torch
        d = self.dims
        g = f.reshape((d[3], d[2], d[1], d[0]) + f.shape[1:])
        return torch.roll(g, -k, 3 - mu).reshape(f.shape)

    def hops(self, v):
        """T_k v for the nine paths of v [V, 3]."""
        out = [v]
        for mu in range(4):
            F = self.F[:, mu]
            out.append((F * self.shift(v, mu, 1)[:, None, :]).sum(-1))
            out.append(self.shift((F.conj().transpose(1, 2) * v[:, None, :]).sum(-1), mu, -1))
        return out

    def layer(self, w, vs):
        """w [cout][cin][9], vs: cin fields [V, 3]."""
        T = [self.hops(v) for v in vs]
        return [sum(w[c][cp][k] * T[cp][k] for cp in range(len(vs)) for k in range(9)) for c in range(len(w))]

    def gradient(self, vs, gs):
        T = [self.hops(v) for v in vs]
        return np.array([[[complex((t.conj() * g).sum()) for t in Tv] for Tv in T] for g in gs])

    def field(self, a, n):
        """n fields [V, 3] of an activation array."""
        import torch
        a = torch.view_as_complex(a.reshape(n, self.V, 3, 2).double())
        return [a[c][self.slot] for c in range(n)]


def _adjoint(w):
    rev = [0, 2, 1, 4, 3, 6, 5, 8, 7]
    return np.conj(np.transpose(w, (1, 0, 2)))[:, :, rev]


def _close(got, want, tol, what):
    import torch
    for c, (g, r) in enumerate(zip(got, want)):
        rel = float((g - r).norm() / r.norm())
        site = float((g - r).norm(dim=1).max() / (r.norm() / math.sqrt(r.shape[0])))
        print(what, c, f"{rel:.2e} {site:.2e}", flush=True)
        assert rel <= tol and site <= 20 * tol, (what, c, rel, site)


@pytest.mark.parametrize("prec", [1, 2])
@pytest.mark.parametrize("dims", DIMS)
def test_layers_beyond_the_caches(dims, prec):
    import torch
    from paper_1712_00143_amd import hisq as H
    gen = torch.Generator(device="cuda").manual_seed(11)

    def rand(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64)

    V = math.prod(dims)
    a = torch.view_as_complex(rand(V, 4, 2, 3, 2))
    r0 = a[..., 0, :] / a[..., 0, :].norm(dim=-1, keepdim=True)
    r1 = a[..., 1, :] - (r0.conj() * a[..., 1, :]).sum(-1, keepdim=True) * r0
    r1 = r1 / r1.norm(dim=-1, keepdim=True)
    x, q, s = [], torch.arange(V, device="cuda"), []
    for L in dims:
        s.append(sum(x) if x else 0 * q)
        x.append(q % L)
        q = q // L
    eta = torch.stack([1.0 - 2.0 * (v % 2) for v in s], 1)[:, :, None, None]
    fat = (0.9 * eta * torch.stack([r0, r1, torch.linalg.cross(r0.conj(), r1.conj())], -2)).contiguous()
    lng = (-fat / 24.0).contiguous()
    lat = H.Lattice(dims)
    torch.cuda.synchronize()
    lat.load_links(fat, lng)
    del lng, a, r0, r1
    ref = _Ref(dims, fat)
    rng = np.random.default_rng(5)
    for chans in ((1, 2, 2, 1), (1, 4, 4, 1), (1, 8, 1), (1, 1), (1, 2, 4, 2)):
        net = H.PTC(lat, chans)
        net.set_transport(prec, 18 if prec == 1 else 12)
        net.set_weights([0.3 * (rng.standard_normal((b, c, 9)) + 1j * rng.standard_normal((b, c, 9)))
                         for c, b in zip(chans[:-1], chans[1:])])
        ws = [np.asarray(w) for w in net.get_weights()]
        for l, (ci, co) in enumerate(zip(chans[:-1], chans[1:])):
            v, g = rand(ci, V, 3, 2).float(), rand(co, V, 3, 2).float()
            out, gin = torch.empty_like(g), torch.empty_like(v)
            torch.cuda.synchronize()   # the lattice has a stream of its own
            net.layer_forward(l, v, out)
            gw = net.layer_backward(l, v, g, gin)
            torch.cuda.synchronize()
            vs, gs = ref.field(v, ci), ref.field(g, co)
            what = (dims, prec, ci, co)
            _close(ref.field(out, co), ref.layer(ws[l], vs), TOL[prec], what + ("forward",))
            _close(ref.field(gin, ci), ref.layer(_adjoint(ws[l]), gs), TOL[prec], what + ("input gradient",))
            want = ref.gradient(vs, gs)
            # sums of V terms of random sign: a relative error of the terms stays one of the sums
            assert np.abs(gw - want).max() <= 3 * TOL[prec] * np.abs(want).max(), what
        if chans[-1] == 1 and len(chans) == 4:
            # z = r + E^+ K^+ K E r with FP16 weights
            r = rand(V // 2, 3, 2).float()
            z = torch.empty_like(r)
            torch.cuda.synchronize()
            net.apply(r, z)
            torch.cuda.synchronize()
            half = [np.asarray(w.real.astype(np.float16), dtype=float) + 1j * w.imag.astype(np.float16) for w in ws]
            full = torch.cat([r, torch.zeros_like(r)])
            vs = ref.field(full, 1)
            for w in half:
                vs = ref.layer(w, vs)
            for w in reversed(half):
                vs = ref.layer(_adjoint(w), vs)
            got = ref.field(torch.cat([z, torch.zeros_like(z)]), 1)[0]
            even = (ref.slot < V // 2)[:, None]
            want = torch.where(even, vs[0] + ref.field(full, 1)[0], 0)
            _close([got], [want], 6 * TOL[prec], (dims, prec, chans, "apply"))
        net.close()
    lat.close()
