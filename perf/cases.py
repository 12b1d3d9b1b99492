"""Performance cases: what programs built on this library have it do, through
the entry points of paper_1712_00143_amd/hisq.py.

Families (kind):
  dslash     one application of D_oe and one of D_eo on device vectors, one or
             several right-hand sides: the inner work of every solver
  cg         one even-odd CG solve, plain FP64 or mixed precision
  multishift the multi-shift CG of a rational approximation
  batch      many uneven solves in one call, on host vectors
  learned    flexible CG with the parallel-transport preconditioner
  train      Adam steps of that network on harvested pairs
  smear      HISQ links from thin links
  gauge      Symanzik gauge force
  fermion    HISQ fermion force from solution vectors

Lattices, masses, link recipes, shift lists, network shapes and solver options
are those of this repository's workloads (synth.py, bench.py) and of its
tests.  Solves run to 1e-12, the accuracy of the reference solutions that the
training harvest and the benchmark use: at that accuracy the solution is
determined to about 1e-10, whatever the order of the sums.

Fields are made on the GPU from the seed alone.  Every handle works on one
torch stream of this module, as a single-stream program has it.
"""
import math

import numpy as np
import torch

from paper_1712_00143_amd import hisq, synth

_NAMES = {hisq.HISQ_F64: "f64", hisq.HISQ_F32: "f32", hisq.HISQ_F16: "f16"}
_TOL = 1e-12
_state = {}


def _stream():
    if "stream" not in _state:
        _state["stream"] = torch.cuda.Stream()
    return _state["stream"]


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # The smallest solve: a plain FP64 CG on 4^4, latency and launches only.
        dict(name="cg_f64_4x4x4x4", kind="cg", L0=4, L1=4, L2=4, L3=4, eps=0.3, mass=0.1, prec=hisq.HISQ_F64,
             recon=18),
        # A small ragged operator in the most compact format (FP16 recon-12),
        # called from a user's own Krylov method.
        dict(name="dslash_f16_r12_12x10x14x18", kind="dslash", L0=12, L1=10, L2=14, L3=18, eps=0.2,
             prec=hisq.HISQ_F16, recon=12, nrhs=1),
        # The operator alone in the paper's precision, beyond the caches: the
        # headline benchmark's lattice with the default link policy.
        dict(name="dslash_f64_r18_32x32x32x32", kind="dslash", L0=32, L1=32, L2=32, L3=32, eps=0.2,
             prec=hisq.HISQ_F64, recon=18, nrhs=1),
        # Several sources on one operator (a propagator's columns).
        dict(name="dslash_f32_r18_4rhs_24x24x24x48", kind="dslash", L0=24, L1=24, L2=24, L3=48, eps=0.2,
             prec=hisq.HISQ_F32, recon=18, nrhs=4),
        # The ordinary production solve: mixed precision with FP64 reliable
        # updates and captured chunks.
        dict(name="cg_f32_r18_16x16x16x32", kind="cg", L0=16, L1=16, L2=16, L3=32, eps=0.2, mass=0.02,
             prec=hisq.HISQ_F32, recon=18),
        # The RHMD evolution's dominant routine: 12 shifts, 4 sources.
        dict(name="multishift_24x24x24x48", kind="multishift", L0=24, L1=24, L2=24, L3=48, eps=0.2, mass=0.01,
             nshift=12, nrhs=4),
        # Independent uneven solves in one call: two of each of the four
        # shapes of the batched workload.
        dict(name="batch_cg_8_uneven", kind="batch", nper=2),
        # The learned preconditioner inside flexible CG at the light mass.
        dict(name="learned_cg_16x16x16x16", kind="learned", L0=16, L1=16, L2=16, L3=16, eps=0.25, mass=0.005,
             c1=4, c2=4),
        # Training that network (forward, backward, loss, Adam).
        dict(name="train_16x16x16x16", kind="train", L0=16, L1=16, L2=16, L3=16, eps=0.25, mass=0.02, c1=4, c2=4,
             batch=8, steps=16),
        # The three other routines of an RHMD step, at the benchmark's size.
        dict(name="smear_32x32x32x32", kind="smear", L0=32, L1=32, L2=32, L3=32, eps=0.4),
        dict(name="gauge_force_32x32x32x32", kind="gauge", L0=32, L1=32, L2=32, L3=32, eps=0.4),
        dict(name="fermion_force_32x32x32x32", kind="fermion", L0=32, L1=32, L2=32, L3=32, eps=0.4, terms=12),
    ]


def _extents(rng, lo, hi):
    """Four even extents >= 4 whose volume is spread over [lo, hi] on a
    logarithmic scale; most are not powers of two."""
    while True:
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        L = [max(4, 2 * round(0.5 * v ** 0.25 * math.exp(rng.uniform(-0.3, 0.3)))) for _ in range(3)]
        L.append(max(4, 2 * round(0.5 * v / (L[0] * L[1] * L[2]))))
        if lo <= math.prod(L) <= hi and L[3] <= 96:
            return dict(L0=L[0], L1=L[1], L2=L[2], L3=L[3])


def draw(rng):
    kind = rng.choice(["dslash", "dslash", "cg", "cg", "multishift", "batch", "learned", "train", "smear", "gauge",
                       "fermion"])
    if kind == "dslash":
        nrhs = rng.choice([1, 1, rng.randint(2, 12)])
        prec, recon = rng.choice([(hisq.HISQ_F64, 18), (hisq.HISQ_F32, 18), (hisq.HISQ_F32, 12), (hisq.HISQ_F16, 12)])
        if nrhs > 1 and prec == hisq.HISQ_F64:
            prec = hisq.HISQ_F32
        return dict(kind=kind, **_extents(rng, 256, 1 << 20 if nrhs == 1 else 663552), eps=0.2, prec=prec,
                    recon=recon, nrhs=nrhs)
    mass = round(math.exp(rng.uniform(math.log(0.02), math.log(0.2))), 4)
    if kind == "cg":
        prec, recon = rng.choice([(hisq.HISQ_F64, 18), (hisq.HISQ_F32, 18), (hisq.HISQ_F32, 12), (hisq.HISQ_F16, 12)])
        return dict(kind=kind, **_extents(rng, 256, 331776), eps=0.2, mass=mass, prec=prec, recon=recon)
    if kind == "multishift":
        return dict(kind=kind, **_extents(rng, 4096, 331776), eps=0.2, mass=mass, nshift=rng.randint(4, 12),
                    nrhs=rng.randint(1, 4))
    if kind == "batch":
        return dict(kind=kind, nper=rng.choice([1, 2, 3]), part=rng.randint(0, 1 << 16))
    if kind in ("learned", "train"):
        c = dict(kind=kind, **_extents(rng, 4096, 131072), eps=0.25, mass=mass, c1=rng.choice([2, 4]),
                 c2=rng.choice([0, 4]))
        return dict(c, batch=rng.choice([4, 8]), steps=16) if kind == "train" else c
    c = dict(kind=kind, **_extents(rng, 256, 1 << 20), eps=0.4)
    return dict(c, terms=rng.randint(1, 12)) if kind == "fermion" else c


# ------------------------------------------------- fields, made on the GPU

def _dims(case):
    return (case["L0"], case["L1"], case["L2"], case["L3"])


def _mm(a, b):
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _dag(a):
    return a.conj().transpose(-1, -2)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _shift(f, dims, mu, k):
    """f(x + k mu) of a site-major field [V, ...]."""
    g = f.reshape((dims[3], dims[2], dims[1], dims[0]) + f.shape[1:])
    return torch.roll(g, -k, 3 - mu).reshape(f.shape)


def _coords(dims):
    r = torch.arange(math.prod(dims), device="cuda")
    x = []
    for L in dims:
        x.append(r % L)
        r = r // L
    return x


def _eta(dims):
    """Staggered phases [V, 4]."""
    x = _coords(dims)
    s = [torch.zeros_like(x[0]), x[0], x[0] + x[1], x[0] + x[1] + x[2]]
    return torch.stack([1.0 - 2.0 * (v % 2) for v in s], -1).double()


def _thin(dims, eps, gen):
    """SU(3) links exp(i eps H) [V, 4, 3, 3], H = sum_a omega_a lambda_a / 2."""
    V = math.prod(dims)
    om = torch.randn((V, 4, 8), generator=gen, device="cuda", dtype=torch.float64)
    H = torch.zeros((V, 4, 3, 3), device="cuda", dtype=torch.complex128)
    for a in range(8):
        for i in range(3):
            for j in range(3):
                v = complex(synth._GELL_MANN[a][i, j])
                if v:
                    H[..., i, j] += om[..., a] * (0.5 * v)
    # four halvings, a Taylor series, four squarings
    A = H * (1j * eps / 16.0)
    E = torch.eye(3, device="cuda", dtype=torch.complex128).expand_as(A) + A / 14.0
    for n in range(13, 0, -1):
        E = _mm(A, E) / n
        E = E + torch.eye(3, device="cuda", dtype=torch.complex128)
    for _ in range(4):
        E = _mm(E, E)
    return E


def _solver_links(dims, eps, gen):
    """Phased fat (0.9 SU(3)) and long links of the solver workloads."""
    F = synth.FAT_SCALE * _thin(dims, eps, gen)
    N = torch.stack([-(1.0 / 24.0) * _mm(_mm(F[:, m], _shift(F[:, m], dims, m, 1)), _shift(F[:, m], dims, m, 2))
                     for m in range(4)], 1)
    e = _eta(dims)[:, :, None, None]
    return (F * e).contiguous(), (N * e).contiguous()


def _gauss(shape, gen):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=gen, device="cuda", dtype=torch.float64))


def _random_net(chans, seed, scale=0.1):
    rng = np.random.default_rng(seed)
    return [scale * (rng.standard_normal((b, a, 9)) + 1j * rng.standard_normal((b, a, 9)))
            for a, b in zip(chans[:-1], chans[1:])]


def _chans(case):
    return (1, case["c1"], 1) if not case["c2"] else (1, case["c1"], case["c2"], 1)


def _batch_problems(case):
    ws = synth.batch_workload(16)
    at = case.get("part", 0) % 16
    return [ws[16 * s + (at + k) % 16] for s in range(4) for k in range(case["nper"])]


# ----------------------------------------- what a user's program keeps

def _reals(t):
    return torch.view_as_real(t).reshape(-1)


def _lattice(dims, fat, lng, formats):
    lat = hisq.Lattice(dims, use_torch_stream=True)
    lat.load_links(fat, lng)
    for prec, recon in formats:
        lat.prepare_links(prec, recon)
    return lat


def _inputs(case, seed):
    """The seeded inputs of a case (device tensors; host arrays for a batch)."""
    kind, gen = case["kind"], _gen(seed)
    if kind == "batch":
        out = []
        for w in _batch_problems(case):
            fat, lng = _solver_links(w.dims, w.eps, gen)
            b = _gauss((math.prod(w.dims) // 2, 3), gen).cpu().numpy()
            out.append((w, fat, lng, b))
        return out
    dims = _dims(case)
    h = math.prod(dims) // 2
    if kind in ("smear", "gauge"):
        return dict(U=_thin(dims, case["eps"], gen))
    if kind == "fermion":
        X = _gauss((case["terms"], h, 3), gen)
        al = (0.01 + 0.99 * torch.rand(case["terms"], generator=gen, device="cuda", dtype=torch.float64)).tolist()
        return dict(U=_thin(dims, case["eps"], gen), X=X, alphas=al)
    fat, lng = _solver_links(dims, case["eps"], gen)
    n = case.get("nrhs", 1)
    b = _gauss((n, h, 3), gen)
    if kind == "dslash" and (case["prec"] != hisq.HISQ_F64):
        b = b.to(torch.complex64)
    return dict(fat=fat, lng=lng, b=b)


def _params(case):
    p = dict(tol=_TOL, flags=hisq.HISQ_USE_GRAPH)
    if case["kind"] == "cg":
        p.update(sloppy=case["prec"], recon=case["recon"])
        if case["prec"] == hisq.HISQ_F32:
            p.update(delta=0.01)
    elif case["kind"] == "multishift":
        p.update(sloppy=hisq.HISQ_F32)
    else:
        p.update(sloppy=hisq.HISQ_F32, delta=0.01)
    return hisq.hisq_default_params(**p)


def _half_vector(b):
    """An FP16 device vector (values over a per-site scale) of b [h, 3]."""
    v = torch.view_as_real(b).float()
    s = v.abs().amax(dim=(1, 2))
    q = (v / s[:, None, None]).to(torch.float16)
    return torch.cat([q.reshape(-1).view(torch.uint8), s.view(torch.uint8)])


def prepare(case, seed):
    with torch.cuda.stream(_stream()):
        st = _prepare(case, seed)
        torch.cuda.current_stream().synchronize()
        return st


def _prepare(case, seed):
    kind, inp = case["kind"], _inputs(case, seed)
    st = dict(case=case)
    if kind == "batch":
        st["lats"] = [_lattice(w.dims, f, l, [(hisq.HISQ_F32, 18)]) for w, f, l, _ in inp]
        st["masses"] = [max(w.mass, 0.02) for w, _, _, _ in inp]
        st["b"] = [b for _, _, _, b in inp]
        return st
    dims = _dims(case)
    h = math.prod(dims) // 2
    if kind in ("smear", "gauge", "fermion"):
        st["lat"] = hisq.Lattice(dims, use_torch_stream=True)
        st["U"] = inp["U"]
        if kind == "fermion":
            st["X"], st["alphas"] = _reals(inp["X"]).clone(), inp["alphas"]
        if kind == "gauge":
            # tadpole-improved one-loop weights at a mean plaquette of 0.65
            u0 = 0.65 ** 0.25
            a_s = -4.0 * math.log(u0) / 3.0684
            st["coefs"] = (1.0, -(1.0 + 0.4805 * a_s) / (20.0 * u0 * u0), -0.03325 * a_s / (u0 * u0))
        return st
    if kind == "dslash":
        fmts = [(case["prec"], case["recon"])]
    elif kind in ("learned", "train"):
        fmts = [(hisq.HISQ_F32, 18), (hisq.HISQ_F16, 12)]
    else:
        fmts = [(hisq.HISQ_F32, 18) if kind == "multishift" else (case["prec"], case["recon"])]
    lat = st["lat"] = _lattice(dims, inp["fat"], inp["lng"], fmts)
    b = inp["b"]
    if kind == "dslash":
        st["b"] = _half_vector(b[0]) if case["prec"] == hisq.HISQ_F16 and case["nrhs"] == 1 else b
        st["odd"], st["even"] = torch.empty_like(st["b"]), torch.empty_like(st["b"])
    elif kind == "cg" or kind == "learned":
        st["b"], st["x"] = b[0].contiguous(), torch.empty_like(b[0])
    elif kind == "multishift":
        st["b"] = _reals(b).clone()
        st["x"] = torch.empty(case["nrhs"] * case["nshift"] * h * 6, device="cuda", dtype=torch.float64)
        st["shifts"] = synth.shifts_log(case["nshift"])
    if kind == "learned":
        net = st["net"] = hisq.PTC(lat, _chans(case))
        net.set_transport(hisq.HISQ_F16, 12)
        net.set_activations(hisq.HISQ_F16)
        net.init_polynomial(a=4.0, c=1.2)
    elif kind == "train":
        net = st["net"] = hisq.PTC(lat, _chans(case))
        net.set_transport(hisq.HISQ_F16, 12)
        st["w0"] = _random_net(_chans(case), seed)
        net.set_weights(st["w0"])
        net.harvest(lat, case["mass"], b[0].cpu().numpy(), every=10, maxpairs=32)
    return st


# ------------------------------------------------------------------ one pass

def run(st):
    with torch.cuda.stream(_stream()):
        return _run(st)


def _run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "dslash":
        lat, p, r, n = st["lat"], case["prec"], case["recon"], case["nrhs"]
        lat.dslash(hisq.HISQ_ODD, p, r, st["b"], st["odd"], nrhs=n)
        lat.dslash(hisq.HISQ_EVEN, p, r, st["odd"], st["even"], nrhs=n)
        return dict(odd=_vector(st["odd"], lat.h), even=_vector(st["even"], lat.h))
    if kind == "cg":
        return st["lat"].cg(case["mass"], st["b"], x=st["x"], params=_params(case))[0]
    if kind == "multishift":
        return st["lat"].multishift_cg(case["mass"], st["shifts"], st["b"], x=st["x"], params=_params(case))[0]
    if kind == "batch":
        return hisq.hisq_batch_cg(st["lats"], st["masses"], st["b"], params=_params(case))[0]
    if kind == "learned":
        return st["net"].cg_learned(st["lat"], case["mass"], st["b"], x=st["x"], params=_params(case))[0]
    if kind == "train":
        # weights and losses are FP32 results behind a double interface
        net = st["net"]
        net.set_weights(st["w0"])
        loss = net.train(case["steps"], batch=case["batch"], lr=3e-3, seed=1)
        return dict(loss=loss.astype(np.float32), weights=[w.astype(np.complex64) for w in net.get_weights()])
    if kind == "smear":
        return st["lat"].smear_links(st["U"])
    if kind == "gauge":
        return st["lat"].gauge_force(st["U"], 7.0, st["coefs"])
    return st["lat"].fermion_force(st["U"], st["alphas"], st["X"])


def _vector(v, h):
    if v.dtype != torch.uint8:
        return v
    return dict(values=v[:12 * h].view(torch.float16), scales=v[12 * h:].view(torch.float32))


# ------------------------------------------------------- what it cannot avoid

def _cg_iters(mass2, tol):
    """CG iterations at a diagonal 4 m^2 + sigma = mass2: the measured counts of
    this repository's workloads, 0.5 ln(1/tol) / sqrt(mass2 + 0.00026)."""
    return 0.5 * math.log(1.0 / tol) / math.sqrt(mass2 + 0.00026)


def _op(h, prec, recon, nrhs=1, pair=True):
    """Bytes and flops of one D_oe and one D_eo: 16 links a site, the vectors
    once (1146 flops a site: the usual count of this stencil)."""
    size = {hisq.HISQ_F64: 8, hisq.HISQ_F32: 4, hisq.HISQ_F16: 2}[prec]
    vec = 16 if prec == hisq.HISQ_F16 and nrhs == 1 else 6 * max(size, 4)
    k = 2 if pair else 1
    return k * h * (16.0 * recon * size + 2.0 * nrhs * vec), k * 1146.0 * h * nrhs


def work(case):
    kind = case["kind"]
    if kind == "batch":
        by = fl = 0.0
        for w in _batch_problems(case):
            b, f = _op(math.prod(w.dims) // 2, hisq.HISQ_F32, 18)
            n = _cg_iters(4.0 * max(w.mass, 0.02) ** 2, _TOL)
            by, fl = by + n * b, fl + n * f
        return {"bytes": by, "flops": fl}
    V = math.prod(_dims(case))
    h = V // 2
    if kind == "dslash":
        b, f = _op(h, case["prec"], case["recon"], case["nrhs"])
        return {"bytes": b, "flops": f}
    if kind in ("cg", "learned"):
        n = _cg_iters(4.0 * case["mass"] ** 2, _TOL)
        if kind == "learned":
            # a third of plain CG's iterations, each with the fat links of both
            # parities read once per layer application
            b, f = _op(h, hisq.HISQ_F32, 18)
            nl = 2 * (len(_chans(case)) - 1)
            return {"bytes": n / 3 * (b + nl * V * 8 * 24.0), "flops": n / 3 * (f + nl * V * 16 * 9 * 8 * 4.0)}
        b, f = _op(h, case["prec"], case["recon"])
        return {"bytes": n * b, "flops": n * f}
    if kind == "multishift":
        by = fl = 0.0
        b, f = _op(h, hisq.HISQ_F32, 18, case["nrhs"])
        for k, s in enumerate(sorted(synth.shifts_log(case["nshift"]))):
            n = _cg_iters(4.0 * case["mass"] ** 2 + s, _TOL)
            if k == 0:
                by, fl = n * b, n * f
            by += n * case["nrhs"] * h * 24.0 * 4
        return {"bytes": by, "flops": fl}
    if kind == "train":
        ch = _chans(case)
        pairs = sum(a * b for a, b in zip(ch[:-1], ch[1:]))
        sites = float(V) * case["batch"] * case["steps"]
        # two applications forward, and the input and weight gradient of each
        return {"bytes": sites * 6 * 24 * sum(ch), "flops": sites * 6 * pairs * 9 * 24.0}
    link = V * 4 * 144.0
    prod = 198.0 * V
    if kind == "smear":
        return {"bytes": 3 * link, "flops": 464 * prod}
    if kind == "gauge":
        return {"bytes": 2 * link, "flops": 172 * prod}
    return {"bytes": 2 * link + case["terms"] * h * 48.0, "flops": (464 + 1296) * prod}


# --------------------------------------------- the same in plain FP64 torch

class _Exact:
    """D of a lattice from its links: neighbour tables and the sixteen links
    of every output site."""

    def __init__(self, dims, fat, lng):
        x = _coords(dims)
        par = (x[0] + x[1] + x[2] + x[3]) % 2
        lex = torch.arange(math.prod(dims), device="cuda")
        self.nb, self.u = [], []
        for p in (0, 1):
            site = lex[par == p]
            nb, u = [], []
            for mu in range(4):
                for U, k in ((fat, 1), (lng, 3)):
                    f, b = _shift(lex, dims, mu, k)[site], _shift(lex, dims, mu, -k)[site]
                    nb += [f // 2, b // 2]
                    u += [U[site, mu], -_dag(U[b, mu])]
            self.nb.append(nb)
            self.u.append(u)

    def d(self, p, v):
        """D to parity p of v [..., h, 3]."""
        out = torch.zeros_like(v)
        for nb, u in zip(self.nb[p], self.u[p]):
            w = v[..., nb, :]
            for c in range(3):
                out += u[:, :, c] * w[..., c, None]
        return out

    def solve(self, diag, b):
        """A x = b for diagonals diag [n] and b [n, h, 3], refined once."""
        dg = torch.as_tensor(diag, device="cuda", dtype=torch.float64)[:, None, None]

        def A(v):
            return dg * v - self.d(0, self.d(1, v))

        def dot(u, v):
            return (u.conj() * v).sum((1, 2)).real

        x = torch.zeros_like(b)
        for _ in range(2):
            r = b - A(x)
            p, rr = r, dot(r, r)
            stop = rr.clamp_min(1e-300) * (1e-13 if _ == 0 else 1e-5) ** 2
            for it in range(20000):
                if it % 20 == 0 and bool((rr <= stop).all()):
                    break
                q = A(p)
                al = rr / dot(p, q).clamp_min(1e-300)
                x = x + al[:, None, None] * p
                r = r - al[:, None, None] * q
                rn = dot(r, r)
                p = r + (rn / rr.clamp_min(1e-300))[:, None, None] * p
                rr = rn
        return x


def _fat7(U, dims, c):
    """One smearing level (c1, c3, c5, c7, cL) of links [4] of [V, 3, 3]."""
    def stap(nu, mu, P, M):
        s, m = _shift(U[nu], dims, nu, -1), _shift(M, dims, nu, -1)
        up = _mm(_mm(U[nu], _shift(P, dims, nu, 1)), _dag(_shift(U[nu], dims, mu, 1)))
        return up, _mm(_mm(_dag(s), m), _shift(s, dims, mu, 1))

    out = []
    for mu in range(4):
        perp = [d for d in range(4) if d != mu]
        F = c[0] * U[mu]
        T1 = {}
        for nu in perp:
            hp, hm = stap(nu, mu, U[mu], U[mu])
            T1[nu] = hp + hm
            F = F + c[1] * T1[nu]
            if c[4]:
                F = F + c[4] * sum(stap(nu, mu, hp, hm))
        for sig in perp:
            nu, rho = [d for d in perp if d != sig]
            T2 = sum(stap(rho, mu, T1[nu], T1[nu])) + sum(stap(nu, mu, T1[rho], T1[rho]))
            F = F + c[2] * T2 + c[3] * sum(stap(sig, mu, T2, T2))
        out.append(F)
    return out


def _inverse(m):
    a, b, c = m[..., 0, :], m[..., 1, :], m[..., 2, :]
    ia, ib, ic = torch.linalg.cross(b, c), torch.linalg.cross(c, a), torch.linalg.cross(a, b)
    det = (a * ia).sum(-1)
    return torch.stack([ia, ib, ic], -1) / det[..., None, None]


def _polar(V):
    for _ in range(9):
        V = 0.5 * (V + _dag(_inverse(V)))
    return V


def _hisq(U, dims):
    """Unphased level-2 links and Naik products of thin links [4] of [V, 3, 3]."""
    W = [_polar(v) for v in _fat7(U, dims, (1 / 8, 1 / 16, 1 / 64, 1 / 384, 0.0))]
    X = _fat7(W, dims, (5 / 8, 1 / 16, 1 / 64, 1 / 384, -1 / 16))
    N = [-(1.0 / 24.0) * _mm(_mm(W[m], _shift(W[m], dims, m, 1)), _shift(W[m], dims, m, 2)) for m in range(4)]
    return X, N


def _ta(M):
    A = 0.5 * (M - _dag(M))
    return A - torch.diagonal(A, dim1=-2, dim2=-1).sum(-1)[..., None, None] / 3.0 * torch.eye(3, device="cuda")


def _loop_sum(U, dims, coefs):
    """sum over loops of c Re Tr U_loop, each loop once."""
    def path(steps):
        x = [0, 0, 0, 0]
        P = None
        for d in steps:
            mu = abs(d) - 1
            if d < 0:
                x[mu] -= 1
            u = U[mu]
            for k in range(4):
                if x[k]:
                    u = _shift(u, dims, k, x[k])
            if d < 0:
                u = _dag(u)
            else:
                x[mu] += 1
            P = u if P is None else _mm(P, u)
        return torch.diagonal(P, dim1=-2, dim2=-1).sum().real

    S = 0.0
    for m in range(1, 5):
        for n in range(1, 5):
            if n > m:
                S = S + coefs[0] * path((m, n, -m, -n))
            if n != m:
                S = S + coefs[1] * path((m, m, n, -m, -m, -n))
            for r in range(n + 1, 5):
                if m < n:
                    for a, b in ((n, r), (n, -r), (-n, r), (-n, -r)):
                        S = S + coefs[2] * path((m, a, b, -m, -a, -b))
    return S


# above these volumes the plain version takes too long or too much memory
_EXACT_SITES = {"gauge": 300000, "fermion": 70000, "smear": 1 << 20, "multishift": 140000}


def exact(case, seed):
    with torch.cuda.stream(_stream()):
        v = _exact(case, seed)
        torch.cuda.current_stream().synchronize()
        return v


def _exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return None
    inp = _inputs(case, seed)
    if kind == "batch":
        return [_Exact(w.dims, f, l).solve([4.0 * max(w.mass, 0.02) ** 2], torch.from_numpy(b).cuda()[None])[0]
                .cpu().numpy() for w, f, l, b in inp]
    dims = _dims(case)
    V = math.prod(dims)
    if V > _EXACT_SITES.get(kind, V):
        return None
    if kind in ("smear", "gauge", "fermion"):
        U = [inp["U"][:, m].clone() for m in range(4)]
        e = _eta(dims)
        if kind == "smear":
            X, N = _hisq(U, dims)
            return tuple(torch.stack([f[m] * e[:, m, None, None] for m in range(4)], 1) for f in (X, N))
        for u in U:
            u.requires_grad_(True)
        if kind == "gauge":
            st = _prepare(case, seed)
            Q, k = _loop_sum(U, dims, st["coefs"]), 7.0 / 3.0
            Q.backward()
            # the gradient (torch's convention) of Re Tr(U B^+) is B: F = k TA[U B^+]
            return torch.stack([k * _ta(_mm(u.detach(), _dag(u.grad))) for u in U], 1)
        X, N = _hisq(U, dims)
        D = _Exact(dims, torch.stack([X[m] * e[:, m, None, None] for m in range(4)], 1),
                   torch.stack([N[m] * e[:, m, None, None] for m in range(4)], 1))
        # X^+ A X at fixed X, up to the constant 4 m^2 |X|^2: |D_oe X|^2
        Q = 0.0
        for a, v in zip(inp["alphas"], inp["X"]):
            Q = Q + a * D.d(1, v).abs().square().sum()
        Q.backward()
        # dQ = Re Tr(dU G) with G the conjugate transpose of torch's gradient
        return torch.stack([_ta(_mm(u.detach(), _dag(u.grad))) for u in U], 1)
    D = _Exact(dims, inp["fat"], inp["lng"])
    b = inp["b"].to(torch.complex128)
    if kind == "dslash":
        odd = D.d(1, b)
        even = D.d(0, odd)
        if case["prec"] == hisq.HISQ_F16 and case["nrhs"] == 1:
            return dict(odd=_exact_half(odd[0]), even=_exact_half(even[0]))
        return dict(odd=odd, even=even)
    if kind == "multishift":
        diag = [4.0 * case["mass"] ** 2 + s for s in synth.shifts_log(case["nshift"])]
        x = [D.solve(diag, b[j].expand(len(diag), -1, -1).contiguous()) for j in range(case["nrhs"])]
        return _reals(torch.stack(x))
    return D.solve([4.0 * case["mass"] ** 2], b)[0]


def _exact_half(v):
    r = torch.view_as_real(v)
    s = r.abs().amax(dim=(1, 2))
    return dict(values=(r / s[:, None, None]).reshape(-1), scales=s)
