// HISQ fermion-force kernels (FP64): the chain rule of the force from the
// multi-shift solutions back to the thin links (Section 4.2's fermion
// force; the smearing it differentiates is the HISQ construction of
// smear.hip).
//
// The gradient flows backwards through the forward passes: outer products
// of the solution vectors give the gradients with respect to the fat and
// long links; the Naik product and every staple pass of the two fat7 levels
// have a gather-form adjoint (each thread owns the gradient of its own
// site's links, so there are no scattered updates); the U(3) projection has
// a closed-form adjoint from the Cayley-Hamilton form of (V^+ V)^{-1/2},
// whose coefficients are symmetric functions of the singular values and
// stay finite when they coincide.  Every kernel is an FP64 pass over planar
// fields, bound by memory traffic and latency.
#include "fforce.h"
#include "gforce.h"
#include "hisq_dev.h"
#include "su3.h"

namespace hisq {

using namespace su3;

namespace {

__device__ __forceinline__ void coords4(const SmearGeom &g, long long s, int x[4])
{
    unsigned r = (unsigned)s;   // V <= 2^31
    x[0] = (int)(r % (unsigned)g.L[0]);
    r /= (unsigned)g.L[0];
    x[1] = (int)(r % (unsigned)g.L[1]);
    r /= (unsigned)g.L[1];
    x[2] = (int)(r % (unsigned)g.L[2]);
    x[3] = (int)(r / (unsigned)g.L[2]);
}

__device__ __forceinline__ void scale3(M3 &m, double k)
{
#pragma unroll
    for (int i = 0; i < 9; i++) m.e[i] = make_double2(k * m.e[i].x, k * m.e[i].y);
}

__global__ void __launch_bounds__(256) k_ff_outer(SmearGeom g, OuterArgs a)
{
    const long long s = (long long)blockIdx.x * 256 + threadIdx.x;
    if (s >= g.V) return;
    const size_t V = (size_t)g.P;   // plane stride
    int x[4];
    coords4(g, s, x);
    const int par = (x[0] + x[1] + x[2] + x[3]) & 1;
    const double eps2 = par ? 2.0 : -2.0;   // -2 eps(x)
    const double2 *vs = par ? a.Y : a.X, *vo = par ? a.X : a.Y;
    const long long cb = s >> 1;
#pragma unroll 1
    for (int mu = 0; mu < 4; mu++) {
        const int xm = pick(x, mu), Sm = pick(g.S, mu), Lm = pick(g.L, mu);
        const long long cb1 = shift(s, xm, Sm, Lm, 1) >> 1, cb3 = shift(s, xm, Sm, Lm, 3) >> 1;
        M3 F = zero3(), L = zero3();
#pragma unroll 1
        for (int k = 0; k < a.n; k++) {
            const double al = a.alpha[k];
            const double2 *p0 = vs + ((long long)k * a.h + cb) * 3;
            const double2 *p1 = vo + ((long long)k * a.h + cb1) * 3;
            const double2 *p3 = vo + ((long long)k * a.h + cb3) * 3;
            double2 c0[3], c1[3], c3[3];
#pragma unroll
            for (int i = 0; i < 3; i++) {
                c0[i] = p0[i];
                c1[i] = make_double2(al * p1[i].x, al * p1[i].y);
                c3[i] = make_double2(al * p3[i].x, al * p3[i].y);
            }
#pragma unroll
            for (int i = 0; i < 3; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    // alpha psi(x+mu)_i conj(psi(x)_j)
                    F.e[3 * i + j].x = __builtin_fma(c1[i].x, c0[j].x, __builtin_fma(c1[i].y, c0[j].y, F.e[3 * i + j].x));
                    F.e[3 * i + j].y = __builtin_fma(c1[i].y, c0[j].x, __builtin_fma(-c1[i].x, c0[j].y, F.e[3 * i + j].y));
                    L.e[3 * i + j].x = __builtin_fma(c3[i].x, c0[j].x, __builtin_fma(c3[i].y, c0[j].y, L.e[3 * i + j].x));
                    L.e[3 * i + j].y = __builtin_fma(c3[i].y, c0[j].x, __builtin_fma(-c3[i].x, c0[j].y, L.e[3 * i + j].y));
                }
        }
        double kf = eps2, kl = eps2;
        if (a.fold) {
            const int ph = mu == 0 ? 0 : mu == 1 ? x[0] : mu == 2 ? x[0] + x[1] : x[0] + x[1] + x[2];
            const double eta = (ph & 1) ? -1.0 : 1.0;
            kf *= eta;
            kl *= eta * a.cN;
        }
        scale3(F, kf);
        scale3(L, kl);
        st(a.OF + (size_t)mu * 9 * V, V, s, F);
        st(a.OL + (size_t)mu * 9 * V, V, s, L);
    }
}

// ---- adjoint of a fat7 level
//
// The staple of fields M+ (through +d) and M- (through -d) for output
// direction mu,
//   T(x) = U_d(x) M+(x+d) U_d(x+mu)^+ + U_d(x-d)^+ M-(x-d) U_d(x-d+mu),
// has, for the gradients G+, G- of its two terms, the gather-form adjoint
//   t+(z) = U_d(z-d+mu)^+ G+(z-d) U_d(z-d)        (with respect to M+)
//   t-(z) = U_d(z+mu) G-(z+d) U_d(z)^+            (with respect to M-)
//   u(z)  = M+(z+d) U_d(z+mu)^+ G+(z) + (G+(z-mu) U_d(z-mu) M+(z-mu+d))^+
//         + (M-(z) U_d(z+mu) G-(z+d))^+ + G-(z-mu+d) U_d(z-mu)^+ M-(z-mu)
// (with respect to U_d).  The passes below take every (mu, d) of a level at
// once: a block holds 64 sites of an x-y-z slab and one wave per direction e
// and walks a run of time slices; a wave gathers what every (mu, e) or (e, mu)
// adds to its gradient fields in registers, so that each gradient field is read
// and written once per pass and the four waves share what they gather through
// L1 / L2.  (One launch per (mu, d) and sign pair, each updating its link
// gradient in memory, took 108 launches and 27 ms of the force at 32^4.)
//
// What bounds them is traffic beyond L2: a site's fields here are 3 to 10 KB,
// so that the sites 256 CUs hold at once exceed the L2s, and every extra site
// in flight costs refetched neighbours.  One wave per SIMD with a term's six to
// ten matrices requested before its first product (loads_first) therefore
// beats two waves with a few each: mid 1.77 against 2.11 ms at 32^4.

// Positions of the adjoint of (mu, d) at one site.
struct StapNb {
    int s, pd, md, pm, mm, md_pm, mm_pd;
};

__device__ __forceinline__ StapNb stap_nb(const SmearGeom &g, int s, const int x[4], int mu, int d)
{
    StapNb n;
    const int Sm = pick(g.S, mu), Lm = pick(g.L, mu), xm = pick(x, mu);
    const int Sd = pick(g.S, d), Ld = pick(g.L, d), xd = pick(x, d);
    n.s = s;
    n.pd = shift(s, xd, Sd, Ld, 1);
    n.md = shift(s, xd, Sd, Ld, -1);
    n.pm = shift(s, xm, Sm, Lm, 1);
    n.mm = shift(s, xm, Sm, Lm, -1);
    n.md_pm = shift(n.md, xm, Sm, Lm, 1);
    n.mm_pd = shift(n.mm, xd, Sd, Ld, 1);
    return n;
}

// The w-th direction other than e, and the index of direction d among those
// other than mu (fields 3 mu + k hold (mu, d)).
__device__ __forceinline__ int other_dir(int w, int e) { return w + (w >= e ? 1 : 0); }
__device__ __forceinline__ int other_idx(int d, int mu) { return d - (d > mu ? 1 : 0); }

// Block index -> tile and time slices of the walk; wave -> direction.  The brick
// order of the tiles is the plain one unless L0 = 32 (brick_tile); without it the
// force at 32^4 takes 35.1 ms instead of 33.6.  Extents in plain order: 24^4
// 14.7 -> 12.3 ms against one launch per staple, 24^3x48 29.6 -> 24.9, 28^4 28.9
// -> 24.7, 48x16^2x32 17.8 -> 15.1, 16^4 3.01 -> 2.28.
struct AdjWalk {
    int e, t0, t1, i;
    bool valid;
    int x[4];
};

__device__ __forceinline__ AdjWalk adj_walk(const SmearGeom &g, int ntile, int tch)
{
    AdjWalk w;
    const int lb = xcd_tile(blockIdx.x, gridDim.x, 1);
    const int chunk = lb / ntile, tile = brick_tile(lb - chunk * ntile, g);
    w.e = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    w.i = tile * 64 + (int)(threadIdx.x & 63);
    w.valid = w.i < g.S[3];
    unsigned q = w.valid ? (unsigned)w.i : 0u;
    w.x[0] = (int)(q % (unsigned)g.L[0]);
    q /= (unsigned)g.L[0];
    w.x[1] = (int)(q % (unsigned)g.L[1]);
    w.x[2] = (int)(q / (unsigned)g.L[1]);
    w.x[3] = 0;
    w.t0 = chunk * tch;
    w.t1 = w.t0 + tch < g.L[3] ? w.t0 + tch : g.L[3];
    return w;
}

__device__ __forceinline__ M3 scaled(double k, M3 m)
{
    scale3(m, k);
    return m;
}

// GU(s) += u.
__device__ __forceinline__ void add_to(double2 *GU, size_t V, int s, const M3 &u)
{
    stb(GU, V, s, add(ldb_nt(GU, V, s), u));
}

#define ADJ_KERNEL __global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))

// The last staples of a level: F_mu holds the staple through d of
// c7 T2_(mu,d) + cL H+-_(mu,d) (the 7-link and, at level 2, the Lepage
// staples: one transported field, one set of products) and c5 T2_(mu,d).
// Wave: link direction e = d, every mu in turn.
template <bool LEP>
ADJ_KERNEL k_adj_top(SmearGeom g, AdjTopArgs a, int ntile, int tch)
{
    AdjWalk w = adj_walk(g, ntile, tch);
    if (!w.valid) return;
    const size_t V = (size_t)g.P, fsz = 9 * V;
    const int e = w.e;
    const double2 *U = a.U + e * fsz;
#pragma unroll 1
    for (int t = w.t0; t < w.t1; t++) {
        w.x[3] = t;
        const int s = w.i + t * g.S[3];
        M3 u = zero3();
#pragma unroll 1
        for (int k = 0; k < 3; k++) {
            const int mu = other_dir(k, e), f = 3 * mu + other_idx(e, mu);
            const double2 *G = a.G + mu * fsz, *T2 = a.T2 + f * fsz;
            const double2 *Hp = LEP ? a.H + 2 * f * fsz : nullptr, *Hm = LEP ? Hp + fsz : nullptr;
            const StapNb n = stap_nb(g, s, w.x, mu, e);
            // c7 T2 + cL H, from loads already issued
            auto field = [&](M3 t2, const M3 &h) {
                scale3(t2, a.c7);
                if constexpr (LEP) axpy(t2, a.cL, h);
                return t2;
            };
            auto half = [&](const double2 *h, int y) { return LEP ? ldb(h, V, y) : M3(); };
            const M3 Gs = ldb(G, V, s);
            {
                const M3 Upm = ldb(U, V, n.pm), Gpd = ldb(G, V, n.pd), T2s = ldb(T2, V, s), Hs = half(Hm, s);
                const M3 Us = ldb(U, V, s), Udp = ldb(U, V, n.md_pm), Gmd = ldb(G, V, n.md), Umd = ldb(U, V, n.md);
                loads_first();
                const M3 Q = mul_nn(Upm, Gpd);
                u = add(u, dag(mul_nn(field(T2s, Hs), Q)));
                const M3 tm = mul_na(Q, Us);
                const M3 tp = mul_nn(mul_an(Udp, Gmd), Umd);
                M3 gt = scaled(a.c5, Gs);
                axpy(gt, a.c7, add(tp, tm));
                stb(a.GT2 + f * fsz, V, s, gt);
            }
            loads_first();
            {
                const M3 Upm = ldb(U, V, n.pm), Tpd = ldb(T2, V, n.pd), Hpd = half(Hp, n.pd);
                const M3 Gmm = ldb(G, V, n.mm), Umm = ldb(U, V, n.mm), Tmp = ldb(T2, V, n.mm_pd), Hmp = half(Hp, n.mm_pd);
                const M3 Gmp = ldb(G, V, n.mm_pd), Tmm = ldb(T2, V, n.mm), Hmm = half(Hm, n.mm);
                loads_first();
                u = add(u, mul_nn(mul_na(field(Tpd, Hpd), Upm), Gs));
                u = add(u, dag(mul_nn(mul_nn(Gmm, Umm), field(Tmp, Hmp))));
                u = add(u, mul_nn(mul_na(Gmp, Umm), field(Tmm, Hmm)));
            }
        }
        add_to(a.GU + e * fsz, V, s, u);
    }
}

// t+ and t- of the adjoint of (mu, d) at n, from the fields of G+ and G-.
__device__ __forceinline__ void adj_halves(const double2 *U, const double2 *Gp, const double2 *Gm, size_t V,
                                           const StapNb &n, M3 &tp, M3 &tm)
{
    const M3 a = ldb(U, V, n.md_pm), p = ldb(Gp, V, n.md), b = ldb(U, V, n.md);
    const M3 c = ldb(U, V, n.pm), m = ldb(Gm, V, n.pd), d = ldb(U, V, n.s);
    loads_first();
    tp = mul_nn(mul_an(a, p), b);
    tm = mul_na(mul_nn(c, m), d);
}
__device__ __forceinline__ M3 adj_field(const double2 *U, const double2 *Gp, const double2 *Gm, size_t V,
                                        const StapNb &n)
{
    M3 tp, tm;
    adj_halves(U, Gp, Gm, V, n, tp, tm);
    return add(tp, tm);
}

// GT1_(mu,j) = c3 G_mu + the adjoints of the two 5-link staples that transport
// T1_(mu,j): through x of T2_(mu,y) and through y of T2_(mu,x), {x, y} the
// other two directions.  Wave: mu, every j in turn.
ADJ_KERNEL k_adj_mid(SmearGeom g, AdjMidArgs a, int ntile, int tch)
{
    AdjWalk w = adj_walk(g, ntile, tch);
    if (!w.valid) return;
    const size_t V = (size_t)g.P, fsz = 9 * V;
    const int mu = w.e;
#pragma unroll 1
    for (int t = w.t0; t < w.t1; t++) {
        w.x[3] = t;
        const int s = w.i + t * g.S[3];
        const M3 Gs = scaled(a.c3, ldb(a.G + mu * fsz, V, s));
#pragma unroll 1
        for (int j = 0; j < 3; j++) {
            const int kx = j == 0 ? 1 : 0, ky = j == 2 ? 1 : 2;
            M3 o = Gs;
#pragma unroll 1
            for (int q = 0; q < 2; q++) {
                const int d = other_dir(q ? ky : kx, mu);
                const double2 *G = a.GT2 + (3 * mu + (q ? kx : ky)) * fsz;
                o = add(o, adj_field(a.U + d * fsz, G, G, V, stap_nb(g, s, w.x, mu, d)));
            }
            stb(a.GT1 + (3 * mu + j) * fsz, V, s, o);
        }
    }
}

// With a Lepage term the two signs of the 3-link staple (mu, j) have their own
// gradients: H+-_(mu,j) is transported through j into F_mu, so they are
// GT1_(mu,j) + cL t+- of G_mu (the first over GT1, the second to Gm).  Wave:
// mu, every j in turn.
ADJ_KERNEL k_adj_split(SmearGeom g, AdjSplitArgs a, int ntile, int tch)
{
    AdjWalk w = adj_walk(g, ntile, tch);
    if (!w.valid) return;
    const size_t V = (size_t)g.P, fsz = 9 * V;
    const int mu = w.e;
    const double2 *G = a.G + mu * fsz;
#pragma unroll 1
    for (int t = w.t0; t < w.t1; t++) {
        w.x[3] = t;
        const int s = w.i + t * g.S[3];
#pragma unroll 1
        for (int j = 0; j < 3; j++) {
            const int d = other_dir(j, mu);
            double2 *Gp = a.Gp + (3 * mu + j) * fsz;
            const M3 o = ldb_nt(Gp, V, s);
            M3 tp, tm, p = o, m = o;
            adj_halves(a.U + d * fsz, G, G, V, stap_nb(g, s, w.x, mu, d), tp, tm);
            axpy(p, a.cL, tp);
            axpy(m, a.cL, tm);
            stb(Gp, V, s, p);
            stb(a.Gm + (3 * mu + j) * fsz, V, s, m);
        }
    }
}

// u of the adjoint of (mu, d) for M+ = M- = M.
__device__ __forceinline__ void adj_link(M3 &u, const double2 *U, const double2 *M, const double2 *Gp,
                                         const double2 *Gm, size_t V, const StapNb &n)
{
    const M3 Upm = ldb(U, V, n.pm), Mpd = ldb(M, V, n.pd), Gs = ldb(Gp, V, n.s);
    const M3 Ms = ldb(M, V, n.s), Gpd = ldb(Gm, V, n.pd);
    const M3 Umm = ldb(U, V, n.mm), Gmm = ldb(Gp, V, n.mm), Mmp = ldb(M, V, n.mm_pd);
    const M3 Gmp = ldb(Gm, V, n.mm_pd), Mmm = ldb(M, V, n.mm);
    loads_first();
    u = add(u, mul_nn(mul_na(Mpd, Upm), Gs));
    u = add(u, dag(mul_nn(mul_nn(Ms, Upm), Gpd)));
    u = add(u, dag(mul_nn(mul_nn(Gmm, Umm), Mmp)));
    u = add(u, mul_nn(mul_na(Gmp, Umm), Mmm));
}

// The 5-link staples' share of the gradient of the links of direction e
// (wave): those through e of every mu in turn.
ADJ_KERNEL k_adj_mid_links(SmearGeom g, AdjMidArgs a, int ntile, int tch)
{
    AdjWalk w = adj_walk(g, ntile, tch);
    if (!w.valid) return;
    const size_t V = (size_t)g.P, fsz = 9 * V;
    const int e = w.e;
#pragma unroll 1
    for (int t = w.t0; t < w.t1; t++) {
        w.x[3] = t;
        const int s = w.i + t * g.S[3];
        M3 u = zero3();
#pragma unroll 1
        for (int k = 0; k < 6; k++) {
            const int mu = other_dir(k >> 1, e), ke = other_idx(e, mu);
            const int ka = ke == 0 ? 1 : 0, kb = ke == 2 ? 1 : 2;
            const double2 *M = a.T1 + (3 * mu + (k & 1 ? kb : ka)) * fsz, *G = a.GT2 + (3 * mu + (k & 1 ? ka : kb)) * fsz;
            adj_link(u, a.U + e * fsz, M, G, G, V, stap_nb(g, s, w.x, mu, e));
        }
        add_to(a.GU + e * fsz, V, s, u);
    }
}

// The rest of the gradient of the links of direction e (wave): for every mu in
// turn the 3-link staples through e of U_mu and those of U_e through mu, and
// c1 G_e.
ADJ_KERNEL k_adj_low(SmearGeom g, AdjLowArgs a, int ntile, int tch)
{
    AdjWalk w = adj_walk(g, ntile, tch);
    if (!w.valid) return;
    const size_t V = (size_t)g.P, fsz = 9 * V;
    const int e = w.e;
#pragma unroll 1
    for (int t = w.t0; t < w.t1; t++) {
        w.x[3] = t;
        const int s = w.i + t * g.S[3];
        M3 u = scaled(a.c1, ldb(a.G + e * fsz, V, s));
#pragma unroll 1
        for (int k = 0; k < 3; k++) {
            const int mu = other_dir(k, e), f = 3 * mu + other_idx(e, mu), fe = 3 * e + k;
            u = add(u, adj_field(a.U + mu * fsz, a.Gp + fe * fsz, a.Gm + fe * fsz, V, stap_nb(g, s, w.x, e, mu)));
            loads_first();
            adj_link(u, a.U + e * fsz, a.U + mu * fsz, a.Gp + f * fsz, a.Gm + f * fsz, V, stap_nb(g, s, w.x, mu, e));
        }
        add_to(a.GU + e * fsz, V, s, u);
    }
}

__global__ void __launch_bounds__(256) k_ff_naik_adjoint(SmearGeom g, const double2 *W, const double2 *GN,
                                                         double2 *GW)
{
    const long long s = (long long)blockIdx.x * 256 + threadIdx.x;
    if (s >= g.V) return;
    const size_t V = (size_t)g.P;   // plane stride
    const int mu = blockIdx.y;
    int x[4];
    coords4(g, s, x);
    const int Sm = pick(g.S, mu), Lm = pick(g.L, mu), xm = pick(x, mu);
    const double2 *w = W + (size_t)mu * 9 * V, *gn = GN + (size_t)mu * 9 * V;
    double2 *gw = GW + (size_t)mu * 9 * V;
    const long long p1 = shift(s, xm, Sm, Lm, 1), p2 = shift(s, xm, Sm, Lm, 2);
    const long long m1 = shift(s, xm, Sm, Lm, -1), m2 = shift(s, xm, Sm, Lm, -2);
    // W(z) is the first, second and third factor of N at z, z - mu, z - 2 mu
    M3 acc = mul_nn(mul_nn(ld(w, V, p1), ld(w, V, p2)), ld(gn, V, s));
    acc = add(acc, mul_nn(mul_nn(ld(w, V, p1), ld(gn, V, m1)), ld(w, V, m1)));
    acc = add(acc, mul_nn(mul_nn(ld(gn, V, m2), ld(w, V, m2)), ld(w, V, m1)));
    st(gw, V, s, add(ld(gw, V, s), acc));
}

// G <- M G + 2 Kh V^+: the gradient of Re Tr(W G) with respect to V for
// W = V M, M = (V^+ V)^{-1/2} = f0 + f1 Q + f2 Q^2, Q = V^+ V.  The f's are
// rational in u, v, w (sum, pairwise products and product of the square
// roots of Q's eigenvalues), which are functions of the invariants
// I = (Tr Q, Tr Q^2, det Q) with an invertible Jacobian (det = -16 w (uv - w));
// dM = sum_a (df/dI_a) dI_a + f1 dQ + f2 (dQ Q + Q dQ), dI = (Tr dQ,
// 2 Tr Q dQ, Tr adj(Q) dQ), and dQ = dV^+ V + V^+ dV gives the V^+ factor.
__global__ void __launch_bounds__(256) k_ff_unitarize_adjoint(SmearGeom g, const double2 *Vf, double2 *Gf)
{
    const long long s = (long long)blockIdx.x * 256 + threadIdx.x;
    if (s >= g.V) return;
    const size_t V = (size_t)g.P;   // plane stride
    const double2 *vf = Vf + (size_t)blockIdx.y * 9 * V;
    double2 *gf = Gf + (size_t)blockIdx.y * 9 * V;
    const M3 Vm = ld(vf, V, s), G = ld(gf, V, s);
    const M3 Q = mul_an(Vm, Vm);
    const double c0 = (Q.e[0].x + Q.e[4].x + Q.e[8].x) * (1.0 / 3.0);
    const double a0 = Q.e[0].x - c0, a1 = Q.e[4].x - c0, a2 = Q.e[8].x - c0;
    const double2 q01 = Q.e[1], q02 = Q.e[2], q12 = Q.e[5];
    const double n01 = q01.x * q01.x + q01.y * q01.y, n02 = q02.x * q02.x + q02.y * q02.y;
    const double n12 = q12.x * q12.x + q12.y * q12.y;
    const double p = (a0 * a0 + a1 * a1 + a2 * a2 + 2.0 * (n01 + n02 + n12)) * (1.0 / 6.0);
    const double re3 = (q01.x * q12.x - q01.y * q12.y) * q02.x + (q01.x * q12.y + q01.y * q12.x) * q02.y;
    const double detd = a0 * a1 * a2 + 2.0 * re3 - a0 * n12 - a1 * n02 - a2 * n01;
    double g0 = c0, g1 = c0, g2 = c0;
    if (p > 1e-28 * c0 * c0) {
        const double sp = sqrt(p);
        double r = 0.5 * detd / (p * sp);
        r = r > 1.0 ? 1.0 : (r < -1.0 ? -1.0 : r);
        const double th = acos(r) * (1.0 / 3.0);
        const double tp = 2.0943951023931954923;   // 2 pi / 3
        g0 = c0 + 2.0 * sp * cos(th);
        g1 = c0 + 2.0 * sp * cos(th + tp);
        g2 = c0 + 2.0 * sp * cos(th - tp);
    }
    const double r0 = sqrt(fmax(g0, 0.0)), r1 = sqrt(fmax(g1, 0.0)), r2 = sqrt(fmax(g2, 0.0));
    const double u = r0 + r1 + r2, v = r0 * r1 + r0 * r2 + r1 * r2, w = r0 * r1 * r2;
    const double D = w * (u * v - w), iD = 1.0 / D;
    const double f[3] = {(u * v * v - w * (u * u + v)) * iD, (2.0 * u * v - w - u * u * u) * iD, u * iD};
    const double dN[3][3] = {{v * v - 2.0 * u * w, 2.0 * u * v - w, -u * u - v}, {2.0 * v - 3.0 * u * u, 2.0 * u, -1.0},
                             {1.0, 0.0, 0.0}};
    const double dD[3] = {v * w, u * w, u * v - 2.0 * w};
    // J = d(I1, I2, I3)/d(u, v, w) and its inverse
    const double J[3][3] = {{2.0 * u, -2.0, 0.0},
                            {4.0 * u * (u * u - 2.0 * v) + 4.0 * w, -4.0 * (u * u - 2.0 * v) - 4.0 * v, 4.0 * u},
                            {0.0, 0.0, 2.0 * w}};
    double Ji[3][3];
    {
        const double det = J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) - J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
                           J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
        const double id = 1.0 / det;
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const int i1 = (j + 1) % 3, i2 = (j + 2) % 3, j1 = (i + 1) % 3, j2 = (i + 2) % 3;
                Ji[i][j] = (J[i1][j1] * J[i2][j2] - J[i1][j2] * J[i2][j1]) * id;
            }
    }
    const M3 Q2 = mul_nn(Q, Q);
    const M3 R = mul_nn(G, Vm);
    const M3 QR = mul_nn(Q, R), RQ = mul_nn(R, Q);
    double rho[3] = {R.e[0].x + R.e[4].x + R.e[8].x, QR.e[0].x + QR.e[4].x + QR.e[8].x, 0.0};
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int k = 0; k < 3; k++)   // Re Tr(Q QR)
            rho[2] += Q.e[3 * i + k].x * QR.e[3 * k + i].x - Q.e[3 * i + k].y * QR.e[3 * k + i].y;
    double beta[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 3; i++) {
        double df[3];
#pragma unroll
        for (int j = 0; j < 3; j++) df[j] = (dN[i][j] - f[i] * dD[j]) * iD;
#pragma unroll
        for (int a = 0; a < 3; a++) beta[a] += (df[0] * Ji[0][a] + df[1] * Ji[1][a] + df[2] * Ji[2][a]) * rho[i];
    }
    // adj(Q)_ij = cofactor C_ji
    M3 K;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const int i1 = (j + 1) % 3, i2 = (j + 2) % 3, j1 = (i + 1) % 3, j2 = (i + 2) % 3;
            const double2 a11 = Q.e[3 * i1 + j1], a22 = Q.e[3 * i2 + j2], a12 = Q.e[3 * i1 + j2], a21 = Q.e[3 * i2 + j1];
            const double2 adj = make_double2(a11.x * a22.x - a11.y * a22.y - (a12.x * a21.x - a12.y * a21.y),
                                             a11.x * a22.y + a11.y * a22.x - (a12.x * a21.y + a12.y * a21.x));
            const double2 q = Q.e[3 * i + j], r = R.e[3 * i + j], qr = QR.e[3 * i + j], rq = RQ.e[3 * i + j];
            K.e[3 * i + j] = make_double2(2.0 * beta[1] * q.x + beta[2] * adj.x + f[1] * r.x + f[2] * (qr.x + rq.x),
                                          2.0 * beta[1] * q.y + beta[2] * adj.y + f[1] * r.y + f[2] * (qr.y + rq.y));
        }
    K.e[0].x += beta[0];
    K.e[4].x += beta[0];
    K.e[8].x += beta[0];
    M3 Kh;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++)
            Kh.e[3 * i + j] = make_double2(K.e[3 * i + j].x + K.e[3 * j + i].x, K.e[3 * i + j].y - K.e[3 * j + i].y);   // 2 Kh
    M3 Mx;
#pragma unroll
    for (int i = 0; i < 9; i++)
        Mx.e[i] = make_double2(__builtin_fma(f[1], Q.e[i].x, f[2] * Q2.e[i].x), __builtin_fma(f[1], Q.e[i].y, f[2] * Q2.e[i].y));
    Mx.e[0].x += f[0];
    Mx.e[4].x += f[0];
    Mx.e[8].x += f[0];
    st(gf, V, s, add(mul_nn(Mx, G), mul_na(Kh, Vm)));
}

__global__ void k_field_copy(double2 *out, const double2 *in, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        out[i] = in[i];
}

__global__ void __launch_bounds__(256) k_ff_project(SmearGeom g, const double2 *U, const double2 *G, double2 *F)
{
    const long long s = (long long)blockIdx.x * 256 + threadIdx.x;
    if (s >= g.V) return;
    const size_t V = (size_t)g.P;   // plane stride
    const size_t off = (size_t)blockIdx.y * 9 * V;
    const M3 M = mul_nn(ld(U + off, V, s), ld(G + off, V, s));
    const double im3 = (M.e[0].y + M.e[4].y + M.e[8].y) * (1.0 / 3.0);
    M3 T;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const double2 p = M.e[3 * i + j], r = M.e[3 * j + i];
            T.e[3 * i + j] = make_double2(0.5 * (p.x - r.x), 0.5 * (p.y + r.y) - (i == j ? im3 : 0.0));
        }
    st(F + off, V, s, T);
}

}  // namespace

hipError_t launch_ff_outer(const SmearGeom &g, const OuterArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_ff_outer, dim3((unsigned)((g.V + 255) / 256)), dim3(256), 0, s, g, a);
    return hipGetLastError();
}

// Blocks of the adjoint passes: 1024, four per CU one after the other (the
// force at 32^4: 34.2 ms; 512 34.5, 2048 34.8, 8192 35.3).
static int adj_grid(const SmearGeom &g, int *ntile, int *tch)
{
    int nb;
    tile_grid(g, 1024, ntile, tch, &nb);
    return nb;
}

hipError_t launch_adj_top(const SmearGeom &g, const AdjTopArgs &a, hipStream_t s)
{
    if (g.P >= BUF_MAX_P) return hipErrorInvalidValue;
    int ntile, tch;
    const int nb = adj_grid(g, &ntile, &tch);
    if (a.H) hipLaunchKernelGGL((k_adj_top<true>), dim3(nb), dim3(256), 0, s, g, a, ntile, tch);
    else hipLaunchKernelGGL((k_adj_top<false>), dim3(nb), dim3(256), 0, s, g, a, ntile, tch);
    return hipGetLastError();
}

hipError_t launch_adj_mid(const SmearGeom &g, const AdjMidArgs &a, hipStream_t s)
{
    int ntile, tch;
    const int nb = adj_grid(g, &ntile, &tch);
    hipLaunchKernelGGL(k_adj_mid, dim3(nb), dim3(256), 0, s, g, a, ntile, tch);
    hipLaunchKernelGGL(k_adj_mid_links, dim3(nb), dim3(256), 0, s, g, a, ntile, tch);
    return hipGetLastError();
}

hipError_t launch_adj_split(const SmearGeom &g, const AdjSplitArgs &a, hipStream_t s)
{
    int ntile, tch;
    const int nb = adj_grid(g, &ntile, &tch);
    hipLaunchKernelGGL(k_adj_split, dim3(nb), dim3(256), 0, s, g, a, ntile, tch);
    return hipGetLastError();
}

hipError_t launch_adj_low(const SmearGeom &g, const AdjLowArgs &a, hipStream_t s)
{
    int ntile, tch;
    const int nb = adj_grid(g, &ntile, &tch);
    hipLaunchKernelGGL(k_adj_low, dim3(nb), dim3(256), 0, s, g, a, ntile, tch);
    return hipGetLastError();
}

hipError_t launch_ff_naik_adjoint(const SmearGeom &g, const double2 *W, const double2 *GN, double2 *GW,
                                  hipStream_t s)
{
    hipLaunchKernelGGL(k_ff_naik_adjoint, dim3((unsigned)((g.V + 255) / 256), 4), dim3(256), 0, s, g, W, GN, GW);
    return hipGetLastError();
}

hipError_t launch_ff_unitarize_adjoint(const SmearGeom &g, const double2 *V, double2 *G, hipStream_t s)
{
    hipLaunchKernelGGL(k_ff_unitarize_adjoint, dim3((unsigned)((g.V + 255) / 256), 4), dim3(256), 0, s, g, V, G);
    return hipGetLastError();
}

hipError_t launch_field_copy(double2 *out, const double2 *in, size_t n, hipStream_t s)
{
    const size_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_field_copy, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, s, out, in, n);
    return hipGetLastError();
}

hipError_t launch_ff_project(const SmearGeom &g, const double2 *U, const double2 *G, double2 *F, hipStream_t s)
{
    hipLaunchKernelGGL(k_ff_project, dim3((unsigned)((g.V + 255) / 256), 4), dim3(256), 0, s, g, U, G, F);
    return hipGetLastError();
}

}  // namespace hisq
