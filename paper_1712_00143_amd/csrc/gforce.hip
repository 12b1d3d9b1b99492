// Symanzik-improved gauge force and action (FP64), the gauge-field half of
// the RHMC step the paper benchmarks beside the fermion force (Section 4.2).
//
// S = beta sum over loops of c (1 - Re Tr U_loop / 3) over the 1x1
// plaquettes, the 1x2 / 2x1 rectangles and the six-link parallelograms;
// the force on U_mu(x) is (beta/3) TA[U_mu(x) B^+], B the weighted sum of
// the paths from x to x+mu that close each loop through the link.
//
// The force comes from k_gauge_force_even (below), on small lattices and on
// those beyond its 32-bit offsets from the direct sum (gauge_force_even_serves),
// as the action always does: one thread per link, the whole staple sum in
// registers:
// 6 signed transverse steps n, each giving the plaquette and the three
// rectangles (11 products with the shared prefix and suffix factored out),
// and 24 parallelograms (b, a, mu, -b, -a), summed over b before the common
// last step along -a (13 products per signed a).  145 3x3 products per link:
// about 29 kflop against 288 B of link reads and writes, so the kernel is
// bound by the FP64 units and load latency, not by HBM bandwidth; the
// neighbour links come from L1 / L2.
#include "gforce.h"
#include "hisq_dev.h"
#include "su3.h"

namespace hisq {

using namespace su3;

namespace {

// Link of the step from site `from` to `to` = from + SG * axis.
template <int SG>
__device__ __forceinline__ M3 stp(const double2 *__restrict__ Ua, size_t V, long long from, long long to)
{
    if constexpr (SG > 0) return ld(Ua, V, from);
    else return dag(ld(Ua, V, to));
}

struct Geo {
    long long s;
    int x[4];
};

// x + ka * a + kb * b (distinct axes a, b)
__device__ __forceinline__ long long at2(const SmearGeom &g, const Geo &q, int a, int ka, int b, int kb)
{
    long long y = q.s;
    if (ka) y = shift(y, pick(q.x, a), pick(g.S, a), pick(g.L, a), ka);
    if (kb) y = shift(y, pick(q.x, b), pick(g.S, b), pick(g.L, b), kb);
    return y;
}

__device__ __forceinline__ long long at3(const SmearGeom &g, const Geo &q, int a, int ka, int b, int kb, int c, int kc)
{
    long long y = at2(g, q, a, ka, b, kb);
    if (kc) y = shift(y, pick(q.x, c), pick(g.S, c), pick(g.L, c), kc);
    return y;
}

// Plaquette and rectangle paths for the signed transverse step n = SN nu:
//   plaquette      L(x->x+n) U_mu(x+n) L(x+n+mu->x+mu)
//   nu-long        L(x->x+n) L(x+n->x+2n) U_mu(x+2n) L(x+2n+mu->x+n+mu) L(x+n+mu->x+mu)
//   mu-long, link first   L(x->x+n) U_mu(x+n) U_mu(x+n+mu) L(x+n+2mu->x+2mu) U_mu(x+mu)^+
//   mu-long, link second  U_mu(x-mu)^+ L(x-mu->x-mu+n) U_mu(x-mu+n) U_mu(x+n) L(x+n+mu->x+mu)
template <int SN>
__device__ __forceinline__ void plaq_rect(const SmearGeom &g, const Geo &q, const double2 *__restrict__ U, size_t V,
                                          int mu, int nu, double cp, double cr, M3 &B)
{
    const double2 *Un = U + (size_t)nu * 9 * V, *Um = U + (size_t)mu * 9 * V;
    const long long xn1 = at2(g, q, nu, SN, mu, 0), xn2 = at2(g, q, nu, 2 * SN, mu, 0);
    const long long xm1 = at2(g, q, nu, 0, mu, 1), xn1m1 = at2(g, q, nu, SN, mu, 1), xn2m1 = at2(g, q, nu, 2 * SN, mu, 1);
    const long long xm2 = at2(g, q, nu, 0, mu, 2), xn1m2 = at2(g, q, nu, SN, mu, 2);
    const long long xmm = at2(g, q, nu, 0, mu, -1), xn1mm = at2(g, q, nu, SN, mu, -1);
    const M3 Ln0 = stp<SN>(Un, V, q.s, xn1);
    const M3 H = mul_nn(Ln0, ld(Um, V, xn1));
    M3 X = H;
#pragma unroll
    for (int i = 0; i < 9; i++) X.e[i] = make_double2(cp * X.e[i].x, cp * X.e[i].y);
    {
        M3 P = mul_an(ld(Um, V, xmm), stp<SN>(Un, V, xmm, xn1mm));
        P = mul_nn(P, ld(Um, V, xn1mm));
        P = mul_nn(P, ld(Um, V, xn1));
        axpy(X, cr, P);
    }
    {
        M3 P = mul_nn(Ln0, stp<SN>(Un, V, xn1, xn2));
        P = mul_nn(P, ld(Um, V, xn2));
        P = mul_nn(P, stp<-SN>(Un, V, xn2m1, xn1m1));
        axpy(X, cr, P);
    }
    B = add(B, mul_nn(X, stp<-SN>(Un, V, xn1m1, xm1)));
    {
        M3 P = mul_nn(H, ld(Um, V, xn1m1));
        P = mul_nn(P, stp<-SN>(Un, V, xn1m2, xm2));
        P = mul_na(P, ld(Um, V, xm1));
        axpy(B, cr, P);
    }
}

// Parallelograms with first step a = SA * ax_a: sum over the four signed b
// on the two remaining axes of L(x->x+b) L(x+b->x+a+b) U_mu(x+a+b)
// L(x+a+b+mu->x+a+mu), then the common last step L(x+a+mu->x+mu).
template <int SA>
__device__ __forceinline__ void parallelograms(const SmearGeom &g, const Geo &q, const double2 *__restrict__ U,
                                               size_t V, int mu, int a, int b0, int b1, double cg, M3 &B)
{
    const double2 *Ua = U + (size_t)a * 9 * V, *Um = U + (size_t)mu * 9 * V;
    M3 S = zero3();
#pragma unroll 1
    for (int k = 0; k < 2; k++) {
        const int b = k == 0 ? b0 : b1;
        const double2 *Ub = U + (size_t)b * 9 * V;
#pragma unroll
        for (int sb = 0; sb < 2; sb++) {
            const int SB = sb == 0 ? 1 : -1;
            const long long xb = at3(g, q, b, SB, a, 0, mu, 0), xab = at3(g, q, b, SB, a, SA, mu, 0);
            const long long xabm = at3(g, q, b, SB, a, SA, mu, 1), xam = at3(g, q, b, 0, a, SA, mu, 1);
            M3 P = sb == 0 ? stp<1>(Ub, V, q.s, xb) : stp<-1>(Ub, V, q.s, xb);
            P = mul_nn(P, stp<SA>(Ua, V, xb, xab));
            P = mul_nn(P, ld(Um, V, xab));
            P = mul_nn(P, sb == 0 ? stp<-1>(Ub, V, xabm, xam) : stp<1>(Ub, V, xabm, xam));
            S = add(S, P);
        }
    }
    const long long xam = at2(g, q, a, SA, mu, 1), xm1 = at2(g, q, a, 0, mu, 1);
    axpy(B, cg, mul_nn(S, stp<-SA>(Ua, V, xam, xm1)));
}

template <int MODE>   // 0: force, 1: action partials
__global__ void __launch_bounds__(256) k_gauge_force(SmearGeom g, GForceArgs a)
{
    // A block holds the four links (one wave per direction) of 64 sites of
    // one x-y-z slab and walks a run of tch time slices: the links one
    // direction's staples fetch serve the other directions, and those of the
    // next slices, from L1 / L2 (the t neighbours are the block's own recent
    // loads instead of a lattice-volume stride away).
    const int lb = xcd_tile(blockIdx.x, gridDim.x, 1);
    const int chunk = lb / a.ntile, tile = brick_tile(lb - chunk * a.ntile, g);
    const long long nxyz = (long long)g.L[0] * g.L[1] * g.L[2];
    const long long i = (long long)tile * 64 + (threadIdx.x & 63);
    const bool valid = i < nxyz;
    const size_t V = (size_t)g.P;   // plane stride
    const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Geo q;
    {
        unsigned r = valid ? (unsigned)i : 0u;
        q.x[0] = (int)(r % (unsigned)g.L[0]);
        r /= (unsigned)g.L[0];
        q.x[1] = (int)(r % (unsigned)g.L[1]);
        q.x[2] = (int)(r / (unsigned)g.L[1]);
    }
    const long long ixyz = valid ? i : 0;
    const int t0 = chunk * a.tch, t1 = t0 + a.tch < g.L[3] ? t0 + a.tch : g.L[3];
    const int perp[3] = {mu == 0 ? 1 : 0, mu <= 1 ? 2 : 1, mu <= 2 ? 3 : 2};
    double v = 0.0;
#pragma unroll 1
    for (int t = t0; t < t1; t++) {
        q.x[3] = t;
        q.s = ixyz + (long long)t * g.S[3];
    M3 B = zero3();
#pragma unroll 1
    for (int k = 0; k < 3; k++) {
        const int nu = k == 0 ? perp[0] : k == 1 ? perp[1] : perp[2];
        plaq_rect<1>(g, q, a.U, V, mu, nu, a.cp, a.cr, B);
        plaq_rect<-1>(g, q, a.U, V, mu, nu, a.cp, a.cr, B);
    }
    if (a.cg != 0.0) {
#pragma unroll 1
        for (int k = 0; k < 3; k++) {
            const int ax = k == 0 ? perp[0] : k == 1 ? perp[1] : perp[2];
            const int b0 = k == 0 ? perp[1] : perp[0], b1 = k == 2 ? perp[1] : perp[2];
            parallelograms<1>(g, q, a.U, V, mu, ax, b0, b1, a.cg, B);
            parallelograms<-1>(g, q, a.U, V, mu, ax, b0, b1, a.cg, B);
        }
    }
    const M3 M = mul_na(ld(a.U + (size_t)mu * 9 * V, V, q.s), B);
    if constexpr (MODE == 0) {
        if (valid) {
            const double im3 = (M.e[0].y + M.e[4].y + M.e[8].y) * (1.0 / 3.0);
            M3 F;
#pragma unroll
            for (int i2 = 0; i2 < 3; i2++)
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    const double2 p = M.e[3 * i2 + j], r = M.e[3 * j + i2];
                    F.e[3 * i2 + j] = make_double2(a.scale * 0.5 * (p.x - r.x),
                                                   a.scale * (0.5 * (p.y + r.y) - (i2 == j ? im3 : 0.0)));
                }
            st(a.F + (size_t)mu * 9 * V, V, q.s, F);
        }
    } else {
        if (valid) v += M.e[0].x + M.e[4].x + M.e[8].x;
    }
    }
    if constexpr (MODE == 1) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        __shared__ double red[4];
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        if (threadIdx.x == 0) a.part[lb] = ((red[0] + red[1]) + red[2]) + red[3];
    }
}

// ---- the force around even sites
//
// Every loop of the action alternates between even and odd sites.  With the
// eight legs L_p(y) of a site (L_{+mu}(y) = U_mu(y), L_{-mu}(y) = U_mu(y-mu)^+)
// the loops that turn (or go straight) from leg s to leg b at an even site c
// close the path c+s -> c -> c+b along
//   G_{s,b}(c) = cp L_s(c+b) L_{-b}(c+b+s)
//              + sum_k w_k L_k(c+b) L_s(c+b+k) L_{-b}(c+b+k+s) L_{-k}(c+s+k)
// over the six signed directions k other than -s and -b; w_k = cr (a rectangle)
// where k is s or b or the pair is straight (s = -b, then no plaquette), cg (a
// parallelogram) otherwise.  Every link has one even end, so
//   A_b(c) = sum_{s != b} G_{s,b}(c) L_s(c)^+,   G_{b,s} = G_{s,b}^+,
// is the whole staple sum of the link (c, c+b): the 28 pairs of an even site
// cost 21 products each and give eight links, 74 products per link instead of
// the 145 of the direct sum (k_gauge_force), and 98 matrix loads instead of 166.
//
// A block holds 64 even sites.  The 28 pairs fall into seven rounds of four
// disjoint ones, one per wave, so that the waves add into the eight sums in LDS
// without conflicts: the four straight pairs, then for each of the three ways
// to pair the axes the two matchings of their legs.  Even and odd sites have
// their own half of every plane, so that a wavefront's loads stay contiguous.
// Bound by links fetched past L2 (7 TB/s).
// (Storing the 28 corners L_s^+ L_b of every even site, 2.1 GB at 32^4, leaves
// 50 products per link but took 7.4 ms: 98 corner loads a link miss L2.)
//
// Leg p: axis p >> 1, negative direction if p & 1; p ^ 1 is the opposite.

// A lane's even site: its lex index and, in LDS (64 lanes apart), the lex
// offsets of the steps -2 .. 2 along each axis (entry 5 a + k + 2), computed
// once per block instead of with every load.
struct EvenSite {
    int lex;
    const int *off;
};

// Block -> tile: the chip takes one run of `slice` tiles (a multiple of 8, about
// four time slices) after the other, each XCD a contiguous part of it, so that
// the neighbour links that miss L2 come from the Infinity Cache: with a
// contiguous eighth of the lattice per XCD the slices in use are all over the
// lattice (3 % slower at 32^4).
__device__ __forceinline__ int slice_tile(int b, int nb, int slice)
{
    const int g0 = b / slice * slice;
    return g0 + xcd_tile(b - g0, nb - g0 < slice ? nb - g0 : slice, 1);
}

// Slot of c + d (d uniform) in the parity-split planes: even sites first.
__device__ __forceinline__ int split_slot(const SmearGeom &g, const EvenSite &e, const int d[4])
{
    int y = e.lex;
#pragma unroll
    for (int a = 0; a < 4; a++)
        if (d[a]) y += e.off[(5 * a + d[a] + 2) * 64];
    return (y >> 1) + (((d[0] ^ d[1] ^ d[2] ^ d[3]) & 1) ? (int)(g.V >> 1) : 0);
}

__device__ __forceinline__ void go(int d[4], int p)
{
    const int k = p & 1 ? -1 : 1;
#pragma unroll
    for (int a = 0; a < 4; a++) d[a] += (p >> 1) == a ? k : 0;
}

// L_p(c + d); the conjugate transpose is taken by reading the transposed
// planes and flipping the sign of the imaginary parts.
__device__ __forceinline__ M3 ld_leg(const SmearGeom &g, const double2 *U, const EvenSite &e, const int d0[4], int p)
{
    int d[4] = {d0[0], d0[1], d0[2], d0[3]};
    const bool neg = p & 1;
    if (neg) go(d, p);
    const size_t V = (size_t)g.P;
    const double2 *f = U + (size_t)(p >> 1) * 9 * V;
    const unsigned pb = (unsigned)V * 16u, off = (unsigned)split_slot(g, e, d) * 16u, flip = neg ? 0x80000000u : 0u;
    M3 m;
#pragma unroll
    for (int i = 0; i < 9; i++) {
        const int q = neg ? 3 * (i % 3) + i / 3 : i, hi = q >= 5 ? 1 : 0;
        b128 v = __builtin_bit_cast(b128, __builtin_amdgcn_raw_buffer_load_b128(plane_rsrc(f, V, hi), (int)off,
                                                                              (int)((unsigned)(q - 5 * hi) * pb), 0));
        v.w ^= flip;
        m.e[i] = __builtin_bit_cast(double2, v);
    }
    return m;
}

// The path c+b -> k -> s -> -b -> -k -> c+s.
struct Path4 {
    M3 l[4];
};
__device__ __forceinline__ void ld_path(const SmearGeom &g, const double2 *U, const EvenSite &e, int s, int b, int k,
                                        Path4 &p)
{
    int d[4] = {0, 0, 0, 0};
    go(d, b);
    p.l[0] = ld_leg(g, U, e, d, k);
    go(d, k);
    p.l[1] = ld_leg(g, U, e, d, s);
    go(d, s);
    p.l[2] = ld_leg(g, U, e, d, b ^ 1);
    go(d, b ^ 1);
    p.l[3] = ld_leg(g, U, e, d, k ^ 1);
}
__device__ __forceinline__ M3 product(const Path4 &p)
{
    return mul_nn(mul_nn(mul_nn(p.l[0], p.l[1]), p.l[2]), p.l[3]);
}

// acc (in LDS, 64 lanes apart) = or += m.
__device__ __forceinline__ void lds_add(double2 *acc, bool first, const M3 &m)
{
#pragma unroll
    for (int i = 0; i < 9; i++) {
        double2 o = first ? make_double2(0.0, 0.0) : acc[i * 64];
        acc[i * 64] = make_double2(o.x + m.e[i].x, o.y + m.e[i].y);
    }
}

// Two groups of four waves take every other round, each with its own sums in
// LDS (147 KB, one block per CU), added at the end: with four waves and two
// blocks per CU the sites in flight, and with them the neighbour links fetched
// again past L2, double (39 GB a launch at 32^4, 5.1 ms; 27 GB and 3.9 ms so;
// the direct sum 6.3 ms, 5.9 with its loads first).
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_gauge_force_even(SmearGeom g, GForceArgs a, int slice)
{
    __shared__ double2 acc2[2][8 * 9 * 64];
    __shared__ int off[20 * 64];
    const int lane = threadIdx.x & 63, w8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = w8 >> 2, w = w8 & 3;
    double2 *acc = acc2[half];
    const int cb0 = slice_tile(blockIdx.x, gridDim.x, slice) * 64 + lane;
    const bool valid = cb0 < (int)(g.V >> 1);
    EvenSite e;
    {
        int x[4];
        unsigned q = valid ? 2u * (unsigned)cb0 : 0u;
        e.lex = (int)q;
        x[0] = (int)(q % (unsigned)g.L[0]);
        q /= (unsigned)g.L[0];
        x[1] = (int)(q % (unsigned)g.L[1]);
        q /= (unsigned)g.L[1];
        x[2] = (int)(q % (unsigned)g.L[2]);
        x[3] = (int)(q / (unsigned)g.L[2]);
        const int odd = (x[1] + x[2] + x[3]) & 1;
        x[0] += odd;
        e.lex += odd;
        e.off = off + lane;
        if (w8 < 4)
#pragma unroll
            for (int k = -2; k <= 2; k++)
                off[(5 * w8 + k + 2) * 64 + lane] = shift(0, pick(x, w8), pick(g.S, w8), pick(g.L, w8), k);
        __syncthreads();
    }
    const int zero[4] = {0, 0, 0, 0};
#pragma unroll 1
    for (int r0 = 0; r0 < 8; r0 += 2) {
        const int r = r0 + half;
        // round 0: the straight pair of axis w; then axes (0, t + 1) in waves 0
        // and 1 and the other two in waves 2 and 3, legs of equal or of
        // opposite signs
        int s = 2 * w, b = 2 * w + 1;
        const bool straight = r == 0;
        if (!straight) {
            const int t = (r - 1) >> 1, x = (r - 1) & 1;
            const int i = w < 2 ? 0 : (t == 0 ? 2 : 1), j = w < 2 ? t + 1 : (t == 2 ? 2 : 3);
            s = 2 * i + (w & 1);
            b = 2 * j + ((w & 1) ^ x);
        }
        if (valid && r < 7) {
            M3 G = zero3();
            if (!straight) {
                int d[4] = {0, 0, 0, 0};
                go(d, b);
                const M3 p0 = ld_leg(g, a.U, e, d, s);
                go(d, s);
                const M3 p1 = ld_leg(g, a.U, e, d, b ^ 1);
                axpy(G, a.cp, mul_nn(p0, p1));
            }
#pragma unroll 1
            for (int k = 0; k < 8; k++) {
                if (k == (b ^ 1) || k == (s ^ 1)) continue;
                const double wk = straight || k == b || k == s ? a.cr : a.cg;
                if (wk == 0.0) continue;
                Path4 p;
                ld_path(g, a.U, e, s, b, k, p);
                loads_first();
                axpy(G, wk, product(p));
            }
            loads_first();
            const M3 ls = ld_leg(g, a.U, e, zero, s), lb = ld_leg(g, a.U, e, zero, b);
            lds_add(acc + b * 9 * 64 + lane, r0 == 0, mul_na(G, ls));
            lds_add(acc + s * 9 * 64 + lane, r0 == 0, mul_an(G, dag(lb)));
        }
        __syncthreads();
    }
    if (!valid) return;
    {
        const int p = w8;
        M3 A;
#pragma unroll
        for (int i = 0; i < 9; i++) {
            const double2 u = acc2[0][(p * 9 + i) * 64 + lane], v = acc2[1][(p * 9 + i) * 64 + lane];
            A.e[i] = make_double2(u.x + v.x, u.y + v.y);
        }
        // U_mu(c) A, or for the link U_mu(c-mu) = L_p(c)^+ its product with A^+
        const M3 l = ld_leg(g, a.U, e, zero, p);
        const M3 M = p & 1 ? mul_an(l, dag(A)) : mul_nn(l, A);
        const double im3 = (M.e[0].y + M.e[4].y + M.e[8].y) * (1.0 / 3.0);
        M3 F;
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const double2 u = M.e[3 * i + j], v = M.e[3 * j + i];
                F.e[3 * i + j] = make_double2(a.scale * 0.5 * (u.x - v.x),
                                              a.scale * (0.5 * (u.y + v.y) - (i == j ? im3 : 0.0)));
            }
        int d[4] = {0, 0, 0, 0};
        if (p & 1) go(d, p);
        stb(a.F + (size_t)(p >> 1) * 9 * g.P, (size_t)g.P, split_slot(g, e, d), F);
    }
}

}  // namespace

void gauge_force_grid(const SmearGeom &g, int *ntile, int *tch, int *nblocks)
{
    const long long nxyz = (long long)g.L[0] * g.L[1] * g.L[2];
    *ntile = (int)((nxyz + 63) / 64);
    // enough blocks to fill the chip (about 2048), each with a run of slices
    int nchunk = (int)((2048 + *ntile - 1) / *ntile);
    nchunk = nchunk < 1 ? 1 : (nchunk > g.L[3] ? g.L[3] : nchunk);
    *tch = (g.L[3] + nchunk - 1) / nchunk;
    nchunk = (g.L[3] + *tch - 1) / *tch;
    *nblocks = *ntile * nchunk;
}

hipError_t launch_gauge_force_even(const SmearGeom &g, const GForceArgs &a, hipStream_t s)
{
    if (g.P >= BUF_MAX_P) return hipErrorInvalidValue;
    const int per = (int)((g.S[3] / 2 + 63) / 64), slice = (4 * per + 7) / 8 * 8;
    hipLaunchKernelGGL(k_gauge_force_even, dim3((unsigned)((g.V / 2 + 63) / 64)), dim3(512), 0, s, g, a, slice);
    return hipGetLastError();
}

hipError_t launch_gauge_force(const SmearGeom &g, const GForceArgs &a0, int mode, hipStream_t s)
{
    GForceArgs a = a0;
    int nb;
    gauge_force_grid(g, &a.ntile, &a.tch, &nb);
    const dim3 grid((unsigned)nb), blk(256);
    if (mode == 0) hipLaunchKernelGGL((k_gauge_force<0>), grid, blk, 0, s, g, a);
    else hipLaunchKernelGGL((k_gauge_force<1>), grid, blk, 0, s, g, a);
    return hipGetLastError();
}

}  // namespace hisq
