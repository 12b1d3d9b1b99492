// Gauge-covariant parallel-transport convolution (PTC) layers of the learned
// preconditioner: forward / inference, input gradient, weight gradient, loss
// and Adam.  The network maps Cin to Cout channels of colour vectors:
//   out_c(x) = sum_{c'} [ w_{c c' 0} psi_{c'}(x)
//              + sum_mu ( w_{c c' 1+2mu} F_mu(x) psi_{c'}(x+mu)
//                       + w_{c c' 2+2mu} F_mu(x-mu)^+ psi_{c'}(x-mu) ) ]
// with the fat links F (no bias: a bias would break gauge covariance).
//
// Activations are parity-split: channel c of batch entry b is
// [2 parities][h sites][3 colours] complex FP32.  The hops reuse the packed
// fat-link directions of the Dslash operator (direction 4mu: F_mu(x);
// direction 4mu+1: -F_mu(x-mu)^+, hence the sign).  A parity known to be zero
// in the input (an even vector embedded on the full lattice) is skipped.
#include "fields.h"
#include "finish.h"
#include "launch.h"
#include "ptc.h"
#include "reduce.h"

namespace hisq {

// Weight idx (uniform over the wavefront) through the scalar cache: no kernel
// writes the weights that it reads, which the address space tells the compiler
// (in a loop with stores it would load them per lane otherwise).
template <class WT> __device__ __forceinline__ float2 ldw(const void *w, int idx)
{
    if constexpr (sizeof(WT) == 2) {
        const uint32_t t = ((const __attribute__((address_space(4))) uint32_t *)w)[idx];
        return __half22float2(__builtin_bit_cast(__half2, t));
    } else {
        const uint64_t t = ((const __attribute__((address_space(4))) uint64_t *)w)[idx];
        return __builtin_bit_cast(float2, t);
    }
}

// neighbour cb index of (co, lex) along mu by +-1
__device__ __forceinline__ int nb1(const Coord &co, int lex, int mu, int k, int L0, int L1, int L2, int L3)
{
    const int x = mu == 0 ? co.x[0] : mu == 1 ? co.x[1] : mu == 2 ? co.x[2] : co.x[3];
    const int Lm = mu == 0 ? L0 : mu == 1 ? L1 : mu == 2 ? L2 : L3;
    const int Sm = mu == 0 ? 1 : mu == 1 ? L0 : mu == 2 ? L0 * L1 : L0 * L1 * L2;
    int v = x + k;
    v -= v >= Lm ? Lm : 0;
    v += v < 0 ? Lm : 0;
    return (lex + (v - x) * Sm) >> 1;
}

// Path k (0 identity, 1+2mu forward, 2+2mu backward) contributes unless the
// input parity it reads is known to be zero.  Uniform over the wavefront.
__device__ __forceinline__ bool path_live(const PtcLaunch &a, int par, int k)
{
    return k == 0 ? a.in_zero_par != par : a.in_zero_par != 1 - par;
}

// Index of W[c][c'][k] of a layer with cout outputs in its adjoint W'[c'][c][k'],
// k' the reversed hop (the adjoint of a forward hop is a backward hop).
__device__ __forceinline__ int adjoint_index(int c, int cp, int k, int cout)
{
    return (cp * cout + c) * 9 + (k == 0 ? 0 : (k & 1) ? k + 1 : k - 1);
}

// packed link direction of hop k: 4mu forward, 4mu + 1 backward
__device__ __forceinline__ int path_dir(int k) { return 4 * ((k - 1) >> 1) + ((k - 1) & 1); }

// The packed link of path k at output site (par, i); k and par must be uniform
// over the wavefront (the link block is addressed through a wave-uniform
// buffer resource).  The fat links are re-read by every layer of every
// application: cached (temporal) loads.
template <class LT, int R>
__device__ __forceinline__ void path_link(const LinkSet &ls, int par, int i, int k, RawLink<LT, R> &raw)
{
    if (k == 0) return;
    using F = LinkFmt<LT, R>;
    load_link_raw_wave<LT, R, 1>((const char *)ls.ptr[par] + (size_t)path_dir(k) * ls.hs * F::BYTES, i, ls.hs, raw);
}

// The site that path k reads (on the other parity, except for the identity).
__device__ __forceinline__ int path_site(const ProbDesc &pd, int i, const Coord &co, int lex, int k)
{
    return k == 0 ? i : nb1(co, lex, (k - 1) >> 1, (k & 1) ? 1 : -1, pd.L[0], pd.L[1], pd.L[2], pd.L[3]);
}

// NC colour vectors of one site: channel c of parity sp (of np stored ones)
// starts at base + (c np + sp) h vectors.  A vector is 24 bytes at a stride of
// 24: one 16-byte and one 8-byte access, with a uniform base per channel.
typedef float f4a8 __attribute__((ext_vector_type(4), aligned(8)));

template <int NC>
__device__ __forceinline__ void load_site(const float *base, int np, int sp, long long h, int site, Cx<float> v[NC][3])
{
#pragma unroll
    for (int c = 0; c < NC; c++) {
        const char *p = reinterpret_cast<const char *>(base) + (c * np + sp) * h * 24;
        const f4a8 t = *reinterpret_cast<const f4a8 *>(p + (unsigned)site * 24u);
        const float2 u = *reinterpret_cast<const float2 *>(p + (unsigned)site * 24u + 16);
        v[c][0] = {t.x, t.y};
        v[c][1] = {t.z, t.w};
        v[c][2] = {u.x, u.y};
    }
}

__device__ __forceinline__ void store_vec(float2 *p, const Cx<float> v[3])
{
    f4a8 t;
    t.x = v[0].re;
    t.y = v[0].im;
    t.z = v[1].re;
    t.w = v[1].im;
    *reinterpret_cast<f4a8 *>(p) = t;
    p[2] = make_float2(v[2].re, v[2].im);
}

// The matrix of hop k, T_k v = u v, from its packed form: the format's scale,
// phase and the sign of the stored backward links (-F^+) included.
template <class LT, int R>
__device__ __forceinline__ void path_matrix(const LinkSet &ls, const Coord &co, int k, const RawLink<LT, R> &raw,
                                            Cx<float> u[3][3])
{
    const int mu = (k - 1) >> 1, d = path_dir(k);
    decode_link<LT, R, float>(raw, u);
    float coef = 1.f;
    if constexpr (R == 12 || sizeof(LT) == 2) {
        coef = (float)ls.a[0];
        if constexpr (R == 12) {
            const int eb = mu == 0 ? 0 : ((co.x[0] + (mu > 1 ? co.x[1] : 0) + (mu > 2 ? co.x[2] : 0)) & 1);
            const int neg = (ls.s[0] < 0) ^ eb ^ (d & 1);
            coef = neg ? -coef : coef;
        }
    }
    if (d & 1) coef = -coef;
#pragma unroll
    for (int r = 0; r < 3; r++)
#pragma unroll
        for (int c = 0; c < 3; c++) u[r][c] = {coef * u[r][c].re, coef * u[r][c].im};
}

// acc += w v for one colour vector
__device__ __forceinline__ void mix_acc(const float2 w, const Cx<float> v[3], Cx<float> acc[3])
{
#pragma unroll
    for (int q = 0; q < 3; q++) {
        acc[q].re = fmaa(-w.y, v[q].im, fmaa(w.x, v[q].re, acc[q].re));
        acc[q].im = fmaa(w.y, v[q].re, fmaa(w.x, v[q].im, acc[q].im));
    }
}

// Forward layer (also the input-gradient layer, given the adjoint weights) of
// a.bper batch entries per block of four waves: wave w takes the two hops along
// direction w and every fourth input channel of the identity path, so that the
// waves and the four SIMDs are evenly loaded (three waves of three paths each,
// or nine of one, left a SIMD with half or twice the work of another).
//
// Issue of vector instructions bounds it: a 4 -> 4 layer needs 336 FP32
// multiply-adds per site and hop, and unpacking and scaling the link took as
// many again as a third of them.  So the links are unpacked once, with their
// coefficient folded in, and stay in registers over the batch entries.  With
// fewer outputs than inputs the channels are mixed first and COUT vectors
// transported (the transport is linear).  The waves' outputs are joined
// through LDS, channel c by wave c mod 4.
//
// 16^4, 8 entries, FP16 recon-12 links: 4 -> 4 70 -> 57 us, 4 -> 1 49 -> 29 us,
// against one entry per block, three waves of three paths and the link
// unpacked for each entry.  The matrix cores are no help: FP32 4x4x1 products
// (nine cycles for what takes four multiply-adds) on the mixing gave 62 us.
//
// STREAM (one entry, links beyond the Infinity Cache: see layer_form): memory
// bounds it, so the blocks take the sites of one parity after the other in plain
// order (a contiguous eighth per XCD costs 5 % of the rate), and the vectors are
// requested before the links are unpacked.  W = 1: a wave takes the whole
// stencil of its sites, two hops at a time, without a join.
template <class LT, int R, class WT, int CIN, int COUT, int W, bool STREAM>
__global__ void __launch_bounds__(64 * W) k_ptc_layer(PtcLaunch a)
{
    if (a.gate && a.gate->status != a.gate_want) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const ProbDesc &pd = a.probs[0];
    const int ntile = pd.ntile;
    const int npar = gridDim.x / ntile;
    const int unit = xcd_tile(blockIdx.x, gridDim.x, !STREAM);
    const int par = a.par_lo + (STREAM ? unit / ntile : unit % npar), tile = STREAM ? unit % ntile : unit / npar;
    const bool valid = tile * TILE + lane < pd.h;
    const int i = valid ? tile * TILE + lane : pd.h - 1;   // idle lanes repeat the last site
    const long long h = pd.h;
    const LinkSet &ls = pd.ls[a.lslot];
    const Coord co = cb_to_coord_pd(i, par, pd);
    const int lex = 2 * i + (co.x[0] & 1);
    constexpr int H = 8 / W, G = 2;   // hops of a wave, hops in hand
    constexpr bool KEEP = H == G;     // the links stay in registers
    static_assert(KEEP || STREAM, "a block of several entries keeps its links");
    __shared__ float red[W > 1 ? W * COUT * 6 * 64 : 1];
    const bool hops = path_live(a, par, 1), ident = path_live(a, par, 0);
    const int b0 = blockIdx.y * a.bper, b1 = b0 + a.bper < a.batch ? b0 + a.bper : a.batch;
    RawLink<LT, R> raw[G];
    Cx<float> u[G][3][3], sv[G][CIN][3];
    int site[G];
    auto links = [&](int k0) {
#pragma unroll
        for (int g = 0; g < G; g++) {
            site[g] = path_site(pd, i, co, lex, k0 + g);
            path_link<LT, R>(ls, par, i, k0 + g, raw[g]);
        }
    };
    auto vectors = [&](const float *in_b) {
#pragma unroll
        for (int g = 0; g < G; g++) load_site<CIN>(in_b, 2, 1 - par, h, site[g], sv[g]);
    };
    auto unpack = [&](int k0) {
#pragma unroll
        for (int g = 0; g < G; g++) path_matrix<LT, R>(ls, co, k0 + g, raw[g], u[g]);
    };
    if (KEEP && hops) {
        links(1 + wave * G);
        if (STREAM) vectors(a.in + (size_t)b0 * a.in_bstride);
        unpack(1 + wave * G);
    }
    for (int b = b0; b < b1; b++) {
        const float *in_b = a.in + (size_t)b * a.in_bstride;
        Cx<float> acc[COUT][3];
#pragma unroll
        for (int c = 0; c < COUT; c++)
#pragma unroll
            for (int q = 0; q < 3; q++) acc[c][q] = {0.f, 0.f};
        if (ident)
#pragma unroll
            for (int cp = 0; cp < CIN; cp++) {
                if (cp % W != wave) continue;
                Cx<float> v[1][3];
                load_site<1>(in_b + (size_t)(2 * cp + par) * h * 6, 2, 0, h, i, v);
#pragma unroll
                for (int c = 0; c < COUT; c++) mix_acc(ldw<WT>(a.w, (c * CIN + cp) * 9), v[0], acc[c]);
            }
        if (hops)
#pragma unroll
            for (int h0 = 0; h0 < H; h0 += G) {
                if (!KEEP) links(1 + wave * H + h0);
                if (!(KEEP && STREAM)) vectors(in_b);
                if (!KEEP) unpack(1 + wave * H + h0);
#pragma unroll
                for (int g = 0; g < G; g++) {
                    const int k = 1 + wave * H + h0 + g;
                    if constexpr (COUT < CIN) {
#pragma unroll
                        for (int c = 0; c < COUT; c++) {
                            Cx<float> ph[3] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
#pragma unroll
                            for (int cp = 0; cp < CIN; cp++)
                                mix_acc(ldw<WT>(a.w, (c * CIN + cp) * 9 + k), sv[g][cp], ph);
                            matvec_acc(u[g], ph, acc[c]);
                        }
                    } else {
#pragma unroll
                        for (int cp = 0; cp < CIN; cp++) {
                            Cx<float> t[3] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
                            matvec_acc(u[g], sv[g][cp], t);
#pragma unroll
                            for (int c = 0; c < COUT; c++) mix_acc(ldw<WT>(a.w, (c * CIN + cp) * 9 + k), t, acc[c]);
                        }
                    }
                }
            }
        if constexpr (W > 1) {
            float *mine = red + (size_t)wave * COUT * 6 * 64 + lane;
#pragma unroll
            for (int c = 0; c < COUT; c++)
                if (c % W != wave)
#pragma unroll
                    for (int q = 0; q < 3; q++) {
                        mine[(6 * c + 2 * q) * 64] = acc[c][q].re;
                        mine[(6 * c + 2 * q + 1) * 64] = acc[c][q].im;
                    }
            __syncthreads();
#pragma unroll
            for (int c = 0; c < COUT; c++)
                if (c % W == wave)
#pragma unroll
                    for (int q = 0; q < 3; q++) {
                        Cx<float> t = {0.f, 0.f};
#pragma unroll
                        for (int w = 0; w < W; w++) {   // the waves in order
                            const float *o = red + ((size_t)w * COUT + c) * 6 * 64 + lane;
                            t.re += w == c % W ? acc[c][q].re : o[2 * q * 64];
                            t.im += w == c % W ? acc[c][q].im : o[(2 * q + 1) * 64];
                        }
                        acc[c][q] = t;
                    }
            if (b + 1 < b1) __syncthreads();
        }
        double dr = 0.0, di = 0.0;
#pragma unroll
        for (int c = 0; c < COUT; c++) {
            if (c % W != wave || !valid) continue;
            const long long o = ((c * a.out_pstride + (par - a.out_par0)) * h + i) * 3;
            if (a.addin) {   // the identity term of M, added in the same rounding as a separate pass
                const float2 *ad = reinterpret_cast<const float2 *>(a.addin + (size_t)b * a.addin_bstride) + o;
#pragma unroll
                for (int q = 0; q < 3; q++) {
                    const float2 t = ad[q];
                    acc[c][q].re += t.x;
                    acc[c][q].im += t.y;
                }
            }
            store_vec(reinterpret_cast<float2 *>(a.out + (size_t)b * a.out_bstride) + o, acc[c]);
            if (COUT == 1 && a.dotred) {   // (q, out) = sum conj(q) out over this tile
                const float2 *qv = reinterpret_cast<const float2 *>(a.dotq) + (size_t)i * 3;
#pragma unroll
                for (int q = 0; q < 3; q++) {
                    const float2 t = qv[q];
                    dr += (double)t.x * acc[0][q].re + (double)t.y * acc[0][q].im;
                    di += (double)t.x * acc[0][q].im - (double)t.y * acc[0][q].re;
                }
            }
        }
        if (COUT == 1 && a.dotred && wave == 0) {   // wave 0 covers the whole 64-site tile
            dr = wave_sum(dr);
            di = wave_sum(di);
            if (lane == 0) {
                a.dotred[tile] = dr;
                a.dotred[a.dot_nt + tile] = di;
            }
        }
    }
}

// Weight gradient: sums of (T_k in_{c'})(x)^+ g_c(x) over sites and batch
// entries, one wavefront per path k.  Row j walks the work units (batch chunk,
// output parity, tile) j, j + nrow, ..., accumulating in FP64 per lane, and
// reduces once at the end: partials [row][9][COUT][CIN] complex FP64, in a
// fixed order for a given grid.  A unit unpacks its link once for a.bper batch
// entries.  The hops of a row are two blocks (blockIdx.y 0, 1) of four waves,
// one per SIMD; the lighter identity path is taken by further blocks, a row per
// wave.
//
// The vector ALU bounds it (4 -> 4: 144 transport, 192 product and 64
// conversion or FP64 instructions per site, path and entry); with fewer
// outputs than inputs the gradient is transported instead,
// (T_k in)^+ g = in^+ (T_k^+ g).  16^4, 8 entries: 4 -> 4 110 -> 75 us, 4 -> 1
// 53 -> 42 us, 1 -> 4 40 -> 38 us, against blocks of nine waves, a path each
// (two or three on a SIMD), that unpacked the link for every entry.
//
// W = 9: those blocks, for one entry per unit on lattices that stream from
// memory (wgrad_nine): a row's nine waves read the same vectors at the same time,
// which blocks of their own would fetch again.
template <class LT, int R, int CIN, int COUT, int W>
__global__ void __launch_bounds__(64 * W) k_ptc_wgrad(PtcLaunch a, int npar, int nrow)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k = W == 9 ? wave : blockIdx.y < 2 ? 1 + 4 * blockIdx.y + wave : 0;
    const int row = W == 9 || blockIdx.y < 2 ? blockIdx.x : 4 * blockIdx.x + wave;
    if (row >= nrow) return;
    const ProbDesc &pd = a.probs[0];
    const int ntile = pd.ntile;
    const long long h = pd.h;
    const LinkSet &ls = pd.ls[a.lslot];
    const int nunit = (a.batch + a.bper - 1) / a.bper * npar * ntile;
    double acc[COUT][CIN][2];
#pragma unroll
    for (int c = 0; c < COUT; c++)
#pragma unroll
        for (int cp = 0; cp < CIN; cp++) acc[c][cp][0] = acc[c][cp][1] = 0.0;
    for (int j = row; j < nunit; j += nrow) {
        const int u = xcd_tile(j, nunit, 1);
        const int b0 = u / (npar * ntile) * a.bper;
        const int b1 = b0 + a.bper < a.batch ? b0 + a.bper : a.batch;
        const int rem = u % (npar * ntile);
        const int par = a.par_lo + rem % npar;
        const int i = rem / npar * TILE + lane;
        if (i >= pd.h || !path_live(a, par, k)) continue;
        const Coord co = cb_to_coord_pd(i, par, pd);
        const int site = path_site(pd, i, co, 2 * i + (co.x[0] & 1), k);
        RawLink<LT, R> raw;
        path_link<LT, R>(ls, par, i, k, raw);
        Cx<float> m[3][3], v[CIN][3], g[COUT][3];
        auto vectors = [&](int b) {
            load_site<CIN>(a.in + (size_t)b * a.in_bstride, 2, k == 0 ? par : 1 - par, h, site, v);
            load_site<COUT>(a.g + (size_t)b * a.g_bstride, a.g_pstride, par - a.g_par0, h, i, g);
        };
        if (W == 9) vectors(b0);   // its only entry, requested before the link is unpacked
        if (k != 0) path_matrix<LT, R>(ls, co, k, raw, m);
        for (int b = b0; b < b1; b++) {
            if (W != 9) vectors(b);
            if (k != 0) {
                if constexpr (COUT < CIN) {
#pragma unroll
                    for (int c = 0; c < COUT; c++) {
                        Cx<float> t[3] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
#pragma unroll
                        for (int q = 0; q < 3; q++)
#pragma unroll
                            for (int r = 0; r < 3; r++) {   // conj(m) g
                                t[q].re = fmaa(m[r][q].re, g[c][r].re, t[q].re);
                                t[q].re = fmaa(m[r][q].im, g[c][r].im, t[q].re);
                                t[q].im = fmaa(m[r][q].re, g[c][r].im, t[q].im);
                                t[q].im = fmaa(-m[r][q].im, g[c][r].re, t[q].im);
                            }
#pragma unroll
                        for (int q = 0; q < 3; q++) g[c][q] = t[q];
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < CIN; c++) {
                        Cx<float> t[3] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
                        matvec_acc(m, v[c], t);
#pragma unroll
                        for (int q = 0; q < 3; q++) v[c][q] = t[q];
                    }
                }
            }
#pragma unroll
            for (int c = 0; c < COUT; c++)
#pragma unroll
                for (int cp = 0; cp < CIN; cp++) {
                    float re = 0.f, im = 0.f;
#pragma unroll
                    for (int q = 0; q < 3; q++) {   // conj(v) g
                        re = fmaa(v[cp][q].re, g[c][q].re, re);
                        re = fmaa(v[cp][q].im, g[c][q].im, re);
                        im = fmaa(v[cp][q].re, g[c][q].im, im);
                        im = fmaa(-v[cp][q].im, g[c][q].re, im);
                    }
                    acc[c][cp][0] += re;
                    acc[c][cp][1] += im;
                }
        }
    }
    double *out = a.partials + ((size_t)row * 9 + k) * (COUT * CIN * 2);
#pragma unroll
    for (int c = 0; c < COUT; c++)
#pragma unroll
        for (int cp = 0; cp < CIN; cp++) {
            const double re = wave_sum(acc[c][cp][0]), im = wave_sum(acc[c][cp][1]);
            if (lane == 0) {
                out[(c * CIN + cp) * 2] = re;
                out[(c * CIN + cp) * 2 + 1] = im;
            }
        }
}

// g_w[c][c'][k] = sum over the partial rows: one block per value, each thread
// summing rows t, t + 256, ... in order, then a fixed-order block sum, so the
// result does not depend on scheduling.  WSUM_ADJOINT: the rows are a gradient
// with respect to adjoint weights W' = conj(P W), P the index map; it is stored
// as conj of the value at the reversed index, as a gradient of W.
__global__ void __launch_bounds__(256) k_ptc_wsum(const double *partials, long long nrow, int cin, int cout,
                                                  double *gw, int mode)
{
    __shared__ double lds[16];
    const int v = blockIdx.x;   // value index in [9][cout][cin][2]
    const int nv = 9 * cout * cin * 2;
    double s[1] = {0.0};
    for (long long r = threadIdx.x; r < nrow; r += blockDim.x) s[0] += partials[r * nv + v];
    block_sum<1>(s, lds);
    if (threadIdx.x == 0) {
        const int ri = v & 1, q = v >> 1;
        const int k = q / (cout * cin), c = (q / cin) % cout, cp = q % cin;
        if (mode == WSUM_ADJOINT) {
            gw[2 * adjoint_index(c, cp, k, cout) + ri] = ri ? -s[0] : s[0];
        } else {
            const int o = ((c * cin + cp) * 9 + k) * 2 + ri;
            gw[o] = mode == WSUM_ADD ? gw[o] + s[0] : s[0];
        }
    }
}

// Drawn pairs gathered into the batch: one launch per step in place of two
// copies per pair (about 3 us each, 50 us of a step at a batch of 8).
__global__ void __launch_bounds__(256) k_ptc_pairs(PtcPairs a)
{
    const int j = blockIdx.y;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.norm[j] = a.norm_of[j];
    const float2 *src = reinterpret_cast<const float2 *>(a.mem) + 2 * a.nv * a.index[j];
    float2 *r = reinterpret_cast<float2 *>(a.r) + a.nv * j, *e = reinterpret_cast<float2 *>(a.e) + a.nv * j;
    for (long long t = (long long)blockIdx.x * 256 + threadIdx.x; t < a.nv; t += (long long)gridDim.x * 256) {
        const float2 u = src[t], v = src[a.nv + t];
        r[t] = u;
        e[t] = v;
    }
}

// Loss of a batch of B pairs (z_b = M r_b, e_b the target):
//   L = 1 - |S|^2 / (B Q),  S = sum_b <z_b, e_b> / |e_b|^2,  Q = sum_b |z_b|^2 / |e_b|^2,
// the normalised least-squares misfit of z_b ~ c e_b with one common c (M A
// close to a multiple of 1 on the error directions), invariant to the scale
// of M.  Passes: per-tile partials of (Re, Im <z, e>, |z|^2); per-pair totals;
// S, Q and L; the gradient g_b = -2 (conj(S) e_b Q - |S|^2 z_b) / (B Q^2 |e_b|^2)
// on even sites.
// The vector the loss measures z against: z itself (Euclidean), or A z =
// wdiag z - D_eo D_oe z (energy norm), element f of batch entry b.
__device__ __forceinline__ float2 weighted(const PtcLaunch &a, int b, long long f, float2 z)
{
    if (!a.wvec) return z;
    const float2 u = reinterpret_cast<const float2 *>(a.wvec + (size_t)b * a.in_bstride)[f];
    const float dg = (float)a.wdiag;
    return make_float2(dg * z.x - u.x, dg * z.y - u.y);
}

__global__ void __launch_bounds__(192) k_ptc_loss_dots(PtcLaunch a)
{
    const ProbDesc &pd = a.probs[0];
    const int tile = blockIdx.x, b = blockIdx.y;
    const long long f = (long long)tile * TILE * 3 + threadIdx.x;
    double part[3] = {0.0, 0.0, 0.0};
    if (f < (long long)pd.h * 3) {
        const float2 z = reinterpret_cast<const float2 *>(a.in + (size_t)b * a.in_bstride)[f];
        const float2 t = reinterpret_cast<const float2 *>(a.tgt + (size_t)b * a.tgt_bstride)[f];
        const float2 zw = weighted(a, b, f, z);
        part[0] = (double)z.x * t.x + (double)z.y * t.y;
        part[1] = (double)z.x * t.y - (double)z.y * t.x;
        part[2] = (double)z.x * zw.x + (double)z.y * zw.y;
    }
    publish_partials<3>(part, a.partials, b * gridDim.x + tile);
}

__global__ void __launch_bounds__(256) k_ptc_loss_fin(const double *partials, int ntile, double *pstat)
{
    __shared__ double lds[16 * 3];
    const int b = blockIdx.x;
    double acc[3] = {0.0, 0.0, 0.0};
    for (int j = threadIdx.x; j < ntile; j += blockDim.x) {
        const double *p = partials + ((size_t)b * ntile + j) * NPART;
        acc[0] += p[0];
        acc[1] += p[1];
        acc[2] += p[2];
    }
    block_sum<3>(acc, lds);
    if (threadIdx.x == 0) {
        pstat[4 * b + 0] = acc[0];
        pstat[4 * b + 1] = acc[1];
        pstat[4 * b + 2] = acc[2];
    }
}

// one thread: S, Q, L over the batch (fixed order); S, Q, L kept after the pairs
__global__ void k_ptc_lsum(double *pstat, const double *ee, int npair, double *loss)
{
    if (threadIdx.x != 0) return;
    double sr = 0, si = 0, q = 0;
    for (int b = 0; b < npair; b++) {
        sr += pstat[4 * b] / ee[b];
        si += pstat[4 * b + 1] / ee[b];
        q += pstat[4 * b + 2] / ee[b];
    }
    const double l = 1.0 - (sr * sr + si * si) / (npair * q);
    pstat[4 * npair + 0] = sr;
    pstat[4 * npair + 1] = si;
    pstat[4 * npair + 2] = q;
    *loss = l;
}

__global__ void __launch_bounds__(192) k_ptc_loss_grad(PtcLaunch a, const double *pstat)
{
    const ProbDesc &pd = a.probs[0];
    const int tile = blockIdx.x, b = blockIdx.y, B = gridDim.y;
    const long long f = (long long)tile * TILE * 3 + threadIdx.x;
    if (f >= (long long)pd.h * 3) return;
    const double sr = pstat[4 * B], si = pstat[4 * B + 1], q = pstat[4 * B + 2];
    const double den = (double)B * q * q * a.ee[b];
    // g = Ac t + Bc z_w,  Ac = -2 conj(S) Q / den,  Bc = 2 |S|^2 / den (t the
    // target: e, or r for the energy norm; z_w = z, or A z)
    const float ar = (float)(-2.0 * sr * q / den), ai = (float)(2.0 * si * q / den);
    const float bc = (float)(2.0 * (sr * sr + si * si) / den);
    const float2 z = reinterpret_cast<const float2 *>(a.in + (size_t)b * a.in_bstride)[f];
    const float2 t = reinterpret_cast<const float2 *>(a.tgt + (size_t)b * a.tgt_bstride)[f];
    const float2 zw = weighted(a, b, f, z);
    reinterpret_cast<float2 *>(a.out + (size_t)b * a.out_bstride)[f] =
        make_float2(ar * t.x - ai * t.y + bc * zw.x, ar * t.y + ai * t.x + bc * zw.y);
}

// The working copies of complex weight j (FP32 master value w): the adjoint's
// in FP32 and FP16, W'[c'][c][k'] = conj(W[c][c'][k]).
__device__ __forceinline__ void put_adjoint(const PtcNet &net, int j, float re, float im)
{
    int l = 0;
    while (j >= net.woff[l + 1]) l++;
    const int cin = net.chans[l], cout = net.chans[l + 1];
    const int t = j - net.woff[l], k = t % 9, cp = (t / 9) % cin, c = t / (9 * cin);
    const int o = net.woff[l] + adjoint_index(c, cp, k, cout);
    net.wa32[2 * o] = re;
    net.wa32[2 * o + 1] = -im;
    net.wa16[2 * o] = __float2half_rn(re);
    net.wa16[2 * o + 1] = __float2half_rn(-im);
}

__global__ void k_ptc_adjoint(PtcNet net)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < net.woff[net.nlayer]) put_adjoint(net, j, net.w32[2 * j], net.w32[2 * j + 1]);
}

// Adam on the FP32 master weights (one complex weight per thread, its parts
// separate parameters); refreshes the working copies of the weight and of the
// adjoint (one launch instead of one more per layer, 4.4 us each).
__global__ void k_adam(PtcNet net, float *m, float *v, const double *g, int step, float lr, float b1, float b2,
                       float eps)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= net.woff[net.nlayer]) return;
    float wn[2];
#pragma unroll
    for (int ri = 0; ri < 2; ri++) {
        const int j = 2 * t + ri;
        const float gj = (float)g[j];
        const float mj = b1 * m[j] + (1.f - b1) * gj;
        const float vj = b2 * v[j] + (1.f - b2) * gj * gj;
        m[j] = mj;
        v[j] = vj;
        const float mh = mj / (1.f - powf(b1, (float)step));
        const float vh = vj / (1.f - powf(b2, (float)step));
        wn[ri] = net.w32[j] - lr * mh / (sqrtf(vh) + eps);
        net.w32[j] = wn[ri];
        net.w16[j] = __float2half_rn(wn[ri]);
    }
    put_adjoint(net, t, wn[0], wn[1]);
}

// ------------------------------------------------------------- launchers

// How a layer is applied: 0 four waves, batch entries sharing the unpacked
// links; the others for one entry per block on lattices whose fat links stream
// past the Infinity Cache (FP32 recon-18: 576 bytes a site, FP16 recon-12: 192):
// 1 four waves, 2 one wave, both in plain order.  One layer in us by form 0 / 1 /
// 2:
//             1 -> 1            2 -> 2            4 -> 4            8 -> 1
//   FP32 24^4     33 / 38 / 40     41 / 46 / 47    56 / 64 / 69    59 / 73 / 86
//        24^3x48  82 / 78 / 82     94 / 88 / 94   122 / 117 / 132  134 / 162 / 167
//        28^4     80 / 75 / 77     91 / 88 / 93   116 / 119 / 129  118 / 164 / 174
//        32^4    134 / 127 / 125  150 / 146 / 142 200 / 197 / 205  267 / 261 / 246
//   FP16 24^3x48  33 / 39 / 36     47 / 51 / 49    90 / 98 / 100   89 / 124 / 121
//        32^4     51 / 54 / 51     81 / 80 / 72   148 / 158 / 158 154 / 200 / 174
//        32^3x64 114 / 120 / 104  165 / 174 / 145 298 / 309 / 321 336 / 397 / 363
// Where four or more channels are gathered for fewer, the vectors count for more
// than the links, and form 0 keeps their neighbours in an XCD's L2.
static int layer_form(int prec, int cin, int cout, long long V, int bper)
{
    if (bper > 1 || cin * cout >= 64 || (cin > 2 && cin > cout)) return 0;
    if (prec == 2) return V >= 1 << 20 && cin <= 2 ? 2 : 0;
    if (V <= 1 << 19) return 0;
    return V >= 1 << 20 && (cin == 1 || cout == 1) ? 2 : 1;
}

template <class LT, int R, class WT, int I, int O>
static hipError_t layer_f(int form, const PtcLaunch &a, dim3 g, hipStream_t s)
{
    if constexpr (I * O < 64) {
        if (form == 2) {
            hipLaunchKernelGGL((k_ptc_layer<LT, R, WT, I, O, 1, true>), g, dim3(64), 0, s, a);
            return hipGetLastError();
        }
        if constexpr (sizeof(LT) == 4)
            if (form == 1) {
                hipLaunchKernelGGL((k_ptc_layer<LT, R, WT, I, O, 4, true>), g, dim3(256), 0, s, a);
                return hipGetLastError();
            }
    }
    hipLaunchKernelGGL((k_ptc_layer<LT, R, WT, I, O, 4, false>), g, dim3(256), 0, s, a);
    return hipGetLastError();
}

template <class LT, int R, class WT>
static hipError_t layer_c(int form, int cin, int cout, const PtcLaunch &a, dim3 g, hipStream_t s)
{
#define PTC_CASE(I, O) \
    if (cin == I && cout == O) return layer_f<LT, R, WT, I, O>(form, a, g, s);
    PTC_CASE(1, 1) PTC_CASE(1, 4) PTC_CASE(4, 4) PTC_CASE(4, 1) PTC_CASE(1, 2) PTC_CASE(2, 2) PTC_CASE(2, 1)
    PTC_CASE(2, 4) PTC_CASE(4, 2) PTC_CASE(1, 8) PTC_CASE(8, 8) PTC_CASE(8, 1)
#undef PTC_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_ptc_layer(int prec, int recon, bool w16, int cin, int cout, const PtcLaunch &a, int nblk,
                            long long V, hipStream_t s)
{
    dim3 g(nblk, (a.batch + a.bper - 1) / a.bper);
    const int f = layer_form(prec, cin, cout, V, a.bper);
    if (prec == 1 && recon == 18)
        return w16 ? layer_c<float, 18, __half>(f, cin, cout, a, g, s) : layer_c<float, 18, float>(f, cin, cout, a, g, s);
    if (prec == 2 && recon == 12)
        return w16 ? layer_c<__half, 12, __half>(f, cin, cout, a, g, s) : layer_c<__half, 12, float>(f, cin, cout, a, g, s);
    return hipErrorInvalidValue;
}

template <class LT, int R, int I, int O>
static hipError_t wgrad_w(bool nine, const PtcLaunch &a, int npar, int nrow, hipStream_t s)
{
    if constexpr (I == 1 || O == 1 || I * O <= 4)
        if (nine) {
            hipLaunchKernelGGL((k_ptc_wgrad<LT, R, I, O, 9>), dim3(nrow), dim3(576), 0, s, a, npar, nrow);
            return hipGetLastError();
        }
    hipLaunchKernelGGL((k_ptc_wgrad<LT, R, I, O, 4>), dim3(nrow, 3), dim3(256), 0, s, a, npar, nrow);
    return hipGetLastError();
}

template <class LT, int R>
static hipError_t wgrad_c(bool nine, int cin, int cout, const PtcLaunch &a, int npar, int nrow, hipStream_t s)
{
#define WG_CASE(I, O) \
    if (cin == I && cout == O) return wgrad_w<LT, R, I, O>(nine, a, npar, nrow, s);
    WG_CASE(1, 1) WG_CASE(1, 4) WG_CASE(4, 4) WG_CASE(4, 1) WG_CASE(1, 2) WG_CASE(2, 2) WG_CASE(2, 1)
    WG_CASE(2, 4) WG_CASE(4, 2) WG_CASE(1, 8) WG_CASE(8, 8) WG_CASE(8, 1)
#undef WG_CASE
    return hipErrorInvalidValue;
}

// transports on FP32 recon-18 (prec 1) or FP16 recon-12 (prec 2) fat links
hipError_t launch_ptc_wgrad(int prec, int recon, bool nine, int cin, int cout, const PtcLaunch &a, int npar, int nrow,
                            hipStream_t s)
{
    if (prec == 1 && recon == 18) return wgrad_c<float, 18>(nine, cin, cout, a, npar, nrow, s);
    if (prec == 2 && recon == 12) return wgrad_c<__half, 12>(nine, cin, cout, a, npar, nrow, s);
    return hipErrorInvalidValue;
}

hipError_t launch_ptc_wsum(const double *partials, long long nrow, int cin, int cout, double *gw, int mode,
                           hipStream_t s)
{
    const int nv = 9 * cout * cin * 2;
    hipLaunchKernelGGL(k_ptc_wsum, dim3(nv), dim3(256), 0, s, partials, nrow, cin, cout, gw, mode);
    return hipGetLastError();
}

hipError_t launch_ptc_pairs(const PtcPairs &a, hipStream_t s)
{
    const long long nb = (a.nv + 255) / 256;
    hipLaunchKernelGGL(k_ptc_pairs, dim3((unsigned)(nb < 1024 ? nb : 1024), a.n), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_ptc_loss(const PtcLaunch &a, int ntile, int batch, double *loss, hipStream_t s)
{
    double *pstat = a.partials + (size_t)batch * ntile * NPART;
    hipLaunchKernelGGL(k_ptc_loss_dots, dim3(ntile, batch), dim3(192), 0, s, a);
    hipLaunchKernelGGL(k_ptc_loss_fin, dim3(batch), dim3(256), 0, s, a.partials, ntile, pstat);
    hipLaunchKernelGGL(k_ptc_lsum, dim3(1), dim3(64), 0, s, pstat, a.ee, batch, loss);
    hipLaunchKernelGGL(k_ptc_loss_grad, dim3(ntile, batch), dim3(192), 0, s, a, (const double *)pstat);
    return hipGetLastError();
}

hipError_t launch_adam(const PtcNet &net, float *m, float *v, const double *g, int step, float lr, hipStream_t s)
{
    hipLaunchKernelGGL(k_adam, dim3((net.woff[net.nlayer] + 255) / 256), dim3(256), 0, s, net, m, v, g, step, lr, 0.9f,
                       0.999f, 1e-8f);
    return hipGetLastError();
}

hipError_t launch_ptc_adjoint(const PtcNet &net, hipStream_t s)
{
    hipLaunchKernelGGL(k_ptc_adjoint, dim3((net.woff[net.nlayer] + 255) / 256), dim3(256), 0, s, net);
    return hipGetLastError();
}

}  // namespace hisq
