// Launch descriptors of the PTC preconditioner and flexible-CG kernels.
#pragma once
#include "hisq_dev.h"

namespace hisq {

struct PtcLaunch {
    const ProbDesc *probs;   // the lattice (links, geometry)
    int lslot;               // link set for the transports
    int in_zero_par;         // parity whose input is known zero (-1: none)
    const void *w;           // weights [Cout][Cin][9] complex (float2 or half2)
    const float *in;         // input activations [B][Cin][2][h][3] complex
    long long in_bstride;    // floats between batch entries
    float *out;              // output [B][Cout][out_pstride][h][3]
    long long out_bstride;
    int out_pstride;         // parities stored per output channel (1 or 2)
    int out_par0;            // first stored output parity
    int par_lo;              // first output parity computed (grid: npar * ntile blocks)
    int batch, bper;         // batch entries, and how many of them one block (layer) or unit (weight gradient) takes
    const float *g;          // weight gradient: output gradient [B][Cout][g_pstride][h][3]
    long long g_bstride;
    int g_pstride, g_par0;
    double *partials;
    const float *tgt;        // loss: targets [B][h][3]
    long long tgt_bstride;
    const double *ee;        // loss: normalisation per batch entry (|e|^2, or <e, r> for the energy norm)
    const float *wvec;       // energy-norm loss: D_eo D_oe z, so that A z = wdiag z - wvec (null: Euclidean)
    double wdiag;
    // flexible-CG fusion (all null / unused otherwise)
    const SolveState *gate;  // skip the launch unless gate->status == gate_want
    int gate_want;
    int dot_nt;              // tiles of the dot partials below
    const float *addin;      // out += addin (same layout as out, COUT = 1, one parity)
    long long addin_bstride;
    const float *dotq;       // with dotred: per-tile (dotq, out) into dotred[tile], dotred[dot_nt + tile]
    double *dotred;
};

// Fusion of the preconditioner into the flexible CG's iteration: launches are
// skipped unless gate->status == want, and the final layer also forms the
// per-tile partials of (q, z) (re in red[tile], im in red[nt + tile]).
struct PtcFuse {
    const SolveState *gate;
    int want;
    const float *q;
    double *red;
    int nt;
};

// V: sites of the lattice
hipError_t launch_ptc_layer(int prec, int recon, bool w16, int cin, int cout, const PtcLaunch &a, int nblk,
                            long long V, hipStream_t s);

// Blocks that a layer launch should have before its batch entries share blocks:
// one full load of the 256 CUs at the three or four waves per SIMD that the
// kernels' registers allow (16^4, batch 8: 1024 blocks 57 / 22 / 30 us for
// 4->4 / 1->4 / 4->1, 2048 blocks 55 / 24 / 30, 4096 blocks 60 / 26 / 33; with it
// training steps of 1 to 64 pairs from 4^4 to 16^3x32 take 0.24 to 0.92 of the
// time that one entry per block took, of 2 to 8 pairs at 32^4 0.45 to 1.01)
constexpr int LAYER_BLOCKS = 1024;

// Inference layer with FP16 activation storage (ptc_infer.hip): activations
// [2 parities][h][C][3] half2 plus one FP32 scale per (parity, site).
struct PtcInferLaunch {
    const ProbDesc *probs;
    int lslot;
    int par_lo;              // first output parity (grid: npar * ntile blocks)
    const void *w;           // FP16 weights [Cout][Cin][9] complex
    const float *in32;       // input kind 0: even FP32 vector [h][3] complex (odd parity zero)
    const __half2 *in16;     // input kind 1: FP16 activation
    const float *in_scale;
    __half2 *out16;          // output kind 0: FP16 activation
    float *out_scale;
    float *out32;            // output kind 1: even FP32 vector z = addin + layer output
    const float *addin;
    const float *dotq;       // with dotred: per-tile (dotq, z) into dotred[tile], dotred[dot_nt + tile]
    double *dotred;
    int dot_nt;
    int gate_want;
    const SolveState *gate;  // skip the launch unless gate->status == gate_want
};
// W: 1, 3 or 9 waves per block, or'ed with PTC_MFMA (3 and 9, cout >= cin)
// for the matrix-core channel mixing
constexpr int PTC_MFMA = 0x100;
hipError_t launch_ptc_infer(int prec, int recon, int cin, int cout, int ik, int ok, int W, const PtcInferLaunch &a,
                            int nblk, hipStream_t s);
// Weight-gradient partial rows at most (a multiple of the 8 XCDs): the 9 waves
// of a row, in blocks of four, load the 256 CUs once at three waves per SIMD.
// Units wanted before batch entries share one: the rows that take one unit more
// than others then cost at most a tenth.
constexpr int WGRAD_ROWS = 336, WGRAD_UNITS = 10 * WGRAD_ROWS;
// Rows of nine-wave blocks, a path each, for a single entry on lattices beyond
// the caches and few channels (32^4, FP16 links, layer_backward: 1 -> 1 115 us
// with WGRAD_ROWS rows of four-wave blocks, 94 so; 2 -> 2 143 and 125, 8 -> 1 in
// FP32 303 and 292; 4 -> 4 216 and 258; at 24^4 55 and 53, 62 and 62).
constexpr int WGRAD_NINE_ROWS = 1024;
inline bool wgrad_nine(int cin, int cout, long long V, int bper)
{
    return bper == 1 && V > 1 << 19 && (cin == 1 || cout == 1 || cin * cout <= 4);
}

// Weight-gradient partials of npar output parities x a.batch entries, reduced
// into nrow rows of [9][cout][cin] complex FP64.
hipError_t launch_ptc_wgrad(int prec, int recon, bool nine, int cin, int cout, const PtcLaunch &a, int npar, int nrow,
                            hipStream_t s);
enum : int { WSUM_SET = 0, WSUM_ADD = 1, WSUM_ADJOINT = 2 };
hipError_t launch_ptc_wsum(const double *partials, long long nrow, int cin, int cout, double *gw, int mode,
                           hipStream_t s);
// Gather of drawn training pairs (r, e) and their normalisations.
constexpr int PTC_PAIRS = 16;   // pairs per launch (their indices travel in the kernel arguments)
struct PtcPairs {
    const float *mem;        // pair j: r at 2j nv, e at (2j + 1) nv complex values
    float *r, *e;            // [n][nv] complex
    double *norm;            // [n]
    long long nv;            // complex values of a vector
    int n;
    int index[PTC_PAIRS];
    double norm_of[PTC_PAIRS];
};
hipError_t launch_ptc_pairs(const PtcPairs &a, hipStream_t s);
hipError_t launch_ptc_loss(const PtcLaunch &a, int ntile, int batch, double *loss, hipStream_t s);
// A network's weights: layer l has chans[l] inputs, chans[l + 1] outputs and
// starts at complex weight woff[l] (woff[nlayer]: all of them).
constexpr int PTC_MAX_LAYERS = 8;
struct PtcNet {
    float *w32, *wa32;       // FP32 master weights, their adjoint
    __half *w16, *wa16;      // FP16 copies
    int nlayer;
    int chans[PTC_MAX_LAYERS + 1], woff[PTC_MAX_LAYERS + 1];
};
// One Adam step on w32, and the copies it leaves stale; launch_ptc_adjoint
// refreshes the adjoints alone.
hipError_t launch_adam(const PtcNet &net, float *m, float *v, const double *g, int step, float lr, hipStream_t s);
hipError_t launch_ptc_adjoint(const PtcNet &net, hipStream_t s);
hipError_t launch_to_half(const float *w, __half *w16, int n, hipStream_t s);

// flexible CG vector kernels (FP32 vectors, complex FP64 scalars in SolveState::cplx)
struct FcgLaunch {
    const ProbDesc *probs;
    SolveState *states;
    int want;
    int op;
    double *partials;
    float *r, *x, *p, *q, *z;
    double *red;   // fused ops: compact tile sums [(p,q)][Re (p,r)][Im (p,r)][|r|^2][Re (q,z)][Im (q,z)], nt each
    int nt;
};
enum : int { FCG_DOTS_B = 2, FCG_P = 3, FCG_XR_F = 4, FCG_P_F = 5, FCG_DOT_PR = 6 };
// offsets of the compact sums in FcgLaunch::red, in units of nt
// (the three sums each fused op reads are adjacent)
enum : int { FRED_PQ = 0, FRED_PR = 1, FRED_RR = 3, FRED_QZ = 4, FRED_N = 6 };
hipError_t launch_fcg(const FcgLaunch &a, int ntile, hipStream_t s);

}  // namespace hisq
