// Launchers of the HISQ fermion-force kernels (FP64).  Fields are the
// site-planar link fields of smear.h; gradients G of a real scalar Q with
// respect to a link field Y are fields with dQ = sum Re Tr(dY_mu(x) G_mu(x)).
#pragma once
#include <hip/hip_runtime.h>

#include "smear.h"

namespace hisq {

// Gradients of Q = sum_k alpha_k X_k^+ A X_k with respect to the fat and long
// links, from the even vectors X_k and Y_k = D_oe X_k ([n][h][3] complex
// each): with Psi = (X on even, Y on odd sites) and eps = +1 / -1 on even /
// odd sites,
//   OF_mu(x) = -2 eps(x) sum_k alpha_k Psi_k(x+mu) Psi_k(x)^+,
//   OL_mu(x) = -2 eps(x) sum_k alpha_k Psi_k(x+3mu) Psi_k(x)^+.
// fold: write eta_mu(x) OF and cN eta_mu(x) OL instead (the gradients with
// respect to the unphased level-2 sum and the Naik product).
struct OuterArgs {
    const double2 *X, *Y;
    const double *alpha;
    int n;
    long long h;
    double2 *OF, *OL;   // four planar fields each
    int fold;
    double cN;
};
hipError_t launch_ff_outer(const SmearGeom &g, const OuterArgs &a, hipStream_t s);

// Adjoint of a fat7 level (see smear.h for its fields): for the gradient G of F
// (four fields), GU (four fields) += the gradient with respect to the links U.
// T1, T2 (twelve fields, 3 mu + k) and, with a Lepage term, H (twenty-four) are
// the forward intermediates, GT1, GT2 the gradients of T1, T2.
//   top    from F_mu's last staples: GT2 and their share of GU;
//   mid    the 5-link staples: GT1 from GT2 and G, and their share of GU; GT1
//          may overwrite T2 (read by top only);
//   split  (with a Lepage term) the gradients of the two signs of the 3-link
//          staples, Gp over GT1 and Gm over anything else (T1 is free now);
//   low    the shares of the 3-link staples (Gp = Gm = GT1 without a Lepage
//          term) and of c1 U.
struct AdjTopArgs {
    const double2 *U, *G, *T2, *H;   // H null: no Lepage term
    double2 *GT2, *GU;
    double c5, c7, cL;
};
struct AdjMidArgs {
    const double2 *U, *G, *T1, *GT2;
    double2 *GT1, *GU;
    double c3;
};
struct AdjSplitArgs {
    const double2 *U, *G;
    double2 *Gp, *Gm;
    double cL;
};
struct AdjLowArgs {
    const double2 *U, *G, *Gp, *Gm;
    double2 *GU;
    double c1;
};
hipError_t launch_adj_top(const SmearGeom &g, const AdjTopArgs &a, hipStream_t s);
hipError_t launch_adj_mid(const SmearGeom &g, const AdjMidArgs &a, hipStream_t s);
hipError_t launch_adj_split(const SmearGeom &g, const AdjSplitArgs &a, hipStream_t s);
hipError_t launch_adj_low(const SmearGeom &g, const AdjLowArgs &a, hipStream_t s);

// GW += gradient of sum Re Tr(N_mu(x) GN_mu(x)), N_mu(x) = W_mu(x) W_mu(x+mu) W_mu(x+2mu)
// (four-direction planar fields).
hipError_t launch_ff_naik_adjoint(const SmearGeom &g, const double2 *W, const double2 *GN, double2 *GW,
                                  hipStream_t s);

// In place: G <- gradient with respect to V of Re Tr(W(V) G), W = V (V^+ V)^{-1/2},
// four-direction planar fields.
hipError_t launch_ff_unitarize_adjoint(const SmearGeom &g, const double2 *V, double2 *G, hipStream_t s);

// out = in over n double2.
hipError_t launch_field_copy(double2 *out, const double2 *in, size_t n, hipStream_t s);

// F_mu(x) = TA[U_mu(x) G_mu(x)] (four-direction planar fields; F may alias G).
hipError_t launch_ff_project(const SmearGeom &g, const double2 *U, const double2 *G, double2 *F, hipStream_t s);

}  // namespace hisq
