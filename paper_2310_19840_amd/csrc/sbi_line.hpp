// sbi_line.hpp -- operands of the one-dimensional solve and step kernel (sbi_line.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "sbi_internal.hpp"
#include "sbi_kernels.hpp"

namespace sbi {

// fields at the points: eta, delta, eta_x, phi_x, the damping weight, a work
// field, the orders V_1 .. V_6 (the iterate in the first) and their d_x phi_b
enum { LF_ETA, LF_DELTA, LF_EX, LF_PX, LF_MU, LF_NL, LF_V0, LF_B0 = LF_V0 + 6, LF_COUNT = LF_B0 + 6 };

struct LineParams {
    GridDev g;
    int sa;              // 1: successive approximation, 0: iteration
    int vd, aa;          // variable bed; Anderson-mixed sweeps
    int max_sweeps;
    double tol;
    // steps > 0: that many steps of rk.h from time t0 on the state (rk.eh, rk.ph);
    // 0: one solve at (eta_in, phi_in)
    int steps;
    int load;            // first transform the physical phi_in (and eta_in when stepping) to the state
    int acc_reset;       // clear the totals over solves first
    int keep;            // go on stepping after a failed solve (ensembles)
    double t0;
    const void* eta_in;
    const void* phi_in;
    RkParams rk;         // state, stage state, accumulators, W spectrum, N_phi, damping pressure, filter
    void* pd;            // damping pressure's divergence (rk.Pdiv), written
    void* np;            // N_phi (rk.Nph), written; the sweeps keep f_n there
    void* vh;            // W spectrum: the SA sum, or T(V_n) of the iteration (rk.Vh)
    void* vn;            // current order / iterate (V, phi_b)
    void* bn;
    void* bv;            // forcing of the iteration
    void* bb;
    void* ring[4][kAASlots];  // residual and relaxed-sweep history: f (V, phi_b), g (V, phi_b)
    void* gv;            // half forms left for the caller of a solve: V (SA: W), D, T
    void* gd;
    void* gt;
    void* f[LF_COUNT];   // fields at the points (where the kernel does not keep them in LDS)
    Ctl* ctl;
    // wave tank and relaxation zones, as in RowNphiParams and RowBlendParams
    int wm_n;
    double wm[kMaxWavemaker][4];
    double wm_h, dmp_x0, dmp_w;
    int rz_on;
    double rz[6];
};

// threads per member (0: the kernel does not take this row length)
int line_threads(int nx);
template <typename R> hipError_t launch_line_t(const LineParams&, int batch, const Twiddles&, hipStream_t);
hipError_t launch_line(int fp64, const LineParams& p, int batch, const Twiddles& tw, hipStream_t s);

}  // namespace sbi
