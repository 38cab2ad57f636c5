// sbi_stage.hpp -- device functions of one kept mode or one workgroup that the
// pass kernels and the one-dimensional step kernel share: mode geometry, the
// Runge-Kutta stage update, the Anderson weights.
#pragma once
#include "sbi_device.hpp"
#include "sbi_fft.hpp"
#include "sbi_kernels.hpp"

namespace sbi {

__device__ __forceinline__ double sech_d(double x) {
    double e = exp(-fabs(x));
    return 2.0 * e / (1.0 + e * e);
}

struct ModeGeo {
    int r, mx;
    bool valid;
    double kx, ky, k;
};
__device__ __forceinline__ ModeGeo mode_geo(const GridDev& g, long long idx) {
    ModeGeo m;
    m.mx = (int)(idx / g.Ky);
    m.r = (int)(idx % g.Ky);
    m.valid = m.r < g.Ky && m.mx < g.Kx;
    const int my = m.r <= g.My ? m.r : m.r - g.Ky;
    m.kx = 2.0 * M_PI * m.mx / g.lx;
    m.ky = g.ny == 1 ? 0.0 : 2.0 * M_PI * my / g.ly;
    m.k = sqrt(m.kx * m.kx + m.ky * m.ky);
    return m;
}

// Stage `stage` of the integrating-factor Runge-Kutta step (Lawson form) of one mode, at
// element o of the compact fields
template <typename R>
__device__ __forceinline__ void rk_mode(const RkParams& p, int stage, const ModeGeo& m, long long o, double href) {
    using V = typename cplx_of<R>::type;
    const double om2 = m.k * tanh(m.k * href);
    const double om = sqrt(om2);
    const double h = p.h;
    V* eh = static_cast<V*>(p.eh);
    V* ph = static_cast<V*>(p.ph);
    V* es = static_cast<V*>(p.es);
    V* ps = static_cast<V*>(p.ps);
    V* ae = static_cast<V*>(p.ae);
    V* ap = static_cast<V*>(p.ap);
    const V vh = static_cast<const V*>(p.Vh)[o];
    const V nph = static_cast<const V*>(p.Nph)[o];
    const V psv = ps[o];
    // derivative of the stage: (W_hat - omega^2 phi_hat, N_phi [- p_d_hat])
    const double de_r = (double)vh.x - om2 * (double)psv.x, de_i = (double)vh.y - om2 * (double)psv.y;
    double dp_r = (double)nph.x, dp_i = (double)nph.y;
    if (p.Pdiv && m.k > 0.0) {
        const V pd = static_cast<const V*>(p.Pdiv)[o];
        dp_r += (double)pd.x / (m.k * m.k);
        dp_i += (double)pd.y / (m.k * m.k);
    }
    const double u_er = (double)eh[o].x, u_ei = (double)eh[o].y;
    const double u_pr = (double)ph[o].x, u_pi = (double)ph[o].y;
    auto prop = [&](double tau, double er, double ei, double pr, double pi_, double* oer, double* oei, double* opr,
                    double* opi) {
        const double c = cos(om * tau), s = sin(om * tau);
        const double sw = om > 0.0 ? s / om : tau;
        *oer = c * er + om * s * pr;
        *oei = c * ei + om * s * pi_;
        *opr = -sw * er + c * pr;
        *opi = -sw * ei + c * pi_;
    };
    double a_er, a_ei, a_pr, a_pi;   // accumulator
    double n_er, n_ei, n_pr, n_pi;   // next stage state
    if (stage == 0) {
        prop(h, de_r, de_i, dp_r, dp_i, &a_er, &a_ei, &a_pr, &a_pi);
        prop(0.5 * h, u_er + 0.5 * h * de_r, u_ei + 0.5 * h * de_i, u_pr + 0.5 * h * dp_r, u_pi + 0.5 * h * dp_i,
             &n_er, &n_ei, &n_pr, &n_pi);
    } else if (stage == 1 || stage == 2) {
        double b_er, b_ei, b_pr, b_pi;
        prop(0.5 * h, de_r, de_i, dp_r, dp_i, &b_er, &b_ei, &b_pr, &b_pi);
        a_er = (double)ae[o].x + 2.0 * b_er;
        a_ei = (double)ae[o].y + 2.0 * b_ei;
        a_pr = (double)ap[o].x + 2.0 * b_pr;
        a_pi = (double)ap[o].y + 2.0 * b_pi;
        if (stage == 1) {
            prop(0.5 * h, u_er, u_ei, u_pr, u_pi, &n_er, &n_ei, &n_pr, &n_pi);
            n_er += 0.5 * h * de_r;
            n_ei += 0.5 * h * de_i;
            n_pr += 0.5 * h * dp_r;
            n_pi += 0.5 * h * dp_i;
        } else {
            prop(h, u_er, u_ei, u_pr, u_pi, &n_er, &n_ei, &n_pr, &n_pi);
            n_er += h * b_er;
            n_ei += h * b_ei;
            n_pr += h * b_pr;
            n_pi += h * b_pi;
        }
    } else {
        prop(h, u_er, u_ei, u_pr, u_pi, &n_er, &n_ei, &n_pr, &n_pi);
        n_er += h / 6.0 * ((double)ae[o].x + de_r);
        n_ei += h / 6.0 * ((double)ae[o].y + de_i);
        n_pr += h / 6.0 * ((double)ap[o].x + dp_r);
        n_pi += h / 6.0 * ((double)ap[o].y + dp_i);
        if (p.fb1 > 0.0 && p.fb2 > 0.0) {
            const double lam = exp(-pow(fabs(m.k / p.fb1), p.fb2));
            n_er *= lam;
            n_ei *= lam;
            n_pr *= lam;
            n_pi *= lam;
        }
        eh[o] = cx<V>(R(n_er), R(n_ei));
        ph[o] = cx<V>(R(n_pr), R(n_pi));
        es[o] = cx<V>(R(n_er), R(n_ei));
        ps[o] = cx<V>(R(n_pr), R(n_pi));
        return;
    }
    ae[o] = cx<V>(R(a_er), R(a_ei));
    ap[o] = cx<V>(R(a_pr), R(a_pi));
    es[o] = cx<V>(R(n_er), R(n_ei));
    ps[o] = cx<V>(R(n_pr), R(n_pi));
}

// entry i of a register array, with i known only at run time: a chain of
// selects, so the array is never placed in memory
static __device__ __forceinline__ double aa_sel(const double (&v)[kAASlots], int i) {
    double r = 0.0;
#pragma unroll
    for (int q = 0; q < kAASlots; ++q) r = q == i ? v[q] : r;
    return r;
}

// Anderson mixing of the relaxed sweep: from dots[i] = <F_i, f_n> over the
// ring slots of sweep n, complete the Gram matrix of the residual history,
// solve the normal equations of min |f_n - sum_a gamma_a dF_a|,
// dF_a = F_(a+1) - F_a over the history in sweep order (regularised by
// 1e-12 trace / k; gamma = 0 when they fail), and write to w the weights of
// x_(n+1) = g_n - sum_a gamma_a (G_(a+1) - G_a) on the history slots.
// commit: store the new Gram entries (row and column of slot n) in the control
// block, whose entries (or a copy) gram gives.  Those read here are not in that
// row and column: they
// were stored by earlier sweeps, so workgroups of one pass that solve
// side by side while one of them commits read the same values.
// dots and w are indexed with compile-time indices only (registers); the
// history slots in sweep order are H_a = (n - k + a) mod kAASlots, a <= k
static __device__ void aa_weights(Ctl* ctl, const double* gram, int n, const double (&dots)[kAASlots],
                                  double (&w)[kAASlots], bool commit) {
    static_assert(kAADepth == 2, "the elimination below is written out for two residual differences");
    const int s = n % kAASlots, k = n < kAADepth ? n : kAADepth;
    const int H0 = (n - k) % kAASlots, H1 = (n - k + 1) % kAASlots, H2 = (n - k + 2) % kAASlots;
    // the new row and column of slot s (over the slots of the history) come
    // from dots; the other entries were stored by earlier sweeps
    if (commit) {
#pragma unroll
        for (int i = 0; i < kAASlots; ++i) {
            const bool hi = i == H0 || (k >= 1 && i == H1) || (k >= 2 && i == H2);
            if (hi) {
                ctl->aa_gram[s][i] = aa_sel(dots, i);
                ctl->aa_gram[i][s] = aa_sel(dots, i);
            }
        }
    }
    auto M = [&](int a, int b) {
        const int r = a == 0 ? H0 : (a == 1 ? H1 : H2), c = b == 0 ? H0 : (b == 1 ? H1 : H2);
        if (r == s) return aa_sel(dots, c);
        if (c == s) return aa_sel(dots, r);
        return gram[r * kAASlots + c];
    };
    double gam0 = 0.0, gam1 = 0.0;
    if (k == 1) {
        double A00 = M(1, 1) - M(1, 0) - M(0, 1) + M(0, 0);
        const double y0 = M(1, 1) - M(0, 1);
        const double tr = A00;
        A00 += 1e-12 * tr;
        const bool ok = tr > 0.0 && isfinite(tr) && fabs(A00) > 0.0;
        gam0 = ok ? y0 / A00 : 0.0;
        if (!isfinite(gam0)) gam0 = 0.0;
    } else if (k == 2) {
        double A00 = M(1, 1) - M(1, 0) - M(0, 1) + M(0, 0);
        double A01 = M(1, 2) - M(1, 1) - M(0, 2) + M(0, 1);
        double A10 = M(2, 1) - M(2, 0) - M(1, 1) + M(1, 0);
        double A11 = M(2, 2) - M(2, 1) - M(1, 2) + M(1, 1);
        double y0 = M(1, 2) - M(0, 2), y1 = M(2, 2) - M(1, 2);
        const double tr = A00 + A11;
        const double reg = 1e-12 * tr / 2;
        A00 += reg;
        A11 += reg;
        bool ok = tr > 0.0 && isfinite(tr);
        // Gaussian elimination with partial pivoting on the first column
        if (fabs(A10) > fabs(A00)) {
            double t = A00; A00 = A10; A10 = t;
            t = A01; A01 = A11; A11 = t;
            t = y0; y0 = y1; y1 = t;
        }
        ok = ok && fabs(A00) > 0.0;
        if (ok) {
            const double f = A10 / A00;
            A11 -= f * A01;
            y1 -= f * y0;
            ok = fabs(A11) > 0.0;
        }
        if (ok) {
            gam1 = y1 / A11;
            gam0 = (y0 - A01 * gam1) / A00;
            ok = isfinite(gam0) && isfinite(gam1);
        }
        if (!ok) gam0 = gam1 = 0.0;
    }
    // x_(n+1) = G_k - sum_a gamma_a (G_(a+1) - G_a): weights of the history slots
    const double c0 = k == 0 ? 1.0 : gam0;
    const double c1 = k == 1 ? 1.0 - gam0 : gam1 - gam0;
    const double c2 = 1.0 - gam1;
#pragma unroll
    for (int i = 0; i < kAASlots; ++i)
        w[i] = i == H0 ? c0 : ((k >= 1 && i == H1) ? c1 : ((k >= 2 && i == H2) ? c2 : 0.0));
}

// block sums of d -> out[0 .. kAASlots) (fixed order; s_red: kAASlots per wavefront)
__device__ __forceinline__ void col_aa_reduce(double (&d)[kAASlots], double* s_red, double* out) {
#pragma unroll
    for (int i = 0; i < kAASlots; ++i)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) d[i] += __shfl_xor(d[i], off, 64);
    const int wv = threadIdx.x / 64, nw = blockDim.x / 64;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int i = 0; i < kAASlots; ++i) s_red[wv * kAASlots + i] = d[i];
    lds_sync();
    if (threadIdx.x < kAASlots) {
        double v = 0.0;
        for (int w = 0; w < nw; ++w) v += s_red[w * kAASlots + threadIdx.x];
        out[threadIdx.x] = v;
    }
}

// the weights inside a column-pass workgroup: its first wavefront adds the
// member's partials in a fixed order (strided per lane, then across the lanes),
// so every workgroup forms the same weights; s_w receives them.  head: the first
// 64 partials, read ahead by aa_head.
__device__ __forceinline__ void aa_head(const ColParams& p, int mem, double (&head)[kAASlots]) {
#pragma unroll
    for (int i = 0; i < kAASlots; ++i)
        head[i] = (int)threadIdx.x < min(64, p.aa_nblk) ? p.aa_partial[((long long)mem * p.aa_nblk + threadIdx.x) * kAASlots + i] : 0.0;
}
static __device__ __forceinline__ void aa_block_weights(const ColParams& p, Ctl* ctl, int mem, bool commit,
                                                        const double (&head)[kAASlots], double* s_gram, double* s_w) {
    if (threadIdx.x < 64) {
        double d[kAASlots], w[kAASlots];
        if (threadIdx.x < kAASlots * kAASlots) s_gram[threadIdx.x] = (&ctl->aa_gram[0][0])[threadIdx.x];
#pragma unroll
        for (int i = 0; i < kAASlots; ++i) d[i] = head[i];
        const double* part = p.aa_partial + (long long)mem * p.aa_nblk * kAASlots;
#pragma unroll 4
        for (int b = threadIdx.x + 64; b < p.aa_nblk; b += 64)
#pragma unroll
            for (int i = 0; i < kAASlots; ++i) d[i] += part[b * kAASlots + i];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            if (off >= p.aa_nblk) continue;  // the lanes from there on hold zeros
#pragma unroll
            for (int i = 0; i < kAASlots; ++i) d[i] += __shfl_xor(d[i], off, 64);
        }
        wave_lds_sync();
        if (threadIdx.x == 0) {
            aa_weights(ctl, s_gram, p.aa_sweep, d, w, commit);
#pragma unroll
            for (int i = 0; i < kAASlots; ++i) s_w[i] = w[i];
        }
    }
    lds_sync();
}

}  // namespace sbi
