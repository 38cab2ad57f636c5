// sbi_line.hip -- W solves and time steps of one-dimensional grids in one
// kernel: a workgroup per member carries the whole solve, or whole steps, with
// every transform in LDS and the kept modes owned by its threads.
//
// As separate passes a 1D solve is a chain of some fourteen (SA) or two or
// three per sweep (iteration) launches of a few microseconds each, nearly all
// latency: launch, parameters, a single row's transform on one or a dozen of
// the 256 CUs, store.  Here a pass costs its transforms and a few barriers, and
// is bound by the chain through them: one CU does all the work of a member, so
// the kernel serves rows of up to 1024 points, whose transforms lie in single
// wavefronts.  FP64, one member: 256 points iterated to 1e-9, 237 us a solve
// against 613 as separate passes; 1024 points, 371 against 598.
//
// The workgroup is G groups of P threads, one transform of n = nx / 2 complex
// points each (real rows by the half-length transform, as in the row passes).
// A pass is: inverse transforms of a list of spectra (owners write each into a
// group's LDS area, the group transforms it and stores the field); then forward
// transforms of a list of products src w^j, whose kept values the owners read
// from the areas and add, with their multipliers, to their mode's sums (the
// owners of a mode share a round's products over `lanes` threads); then the
// owners' update.  The main loop below runs such passes; what they transform
// and add depends on the phase.  Spectra live in the context's compact fields,
// each element read and written by its owner only, what the next pass transforms
// in the owners' registers; fields at the points in LDS where they all fit, else
// in the context's work fields, handed on at workgroup barriers.
#include <hip/hip_runtime.h>
#include <math.h>

#include "sbi_line.hpp"
#include "sbi_stage.hpp"

#ifndef SBI_REAL
#define SBI_REAL double
#endif

namespace sbi {

template <typename R, int NX> struct LineShape {
    using V = typename cplx_of<R>::type;
    static constexpr int N = NX / 2;
    static constexpr int E = FftShape<N>::E;
    static constexpr int P = N / E;
    // groups: the twelve products of a sweep at once, in whole wavefronts; eight at
    // 1024 points, where twelve would halve each thread's registers
    static constexpr int G = P >= 64 ? 8 : P >= 16 ? 12 : (P >= 4 ? 16 : 64 / P);
    static constexpr int T = G * P;
    static constexpr int AREA = fft_lds_elems<N, E>();
    static_assert(P <= 64, "a transform lies in one wavefront: its exchanges order that wavefront only");
    static_assert(T % 64 == 0 && G >= 5, "whole wavefronts, and a pass's inverse transforms at once");
    // fields in LDS where all of them fit beside the areas
    static constexpr size_t AREAS_BYTES = (size_t)G * AREA * sizeof(V);
    static constexpr size_t FIELD_BYTES = (size_t)LF_COUNT * NX * sizeof(R);
    static constexpr bool FLDS = AREAS_BYTES + FIELD_BYTES + 8192 <= kMaxLdsBytes;
    static constexpr size_t LDS = AREAS_BYTES + (FLDS ? FIELD_BYTES : 0);
};

enum LinePhase { LINE_LOAD, LINE_START, LINE_ORDER, LINE_SWEEP, LINE_NPHI, LINE_BLEND };

static __constant__ double kInvFact[8] = {1.0, 1.0, 1.0 / 2.0, 1.0 / 6.0, 1.0 / 24.0, 1.0 / 120.0, 1.0 / 720.0, 1.0 / 5040.0};

// What a phase does once and pointwise stays out of line: inlined, its constants
// would be held in registers across the whole loop.
template <typename R> __device__ __attribute__((noinline)) void line_rk(const LineParams* p, int stage, int om, long long co, double href) {
    rk_mode<R>(p->rk, stage, mode_geo(p->g, om), co, href);
}
static __device__ __attribute__((noinline)) void line_weights(Ctl* ctl, int n, const double* s_tot, double* s_w) {
    double tot[kAASlots], w[kAASlots];
#pragma unroll
    for (int i = 0; i < kAASlots; ++i) tot[i] = s_tot[i];
    aa_weights(ctl, &ctl->aa_gram[0][0], n, tot, w, true);
#pragma unroll
    for (int i = 0; i < kAASlots; ++i) s_w[i] = w[i];
}
// wavemaker pressure at point i
static __device__ __attribute__((noinline)) double line_pressure(const LineParams* p, const double* amp, int i) {
    const double lx = p->g.lx, x = i * (lx / p->g.nx);
    const double xs = x < 0.5 * lx ? x : x - lx;
    double pg = 0.0;
#pragma unroll 1
    for (int c = 0; c < p->wm_n; ++c) {
        const double kx = p->wm[c][1] * xs;
        pg += amp[c] * exp(-0.5 * kx * kx);
    }
    return pg;
}
// radiated amplitude of wavemaker component c at time ts
static __device__ __attribute__((noinline)) double line_amplitude(const LineParams* p, int c, double ts, double href) {
    const double hg = p->wm_h > 0.0 ? p->wm_h : href;
    const double kh2 = 2.0 * p->wm[c][1] * hg;
    const double gn = kh2 < 700.0 ? kh2 / sinh(kh2) : 0.0;
    return p->wm[c][0] * sqrt(M_E / (2.0 * M_PI)) * (1.0 + gn) * sin(p->wm[c][2] * ts + p->wm[c][3]);
}
// relaxation zones at point i: towards the target near x = 0, to rest near x = lx (pot: phi_s, else eta)
static __device__ __attribute__((noinline)) double line_blend(const LineParams* p, double f, int i, bool pot, double tm) {
    const double gen = p->rz[3], absl = p->rz[4], ramp = p->rz[5] * 2.0 * M_PI / p->rz[2];
    const double lx = p->g.lx, x = i * (lx / p->g.nx);
    if (x < gen) {
        const double r = tm < ramp ? 0.5 * (1.0 - cos(M_PI * tm / ramp)) : 1.0;
        const double amp = pot ? p->rz[0] * r / p->rz[2] : p->rz[0] * r;
        const double s = x / gen, w = 1.0 - (3 * s * s - 2 * s * s * s);
        const double th = p->rz[1] * x - p->rz[2] * tm;
        f = (1.0 - w) * f + w * (amp * (pot ? sin(th) : cos(th)));
    }
    if (x > lx - absl) {
        const double s = (lx - x) / absl;
        f *= 1.0 - (1.0 - (3 * s * s - 2 * s * s * s));
    }
    return f;
}
// damping weight of the tank at point i
static __device__ __attribute__((noinline)) double line_damping(const LineParams* p, int i) {
    const double lx = p->g.lx;
    const double d = fmod(i * (lx / p->g.nx) - p->dmp_x0 + 1.5 * lx, lx) - 0.5 * lx;
    return exp(-(d / p->dmp_w) * (d / p->dmp_w));
}
static __device__ __attribute__((noinline)) double line_omega(const LineParams* p, double emax, double emin) {
    // relaxation weight from the local symbol sum_{j<=L-1} (k eta)^j / j!
    const int L = p->g.order;
    if (!p->g.relax || L < 2) return 1.0;
    double lmax = 0.0, lmin = 0.0, tmax = 1.0, tmin = 1.0;
    const double xmax = p->g.kband * emax, xmin = p->g.kband * emin;
    for (int i = 0; i < L; ++i) {
        if (i > 0) {
            tmax *= xmax / i;
            tmin *= xmin / i;
        }
        lmax += tmax;
        lmin += tmin;
    }
    const double s = lmin + lmax;
    return isfinite(s) && s > 0.0 ? fmin(1.0, 2.0 / s) : 1.0;
}

template <typename R, int NX>
__global__ void __launch_bounds__((LineShape<R, NX>::T)) k_line(const LineParams pk, const typename cplx_of<R>::type* __restrict__ twN,
                                                              const typename cplx_of<R>::type* __restrict__ twX) {
    using LS = LineShape<R, NX>;
    using V = typename LS::V;
    constexpr int N = LS::N, E = LS::E, P = LS::P, G = LS::G, T = LS::T, AREA = LS::AREA;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    __shared__ double s_red[16 * kAASlots], s_tot[kAASlots], s_w[kAASlots], s_amp[kMaxWavemaker];
    // the parameters in LDS: as kernel arguments the loop would hold all of them
    // in scalar registers at once
    __shared__ LineParams p;
    for (int i = threadIdx.x; i < (int)(sizeof(LineParams) / 4); i += T)
        reinterpret_cast<int*>(&p)[i] = reinterpret_cast<const int*>(&pk)[i];
    __syncthreads();
    V* const areas = reinterpret_cast<V*>(smem_raw);
    const int t = threadIdx.x;
    const int grp = P == 64 ? __builtin_amdgcn_readfirstlane(t / P) : t / P;
    const int j = t % P;
    const int mem = blockIdx.x;
    const GridDev& g = pk.g;
    Ctl* const ctl = pk.ctl + mem;
    V* const area = areas + grp * AREA;
    Twid<V, N, E> twc;
    twc.load(twN, j);

    // owners: mode om, lane ol of `lanes`; the lead lane holds the mode's state
    const int KP = (g.Kx + 63) / 64 * 64, lanes = T / KP;
    const int om = t % KP, ol = t / KP;
    const bool own = om < g.Kx && ol < lanes, lead = own && ol == 0;
    const double href = g.href[mem];
    const double kd = 2.0 * M_PI * om / g.lx;
    const R kk = R(kd), kT = R(tanh(kd * href)), kS = R(sech_d(kd * href));
    const V tw1 = twX[own ? om : 0], tw2 = twX[own ? N - om : 0];
    const long long co = mem * g.s_cmp + om, ho = mem * g.s_half + om, po = mem * g.s_phys;
    const V zero = cx<V>(R(0), R(0));
    auto C = [&](void* f) __attribute__((always_inline)) -> V& { return static_cast<V*>(f)[co]; };
    // field id at the points, this member's
    R* const lds_fields = reinterpret_cast<R*>(areas + G * AREA);
    auto field = [&](int id) __attribute__((always_inline)) -> R* {
        if constexpr (LS::FLDS) return lds_fields + id * NX;
        else return static_cast<R*>(p.f[id]) + po;
    };
    auto pairs = [&](int id) __attribute__((always_inline)) { return reinterpret_cast<V*>(field(id)); };

    const int L = g.order;
    const bool sa = pk.sa, vd = pk.vd, step = pk.steps > 0, damp = pk.dmp_w > 0.0;
    if (t == 0 && p.acc_reset) {
        ctl->acc_solves = ctl->acc_sweeps = 0;
        ctl->acc_sweeps_max = ctl->acc_worst = 0;
        ctl->acc_residual_max = 0.0;
    }
    if (step && damp) {
        // damping weight of the tank at the points, once
#pragma unroll 1
        for (int i = t; i < NX; i += T) field(LF_MU)[i] = R(line_damping(&p, i));
    }
    if constexpr (LS::FLDS) {
        const R* const d = static_cast<const R*>(pk.f[LF_DELTA]) + po;
        const R* const e = step ? nullptr : static_cast<const R*>(pk.eta_in) + po;
#pragma unroll 1
        for (int i = t; i < NX; i += T) {
            field(LF_DELTA)[i] = d[i];
            if (e) field(LF_ETA)[i] = e[i];
        }
    }

    int phase = pk.load ? LINE_LOAD : LINE_START;
    int l = 2, n = 0, stage = 0, left = pk.steps;   // SA order formed; sweep; Runge-Kutta stage; steps to go
    double tm = pk.t0, omega = 1.0, rmin = INFINITY;
    // a lead owner's spectral values that the next pass transforms, in the order of its jobs
    V sv[5] = {zero, zero, zero, zero, zero};
    if (lead && !pk.load) {
        sv[0] = C(p.rk.es);
        sv[2] = C(p.rk.ps);
    }

    for (;;) {
        asm volatile("" : "+v"(phase));  // one body for every phase, not one per phase
        phase = __builtin_amdgcn_readfirstlane(phase);
        // ---- what the phase transforms: spectra and where they go, then products
        int ni = 0, nf = 0, J = 1;                  // J: products of a family
        V x = zero, y = zero;                       // the mode's sums (V and phi_b parts)
        const int nb = vd ? 1 : 0;
        switch (phase) {
            case LINE_LOAD: nf = step ? 2 : 1; break;
            case LINE_START:
                ni = (step ? 3 : 1) + (sa ? 1 + nb : 0);
                if (sa) nf = L > 1 ? 2 + nb : 0;    // order 2
                else nf = J = L - 1;
                if (t == 0) {
                    ctl->done = ctl->status = ctl->sweeps = ctl->nonfinite = ctl->sweeps_inner = 0;
                    ctl->omega = 1.0;
                    ctl->residual = 0.0;
                    ctl->rmin = INFINITY;
                }
                l = 2;
                n = 0;
                rmin = INFINITY;
                if (lead) {
                    // in sv: eta_hat (when stepping) and phi_hat; then eta, eta_x, phi_x and the
                    // linear guess, order 1 or the iteration's first iterate
                    const V e = sv[0], f = sv[2];
                    const V v1 = cscale(f, kT * kk), b1 = cscale(f, kS);
                    C(p.vn) = v1;
                    C(p.bn) = b1;
                    if (sa) C(p.vh) = v1;
                    sv[1] = mul_i(cscale(e, kk));
                    sv[2] = mul_i(cscale(f, kk));
                    sv[3] = v1;
                    sv[4] = mul_i(cscale(b1, kk));
                }
                break;
            case LINE_ORDER:
                J = l - 1;
                ni = 1 + nb;
                nf = J * (1 + nb) + 1;
                break;
            case LINE_SWEEP:
                J = L - 1;
                ni = 1 + nb + (n > 0 ? 2 : 0);
                nf = J * (1 + nb);
                break;
            case LINE_NPHI:
                ni = 1;
                nf = 1 + (damp ? 1 : 0);
                if (t < p.wm_n) s_amp[t] = line_amplitude(&p, t, tm + (stage == 0 ? 0.0 : (stage == 3 ? 1.0 : 0.5)) * p.rk.h, href);
                break;
            default:
                ni = nf = 2;
                break;
        }
        J = max(J, 1);
        // the first of START's values that are transformed (a solve is given eta)
        const int v0 = phase == LINE_START && !step ? 2 : 0;
        // field of job q of the inverse transforms (-1: none kept, the residual's two maxima)
        auto inv_field = [&](int q) __attribute__((always_inline)) -> int {
            if (phase == LINE_START) {
                const int u = q + v0;
                return u == 0 ? LF_ETA : (u == 1 ? LF_EX : (u == 2 ? LF_PX : (u == 3 ? LF_V0 : LF_B0)));
            }
            if (q > nb) return -1;
            return (q == 0 ? LF_V0 : LF_B0) + (phase == LINE_ORDER ? l - 2 : 0);  // the order l - 1
        };
        unsigned long long nu = 0ull, de = 0ull;
        V v[E];
        if (ni > 0) {
            if (lead) {
#pragma unroll
                for (int u = 0; u < 5; ++u) {
                    const int q = u - v0;
                    if (q < 0 || q >= ni) continue;
                    // Z[m] = (F[m] + conj F[n-m]) / 2 + i (F[m] - conj F[n-m]) / 2 e^(2 pi i m / nx);
                    // the kept band lies below n / 2, so F[m] alone gives Z[m] and Z[n-m]
                    V* const z = areas + q * AREA;
                    const V h = cscale(sv[u], R(0.5));
                    z[om] = cadd(h, mul_i(cmul(h, cconj(tw1))));
                    if (om > 0) {
                        const V hc = cconj(h);
                        const V w = mul_i(cmul(hc, cconj(tw2)));
                        z[N - om] = cx<V>(hc.x - w.x, hc.y - w.y);
                    }
                }
            }
            lds_sync();
#pragma unroll
            for (int q = 0; q < E; ++q) {
                const int i = j + q * P;
                v[q] = (i <= g.Mx || i >= N - g.Mx) ? area[i] : zero;
            }
            wave_lds_sync();
            fft<V, N, true, 1, 8, true>(v, area, 0, j, twc);
#pragma unroll
            for (int q = 0; q < E; ++q) v[q] = cscale(v[q], R(1.0 / N));
            const int job = grp;
            if (job < ni) {
                const int out = inv_field(job);
                if (phase == LINE_NPHI) {
                    // (V + eta_x phi_x)^2 / (2 (1 + eta_x^2)) - phi_x^2 / 2 - p_g
                    const V* ex = pairs(LF_EX);
                    const V* px = pairs(LF_PX);
#pragma unroll
                    for (int q = 0; q < E; ++q) {
                        const int i = j + q * P;
                        const V a = ex[i], b = px[i];
                        const R qx = v[q].x + a.x * b.x, qy = v[q].y + a.y * b.y;
                        V r = cx<V>(R(0.5) * (qx * qx / (R(1) + a.x * a.x) - b.x * b.x),
                                    R(0.5) * (qy * qy / (R(1) + a.y * a.y) - b.y * b.y));
                        if (p.wm_n > 0)
                            r = cx<V>(R((double)r.x - line_pressure(&p, s_amp, 2 * i)),
                                      R((double)r.y - line_pressure(&p, s_amp, 2 * i + 1)));
                        pairs(LF_NL)[i] = r;
                    }
                } else if (phase == LINE_BLEND) {
                    V* const o = pairs(job == 0 ? LF_NL : LF_V0);
#pragma unroll
                    for (int q = 0; q < E; ++q) {
                        const int i = j + q * P;
                        o[i] = cx<V>(R(line_blend(&p, (double)v[q].x, 2 * i, job == 1, tm)),
                                     R(line_blend(&p, (double)v[q].y, 2 * i + 1, job == 1, tm)));
                    }
                } else if (out >= 0) {
                    V* const o = pairs(out);
#pragma unroll
                    for (int q = 0; q < E; ++q) o[j + q * P] = v[q];
                } else {
#pragma unroll
                    for (int q = 0; q < E; ++q) {
                        const unsigned long long a = abs_bits((double)v[q].x), b = abs_bits((double)v[q].y);
                        unsigned long long& r = job == nb + 1 ? nu : de;
                        r = a > r ? a : r;
                        r = b > r ? b : r;
                    }
                }
            }
            __syncthreads();  // the areas are free, the fields visible to every group
        }
        if (phase == LINE_START) {
            // extrema of eta (relaxation weight), non-finite inputs
            unsigned long long mx = 0ull, mn = ~0ull;
            int bad = 0;
            const R* e = field(LF_ETA);
            const R* f = field(LF_PX);
#pragma unroll 1
            for (int i = t; i < NX; i += T) {
                const double a = (double)e[i];
                bad |= !isfinite(a) || !isfinite((double)f[i]);
                const unsigned long long b = ord_bits(a);
                mx = b > mx ? b : mx;
                mn = b < mn ? b : mn;
            }
            if (bad) atomicOr(&ctl->nonfinite, 1);
            if (!sa) {
                const double emax = unord_bits(block_reduce_u64<true>(mx)), emin = unord_bits(block_reduce_u64<false>(mn));
                omega = line_omega(&p, emax, emin);
                if (t == 0) ctl->omega = omega;
            }
        } else if (phase == LINE_SWEEP && n > 0) {
            // the decision on sweep n - 1 (the rules of the sweep passes)
            block_reduce2_max_u64(nu, de);
            const double num = bits_to_double(nu), den = bits_to_double(de);
            double r = 0.0;
            int dec = 0;
            if (!isfinite(num) || !isfinite(den)) {
                r = __longlong_as_double(0x7ff8000000000000ll);
                dec = 100 - 5;
            } else {
                r = num == 0.0 ? 0.0 : (den > 0.0 ? num / den : INFINITY);
                if (r <= p.tol) {
                    dec = 100;
                } else {
                    rmin = fmin(rmin, r);
                    if (r > 1e6 || (n - 1 >= 3 && r > 10.0 * rmin)) dec = 100 - 6;
                    else if (n >= p.max_sweeps) dec = 100 + 1;
                }
            }
            dec = __builtin_amdgcn_readfirstlane(dec);
            if (dec) {
                if (t == 0) ctl_commit(ctl, dec - 100, n, r);
                if (!step || (dec < 100 && !p.keep)) {
                    if (lead && !step) {
                        static_cast<V*>(p.gv)[ho] = C(p.vn);
                        static_cast<V*>(p.gd)[ho] = C(p.np);
                        static_cast<V*>(p.gt)[ho] = C(p.vh);
                    }
                    return;  // the whole workgroup: the decision is uniform
                }
                phase = LINE_NPHI;
                if (lead) sv[0] = C(p.vh);
                continue;
            }
        }

        // ---- forward transforms of the products
#pragma unroll 1
        for (int q0 = 0; q0 < nf; q0 += G) {
            const int job = q0 + grp;
            // products of an order or a sweep: eta^j V, (delta^j phi_b,x,) j = 1 .. J, then the forcing
            // eta^(l-1) phi_x of an order; of the iteration's start: the forcing of every order
            const bool forcing = phase == LINE_START ? (!sa || job == 1 + nb) : (phase == LINE_ORDER && job == J * (1 + nb));
            const int fam = forcing ? 0 : job / J, jj = forcing ? (sa ? l - 1 : job + 1) : job % J + 1;
            int src, w = LF_ETA, pw = jj;
            if (phase == LINE_NPHI) {
                src = job == 0 ? LF_NL : LF_PX;
                w = LF_MU;
                pw = job;
            } else if (phase == LINE_BLEND) {
                src = job == 0 ? LF_NL : LF_V0;
                pw = 0;
            } else {
                const int slot = sa ? min(max(l - jj - 1, 0), 5) : 0;   // V_(l-j)
                src = forcing ? LF_PX : (fam == 0 ? LF_V0 : LF_B0) + slot;
                w = forcing || fam == 0 ? LF_ETA : LF_DELTA;
            }
            if (job < nf && phase == LINE_LOAD) {
                const V* s = reinterpret_cast<const V*>(static_cast<const R*>(step && job == 0 ? p.eta_in : p.phi_in) + po);
#pragma unroll
                for (int q = 0; q < E; ++q) v[q] = s[j + q * P];
            } else if (job < nf) {
                const V* s = pairs(src);
#pragma unroll
                for (int q = 0; q < E; ++q) v[q] = s[j + q * P];
                if (pw > 0) {
                    V wv[E];
                    const V* ws = pairs(w);
#pragma unroll
                    for (int q = 0; q < E; ++q) wv[q] = ws[j + q * P];
#pragma unroll 1
                    for (int e = 0; e < pw; ++e)
#pragma unroll
                        for (int q = 0; q < E; ++q) v[q] = cx<V>(v[q].x * wv[q].x, v[q].y * wv[q].y);
                }
            } else {
#pragma unroll
                for (int q = 0; q < E; ++q) v[q] = zero;
            }
            fft<V, N, false, 1, 8, true>(v, area, 0, j, twc);
            wave_lds_sync();
#pragma unroll
            for (int q = 0; q < E; ++q) area[j + q * P] = v[q];
            lds_sync();
            if (own) {
#pragma unroll 1
                for (int q = ol; q < min(G, nf - q0); q += lanes) {
                    const int jb = q0 + q;
                    const V zm = areas[q * AREA + om], zc = cconj(areas[q * AREA + ((N - om) & (N - 1))]);
                    const V ev = cx<V>(R(0.5) * (zm.x + zc.x), R(0.5) * (zm.y + zc.y));
                    const V od = mul_mi<false>(cx<V>(R(0.5) * (zm.x - zc.x), R(0.5) * (zm.y - zc.y)));
                    V F = cadd(ev, cmul(tw1, od));
                    // coef fn(k) k^pw F added to the V part (the phi_b part)
                    auto add = [&](bool b, double coef, int fn, int kpw) __attribute__((always_inline)) {
                        R f = R(coef);
                        if (fn == FN_T) f *= kT;
                        else if (fn == FN_S) f *= kS;
                        if (kpw >= 0) {
                            for (int e = 0; e < kpw; ++e) f *= kk;
                        } else {
                            f = kk > R(0) ? f / kk : R(0);
                        }
                        if (b) y = cx<V>(y.x + F.x * f, y.y + F.y * f);
                        else x = cx<V>(x.x + F.x * f, x.y + F.y * f);
                    };
                    if (phase == LINE_LOAD || phase == LINE_BLEND) {
                        if (jb == 0) x = F;
                        else y = F;
                        continue;
                    }
                    if (phase == LINE_NPHI) {
                        if (jb == 0) x = F;
                        else y = mul_i(cscale(F, kk));
                        continue;
                    }
                    const bool fo = phase == LINE_START ? (!sa || jb == 1 + nb) : (phase == LINE_ORDER && jb == J * (1 + nb));
                    const int pj = fo ? (sa ? l - 1 : jb + 1) : jb % J + 1;
                    const bool want_b = vd && (!sa || l < L);
                    const double f = kInvFact[pj];
                    const bool odd = pj & 1;
                    if (fo) {
                        F = mul_i(cscale(F, kk));
                        add(false, -f, odd ? FN_ONE : FN_T, pj - 1);
                        if (want_b && !odd) add(true, -f, FN_S, pj - 2);
                    } else if (jb < J) {
                        add(false, -f, odd ? FN_T : FN_ONE, pj);
                        if (want_b && odd) add(true, -f, FN_S, pj - 1);
                    } else {
                        F = mul_i(cscale(F, kk));
                        if (odd) add(false, f, FN_S, pj - 1);
                        if (want_b) add(true, odd ? -f : f, odd ? FN_T : FN_ONE, pj - 2);
                    }
                }
            }
            lds_sync();  // the areas are free
        }

        // ---- the owners' update
        // the sums, folded over the lanes
        if (lanes > 1) {
            if (phase == LINE_LOAD || phase == LINE_NPHI || phase == LINE_BLEND) {
                // one product each: lane 0 holds the first, lane 1 the second
                if (own && ol == 1) areas[om] = y;
                lds_sync();
                if (lead && nf > 1) y = areas[om];
            } else {
                if (own && ol > 0) {
                    areas[(2 * ol - 2) * KP + om] = x;
                    areas[(2 * ol - 1) * KP + om] = y;
                }
                lds_sync();
                if (lead)
                    for (int l = 1; l < lanes; ++l) {
                        x = cadd(x, areas[(2 * l - 2) * KP + om]);
                        y = cadd(y, areas[(2 * l - 1) * KP + om]);
                    }
            }
            lds_sync();
        }
        if (phase == LINE_LOAD) {
            if (lead) {
                if (step) {
                    C(p.rk.eh) = x;
                    C(p.rk.es) = x;
                    C(p.rk.ph) = y;
                    C(p.rk.ps) = y;
                    sv[0] = x;
                    sv[2] = y;
                } else {
                    C(p.rk.ps) = x;
                    sv[2] = x;
                }
            }
            phase = LINE_START;
        } else if (phase == LINE_START && !sa) {
            if (lead) {
                const V s = C(p.rk.ps);
                C(p.bv) = cadd(cscale(s, kT * kk), x);
                C(p.bb) = cadd(cscale(s, kS), y);
                sv[0] = C(p.vn);
                sv[1] = mul_i(cscale(C(p.bn), kk));
            }
            phase = LINE_SWEEP;
        } else if (phase == LINE_START || phase == LINE_ORDER) {
            // order l is complete
            if (lead && L > 1) {
                C(p.vh) = cadd(C(p.vh), x);
                sv[0] = x;
                sv[1] = mul_i(cscale(y, kk));
            }
            if (++l <= L) {
                phase = LINE_ORDER;
            } else {
                if (!step) {
                    if (lead) static_cast<V*>(p.gv)[ho] = C(p.vh);
                    return;
                }
                phase = LINE_NPHI;
                if (lead) sv[0] = C(p.vh);
            }
        } else if (phase == LINE_SWEEP) {
            const int s = n % kAASlots, k = n < kAADepth ? n : kAADepth;
            double d[kAASlots];
#pragma unroll
            for (int i = 0; i < kAASlots; ++i) d[i] = 0.0;
            if (lead) {
                const V xv = C(p.vn), xb = C(p.bn);
                const V tv = cadd(C(p.bv), x), tb = cadd(C(p.bb), y);
                const V fv = csub(tv, xv), fb = csub(tb, xb);
                const V gv = cadd(xv, cscale(fv, R(omega))), gb = cadd(xb, cscale(fb, R(omega)));
                C(p.vh) = tv;
                C(p.np) = fv;
                // next pass: the iterate, then the residual's f_n and T(x_n)
                if (vd) {
                    sv[2] = fv;
                    sv[3] = tv;
                } else {
                    sv[1] = fv;
                    sv[2] = tv;
                }
                if (!p.aa) {
                    C(p.vn) = gv;
                    C(p.bn) = gb;
                    sv[0] = gv;
                    if (vd) sv[1] = mul_i(cscale(gb, kk));
                } else {
                    C(p.ring[0][s]) = fv;
                    C(p.ring[1][s]) = fb;
                    C(p.ring[2][s]) = gv;
                    C(p.ring[3][s]) = gb;
                    const double wt = om == 0 ? 1.0 : 2.0;
                    for (int a = 0; a <= k; ++a) {
                        const int si = (n - a) % kAASlots;
                        const V qv = C(p.ring[0][si]);
                        double e = (double)qv.x * (double)fv.x + (double)qv.y * (double)fv.y;
                        if (vd) {
                            const V qb = C(p.ring[1][si]);
                            e += (double)qb.x * (double)fb.x + (double)qb.y * (double)fb.y;
                        }
#pragma unroll
                        for (int i = 0; i < kAASlots; ++i)
                            if (i == si) d[i] = wt * e;
                    }
                }
            }
            if (p.aa) {
                col_aa_reduce(d, s_red, s_tot);
                lds_sync();
                if (t == 0) line_weights(ctl, n, s_tot, s_w);
                lds_sync();
                if (lead) {
                    V nv = zero, nbv = zero;
                    for (int a = 0; a <= k; ++a) {
                        const int si = (n - a) % kAASlots;
                        const R w = R(s_w[si]);
                        nv = cadd(nv, cscale(C(p.ring[2][si]), w));
                        nbv = cadd(nbv, cscale(C(p.ring[3][si]), w));
                    }
                    C(p.vn) = nv;
                    C(p.bn) = nbv;
                    sv[0] = nv;
                    if (vd) sv[1] = mul_i(cscale(nbv, kk));
                }
            }
            ++n;
        } else if (phase == LINE_NPHI) {
            if (lead) {
                C(p.np) = x;
                if (damp) C(p.pd) = y;
                line_rk<R>(&p, stage, om, co, href);
                sv[0] = C(p.rk.es);
                sv[2] = C(p.rk.ps);
            }
            phase = LINE_START;
            if (++stage == 4) {
                stage = 0;
                tm += p.rk.h;
                --left;
                if (p.rz_on) {
                    phase = LINE_BLEND;
                    sv[1] = sv[2];
                } else if (left == 0) {
                    return;
                }
            }
        } else {
            if (lead) {
                C(p.rk.eh) = x;
                C(p.rk.es) = x;
                C(p.rk.ph) = y;
                C(p.rk.ps) = y;
                sv[0] = x;
                sv[2] = y;
            }
            if (left == 0) return;
            phase = LINE_START;
        }
    }
}

using Real = SBI_REAL;

template <int NX> static hipError_t line_go(const LineParams& p, int batch, const Twiddles& tw, hipStream_t s) {
    using LS = LineShape<Real, NX>;
    using V = typename LS::V;
    // every kept mode has an owner, and a kept band below half the transform
    if (p.g.ny != 1 || (p.g.Kx + 63) / 64 * 64 > LS::T || 2 * p.g.Mx >= LS::N || p.g.order < 1 || p.g.order > 7)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_line<Real, NX>), dim3(batch), dim3(LS::T), LS::LDS, s, p,
                       (const V*)tw.tn, (const V*)tw.tx);
    return hipGetLastError();
}

template <> hipError_t launch_line_t<Real>(const LineParams& p, int batch, const Twiddles& tw, hipStream_t s) {
    switch (p.g.nx) {
        case 16: return line_go<16>(p, batch, tw, s);
        case 32: return line_go<32>(p, batch, tw, s);
        case 64: return line_go<64>(p, batch, tw, s);
        case 128: return line_go<128>(p, batch, tw, s);
        case 256: return line_go<256>(p, batch, tw, s);
        case 512: return line_go<512>(p, batch, tw, s);
        case 1024: return line_go<1024>(p, batch, tw, s);
        default: return hipErrorInvalidValue;
    }
}

template <int NX> static constexpr int line_t() { return LineShape<Real, NX>::T; }
#ifdef SBI_LINE_MAIN
int line_threads(int nx) {
    switch (nx) {
        case 16: return line_t<16>();
        case 32: return line_t<32>();
        case 64: return line_t<64>();
        case 128: return line_t<128>();
        case 256: return line_t<256>();
        case 512: return line_t<512>();
        case 1024: return line_t<1024>();
        default: return 0;
    }
}
hipError_t launch_line(int fp64, const LineParams& p, int batch, const Twiddles& tw, hipStream_t s) {
    return fp64 ? launch_line_t<double>(p, batch, tw, s) : launch_line_t<float>(p, batch, tw, s);
}
#endif

}  // namespace sbi
