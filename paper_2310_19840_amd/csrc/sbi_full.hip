// sbi_full.hip -- the fully nonlinear W solve of one-dimensional grids: the
// boundary-integral equations of Sec. 2.3 with the remaining integrals I^(S)
// of App. A kept (Eq. con-V: V = sum_j V^(j) + I^(S), whose sum is the exact
// equation) and, over a variable bed, the bed's remainder I^(B) of App. B.
//
// Two-dimensional flow (one horizontal dimension): Green function -ln r with
// the image of the source in the bed z = -h, jump coefficient pi; for the
// periodic surface z = x + i eta(x), 0 <= x < L,
//
//   S[V] = pi phi_s + D[phi_s],
//   S[V](x_i) = int V(x') G dx',  D[f](x_i) = int f(x') dG/dn' sqrt(1 + eta_x'^2) dx',
//   G = -ln|2 sin(pi (z - z') / L)| - ln|2 sin(pi (z - conj(z') + 2 i h) / L)|.
//
// The solve iterates V_(n+1) = S0^-1 [pi phi_s + D[phi_s] - (S - S0)[V_n]]
// from V_0 = 0, where S0 is S on the undisturbed surface (Fourier multiplier
// (pi / |k|) (1 + exp(-2 |k| h))).  The kernels of S - S0 and D are smooth and
// periodic, so the trapezoidal rule over the grid is spectrally accurate;
// S0^-1 and the derivatives eta_x, eta_xx are circulant matrices on the grid
// (their discrete Fourier multipliers), applied by direct summation.  The work
// is O(n^2) per application: every kernel evaluates point pairs, split over
// workgroups along both the evaluation and the source points.  Deep water
// (k_1 h > 18, k_1 = 2 pi / L) drops the image terms.
//
// Over a variable bed z = b(x) = -h + delta(x) the image no longer applies; the
// bed is a boundary of its own with the potential phi_b on it (dphi/dn = 0):
//
//   S[V] = pi phi_s + D_SS[phi_s] + D_SB[phi_b]       at the surface points,
//   pi phi_b = S_BS[V] - D_BS[phi_s] - D_BB[phi_b]     at the bed points,
//
// (S, D without image; D_XY the double layer of boundary Y seen from the
// points of X, outward normals (-eta_x, 1) and (b_x, -1) times ds/dx).  A
// sweep updates phi_b from the bed equation with V_n, then
// V_(n+1) = S0^-1 [pi phi_s + D_SS[phi_s] + D_SB[phi_b] - (S - S_flat)[V_n]]
//           + S0^-1 (S0 - S_flat)[V_n],
// S0 the image form's flat operator, S_flat = pi / |k| that of the flat surface
// alone.  A bed too deep to matter (k_1 times the smallest depth beyond 18)
// keeps the image form, which then drops the image.
//
// One object per precision (SBI_REAL): fields and the pair arithmetic run in
// that type; the tables of the heights and of the flat geometry and the distances
// formed from them, the circulant tables, the slices of the pair sums and every
// accumulation are FP64 (the direct sums over n points would otherwise lose
// about log10(sqrt(n)) digits in FP32).
#include <hip/hip_runtime.h>
#include <math.h>

#include "sbi_device.hpp"
#include "sbi_full.hpp"
#include "sbi_kernels.hpp"

#ifndef SBI_REAL
#define SBI_REAL double
#endif

namespace sbi {

using Real = SBI_REAL;

constexpr int kFullThreads = 256;       // evaluation points per workgroup
constexpr double kDeepK1H = 18.0;       // exp(-2 k_1 h) < 1e-15 beyond this

__device__ __forceinline__ bool full_deep(const FullParams& p, int m) {
    return (2.0 * M_PI / p.lx) * p.href[m] > kDeepK1H;
}

__device__ __forceinline__ bool full_bed(const FullParams& p, int m) { return p.bed && p.bed[m]; }
// scaled distance of the flat geometry: surface to image 2 pi h / L, surface to bed pi h / L
__device__ __forceinline__ double full_flat(const FullParams& p, int m) {
    return (full_bed(p, m) ? 1.0 : 2.0) * M_PI * p.href[m] / p.lx;
}

// --- tables: S0^-1 (per member: its depth), eta_x and eta_xx circulants,
// sin^2(pi j / n), and the circulant cm of S0^-1 (S0 - S_flat) (multiplier
// exp(-2|k|h) / (1 + exp(-2|k|h))).  c[j] = (1/n) sum_m s(k_m) cos(2 pi m j / n) with
// s = |k| / (pi (1 + exp(-2 |k| h))), k_m the m-th discrete wavenumber (the
// Nyquist mode included); d1[j] = (1/n) sum_(0<m<n/2) (-2 k_m) sin(2 pi m j / n)
// (the Nyquist mode drops out of a first derivative of a real field);
// d2[j] = (1/n) sum_m (-k_m^2) cos(2 pi m j / n).
template <typename R>
__global__ void __launch_bounds__(kFullThreads) k_full_tables(const FullParams p) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int m = blockIdx.y;
    const int n = p.n;
    if (j >= n) return;
    const double dk = 2.0 * M_PI / p.lx;
    const bool deep = full_deep(p, m);
    const double h = p.href[m];
    double c = 0.0, cm = 0.0, d1 = 0.0, d2 = 0.0;
    for (int q = 1; q < n; ++q) {
        const int qq = q <= n / 2 ? q : n - q;
        const double k = dk * qq;
        // angle 2 pi q j / n reduced exactly in integers
        const long long r = ((long long)q * j) % n;
        const double cs = cospi(2.0 * (double)r / n);
        const double e2 = deep ? 0.0 : exp(-2.0 * k * h);
        const double s = k / (M_PI * (1.0 + e2));
        c += s * cs;
        cm += e2 / (1.0 + e2) * cs;  // S0^-1 (S0 - S_flat): exp(-2|k|h) / (1 + exp(-2|k|h))
        if (m == 0) {
            d2 -= k * k * cs;
            if (q < n / 2) d1 -= 2.0 * k * sinpi(2.0 * (double)r / n);
        }
    }
    static_cast<double*>(p.c0)[(long long)m * n + j] = c / n;
    if (p.cm) static_cast<double*>(p.cm)[(long long)m * n + j] = cm / n;
    {
        // the flat geometry a pair kernel's logarithm is taken against: between
        // the surface and its image, or (two-boundary members) surface and bed;
        // 1/2 ln(sin^2(pi j / n) + sinh^2) and 1 / (sin^2 + sinh^2)
        const double sn = sinpi((double)j / n), sh = deep && !full_bed(p, m) ? 0.0 : sinh(full_flat(p, m));
        const bool none = deep && !full_bed(p, m);
        static_cast<double*>(p.lfl)[(long long)m * n + j] = none ? 0.0 : 0.5 * log(sn * sn + sh * sh);
        static_cast<double*>(p.rfl)[(long long)m * n + j] = none ? 0.0 : 1.0 / (sn * sn + sh * sh);
    }
    if (m == 0) {
        static_cast<double*>(p.d1)[j] = d1 / n;
        static_cast<double*>(p.d2)[j] = d2 / n;
        const double sn = sinpi((double)j / n);
        static_cast<double*>(p.s2)[j] = sn * sn;
        static_cast<double*>(p.s2a)[j] = sinpi(2.0 * (double)j / n);
        static_cast<double*>(p.rs2)[j] = j == 0 ? 0.0 : 1.0 / (sn * sn);  // unused at j = 0 (the pair limit)
    }
}

// Circulant sums are split over kLanes lanes per output point (the lanes of
// an output take every kLanes-th source point, so the lanes of a wavefront
// read consecutive table and source entries) and folded by lane exchanges.
constexpr int kLanes = 16;
constexpr int kOutPerBlock = kFullThreads / kLanes;

__device__ __forceinline__ double lane_fold(double v) {
#pragma unroll
    for (int off = kLanes / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, kLanes);
    return v;
}

// --- b_x, b_xx of each member's bed (FP64 heights bz) at set-up
template <typename R>
__global__ void __launch_bounds__(kFullThreads) k_full_bedgeom(const FullParams p) {
    const int t = threadIdx.x;
    const int i = blockIdx.x * kOutPerBlock + t / kLanes;
    const int l = t % kLanes;
    const int m = blockIdx.z;
    const int n = p.n;
    const double* bz = static_cast<const double*>(p.bz) + (long long)m * n;
    const double* d1 = static_cast<const double*>(p.d1);
    const double* d2 = static_cast<const double*>(p.d2);
    double a1 = 0.0, a2 = 0.0;
    if (i < n)
        for (int j = l; j < n; j += kLanes) {
            const int d = (i - j + n) & (n - 1);
            a1 += d1[d] * bz[j];
            a2 += d2[d] * bz[j];
        }
    a1 = lane_fold(a1);
    a2 = lane_fold(a2);
    if (i < n && l == 0) {
        static_cast<double*>(p.bx)[(long long)m * n + i] = a1;
        static_cast<double*>(p.bxx)[(long long)m * n + i] = a2;
    }
}

// Decision of launch `sweep` from the residual of the previous one (the
// iteration mode's rules); every workgroup decides alike, the leader records.
__device__ __forceinline__ bool full_decided(const FullParams& p, Ctl* ctl, bool leader) {
    if (ctl->done) return true;
    double r, rmin;
    const int dec = sweep_decision(ctl, p.sweep, p.max_sweeps, p.tol, &r, &rmin);
    if (dec) {
        if (leader) ctl_commit(ctl, dec - 100, p.sweep, r);
        return true;
    }
    if (leader) {
        ctl->rmin = rmin;
        ctl->residual = r;
    }
    return false;
}

// --- pair sums over a slice of the source points, at the surface points.
// KIND 0: the double layer D[phi_s] (every member); KIND 1: the single layer
// (S - S0)[V_n] of the image-form members.  Partial sums go to
// part[split][member][point]; the consumer adds the slices in order.
// sinh of the small arguments of the pair kernels (scaled height differences
// pi (y_j - y_i) / L): below 1/8 by its Taylor series to the x^11 term, nested
// as x (1 + x^2/(2*3) (1 + x^2/(4*5) (...))), whose remainder is below 3e-21
// of the value there; beyond it by the library function.  A difference is
// passed as such (from exponentials of each point the sinh would lose its
// relative accuracy for nearby points).
template <typename R> __device__ __forceinline__ R sinh_series(R x) {
    if (fabs(x) >= R(0.125)) return sinh(x);
    const R x2 = x * x;
    R s = R(1) + x2 * R(1.0 / 110.0);
    s = R(1) + x2 * R(1.0 / 72.0) * s;
    s = R(1) + x2 * R(1.0 / 42.0) * s;
    s = R(1) + x2 * R(1.0 / 20.0) * s;
    s = R(1) + x2 * R(1.0 / 6.0) * s;
    return x * s;
}

// sinh and cosh of a small argument together: below 1/8 both by their Taylor
// series (cosh to the x^12 term, nested as 1 + x^2/(1*2) (1 + x^2/(3*4) (...)),
// remainder below 3e-24), beyond it the library sinh and cosh = sqrt(1 + sinh^2)
template <typename R> __device__ __forceinline__ R sinh_cosh_series(R x, R* ch) {
    if (fabs(x) >= R(0.125)) {
        const R sh = sinh(x);
        *ch = sqrt(R(1) + sh * sh);
        return sh;
    }
    const R x2 = x * x;
    R c = R(1) + x2 * R(1.0 / 132.0);
    c = R(1) + x2 * R(1.0 / 90.0) * c;
    c = R(1) + x2 * R(1.0 / 56.0) * c;
    c = R(1) + x2 * R(1.0 / 30.0) * c;
    c = R(1) + x2 * R(1.0 / 12.0) * c;
    *ch = R(1) + x2 * R(0.5) * c;
    return sinh_series(x);
}

// a / b for a positive, normal b: the reciprocal's two Newton steps and a
// correction of the quotient, without the scaling of the general division
__device__ __forceinline__ double pair_div(double a, double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = fma(fma(-b, r, 1.0), r, r);
    r = fma(fma(-b, r, 1.0), r, r);
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}
__device__ __forceinline__ float pair_div(float a, float b) { return a / b; }

// log(1 + x).  The pair kernels' arguments are the height differences' effect
// on a squared distance, small except for the nearest points: pair_small, as
// 2 atanh(s), s = x / (2 + x), by its series to s^21 (the next term is below
// 2e-18 of the value for |s| <= 0.177); the library function elsewhere.
__device__ __forceinline__ bool pair_is_small(double x) { return x > -0.3 && x < 0.42; }
__device__ __forceinline__ double pair_small(double x) {
    const double s = pair_div(x, 2.0 + x), z = s * s;
    double q = 1.0 / 21.0;
    q = fma(q, z, 1.0 / 19.0);
    q = fma(q, z, 1.0 / 17.0);
    q = fma(q, z, 1.0 / 15.0);
    q = fma(q, z, 1.0 / 13.0);
    q = fma(q, z, 1.0 / 11.0);
    q = fma(q, z, 1.0 / 9.0);
    q = fma(q, z, 1.0 / 7.0);
    q = fma(q, z, 1.0 / 5.0);
    q = fma(q, z, 1.0 / 3.0);
    return fma(2.0 * s * z, q, 2.0 * s);
}
__device__ __forceinline__ double pair_log1p(double x) { return pair_is_small(x) ? pair_small(x) : log1p(x); }
__device__ __forceinline__ float pair_small(float x) { return log1p(x); }
__device__ __forceinline__ float pair_log1p(float x) { return log1p(x); }

// A pair pass: kFullThreads evaluation points per workgroup, each served by
// kPairLanes threads over a part of every staged block of sources (one thread
// per point leaves one wavefront per SIMD, and its chains of dependent FP64
// operations then wait on themselves); the lanes' sums are added in order.
// Bound by the issue of FP64 operations, 60 to 75 a pair.  FP64, 4096 points,
// per pass: the bed pass 75 us, the surface pass 56, the double layer 52 (148,
// 174 and 114 with one thread per point, the library's logarithms, the general
// division and a sinh of each pair's height difference).
constexpr int kPairLanes = 4;
constexpr int kPairThreads = kFullThreads * kPairLanes;
// sum over the lanes of a point; red holds (kPairLanes - 1) * kFullThreads values
__device__ __forceinline__ double pair_fold(double acc, double* red, int lane, int il) {
    if (lane > 0) red[(lane - 1) * kFullThreads + il] = acc;
    __syncthreads();
    if (lane == 0)
#pragma unroll
        for (int l = 1; l < kPairLanes; ++l) acc += red[(l - 1) * kFullThreads + il];
    return acc;
}
// Source block j0 .. of a slice: lane's points [jl0, jl1) within the block
struct PairBlock {
    int jl0, jl1;
};
__device__ __forceinline__ PairBlock pair_block(int j0, int jend, int lane) {
    const int jn = min(kFullThreads, jend - j0);
    const int per = (jn + kPairLanes - 1) / kPairLanes;
    return {min(jn, lane * per), min(jn, (lane + 1) * per)};
}

// The sinh and cosh of the distance between two boundaries, pi (y - y') / L =
// a + b, come from per-point tables: sinh a cosh b + cosh a sinh b.  Between
// surface and bed, a is the surface's height above a level and b the bed's depth
// below it; the level is the surface's lowest point (the solve's set-up left it in
// the control header), so that a >= 0, b >= 0 wherever the bed lies below every
// trough, and the sums add terms of one sign: against z = 0 a surface far below it
// would lose exp(2 pi |eta| / L) in relative accuracy.  The tables and sums are FP64
// in both precisions and rounded once, as the difference of the heights would be.
__device__ __forceinline__ double full_lowest(const FullParams& p, int m) { return unord_bits(p.ctl[m].eta_min); }

// Between surface and image the level is the bed itself, halfway between them: a
// and b are pi / L times the two points' heights above it.
//
// Single layer of the image form, direct part and image minus flat image,
//     -1/2 ln(1 + x) - 1/2 ln((sin^2 + sinh^2(pi (eta_i + eta_j + 2 h) / L)) / (sin^2 + sinh^2(2 pi h / L))),
// as one logarithm of (1 + x)(1 + y), y from the difference of the squares.  For a
// surface far below z = 0 y tends to -1 and 1 + y would cancel: it is then the ratio
// itself.  sh: sinh of the image's distance, sh0 of the flat one, s2, rfl: the flat
// geometry's tables at the pair's index distance.
template <typename R>
__device__ __forceinline__ R pair_single(R x, double sh, double sh0, const double* s2, double rfl) {
    const double y = (sh - sh0) * (sh + sh0) * rfl;
    const R yr = R(y), z = x + yr + x * yr;
    if (y > -0.3 && z < R(0.42)) return R(-0.5) * pair_small(z);  // z >= y, as x >= 0
    return R(-0.5) * (y > -0.3 ? log1p(z) : log((R(1) + x) * R((*s2 + sh * sh) * rfl)));
}

template <typename R, int KIND>
__global__ void __launch_bounds__(kPairThreads) k_full_pairs(const FullParams p) {
    __shared__ R te[kFullThreads], tex[kFullThreads], tsrc[kFullThreads];
    __shared__ double tsj[kFullThreads], tcj[kFullThreads];
    __shared__ double red[(kPairLanes - 1) * kFullThreads];
    const int t = threadIdx.x;
    const int il = t % kFullThreads, lane = __builtin_amdgcn_readfirstlane(t / kFullThreads);
    const int i = blockIdx.x * kFullThreads + il;
    const int split = blockIdx.y;
    const int m = blockIdx.z;
    const int n = p.n;
    if (KIND == 1) {
        Ctl* ctl = p.ctl + m;
        const bool leader = blockIdx.x == 0 && blockIdx.y == 0 && t == 0;
        if (full_decided(p, ctl, leader)) return;  // workgroup-uniform
    }
    const long long mo = m * p.s_phys;
    const R* eta = static_cast<const R*>(p.eta) + mo;
    const R* ex = static_cast<const R*>(p.ex) + mo;
    if (KIND == 1 && full_bed(p, m)) return;  // the two-boundary surface pass serves it
    const R* src = static_cast<const R*>(KIND == 0 ? p.phi : p.vin) + mo;
    const double* s2 = static_cast<const double*>(p.s2);
    const double* rs2 = static_cast<const double*>(p.rs2);
    const double* s2at = static_cast<const double*>(p.s2a);
    const double* rfl = static_cast<const double*>(p.rfl) + (long long)m * n;
    const R pl = R(M_PI / p.lx);
    const bool img = !full_deep(p, m) && !full_bed(p, m);  // the image form keeps the bed's image
    const double pld = M_PI / p.lx, h = p.href[m];
    const double sh0 = img ? sinh(2.0 * pld * h) : 0.0;
    // this point's values
    const bool on = i < n;
    const R etai = on ? eta[i] : R(0);
    const R exi = on ? ex[i] : R(0);
    double sbi = 0.0, cbi = 1.0;
    if (img) {
        const double b = pld * ((double)etai + h);
        sbi = sinh(b);
        cbi = cosh(b);
    }
    double acc = 0.0;
    const int chunk = (n + gridDim.y - 1) / gridDim.y;
    const int jbeg = split * chunk, jend = min(n, jbeg + chunk);
    for (int j0 = jbeg; j0 < jend; j0 += kFullThreads) {
        __syncthreads();
        if (t < kFullThreads && j0 + t < jend) {
            te[t] = eta[j0 + t];
            tex[t] = ex[j0 + t];
            tsrc[t] = src[j0 + t];
            if (img) {
                const double a = pld * ((double)te[t] + h);
                tsj[t] = sinh(a);
                tcj[t] = cosh(a);
            }
        }
        __syncthreads();
        if (!on) continue;
        const PairBlock pb = pair_block(j0, jend, lane);
        for (int jj = pb.jl0; jj < pb.jl1; ++jj) {
            const int j = j0 + jj;
            const int d = (j - i + n) & (n - 1);
            R kv;
            if (KIND == 1) {
                // direct part -1/2 ln(1 + sinh^2 / sin^2) (its limit -1/2 ln(1 + eta_x^2) at j = i), and the image's
                const R shb = sinh_series(pl * (te[jj] - etai));
                const R x = j == i ? exi * exi : shb * shb * R(rs2[d]);
                kv = img ? pair_single(x, tsj[jj] * cbi + tcj[jj] * sbi, sh0, s2 + d, rfl[d]) : R(-0.5) * pair_log1p(x);
            } else {
                // Im[(pi/L) cot(a + i b) (1 + i eta_x,j)], a = pi (x_j - x_i)/L, b = pi (eta_j - eta_i)/L:
                // cot(a + i b) = (sin 2a - i sinh 2b) / (2 (sin^2 a + sinh^2 b))
                const R sa2 = R(s2[d]);  // sin^2 a
                const R s2a = R(s2at[d]);  // sin 2a
                R chb;
                const R shb = sinh_cosh_series(pl * (te[jj] - etai), &chb);
                // the curvature limit at j = i is added below
                kv = j == i ? R(0) : pair_div(R(-2) * shb * chb + s2a * tex[jj], sa2 + shb * shb);
                if (img) {
                    // the image partner: b' = pi (eta_i + eta_j + 2h) / L
                    const R shp = R(tsj[jj] * cbi + tcj[jj] * sbi), chp = R(tcj[jj] * cbi + tsj[jj] * sbi);
                    kv += pair_div(R(-2) * shp * chp + s2a * tex[jj], sa2 + shp * shp);
                }
                kv *= R(0.5) * pl;
            }
            acc += (double)kv * (double)tsrc[jj];
        }
    }
    acc = pair_fold(acc, red, lane, il);
    if (!on || lane > 0) return;
    const double dx = p.lx / n;
    double out = acc * dx;
    if (KIND == 0 && i >= jbeg && i < jend) {
        // the diagonal of the direct double layer: eta_xx / (2 (1 + eta_x^2))
        const double exx = (double)static_cast<const R*>(p.exx)[mo + i];
        out += dx * exx / (2.0 * (1.0 + (double)exi * (double)exi)) * (double)src[i];
    }
    static_cast<double*>(p.part)[((long long)split * p.batch + m) * n + i] = out;
}

// --- the single layer (S - S0)[V_n] of the image-form members from the
// symmetry of its kernel: K(i, j) = K(j, i) (both the direct part and the
// image depend on |eta_j - eta_i|, eta_i + eta_j and sin^2(pi (x_j - x_i)/L)).
// The n x n pairs split into blocks of Q kSymT x Q kSymT points; a workgroup
// takes block (I, J), I <= J, tile by tile of kSymT x kSymT, evaluates each of
// its pairs once and adds K V_j to the row sums of its points i in block I and
// K V_i to the column sums of its points j in block J.  Row sums go to slice J
// of the points of block I, column sums to slice I of those of block J, so every
// point receives n / (Q kSymT) slices, one from each block, each written once; a
// diagonal tile evaluates all its pairs and adds to the rows only, and the tiles
// below the diagonal of a diagonal block are left out.
//
// Bound by the issue of FP64 operations (about 50 a pair).  A tile's 64 columns
// are the lanes of a wavefront and its four wavefronts take a quarter of the
// tile's diagonals each: at 4096 points 2080 workgroups, eight to nine per CU
// (blocks of two tiles a side leave two or three, a third of the chip idle at the
// end: those are for where the slices of many members would fill memory instead).
// FP64, 4096 points: 41 us per pass, against 109 with tiles of 128 and two
// library logarithms a pair.
constexpr int kSymT = kFullSymTile;
constexpr int kSymWaves = 4;
static_assert(kSymT == 64, "a tile's columns are the lanes of one wavefront");

template <typename R, int Q>
__global__ void __launch_bounds__(64 * kSymWaves) k_full_sympairs(const FullParams p) {
    __shared__ R tej[kSymT], tvj[kSymT];
    __shared__ double tsj[kSymT], tcj[kSymT];
    __shared__ double colp[kSymWaves][kSymT], rowp[kSymWaves][kSymT];
    __shared__ double rsum[Q][kSymT], csum[Q][kSymT];
    const int t = threadIdx.x;
    const int m = blockIdx.z;
    const int n = p.n;
    const int nb = n / (Q * kSymT);
    {
        Ctl* ctl = p.ctl + m;
        const bool leader = blockIdx.x == 0 && t == 0;
        if (full_decided(p, ctl, leader)) return;  // workgroup-uniform
    }
    if (full_bed(p, m)) return;
    // block (I, J), I <= J, of this workgroup's linear index (row-major upper triangle)
    int L = blockIdx.x, I = 0;
    while (L >= nb - I) {
        L -= nb - I;
        ++I;
    }
    const int J = I + L;
    const bool diag = I == J;
    const long long mo = m * p.s_phys;
    const R* eta = static_cast<const R*>(p.eta) + mo;
    const R* ex = static_cast<const R*>(p.ex) + mo;
    const R* v = static_cast<const R*>(p.vin) + mo;
    const double* s2 = static_cast<const double*>(p.s2);
    const double* rs2 = static_cast<const double*>(p.rs2);
    const double* rfl = static_cast<const double*>(p.rfl) + (long long)m * n;
    const R pl = R(M_PI / p.lx);
    const bool img = !full_deep(p, m);
    const double pld = M_PI / p.lx, h = p.href[m];
    const double sh0 = img ? sinh(2.0 * pld * h) : 0.0;
    const int wv = t / 64, ln = t & 63;
    if (t < kSymT) {
#pragma unroll
        for (int q = 0; q < Q; ++q) rsum[q][t] = csum[q][t] = 0.0;
    }
#pragma unroll 1
    for (int q = 0; q < Q * Q; ++q) {
        const int qa = q / Q, qb = q % Q;
        const bool own = diag && qa == qb;
        if (diag && qa > qb) continue;
        if (Q > 1) __syncthreads();  // the tile before is done with the shared columns
        const int i = (I * Q + qa) * kSymT + ln;
        const R etai = eta[i], exi = ex[i];
        const double vi = (double)v[i];
        double sbi = 0.0, cbi = 1.0;
        if (img) {
            const double b = pld * ((double)etai + h);
            sbi = sinh(b);
            cbi = cosh(b);
        }
        if (t < kSymT) {
            const R ej = eta[(J * Q + qb) * kSymT + t];
            tej[t] = ej;
            tvj[t] = v[(J * Q + qb) * kSymT + t];
            if (img) {
                const double a = pld * ((double)ej + h);
                tsj[t] = sinh(a);
                tcj[t] = cosh(a);
            }
        }
        __syncthreads();
        const int from = (ln + 1) & 63;
        constexpr int kSteps = kSymT / kSymWaves;
        double acc = 0.0, cacc = 0.0;
#pragma unroll 2
        for (int s = 0; s < kSteps; ++s) {
            // lane ln takes the columns ln + kSteps wv, + 1, ... (mod 64): at each
            // step the lanes of a wavefront hold 64 different columns, and the
            // running column sum moves one lane down with its column
            const int jl = (ln + wv * kSteps + s) & 63;
            const int j = (J * Q + qb) * kSymT + jl;
            const int d = (j - i + n) & (n - 1);
            const R shb = sinh_series(pl * (tej[jl] - etai));
            const R x = j == i ? exi * exi : shb * shb * R(rs2[d]);
            const double kv = (double)(img ? pair_single(x, tsj[jl] * cbi + tcj[jl] * sbi, sh0, s2 + d, rfl[d])
                                           : R(-0.5) * pair_log1p(x));
            acc += kv * (double)tvj[jl];
            if (!own) {
                // the pair seen from j: K V_i added to column jl's sum over this
                // wavefront's rows, which lane ln - 1 continues at the next step
                cacc += kv * vi;
                cacc = __shfl(cacc, from, 64);
            }
        }
        rowp[wv][ln] = acc;
        if (!own) colp[wv][(ln + (wv + 1) * kSteps) & 63] = cacc;
        __syncthreads();
        if (t < kSymT) {  // thread t adds to its own points' sums only
#pragma unroll
            for (int w = 0; w < kSymWaves; ++w) rsum[qa][t] += rowp[w][t];
            if (!own) {
                double* c = diag ? rsum[qb] : csum[qb];
#pragma unroll
                for (int w = 0; w < kSymWaves; ++w) c[t] += colp[w][t];
            }
        }
    }
    if (t < kSymT) {
        const double dx = p.lx / n;
        double* part = static_cast<double*>(p.part);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            // rows of block I: slice J; columns of block J: slice I
            part[((long long)J * p.batch + m) * n + (I * Q + q) * kSymT + t] = rsum[q][t] * dx;
            if (!diag) part[((long long)I * p.batch + m) * n + (J * Q + q) * kSymT + t] = csum[q][t] * dx;
        }
    }
}

// --- the surface pass of the two-boundary members: (S - S_flat)[V_n] (no
// image; V_n absent at the first sweep) minus D_SB[phi_b] with the phi_b of
// this sweep, at the surface points over a slice of the source points
template <typename R>
__global__ void __launch_bounds__(kPairThreads) k_full_spairs(const FullParams p) {
    __shared__ R te[kFullThreads], tsrc[kFullThreads], tbx[kFullThreads];
    __shared__ double tpb[kFullThreads], tsj[kFullThreads], tcj[kFullThreads];
    __shared__ double red[(kPairLanes - 1) * kFullThreads];
    const int t = threadIdx.x;
    const int il = t % kFullThreads, lane = __builtin_amdgcn_readfirstlane(t / kFullThreads);
    const int i = blockIdx.x * kFullThreads + il;
    const int split = blockIdx.y;
    const int m = blockIdx.z;
    const int n = p.n;
    {
        Ctl* ctl = p.ctl + m;
        const bool leader = blockIdx.x == 0 && blockIdx.y == 0 && t == 0;
        if (full_decided(p, ctl, leader)) return;  // workgroup-uniform
    }
    if (!full_bed(p, m)) return;
    const long long mo = m * p.s_phys, mb = (long long)m * n;
    const R* eta = static_cast<const R*>(p.eta) + mo;
    const R* ex = static_cast<const R*>(p.ex) + mo;
    const bool hasv = p.vin != nullptr;
    const R* src = hasv ? static_cast<const R*>(p.vin) + mo : nullptr;
    const double* bz = static_cast<const double*>(p.bz) + mb;
    const double* bxs = static_cast<const double*>(p.bx) + mb;
    const double* pbs = static_cast<const double*>(p.pbout) + mb;
    const double* s2 = static_cast<const double*>(p.s2);
    const double* rs2 = static_cast<const double*>(p.rs2);
    const double* s2at = static_cast<const double*>(p.s2a);
    const R pl = R(M_PI / p.lx);
    const double pld = M_PI / p.lx;
    const bool on = i < n;
    const R etai = on ? eta[i] : R(0);
    const R exi = on ? ex[i] : R(0);
    const double low = full_lowest(p, m), hi = pld * ((double)etai - low);  // the surface point above the level
    const double sei = sinh(hi), cei = cosh(hi);
    double accb = 0.0, accs = 0.0;
    const int chunk = (n + gridDim.y - 1) / gridDim.y;
    const int jbeg = split * chunk, jend = min(n, jbeg + chunk);
    for (int j0 = jbeg; j0 < jend; j0 += kFullThreads) {
        __syncthreads();
        const int jl = j0 + t;
        if (t < kFullThreads && jl < jend) {
            te[t] = eta[jl];
            tsrc[t] = hasv ? src[jl] : R(0);
            const double b = pld * (low - bz[jl]);  // the bed's depth below the level
            tsj[t] = sinh(b);
            tcj[t] = cosh(b);
            tbx[t] = R(bxs[jl]);
            tpb[t] = pbs[jl];
        }
        __syncthreads();
        if (!on) continue;
        const PairBlock pb = pair_block(j0, jend, lane);
#pragma unroll 2
        for (int jj = pb.jl0; jj < pb.jl1; ++jj) {
            const int j = j0 + jj;
            const int d = (j - i + n) & (n - 1);
            const R sa2 = R(s2[d]);
            const R s2a = R(s2at[d]);
            // the bed source (x_j, b_j): -D_SB = Im[(pi/L) cot(a + i b) (1 + i b_x,j)],
            // b = pi (b_j - eta_i) / L (the bed lies below every surface point): -b from the tables
            const R sh = R(tsj[jj] * cei + tcj[jj] * sei), ch = R(tcj[jj] * cei + tsj[jj] * sei);
            accb += (double)pair_div(R(2) * sh * ch + s2a * tbx[jj], sa2 + sh * sh) * tpb[jj];
            if (hasv) {
                // the direct single layer minus the flat one, as in the image form
                const R shb = sinh_series(pl * (te[jj] - etai));
                accs += (double)pair_log1p(j == i ? exi * exi : shb * shb * R(rs2[d])) * (double)tsrc[jj];
            }
        }
    }
    const double acc = pair_fold(0.5 * (double)pl * accb - 0.5 * accs, red, lane, il);
    if (!on || lane > 0) return;
    static_cast<double*>(p.part)[((long long)split * p.batch + m) * n + i] = acc * (p.lx / n);
}

// --- pair sums at the bed points of two-boundary members, over a slice of
// the source points.  KIND 2: D_BS[phi_s] (surface sources); KIND 3:
// S_BS[V_n] - D_BB[phi_b] (surface and bed sources, phi_b of this sweep),
// which also decides the sweep.  With a = pi (x_j - x_i) / L and b the scaled
// height difference pi (y_j - y_i) / L of source and evaluation point:
// G = -1/2 ln(4 (sin^2 a + sinh^2 b)), taken against the flat geometry's table
// where the distances are alike;
// the double layer of a surface source is Im[(pi/L) cot(a + i b) (1 + i eta_x,j)],
// that of a bed source -Im[(pi/L) cot(a + i b) (1 + i b_x,j)], with the curvature
// limit -b_xx / (2 (1 + b_x^2)) at coincident bed points.
template <typename R, int KIND>
__global__ void __launch_bounds__(kPairThreads) k_full_bpairs(const FullParams p) {
    __shared__ R tex[kFullThreads], tsrc[kFullThreads];
    __shared__ double tsj[kFullThreads], tcj[kFullThreads];
    __shared__ double tbz[kFullThreads], tbx[kFullThreads], tpb[kFullThreads];
    __shared__ double red[(kPairLanes - 1) * kFullThreads];
    const int t = threadIdx.x;
    const int il = t % kFullThreads, lane = __builtin_amdgcn_readfirstlane(t / kFullThreads);
    const int i = blockIdx.x * kFullThreads + il;
    const int split = blockIdx.y;
    const int m = blockIdx.z;
    const int n = p.n;
    if (KIND == 3) {
        Ctl* ctl = p.ctl + m;
        const bool leader = blockIdx.x == 0 && blockIdx.y == 0 && t == 0;
        if (full_decided(p, ctl, leader)) return;  // workgroup-uniform
    }
    if (!full_bed(p, m)) return;
    const long long mo = m * p.s_phys, mb = (long long)m * n;
    const R* eta = static_cast<const R*>(p.eta) + mo;
    const R* ex = static_cast<const R*>(p.ex) + mo;
    const R* src = static_cast<const R*>(KIND == 2 ? p.phi : p.vin) + mo;
    const double* bz = static_cast<const double*>(p.bz) + mb;
    const double* bxs = static_cast<const double*>(p.bx) + mb;
    const double* pbs = KIND == 3 ? static_cast<const double*>(p.pbin) + mb : nullptr;
    const double* s2 = static_cast<const double*>(p.s2);
    const double* s2at = static_cast<const double*>(p.s2a);
    const double* lfl = static_cast<const double*>(p.lfl) + mb;
    const double* rfl = static_cast<const double*>(p.rfl) + mb;
    const R pl = R(M_PI / p.lx);
    const double pld = M_PI / p.lx;
    const double sh0 = sinh(full_flat(p, m));
    const bool on = i < n;
    const double bzi = on ? bz[i] : 0.0;
    const double low = full_lowest(p, m), bi = pld * (low - bzi);  // the bed point's depth below the level
    const double sbi = sinh(bi), cbi = cosh(bi);
    double acc = 0.0, accb = 0.0;
    const int chunk = (n + gridDim.y - 1) / gridDim.y;
    const int jbeg = split * chunk, jend = min(n, jbeg + chunk);
    for (int j0 = jbeg; j0 < jend; j0 += kFullThreads) {
        __syncthreads();
        const int jl = j0 + t;
        if (t < kFullThreads && jl < jend) {
            const double e = pld * ((double)eta[jl] - low);  // the surface above the level
            tsj[t] = sinh(e);
            tcj[t] = cosh(e);
            tex[t] = ex[jl];
            tsrc[t] = src[jl];
            if (KIND == 3) {
                tbz[t] = bz[jl];
                tbx[t] = bxs[jl];
                tpb[t] = pbs[jl];
            }
        }
        __syncthreads();
        if (!on) continue;
        const PairBlock pb = pair_block(j0, jend, lane);
#pragma unroll 2
        for (int jj = pb.jl0; jj < pb.jl1; ++jj) {
            const int j = j0 + jj;
            const int d = (j - i + n) & (n - 1);
            const R s2a = R(s2at[d]);
            const R sa2 = R(s2[d]);
            // the surface source (x_j, eta_j) seen from the bed point (x_i, b_i)
            const double shd = tsj[jj] * cbi + tcj[jj] * sbi;
            const R sh = R(shd);
            if (KIND == 2) {
                const R ch = R(tcj[jj] * cbi + tsj[jj] * sbi);
                acc += (double)pair_div(R(-2) * sh * ch + s2a * tex[jj], sa2 + sh * sh) * (double)tsrc[jj];
            } else {
                // 1/2 ln(4 (sin^2 a + sinh^2 b)).  Against the flat geometry only near it: where
                // the bed rises far above the reference depth y tends to -1, 1 + y would cancel
                // (and the flat distance may overflow), and the logarithm is that of the distance
                const double y = (shd - sh0) * (shd + sh0) * rfl[d];
                const double l = pair_is_small(y) ? lfl[d] + 0.5 * (double)pair_small(R(y)) : 0.5 * (double)log(sa2 + sh * sh);
                acc += (l + M_LN2) * (double)tsrc[jj];
                if (j != i) {
                    // minus the bed's double layer at (x_j, b_j)
                    R chb;
                    const R shb = sinh_cosh_series(R(pld * (tbz[jj] - bzi)), &chb);
                    accb += (double)pair_div(R(-2) * shb * chb + s2a * R(tbx[jj]), sa2 + shb * shb) * tpb[jj];
                }
            }
        }
    }
    const double hpl = 0.5 * (double)pl;
    acc = pair_fold(KIND == 2 ? hpl * acc : hpl * accb - acc, red, lane, il);
    if (!on || lane > 0) return;
    const double dx = p.lx / n;
    double out = acc * dx;
    if (KIND == 3 && i >= jbeg && i < jend) {
        // minus the diagonal of the bed's double layer: + b_xx / (2 (1 + b_x^2)) phi_b
        const double bxi = bxs[i], bxxi = static_cast<const double*>(p.bxx)[mb + i];
        out += dx * bxxi / (2.0 * (1.0 + bxi * bxi)) * pbs[i];
    }
    static_cast<double*>(p.part)[((long long)split * p.batch + m) * n + i] = out;
}

// --- rb = -D_BS[phi_s] of the two-boundary members (slices added in order)
template <typename R>
__global__ void k_full_rb(const FullParams p) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int m = blockIdx.z;
    if (i >= p.n || !full_bed(p, m)) return;
    double a = 0.0;
    for (int s = 0; s < p.nsplit; ++s) a -= static_cast<const double*>(p.part)[((long long)s * p.batch + m) * p.n + i];
    static_cast<double*>(p.rb)[(long long)m * p.n + i] = a;
}

// --- phi_b of the next sweep, (rb + S_BS[V_n] - D_BB[phi_b]) / pi, for the
// undecided two-boundary members (no bed pass at the first sweep: V_0 = 0,
// phi_b = 0)
template <typename R>
__global__ void k_full_pb(const FullParams p) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int m = blockIdx.z;
    if (i >= p.n || !full_bed(p, m) || p.ctl[m].done) return;
    const long long o = (long long)m * p.n + i;
    double a = static_cast<const double*>(p.rb)[o];
    if (p.pbin)
        for (int s = 0; s < p.nsplit; ++s) a += static_cast<const double*>(p.part)[((long long)s * p.batch + m) * p.n + i];
    static_cast<double*>(p.pbout)[o] = a / M_PI;
}

// --- rhs = pi phi_s + D[phi_s] (slices added in order)
template <typename R>
__global__ void k_full_rhs(const FullParams p) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int m = blockIdx.z;
    if (i >= p.n) return;
    const long long mo = m * p.s_phys;
    double a = M_PI * (double)static_cast<const R*>(p.phi)[mo + i];
    for (int s = 0; s < p.nsplit; ++s) a += static_cast<const double*>(p.part)[((long long)s * p.batch + m) * p.n + i];
    static_cast<double*>(p.rhs)[(long long)m * p.n + i] = a;
}

// --- w = rhs - (S - S0)[V_n], or rhs - (S - S_flat)[V_n] + D_SB[phi_b] (the
// slices of the surface pass, in order; w = rhs at the first sweep of the
// image form, from V_0 = 0)
// The slices of 64 points are shared by kCombLanes wavefronts, whose sums are
// added in order: one thread per point would wait for its loads slice by slice.
constexpr int kCombLanes = 8;
template <typename R>
__global__ void __launch_bounds__(64 * kCombLanes) k_full_combine(const FullParams p) {
    __shared__ double red[kCombLanes][64];
    const int t = threadIdx.x & 63, lane = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + t;
    const int m = blockIdx.z;
    if (p.ctl[m].done) return;  // decided by this sweep's pair pass (workgroup-uniform)
    const long long o = (long long)m * p.n + i;
    // slices: those of the two-boundary surface pass, or of the image form's
    // single layer (nsym of the symmetric pass when it ran)
    const int ns = !(p.vin || full_bed(p, m)) ? 0 : (full_bed(p, m) ? p.nsplit : (p.nsym > 0 ? p.nsym : p.nsplit));
    double a = 0.0;
    if (i < p.n) {
#pragma unroll 4
        for (int s = lane; s < ns; s += kCombLanes) a += static_cast<const double*>(p.part)[((long long)s * p.batch + m) * p.n + i];
    }
    red[lane][t] = a;
    __syncthreads();
    if (lane > 0 || i >= p.n) return;
    double w = static_cast<const double*>(p.rhs)[o];
#pragma unroll
    for (int l = 0; l < kCombLanes; ++l) w -= red[l][t];
    static_cast<double*>(p.w)[o] = w;
}

// --- V_(n+1) = S0^-1 w (+ S0^-1 (S0 - S_flat)[V_n] in the two-boundary form)
// in two passes.  The sum pass: workgroup (x, s) forms the kApOuts outputs of
// block x over source slice s; a thread forms kApR consecutive outputs over one
// of kApLanes ranges of the slice (its wavefront's: the source value is
// wave-uniform), keeping the kApR circulant entries c[i + r - j] as a window
// that moves by one entry per source point, so each step loads one table entry
// for kApR products; the ranges are added in LDS in a fixed order and the
// slice's sums go to the pair-pass slices, spent by then.  The finish pass adds
// the slices in order and takes the residual maxima max|V_(n+1) - V_n|,
// max|V_(n+1)| into the member's slot `sweep`.
constexpr int kApR = 4, kApLanes = 8, kApB = 16;
constexpr int kApThreads = 64 * kApLanes;
constexpr int kApOuts = 64 * kApR;  // outputs per workgroup
// source slices of the sum pass: enough workgroups to cover the chip at 4096
// points, each lane's range at least kApB points when n allows
__host__ __device__ constexpr int apply_slices(int n) { return n / 128 < 1 ? 1 : (n / 128 > 16 ? 16 : n / 128); }


// acc[k][r] += sum_j tab[k][(i0 + r - j) mod n] src_j over j in [jb, je), for
// NT tables against one source, in blocks of kApB source points whose table
// entries and source values are all requested before the block's products
// (one memory latency per block)
template <int NT, typename S>
__device__ __forceinline__ void circ_window(const double* const (&tab)[NT], const S* src, int i0, int jb, int je,
                                            int msk, double (&acc)[NT][kApR]) {
    double cw[NT][kApR];
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int r = 0; r < kApR; ++r) cw[k][r] = tab[k][(i0 + r - jb) & msk];
    for (int j0 = jb; j0 < je; j0 += kApB) {
        double nx[NT][kApB], sv[kApB];
#pragma unroll
        for (int q = 0; q < kApB; ++q) {
            const int j = j0 + q;
#pragma unroll
            for (int k = 0; k < NT; ++k) nx[k][q] = tab[k][(i0 - j - 1) & msk];  // enters the window after point j
            sv[q] = j < je ? (double)src[j] : 0.0;  // a short range (small n) ends inside a block
        }
#pragma unroll
        for (int q = 0; q < kApB; ++q)
#pragma unroll
            for (int k = 0; k < NT; ++k) {
#pragma unroll
                for (int r = 0; r < kApR; ++r) acc[k][r] += cw[k][r] * sv[q];
#pragma unroll
                for (int r = kApR - 1; r > 0; --r) cw[k][r] = cw[k][r - 1];
                cw[k][0] = nx[k][q];
            }
    }
}

template <typename R>
__global__ void __launch_bounds__(kApThreads) k_full_apply(const FullParams p) {
    __shared__ double red[kApLanes][kApOuts];
    const int t = threadIdx.x;
    const int m = blockIdx.z;
    const int n = p.n;
    const int msk = n - 1;
    if (p.ctl[m].done) return;  // decided by this sweep's pair pass (workgroup-uniform)
    const long long mo = m * p.s_phys;
    const int lane = __builtin_amdgcn_readfirstlane(t / 64);
    const int o0 = (t & 63) * kApR;  // this thread's first output within the workgroup
    const int i0 = blockIdx.x * kApOuts + o0;
    const int ns = apply_slices(n);
    const int sl = n / ns;  // points per slice (n and ns are powers of two)
    const int jn = (sl + kApLanes - 1) / kApLanes;
    const int jb = blockIdx.y * sl + lane * jn, je = min(blockIdx.y * sl + sl, jb + jn);
    double acc[1][kApR];
#pragma unroll
    for (int r = 0; r < kApR; ++r) acc[0][r] = 0.0;
    if (jb < je) {
        const double* const c0[1] = {static_cast<const double*>(p.c0) + (long long)m * n};
        circ_window<1>(c0, static_cast<const double*>(p.w) + (long long)m * n, i0, jb, je, msk, acc);
        if (p.vin && full_bed(p, m)) {
            // + S0^-1 (S0 - S_flat)[V_n] of the two-boundary form
            const double* const cm[1] = {static_cast<const double*>(p.cm) + (long long)m * n};
            circ_window<1>(cm, static_cast<const R*>(p.vin) + mo, i0, jb, je, msk, acc);
        }
    }
#pragma unroll
    for (int r = 0; r < kApR; ++r) red[lane][o0 + r] = acc[0][r];
    __syncthreads();
    const int i = blockIdx.x * kApOuts + t;
    if (t < kApOuts && i < n) {
        double a = 0.0;
#pragma unroll
        for (int l = 0; l < kApLanes; ++l) a += red[l][t];
        static_cast<double*>(p.part)[((long long)blockIdx.y * p.batch + m) * n + i] = a;
    }
}

template <typename R>
__global__ void __launch_bounds__(kFullThreads) k_full_finish(const FullParams p) {
    const int t = threadIdx.x;
    const int i = blockIdx.x * kFullThreads + t;
    const int m = blockIdx.z;
    const int n = p.n;
    Ctl* ctl = p.ctl + m;
    if (ctl->done) return;  // workgroup-uniform
    const long long mo = m * p.s_phys;
    unsigned long long nu = 0ull, de = 0ull;
    if (i < n) {
        const int ns = apply_slices(n);
        double a = 0.0;
        for (int s2 = 0; s2 < ns; ++s2) a += static_cast<const double*>(p.part)[((long long)s2 * p.batch + m) * n + i];
        const R v = R(a);
        static_cast<R*>(p.vout)[mo + i] = v;
        const double vold = p.vin ? (double)static_cast<const R*>(p.vin)[mo + i] : 0.0;
        nu = abs_bits((double)v - vold);
        de = abs_bits((double)v);
        if (!isfinite((double)v)) nu = de = 0x7ff8000000000000ull;  // a NaN key outranks every finite one
    }
    block_reduce2_max_u64(nu, de);
    if (t == 0) {
        atomicMax(&ctl->slots->num[p.sweep], nu);
        atomicMax(&ctl->slots->den[p.sweep], de);
    }
}

// --- eta_x, eta_xx at every point: the circulant sums d1 * eta and d2 * eta
// by the apply's sum pass (both tables against eta; the ex slices first, then
// the exx slices, in the pair-pass slices, free at the start of a solve) and a
// pass that adds the slices in order
__host__ __device__ constexpr int geom_slices(int n) { return apply_slices(n) / 2 < 1 ? 1 : apply_slices(n) / 2; }

template <typename R>
__global__ void __launch_bounds__(kApThreads) k_full_geom(const FullParams p) {
    __shared__ double red[2][kApLanes][kApOuts];
    const int t = threadIdx.x;
    const int m = blockIdx.z;
    const int n = p.n;
    const int msk = n - 1;
    const int lane = __builtin_amdgcn_readfirstlane(t / 64);
    const int o0 = (t & 63) * kApR;
    const int i0 = blockIdx.x * kApOuts + o0;
    const int ns = geom_slices(n);
    const int sl = n / ns;
    const int jn = (sl + kApLanes - 1) / kApLanes;
    const int jb = blockIdx.y * sl + lane * jn, je = min(blockIdx.y * sl + sl, jb + jn);
    double acc[2][kApR];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < kApR; ++r) acc[k][r] = 0.0;
    if (jb < je) {
        const double* const tab[2] = {static_cast<const double*>(p.d1), static_cast<const double*>(p.d2)};
        circ_window<2>(tab, static_cast<const R*>(p.eta) + m * p.s_phys, i0, jb, je, msk, acc);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < kApR; ++r) red[k][lane][o0 + r] = acc[k][r];
    __syncthreads();
    const int i = blockIdx.x * kApOuts + t;
    if (t < kApOuts && i < n) {
        double* part = static_cast<double*>(p.part);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            double a = 0.0;
#pragma unroll
            for (int l = 0; l < kApLanes; ++l) a += red[k][l][t];
            part[((long long)(k * ns + blockIdx.y) * p.batch + m) * n + i] = a;
        }
    }
}

template <typename R>
__global__ void k_full_geomfin(const FullParams p) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int m = blockIdx.z;
    const int n = p.n;
    if (i >= n) return;
    const int ns = geom_slices(n);
    const double* part = static_cast<const double*>(p.part);
    double a1 = 0.0, a2 = 0.0;
    for (int s = 0; s < ns; ++s) {
        a1 += part[((long long)s * p.batch + m) * n + i];
        a2 += part[((long long)(ns + s) * p.batch + m) * n + i];
    }
    static_cast<R*>(p.ex)[m * p.s_phys + i] = R(a1);
    static_cast<R*>(p.exx)[m * p.s_phys + i] = R(a2);
}

// --- the decided iterate V_s of every member (s = its sweep count) -> out
template <typename R>
__global__ void k_full_select(const FullParams p) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int m = blockIdx.z;
    if (i >= p.n) return;
    const int s = p.ctl[m].sweeps;
    const long long mo = m * p.s_phys;
    static_cast<R*>(p.vfinal)[mo + i] = static_cast<const R*>(p.vbuf[s & 1])[mo + i];
}

// ---------------------------------------------------------------------------
template <> hipError_t launch_full_t<Real>(const FullParams& p, int what, hipStream_t s) {
    const int n = p.n;
    const int tiles = (n + kFullThreads - 1) / kFullThreads;
    const int outs = (n + kOutPerBlock - 1) / kOutPerBlock;
    switch (what) {
        case FULL_TABLES:
            hipLaunchKernelGGL(k_full_tables<Real>, dim3(tiles, p.batch), dim3(kFullThreads), 0, s, p);
            break;
        case FULL_GEOM: {
            hipLaunchKernelGGL(k_full_geom<Real>, dim3((n + kApOuts - 1) / kApOuts, geom_slices(n), p.batch),
                               dim3(kApThreads), 0, s, p);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(k_full_geomfin<Real>, dim3(tiles, 1, p.batch), dim3(kFullThreads), 0, s, p);
            break;
        }
        case FULL_DOUBLE:
            hipLaunchKernelGGL((k_full_pairs<Real, 0>), dim3(tiles, p.nsplit, p.batch), dim3(kPairThreads), 0, s, p);
            break;
        case FULL_RHS:
            hipLaunchKernelGGL(k_full_rhs<Real>, dim3(tiles, 1, p.batch), dim3(kFullThreads), 0, s, p);
            break;
        case FULL_SINGLE:
            hipLaunchKernelGGL((k_full_pairs<Real, 1>), dim3(tiles, p.nsplit, p.batch), dim3(kPairThreads), 0, s, p);
            break;
        case FULL_COMBINE:
            hipLaunchKernelGGL(k_full_combine<Real>, dim3((n + 63) / 64, 1, p.batch), dim3(64 * kCombLanes), 0, s, p);
            break;
        case FULL_APPLY: {
            hipLaunchKernelGGL(k_full_apply<Real>, dim3((n + kApOuts - 1) / kApOuts, apply_slices(n), p.batch),
                               dim3(kApThreads), 0, s, p);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(k_full_finish<Real>, dim3(tiles, 1, p.batch), dim3(kFullThreads), 0, s, p);
            break;
        }
        case FULL_SELECT:
            hipLaunchKernelGGL(k_full_select<Real>, dim3(tiles, 1, p.batch), dim3(kFullThreads), 0, s, p);
            break;
        case FULL_BEDGEOM:
            hipLaunchKernelGGL(k_full_bedgeom<Real>, dim3(outs, 1, p.batch), dim3(kFullThreads), 0, s, p);
            break;
        case FULL_RHSB:
            hipLaunchKernelGGL((k_full_bpairs<Real, 2>), dim3(tiles, p.nsplit, p.batch), dim3(kPairThreads), 0, s, p);
            break;
        case FULL_RB:
            hipLaunchKernelGGL(k_full_rb<Real>, dim3(tiles, 1, p.batch), dim3(kFullThreads), 0, s, p);
            break;
        case FULL_BED:
            hipLaunchKernelGGL((k_full_bpairs<Real, 3>), dim3(tiles, p.nsplit, p.batch), dim3(kPairThreads), 0, s, p);
            break;
        case FULL_SYM:
        {
            const int nb = p.nsym;
            if (n == nb * kSymT)
                hipLaunchKernelGGL((k_full_sympairs<Real, 1>), dim3(nb * (nb + 1) / 2, 1, p.batch), dim3(64 * kSymWaves), 0, s, p);
            else if (n == nb * 2 * kSymT)
                hipLaunchKernelGGL((k_full_sympairs<Real, 2>), dim3(nb * (nb + 1) / 2, 1, p.batch), dim3(64 * kSymWaves), 0, s, p);
            else
                return hipErrorInvalidValue;
            break;
        }
        case FULL_SURF:
            hipLaunchKernelGGL(k_full_spairs<Real>, dim3(tiles, p.nsplit, p.batch), dim3(kPairThreads), 0, s, p);
            break;
        case FULL_PB:
            hipLaunchKernelGGL(k_full_pb<Real>, dim3(tiles, 1, p.batch), dim3(kFullThreads), 0, s, p);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace sbi
