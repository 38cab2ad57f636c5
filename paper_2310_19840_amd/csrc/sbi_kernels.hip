// sbi_kernels.hip -- gfx950 kernels of the SBI wave solver.
//
// Every 2D transform is split into a row pass (real <-> half form, one row per
// group of P threads, half-length complex FFT plus the standard real/complex
// twist) and a column pass (C adjacent columns per workgroup, length-ny complex
// FFT).  The products of the method (eta^j V, delta^j grad phi_b, ...) are
// formed in registers inside the row pass; the Fourier multipliers of the
// method (k^j/j! tanh(kh), sech(kh), i k, ...) are applied and summed inside
// the column pass, which then runs the inverse column transforms of the new
// iterate directly from registers.  Only kept modes are ever written, so the
// spectra in memory are 1/4 (2D) of the full size.
#include <math.h>
#include <algorithm>
#include <type_traits>
#include "sbi_device.hpp"
#include "sbi_fft.hpp"
#include "sbi_kernels.hpp"
#include "sbi_stage.hpp"

#ifndef SBI_REAL
#error "compile with -DSBI_REAL=double or -DSBI_REAL=float"
#endif

namespace sbi {

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------

template <typename V> __device__ __forceinline__ V rmul(V a, V b) {  // componentwise real product
    return cx<V>(a.x * b.x, a.y * b.y);
}

// ---------------------------------------------------------------------------
// Row pass helpers: real row of length NX <-> kept half spectrum F[0..Mx]
// via the length-NX/2 complex transform of z[n] = f[2n] + i f[2n+1].
// ---------------------------------------------------------------------------
// Per-thread view of a row-pass workgroup: rpw rows of P threads each.
struct RowCtx {
    int t, nthr, j, rl, y0, rpw, rsh, ny, ldh, Mx, mem;  // rpw = 1 << rsh rows per workgroup
    bool valid;
};

// LDS pitch of a row (elements): room for the padded transform, rounded up so
// that consecutive rows start 16 banks apart -- the staging loops read and
// write (row, mode) with the row index fastest, and a quarter wave of 16-byte
// (half wave of 8-byte) accesses then covers distinct banks
constexpr int row_pitch(int e0, int vbytes) {
    const int unit = 256 / vbytes, want = 64 / vbytes;
    int ls = e0;
    while (ls % unit != want) ++ls;
    return ls;
}

// EM: elements per thread of the row transform (its radix sequence: 8 gives
// radix-8 passes, 16 radix-16 ones); TWC: every twiddle power held in
// registers instead of formed by recurrence.  Both are launch-plan choices.
template <typename R, int NX, int EM = 8, bool TWC = false> struct Row {
    using V = typename cplx_of<R>::type;
    static constexpr int N = NX / 2;
    static constexpr int E = FftShape<N, EM>::E;
    static constexpr int P = FftShape<N, EM>::P;
    static constexpr int LS = row_pitch(fft_lds_elems<N, E>(), (int)sizeof(V));
    // a row of up to 64 threads lies in one wavefront: its transform's LDS
    // exchanges need only wave-level ordering
    static constexpr bool WAVE = P <= 64;

    // A thread's modes come in batches whose reads are issued together, the index
    // clamped to the last one: a loop that tests each mode before its read waits out
    // the latency once a mode.  128 x 64, FP64: sweeps 9.8 -> 8.3 us, N_phi 16.5 -> 13.8;
    // 512 x 512, FP32: products of an order 8.0 -> 7.3 us, N_phi 16.9 -> 13.5; 1024 x 1024,
    // FP32: sweeps 27.1 -> 25.3 us (in FP64 unchanged at 35.5).  Rows of 8192 points in FP64 read
    // two at a time: with four the mixed sweeps spill (8192 x 16, 16 members 159 us, with two 138).
    static constexpr int kBatch = sizeof(R) == 8 && NX >= 8192 ? 2 : 4;
    static __device__ __forceinline__ void fetch(V (&f)[kBatch], const V* __restrict__ Gr, const V* __restrict__ G2r, R c2,
                                                 int k0, int kstep, int K, int ldh) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) f[u] = Gr[min(k0 + u * kstep, K - 1) * ldh];
        if (G2r) {
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const V f2 = G2r[min(k0 + u * kstep, K - 1) * ldh];
                f[u] = cx<V>(f[u].x + c2 * f2.x, f[u].y + c2 * f2.y);
            }
        }
    }

    // v <- z = inverse row transform of (G + c2 G2) for the thread's row.
    // G, G2: member base of a half form [m_x][ny]; all rows of the workgroup
    // stage their kept spectra through LDS with coalesced column segments.
    // z[n] = f[2n] + i f[2n+1] has Z[m] = (F[m] + conj F[N-m]) / 2
    //   + i (F[m] - conj F[N-m]) / 2 * exp(+2 pi i m / NX).
    using TW = typename std::conditional<TWC, TwidAll<V, N, E>, Twid<V, N, E>>::type;
    static __device__ __forceinline__ void inverse(V (&v)[E], const V* __restrict__ G, const V* __restrict__ G2,
                                                   R c2, const RowCtx& rc, V* lds_all,
                                                   const TW& twN, const V* __restrict__ twX, R scale) {
        V* lds = lds_all + rc.rl * LS;
        // a thread stages modes k0, k0 + kstep, ... of row r2 of the workgroup
        // (the block is a whole number of rows, and ny a multiple of rpw)
        const int r2 = rc.t & (rc.rpw - 1);
        const int k0 = rc.t >> rc.rsh, kstep = rc.nthr >> rc.rsh;
        V* const zr = lds_all + r2 * LS;
        const V* const Gr = G + rc.y0 + r2;
        const V* const G2r = G2 ? G2 + rc.y0 + r2 : nullptr;
        const int K = rc.Mx + 1;
        V f[kBatch];
        fetch(f, Gr, G2r, c2, k0, kstep, K, rc.ldh);
        lds_sync();  // other rows' transforms are done with the area the staging loop writes
        if (2 * rc.Mx < N) {
            // kept band below N/2: F[k] alone gives Z[k] and Z[N-k], Z is zero
            // between them; the staging loop writes Z directly
            for (int kb = k0; kb < K; kb += kBatch * kstep) {
                if (kb > k0) fetch(f, Gr, G2r, c2, kb, kstep, K, rc.ldh);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int k = kb + u * kstep;
                    if (k >= K) break;
                    const V h = cscale(f[u], R(0.5));
                    zr[k] = cadd(h, mul_i(cmul(h, cconj(twX[k]))));
                    if (k > 0) {
                        const V hc = cconj(h);
                        const V w = mul_i(cmul(hc, cconj(twX[N - k])));
                        zr[N - k] = cx<V>(hc.x - w.x, hc.y - w.y);
                    }
                }
            }
            for (int k = K + k0; k <= N - K; k += kstep) zr[k] = cx<V>(R(0), R(0));
            lds_sync();
#pragma unroll
            for (int q = 0; q < E; ++q) v[q] = lds[rc.j + q * P];
        } else {
            for (int mb = k0; mb < N; mb += kBatch * kstep) {
                if (mb > k0) fetch(f, Gr, G2r, c2, mb, kstep, K, rc.ldh);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int m = mb + u * kstep;
                    if (m < N) zr[m] = m <= rc.Mx ? f[u] : cx<V>(R(0), R(0));
                }
            }
            lds_sync();
#pragma unroll
            for (int q = 0; q < E; ++q) {
                const int m = rc.j + q * P;
                V fm = lds[m];
                V fc = (m == 0) ? cx<V>(R(0), R(0)) : cconj(lds[N - m]);
                V ev = cx<V>(R(0.5) * (fm.x + fc.x), R(0.5) * (fm.y + fc.y));
                V od = cx<V>(R(0.5) * (fm.x - fc.x), R(0.5) * (fm.y - fc.y));
                od = cmul(od, cconj(twX[m]));           // exp(+2 pi i m / NX)
                v[q] = cadd(ev, mul_i(od));
            }
        }
        xfer_sync<WAVE>();  // the row's staged values are in registers before the exchanges reuse them
        fft<V, N, true, 1, EM, WAVE>(v, lds, 0, rc.j, twN);
#pragma unroll
        for (int q = 0; q < E; ++q) v[q] = cscale(v[q], scale);
    }

    // H[kept m][row] <- forward row transform of the real pairs in v (v is
    // destroyed): F[m] = (Z[m] + conj Z[N-m]) / 2 - i (Z[m] - conj Z[N-m]) / 2
    // * exp(-2 pi i m / NX), formed by the cooperative column-segment store.
    static __device__ __forceinline__ void forward(V (&v)[E], V* __restrict__ H, const RowCtx& rc, V* lds_all,
                                                   const TW& twN, const V* __restrict__ twX) {
        V* lds = lds_all + rc.rl * LS;
        // other rows touch this row's LDS only in the staging and store loops,
        // each closed by a workgroup barrier
        fft<V, N, false, 1, EM, WAVE>(v, lds, 0, rc.j, twN);
        xfer_sync<WAVE>();  // the row's last exchange reads are done before it is overwritten
#pragma unroll
        for (int q = 0; q < E; ++q) lds[rc.j + q * P] = v[q];
        lds_sync();
        // a thread stores modes m0, m0 + mstep, ... of row r2 of the workgroup
        const int r2 = rc.t & (rc.rpw - 1);
        const V* const zr = lds_all + r2 * LS;
        V* const Hr = H + rc.y0 + r2;
        const int mstep = rc.nthr >> rc.rsh;
        for (int mb = rc.t >> rc.rsh; mb <= rc.Mx; mb += kBatch * mstep) {
            V zm[kBatch], zc[kBatch], tw[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int m = min(mb + u * mstep, rc.Mx);
                zm[u] = zr[m];
                zc[u] = zr[(N - m) & (N - 1)];
                tw[u] = twX[m];
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int m = mb + u * mstep;
                const V c = cconj(zc[u]);
                const V ev = cx<V>(R(0.5) * (zm[u].x + c.x), R(0.5) * (zm[u].y + c.y));
                const V od = mul_mi<false>(cx<V>(R(0.5) * (zm[u].x - c.x), R(0.5) * (zm[u].y - c.y)));
                const V F = cadd(ev, cmul(tw[u], od));
                if (m <= rc.Mx) Hr[m * rc.ldh] = F;
            }
        }
        lds_sync();
    }

    static __device__ __forceinline__ void load(V (&v)[E], const R* __restrict__ row, int j, bool valid) {
        const V* r2 = reinterpret_cast<const V*>(row);
#pragma unroll
        for (int q = 0; q < E; ++q) v[q] = valid ? r2[j + q * P] : cx<V>(R(0), R(0));
    }
    static __device__ __forceinline__ void store(const V (&v)[E], R* __restrict__ row, int j, bool valid) {
        if (!valid) return;
        V* r2 = reinterpret_cast<V*>(row);
#pragma unroll
        for (int q = 0; q < E; ++q) r2[j + q * P] = v[q];
    }
};

// threads per row-pass workgroup: rows of P threads packed up to 256 threads
template <int NX, int EM = 8> __host__ __device__ constexpr int row_threads() {
    return FftShape<NX / 2, EM>::P > 256 ? FftShape<NX / 2, EM>::P : 256;
}

// Row transform of launch-plan variant VAR of the sweep and SA kernels:
// 0 radix-8 passes with twiddle recurrence, 1 the same with every twiddle
// power cached, 2 radix-16 passes, 3 radix-4 passes
template <typename R, int NX, int VAR> struct RowVarT {
    using type = Row<R, NX, VAR == 2 ? 16 : (VAR == 3 ? 4 : 8), VAR == 1>;
};
template <typename R, int NX, int VAR> using RowVar = typename RowVarT<R, NX, VAR>::type;

// Workgroups are dealt to the 8 XCDs round-robin by launch order, and each
// XCD has its own L2.  Neighbouring row groups read neighbouring pieces of the
// same cache lines of the column-major half forms, so they are mapped to the
// same XCD: launch index b runs row group (b % 8) * (G / 8) + b / 8.
__device__ __forceinline__ int xcd_row_group(int b, int G) {
    constexpr int kXcd = 8;
    return (G % kXcd) ? b : (b % kXcd) * (G / kXcd) + b / kXcd;
}

template <int P> __device__ __forceinline__ RowCtx row_ctx(const GridDev& g) {
    RowCtx r;
    r.t = threadIdx.x;
    r.nthr = blockDim.x;
    r.j = r.t % P;
    r.rl = r.t / P;
    r.rpw = blockDim.x / P;  // a power of two (grid sizes are)
    r.rsh = __builtin_ctz((unsigned)r.rpw);
    r.y0 = xcd_row_group(blockIdx.x, gridDim.x) * r.rpw;
    r.ny = g.ny;
    r.ldh = g.ldh;
    r.Mx = g.Mx;
    r.mem = blockIdx.z;
    r.valid = r.y0 + r.rl < g.ny;
    return r;
}

#define ROW_PROLOGUE_T(...)                                              \
    using RW = __VA_ARGS__;                                              \
    using V = typename RW::V;                                            \
    constexpr int E = RW::E;                                             \
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];                          \
    const RowCtx rc = row_ctx<RW::P>(p.g);                               \
    const struct {                                                       \
        int j, mem;                                                      \
        bool valid;                                                      \
    } ri = {rc.j, rc.mem, rc.valid};                                     \
    V* lds_all = reinterpret_cast<V*>(smem_raw);                         \
    const long long hb = (long long)rc.mem * p.g.s_half;                 \
    const long long po = rc.mem * p.g.s_phys + (long long)(rc.valid ? rc.y0 + rc.rl : 0) * p.g.nx; \
    const R iscale = R(1.0 / ((double)RW::N * (double)p.g.ny));          \
    typename RW::TW twN;                                                 \
    twN.load(twN_tab, rc.j);                                             \
    /* the twist table exp(-2 pi i m / NX), m < N, staged after the rows'  \
       areas: the staging and store loops then read it from LDS (a global  \
       read there would wait behind the loop's own stores) */             \
    V* const twX = lds_all + rc.rpw * RW::LS;                            \
    for (int i_ = rc.t; i_ < RW::N; i_ += rc.nthr) twX[i_] = twX_tab[i_]; \
    (void)po; (void)iscale; (void)hb;
#define ROW_PROLOGUE(R, NX) ROW_PROLOGUE_T(Row<R, NX>)

// ---------------------------------------------------------------------------
// Row kernels
// ---------------------------------------------------------------------------
template <typename R, int NX>
__global__ void __launch_bounds__(row_threads<NX>()) k_row_fwd(const RowFwdParams p, const typename cplx_of<R>::type* twN_tab,
                          const typename cplx_of<R>::type* twX_tab) {
    ROW_PROLOGUE(R, NX)
    for (int f = 0; f < p.nf; ++f) {
        V v[E];
        RW::load(v, static_cast<const R*>(p.in[f]) + po, ri.j, ri.valid);
        RW::forward(v, static_cast<V*>(p.out[f]) + hb, rc, lds_all, twN, twX);
    }
}

template <typename R, int NX>
__global__ void __launch_bounds__(row_threads<NX>()) k_row_inv(const RowInvParams p, const typename cplx_of<R>::type* twN_tab,
                          const typename cplx_of<R>::type* twX_tab) {
    ROW_PROLOGUE(R, NX)
    for (int f = 0; f < p.nf; ++f) {
        V v[E];
        const V* g2 = p.in2[f] ? static_cast<const V*>(p.in2[f]) + hb : nullptr;
        R c2 = R(0);
        if (g2) c2 = R(1.0 - p.ctl[ri.mem].omega);
        RW::inverse(v, static_cast<const V*>(p.in[f]) + hb, g2, c2, rc, lds_all, twN, twX, iscale);
        RW::store(v, static_cast<R*>(p.out[f]) + po, ri.j, ri.valid);
    }
}

// Forward half forms of the running products v w^j, j = j0 + 1 .. j1, of a row
// (v is destroyed; every chunk of a chain forms the same products).
template <typename RW, typename V, int E>
__device__ __forceinline__ void row_chain(V (&v)[E], const V (&w)[E], int j0, int j1, void* const* h, long long hb,
                                          const RowCtx& rc, V* lds_all, const typename RW::TW& twN, const V* twX) {
    for (int jj = 1; jj <= j1; ++jj) {
#pragma unroll
        for (int q = 0; q < E; ++q) v[q] = rmul(v[q], w[q]);
        if (jj <= j0) continue;
        V o[E];
#pragma unroll
        for (int q = 0; q < E; ++q) o[q] = v[q];
        RW::forward(o, static_cast<V*>(h[jj - 1]) + hb, rc, lds_all, twN, twX);
    }
}

// Product families of a W solve: src w^j, j = 1 .. J, for each family's half
// form src and its weight w (eta, or delta for the bed's gradients) -- the
// forcing eta^j grad phi_s of every order, and in SA mode the products of the
// order last formed.  Workgroup row y takes products pc ch + 1 .. pc (ch + 1) of
// family y / nch.  The lead family also serves the stage: it stores eta, its
// extrema (relaxation weight) and the checks for non-finite values.
//
// A workgroup is one chain of transforms, so few rows leave the chip idle
// however short the rows: there each product takes a workgroup of its own and
// the inverse transform before it is repeated (row_chunk).
template <typename R, int NX, int VAR>
__global__ void __launch_bounds__((row_threads<NX, RowVar<R, NX, VAR>::E>()))
    k_row_prod(const RowProdParams p, const typename cplx_of<R>::type* twN_tab,
               const typename cplx_of<R>::type* twX_tab) {
    ROW_PROLOGUE_T(RowVar<R, NX, VAR>)
    const int fam = blockIdx.y / p.nch, ch = blockIdx.y % p.nch;
    const bool bed = (p.bed >> fam) & 1;
    const bool check = ch == 0 && ((p.check >> fam) & 1);
    const bool lead = ch == 0 && fam == p.lead;
    V w[E];
    if (bed) {
        RW::load(w, static_cast<const R*>(p.delta) + po, ri.j, ri.valid);
    } else if (p.g_eta) {
        RW::inverse(w, static_cast<const V*>(p.g_eta) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
    } else {
        RW::load(w, static_cast<const R*>(p.eta_in) + po, ri.j, ri.valid);
    }
    int bad = 0;
    if (lead) {
        if (p.eta_out) RW::store(w, static_cast<R*>(p.eta_out) + po, ri.j, ri.valid);
        if (p.extrema) {
            unsigned long long mx = 0ull, mn = ~0ull;
            if (ri.valid) {
#pragma unroll
                for (int q = 0; q < E; ++q) {
                    unsigned long long a = ord_bits((double)w[q].x), b = ord_bits((double)w[q].y);
                    mx = a > mx ? a : mx;
                    mx = b > mx ? b : mx;
                    mn = a < mn ? a : mn;
                    mn = b < mn ? b : mn;
                }
            }
            mx = block_reduce_u64<true>(mx);
            mn = block_reduce_u64<false>(mn);
            if (threadIdx.x == 0) {
                atomicMax(&p.ctl[ri.mem].eta_max, mx);
                atomicMin(&p.ctl[ri.mem].eta_min, mn);
            }
        }
        if (ri.valid) {
#pragma unroll
            for (int q = 0; q < E; ++q) bad |= !isfinite((double)w[q].x) || !isfinite((double)w[q].y);
        }
    }
    V v[E];
    RW::inverse(v, static_cast<const V*>(p.src[fam]) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
    if (check && ri.valid) {
#pragma unroll
        for (int q = 0; q < E; ++q) bad |= !isfinite((double)v[q].x) || !isfinite((double)v[q].y);
    }
    if (bad) atomicOr(&p.ctl[ri.mem].nonfinite, 1);
    row_chain<RW, V, E>(v, w, ch * p.pc, min(p.J, (ch + 1) * p.pc), p.h + fam * p.J, hb, rc, lds_all, twN, twX);
}

template <typename R, int NX, bool AA, int VAR>
__device__ __forceinline__ void row_sweep_body(const RowSweepParams& p, const typename cplx_of<R>::type* twN_tab,
                                               const typename cplx_of<R>::type* twX_tab) {
    Ctl* ctl = p.ctl + blockIdx.z;
    if (ctl->done) return;  // block-uniform: the member's solve is decided
    ROW_PROLOGUE_T(RowVar<R, NX, VAR>)
    // product family and chunk of this workgroup; with several chunks the
    // residual test has a workgroup row of its own after them.  The iterate and the
    // products come from one piece of code however the chains are cut: copies of it may
    // round apart, and a member's results must not depend on how many others there are
    const int fam = blockIdx.y / p.nch, ch = blockIdx.y % p.nch;
    const bool rest = fam == p.nfam;
    const bool test = p.residual && (rest || (fam == 0 && p.nch == 1)), products = p.products && !rest;
    V v[E];
    // the iterate: for its products, and for the residual's denominator
    // of the relaxed update (a residual-only Anderson pass needs neither)
    if (products || (test && !AA))
        RW::inverse(v, static_cast<const V*>(fam == 0 || rest ? p.gV : (fam == 1 ? p.gbx : p.gby)) + hb, nullptr, R(0), rc,
                    lds_all, twN, twX, iscale);
    if (test) {
        V dd[E];
        RW::inverse(dd, static_cast<const V*>(p.gD) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
        const double c = 1.0 - ctl->omega;
        unsigned long long nu = 0ull, de = 0ull;
        if (ri.valid) {
#pragma unroll
            for (int q = 0; q < E; ++q) {
                const double d0 = (double)dd[q].x, d1 = (double)dd[q].y;
                unsigned long long a = abs_bits(d0), b = abs_bits(d1);
                nu = a > nu ? a : nu;
                nu = b > nu ? b : nu;
                if constexpr (!AA) {
                    // denominator T(V_(n-1)) = V_n + (1 - omega) D from the relaxed update
                    a = abs_bits((double)v[q].x + c * d0);
                    b = abs_bits((double)v[q].y + c * d1);
                    de = a > de ? a : de;
                    de = b > de ? b : de;
                }
            }
        }
        if constexpr (AA) {
            // denominator T(V_(n-1)) given as its own half form (in D's registers)
            RW::inverse(dd, static_cast<const V*>(p.gT) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
            if (ri.valid) {
#pragma unroll
                for (int q = 0; q < E; ++q) {
                    const unsigned long long a = abs_bits((double)dd[q].x), b = abs_bits((double)dd[q].y);
                    de = a > de ? a : de;
                    de = b > de ? b : de;
                }
            }
        }
        block_reduce2_max_u64(nu, de);
        if (threadIdx.x == 0) {
            atomicMax(&ctl->slots->num[p.slot], nu);
            atomicMax(&ctl->slots->den[p.slot], de);
        }
    }
    if (!products) return;
    // eta^j V, delta^j d_x phi_b, delta^j d_y phi_b
    V w[E];
    RW::load(w, static_cast<const R*>(fam == 0 ? p.eta : p.delta) + po, ri.j, ri.valid);
    row_chain<RW, V, E>(v, w, ch * p.pc, min(p.J, (ch + 1) * p.pc), p.h + fam * p.J, hb, rc, lds_all, twN, twX);
}

template <typename R, int NX, int VAR>
__global__ void __launch_bounds__((row_threads<NX, RowVar<R, NX, VAR>::E>()), 3)
    k_row_sweep(const RowSweepParams p, const typename cplx_of<R>::type* twN_tab,
                const typename cplx_of<R>::type* twX_tab) {
    row_sweep_body<R, NX, false, VAR>(p, twN_tab, twX_tab);
}

// the same with the residual's denominator given as a third half form (Anderson mixing)
template <typename R, int NX, int VAR>
__global__ void __launch_bounds__((row_threads<NX, RowVar<R, NX, VAR>::E>()), 3)
    k_row_sweep_aa(const RowSweepParams p, const typename cplx_of<R>::type* twN_tab,
                   const typename cplx_of<R>::type* twX_tab) {
    row_sweep_body<R, NX, true, VAR>(p, twN_tab, twX_tab);
}

// nonlinear term of the potential equation; TANK adds the wave tank's surface
// pressures (a separate instance, so that the plain one keeps its registers)
template <typename R, int NX, bool TANK>
__device__ __forceinline__ void row_nphi_body(const RowNphiParams& p, const typename cplx_of<R>::type* twN_tab,
                                              const typename cplx_of<R>::type* twX_tab) {
    ROW_PROLOGUE(R, NX)
    V q[E], gg[E], pp[E], a[E], b[E];
    const V* gD = p.gD ? static_cast<const V*>(p.gD) + hb : nullptr;
    const R c2 = gD ? R(1.0 - p.ctl[ri.mem].omega) : R(0);
    RW::inverse(q, static_cast<const V*>(p.gV) + hb, gD, c2, rc, lds_all, twN, twX, iscale);
    RW::inverse(a, static_cast<const V*>(p.gex) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
    RW::inverse(b, static_cast<const V*>(p.gpx) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
    const double dx = p.g.lx / p.g.nx;
    // damping weight mu(x) of the wave tank times a potential gradient, in
    // place (the gradient is spent by then) -> forward half form
    auto damped = [&](V (&grad)[E], void* out) {
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int n = ri.j + k * RW::P;
            double mv[2];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const double d = fmod((2 * n + hh) * dx - p.dmp_x0 + 1.5 * p.g.lx, p.g.lx) - 0.5 * p.g.lx;
                mv[hh] = exp(-(d / p.dmp_w) * (d / p.dmp_w));
            }
            grad[k] = cx<V>(R(mv[0] * (double)grad[k].x), R(mv[1] * (double)grad[k].y));
        }
        RW::forward(grad, static_cast<V*>(out) + hb, rc, lds_all, twN, twX);
    };
#pragma unroll
    for (int k = 0; k < E; ++k) {
        q[k] = cx<V>(q[k].x + a[k].x * b[k].x, q[k].y + a[k].y * b[k].y);
        gg[k] = rmul(a[k], a[k]);
        pp[k] = rmul(b[k], b[k]);
    }
    if (p.g.ny > 1) {
        if constexpr (TANK)
            if (p.dmp_w > 0.0) damped(b, p.hdx);
        RW::inverse(a, static_cast<const V*>(p.gey) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
        RW::inverse(b, static_cast<const V*>(p.gpy) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
#pragma unroll
        for (int k = 0; k < E; ++k) {
            q[k] = cx<V>(q[k].x + a[k].x * b[k].x, q[k].y + a[k].y * b[k].y);
            gg[k] = cx<V>(gg[k].x + a[k].x * a[k].x, gg[k].y + a[k].y * a[k].y);
            pp[k] = cx<V>(pp[k].x + b[k].x * b[k].x, pp[k].y + b[k].y * b[k].y);
        }
    }
#pragma unroll
    for (int k = 0; k < E; ++k) {
        q[k] = cx<V>(R(0.5) * (q[k].x * q[k].x / (R(1) + gg[k].x) - pp[k].x),
                     R(0.5) * (q[k].y * q[k].y / (R(1) + gg[k].y) - pp[k].y));
    }
    // the last potential gradient (d_x phi in 1D, d_y phi in 2D), after the
    // products, when only q is live beside it
    if constexpr (TANK)
        if (p.dmp_w > 0.0) damped(b, p.g.ny > 1 ? p.hdy : p.hdx);
    if (TANK && p.wm_n > 0) {
        // pneumatic wavemaker: bell-shaped pressures centred on x = 0, i.e. split
        // over both ends of the periodic domain; the prefactor
        // a_j sqrt(e/(2 pi)) (1 + 2 k_j h / sinh(2 k_j h)) radiates waves of amplitude a_j
        const double hg = p.wm_h > 0.0 ? p.wm_h : p.g.href[ri.mem];
        double amp[kMaxWavemaker];
#pragma unroll
        for (int c = 0; c < kMaxWavemaker; ++c) {
            amp[c] = 0.0;
            if (c < p.wm_n) {
                const double kh2 = 2.0 * p.wm[c][1] * hg;
                const double G = kh2 < 700.0 ? kh2 / sinh(kh2) : 0.0;
                amp[c] = p.wm[c][0] * sqrt(M_E / (2.0 * M_PI)) * (1.0 + G) * sin(p.wm[c][2] * p.t + p.wm[c][3]);
            }
        }
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int n = ri.j + k * RW::P;
            double pg[2] = {0.0, 0.0};
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const double x = (2 * n + hh) * dx;
                const double xs = x < 0.5 * p.g.lx ? x : x - p.g.lx;
#pragma unroll
                for (int c = 0; c < kMaxWavemaker; ++c) {
                    if (c < p.wm_n) {
                        const double kx = p.wm[c][1] * xs;
                        pg[hh] += amp[c] * exp(-0.5 * kx * kx);
                    }
                }
            }
            q[k] = cx<V>(R((double)q[k].x - pg[0]), R((double)q[k].y - pg[1]));
        }
    }
    RW::forward(q, static_cast<V*>(p.h) + hb, rc, lds_all, twN, twX);
}

// (two wavefronts a SIMD: left to itself the compiler takes registers for one in FP64
// at 256 and 2048 points, for the reads in batches; 2048 x 64, 16 members 51 -> 37 us,
// 256 x 256, 32 members 38 -> 28)
template <typename R, int NX>
__global__ void __launch_bounds__(row_threads<NX>(), 2) k_row_nphi(const RowNphiParams p, const typename cplx_of<R>::type* twN_tab,
                           const typename cplx_of<R>::type* twX_tab) {
    row_nphi_body<R, NX, false>(p, twN_tab, twX_tab);
}

template <typename R, int NX>
__global__ void __launch_bounds__(row_threads<NX>()) k_row_nphi_tank(const RowNphiParams p,
                                                                     const typename cplx_of<R>::type* twN_tab,
                                                                     const typename cplx_of<R>::type* twX_tab) {
    row_nphi_body<R, NX, true>(p, twN_tab, twX_tab);
}

template <typename R, int NX>
__global__ void __launch_bounds__(row_threads<NX>()) k_row_blend(const RowBlendParams p, const typename cplx_of<R>::type* twN_tab,
                            const typename cplx_of<R>::type* twX_tab) {
    ROW_PROLOGUE(R, NX)
    const double dx = p.g.lx / p.g.nx;
    const double r = p.t < p.ramp_time ? 0.5 * (1.0 - cos(M_PI * p.t / p.ramp_time)) : 1.0;
    // the zones' reciprocal lengths, once: a division per point, unrolled over
    // the row's elements, would hold more registers than the transforms
    const double igen = p.gen > 0.0 ? 1.0 / p.gen : 0.0, iabs = p.absl > 0.0 ? 1.0 / p.absl : 0.0;
    // one field at a time (eta against a r cos, phi against a r / om sin), so
    // that a single row of values is live
    auto blend = [&](const void* in, void* out, bool pot) {
        V v[E];
        RW::inverse(v, static_cast<const V*>(in) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
        const double amp = pot ? p.a * r / p.om : p.a * r;
        // target a r cos(k x - om t) for eta and a r / om cos(k x - om t - pi/2)
        // for phi: one sincos at the thread's first point 2j, then rotations by
        // k dx (to point 2n + 1) and by 2 P k dx (to the next element), each
        // exact to rounding (the two fields' phases differ, so that the first
        // field's rotated values are not kept for the second)
        double c0, s0, ch, sh, cq, sq;
        sincos(p.k * (2 * ri.j) * dx - p.om * p.t - (pot ? 0.5 * M_PI : 0.0), &s0, &c0);
        sincos(p.k * dx, &sh, &ch);
        sincos(p.k * (2 * RW::P) * dx, &sq, &cq);
#pragma unroll
        for (int q = 0; q < E; ++q) {
            const int n = ri.j + q * RW::P;
            double fv[2] = {(double)v[q].x, (double)v[q].y};
            double c = c0, sn = s0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const double x = (2 * n + h) * dx;
                double wg = 0.0, wa = 0.0;
                if (x < p.gen) {
                    const double s = x * igen;
                    wg = 1.0 - (3 * s * s - 2 * s * s * s);
                }
                if (x > p.g.lx - p.absl) {
                    const double s = (p.g.lx - x) * iabs;
                    wa = 1.0 - (3 * s * s - 2 * s * s * s);
                }
                fv[h] = (1.0 - wg) * fv[h] + wg * (amp * c);
                fv[h] *= (1.0 - wa);
                const double cn = c * ch - sn * sh;
                sn = sn * ch + c * sh;
                c = cn;
            }
            const double cn = c0 * cq - s0 * sq;
            s0 = s0 * cq + c0 * sq;
            c0 = cn;
            v[q] = cx<V>(R(fv[0]), R(fv[1]));
        }
        RW::forward(v, static_cast<V*>(out) + hb, rc, lds_all, twN, twX);
    };
    blend(p.ge, p.he, false);
    blend(p.gp, p.hp, true);
}

// Learned-warm-start features of each point, channel-last FP32:
// (eta, W_lin, d_x eta, d_y eta, d_x phi, d_y phi, delta, eta * W_lin), each
// multiplied by its channel scale in the working precision before rounding.
template <typename R, int NX>
__global__ void __launch_bounds__(row_threads<NX>()) k_row_feat(const RowFeatParams p, const typename cplx_of<R>::type* twN_tab,
                           const typename cplx_of<R>::type* twX_tab) {
    ROW_PROLOGUE(R, NX)
    V wl[E], a[E];
    RW::inverse(wl, static_cast<const V*>(p.gV) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
    if (p.wlin) RW::store(wl, static_cast<R*>(p.wlin) + po, ri.j, ri.valid);
    float2 fe[4][E];
    const void* src[4] = {p.gex, p.gey, p.gpx, p.gpy};
    const int ch[4] = {2, 3, 4, 5};
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        RW::inverse(a, static_cast<const V*>(src[f]) + hb, nullptr, R(0), rc, lds_all, twN, twX, iscale);
        const R sc = R(p.scale[ch[f]]);
#pragma unroll
        for (int q = 0; q < E; ++q) fe[f][q] = make_float2((float)(a[q].x * sc), (float)(a[q].y * sc));
    }
    if (!ri.valid) return;  // after the last workgroup barrier
    V ev[E], dv[E];
    RW::load(ev, static_cast<const R*>(p.eta) + po, ri.j, true);
    RW::load(dv, static_cast<const R*>(p.delta) + po, ri.j, true);
    const R s0 = R(p.scale[0]), s1 = R(p.scale[1]), s6 = R(p.scale[6]), s7 = R(p.scale[7]);
    float4* out = reinterpret_cast<float4*>(p.feat + po * 8);
#pragma unroll
    for (int q = 0; q < E; ++q) {
        const int n = ri.j + q * RW::P;  // points 2n and 2n + 1 of the row
        out[4 * n + 0] = make_float4((float)(ev[q].x * s0), (float)(wl[q].x * s1), fe[0][q].x, fe[1][q].x);
        out[4 * n + 1] = make_float4(fe[2][q].x, fe[3][q].x, (float)(dv[q].x * s6), (float)(ev[q].x * wl[q].x * s7));
        out[4 * n + 2] = make_float4((float)(ev[q].y * s0), (float)(wl[q].y * s1), fe[0][q].y, fe[1][q].y);
        out[4 * n + 3] = make_float4(fe[2][q].y, fe[3][q].y, (float)(dv[q].y * s6), (float)(ev[q].y * wl[q].y * s7));
    }
}

// ---------------------------------------------------------------------------
// Column pass: forward column transforms of the products, multiplier sums,
// relaxation, compact outputs, inverse column transforms of the results.
//
// A workgroup owns the columns of one wavefront's transform (ColShape::CW of
// them; a single one from 512 rows on) and the kept modes in them.  Its
// wavefronts take the products as jobs, one column transform each, which never
// leave the wavefront; after a round of transforms the kept values stand in
// the wavefronts' LDS areas, and each thread -- the owner of one kept mode --
// adds the round's products to its mode's sums, the multipliers formed once
// per mode and product with the term's exponents in scalar registers.  The
// next round's columns are requested before the sums, so the loads run under
// them.  The owners read and write the compact fields themselves (one
// contiguous run per column) and hand the wavefronts the spectra of the
// inverse transforms through the same areas.
//
// What bounds it: at 1024 rows the transforms' issue and LDS exchanges, on
// small grids the chain of dependent loads and barriers of one workgroup.
// Measured per launch, against one whose transform threads also formed the sums
// of the modes they held: FP64 1024 x 1024 sweep 36 us (37, and 5.6 for the
// inner products in a kernel of their own), its inverse pass 15.4 (17.5); FP32
// 512 x 512 SA order 7.6 (21.7); FP64 128 x 64 sweep 14.6 (31); a single product
// without inverse at 1024 rows 6.9 (11.8).
//
// S ("classes"): columns of more than 512 rows are split by decimation in frequency
// into S = ny / 512 transforms of 512 points, one wavefront each: wave h forms u_h[n]
// = sum_p x[n + 512 p] W_S^(h p) W^(h n), W = exp(-2 pi i / ny), whose transform holds
// the modes S k + h. Both waves of S = 2 read the whole column (the second reads are
// served by the cache). Four would read it four times and hold no next round's values:
// there wave q loads the positions n of its quarter of the 512, forms u_0 .. u_3 from
// them and leaves each in its class's area, so that a value is read once and requested
// a round ahead (16 members of 16 x 2048, FP64: a sweep's pass 46 us, 103 with four
// reads; FP32 28 against 61). The inverse runs the other way: each wave inverts its
// class of modes, multiplies by W^(-h n), and the S waves form x[n + 512 p] = sum_h
// W_S^(-h p) e_h[n] through LDS (four classes: wave q those of its quarter, for every
// p).
// ---------------------------------------------------------------------------
template <typename R, int NY> struct ColShape {
    using V = typename cplx_of<R>::type;
    static constexpr int S = NY <= 512 ? 1 : NY / 512;
    static constexpr int NH = NY / S;
    static constexpr int E = FftShape<NH>::E;
    static constexpr int P = NH / E;
    static constexpr int CW = 64 / P;   // columns per workgroup
    static constexpr int REG = fft_lds_elems<NH, E>();
    // a wavefront's LDS area; the areas of the S classes of a column start
    // 256 / S bytes apart modulo the banks, so that consecutive modes, which
    // alternate between the classes, are read without conflicts
    static constexpr int AREA = CW * REG + (S > 1 ? 256 / S / (int)sizeof(V) : 0);
    // wavefronts of a workgroup at most: twelve leave each thread 168 registers, which
    // hold the next round's column in FP64 too, but for 7 registers of a sweep and 47 of
    // the state pass at 1024 rows, and 13 to 23 at 2048 rows with two modes an owner
    static constexpr int WMAX = 12;
    // kept modes per owner thread when all of a column's are kept: 1 below 1024 rows,
    // 2 at 1024 and 3 at 2048 rows, where half bands take 1 and 2
    static constexpr int ITMAX = (CW * (NY - 1) + 64 * WMAX - 1) / (64 * WMAX);
    static_assert(WMAX % S == 0 && WMAX * AREA * sizeof(V) + 4096 <= kMaxLdsBytes, "the workgroup's LDS");
};

// Sweep control of a column pass: decides the solve from the previous
// sweep's residual (false: this launch has nothing to do) and gives the
// relaxation weight; the leader thread updates the control header.
__device__ __forceinline__ bool col_control(const ColParams& p, Ctl* ctl, bool leader, double* omega) {
    const GridDev& g = p.g;
    if (p.ctl_mode == CTL_SWEEP) {
        if (ctl->done) return false;
        double r, rmin;
        const int dec = sweep_decision(ctl, p.sweep, p.max_sweeps, p.tol, &r, &rmin);
        if (dec) {
            if (leader) ctl_commit(ctl, dec - 100, p.sweep, r);
            return false;
        }
        if (leader) {
            ctl->rmin = rmin;
            ctl->residual = r;
        }
        *omega = ctl->omega;
    } else if (p.ctl_mode == CTL_SKIP) {
        if (ctl->done) return false;
        *omega = ctl->omega;
    } else if (p.ctl_mode == CTL_OMEGA) {
        // relaxation weight from the local symbol sum_{j<=J} (k eta)^j / j!
        const double emax = unord_bits(ctl->eta_max), emin = unord_bits(ctl->eta_min);
        const int J = g.order - 1;
        double w = 1.0;
        if (g.relax && J >= 1) {
            double lmax = 0.0, lmin = 0.0, tmax = 1.0, tmin = 1.0;
            const double xmax = g.kband * emax, xmin = g.kband * emin;
            for (int jj = 0; jj <= J; ++jj) {
                if (jj > 0) {
                    tmax *= xmax / jj;
                    tmin *= xmin / jj;
                }
                lmax += tmax;
                lmin += tmin;
            }
            const double s = lmin + lmax;
            if (isfinite(s) && s > 0.0) w = fmin(1.0, 2.0 / s);
        }
        *omega = w;
        if (leader) ctl->omega = w;
    }
    return true;
}

// geometry of one kept mode
template <typename R> struct ColGeo {
    R k, ik, T, S, kx, ky;   // ik: 1 / k, 0 at k = 0
};
// (mx, r): column and compact row; T = tanh(kh) and S = sech(kh) only when
// the pass uses them
template <typename R>
__device__ __forceinline__ ColGeo<R> col_geo(const ColParams& p, int mx, int r, double href) {
    const GridDev& g = p.g;
    const int my = r <= g.My ? r : r - g.Ky;
    const double kx = 2.0 * M_PI * (double)mx / g.lx;
    const double ky = (g.ny == 1) ? 0.0 : 2.0 * M_PI * (double)my / g.ly;
    const double k = sqrt(kx * kx + ky * ky);
    ColGeo<R> o;
    o.k = R(k);
    o.ik = k > 0.0 ? R(1) / R(k) : R(0);
    o.T = o.S = R(1);
    if (p.hyper) {
        o.T = R(tanh(k * href));
        o.S = R(sech_d(k * href));
    }
    o.kx = R(kx);
    o.ky = R(ky);
    return o;
}

// A pass's parameters are staged in LDS by one parallel load: read where they
// are needed, each source's description would cost a dependent miss of the
// scalar cache (the kernel arguments are new to it in every launch).
__device__ __forceinline__ void col_stage(const ColParams& p, ColParams* sp) {
    const int* src = reinterpret_cast<const int*>(&p);
    int* dst = reinterpret_cast<int*>(sp);
    for (int i = threadIdx.x; i < (int)(sizeof(ColParams) / 4); i += blockDim.x) dst[i] = src[i];
}
// a source's description; every thread reads the same one, so what steers
// branches goes to scalar registers
__device__ __forceinline__ ColSrc col_src(const ColSrc* s) {
    ColSrc o = *s;
    int ctl[2];
    __builtin_memcpy(ctl, o.acc, 8);
    ctl[0] = __builtin_amdgcn_readfirstlane(ctl[0]);
    ctl[1] = __builtin_amdgcn_readfirstlane(ctl[1]);
    __builtin_memcpy(o.acc, ctl, 8);
    return o;
}
__device__ __forceinline__ int col_uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T> __device__ __forceinline__ T* col_uni(T* ptr) {
    const unsigned long long a = (unsigned long long)ptr;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)a);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(a >> 32));
    return reinterpret_cast<T*>(((unsigned long long)hi << 32) | lo);
}

// Adds a source's terms to the sums of one mode: acc[t.acc] += coef fn(k) k^pw
// (i kx or i ky) val for its at most two terms (the branches are uniform).
template <typename R, typename V, int NACC>
__device__ __forceinline__ void col_add(const ColSrc& s, V val, V (&acc)[NACC], const ColGeo<R>& q) {
    if (s.dv == DV_X) val = mul_i(cscale(val, q.kx));
    else if (s.dv == DV_Y) val = mul_i(cscale(val, q.ky));
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        if (s.acc[t] < 0) continue;
        R m = R(s.coef[t]);
        if (s.fn[t] == FN_T) m *= q.T;
        else if (s.fn[t] == FN_S) m *= q.S;
        const int pw = s.pw[t];
        if (pw < 0) {
            m *= q.ik;
        } else {
            if (pw & 1) m *= q.k;
            if (pw & 2) m *= q.k * q.k;
            if (pw & 4) m *= (q.k * q.k) * (q.k * q.k);
        }
#pragma unroll
        for (int a = 0; a < NACC; ++a)
            if (a == s.acc[t]) acc[a] = cx<V>(acc[a].x + val.x * m, acc[a].y + val.y * m);
    }
}

// The products of a sweep (ColParams::nfam), value F of order j and family f, the
// same in every thread:
//     eta^j V:                  V -= <odd: T> k^j / j! F,          phi_b -= <odd> S k^(j-1) / j! F
//     delta^j d_x,y phi_b:      D = i k_x,y F;  V += <odd> S k^(j-1) / j! D,
//                               phi_b -= <odd: T, even: -1> k^(j-2) / j! D
// kq: k^(j-2), carried from order to order.  Read from the sources' descriptions,
// a term is a chain of branches and LDS reads: the sums of a sweep (FP64, the
// waits for the slowest transform included) took 8.0 us at 128 x 64 and 13.4 us at
// 1024 x 1024; this way 4.9 and 10.4.
static __constant__ double kSweepFact[7] = {1.0, 1.0, 1.0 / 2.0, 1.0 / 6.0, 1.0 / 24.0, 1.0 / 120.0, 1.0 / 720.0};
template <typename R, typename V, int NACC>
__device__ __forceinline__ void col_sweep_add(int j, int f, R fact, V F, V (&acc)[NACC], R& kq, const ColGeo<R>& g) {
    const bool odd = j & 1;
    if (f == 0) kq = j == 1 ? g.ik : (j == 2 ? R(1) : kq * g.k);
    const R kp = (j == 1 ? R(1) : kq * g.k) * fact;  // k^(j-1) / j!
    if (f == 0) {
        const R m = kp * g.k * (odd ? g.T : R(1));
        acc[0] = cx<V>(acc[0].x - F.x * m, acc[0].y - F.y * m);
        if (NACC > 1 && odd) {
            const R s = kp * g.S;
            acc[NACC - 1] = cx<V>(acc[NACC - 1].x - F.x * s, acc[NACC - 1].y - F.y * s);
        }
    } else {
        const V D = mul_i(cscale(F, f == 1 ? g.kx : g.ky));
        if (odd) {
            const R s = kp * g.S;
            acc[0] = cx<V>(acc[0].x + D.x * s, acc[0].y + D.y * s);
        }
        const R m = kq * fact * (odd ? -g.T : R(1));
        if (NACC > 1) acc[NACC - 1] = cx<V>(acc[NACC - 1].x + D.x * m, acc[NACC - 1].y + D.y * m);
    }
}

// value of output source `src` of one mode; pv: the previous iterates
template <typename V, int NACC>
__device__ __forceinline__ V col_source(int src, const V (&acc)[NACC], const V (&pv)[2], decltype(V::x) omega) {
    const bool relaxed = src >= SRC_NEW0;
    const int a = relaxed ? ((src == SRC_NEW0 || src == SRC_DIFF0) ? 0 : 1) : src;
    V cur = cx<V>(0, 0);
#pragma unroll
    for (int k = 0; k < NACC; ++k)
        if (k == a) cur = acc[k];
    if (!relaxed) return cur;
    const V pq = a == 0 ? pv[0] : pv[1];
    const V d = csub(cur, pq);
    return src >= SRC_DIFF0 ? d : cadd(pq, cscale(d, omega));
}

// inner products of the residual history for the Anderson mixing, formed by
// the sweep's own owners: d[i] += wt <F_i, f_n> of one mode over the ring slots
// of sweep n (f: f_n's V and phi_b parts, old: those of the two sweeps before)
template <typename V>
__device__ __forceinline__ void col_aa_old(const ColParams& p, long long o, V (&old)[kAADepth][2]) {
#pragma unroll
    for (int j = 1; j <= kAADepth; ++j)
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            old[j - 1][part] = cx<V>(0, 0);
            if (j <= p.sweep && p.aa_f[part][0])
                old[j - 1][part] = static_cast<const V*>(p.aa_f[part][(p.sweep - j) % kAASlots])[o];
        }
}
template <typename V>
__device__ __forceinline__ void col_aa_dots(const ColParams& p, const V (&f)[2], const V (&old)[kAADepth][2], double wt,
                                            double (&d)[kAASlots]) {
    const int n = p.sweep;
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        if (part == 1 && !p.aa_f[1][0]) break;
        const V f0 = f[part];
#pragma unroll
        for (int j = 0; j <= kAADepth; ++j) {
            if (j > n) break;
            const int si = (n - j) % kAASlots;
            const V fj = j == 0 ? f0 : old[j - 1][part];
            const double v = wt * ((double)fj.x * (double)f0.x + (double)fj.y * (double)f0.y);
#pragma unroll
            for (int i = 0; i < kAASlots; ++i)
                if (i == si) d[i] += v;
        }
    }
}

// (16 rows: four wavefronts a SIMD, whose loads in flight cover the latency; with three
// 256 x 16 FP64, 512 members, took 41 us a sweep's pass, now 38)
template <typename R, int NY, int NACC, int IT>
__global__ void __launch_bounds__((64 * ColShape<R, NY>::WMAX), (NY <= 16 && NACC <= 2 ? 4 : 1)) k_col(const ColParams p, const typename cplx_of<R>::type* __restrict__ twY) {
    using CS = ColShape<R, NY>;
    using V = typename CS::V;
    constexpr int S = CS::S, NH = CS::NH, E = CS::E, P = CS::P, CW = CS::CW, REG = CS::REG, AREA = CS::AREA;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    __shared__ double s_aa[(16 + 1) * kAASlots];  // wavefront sums, then the Anderson weights
    __shared__ ColParams sp;
    V* const areas = reinterpret_cast<V*>(smem_raw);
    const int t = threadIdx.x;
    const int W = blockDim.x >> 6;                             // a multiple of S
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int ln = t & 63;
    const int c = ln / P, j = ln % P;                          // column of the workgroup, thread of the column
    const int h = S > 1 ? wv % S : 0;                          // class of modes of this wavefront
    const int mem = blockIdx.z;
    const int x0 = blockIdx.x * CW;
    const GridDev& g = p.g;
    const ColSub& sub = p.sub[blockIdx.y];
    Ctl* ctl = p.ctl ? p.ctl + mem : nullptr;
    if ((p.ctl_mode == CTL_SWEEP || p.ctl_mode == CTL_SKIP) && ctl->done) return;
    col_stage(p, &sp);

    const int np = sub.p1 - sub.p0;
    const int njob = np * S;
    const int rounds = (njob + W - 1) / W;
    const int per = W / S;                                     // products per round
    // column of job jb (product jb / S): the raw values of its thread
    // (not for columns of several modes an owner in FP64: their registers hold those)
    constexpr bool SPREAD = S > 2;   // each value read by one wavefront of the column, see above
    static_assert(!SPREAD || (S == 4 && P == 64 && E % S == 0), "the radix-4 step of a spread column");
    constexpr bool AHEAD = S == 1 || SPREAD || IT == 1 || sizeof(R) == 4;
    constexpr int RAW = AHEAD ? (SPREAD ? 1 : S) : 1;
    V raw[RAW][E];
    auto column = [&](int jb) __attribute__((always_inline)) {
        return static_cast<const V*>(jb < W ? p.src[sub.p0 + jb / S].ptr : col_uni(sp.src[sub.p0 + jb / S].ptr)) + mem * g.s_half + (long long)(x0 + c) * g.ldh + j;
    };
    auto request = [&](int jb) __attribute__((always_inline)) {
        if constexpr (SPREAD) {
            const V* H = column(jb) + h * (NH / S);
#pragma unroll
            for (int q = 0; q < E; ++q) raw[0][q] = H[(q / S) * P + (q % S) * NH];
        } else if constexpr (AHEAD) {
            const V* H = column(jb);
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int q = 0; q < E; ++q) raw[s][q] = H[q * P + s * NH];
        }
    };
    if (wv < njob) request(wv);
    // compact inputs an owner of one mode loads ahead of their use, into the
    // columns' registers: in a pass without products before everything else
    constexpr bool EARLY = IT == 1 && AHEAD;
    constexpr int kPre = !EARLY ? 0 : (RAW * E < 6 ? RAW * E : 6);
    const int nc = sub.c1 - sub.c0;
    auto preload = [&](long long o, bool on) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < kPre; ++s)
            raw[s / E][s % E] = s < nc && on ? static_cast<const V*>(p.src[kMaxProd + sub.c0 + s].ptr)[o] : cx<V>(R(0), R(0));
    };
    Twid<V, NH, E> twc;
    twc.load(twY, j, S);                                       // the NH-point twiddles: every S-th entry
    V wn = cx<V>(R(1), R(0)), wq = wn;                         // W^(h j), W^(h P)
    if constexpr (S == 2) {
        wn = twY[h * j];
        wq = twY[h * P];
    }
    V ws[SPREAD ? E / S : 1];                                  // W^n of the thread's positions of the radix-4 step
    if constexpr (SPREAD) {
#pragma unroll
        for (int r = 0; r < E / S; ++r) ws[r] = twY[h * (NH / S) + j + r * P];
    }
    // the owner's mode(s): entry i = t + it owners of the workgroup's compact modes.  The owners'
    // number follows from the band alone, not from the wavefronts of the launch, which follow from
    // the member count too: a member's inner products are to round alike among many and alone
    const int owners = IT == 1 ? 0 : (CW * g.Ky + 64 * IT - 1) / (64 * IT) * 64;
    const double href = g.href[mem];
    ColGeo<R> geo[IT];
    int slot[IT];          // element of the areas holding the mode: class area, column, transform index (0: no mode,
                           // so that a thread without one reads inside the areas too)
    int co[IT];            // compact offset from the workgroup's first column, -1: no mode
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int i = t + it * owners;
        const int c2 = i / g.Ky, r = i - c2 * g.Ky;
        const bool on = (IT == 1 || t < owners) && c2 < CW && x0 + c2 < g.Kx;
        const int n = r <= g.My ? r : r + NY - g.Ky;
        co[it] = on ? i : -1;
        slot[it] = on ? (n % S) * AREA + c2 * REG + n / S : 0;
        geo[it] = col_geo<R>(p, x0 + c2, r, href);
    }
    const long long cb = mem * g.s_cmp + (long long)x0 * g.Ky;  // compact base of the workgroup
    if (njob == 0) preload(cb + co[0], co[0] >= 0);
    double head[kAASlots] = {};
    if (p.aa_partial) aa_head(p, mem, head);
    double omega = 1.0;
    // the decision is the same in every thread (the leader's header updates
    // cannot change it), so the workgroup returns as a whole
    if (!col_control(p, ctl, blockIdx.x == 0 && blockIdx.y == 0 && t == 0, &omega)) return;
    if (p.aa_partial) aa_block_weights(p, ctl, mem, blockIdx.x == 0, head, s_aa, s_aa + 16 * kAASlots);

    V acc[IT][NACC];
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
        for (int a = 0; a < NACC; ++a) acc[it][a] = cx<V>(R(0), R(0));
    R kq[IT];              // power of k carried over a sweep's products
    int sj = 1, sf = 0;    // their order and family
    const int nfam = p.nfam;
#pragma unroll
    for (int it = 0; it < IT; ++it) kq[it] = R(0);

    V* const area = areas + wv * AREA;
    lds_sync();  // the staged parameters: every wavefront's part of them is written
    for (int rd = 0; rd < rounds; ++rd) {
        const int jb = rd * W + wv;
        if constexpr (SPREAD) {
            if (jb < njob) {
                V* const cls = areas + (wv - h) * AREA + h * (NH / S) + j;
#pragma unroll
                for (int r = 0; r < E / S; ++r) {
                    const V* x = &raw[0][r * S];
                    const V a = cadd(x[0], x[2]), b = csub(x[0], x[2]), e = cadd(x[1], x[3]);
                    const V d = mul_mi<false>(csub(x[1], x[3]));
                    V w = ws[r];
                    asm volatile("" : "+v"(w.x), "+v"(w.y));  // powers formed here, not held across rounds
                    const V w2 = cmul(w, w);
                    cls[0 * AREA + r * P] = cadd(a, e);
                    cls[1 * AREA + r * P] = cmul(cadd(b, d), w);
                    cls[2 * AREA + r * P] = cmul(csub(a, e), w2);
                    cls[3 * AREA + r * P] = cmul(csub(b, d), cmul(w2, w));
                }
            }
            lds_sync();  // every part of the column's classes is written
        }
        if (jb < njob) {
            V v[E];
            if constexpr (S == 1) {
#pragma unroll
                for (int q = 0; q < E; ++q) v[q] = raw[0][q];
            } else if constexpr (SPREAD) {
#pragma unroll
                for (int q = 0; q < E; ++q) v[q] = area[j + q * P];
                wave_lds_sync();
            } else {
                if constexpr (AHEAD) {
                    if (h == 0) {
#pragma unroll
                        for (int q = 0; q < E; ++q) v[q] = cadd(raw[0][q], raw[1][q]);
                    } else {
#pragma unroll
                        for (int q = 0; q < E; ++q) v[q] = csub(raw[0][q], raw[1][q]);
                    }
                } else {
                    const V* H = column(jb);
#pragma unroll
                    for (int q = 0; q < E; ++q) v[q] = H[q * P];
#pragma unroll
                    for (int q = 0; q < E; ++q) {
                        const V x = H[q * P + NH];
                        v[q] = h == 0 ? cadd(v[q], x) : csub(v[q], x);
                    }
                }
                if (h > 0) {
                    V w = wn;
                    asm volatile("" : "+v"(w.x), "+v"(w.y));  // powers formed here, not held across rounds
#pragma unroll
                    for (int q = 0; q < E; ++q) {
                        v[q] = cmul(v[q], w);
                        w = cmul(w, wq);
                    }
                }
            }
            fft<V, NH, false, 1, E, true>(v, area + c * REG, 0, j, twc);
            wave_lds_sync();
#pragma unroll
            for (int q = 0; q < E; ++q) area[c * REG + j + q * P] = v[q];
        }
        if (jb + W < njob) request(jb + W);
        lds_sync();
        const int s0 = rd * per, s1 = min(np, s0 + per);
        if (NACC <= 2 && nfam > 0) {
            V F[IT];
#pragma unroll
            for (int it = 0; it < IT; ++it) F[it] = areas[slot[it]];
            for (int s = s0; s < s1; ++s) {
                V nx[IT];  // the next product's values, on their way over this one's sums
#pragma unroll
                for (int it = 0; it < IT; ++it) nx[it] = areas[(min(s + 1, s1 - 1) - s0) * S * AREA + slot[it]];
                const R fact = R(kSweepFact[sj]);
#pragma unroll
                for (int it = 0; it < IT; ++it) col_sweep_add<R, V, NACC>(sj, sf, fact, F[it], acc[it], kq[it], geo[it]);
                if (++sf == nfam) {
                    sf = 0;
                    ++sj;
                }
#pragma unroll
                for (int it = 0; it < IT; ++it) F[it] = nx[it];
            }
            lds_sync();
            continue;
        }
#pragma unroll 2
        for (int s = s0; s < s1; ++s) {
            const ColSrc src = col_src(&sp.src[sub.p0 + s]);
#pragma unroll
            for (int it = 0; it < IT; ++it)
                if (co[it] >= 0) col_add<R, V, NACC>(src, areas[(s - s0) * S * AREA + slot[it]], acc[it], geo[it]);
        }
        lds_sync();
    }
    // what the owners read from here on, requested at once
    if (njob > 0) preload(cb + co[0], co[0] >= 0);
    V pv[IT][2], old[IT][kAADepth][2];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
            pv[it][a] = (p.prev[a] && co[it] >= 0) ? static_cast<const V*>(p.prev[a])[cb + co[it]] : cx<V>(R(0), R(0));
        if (EARLY && p.aa_dots && co[it] >= 0) col_aa_old<V>(p, cb + co[it], old[it]);
    }
    // a mixing pass's sums and a sweep's forcing need no descriptions (decoded, an
    // input costs some 0.4 us; a mixing pass of 128 x 64 FP64 took 10.6 us, now 8.8,
    // of 1024 x 1024 17.8, now 15.4)
    const int kmix = kPre >= 2 * kAASlots && NACC <= 2 ? p.nmix : 0;
    const bool forced = kPre >= 2 && NACC <= 2 && nfam > 0;
    if constexpr (kPre >= 2) {
        if (kmix > 0) {
#pragma unroll
            for (int a = 0; a < (kPre >= 2 * kAASlots ? kAASlots : 0); ++a) {
                if (a >= kmix) break;
                const R w = R(s_aa[16 * kAASlots + (p.aa_sweep - kmix + 1 + a) % kAASlots]);
                if (NACC == 1) {
                    acc[0][0] = cadd(acc[0][0], cscale(raw[a / E][a % E], w));
                } else {
                    acc[0][0] = cadd(acc[0][0], cscale(raw[2 * a / E][2 * a % E], w));
                    acc[0][NACC - 1] = cadd(acc[0][NACC - 1], cscale(raw[(2 * a + 1) / E][(2 * a + 1) % E], w));
                }
            }
        } else if (forced) {
            acc[0][0] = cadd(acc[0][0], raw[0][0]);
            if (NACC > 1) acc[0][NACC - 1] = cadd(acc[0][NACC - 1], raw[1 / E][1 % E]);
        }
    }
#pragma unroll
    for (int s = 0; s < kPre; ++s) {
        if (s >= nc || kmix > 0 || forced) break;
        const ColSrc src = col_src(&sp.src[kMaxProd + sub.c0 + s]);
        const R cw = src.widx >= 0 ? R(s_aa[16 * kAASlots + src.widx]) : R(1);
        if (co[0] >= 0) col_add<R, V, NACC>(src, cscale(raw[s / E][s % E], cw), acc[0], geo[0]);
    }
#pragma unroll 2
    for (int s = sub.c0 + kPre; s < sub.c1; ++s) {
        const ColSrc src = col_src(&sp.src[kMaxProd + s]);
        const R cw = src.widx >= 0 ? R(s_aa[16 * kAASlots + src.widx]) : R(1);
#pragma unroll
        for (int it = 0; it < IT; ++it)
            if (co[it] >= 0)
                col_add<R, V, NACC>(src, cscale(static_cast<const V*>(col_uni(src.ptr))[cb + co[it]], cw), acc[it],
                                    geo[it]);
    }

    // inverse column transforms, W / S outputs a round
    V* const ownarea = areas;
    const int ninv = sub.i1 - sub.i0;
    for (int o0 = 0; o0 < ninv; o0 += per) {
        if (o0 > 0) lds_sync();  // the last round's areas have been read
        const int on = min(per, ninv - o0);
        for (int o = 0; o < on; ++o) {
            const int isrc = col_uni(sp.inv_src[sub.i0 + o0 + o]), dv = col_uni(sp.inv_dv[sub.i0 + o0 + o]);
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                if (co[it] < 0) continue;
                V sv = col_source<V, NACC>(isrc, acc[it], pv[it], R(omega));
                if (dv == DV_X) sv = mul_i(cscale(sv, geo[it].kx));
                else if (dv == DV_Y) sv = mul_i(cscale(sv, geo[it].ky));
                ownarea[o * S * AREA + slot[it]] = sv;
            }
        }
        lds_sync();
        const int o = wv / S;
        V v[E];
        if (o < on) {
#pragma unroll
            for (int q = 0; q < E; ++q) {
                const int n = S * (j + q * P) + h;
                const int my = n <= NY / 2 ? n : n - NY;
                const bool keep = x0 + c < g.Kx && my <= g.My && my >= -g.My;
                v[q] = keep ? area[c * REG + j + q * P] : cx<V>(R(0), R(0));
            }
            wave_lds_sync();
            fft<V, NH, true, 1, E, true>(v, area + c * REG, 0, j, twc);
            if constexpr (S > 1) {
                if (!SPREAD && h > 0) {
                    V w = cconj(wn);
                    asm volatile("" : "+v"(w.x), "+v"(w.y));
                    const V wc = cconj(wq);
#pragma unroll
                    for (int q = 0; q < E; ++q) {
                        v[q] = cmul(v[q], w);
                        w = cmul(w, wc);
                    }
                }
                wave_lds_sync();
#pragma unroll
                for (int q = 0; q < E; ++q) area[j + q * P] = v[q];
            }
        }
        V* const G = o < on ? static_cast<V*>(col_uni(sp.inv[sub.i0 + o0 + o])) + mem * g.s_half + (long long)(x0 + c) * g.ldh : nullptr;
        if constexpr (SPREAD) {
            lds_sync();
            if (o < on) {
                const V* const e = areas + o * S * AREA + h * (NH / S) + j;
                V* const x = G + h * (NH / S) + j;
#pragma unroll
                for (int r = 0; r < E / S; ++r) {
                    V w = cconj(ws[r]);
                    asm volatile("" : "+v"(w.x), "+v"(w.y));
                    const V w2 = cmul(w, w);
                    const V e0 = e[r * P], e1 = cmul(e[AREA + r * P], w), e2 = cmul(e[2 * AREA + r * P], w2);
                    const V e3 = cmul(e[3 * AREA + r * P], cmul(w2, w));
                    const V a = cadd(e0, e2), b = csub(e0, e2), d = cadd(e1, e3), f = mul_i(csub(e1, e3));
                    x[r * P] = cadd(a, d);
                    x[NH + r * P] = cadd(b, f);
                    x[2 * NH + r * P] = csub(a, d);
                    x[3 * NH + r * P] = csub(b, f);
                }
            }
        } else if constexpr (S > 1) {
            lds_sync();
            if (o < on) {
                const V* const e = areas + o * S * AREA;
#pragma unroll
                for (int q = 0; q < E; ++q) {
                    const V a = e[j + q * P], b = e[AREA + j + q * P];
                    v[q] = h == 0 ? cadd(a, b) : csub(a, b);
                }
            }
        }
        if (!SPREAD && o < on) {
#pragma unroll
            for (int q = 0; q < E; ++q) G[h * NH + j + q * P] = v[q];
        }
    }
    // compact outputs: a mode's inputs were all read by its owner, so an output
    // may overwrite an input of the same pass
    for (int o = sub.o0; o < sub.o1; ++o) {
        V* const out = static_cast<V*>(col_uni(sp.cout[o])) + cb;
        const int src = col_uni(sp.cout_src[o]);
#pragma unroll
        for (int it = 0; it < IT; ++it)
            if (co[it] >= 0) out[co[it]] = col_source<V, NACC>(src, acc[it], pv[it], R(omega));
    }
    if (p.aa_dots) {
        double d[kAASlots];
#pragma unroll
        for (int i = 0; i < kAASlots; ++i) d[i] = 0.0;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            if (co[it] < 0) continue;
            const V f[2] = {col_source<V, NACC>(SRC_DIFF0, acc[it], pv[it], R(1)),
                            col_source<V, NACC>(SRC_DIFF1, acc[it], pv[it], R(1))};
            const int mx = x0 + co[it] / g.Ky;
            if (!EARLY) col_aa_old<V>(p, cb + co[it], old[it]);
            col_aa_dots<V>(p, f, old[it], mx == 0 ? 1.0 : 2.0, d);
        }
        col_aa_reduce(d, s_aa, p.aa_dots + ((long long)mem * gridDim.x + blockIdx.x) * kAASlots);
    }
}

// Column pass of one-dimensional grids: a "column" is one mode, so a thread
// reads its mode of a source itself.  Bound by the latency of one chain (control
// header, parameters, loads, sums, store); the sources are shared by up to
// eight lanes whose partial sums meet in LDS, a lane taking every lanes-th
// source.  A wavefront serves one lane or several in turn (col1_waves): the
// lanes, and with them the rounding, do not depend on the number of members.
constexpr int kCol1Lanes = 8;
template <typename R, int NACC>
__global__ void __launch_bounds__(64 * kCol1Lanes) k_col1(const ColParams p) {
    using V = typename cplx_of<R>::type;
    __shared__ double s_aa[(16 + 1) * kAASlots];
    __shared__ ColParams sp;
    __shared__ V sums[kCol1Lanes - 1][NACC][64];
    const int t = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), W = blockDim.x >> 6;
    const int mem = blockIdx.z;
    const int mx = blockIdx.x * 64 + t;
    const GridDev& g = p.g;
    const ColSub& sub = p.sub[blockIdx.y];
    Ctl* ctl = p.ctl ? p.ctl + mem : nullptr;
    if ((p.ctl_mode == CTL_SWEEP || p.ctl_mode == CTL_SKIP) && ctl->done) return;
    col_stage(p, &sp);
    const bool on = mx < g.Kx;
    const long long cb = mem * g.s_cmp + mx, hb = mem * g.s_half + mx;
    const V zero = cx<V>(R(0), R(0));
    V pv[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) pv[a] = (p.prev[a] && on) ? static_cast<const V*>(p.prev[a])[cb] : zero;
    const ColGeo<R> geo = col_geo<R>(p, mx, 0, g.href[mem]);
    double omega = 1.0;
    double head[kAASlots] = {};
    if (p.aa_partial) aa_head(p, mem, head);
    if (!col_control(p, ctl, blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0, &omega)) return;
    if (p.aa_partial) aa_block_weights(p, ctl, mem, blockIdx.x == 0, head, s_aa, s_aa + 16 * kAASlots);
    lds_sync();
    V acc[NACC];
    const int np = sub.p1 - sub.p0, ns = np + sub.c1 - sub.c0, lanes = p.lanes;
    // the last lane first, so that the first wavefront ends with lane 0 in its sums
    for (int lane = wv + (lanes - 1 - wv) / W * W; lane >= 0; lane -= W) {
#pragma unroll
        for (int a = 0; a < NACC; ++a) acc[a] = zero;
#pragma unroll 2
        for (int s = lane; s < ns; s += lanes) {
            const bool prod = s < np;
            const ColSrc src = col_src(&sp.src[prod ? sub.p0 + s : kMaxProd + sub.c0 + s - np]);
            V val = on ? static_cast<const V*>(col_uni(src.ptr))[prod ? hb : cb] : zero;
            if (src.widx >= 0) val = cscale(val, R(s_aa[16 * kAASlots + src.widx]));
            col_add<R, V, NACC>(src, val, acc, geo);
        }
        if (lane > 0)
#pragma unroll
            for (int a = 0; a < NACC; ++a) sums[lane - 1][a][t] = acc[a];
    }
    if (lanes > 1) {
        lds_sync();
        if (wv == 0)
            for (int w = 1; w < lanes; ++w)
#pragma unroll
                for (int a = 0; a < NACC; ++a) acc[a] = cadd(acc[a], sums[w - 1][a][t]);
    }
    if (wv == 0 && on) {
        for (int o = sub.i0; o < sub.i1; ++o) {
            V sv = col_source<V, NACC>(col_uni(sp.inv_src[o]), acc, pv, R(omega));
            const int dv = col_uni(sp.inv_dv[o]);
            if (dv == DV_X) sv = mul_i(cscale(sv, geo.kx));
            else if (dv == DV_Y) sv = zero;
            static_cast<V*>(col_uni(sp.inv[o]))[hb] = sv;
        }
        for (int o = sub.o0; o < sub.o1; ++o)
            static_cast<V*>(col_uni(sp.cout[o]))[cb] = col_source<V, NACC>(col_uni(sp.cout_src[o]), acc, pv, R(omega));
    }
    if (p.aa_dots) {
        double d[kAASlots];
#pragma unroll
        for (int i = 0; i < kAASlots; ++i) d[i] = 0.0;
        if (wv == 0 && on) {
            const V f[2] = {col_source<V, NACC>(SRC_DIFF0, acc, pv, R(1)), col_source<V, NACC>(SRC_DIFF1, acc, pv, R(1))};
            V old[kAADepth][2];
            col_aa_old<V>(p, cb, old);
            col_aa_dots<V>(p, f, old, mx == 0 ? 1.0 : 2.0, d);
        }
        col_aa_reduce(d, s_aa, p.aa_dots + ((long long)mem * gridDim.x + blockIdx.x) * kAASlots);
    }
}

// ---------------------------------------------------------------------------
// Pointwise spectral kernels
// ---------------------------------------------------------------------------
template <typename R>
__global__ void k_rk(const RkParams p) {
    const int mem = blockIdx.y;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= p.g.s_cmp) return;
    const ModeGeo m = mode_geo(p.g, idx);
    if (m.valid) rk_mode<R>(p, p.stage, m, mem * p.g.s_cmp + idx, p.g.href[mem]);
}

// Six-stage fifth-order pair with an embedded fourth-order solution (Sec. 2.2),
// the coefficients of Cash & Karp (ACM TOMS 16, 1990): nodes, stage matrix,
// fifth-order weights and the weight differences fifth minus fourth order.
static __constant__ double kPairC[6] = {0.0, 1.0 / 5.0, 3.0 / 10.0, 3.0 / 5.0, 1.0, 7.0 / 8.0};
static __constant__ double kPairA[6][5] = {
    {0.0, 0.0, 0.0, 0.0, 0.0},
    {1.0 / 5.0, 0.0, 0.0, 0.0, 0.0},
    {3.0 / 40.0, 9.0 / 40.0, 0.0, 0.0, 0.0},
    {3.0 / 10.0, -9.0 / 10.0, 6.0 / 5.0, 0.0, 0.0},
    {-11.0 / 54.0, 5.0 / 2.0, -70.0 / 27.0, 35.0 / 27.0, 0.0},
    {1631.0 / 55296.0, 175.0 / 512.0, 575.0 / 13824.0, 44275.0 / 110592.0, 253.0 / 4096.0}};
static __constant__ double kPairB[6] = {37.0 / 378.0, 0.0, 250.0 / 621.0, 125.0 / 594.0, 0.0, 512.0 / 1771.0};
static __constant__ double kPairE[6] = {37.0 / 378.0 - 2825.0 / 27648.0, 0.0,  250.0 / 621.0 - 18575.0 / 48384.0,
                                 125.0 / 594.0 - 13525.0 / 55296.0, -277.0 / 14336.0, 512.0 / 1771.0 - 0.25};

// One stage of the pair in Lawson form, per kept mode.  With E(tau) the exact
// linear propagator (eta, phi) -> (cos eta + om sin phi, -sin/om eta + cos phi)
// and N_i = (W - om^2 phi, N_phi [- p_d]) at stage state U_i, the stage derivative is
// kept as K_i = E(-c_i h) N_i (carried back to t_n), so that
//   U_{i+1} = E(c_{i+1} h) (u_n + h sum_j a_{i+1,j} K_j),
//   u_5     = E(h) (u_n + h sum_j b_j K_j),   u_5 - u_4 = E(h) h sum_j e_j K_j.
// E preserves |eta|^2 + om^2 |phi|^2 per mode, so the linear-energy norms of
// the difference and of the candidate are summed in the frame of t_n; the last
// stage writes per-block partial sums of both (weights 2 for m_x > 0: the half
// spectrum stands for its conjugate).
template <typename R>
__global__ void k_rk54(const Rk54Params p) {
    using V = typename cplx_of<R>::type;
    __shared__ double red[2][256];
    const int mem = blockIdx.y;
    const int i = p.stage;
    const double h = p.h;
    const double href = p.g.href[mem];
    double num = 0.0, den = 0.0;
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < p.g.s_cmp;
         idx += (long long)gridDim.x * blockDim.x) {
        const ModeGeo m = mode_geo(p.g, idx);
        if (!m.valid) continue;
        const long long o = mem * p.g.s_cmp + idx;
        const double om2 = m.k * tanh(m.k * href);
        const double om = sqrt(om2);
        // (er, ei, pr, pi) -> E(tau) applied
        auto prop = [&](double tau, double& er, double& ei, double& pr, double& pi_) {
            const double c = cos(om * tau), s = sin(om * tau);
            const double sw = om > 0.0 ? s / om : tau;
            const double a = c * er + om * s * pr, b = c * ei + om * s * pi_;
            pr = -sw * er + c * pr;
            pi_ = -sw * ei + c * pi_;
            er = a;
            ei = b;
        };
        const V vh = static_cast<const V*>(p.Vh)[o];
        const V nph = static_cast<const V*>(p.Nph)[o];
        const V psv = static_cast<const V*>(p.ps)[o];
        double ker = (double)vh.x - om2 * (double)psv.x, kei = (double)vh.y - om2 * (double)psv.y;
        double kpr = (double)nph.x, kpi = (double)nph.y;
        if (p.Pdiv && m.k > 0.0) {
            // damping pressure of the wave tank: -p_d_hat = i k . MF{mu grad phi} / k^2
            const V pd = static_cast<const V*>(p.Pdiv)[o];
            kpr += (double)pd.x / (m.k * m.k);
            kpi += (double)pd.y / (m.k * m.k);
        }
        prop(-kPairC[i] * h, ker, kei, kpr, kpi);
        static_cast<V*>(p.ke[i])[o] = cx<V>(R(ker), R(kei));
        static_cast<V*>(p.kp[i])[o] = cx<V>(R(kpr), R(kpi));
        const V ue = static_cast<const V*>(p.eh)[o];
        const V up = static_cast<const V*>(p.ph)[o];
        // the stored value (rounded to R) enters the sums, as it does when read back
        const V kse = cx<V>(R(ker), R(kei)), ksp = cx<V>(R(kpr), R(kpi));
        const double* w = i < 5 ? kPairA[i + 1] : kPairB;
        double ser = 0.0, sei = 0.0, spr = 0.0, spi = 0.0;   // sum_j w_j K_j
        double der = 0.0, dei = 0.0, dpr = 0.0, dpi = 0.0;   // sum_j e_j K_j (last stage)
        for (int j = 0; j <= i; ++j) {
            const V ke = j == i ? kse : static_cast<const V*>(p.ke[j])[o];
            const V kp = j == i ? ksp : static_cast<const V*>(p.kp[j])[o];
            ser += w[j] * (double)ke.x;
            sei += w[j] * (double)ke.y;
            spr += w[j] * (double)kp.x;
            spi += w[j] * (double)kp.y;
            if (i == 5) {
                der += kPairE[j] * (double)ke.x;
                dei += kPairE[j] * (double)ke.y;
                dpr += kPairE[j] * (double)kp.x;
                dpi += kPairE[j] * (double)kp.y;
            }
        }
        double ner = (double)ue.x + h * ser, nei = (double)ue.y + h * sei;
        double npr = (double)up.x + h * spr, npi = (double)up.y + h * spi;
        if (i == 5) {
            const double wt = m.mx == 0 ? 1.0 : 2.0;
            num += wt * h * h * (der * der + dei * dei + om2 * (dpr * dpr + dpi * dpi));
            den += wt * (ner * ner + nei * nei + om2 * (npr * npr + npi * npi));
        }
        prop((i < 5 ? kPairC[i + 1] : 1.0) * h, ner, nei, npr, npi);
        if (i == 5 && p.fb1 > 0.0 && p.fb2 > 0.0) {
            const double lam = exp(-pow(fabs(m.k / p.fb1), p.fb2));
            ner *= lam;
            nei *= lam;
            npr *= lam;
            npi *= lam;
        }
        static_cast<V*>(p.es)[o] = cx<V>(R(ner), R(nei));
        static_cast<V*>(p.ps)[o] = cx<V>(R(npr), R(npi));
    }
    if (i < 5) return;
    red[0][threadIdx.x] = num;
    red[1][threadIdx.x] = den;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            red[0][threadIdx.x] += red[0][threadIdx.x + s];
            red[1][threadIdx.x] += red[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        p.partial[((long long)mem * p.nblk + blockIdx.x) * 2 + 0] = red[0][0];
        p.partial[((long long)mem * p.nblk + blockIdx.x) * 2 + 1] = red[1][0];
    }
}

template <typename R>
__global__ void k_diag(const DiagParams p) {
    using V = typename cplx_of<R>::type;
    __shared__ double red[2][256];
    const int mem = blockIdx.y;
    double se = 0.0, sm = 0.0;
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < p.g.s_cmp;
         idx += (long long)gridDim.x * blockDim.x) {
        const ModeGeo m = mode_geo(p.g, idx);
        if (!m.valid) continue;
        const long long o = mem * p.g.s_cmp + idx;
        const V e = static_cast<const V*>(p.eh)[o];
        const V f = static_cast<const V*>(p.ph)[o];
        const V w = static_cast<const V*>(p.Vh)[o];
        const double wt = m.mx == 0 ? 1.0 : 2.0;
        se += wt * ((double)w.x * (double)f.x + (double)w.y * (double)f.y + (double)e.x * (double)e.x +
                    (double)e.y * (double)e.y);
        if (idx == 0) sm += (double)e.x;
    }
    red[0][threadIdx.x] = se;
    red[1][threadIdx.x] = sm;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            red[0][threadIdx.x] += red[0][threadIdx.x + s];
            red[1][threadIdx.x] += red[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        p.partial[((long long)mem * p.nblk + blockIdx.x) * 2 + 0] = red[0][0];
        p.partial[((long long)mem * p.nblk + blockIdx.x) * 2 + 1] = red[1][0];
    }
}

// ---------------------------------------------------------------------------
// launchers (size dispatch)
// ---------------------------------------------------------------------------
// workgroups along y of a row pass: the sweep splits its product families
template <typename PT> static int row_families(const PT&) { return 1; }
static int row_families(const RowSweepParams& p) { return p.nfam * p.nch + (p.nch > 1 && p.residual ? 1 : 0); }
static int row_families(const RowProdParams& p) { return p.nfam * p.nch; }

template <typename RWT> struct RowLaunch {
    using V = typename RWT::V;
    // rpw_req: rows per workgroup asked for by the launch plan (0: as many as
    // fit 256 threads); it is a power of two, as ny is, which the row
    // kernels rely on, and capped by the kernels' launch bounds
    static void shape(int ny, dim3* grid, dim3* block, size_t* lds, int batch, int nfam, int rpw_req = 0) {
        constexpr int P = RWT::P;
        const int cap = P >= 256 ? 1 : 256 / P;
        int rpw = (rpw_req > 0 && rpw_req < cap) ? rpw_req : cap;
        if (rpw > ny) rpw = ny;
        *block = dim3(P * rpw);
        *grid = dim3((ny + rpw - 1) / rpw, nfam, batch);
        *lds = ((size_t)rpw * RWT::LS + RWT::N) * sizeof(V);
    }
};

#define SBI_ROW_NX_SWITCH(KNAME, PTYPE)                                                                    \
    template <typename R>                                                                                  \
    static hipError_t KNAME##_nx(const PTYPE& p, int batch, const Twiddles& tw, hipStream_t s) {           \
        switch (p.g.nx) {                                                                                  \
            case 16: return KNAME##_go<R, 16>(p, batch, tw, s);                                            \
            case 32: return KNAME##_go<R, 32>(p, batch, tw, s);                                            \
            case 64: return KNAME##_go<R, 64>(p, batch, tw, s);                                            \
            case 128: return KNAME##_go<R, 128>(p, batch, tw, s);                                          \
            case 256: return KNAME##_go<R, 256>(p, batch, tw, s);                                          \
            case 512: return KNAME##_go<R, 512>(p, batch, tw, s);                                          \
            case 1024: return KNAME##_go<R, 1024>(p, batch, tw, s);                                        \
            case 2048: return KNAME##_go<R, 2048>(p, batch, tw, s);                                        \
            case 4096: return KNAME##_go<R, 4096>(p, batch, tw, s);                                        \
            case 8192: return KNAME##_go<R, 8192>(p, batch, tw, s);                                        \
            default: return hipErrorInvalidValue;                                                          \
        }                                                                                                  \
    }

#define SBI_ROW_LAUNCH(KNAME, PTYPE)                                                                       \
    template <typename R, int NX>                                                                          \
    static hipError_t KNAME##_go(const PTYPE& p, int batch, const Twiddles& tw, hipStream_t s) {           \
        using V = typename cplx_of<R>::type;                                                               \
        dim3 grid, block;                                                                                  \
        size_t lds;                                                                                        \
        RowLaunch<Row<R, NX>>::shape(p.g.ny, &grid, &block, &lds, batch, row_families(p));                  \
        hipLaunchKernelGGL((KNAME<R, NX>), grid, block, lds, s, p, (const V*)tw.tn, (const V*)tw.tx);      \
        return hipGetLastError();                                                                          \
    }                                                                                                      \
    SBI_ROW_NX_SWITCH(KNAME, PTYPE)

// kernels with launch-plan variants: p.g.row_var picks the transform's
// radix and twiddle mode, p.g.row_rpw the rows per workgroup
// Only variants that compile without register spills are built: the sweep
// kernels (three workgroups per CU) take the cached twiddle powers in FP32
// only and radix-16 rows only at 512 points; the SA kernel takes both in
// FP32 from 512 points (radix 16 needs two radix-16 passes in the
// half-length row) and the cached powers in FP64 too, below 8192 points.
template <typename R, int NX, int VAR, bool SWEEP> constexpr bool row_var_built() {
    constexpr bool f32 = std::is_same<R, float>::value;
    if constexpr (VAR == 0) return true;
    if constexpr (VAR == 1) return f32 || (!SWEEP && NX < 8192);
    if constexpr (VAR == 2) return f32 && (SWEEP ? NX == 512 : NX >= 512);
    // radix 4 (4 values per thread): a row spans two or more wavefronts, so
    // its exchanges take workgroup barriers; from 256-point rows
    if constexpr (VAR == 3) return NX >= 256 && NX <= 4096;
    return false;
}
#define SBI_ROW_LAUNCH_VAR(KNAME, PTYPE, SWEEP)                                                            \
    template <typename R, int NX, int VAR>                                                                 \
    static hipError_t KNAME##_gv(const PTYPE& p, int batch, const Twiddles& tw, hipStream_t s) {           \
        if constexpr (!row_var_built<R, NX, VAR, SWEEP>()) {                                               \
            return hipErrorInvalidValue;                                                                   \
        } else {                                                                                           \
            using V = typename cplx_of<R>::type;                                                           \
            dim3 grid, block;                                                                              \
            size_t lds;                                                                                    \
            RowLaunch<RowVar<R, NX, VAR>>::shape(p.g.ny, &grid, &block, &lds, batch, row_families(p),      \
                                                 p.g.row_rpw);                                             \
            hipLaunchKernelGGL((KNAME<R, NX, VAR>), grid, block, lds, s, p, (const V*)tw.tn,               \
                               (const V*)tw.tx);                                                           \
            return hipGetLastError();                                                                      \
        }                                                                                                  \
    }                                                                                                      \
    template <typename R, int NX>                                                                          \
    static hipError_t KNAME##_go(const PTYPE& p, int batch, const Twiddles& tw, hipStream_t s) {           \
        switch (p.g.row_var) {                                                                             \
            case 0: return KNAME##_gv<R, NX, 0>(p, batch, tw, s);                                          \
            case 1: return KNAME##_gv<R, NX, 1>(p, batch, tw, s);                                          \
            case 2: return KNAME##_gv<R, NX, 2>(p, batch, tw, s);                                          \
            case 3: return KNAME##_gv<R, NX, 3>(p, batch, tw, s);                                          \
            default: return hipErrorInvalidValue;                                                          \
        }                                                                                                  \
    }                                                                                                      \
    SBI_ROW_NX_SWITCH(KNAME, PTYPE)

SBI_ROW_LAUNCH(k_row_fwd, RowFwdParams)
SBI_ROW_LAUNCH(k_row_inv, RowInvParams)
SBI_ROW_LAUNCH_VAR(k_row_sweep, RowSweepParams, true)
SBI_ROW_LAUNCH_VAR(k_row_sweep_aa, RowSweepParams, true)
SBI_ROW_LAUNCH_VAR(k_row_prod, RowProdParams, false)
SBI_ROW_LAUNCH(k_row_nphi, RowNphiParams)
SBI_ROW_LAUNCH(k_row_nphi_tank, RowNphiParams)
SBI_ROW_LAUNCH(k_row_blend, RowBlendParams)
SBI_ROW_LAUNCH(k_row_feat, RowFeatParams)

// kept modes of an owner thread: one where twelve wavefronts hold a column's, else two or three
template <typename R, int NY> static int col_modes(const GridDev& g) {
    using CS = ColShape<R, NY>;
    return (CS::CW * g.Ky + 64 * CS::WMAX - 1) / (64 * CS::WMAX);
}
// Wavefronts of a column-pass workgroup: one per column transform of a round,
// as few as the same number of rounds takes, and enough to own every kept
// mode.  Few workgroups (up to one per CU) take up to twelve, so that a
// workgroup's chain is short; more of them hide each other's barriers, and
// smaller workgroups then pack the CU better.  Measured, us a sweep's pass with at
// most 4 / 8 / 12 wavefronts: 128 x 128 FP64, 48 members (384 workgroups) 26 / 34 / 38,
// 64 members (512) 27 / 36 / 41, 96 (768) 34 / 52 / 59; FP32 64 members 16.5 / 18.1 /
// 25; 64 x 512 FP64, 64 members (1024) 46 / 65 / 76 and 57 for the pass before this
// one.  One 512 x 512 member (128) 0.67 / 0.65 / 0.65 ms per step.  The usual half band
// of 1024 rows takes eight at any rate, for its owners.
template <typename R, int NY> static int col_waves(const ColParams& p, int batch) {
    using CS = ColShape<R, NY>;
    int np = 0, ni = 0;
    for (int s = 0; s < p.nsub; ++s) {
        np = std::max(np, (int)(p.sub[s].p1 - p.sub[s].p0));
        ni = std::max(ni, (int)(p.sub[s].i1 - p.sub[s].i0));
    }
    const long long groups = (long long)(p.g.Kxp / CS::CW) * p.nsub * batch;
    const int cap = groups <= 256 ? CS::WMAX : 4;
    const int jobs = np * CS::S;
    const int rounds = (jobs + cap - 1) / cap;
    int w = rounds > 0 ? (jobs + rounds - 1) / rounds : 1;
    w = std::max(w, std::min(ni * CS::S, cap));
    const int it = col_modes<R, NY>(p.g);
    w = std::max(w, (CS::CW * p.g.Ky + 64 * it - 1) / (64 * it));
    w = (w + CS::S - 1) / CS::S * CS::S;
    return std::min(w, CS::WMAX);
}
template <typename R, int NY, int NACC, int IT>
static hipError_t col_it(const ColParams& p, int W, int batch, const Twiddles& tw, hipStream_t s) {
    using CS = ColShape<R, NY>;
    using V = typename CS::V;
    if (CS::CW * p.g.Ky > W * 64 * IT) return hipErrorInvalidValue;  // a mode without an owner
    hipLaunchKernelGGL((k_col<R, NY, NACC, IT>), dim3(p.g.Kxp / CS::CW, p.nsub, batch), dim3(64 * W),
                       (size_t)W * CS::AREA * sizeof(V), s, p, (const V*)tw.ty);
    return hipGetLastError();
}
// Wavefronts of a one-dimensional column pass's workgroup, for so many workgroups:
// all lanes side by side while the chip has room, fewer where more wavefronts would
// only wait for each other.  Measured, us a sweep's pass with 8 / 4 / 2 wavefronts:
// 16 workgroups (4096 points) 7.5 / 7.9 / 9.0; 768 (512 points, 256 members) 14.2 /
// 10.1 / 10.4; 8192 (8192 points, 256 members) 96 / 53 / 44.
static int col1_waves(int lanes, long long groups) {
    return (int)std::min<long long>(lanes, std::max<long long>(2, 3072 / groups));
}
template <typename R, int NY, int NACC>
static hipError_t col_go(const ColParams& p, int batch, const Twiddles& tw, hipStream_t s) {
    if constexpr (NY == 1) {
        if (p.g.col_C != 64) return hipErrorInvalidValue;
        int ns = 0;
        for (int i = 0; i < p.nsub; ++i)
            ns = std::max(ns, p.sub[i].p1 - p.sub[i].p0 + p.sub[i].c1 - p.sub[i].c0);
        ColParams q = p;
        q.lanes = std::min(kCol1Lanes, std::max(1, (ns + 1) / 2));
        const int W = col1_waves(q.lanes, (long long)(p.g.Kxp / 64) * p.nsub * batch);
        hipLaunchKernelGGL((k_col1<R, NACC>), dim3(p.g.Kxp / 64, p.nsub, batch), dim3(64 * W), 0, s, q);
        return hipGetLastError();
    } else {
        using CS = ColShape<R, NY>;
        if (p.g.col_C != CS::CW) return hipErrorInvalidValue;  // the layout was made for another tile
        const int W = col_waves<R, NY>(p, batch);
        const int it = col_modes<R, NY>(p.g);
        if constexpr (CS::ITMAX > 2)
            if (it > 2) return col_it<R, NY, NACC, CS::ITMAX>(p, W, batch, tw, s);
        if constexpr (CS::ITMAX > 1)
            if (it > 1) return col_it<R, NY, NACC, 2>(p, W, batch, tw, s);
        return col_it<R, NY, NACC, 1>(p, W, batch, tw, s);
    }
}
template <typename R, int NY>
static hipError_t col_acc(const ColParams& p, int batch, const Twiddles& tw, hipStream_t s) {
    if (p.nacc <= 1) return col_go<R, NY, 1>(p, batch, tw, s);
    if (p.nacc <= 2) return col_go<R, NY, 2>(p, batch, tw, s);
    return col_go<R, NY, 4>(p, batch, tw, s);
}
template <typename R>
static hipError_t col_ny(const ColParams& p, int batch, const Twiddles& tw, hipStream_t s) {
    switch (p.g.ny) {
        case 1: return col_acc<R, 1>(p, batch, tw, s);
        case 16: return col_acc<R, 16>(p, batch, tw, s);
        case 32: return col_acc<R, 32>(p, batch, tw, s);
        case 64: return col_acc<R, 64>(p, batch, tw, s);
        case 128: return col_acc<R, 128>(p, batch, tw, s);
        case 256: return col_acc<R, 256>(p, batch, tw, s);
        case 512: return col_acc<R, 512>(p, batch, tw, s);
        case 1024: return col_acc<R, 1024>(p, batch, tw, s);
        case 2048: return col_acc<R, 2048>(p, batch, tw, s);
        default: return hipErrorInvalidValue;
    }
}
// ---------------------------------------------------------------------------
// Learned history seed: per mode, the nonlinear part of the solve at RK stage
// s is predicted from the backward differences d_q of the last K fixed-step
// solves' parts (newest first) with complex weights w[P][s][b][q] of the
// mode's radial bin b = min(floor(|k| / dk), nb - 1); FP32 weights,
// arithmetic in FP64.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int hist_bin(double k, double dk, int nb) {
    const double f = floor(k / dk);
    return f >= (double)(nb - 1) ? nb - 1 : (int)f;
}
__device__ __forceinline__ int hist_widx(int P, int s, int b, int q, int nb, int K) {
    return (((P * kHistStages + s) * nb + b) * K + q) * 2;
}
// backward differences of the history of part P at element o: d_q = sum_(j<=q) (-1)^j C(q, j) h_j
template <typename V>
__device__ __forceinline__ void hist_diffs(const HistParams& p, int P, long long o, double (&dr)[kHistTaps],
                                           double (&di)[kHistTaps]) {
    double hr[kHistTaps], hi[kHistTaps];
    for (int q = 0; q < p.K; ++q) {
        const V h = static_cast<const V*>(P == 0 ? p.hv[q] : p.hb[q])[o];
        hr[q] = (double)h.x;
        hi[q] = (double)h.y;
    }
    for (int q = 0; q < p.K; ++q) {
        double c = 1.0, ar = 0.0, ai = 0.0;  // c = (-1)^j C(q, j)
        for (int j = 0; j <= q; ++j) {
            ar += c * hr[j];
            ai += c * hi[j];
            c = -c * (double)(q - j) / (double)(j + 1);
        }
        dr[q] = ar;
        di[q] = ai;
    }
}

// pv/pb <- predictions of the V and phi_b parts (zero outside the kept modes)
template <typename R>
__global__ void k_hist_seed(const HistParams p) {
    using V = typename cplx_of<R>::type;
    const int mem = blockIdx.y;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= p.g.s_cmp) return;
    const long long o = mem * p.g.s_cmp + idx;
    const ModeGeo m = mode_geo(p.g, idx);
    const int nparts = p.vd ? 2 : 1;
    for (int P = 0; P < nparts; ++P) {
        double re = 0.0, im = 0.0;
        if (m.valid) {
            const int b = hist_bin(m.k, p.dk, p.nb);
            double dr[kHistTaps], di[kHistTaps];
            hist_diffs<V>(p, P, o, dr, di);
            for (int q = 0; q < p.K; ++q) {
                const int wi = hist_widx(P, p.stage, b, q, p.nb, p.K);
                const double wr = (double)p.dev->w[wi], wm = (double)p.dev->w[wi + 1];
                re += wr * dr[q] - wm * di[q];
                im += wr * di[q] + wm * dr[q];
            }
        }
        static_cast<V*>(P == 0 ? p.pv : p.pb)[o] = cx<V>(R(re), R(im));
    }
}

// history shift: h_q <- h_(q-1) for q = K-1 .. 1, h_0 <- the new entry
template <typename R>
__global__ void k_hist_push(const HistParams p) {
    using V = typename cplx_of<R>::type;
    const int mem = blockIdx.y;
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= p.g.s_cmp) return;
    const long long o = mem * p.g.s_cmp + idx;
    const int nparts = p.vd ? 2 : 1;
    for (int P = 0; P < nparts; ++P) {
        void* const* h = P == 0 ? p.hv : p.hb;
        for (int q = p.K - 1; q >= 1; --q) static_cast<V*>(h[q])[o] = static_cast<const V*>(h[q - 1])[o];
        static_cast<V*>(h[0])[o] = static_cast<const V*>(P == 0 ? p.tv : p.tb)[o];
    }
}

// offsets of a member's per-block partials (layout for the pass's K and nb)
__device__ __forceinline__ int hist_part_tri(const HistParams& p) { return 2 * p.nb * p.K * 2; }
__device__ __forceinline__ int hist_part_ed(const HistParams& p) {
    return hist_part_tri(p) + 2 * p.nb * (p.K * (p.K + 1) / 2) * 2;
}

// loss gradient and Gram sums of predicting the target (tv, tb) from the
// history at stage s: per workgroup, S[P][b][q] = sum c conj(d_q) r,
// T[P][b][q <= r] = sum c conj(d_q) d_r, E_P = sum c |r|^2, D_P = sum c |y|^2
// over its modes (r = pred - y, c = 1 at m_x = 0 else 2), summed in LDS and
// written as the workgroup's partials
template <typename R>
__global__ void __launch_bounds__(256) k_hist_grad(const HistParams p) {
    using V = typename cplx_of<R>::type;
    __shared__ double acc[kHistPart];
    const int mem = blockIdx.y;
    const int oT = hist_part_tri(p), oE = hist_part_ed(p);
    const int ntri = p.K * (p.K + 1) / 2;
    for (int i = threadIdx.x; i < kHistPart; i += blockDim.x) acc[i] = 0.0;
    __syncthreads();
    const int nparts = p.vd ? 2 : 1;
    for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < p.g.s_cmp;
         idx += (long long)gridDim.x * blockDim.x) {
        const ModeGeo m = mode_geo(p.g, idx);
        if (!m.valid) continue;
        const long long o = mem * p.g.s_cmp + idx;
        const int b = hist_bin(m.k, p.dk, p.nb);
        const double c = m.mx == 0 ? 1.0 : 2.0;
        for (int P = 0; P < nparts; ++P) {
            const V y = static_cast<const V*>(P == 0 ? p.tv : p.tb)[o];
            double dr[kHistTaps], di[kHistTaps];
            hist_diffs<V>(p, P, o, dr, di);
            double re = 0.0, im = 0.0;
            for (int q = 0; q < p.K; ++q) {
                const int wi = hist_widx(P, p.stage, b, q, p.nb, p.K);
                const double wr = (double)p.dev->w[wi], wm = (double)p.dev->w[wi + 1];
                re += wr * dr[q] - wm * di[q];
                im += wr * di[q] + wm * dr[q];
            }
            const double rr = re - (double)y.x, ri = im - (double)y.y;
            atomicAdd(&acc[oE + P], c * (rr * rr + ri * ri));
            atomicAdd(&acc[oE + 2 + P], c * ((double)y.x * y.x + (double)y.y * y.y));
            int t = 0;
            for (int q = 0; q < p.K; ++q) {
                // conj(d_q) r
                const int si = ((P * p.nb + b) * p.K + q) * 2;
                atomicAdd(&acc[si], c * (dr[q] * rr + di[q] * ri));
                atomicAdd(&acc[si + 1], c * (dr[q] * ri - di[q] * rr));
                for (int r = q; r < p.K; ++r, ++t) {
                    // conj(d_q) d_r
                    const int ti = oT + ((P * p.nb + b) * ntri + t) * 2;
                    atomicAdd(&acc[ti], c * (dr[q] * dr[r] + di[q] * di[r]));
                    atomicAdd(&acc[ti + 1], c * (dr[q] * di[r] - di[q] * dr[r]));
                }
            }
        }
    }
    __syncthreads();
    double* out = p.partial + ((long long)mem * gridDim.x + blockIdx.x) * kHistPart;
    for (int i = threadIdx.x; i < kHistPart; i += blockDim.x) out[i] = acc[i];
}

// ---------------------------------------------------------------------------
// per-precision entry points (this file is compiled once per precision with
// SBI_REAL defined; sbi_dispatch.hip selects between them)
// ---------------------------------------------------------------------------
using Real = SBI_REAL;
template <> hipError_t launch_row_fwd_t<Real>(const RowFwdParams& p, int b, const Twiddles& tw, hipStream_t s) {
    return k_row_fwd_nx<Real>(p, b, tw, s);
}
template <> hipError_t launch_row_inv_t<Real>(const RowInvParams& p, int b, const Twiddles& tw, hipStream_t s) {
    return k_row_inv_nx<Real>(p, b, tw, s);
}
template <typename R, int NX, bool SWEEP> static int row_var_mask_nx() {
    return (row_var_built<R, NX, 0, SWEEP>() ? 1 : 0) | (row_var_built<R, NX, 1, SWEEP>() ? 2 : 0) |
           (row_var_built<R, NX, 2, SWEEP>() ? 4 : 0) | (row_var_built<R, NX, 3, SWEEP>() ? 8 : 0);
}
template <typename R, int NX> static int row_var_mask_k(int sweep) {
    return sweep ? row_var_mask_nx<R, NX, true>() : row_var_mask_nx<R, NX, false>();
}
template <> int row_var_mask_t<Real>(int sweep, int nx) {
    switch (nx) {
        case 16: return row_var_mask_k<Real, 16>(sweep);
        case 32: return row_var_mask_k<Real, 32>(sweep);
        case 64: return row_var_mask_k<Real, 64>(sweep);
        case 128: return row_var_mask_k<Real, 128>(sweep);
        case 256: return row_var_mask_k<Real, 256>(sweep);
        case 512: return row_var_mask_k<Real, 512>(sweep);
        case 1024: return row_var_mask_k<Real, 1024>(sweep);
        case 2048: return row_var_mask_k<Real, 2048>(sweep);
        case 4096: return row_var_mask_k<Real, 4096>(sweep);
        case 8192: return row_var_mask_k<Real, 8192>(sweep);
        default: return 0;
    }
}
template <> int row_rows_cap_t<Real>(int nx, int var) {
    // rows per workgroup that fill 256 threads (the launch bound)
    const int n = nx / 2;
    const int em = var == 2 ? 16 : (var == 3 ? 4 : 8);
    const int e = n >= em ? em : n;
    const int P = n / e;
    return P >= 256 ? 1 : 256 / P;
}
template <> hipError_t launch_row_sweep_t<Real>(const RowSweepParams& p, int b, const Twiddles& tw, hipStream_t s) {
    return p.gT ? k_row_sweep_aa_nx<Real>(p, b, tw, s) : k_row_sweep_nx<Real>(p, b, tw, s);
}
template <> hipError_t launch_row_prod_t<Real>(const RowProdParams& p, int b, const Twiddles& tw, hipStream_t s) {
    return k_row_prod_nx<Real>(p, b, tw, s);
}
template <> hipError_t launch_row_nphi_t<Real>(const RowNphiParams& p, int b, const Twiddles& tw, hipStream_t s) {
    return (p.wm_n > 0 || p.dmp_w > 0.0) ? k_row_nphi_tank_nx<Real>(p, b, tw, s) : k_row_nphi_nx<Real>(p, b, tw, s);
}
template <> hipError_t launch_row_blend_t<Real>(const RowBlendParams& p, int b, const Twiddles& tw, hipStream_t s) {
    return k_row_blend_nx<Real>(p, b, tw, s);
}
template <> hipError_t launch_row_feat_t<Real>(const RowFeatParams& p, int b, const Twiddles& tw, hipStream_t s) {
    return k_row_feat_nx<Real>(p, b, tw, s);
}
template <> hipError_t launch_col_t<Real>(const ColParams& p, int b, const Twiddles& tw, hipStream_t s) {
    return col_ny<Real>(p, b, tw, s);
}
template <> hipError_t launch_rk_t<Real>(const RkParams& p, int batch, hipStream_t s) {
    dim3 block(256), grid((unsigned)((p.g.s_cmp + 255) / 256), batch);
    hipLaunchKernelGGL(k_rk<Real>, grid, block, 0, s, p);
    return hipGetLastError();
}
template <> hipError_t launch_rk54_t<Real>(const Rk54Params& p, int batch, hipStream_t s) {
    // the last stage reduces over a fixed number of workgroups per member
    const unsigned nb = p.stage == 5 ? (unsigned)p.nblk : (unsigned)((p.g.s_cmp + 255) / 256);
    dim3 block(256), grid(nb, batch);
    hipLaunchKernelGGL(k_rk54<Real>, grid, block, 0, s, p);
    return hipGetLastError();
}
template <> hipError_t launch_hist_seed_t<Real>(const HistParams& p, int batch, hipStream_t s) {
    dim3 block(256), grid((unsigned)((p.g.s_cmp + 255) / 256), batch);
    hipLaunchKernelGGL(k_hist_seed<Real>, grid, block, 0, s, p);
    return hipGetLastError();
}
template <> hipError_t launch_hist_push_t<Real>(const HistParams& p, int batch, hipStream_t s) {
    dim3 block(256), grid((unsigned)((p.g.s_cmp + 255) / 256), batch);
    hipLaunchKernelGGL(k_hist_push<Real>, grid, block, 0, s, p);
    return hipGetLastError();
}
template <> hipError_t launch_hist_grad_t<Real>(const HistParams& p, int batch, hipStream_t s) {
    dim3 block(256), grid(kHistBlocks, batch);
    hipLaunchKernelGGL(k_hist_grad<Real>, grid, block, 0, s, p);
    return hipGetLastError();
}
template <> hipError_t launch_diag_t<Real>(const DiagParams& p, int batch, hipStream_t s) {
    dim3 block(256), grid(p.nblk, batch);
    hipLaunchKernelGGL(k_diag<Real>, grid, block, 0, s, p);
    return hipGetLastError();
}

}  // namespace sbi
