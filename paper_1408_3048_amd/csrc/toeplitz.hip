// Noise weighting N^-1: one symmetric band-limited Toeplitz block per
// stationary interval [Sect. 2.1, eq. N_def], applied by overlap-save with an
// LDS-resident radix-16 FFT.
//
// Kernel construction [Sect. 4.1.4, eq. fknee; App. D, eqs. glsSolFourier,
// apodDef]: the first row of the block of an interval of n samples is the
// inverse real DFT, on the interval's own grid f_m = m f_samp / n, of the
// inverse PSD q_m = 1 / (sigma^2 (1 + (f_knee / f_m)^alpha)) (q_0 = 0 for 1/f
// noise), kept for lags |k| <= lambda and apodised by a window.  Its symbol
// on the FFT grid, H(m) = t_0 + 2 sum_k t_k cos(2 pi k m / n_r), is the real
// spectrum used by the convolution; min H > 0 is required (positive
// definiteness of every block).
//
// Overlap-save: a tile producing outputs [o, o + L) loads the window
// [o - lambda, o + L + lambda) of the interval (zeros outside the interval,
// whose edges are hard boundaries, not periodic) into n_r >= L + 2 lambda real
// points.  The real sequence is packed as n_r/2 complex points, transformed
// in place by decimation in frequency (natural order in, bit-reversed out),
// split into the real spectrum, multiplied by H, merged back, and
// transformed in place by decimation in time (bit-reversed in, natural out),
// so no explicit permutation pass is needed.  Both transforms run as radix-16
// passes held in registers with one LDS exchange per pass.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>

#include "mm_device.h"
#include "mm_fft_reg.h"

namespace mm {
namespace {

// ------------------------------------------------------------------ plan-time transforms

// Inverse PSD q_m = 1 / (sigma^2 (1 + (f_knee / f_m)^alpha)) at f_m = m f_samp / n
// [Sect. 4.1.4, eq. fknee], q_0 = 0 for 1/f noise (1/sigma^2 for white noise), or its
// derivative with respect to sigma (what = 1), f_knee (2) or alpha (3); the f_knee and
// alpha derivatives are taken as 0 for white noise.
__device__ __forceinline__ double inv_psd_at(int64_t m, int64_t n, double f_samp, double sigma,
                                             double fk, double al, int what) {
    if (fk > 0.0) {
        if (m == 0) return 0.0;
        const double f = (double)m * f_samp / (double)n;
        const double ratio = pow(fk / f, al);
        const double q = 1.0 / (sigma * sigma * (1.0 + ratio));
        if (what == 0) return q;
        if (what == 1) return -2.0 * q / sigma;
        if (what == 2) return -q * (al * ratio / fk) / (1.0 + ratio);
        return -q * ratio * log(fk / f) / (1.0 + ratio);
    }
    const double q = 1.0 / (sigma * sigma);
    return what == 0 ? q : (what == 1 ? -2.0 * q / sigma : 0.0);
}

// q_m (or a derivative) for every kernel: a[g][m] = c_m q_m, the coefficients of the real
// inverse DFT written as a cosine sum (c_0 = 1, c_m = 2 for 0 < m < n/2, c_{n/2} = 1 for
// even n).
__global__ void k_inv_psd(const int32_t* __restrict__ klen, const double* __restrict__ kpar,
                          const int64_t* __restrict__ aoff, const int64_t* __restrict__ acnt,
                          double f_samp, double* __restrict__ a, int32_t nk, int what) {
    const int g = blockIdx.y;
    if (g >= nk) return;
    const int64_t n = klen[g];
    const int64_t cnt = acnt[g];  // n/2 + 1, or 0 for kernels whose taps come from the FFT path
    const double sigma = kpar[3 * g], fk = kpar[3 * g + 1], al = kpar[3 * g + 2];
    for (int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; m < cnt;
         m += (int64_t)gridDim.x * blockDim.x) {
        const double q = inv_psd_at(m, n, f_samp, sigma, fk, al, what);
        double c = 2.0;
        if (m == 0 || (2 * m == n)) c = 1.0;
        a[aoff[g] + m] = c * q;
    }
}

// the FFT twiddles exp(-2 pi i q / n), q < count, as (re, im) pairs in FP64 and, where
// tw32 is given, rounded to FP32 (2q/n is exact for the power-of-two lengths used here)
__global__ void k_twiddles(int64_t count, int64_t n, double* __restrict__ tw64,
                           float* __restrict__ tw32) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < count;
         q += (int64_t)gridDim.x * blockDim.x) {
        double s, c;
        sincospi(-2.0 * (double)q / (double)n, &s, &c);
        tw64[2 * q] = c;
        tw64[2 * q + 1] = s;
        if (tw32) {
            tw32[2 * q] = (float)c;
            tw32[2 * q + 1] = (float)s;
        }
    }
}

// out[g][j] = sum_{i < cnt[g]} a[g][i] cos(2 pi i j / n[g]) for j < J[g].
// The cosine of every term comes from a rotation recurrence re-anchored by
// sincospi every 32 terms, and the terms are added in runs of 32, of 256 and of the rest
// (bounded rounding growth).
constexpr int kCtThreads = 256;
__global__ void k_cos_transform(const double* __restrict__ a, const int64_t* __restrict__ aoff,
                                const int64_t* __restrict__ acnt, const int64_t* __restrict__ nper,
                                const int64_t* __restrict__ jcnt, const int64_t* __restrict__ ooff,
                                double* __restrict__ out, int32_t ng) {
    __shared__ double sa[kCtThreads];
    const int g = blockIdx.y;
    if (g >= ng) return;
    const int64_t J = jcnt[g];
    const int64_t j = (int64_t)blockIdx.x * kCtThreads + threadIdx.x;
    if ((int64_t)blockIdx.x * kCtThreads >= J) return;
    const int64_t n = nper[g];
    const int64_t cnt = acnt[g];
    const double* ag = a + aoff[g];
    const int64_t jm = j % n;
    double cs, ss;
    sincospi(2.0 * (double)jm / (double)n, &ss, &cs);
    double acc = 0.0;
    for (int64_t i0 = 0; i0 < cnt; i0 += kCtThreads) {
        __syncthreads();
        sa[threadIdx.x] = (i0 + threadIdx.x < cnt) ? ag[i0 + threadIdx.x] : 0.0;
        __syncthreads();
        double chunk = 0.0;
        for (int s = 0; s < kCtThreads; s += 32) {
            if (i0 + s >= cnt) break;
            const int64_t idx = ((i0 + s) % n) * jm % n;
            double c, sn;
            sincospi(2.0 * (double)idx / (double)n, &sn, &c);
            double run = 0.0;
#pragma unroll 8
            for (int u = 0; u < 32; ++u) {
                run = fma(sa[s + u], c, run);
                const double c2 = c * cs - sn * ss;
                sn = fma(sn, cs, c * ss);
                c = c2;
            }
            chunk += run;
        }
        acc += chunk;
    }
    if (j < J) out[ooff[g] + j] = acc;
}

// apodisation window at lag k (0 <= k <= lambda) [App. D, eq. apodDef]: 1 at k = 0 for
// every window, so lambda = 0 keeps t_0 alone (a diagonal N^-1)
__device__ __forceinline__ double window_at(int64_t k, int lam, int window) {
    if (k == 0) return 1.0;
    const double x = (double)k / (double)lam;
    if (window == MM_WIN_GAUSS) return exp(-x * x);
    if (window == MM_WIN_GAUSS2) return exp(-2.0 * x * x);
    return 1.0;
}

__global__ void k_taps_finish(double* __restrict__ t, const int64_t* __restrict__ toff,
                              const int64_t* __restrict__ tcnt, const int32_t* __restrict__ klen,
                              int lam, int window, int32_t nk) {
    const int g = blockIdx.y;
    if (g >= nk) return;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < tcnt[g];
         k += (int64_t)gridDim.x * blockDim.x) {
        t[toff[g] + k] *= window_at(k, lam, window) / (double)klen[g];
    }
}

__global__ void k_spec_finish(const double* __restrict__ Hraw, int64_t stride, int64_t cnt,
                              double scale, double* __restrict__ H64, float* __restrict__ H32,
                              double* __restrict__ hmin) {
    const int g = blockIdx.x;
    double m = INFINITY;
    for (int64_t i = threadIdx.x; i < cnt; i += blockDim.x) {
        const double h = Hraw[g * stride + i];
        m = fmin(m, h);
        if (H64) H64[g * stride + i] = h * scale;
        if (H32) H32[g * stride + i] = (float)(h * scale);
    }
    __shared__ double red[256];
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) hmin[g] = red[0];
}

// ------------------------------------------------------------------ overlap-save kernel

template <typename T>
struct ToepArgs {
    const int32_t* cid;
    const T* w;           // [n_t][2] time-ordered weights (IQU)
    const double* x;      // map (FP64); I-only mode reads it directly
    const T* xp;          // map packed as [n_obs][4] = (I, Q, U, 0) in T (IQU mode)
    const void* y;        // TOD input
    int y_f64;
    int mode;             // 0 map IQU, 1 map I, 2 TOD FP64, 3 TOD FP32
    T* z;
    const T* H;           // [n_kern][M + 1], or [n_kern][PairSpectrum::LEN]
    const T* tw;          // [M][2], or RegFft's table
    const TileRec* tiles;
    int lam;
    int64_t n_tiles;          // tiles of the launch (blocks are mapped to tiles XCD-major)
    const int* mask;          // per-problem flags: tiles of problems with mask 0 are skipped
    int skip_zero;            // map modes: all-zero windows skip the transform
    const uint8_t* int_on;    // zero-skipping launches: intervals flagged 0 have an all-zero
                              // input (known beforehand) and write zeros without loading it
    // zero-skipping launches over several maps (blockIdx.y = layer y < layers): layer y
    // reads x + y x_step, xp + y xp_step and int_on + y on_step and writes z + y z_step
    int layers;
    int64_t x_step, xp_step, z_step, on_step;
};

// The spectrum product of a frequency pair (k, m = M - k) of the packed real transform.
// With Z the M-point transform of z[n] = y[2n] + i y[2n+1], the real transform of y is
// X_k = ((Z_k + conj Z_m) - i e (Z_k - conj Z_m)) / 2, e = exp(-i pi k / M); the product
// Y_k = H_k X_k (H real and even) is packed back into the input of the inverse transform
// as W_k = (Y_k + conj Y_m) + i conj(e) (Y_k - conj Y_m).  Composed, the three steps are
// one linear map with real coefficients: with c = cos(pi k / M), s = sin(pi k / M),
//   W_k = a_k Z_k + i g conj(Z_m),   W_m = a_m Z_m + i g conj(Z_k),
//   a_k = h_k + h_m - s (h_k - h_m),  a_m = h_k + h_m + s (h_k - h_m),  g = c (h_k - h_m),
// where h = H / n_r is the spectrum as the plan stores it (the inverse transform's 1/M
// and the split's factors folded in).  k = 0 (pair with m = M, the Nyquist bin) and the
// self-paired k = M/2 (c = 0, s = 1) are the same formula.  tw holds e as (c, -s).
template <typename T>
__device__ __forceinline__ void spectrum_pair(T hk, T hm, T c, T s, T zkr, T zki, T zmr,
                                                T zmi, T& wkr, T& wki, T& wmr, T& wmi) {
    const T u = hk + hm, v = hk - hm;
    const T ak = u - s * v, am = u + s * v, g = c * v;
    wkr = ak * zkr + g * zmi;
    wki = ak * zki + g * zmr;
    wmr = am * zmr + g * zki;
    wmi = am * zmi + g * zkr;
}

// A thread's kernel-spectrum and twiddle values for the pairs k = tid + i NT <= M/2 of the
// spectrum product, loaded together, so that their memory latency is paid once, not once per
// pair.
template <typename T, int LOGM, int NT>
struct SpectrumValues {
    static constexpr int M = 1 << LOGM, NI = (M / 2 + NT) / NT;
    T hk[NI], hm[NI], cc[NI], ss[NI];
    __device__ __forceinline__ SpectrumValues(const T* __restrict__ H, const T* __restrict__ tw) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int k0 = threadIdx.x + i * NT;
            const int k = k0 <= M / 2 ? k0 : M / 2;  // valid address; not used past M/2
            hk[i] = H[k];
            hm[i] = H[M - k];
            cc[i] = tw[2 * k];
            ss[i] = -tw[2 * k + 1];
        }
    }
};

// spectrum product on pairs (k, M - k) of the bit-reversed half-length transform
template <typename T, int LOGM, int NT>
__device__ __forceinline__ void spectrum_pass(const CBuf<T>& buf,
                                              const SpectrumValues<T, LOGM, NT>& s) {
    constexpr int M = 1 << LOGM, NI = SpectrumValues<T, LOGM, NT>::NI;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int k = threadIdx.x + i * NT;
        if (i == NI - 1 && k > M / 2) continue;  // only the last can be past M/2
        const int km = M - k;
        const int ak = rev_bits<LOGM>(k);
        const int am = k == 0 ? ak : rev_bits<LOGM>(km);  // bin M is bin 0
        T zkr, zki, zmr, zmi, wkr, wki, wmr, wmi;
        buf.get(ak, zkr, zki);
        buf.get(am, zmr, zmi);
        spectrum_pair(s.hk[i], s.hm[i], s.cc[i], s.ss[i], zkr, zki, zmr, zmi, wkr, wki, wmr, wmi);
        buf.put(ak, wkr, wki);
        if (k != 0 && km != k) buf.put(am, wmr, wmi);
    }
    __syncthreads();
}

// For LOGM = 1 mod 4 the forward transform ends and the inverse starts with a radix-2
// stage on adjacent slots (2j, 2j + 1), which hold the frequencies f and f + M/2 after the
// stage (f = rev(2j)).  The slots {rev(k), rev(k) ^ 1, rev(M - k), rev(M - k) ^ 1} carry the
// frequencies k, M/2 + k, M - k and M/2 - k: the two spectrum pairs (k, M - k) and
// (M/2 + k, M/2 - k).  This pass takes such a group (k = 0 .. M/4) through the forward
// radix-2 stage, the spectrum product of both pairs and the inverse radix-2 stage, which
// saves two passes over LDS and two barriers; the arithmetic is that of the three passes.
template <typename T, int LOGM, int NT>
__device__ __forceinline__ void spectrum_pass_r2(const CBuf<T>& buf, const T* __restrict__ H,
                                                 const T* __restrict__ tw) {
    constexpr int M = 1 << LOGM;
    constexpr int NI = (M / 4 + NT) / NT;  // groups k = tid + i NT <= M/4
    // per group: h at k, M - k, M/2 + k, M/2 - k and the twiddle (c, -s) at k; the pair
    // (M/2 + k, M/2 - k) has c' = -s, s' = c
    T h0[NI], h1[NI], h2[NI], h3[NI], cc[NI], ss[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int k0 = threadIdx.x + i * NT;
        const int k = k0 <= M / 4 ? k0 : M / 4;  // valid address; not used past M/4
        h0[i] = H[k];
        h1[i] = H[M - k];
        h2[i] = H[M / 2 + k];
        h3[i] = H[M / 2 - k];
        cc[i] = tw[2 * k];
        ss[i] = -tw[2 * k + 1];
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int k = threadIdx.x + i * NT;
        if (k > M / 4) break;
        const int a = rev_bits<LOGM>(k);  // even: k < M/2
        // byte offsets: slot a + 1 = a ^ 1 sits at swz(a) ^ 1 (swz is linear over XOR)
        const int ab = swz(a) << 3;
        T ur, ui, vr, vi;
        buf.get_swb(ab, ur, ui);
        buf.get_swb(ab ^ 8, vr, vi);
        // forward radix-2 stage: slot a -> frequency k, slot a + 1 -> k + M/2
        const T z0r = ur + vr, z0i = ui + vi, z1r = ur - vr, z1i = ui - vi;
        T y0r, y0i, y1r, y1i, q0r, q0i, q1r, q1i;
        if (k == 0) {  // DC with the Nyquist bin (pair (0, M)), and the self-paired M/2
            // h2 = h3 = H[M/2]; (c, s) at M/2 is (0, 1)
            spectrum_pair(h0[i], h1[i], (T)1, (T)0, z0r, z0i, z0r, z0i, y0r, y0i, q0r, q0i);
            spectrum_pair(h2[i], h3[i], (T)0, (T)1, z1r, z1i, z1r, z1i, y1r, y1i, q1r, q1i);
        } else if (k == M / 4) {  // the pair (M/4, 3M/4) is the slot pair itself
            spectrum_pair(h0[i], h1[i], cc[i], ss[i], z0r, z0i, z1r, z1i, y0r, y0i, y1r, y1i);
        } else {
            const int b = rev_bits<LOGM>(M - k);  // odd: slot b -> M - k, b - 1 -> M/2 - k
            const int bb = swz(b) << 3;           // slot b - 1 = b ^ 1 at bb ^ 8
            T sr, si, tr, ti;
            buf.get_swb(bb ^ 8, sr, si);
            buf.get_swb(bb, tr, ti);
            const T w0r = sr + tr, w0i = si + ti, w1r = sr - tr, w1i = si - ti;
            spectrum_pair(h0[i], h1[i], cc[i], ss[i], z0r, z0i, w1r, w1i, y0r, y0i, q1r, q1i);
            spectrum_pair(h2[i], h3[i], -ss[i], cc[i], z1r, z1i, w0r, w0i, y1r, y1i, q0r, q0i);
            // inverse radix-2 stage on the slots (b - 1, b)
            buf.put_swb(bb ^ 8, q0r + q1r, q0i + q1i);
            buf.put_swb(bb, q0r - q1r, q0i - q1i);
        }
        // inverse radix-2 stage on the slots (a, a + 1)
        buf.put_swb(ab, y0r + y1r, y0i + y1i);
        buf.put_swb(ab ^ 8, y0r - y1r, y0i - y1i);
    }
    __syncthreads();
}

// element i of an array at a block-uniform base, addressed by a 32-bit byte offset (the
// scalar-base form of the load: no 64-bit vector address arithmetic per element)
template <typename E>
__device__ __forceinline__ E at_u32(const E* base, uint32_t i) {
    return *reinterpret_cast<const E*>(reinterpret_cast<const char*>(base) +
                                       i * (uint32_t)sizeof(E));
}

// Load phase: the tile's window [o - lambda, o + L + lambda) of the interval, zero
// outside, packed as complex points (even sample -> real, odd -> imaginary).  Each
// thread handles 8 samples at a time and issues their index loads, weight loads and
// map gathers as independent batches, so several memory requests per thread are in
// flight.  Out-of-window samples load a valid index (the interval start) and are
// masked to zero.
// returns whether any of the thread's samples is nonzero
template <typename T, int LOGM, int NT, int MODE>
__device__ __forceinline__ bool load_window(const ToepArgs<T>& a, const CBuf<T>& buf,
                                            int64_t base, int win, int64_t lo, int64_t hi) {
    constexpr int NR = 2 << LOGM;
    constexpr int PER = NR / NT;
    // samples in flight per thread (the IQU map gather has batches of its own)
    constexpr int B = PER < 16 ? PER : 16;
    static_assert(PER % B == 0, "tile must split into batches");
    static_assert(NT % 2 == 0, "even thread count");
    // point (tid + c NT) / 2 = tid / 2 + c NT / 2 with bit-disjoint terms
    const int sbase = swz(threadIdx.x >> 1), part = threadIdx.x & 1;
    // indices relative to the window start (a block-uniform base): window positions
    // [i_lo, i_hi) lie inside the interval; others read position i_lo (inside the
    // interval, since the window ends past it) and are masked.  32-bit unsigned offsets
    // from uniform bases keep the address arithmetic out of 64-bit vector instructions.
    const int i_lo = (int)(lo > base ? lo - base : 0);
    const int i_hi = (int)(hi - base < (int64_t)win ? hi - base : (int64_t)win);
    bool nz = false;
    if constexpr (MODE == 0) {
        // IQU map gather, software-pipelined: the indices and weights of batch k + 1 are
        // loaded while the map gathers of batch k are in flight, so a batch waits for one
        // memory latency instead of two;
        // batches of 8 samples in FP32, 4 in FP64 (registers)
        typedef typename std::conditional<sizeof(T) == 4, float4, double4>::type T4;
        typedef typename std::conditional<sizeof(T) == 4, float2, double2>::type T2;
        constexpr int BP = sizeof(T) == 4 ? (PER < 8 ? PER : 8) : (PER < 4 ? PER : 4);
        static_assert(PER % BP == 0, "tile must split into batches");
        const int32_t* cb = a.cid + base;
        const T2* wb = reinterpret_cast<const T2*>(a.w) + base;
        const char* xpb = reinterpret_cast<const char*>(a.xp);
        auto pos = [&](int k) -> uint32_t {
            const int i = threadIdx.x + k * NT;
            return (uint32_t)(i >= i_lo && i < i_hi ? i : i_lo);
        };
        uint32_t cc[BP];
        T2 ww[BP];
#pragma unroll
        for (int u = 0; u < BP; ++u) {
            const uint32_t r = pos(u);
            cc[u] = (uint32_t)at_u32(cb, r);
            ww[u] = at_u32(wb, r);
        }
#pragma unroll
        for (int b0 = 0; b0 < PER; b0 += BP) {
            T4 xx[BP];
#pragma unroll
            for (int u = 0; u < BP; ++u)
                xx[u] = *reinterpret_cast<const T4*>(xpb + cc[u] * (uint32_t)sizeof(T4));
            T2 wcur[BP];
#pragma unroll
            for (int u = 0; u < BP; ++u) wcur[u] = ww[u];
            if (b0 + BP < PER) {
#pragma unroll
                for (int u = 0; u < BP; ++u) {
                    const uint32_t r = pos(b0 + BP + u);
                    cc[u] = (uint32_t)at_u32(cb, r);
                    ww[u] = at_u32(wb, r);
                }
            }
#pragma unroll
            for (int u = 0; u < BP; ++u) {
                const int i = threadIdx.x + (b0 + u) * NT;
                const bool ok = i >= i_lo && i < i_hi;
                const T v = ok ? xx[u].x + wcur[u].x * xx[u].y + wcur[u].y * xx[u].z : (T)0;
                buf.put_part_sw(sbase ^ swz((b0 + u) * (NT / 2)), part, v);
                nz = nz || v != (T)0;
            }
        }
        return nz;
    }
#pragma unroll
    for (int b0 = 0; b0 < PER; b0 += B) {
        uint32_t rr[B];
        bool ok[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int i = threadIdx.x + (b0 + u) * NT;
            ok[u] = i >= i_lo && i < i_hi;
            rr[u] = (uint32_t)(ok[u] ? i : i_lo);
        }
        T v[B];
        if constexpr (MODE == 1) {  // I rows of the map (I-only plans, and IQU maps
                                           // whose Q and U rows are zero: the I weight is 1)
            const int32_t* cb = a.cid + base;
            int32_t cc[B];
#pragma unroll
            for (int u = 0; u < B; ++u) cc[u] = at_u32(cb, rr[u]);
#pragma unroll
            for (int u = 0; u < B; ++u) v[u] = ok[u] ? (T)a.x[cc[u]] : (T)0;
        } else if constexpr (MODE == 2) {  // TOD, FP64
            const double* y = (const double*)a.y + base;
#pragma unroll
            for (int u = 0; u < B; ++u) v[u] = ok[u] ? (T)at_u32(y, rr[u]) : (T)0;
        } else {  // TOD, FP32
            const float* y = (const float*)a.y + base;
#pragma unroll
            for (int u = 0; u < B; ++u) v[u] = ok[u] ? (T)at_u32(y, rr[u]) : (T)0;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            buf.put_part_sw(sbase ^ swz((b0 + u) * (NT / 2)), part, v[u]);
            nz = nz || v[u] != (T)0;
        }
    }
    return nz;
}

// waves per SIMD that the tile's LDS allows (160 KB per CU, 4 SIMDs per CU), capped where
// the butterflies and gathers would spill (4 waves = 128 VGPRs for FP32, 3 = 170
// for FP64): the register budget the compiler must meet so that LDS bounds occupancy
template <typename T, int LOGM, int NT>
constexpr int tile_waves_per_simd() {
    constexpr int blocks = (160 * 1024) / (2 * (1 << LOGM) * (int)sizeof(T));
    constexpr int w = blocks * (NT / 64) / 4;
    constexpr int cap = sizeof(T) == 4 ? 4 : 3;
    return w < 1 ? 1 : (w > cap ? cap : w);
}
// the LDS twiddle table is used where it leaves the number of resident tiles unchanged, by LDS and
// by the 32 waves that a CU holds.  The 8192-point FP32 tile, 5 a CU without the table and 4 with
// it, takes, with / without: N^-1 of a TOD of 2^20 samples 11.2 / 11.1 us, of 48 problems (7.3e6
// samples) 28.6 / 28.1, A x 90.2 / 90.3
template <typename T, int LOGM, int NT>
constexpr bool ltw_enabled() {
    constexpr int cu = 160 * 1024, wmax = 32 / (NT / 64);
    constexpr int bytes = 2 * (1 << LOGM) * (int)sizeof(T);
    constexpr int tbytes = 2 * ltw_total(LOGM) * (int)sizeof(T);
    constexpr int b0 = cu / bytes < wmax ? cu / bytes : wmax;
    constexpr int b1 = cu / (bytes + tbytes) < wmax ? cu / (bytes + tbytes) : wmax;
    return ltw_total(LOGM) > 0 && b0 == b1;
}
static_assert(ltw_enabled<float, 11, 256>() && !ltw_enabled<float, 12, 256>() &&
                  ltw_enabled<float, 13, 512>(),
              "8 tiles of 4096 points fit a CU with the table, 4 of 8192 instead of 5, 2 of 16384");

// threads of a tile: one radix-16 group per thread and pass
template <int LOGM>
constexpr int tile_threads() {
    constexpr int nt = (1 << LOGM) / 16;
    return nt > 1024 ? 1024 : (nt < 256 ? 256 : nt);
}

struct Unused {
    template <class... A>
    __device__ __forceinline__ explicit Unused(const A&...) {}
};

// SKIPZ: a tile whose input window is all zero writes zeros and skips the transform (the
// exact result; used for the sparse A Z columns; costs a block vote in LDS)
template <typename T, int LOGM, int NT, int MODE, bool SKIPZ>
__global__ __launch_bounds__(NT, (tile_waves_per_simd<T, LOGM, NT>())) void k_toeplitz(
    ToepArgs<T> a) {
    constexpr int M = 1 << LOGM;
    constexpr bool LTW = ltw_enabled<T, LOGM, NT>();
    __shared__ __align__(16) unsigned char
        smem[2 * M * sizeof(T) + (LTW ? 2 * ltw_total(LOGM) * sizeof(T) : 0)];
    const CBuf<T> buf = make_cbuf<T>(smem, M);
    T* const lt = reinterpret_cast<T*>(smem + 2 * M * sizeof(T));
    if constexpr (SKIPZ) {
        if (blockIdx.y) {
            const int64_t y = blockIdx.y;
            a.x += y * a.x_step;
            a.xp += y * a.xp_step;
            a.z += y * a.z_step;
            if (a.int_on) a.int_on += y * a.on_step;
        }
    }
    // XCD-major tile order (neighbouring tiles share pointing, map and kernel data in one
    // L2), except for zero-skipping launches: there the few non-zero tiles of a sparse
    // column are neighbours and would all land on one XCD
    const int64_t tile = SKIPZ ? (int64_t)blockIdx.x : xcd_item(blockIdx.x, a.n_tiles);
    if (tile < 0 || tile >= a.n_tiles) return;
    const TileRec tr = a.tiles[tile];
    if (a.mask && !a.mask[tr.prob]) return;
    const int64_t o = tr.out, lo = tr.lo, hi = tr.hi;
    const int L = tr.len;
    const int lam = a.lam;
    if constexpr (SKIPZ) {
        if (a.int_on && !a.int_on[tr.inter]) {
            for (int i = threadIdx.x; i < L; i += NT) a.z[o + i] = (T)0;
            return;
        }
    }
    // the twiddle table is ordered by the barrier after the load (zero-skipping launches:
    // filled only for non-zero windows, behind a barrier of its own)
    if constexpr (LTW && !SKIPZ) fill_ltw<T, LOGM, NT>(a.tw, lt);
    // the shortest tiles, a launch of which is a chain of latencies, have registers to load the
    // spectrum's values with the window (with the tile in one record, N^-1 P of 2^14 samples
    // 9.5 -> 8.9 us; the record alone, 2^20 samples FP64 24.8 -> 24.3)
    constexpr bool EARLY = LOGM == 10;
    [[maybe_unused]] std::conditional_t<EARLY, SpectrumValues<T, LOGM, NT>, Unused> early(
        a.H + (int64_t)tr.kern * (M + 1), a.tw);
    const bool nz = load_window<T, LOGM, NT, MODE>(a, buf, o - lam, L + 2 * lam, lo, hi);
    if constexpr (SKIPZ) {
        if (!__syncthreads_or(nz)) {  // zero window: the exact result is zero
            for (int i = threadIdx.x; i < L; i += NT) a.z[o + i] = (T)0;
            return;
        }
        if constexpr (LTW) {
            fill_ltw<T, LOGM, NT>(a.tw, lt);
            __syncthreads();
        }
    } else {
        (void)nz;
        __syncthreads();
    }
    if constexpr (LOGM % 4 == 1) {  // the radix-2 stages go into the spectrum pass
        fwd_passes<T, LOGM, NT, LOGM, 1, LTW>(buf, a.tw, lt);
        spectrum_pass_r2<T, LOGM, NT>(buf, a.H + (int64_t)tr.kern * (M + 1), a.tw);
        inv_passes<T, LOGM, NT, LOGM, 1, LTW>(buf, a.tw, lt);
    } else if constexpr (EARLY) {
        fwd_passes<T, LOGM, NT, LOGM, 0, LTW>(buf, a.tw, lt);
        spectrum_pass<T, LOGM, NT>(buf, early);
        inv_passes<T, LOGM, NT, LOGM, 0, LTW>(buf, a.tw, lt);
    } else {
        fwd_passes<T, LOGM, NT, LOGM, 0, LTW>(buf, a.tw, lt);
        spectrum_pass<T, LOGM, NT>(
            buf, SpectrumValues<T, LOGM, NT>(a.H + (int64_t)tr.kern * (M + 1), a.tw));
        inv_passes<T, LOGM, NT, LOGM, 0, LTW>(buf, a.tw, lt);
    }
    T* zo = a.z + o;  // block-uniform base, 32-bit offsets
    for (int i = lam + threadIdx.x; i < lam + L; i += NT)
        *reinterpret_cast<T*>(reinterpret_cast<char*>(zo) + (uint32_t)(i - lam) * (uint32_t)sizeof(T)) =
            buf.get_part(i >> 1, i & 1);
}

// ---- FP64, two tiles per workgroup, in registers
//
// The kernel spectrum H is real and even, so the band convolution of y_a + i y_b, two windows
// of one interval as one complex sequence of N = n_r points, leaves y_a's result in the real
// part and y_b's in the imaginary part: the spectrum product is one real factor per point,
// without the split, twiddles and partner access that a packed real transform needs.  The
// transform is RegFft's: a thread loads point t + NT i of both windows straight into its
// registers (samples of consecutive threads are consecutive), and stores its results from
// there; LDS carries the two exchanges each way alone.  H is stored in the order the threads
// hold the bit-reversed spectrum, two values per thread and load (PairSpectrum).
//
// What bounded the LDS-resident FP64 tile was the latency of its passes at 2 waves per SIMD
// (a complex buffer of 64 KB per tile); here 4 are resident.  N^-1 of a TOD / N^-1 P x, in us,
// LDS-resident / in registers: 2^20 samples, lambda = 2048 30.7 / 18.5 and 36 / 28; 2^22 58 / 33
// and 67 / 50; 2^24 172 / 121 and 214 / 181; lambda = 512, 5.8e6 samples in ragged intervals
// 49.0 / 35.6 and 64 / 53; 2^18 samples of one Stokes parameter, lambda = 1024 11.1 / 11.1 and
// 13.2 / 11.4.  The map gather is what is left beside the transform: its loads and the
// transforms of a CU's two workgroups overlap little (counters at 2^24 samples, where the data
// leave the last-level cache: 157 us, 712 MB for 470 that the samples need, 4.5 TB/s: there the
// bytes of the halos bound it; vector issue 45%).  The error against 64-bit FFTs of
// whole intervals fell from 1.0e-15 to 0.6e-15 (twiddle powers rounded once).
//
// The same kernel in FP32 (32 points per thread) gained nothing at 16384 points (raster of
// 2^24: 94.5 / 96.5 us, ring scan of 2^25: 229 / 235) and lost at 8192 and below 2^23 samples
// (half as many workgroups): FP32 keeps the LDS-resident tile.

// The spectrum H (real, H(f) = H(N - f)) as k_toeplitz_pair's threads read it.  Position p > 0 of
// the bit-reversed spectrum and its mirror 3 2^m - 1 - p in [2^m, 2^(m+1)) hold f and N - f, so
// thread t > 1 of [2^k, 2^(k+1)) holds the values of thread 3 2^k - 1 - t in reverse: a row of R
// values is stored for one of the two, value 2 q + e of row r at [q][r][e].  Against all rows
// stored: N^-1 P of 2^22 samples, lambda = 2048 (1024) +0.2 (0) us of 50 (43), of 4096 intervals of
// one tile each +2 of 95.
template <int LOGN>
struct PairSpectrum {
    static constexpr int R = RegFft<LOGN>::R, NT = RegFft<LOGN>::NT, ROWS = NT / 2 + 1,
                         LEN = R * ROWS;
    static __device__ __forceinline__ int top(int t) { return 31 - __clz(t); }
    // whether thread t reads its mirror's row, backwards
    static __device__ __forceinline__ bool mirrored(int t) {
        return t > 1 && ((t >> (top(t) - 1)) & 1);
    }
    static __device__ __forceinline__ int row(int t) {
        if (t < 2) return t;
        const int k = top(t), u = mirrored(t) ? (3 << k) - 1 - t : t;
        return u - (1 << (k - 1)) + 1;
    }
    // the thread whose values row r holds
    static __device__ __forceinline__ int thread(int r) {
        return r < 2 ? r : r - 1 + (1 << top(r - 1));
    }
};

// vr[i], vi[i] = sample t + NT i of the two windows, 0 outside their interval, BP samples at a
// time alternating between the windows; nz: whether any is nonzero
template <int R, int NT, int MODE>
__device__ __forceinline__ void load_pair(const ToepArgs<double>& a, const int64_t (&base)[2],
                                          const int (&i_lo)[2], const int (&i_hi)[2], double* vr,
                                          double* vi, bool (&nz)[2]) {
    // one-value loads: a window's 16 together
    constexpr int BP = MODE == 0 ? 4 : R, NB = 2 * R / BP;
    nz[0] = nz[1] = false;
    // sample u of batch q: window q & 1, point (q / 2) BP + u; samples outside read position
    // i_lo, inside the interval
    auto pos = [&](int q, int u) -> uint32_t {
        const int w = q & 1, i = threadIdx.x + ((q >> 1) * BP + u) * NT;
        return (uint32_t)(i >= i_lo[w] && i < i_hi[w] ? i : i_lo[w]);
    };
    auto put = [&](int q, int u, double v) {
        const int w = q & 1, k = (q >> 1) * BP + u, i = threadIdx.x + k * NT;
        v = i >= i_lo[w] && i < i_hi[w] ? v : 0.0;
        asm volatile("" : "+v"(v));  // formed here, not where it is used
        (w ? vi : vr)[k] = v;
        nz[w] = nz[w] || v != 0.0;
    };
    if constexpr (MODE == 0) {
        // every sample's pixel index first (in the registers that the points will fill), then
        // the weights of a batch one batch ahead of its map gathers
        const char* xpb = reinterpret_cast<const char*>(a.xp);
        const double2* wb = reinterpret_cast<const double2*>(a.w);
        uint32_t cc[2 * R];
        double2 ww[BP];
#pragma unroll
        for (int u = 0; u < BP; ++u) {
            cc[u] = (uint32_t)at_u32(a.cid + base[0], pos(0, u));
            ww[u] = at_u32(wb + base[0], pos(0, u));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 1; q < NB; ++q)
#pragma unroll
            for (int u = 0; u < BP; ++u)
                cc[q * BP + u] = (uint32_t)at_u32(a.cid + base[q & 1], pos(q, u));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            double4 xx[BP];
            double2 wc[BP];
#pragma unroll
            for (int u = 0; u < BP; ++u) {
                xx[u] = *reinterpret_cast<const double4*>(xpb + cc[q * BP + u] *
                                                                    (uint32_t)sizeof(double4));
                wc[u] = ww[u];
            }
            // the gathers before the next batch's loads, so that they can be waited for alone
            __builtin_amdgcn_sched_barrier(0);
            if (q + 1 < NB) {
#pragma unroll
                for (int u = 0; u < BP; ++u)
                    ww[u] = at_u32(wb + base[(q + 1) & 1], pos(q + 1, u));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < BP; ++u)
                put(q, u, xx[u].x + wc[u].x * xx[u].y + wc[u].y * xx[u].z);
        }
    } else {
        [[maybe_unused]] uint32_t cc[2 * R];
        if constexpr (MODE == 1) {
#pragma unroll
            for (int q = 0; q < NB; ++q)
#pragma unroll
                for (int u = 0; u < BP; ++u)
                    cc[q * BP + u] = (uint32_t)at_u32(a.cid + base[q], pos(q, u));
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            double v[BP];
#pragma unroll
            for (int u = 0; u < BP; ++u) {
                if constexpr (MODE == 1) v[u] = a.x[cc[q * BP + u]];
                else if constexpr (MODE == 2) v[u] = at_u32((const double*)a.y + base[q], pos(q, u));
                else v[u] = (double)at_u32((const float*)a.y + base[q], pos(q, u));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < BP; ++u) put(q, u, v[u]);
        }
    }
}

// q[w] = the sum of squares of window w over the workgroup, in floats: it chooses a power of
// two.  red: 2 NT / 64 floats; a barrier lies between the writes and the reads, none after them.
template <int R, int NT>
__device__ __forceinline__ void pair_norms(const double* vr, const double* vi, float* red,
                                           float (&q)[2]) {
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        a = fma(vr[i], vr[i], a);
        b = fma(vi[i], vi[i], b);
    }
    q[0] = wave_sum_last((float)a);
    q[1] = wave_sum_last((float)b);
    if ((threadIdx.x & 63) == 63) {
        red[2 * (threadIdx.x >> 6)] = q[0];
        red[2 * (threadIdx.x >> 6) + 1] = q[1];
    }
    __syncthreads();
    q[0] = q[1] = 0.0f;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) {
        q[0] += red[2 * k];
        q[1] += red[2 * k + 1];
    }
}

// launch bounds: 16 waves per CU (128 registers), which both lengths' LDS allows
template <int LOGN, int MODE, bool SKIPZ>
__global__ __launch_bounds__(RegFft<LOGN>::NT, 4) void k_toeplitz_pair(ToepArgs<double> a) {
    using F = RegFft<LOGN>;
    constexpr int R = F::R, NT = F::NT;
    __shared__ __align__(16) double s[F::ELEMS];
    const int64_t pair = SKIPZ ? (int64_t)blockIdx.x : xcd_item(blockIdx.x, a.n_tiles);
    if (pair < 0 || pair >= a.n_tiles) return;
    const TileRec tr = a.tiles[2 * pair];
    const int64_t o[2] = {tr.out, a.tiles[2 * pair + 1].out};
    const int L[2] = {tr.len, a.tiles[2 * pair + 1].len};  // L[1] may be 0
    if (a.mask && !a.mask[tr.prob]) return;
    const int64_t lo = tr.lo, hi = tr.hi;
    const int lam = a.lam, t = threadIdx.x;
    if constexpr (SKIPZ) {
        if (a.int_on && !a.int_on[tr.inter]) {
#pragma unroll
            for (int w = 0; w < 2; ++w)
                for (int i = t; i < L[w]; i += NT) a.z[o[w] + i] = 0.0;
            return;
        }
    }
    const int64_t base[2] = {o[0] - lam, o[1] - lam};
    int i_lo[2], i_hi[2];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int win = L[w] ? L[w] + 2 * lam : 0;
        i_lo[w] = (int)(lo > base[w] ? lo - base[w] : 0);
        i_hi[w] = (int)(hi - base[w] < (int64_t)win ? hi - base[w] : (int64_t)win);
    }
    double vr[R], vi[R];
    bool nz[2];
    load_pair<R, NT, MODE>(a, base, i_lo, i_hi, vr, vi, nz);
    F::pin(vr, vi);
    // what a window's outputs are instead of the transform's: 0 for a zero window (the exact
    // result), NaN for a window with a sample that is not finite, whose transform would be NaN
    // throughout; it is left out of the common one so that the other window stays clean
    bool fixed[2] = {false, L[1] == 0};
    double value[2] = {0.0, 0.0};
    if constexpr (SKIPZ) {
#pragma unroll
        for (int w = 0; w < 2; ++w) fixed[w] = !__syncthreads_or(nz[w]);
    }
    // The common transform rounds by the norm of both windows, so windows whose norms differ by
    // a power of two or more are brought to the same one and their outputs back: the quiet window
    // keeps the rounding of its own transform, and none overflows for the other.  Beside a
    // window 1e4 (1e10) times louder the outputs were off by 2e-12 (1e-6) of their largest,
    // now by less than 1e-12 at any ratio; the norms take the place of the vote on samples that
    // are not finite, and solves of 2^22 samples take 8.73 ms for 8.68, gradients 12.76 for 12.66
    __shared__ float red[2 * (NT / 64)];
    int e[2] = {0, 0};  // powers of two that are taken out of the windows
    float q[2];
    pair_norms<R, NT>(vr, vi, red, q);
    const auto in_range = [](float x) { return x > 1e-30f && x < 1e36f; };
    if (!((fixed[0] || in_range(q[0])) && (fixed[1] || in_range(q[1])))) {
        // a window that is zero or not finite, or whose squares leave the range of floats: by
        // its largest magnitude first
        __shared__ double redm[NT / 64];
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            double m = 0.0, bad = 0.0;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const double v = w ? vi[i] : vr[i];
                m = fmax(m, fabs(v));
                bad = fma(v, 0.0, bad);  // NaN where a sample is not finite
            }
            const bool nan = __syncthreads_or(bad != 0.0);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
            if ((t & 63) == 0) redm[t >> 6] = m;
            __syncthreads();
            for (int k = 0; k < NT / 64; ++k) m = fmax(m, redm[k]);
            if (nan || m == 0.0) {
                fixed[w] = true;
                value[w] = nan ? __builtin_nan("") : 0.0;
#pragma unroll
                for (int i = 0; i < R; ++i) (w ? vi : vr)[i] = 0.0;
            } else {
                (void)frexp(m, &e[w]);
#pragma unroll
                for (int i = 0; i < R; ++i) (w ? vi : vr)[i] = ldexp((w ? vi : vr)[i], -e[w]);
            }
        }
        pair_norms<R, NT>(vr, vi, red, q);
    }
    double back = 1.0;  // the second window's factor after the transform
    if (!fixed[0] && !fixed[1]) {
        int f[2];  // the norms are in [2^(f-1), 2^f)
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            int x;
            (void)frexpf(q[w], &x);
            f[w] = (x + 1) >> 1;
        }
        if (f[0] != f[1]) {
            const double to = ldexp(1.0, f[0] - f[1]);
            back = ldexp(1.0, f[1] - f[0]);
#pragma unroll
            for (int i = 0; i < R; ++i) vi[i] *= to;
        }
    }
    // without SKIPZ always taken: the transform in a block of its own keeps the compiler from
    // moving its loads and addresses up into the load phase, whose registers they would spill
    int go = 1;
    if constexpr (SKIPZ) go = !(fixed[0] && fixed[1]);
    else asm volatile("" : "+s"(go));
    if (go) {
        F::forward(vr, vi, s, a.tw, t);
        F::pin(vr, vi);
        using S = PairSpectrum<LOGN>;
        const bool mir = S::mirrored(t);
        const double2* h = reinterpret_cast<const double2*>(a.H + (int64_t)tr.kern * S::LEN);
        const uint32_t first = S::row(t) + (mir ? (R / 2 - 1) * S::ROWS : 0);
        const int step = mir ? -S::ROWS : S::ROWS;
        double2 hv[R / 2];
#pragma unroll
        for (int q = 0; q < R / 2; ++q) hv[q] = at_u32(h, first + (uint32_t)(q * step));
        if (mir) {
#pragma unroll
            for (int q = 0; q < R / 2; ++q) hv[q] = make_double2(hv[q].y, hv[q].x);
        }
#pragma unroll
        for (int q = 0; q < R / 2; ++q) {
            vr[2 * q] *= hv[q].x;
            vi[2 * q] *= hv[q].x;
            vr[2 * q + 1] *= hv[q].y;
            vi[2 * q + 1] *= hv[q].y;
        }
        F::pin(vr, vi);
        F::inverse(vr, vi, s, a.tw, F::fresh(t));
        if (back != 1.0) {
#pragma unroll
            for (int i = 0; i < R; ++i) vi[i] *= back;
        }
        if (e[0] | e[1]) {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                vr[i] = ldexp(vr[i], e[0]);
                vi[i] = ldexp(vi[i], e[1]);
            }
        }
    }
    const int ts = F::fresh(t);
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        double* zo = a.z + o[w];
        if (fixed[w]) {
            for (int i = t; i < L[w]; i += NT) zo[i] = value[w];
            continue;
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int k = ts + i * NT - lam;
            if (k >= 0 && k < L[w])
                *reinterpret_cast<double*>(reinterpret_cast<char*>(zo) + (uint32_t)k * 8u) =
                    (w ? vi : vr)[i];
        }
    }
}

// RegFft's twiddle table of 2^logn points, 2^logr per thread
__global__ void k_twiddles_pair(int logn, int logr, double* __restrict__ tw) {
    const int nt = 1 << (logn - logr), q2 = nt >> logr;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < logr * (nt + q2);
         x += gridDim.x * blockDim.x) {
        const bool one = x < logr * nt;
        const int y = one ? x : x - logr * nt, m = one ? nt : q2;
        double sn, cs;
        sincospi(-2.0 * (double)((int64_t)(y % m) << (y / m)) / (double)(one ? 1 << logn : nt), &sn,
                 &cs);
        tw[2 * x] = cs;
        tw[2 * x + 1] = sn;
    }
}

// the spectrum H(f) / N of kernel blockIdx.x
template <int LOGN>
__global__ void k_spec_pair(const double* __restrict__ Hraw, double scale,
                            double* __restrict__ out) {
    using S = PairSpectrum<LOGN>;
    constexpr int n = 1 << LOGN;
    const double* h = Hraw + (int64_t)blockIdx.x * (n / 2 + 1);
    for (int x = threadIdx.x; x < S::LEN; x += blockDim.x) {
        const int e = x & 1, r = (x >> 1) % S::ROWS, q = (x >> 1) / S::ROWS;
        const int f = rev_bits<LOGN>(S::R * S::thread(r) + 2 * q + e);
        out[(int64_t)blockIdx.x * S::LEN + x] = h[f <= n / 2 ? f : n - f] * scale;
    }
}

// ------------------------------------------------------------------ plan-time FFTs (FP64)
//
// X_m, m = 0..mmax <= M, of the real sequence packed in (re, im) after the forward
// passes (bit-reversed order): X_m = ((Z_m + conj Z_{M-m}) - i e^{-2 pi i m/N} (Z_m - conj Z_{M-m})) / 2
template <int LOGM, int NT, class Out>
__device__ __forceinline__ void real_dft_out(const CBuf<double>& buf, const double* __restrict__ tw,
                                             int mmax, Out&& out) {
    constexpr int M = 1 << LOGM;
    for (int m = threadIdx.x; m <= mmax; m += NT) {
        double xr, xi;
        if (m == 0 || m == M) {
            double zr, zi;
            buf.get(0, zr, zi);
            xr = m == 0 ? zr + zi : zr - zi;
            xi = 0.0;
        } else {
            double zkr, zki, zmr, zmi;
            buf.get(rev_bits<LOGM>(m), zkr, zki);
            buf.get(rev_bits<LOGM>(M - m), zmr, zmi);
            const double Ar = zkr + zmr, Ai = zki - zmi, Dr = zkr - zmr, Di = zki + zmi;
            const double er = tw[2 * m], ei = tw[2 * m + 1];
            const double pr = er * Dr - ei * Di, pim = er * Di + ei * Dr;
            xr = 0.5 * (Ar + pim);
            xi = 0.5 * (Ai - pr);
        }
        out(m, xr, xi);
    }
}

// symbol on the n_r = 2M grid: H(m) = t_0 + 2 sum_k t_k cos(2 pi k m / n_r), the real DFT
// of the even kernel h (h_0 = t_0, h_k = h_{n_r-k} = t_k for k <= K)
template <int LOGM, int NT>
__global__ __launch_bounds__(NT) void k_spec_fft(const double* __restrict__ taps,
                                                 const int64_t* __restrict__ toff,
                                                 const int64_t* __restrict__ tcnt,
                                                 const double* __restrict__ tw,
                                                 double* __restrict__ H) {
    constexpr int M = 1 << LOGM, NR = 2 * M;
    __shared__ __align__(16) unsigned char smem[2 * M * sizeof(double)];
    const CBuf<double> buf = make_cbuf<double>(smem, M);
    const int g = blockIdx.x;
    const double* t = taps + toff[g];
    const int K = (int)tcnt[g] - 1;
    for (int i = threadIdx.x; i < NR; i += NT) {
        double v = 0.0;
        if (i <= K) v = t[i];
        else if (i >= NR - K) v = t[NR - i];
        buf.put_part(i >> 1, i & 1, v);
    }
    __syncthreads();
    fwd_passes<double, LOGM, NT, LOGM>(buf, tw);
    double* Hg = H + (int64_t)g * (M + 1);
    real_dft_out<LOGM, NT>(buf, tw, M, [&](int m, double xr, double) { Hg[m] = xr; });
}

// taps by decimation in time: for an interval of n = R * 2M samples,
//   t_k = (1/n) sum_{b<R} Re[ e^{2 pi i b k / n} conj(X_b(k)) ],  X_b = real DFT over a of
//   Q(R a + b), Q(m) = q(min(m, n - m)) the inverse PSD on the interval's grid.
// Block (b, g) writes Re[...] for k <= K to row poff[g] + b of part; k_taps_sum adds over b.
template <int LOGM, int NT>
__global__ __launch_bounds__(NT) void k_taps_fft(const int32_t* __restrict__ kid,
                                                 const int32_t* __restrict__ klen,
                                                 const double* __restrict__ kpar,
                                                 const int64_t* __restrict__ tcnt, double f_samp,
                                                 const double* __restrict__ tw, int kstride,
                                                 const int64_t* __restrict__ poff,
                                                 double* __restrict__ part, int what) {
    constexpr int M = 1 << LOGM, NR = 2 * M;
    __shared__ __align__(16) unsigned char smem[2 * M * sizeof(double)];
    const CBuf<double> buf = make_cbuf<double>(smem, M);
    const int gi = blockIdx.y;
    const int g = kid[gi];
    const int64_t n = klen[g];
    const int R = (int)(n / NR);
    const int b = blockIdx.x;
    if (b >= R) return;
    const double sigma = kpar[3 * g], fk = kpar[3 * g + 1], al = kpar[3 * g + 2];
    for (int i = threadIdx.x; i < NR; i += NT) {
        int64_t m = (int64_t)R * i + b;
        if (m > n - m) m = n - m;
        buf.put_part(i >> 1, i & 1, inv_psd_at(m, n, f_samp, sigma, fk, al, what));
    }
    __syncthreads();
    fwd_passes<double, LOGM, NT, LOGM>(buf, tw);
    const int K = (int)tcnt[g] - 1;
    double* out = part + (poff[gi] + b) * kstride;
    real_dft_out<LOGM, NT>(buf, tw, K, [&](int k, double xr, double xi) {
        double sn, cs;
        sincospi(2.0 * (double)((int64_t)b * k % n) / (double)n, &sn, &cs);
        out[k] = cs * xr + sn * xi;
    });
}

// taps of kernel kid[gi] = window / n times the sum of its partial rows [poff[gi],
// poff[gi + 1]) of part, in order
__global__ void k_taps_sum(const int32_t* __restrict__ kid, const int32_t* __restrict__ klen,
                           const int64_t* __restrict__ toff, const int64_t* __restrict__ tcnt,
                           const double* __restrict__ part, int kstride,
                           const int64_t* __restrict__ poff, int lam, int window,
                           double* __restrict__ t) {
    const int gi = blockIdx.y;
    const int g = kid[gi];
    const int64_t n = klen[g];
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < tcnt[g];
         k += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0;
        for (int64_t b = poff[gi]; b < poff[gi + 1]; ++b) s += part[b * kstride + k];
        t[toff[g] + k] = s * window_at(k, lam, window) / (double)n;
    }
}

// Taps of any interval length n by chirp transforms (Bluestein 1970: m k = (m^2 + k^2 -
// (k - m)^2) / 2 turns a DFT at n points into a convolution).  The cosine sum over the
// frequencies m = 0 .. n/2 is cut into segments of M - K frequencies; with m = m0 + i,
//   sum_i a_{m0+i} e^{-2 pi i (m0 + i) k / n} = e^{-pi i (k^2 + 2 m0 k) / n}
//       sum_i (a_{m0+i} e^{-pi i i^2 / n}) e^{pi i (k - i)^2 / n},   k = 0 .. K,
// one circular convolution of M points per segment with a chirp that depends on n alone
// (k_czt_chirp: its transform, one block per length).  Phases are reduced mod 2n in integers.
// The direct sums (k_cos_transform) cost n/2 rotations per lag.  Whole FP64 plan of 256
// intervals of distinct length, direct / chirps: about 40009 samples and 2049 lags 4.99 / 1.86
// ms, 8195 samples 1.72 / 1.08; error of the taps against extended precision, relative to
// their norm, 0.7-6.8e-15 / 0.2-6.4e-16.
// A launch holds the chirps (128 KB a length) and the partial rows of at most kCztScratch; more
// kernels go in turn.  A workgroup adds up several segments where an interval has more than
// kCztMaxRows.
struct CztSeg {
    int32_t g;       // kernel
    int32_t chirp;   // its length's chirp
    int64_t m0, m1;  // frequencies
};
constexpr int64_t kCztScratch = (int64_t)128 << 20, kCztMaxRows = 1024;

template <int LOGM, int NT>
__global__ __launch_bounds__(NT) void k_czt_chirp(const int32_t* __restrict__ len, int lam,
                                                  const double* __restrict__ tw,
                                                  double2* __restrict__ chirp) {
    constexpr int M = 1 << LOGM;
    __shared__ __align__(16) unsigned char smem[2 * M * sizeof(double)];
    const CBuf<double> buf = make_cbuf<double>(smem, M);
    const int64_t n = len[blockIdx.x];
    const int K = (int)(n - 1 < lam ? n - 1 : lam);
    for (int i = threadIdx.x; i < M; i += NT) {
        const int64_t d = i <= K ? i : M - i;  // |k - i|: lags up to K, and the M - K - 1 below 0
        double sn, cs;
        sincospi((double)(d * d % (2 * n)) / (double)n, &sn, &cs);
        buf.put(i, cs, sn);
    }
    __syncthreads();
    fwd_passes<double, LOGM, NT, LOGM>(buf, tw);
    double2* out = chirp + (int64_t)blockIdx.x * M;
    for (int i = threadIdx.x; i < M; i += NT) {  // in the order of the forward transform
        double2 z;
        buf.get(i, z.x, z.y);
        out[i] = z;
    }
}

template <int LOGM, int NT>
__global__ __launch_bounds__(NT) void k_taps_czt(const CztSeg* __restrict__ seg,
                                                 const int32_t* __restrict__ klen,
                                                 const double* __restrict__ kpar, int lam,
                                                 double f_samp, const double* __restrict__ tw,
                                                 const double2* __restrict__ chirp, int kstride,
                                                 double* __restrict__ part, int what) {
    constexpr int M = 1 << LOGM;
    __shared__ __align__(16) unsigned char smem[2 * M * sizeof(double)];
    const CBuf<double> buf = make_cbuf<double>(smem, M);
    const CztSeg sg = seg[blockIdx.x];
    const int64_t n = klen[sg.g];
    const int K = (int)(n - 1 < lam ? n - 1 : lam);
    const double sigma = kpar[3 * sg.g], fk = kpar[3 * sg.g + 1], al = kpar[3 * sg.g + 2];
    const double2* ch = chirp + (int64_t)sg.chirp * M;
    double* out = part + (int64_t)blockIdx.x * kstride;
    for (int64_t m0 = sg.m0; m0 < sg.m1; m0 += M - K) {
        for (int i = threadIdx.x; i < M; i += NT) {
            const int64_t m = m0 + i;
            double re = 0.0, im = 0.0;
            if (i < M - K && 2 * m <= n) {
                const double a = (m == 0 || 2 * m == n ? 1.0 : 2.0) *
                                 inv_psd_at(m, n, f_samp, sigma, fk, al, what);
                double sn, cs;
                sincospi((double)((int64_t)i * i % (2 * n)) / (double)n, &sn, &cs);
                re = a * cs;
                im = -a * sn;
            }
            buf.put(i, re, im);
        }
        __syncthreads();
        fwd_passes<double, LOGM, NT, LOGM>(buf, tw);
        for (int i = threadIdx.x; i < M; i += NT) {
            const double2 z = ch[i];
            double re, im;
            buf.get(i, re, im);
            buf.put(i, re * z.x - im * z.y, re * z.y + im * z.x);
        }
        __syncthreads();
        inv_passes<double, LOGM, NT, LOGM>(buf, tw);
        for (int k = threadIdx.x; k <= K; k += NT) {
            double sn, cs, re, im;
            sincospi((double)((int64_t)k * (k + 2 * m0) % (2 * n)) / (double)n, &sn, &cs);
            buf.get(k, re, im);
            const double r = (cs * re + sn * im) * (1.0 / M);
            out[k] = m0 == sg.m0 ? r : out[k] + r;
        }
        __syncthreads();  // the next segment overwrites the buffer
    }
}

constexpr int kPlanLogM = 13;  // plan-time FP64 FFTs: n_r = 16384 real points
constexpr int kPlanNT = 512;
// Taps by chirp transforms: for lags that leave a segment at least a quarter of the transform,
// from 4096 samples with 512 lags or more and from 6144 with fewer (by the interval alone, so that
// an interval's taps do not depend on the others).  A plan in us, direct / chirps, of one interval,
// of 16 and of 256: 4097 samples and 64 lags 492 / 498, 540 / 552, 1300 / 1327; 2048 lags 510 / 517,
// 554 / 563, 1665 / 1400; 6001 samples and 64 lags 514 / 502, 582 / 571, 1650 / 1650; 2048 lags 535 /
// 517, 600 / 590, 2160 / 1720; 12289 samples and 64 lags 597 / 514, 722 / 646, 2875 / 2760.
// mm_tap_derivatives, three transforms: one interval of 4097 samples 250 / 320-350, of 6001 316 /
// 325-360, of 8195 396 / 335-370; 256 of 4097 with 512 lags 880 / 820.
constexpr int64_t kCztMinLen = 4096, kCztMinLenFew = 6144, kCztFewLags = 512, kCztMaxLag = 6144;

template <typename T, int LOGM>
int launch_logm(const ToepArgs<T>& a_in, int64_t n_tiles, hipStream_t st) {
    constexpr int NT = tile_threads<LOGM>();
    ToepArgs<T> a = a_in;
    a.n_tiles = n_tiles;
    const unsigned gx = (unsigned)xcd_grid(n_tiles);
    if (a.skip_zero) {
        const dim3 grid((unsigned)n_tiles, a.layers > 1 ? (unsigned)a.layers : 1u);
        if (a.mode == 0)
            hipLaunchKernelGGL((k_toeplitz<T, LOGM, NT, 0, true>), grid, dim3(NT), 0, st, a);
        else
            hipLaunchKernelGGL((k_toeplitz<T, LOGM, NT, 1, true>), grid, dim3(NT), 0, st, a);
    } else {
        switch (a.mode) {
            case 0: hipLaunchKernelGGL((k_toeplitz<T, LOGM, NT, 0, false>), dim3(gx), dim3(NT), 0, st, a); break;
            case 1: hipLaunchKernelGGL((k_toeplitz<T, LOGM, NT, 1, false>), dim3(gx), dim3(NT), 0, st, a); break;
            case 2: hipLaunchKernelGGL((k_toeplitz<T, LOGM, NT, 2, false>), dim3(gx), dim3(NT), 0, st, a); break;
            default: hipLaunchKernelGGL((k_toeplitz<T, LOGM, NT, 3, false>), dim3(gx), dim3(NT), 0, st, a); break;
        }
    }
    MM_HIP(hipGetLastError());
    return MM_OK;
}

template <int LOGN>
int launch_pair(const ToepArgs<double>& a_in, int64_t n_pairs, hipStream_t st) {
    ToepArgs<double> a = a_in;
    a.n_tiles = n_pairs;
    const dim3 g((unsigned)xcd_grid(n_pairs)), gz((unsigned)n_pairs), nt(RegFft<LOGN>::NT);
    if (a.skip_zero) {
        if (a.mode == 0)
            hipLaunchKernelGGL((k_toeplitz_pair<LOGN, 0, true>), gz, nt, 0, st, a);
        else
            hipLaunchKernelGGL((k_toeplitz_pair<LOGN, 1, true>), gz, nt, 0, st, a);
    } else {
        switch (a.mode) {
            case 0: hipLaunchKernelGGL((k_toeplitz_pair<LOGN, 0, false>), g, nt, 0, st, a); break;
            case 1: hipLaunchKernelGGL((k_toeplitz_pair<LOGN, 1, false>), g, nt, 0, st, a); break;
            case 2: hipLaunchKernelGGL((k_toeplitz_pair<LOGN, 2, false>), g, nt, 0, st, a); break;
            default: hipLaunchKernelGGL((k_toeplitz_pair<LOGN, 3, false>), g, nt, 0, st, a); break;
        }
    }
    MM_HIP(hipGetLastError());
    return MM_OK;
}

template <typename T>
int launch(const ToepArgs<T>& a, const FftTiling& ft, hipStream_t st) {
    if (ft.n_tiles == 0) return MM_OK;
    const int64_t n = ft.n_tiles;
    if constexpr (sizeof(T) == 4) {
        switch (ft.logm) {
            case 10: return launch_logm<T, 10>(a, n, st);
            case 11: return launch_logm<T, 11>(a, n, st);
            case 12: return launch_logm<T, 12>(a, n, st);
            case 13: return launch_logm<T, 13>(a, n, st);
            case 14: return launch_logm<T, 14>(a, n, st);
        }
    } else {
        switch (ft.logm) {
            case 10: return launch_logm<T, 10>(a, n, st);
            case 11: return launch_pair<12>(a, n / 2, st);
            case 12: return launch_pair<13>(a, n / 2, st);
            case 13: return launch_logm<T, 13>(a, n, st);
        }
    }
    set_error("no overlap-save kernel for log2(M) = %d", ft.logm);
    return MM_ERR_ARG;
}

// (I, Q, U) per pixel -> (I, Q, U, 0) in T, one aligned 16/32-byte record per pixel
template <typename T>
__global__ void k_pack_map(const double* __restrict__ x, int64_t n_obs, T* __restrict__ xp) {
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n_obs;
         c += (int64_t)gridDim.x * blockDim.x) {
        xp[4 * c] = (T)x[3 * c];
        xp[4 * c + 1] = (T)x[3 * c + 1];
        xp[4 * c + 2] = (T)x[3 * c + 2];
        xp[4 * c + 3] = (T)0;
    }
}

template <typename T>
int pack_map(mm_plan_t pl, const double* x, T* xp) {
    int64_t g = (pl->n_obs + 255) / 256;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(k_pack_map<T>, dim3(g), dim3(256), 0, pl->stream, x, pl->n_obs, xp);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

template <typename T>
ToepArgs<T> base_args(mm_plan_t pl, const FftTiling& ft) {
    ToepArgs<T> a{};
    a.cid = pl->cid.p;
    a.tiles = ft.tiles.p;
    a.lam = pl->opts.lambda;
    if constexpr (sizeof(T) == 8) {
        a.H = ft.H64.p;
        a.tw = ft.tw64.p;
        a.w = pl->w64.p;
    } else {
        a.H = ft.H32.p;
        a.tw = ft.tw32.p;
        a.w = pl->w32.p;
    }
    return a;
}

// t0[g] = t_0 of kernel g (the diagonal of its Toeplitz block)
__global__ void k_gather_t0(const double* __restrict__ taps, const int64_t* __restrict__ toff,
                            int32_t nk, double* __restrict__ t0) {
    const int32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < nk) t0[g] = taps[toff[g]];
}

constexpr int64_t kCus = 256;  // compute units of the chip
constexpr int kMaxLogM64 = 13, kMaxLogM32 = 14, kMinLogM = 10;

// tiles of an interval of n samples, at most lmax outputs each
int64_t tiles_of(int64_t n, int64_t lmax, bool paired) {
    return paired ? 2 * ((n + 2 * lmax - 1) / (2 * lmax)) : (n + lmax - 1) / lmax;
}

int64_t count_tiles(const std::vector<int64_t>& off, int64_t lmax, bool paired) {
    int64_t n = 0;
    for (size_t j = 0; j + 1 < off.size(); ++j) n += tiles_of(off[j + 1] - off[j], lmax, paired);
    return n;
}

// FP64 lengths n_r = 2^(l + 1) whose tiles go in pairs (k_toeplitz_pair): 4096 and 8192.  2048
// points serve short intervals, often of one tile; 16384 points would need 128 KB of LDS, one
// workgroup per CU, as the LDS-resident tile does, and are taken from lambda of about 2900
bool pair_length(bool fp64, int l) { return fp64 && (l == 11 || l == 12); }

}  // namespace

// ------------------------------------------------------------------ host: kernels

// tw[q] = exp(-2 pi i q / n), q < count, as (re, im) pairs
int fft_twiddles(mm_plan_t pl, int64_t count, int64_t n, double* tw) {
    hipLaunchKernelGGL(k_twiddles, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, pl->stream,
                       count, n, tw, (float*)nullptr);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

// Windowed taps t_0..t_K of every distinct kernel (what = 0) or of the derivative of the
// inverse PSD with respect to sigma, f_knee or alpha (what = 1, 2, 3), on the host, flat
// with offsets toff and counts tcnt [App. D: the Toeplitz row is the inverse DFT of the
// inverse PSD on the interval's grid].
int kernel_taps_dev(mm_plan_t pl, int what, DBuf<double>& d_t, std::vector<int64_t>& toff,
                    std::vector<int64_t>& tcnt) {
    hipStream_t st = pl->stream;
    const int32_t nk = pl->n_kern;
    const int lam = pl->opts.lambda;
    std::vector<int64_t> aoff(nk), acnt(nk), nper(nk), jcnt(nk);
    toff.assign(nk, 0);
    tcnt.assign(nk, 0);
    std::vector<double> kpar(3 * nk);
    int64_t atot = 0, ttot = 0;
    int64_t amax = 0;
    constexpr int64_t kNs = (int64_t)2 << kPlanLogM, kCz = (int64_t)1 << kPlanLogM;
    // lengths that are multiples of the plan-time transform by decimation in time, other long
    // ones by chirp transforms, short ones by direct sums
    std::vector<int32_t> fft_ids, czt_ids;
    bool direct = false;
    for (int g = 0; g < nk; ++g) {
        const int64_t n = pl->h_kern_len[g];
        const int64_t K = std::min<int64_t>(lam, n - 1);
        const bool by_fft = n % kNs == 0 && K < kNs / 2;
        const bool by_czt =
            !by_fft && n >= (K < kCztFewLags ? kCztMinLenFew : kCztMinLen) && K <= kCztMaxLag;
        if (by_fft) fft_ids.push_back(g);
        else if (by_czt) czt_ids.push_back(g);
        else direct = true;
        aoff[g] = atot;
        acnt[g] = by_fft || by_czt ? 0 : n / 2 + 1;
        atot += acnt[g];
        amax = std::max(amax, acnt[g]);
        nper[g] = n;
        tcnt[g] = std::min<int64_t>(lam, n - 1) + 1;
        jcnt[g] = tcnt[g];
        toff[g] = ttot;
        ttot += tcnt[g];
        kpar[3 * g] = pl->h_kern_psd[g].sigma;
        kpar[3 * g + 1] = pl->h_kern_psd[g].f_knee;
        kpar[3 * g + 2] = pl->h_kern_psd[g].alpha;
    }
    // the kernels' tables, in one buffer and one copy
    std::vector<int64_t> tab;
    tab.reserve(9 * (size_t)nk + (nk + 1) / 2);
    for (const auto* v : {&aoff, &acnt, &nper, &jcnt, &toff, &tcnt})
        tab.insert(tab.end(), v->begin(), v->end());
    tab.resize(9 * (size_t)nk + (nk + 1) / 2);
    std::memcpy(tab.data() + 6 * (size_t)nk, kpar.data(), 3 * (size_t)nk * 8);
    std::memcpy(tab.data() + 9 * (size_t)nk, pl->h_kern_len.data(), (size_t)nk * 4);
    DBuf<int64_t> d_tab;
    DBuf<double> d_a;
    MM_TRY(d_tab.alloc(tab.size()));
    MM_TRY(d_a.alloc(std::max<int64_t>(1, atot)));
    MM_TRY(d_t.alloc(ttot));
    MM_HIP(hipMemcpyAsync(d_tab.p, tab.data(), tab.size() * 8, hipMemcpyHostToDevice, st));
    const int64_t *d_aoff = d_tab.p, *d_acnt = d_aoff + nk, *d_nper = d_acnt + nk,
                  *d_jcnt = d_nper + nk, *d_toff = d_jcnt + nk, *d_tcnt = d_toff + nk;
    const double* d_kpar = reinterpret_cast<const double*>(d_tcnt + nk);
    const int32_t* d_klen = reinterpret_cast<const int32_t*>(d_kpar + 3 * (size_t)nk);
    if (direct) {
        const int gx = (int)std::max<int64_t>(1, std::min<int64_t>((amax + 255) / 256, 1024));
        hipLaunchKernelGGL(k_inv_psd, dim3(gx, nk), dim3(256), 0, st, d_klen, d_kpar,
                           d_aoff, d_acnt, pl->opts.f_samp, d_a.p, nk, what);
        MM_HIP(hipGetLastError());
        const int64_t jmax = *std::max_element(jcnt.begin(), jcnt.end());
        hipLaunchKernelGGL(k_cos_transform, dim3((jmax + kCtThreads - 1) / kCtThreads, nk),
                           dim3(kCtThreads), 0, st, d_a.p, d_aoff, d_acnt, d_nper, d_jcnt,
                           d_toff, d_t.p, nk);
        MM_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_taps_finish, dim3(std::max<int64_t>(1, (jmax + 255) / 256), nk),
                           dim3(256), 0, st, d_t.p, d_toff, d_tcnt, d_klen, lam,
                           pl->opts.window, nk);
        MM_HIP(hipGetLastError());
    }
    DBuf<double> d_tw, d_part, d_part_c;
    DBuf<int32_t> d_kid, d_kid_c, d_clen;
    DBuf<int64_t> d_poff, d_poff_c;
    DBuf<CztSeg> d_seg;
    DBuf<double2> d_chirp;
    if (!fft_ids.empty() || !czt_ids.empty()) {
        MM_TRY(d_tw.alloc(kNs));
        MM_TRY(fft_twiddles(pl, kNs / 2, kNs, d_tw.p));
    }
    // partial rows [poff[i], poff[i + 1]) of the kernels ids, added into their taps
    auto sum_rows = [&](const std::vector<int32_t>& ids, const std::vector<int64_t>& poff,
                        DBuf<int32_t>& kid, DBuf<int64_t>& po) -> int {
        MM_TRY(kid.alloc(ids.size()));
        MM_TRY(po.alloc(poff.size()));
        MM_HIP(hipMemcpyAsync(kid.p, ids.data(), ids.size() * 4, hipMemcpyHostToDevice, st));
        MM_HIP(hipMemcpyAsync(po.p, poff.data(), poff.size() * 8, hipMemcpyHostToDevice, st));
        return MM_OK;
    };
    if (!fft_ids.empty()) {
        const int nf = (int)fft_ids.size();
        int rmax = 1, kmax = 1;
        std::vector<int64_t> poff(1, 0);
        for (int g : fft_ids) {
            const int R = (int)(pl->h_kern_len[g] / kNs);
            poff.push_back(poff.back() + R);
            rmax = std::max(rmax, R);
            kmax = std::max<int>(kmax, (int)tcnt[g]);
        }
        MM_TRY(sum_rows(fft_ids, poff, d_kid, d_poff));
        MM_TRY(d_part.alloc((size_t)poff[nf] * kmax));
        hipLaunchKernelGGL((k_taps_fft<kPlanLogM, kPlanNT>), dim3(rmax, nf), dim3(kPlanNT), 0, st,
                           d_kid.p, d_klen, d_kpar, d_tcnt, pl->opts.f_samp, d_tw.p, kmax,
                           d_poff.p, d_part.p, what);
        MM_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_taps_sum, dim3((kmax + 255) / 256, nf), dim3(256), 0, st, d_kid.p,
                           d_klen, d_toff, d_tcnt, d_part.p, kmax, d_poff.p, lam,
                           pl->opts.window, d_t.p);
        MM_HIP(hipGetLastError());
    }
    // kernels of one length are neighbours and share its chirp
    std::sort(czt_ids.begin(), czt_ids.end(), [&](int32_t a, int32_t b) {
        return pl->h_kern_len[a] != pl->h_kern_len[b] ? pl->h_kern_len[a] < pl->h_kern_len[b]
                                                      : a < b;
    });
    for (size_t i0 = 0, i1; i0 < czt_ids.size(); i0 = i1) {
        int kmax = 1;
        for (size_t i = i0; i < czt_ids.size(); ++i)
            kmax = std::max<int>(kmax, (int)tcnt[czt_ids[i]]);
        std::vector<int32_t> ids, lens;
        std::vector<int64_t> poff(1, 0);
        std::vector<CztSeg> seg;
        for (i1 = i0; i1 < czt_ids.size(); ++i1) {
            const int32_t g = czt_ids[i1], n = pl->h_kern_len[g];
            const int64_t step = kCz - (tcnt[g] - 1), ns = n / 2 / step + 1;
            const int64_t run = (ns + kCztMaxRows - 1) / kCztMaxRows * step;
            const int64_t rows = (n / 2 + run) / run, nl = (int64_t)lens.size() + 1;
            if (i1 > i0 && nl * kCz * 16 + ((int64_t)seg.size() + rows) * kmax * 8 > kCztScratch)
                break;
            if (lens.empty() || lens.back() != n) lens.push_back(n);
            for (int64_t m0 = 0; m0 <= n / 2; m0 += run)
                seg.push_back({g, (int32_t)lens.size() - 1, m0, std::min<int64_t>(m0 + run, n / 2 + 1)});
            ids.push_back(g);
            poff.push_back((int64_t)seg.size());
        }
        MM_TRY(sum_rows(ids, poff, d_kid_c, d_poff_c));
        MM_TRY(d_seg.alloc(seg.size()));
        MM_TRY(d_clen.alloc(lens.size()));
        MM_TRY(d_chirp.alloc(lens.size() * kCz));
        MM_TRY(d_part_c.alloc(seg.size() * kmax));
        MM_HIP(hipMemcpyAsync(d_seg.p, seg.data(), seg.size() * sizeof(CztSeg),
                              hipMemcpyHostToDevice, st));
        MM_HIP(hipMemcpyAsync(d_clen.p, lens.data(), lens.size() * 4, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL((k_czt_chirp<kPlanLogM, kPlanNT>), dim3((unsigned)lens.size()),
                           dim3(kPlanNT), 0, st, d_clen.p, lam, d_tw.p, d_chirp.p);
        MM_HIP(hipGetLastError());
        hipLaunchKernelGGL((k_taps_czt<kPlanLogM, kPlanNT>), dim3((unsigned)seg.size()),
                           dim3(kPlanNT), 0, st, d_seg.p, d_klen, d_kpar, lam,
                           pl->opts.f_samp, d_tw.p, (const double2*)d_chirp.p, kmax, d_part_c.p,
                           what);
        MM_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_taps_sum, dim3((kmax + 255) / 256, (unsigned)ids.size()), dim3(256), 0,
                           st, d_kid_c.p, d_klen, d_toff, d_tcnt, d_part_c.p, kmax, d_poff_c.p, lam,
                           pl->opts.window, d_t.p);
        MM_HIP(hipGetLastError());
    }
    // the temporaries above are released in stream order after the kernels that read them
    return MM_OK;
}

int kernel_taps(mm_plan_t pl, int what, std::vector<double>& taps, std::vector<int64_t>& toff,
                std::vector<int64_t>& tcnt) {
    DBuf<double> d_t;
    MM_TRY(kernel_taps_dev(pl, what, d_t, toff, tcnt));
    taps.resize(d_t.n);
    MM_HIP(hipMemcpyAsync(taps.data(), d_t.p, d_t.n * 8, hipMemcpyDeviceToHost, pl->stream));
    MM_HIP(hipStreamSynchronize(pl->stream));
    return MM_OK;
}

int host_taps(mm_plan_t pl) {
    if (!pl->h_taps.empty() || pl->taps.n == 0) return MM_OK;
    std::vector<double> t(pl->taps.n);
    MM_HIP(hipMemcpyAsync(t.data(), pl->taps.p, t.size() * 8, hipMemcpyDeviceToHost, pl->stream));
    MM_HIP(hipStreamSynchronize(pl->stream));
    pl->h_taps.swap(t);
    return MM_OK;
}

int build_kernels(mm_plan_t pl) {
    hipStream_t st = pl->stream;
    // distinct kernels: identical (sigma, f_knee, alpha, length) share taps and spectra
    std::map<std::tuple<double, double, double, int64_t>, int32_t> seen;
    pl->h_int_kern.resize(pl->n_int);
    pl->h_kern_len.clear();
    pl->h_kern_psd.clear();
    for (int32_t j = 0; j < pl->n_int; ++j) {
        const int64_t n = pl->h_off[j + 1] - pl->h_off[j];
        const mm_psd& p = pl->h_psd[j];
        const auto key = std::make_tuple(p.sigma, p.f_knee, p.alpha, n);
        auto it = seen.find(key);
        if (it == seen.end()) {
            const int32_t id = (int32_t)pl->h_kern_len.size();
            seen.emplace(key, id);
            pl->h_kern_len.push_back((int32_t)n);
            pl->h_kern_psd.push_back(p);
            pl->h_int_kern[j] = id;
        } else {
            pl->h_int_kern[j] = it->second;
        }
    }
    const int32_t nk = (int32_t)pl->h_kern_len.size();
    pl->n_kern = nk;
    // taps stay on the device (the spectra are formed there); the host copy is fetched on
    // first use
    pl->h_taps.clear();
    MM_TRY(kernel_taps_dev(pl, 0, pl->taps, pl->h_taps_off, pl->h_taps_cnt));
    MM_TRY(pl->taps_off.alloc(nk));
    MM_TRY(pl->taps_cnt.alloc(nk));
    MM_HIP(hipMemcpyAsync(pl->taps_off.p, pl->h_taps_off.data(), nk * 8, hipMemcpyHostToDevice, st));
    MM_HIP(hipMemcpyAsync(pl->taps_cnt.p, pl->h_taps_cnt.data(), nk * 8, hipMemcpyHostToDevice, st));
    MM_TRY(pl->kern_t0.alloc(nk));
    hipLaunchKernelGGL(k_gather_t0, dim3((nk + 255) / 256), dim3(256), 0, st, pl->taps.p,
                       pl->taps_off.p, nk, pl->kern_t0.p);
    MM_HIP(hipGetLastError());
    std::vector<double> t0(nk);
    MM_HIP(hipMemcpyAsync(t0.data(), pl->kern_t0.p, nk * 8, hipMemcpyDeviceToHost, st));
    MM_TRY(pl->int_kern.alloc(pl->n_int));
    MM_HIP(hipMemcpyAsync(pl->int_kern.p, pl->h_int_kern.data(), pl->n_int * 4,
                          hipMemcpyHostToDevice, st));
    std::vector<int64_t> lo(pl->n_int), hi(pl->n_int);
    for (int32_t j = 0; j < pl->n_int; ++j) {
        lo[j] = pl->h_off[j];
        hi[j] = pl->h_off[j + 1];
    }
    MM_TRY(pl->int_lo.alloc(pl->n_int));
    MM_TRY(pl->int_hi.alloc(pl->n_int));
    MM_HIP(hipMemcpyAsync(pl->int_lo.p, lo.data(), pl->n_int * 8, hipMemcpyHostToDevice, st));
    MM_HIP(hipMemcpyAsync(pl->int_hi.p, hi.data(), pl->n_int * 8, hipMemcpyHostToDevice, st));
    MM_HIP(hipStreamSynchronize(st));
    for (int g = 0; g < nk; ++g) {
        // t_0 = 0 happens only for a 1-sample interval with 1/f noise (its mean, the
        // sample itself, is not weighted); a negative or non-finite diagonal is an error
        if (!(t0[g] >= 0.0) || !std::isfinite(t0[g])) {
            set_error("kernel of interval length %d has t_0 = %g < 0", pl->h_kern_len[g], t0[g]);
            return MM_ERR_NOT_SPD;
        }
    }
    return MM_OK;
}

// ------------------------------------------------------------------ host: tiling + spectra

int build_tiling(mm_plan_t pl, FftTiling& ft, bool fp64, int n_r_request) {
    hipStream_t st = pl->stream;
    const int lam = pl->opts.lambda;
    const int maxlogm = fp64 ? kMaxLogM64 : kMaxLogM32;
    int logm = 0;
    if (n_r_request > 0) {
        int l = 0;
        while ((2 << l) < n_r_request) ++l;
        if ((2 << l) != n_r_request || l < kMinLogM || l > maxlogm) {
            set_error("FFT length %d must be a power of two in [%d, %d]", n_r_request,
                      2 << kMinLogM, 2 << maxlogm);
            return MM_ERR_ARG;
        }
        if ((2 << l) <= 2 * lam) {
            set_error("FFT length %d too short for lambda = %d", n_r_request, lam);
            return MM_ERR_ARG;
        }
        logm = l;
    } else {
        // Smallest modelled time: workgroups x points x (log2 n_r + 4), a pair of FP64 tiles being
        // one workgroup of 2 n_r points; fewer workgroups than CUs count as one per CU, since such a
        // launch takes the time of one.  Doubled
        //  - in FP32 for a tile whose LDS leaves room for only one resident tile per CU (160 KB): a
        //    second tile hides the other's window load (32768-point tiles at lambda = 4096 take
        //    1.27x the time of 16384-point ones, for 0.72x the modelled work);
        //  - in FP64 for the lengths that do not go in pairs: N^-1 of a TOD of 2^24 samples
        //    takes 11.4 ns per tile of 2048 points, 24.3 per pair of 4096, 58 of 8192 and 87 per tile
        //    of 16384: 2.0, 1, 1.12 and 1.6 times the model's; at 2^22 samples, where a CU takes two
        //    tiles of 16384 after each other, these count 2.1.
        // Pairs of 8192 points count 6% more (as in A x; N^-1 12%).  A x in us: 2^18 samples, lambda
        // = 512: 2048 points 17.5, 4096 21.4; 2^18, lambda = 1024: 64 pairs of 4096 points 21.3, 32 of
        // 8192 29.4; 2^21, lambda = 512: 4096 44.6, 8192 46.4; 2^24, lambda = 512: 4096 233, 8192 240;
        // 2^22, lambda = 2700: 8192 91, 16384 95.7, lambda = 2850: 99.3, 96.0; 2^24, lambda = 2800:
        // 325, 334, lambda = 3072: 357, 336.  FP32, 2^20, lambda = 2048: 32.0 with 256 tiles of 8192,
        // 34.9 with 96 of 16384
        double best = 0.0;
        for (int l = kMinLogM; l <= maxlogm; ++l) {
            const int64_t nr = (int64_t)2 << l;
            const int64_t lmax = nr - 2 * (int64_t)lam;
            if (lmax < nr / 4) continue;
            const bool paired = pair_length(fp64, l);
            const int64_t wgs = count_tiles(pl->h_off, lmax, paired) / (paired ? 2 : 1);
            double factor = l == kMaxLogM32 || (fp64 && !paired) ? 2.0 : 1.0;
            if (fp64 && l == kMaxLogM64) factor = 2.1;
            if (paired) factor = l == 12 ? 2.12 : 2.0;  // 2 n_r points
            const double cost = (double)std::max<int64_t>(wgs, kCus) * (double)nr * (l + 5) * factor;
            if (logm == 0 || cost < best) {
                best = cost;
                logm = l;
            }
        }
        if (logm == 0) {
            set_error("lambda = %d too large for the %s overlap-save tile (n_r <= %d)", lam,
                      fp64 ? "FP64" : "FP32", 2 << maxlogm);
            return MM_ERR_ARG;
        }
    }
    ft.logm = logm;
    ft.n_r = 2 << logm;
    ft.paired = pair_length(fp64, logm);
    const int M = 1 << logm;
    const int64_t lmax = (int64_t)ft.n_r - 2 * (int64_t)lam;
    // balanced tiles per interval
    std::vector<TileRec> tiles;
    int32_t prob = 0;
    for (int32_t j = 0; j < pl->n_int; ++j) {
        const int64_t a = pl->h_off[j], b = pl->h_off[j + 1], n = b - a;
        while (j >= pl->h_pint[prob + 1]) ++prob;
        const int64_t nt = tiles_of(n, lmax, ft.paired);
        const int64_t len = (n + nt - 1) / nt;
        for (int64_t i = 0; i < nt; ++i) {
            const int64_t s = a + i * len;
            const int64_t e = std::min(b, s + len);
            if (e <= s && (!ft.paired || i % 2 == 0)) break;
            // (the second tile of a pair may be empty)
            tiles.push_back({e > s ? s : tiles.back().out, a, b, (int32_t)std::max<int64_t>(e - s, 0),
                             j, pl->h_int_kern[j], prob, 0});
            if (e <= s) break;
        }
    }
    ft.n_tiles = (int64_t)tiles.size();
    MM_TRY(ft.tiles.alloc(ft.n_tiles));
    MM_HIP(hipMemcpyAsync(ft.tiles.p, tiles.data(), ft.n_tiles * sizeof(TileRec),
                          hipMemcpyHostToDevice, st));
    // twiddles exp(-2 pi i q / n_r), q < M, in FP64 (the spectra below and unpaired FP64
    // tiles) and FP32 for FP32 tiles; pairs have a table of their own
    DBuf<double> d_tw;
    double* tw64 = nullptr;
    if (fp64 && !ft.paired) {
        MM_TRY(ft.tw64.alloc(2 * M));
        tw64 = ft.tw64.p;
    } else {
        MM_TRY(d_tw.alloc(2 * M));
        tw64 = d_tw.p;
    }
    if (!fp64) MM_TRY(ft.tw32.alloc(2 * M));
    hipLaunchKernelGGL(k_twiddles, dim3((M + 255) / 256), dim3(256), 0, st, (int64_t)M,
                       (int64_t)ft.n_r, tw64, fp64 ? (float*)nullptr : ft.tw32.p);
    MM_HIP(hipGetLastError());
    // spectra H(m), m = 0..M, of every kernel on this grid
    const int32_t nk = pl->n_kern;
    DBuf<double> d_h, d_min;
    MM_TRY(d_h.alloc((size_t)nk * (M + 1)));
    MM_TRY(d_min.alloc(nk));
    const double* d_taps = pl->taps.p;
    const int64_t* d_toff = pl->taps_off.p;
    const int64_t* d_tcnt = pl->taps_cnt.p;
    if (logm <= kPlanLogM) {  // FP64 FFT of the even kernel on the tile grid
        switch (logm) {
            case 10:
                hipLaunchKernelGGL((k_spec_fft<10, 256>), dim3(nk), dim3(256), 0, st, d_taps,
                                   d_toff, d_tcnt, tw64, d_h.p);
                break;
            case 11:
                hipLaunchKernelGGL((k_spec_fft<11, 256>), dim3(nk), dim3(256), 0, st, d_taps,
                                   d_toff, d_tcnt, tw64, d_h.p);
                break;
            case 12:
                hipLaunchKernelGGL((k_spec_fft<12, 256>), dim3(nk), dim3(256), 0, st, d_taps,
                                   d_toff, d_tcnt, tw64, d_h.p);
                break;
            default:
                hipLaunchKernelGGL((k_spec_fft<kPlanLogM, kPlanNT>), dim3(nk), dim3(kPlanNT), 0, st,
                                   d_taps, d_toff, d_tcnt, tw64, d_h.p);
                break;
        }
        MM_HIP(hipGetLastError());
    } else {  // 2^15-point tiles (FP32 only): direct cosine sums
        MM_TRY(host_taps(pl));
        std::vector<int64_t> boff(nk), bcnt(nk), nper(nk, ft.n_r), jcnt(nk, M + 1), ooff(nk);
        std::vector<double> b;
        for (int g = 0; g < nk; ++g) {
            boff[g] = (int64_t)b.size();
            bcnt[g] = pl->h_taps_cnt[g];
            const double* t = pl->h_taps.data() + pl->h_taps_off[g];
            for (int64_t k = 0; k < bcnt[g]; ++k) b.push_back((k == 0 ? 1.0 : 2.0) * t[k]);
            ooff[g] = (int64_t)g * (M + 1);
        }
        DBuf<double> d_b;
        DBuf<int64_t> d_boff, d_bcnt, d_nper, d_jcnt, d_ooff;
        MM_TRY(d_b.alloc(b.size()));
        MM_TRY(d_boff.alloc(nk));
        MM_TRY(d_bcnt.alloc(nk));
        MM_TRY(d_nper.alloc(nk));
        MM_TRY(d_jcnt.alloc(nk));
        MM_TRY(d_ooff.alloc(nk));
        MM_HIP(hipMemcpyAsync(d_b.p, b.data(), b.size() * 8, hipMemcpyHostToDevice, st));
        MM_HIP(hipMemcpyAsync(d_boff.p, boff.data(), nk * 8, hipMemcpyHostToDevice, st));
        MM_HIP(hipMemcpyAsync(d_bcnt.p, bcnt.data(), nk * 8, hipMemcpyHostToDevice, st));
        MM_HIP(hipMemcpyAsync(d_nper.p, nper.data(), nk * 8, hipMemcpyHostToDevice, st));
        MM_HIP(hipMemcpyAsync(d_jcnt.p, jcnt.data(), nk * 8, hipMemcpyHostToDevice, st));
        MM_HIP(hipMemcpyAsync(d_ooff.p, ooff.data(), nk * 8, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(k_cos_transform, dim3((M + 1 + kCtThreads - 1) / kCtThreads, nk),
                           dim3(kCtThreads), 0, st, d_b.p, d_boff.p, d_bcnt.p, d_nper.p, d_jcnt.p,
                           d_ooff.p, d_h.p, nk);
        MM_HIP(hipGetLastError());
    }
    const double scale = 1.0 / (double)ft.n_r;
    if (ft.paired) {
        MM_TRY(ft.H64.alloc((size_t)nk *
                            (logm == 11 ? PairSpectrum<12>::LEN : PairSpectrum<13>::LEN)));
    } else if (fp64) {
        MM_TRY(ft.H64.alloc((size_t)nk * (M + 1)));
    } else {
        MM_TRY(ft.H32.alloc((size_t)nk * (M + 1)));
    }
    hipLaunchKernelGGL(k_spec_finish, dim3(nk), dim3(256), 0, st, d_h.p, (int64_t)(M + 1),
                       (int64_t)(M + 1), scale, fp64 && !ft.paired ? ft.H64.p : nullptr,
                       fp64 ? nullptr : ft.H32.p, d_min.p);
    if (ft.paired) {
        constexpr int lr = RegFft<12>::LOGR;
        const int ntw = logm == 11 ? RegFft<12>::TW : RegFft<13>::TW;
        MM_TRY(ft.tw64.alloc(2 * ntw));
        hipLaunchKernelGGL(k_twiddles_pair, dim3((ntw + 255) / 256), dim3(256), 0, st, logm + 1, lr,
                           ft.tw64.p);
        if (logm == 11)
            hipLaunchKernelGGL(k_spec_pair<12>, dim3((unsigned)nk), dim3(256), 0, st, d_h.p, scale,
                               ft.H64.p);
        else
            hipLaunchKernelGGL(k_spec_pair<13>, dim3((unsigned)nk), dim3(256), 0, st, d_h.p, scale,
                               ft.H64.p);
    }
    MM_HIP(hipGetLastError());
    std::vector<double> hmin(nk);
    MM_HIP(hipMemcpyAsync(hmin.data(), d_min.p, nk * 8, hipMemcpyDeviceToHost, st));
    MM_HIP(hipStreamSynchronize(st));
    for (int g = 0; g < nk; ++g) {
        // The symbol bound applies when the whole band fits in the interval; a shorter
        // interval's block is the (windowed) circulant of its own inverse PSD, which is
        // only semi-definite for 1/f noise (its mean is not weighted).
        if ((int64_t)pl->h_kern_len[g] <= 2 * (int64_t)lam) continue;
        if (!(hmin[g] > 0.0)) {
            set_error("Toeplitz symbol min %.3e <= 0 (kernel %d: sigma=%g f_knee=%g alpha=%g, "
                      "length %d): N^-1 block not positive definite",
                      hmin[g], g, pl->h_kern_psd[g].sigma, pl->h_kern_psd[g].f_knee,
                      pl->h_kern_psd[g].alpha, pl->h_kern_len[g]);
            return MM_ERR_NOT_SPD;
        }
    }
    return MM_OK;
}

// ------------------------------------------------------------------ host: launches

int pack_map64(mm_plan_t pl, const double* x) {
    return pl->n_s == 3 ? pack_map<double>(pl, x, pl->xp64.p) : MM_OK;
}

int pack_map32(mm_plan_t pl, const double* x) {
    return pl->n_s == 3 ? pack_map<float>(pl, x, pl->xp32.p) : MM_OK;
}

int toeplitz_map64(mm_plan_t pl, const double* x, double* z, const int* mask, bool skip_zero,
                   const uint8_t* int_on) {
    auto a = base_args<double>(pl, pl->fft64);
    a.skip_zero = skip_zero;
    a.int_on = skip_zero ? int_on : nullptr;
    a.x = x;
    if (pl->n_s == 3) a.xp = pl->xp64.p;
    a.mode = pl->n_s == 3 ? 0 : 1;
    a.z = z;
    a.mask = mask;
    return launch<double>(a, pl->fft64, pl->stream);
}

int toeplitz_map64_i(mm_plan_t pl, const double* xi, double* z, const uint8_t* int_on) {
    auto a = base_args<double>(pl, pl->fft64);
    a.skip_zero = 1;
    a.int_on = int_on;
    a.x = xi;
    a.mode = 1;
    a.z = z;
    return launch<double>(a, pl->fft64, pl->stream);
}

int toeplitz_map32(mm_plan_t pl, const double* x, float* z, const int* mask) {
    auto a = base_args<float>(pl, pl->fft32);
    a.x = x;
    if (pl->n_s == 3) a.xp = pl->xp32.p;
    a.mode = pl->n_s == 3 ? 0 : 1;
    a.z = z;
    a.mask = mask;
    return launch<float>(a, pl->fft32, pl->stream);
}

int toeplitz_map32_layers(mm_plan_t pl, const double* x, int64_t x_step, const float* xp,
                          int64_t xp_step, float* z, int64_t z_step, const uint8_t* int_on,
                          int64_t on_step, int layers) {
    if (layers < 1 || layers > 65535) {
        set_error("toeplitz_map32_layers: %d layers", layers);
        return MM_ERR_ARG;
    }
    auto a = base_args<float>(pl, pl->fft32);
    a.skip_zero = 1;
    a.x = x;
    a.xp = xp;
    a.mode = xp ? 0 : 1;
    a.z = z;
    a.int_on = int_on;
    a.layers = layers;
    a.x_step = x_step;
    a.xp_step = xp_step;
    a.z_step = z_step;
    a.on_step = on_step;
    return launch<float>(a, pl->fft32, pl->stream);
}

int toeplitz_tod64(mm_plan_t pl, const void* y, int y_f64, double* z) {
    auto a = base_args<double>(pl, pl->fft64);
    a.y = y;
    a.y_f64 = y_f64;
    a.mode = y_f64 ? 2 : 3;
    a.z = z;
    return launch<double>(a, pl->fft64, pl->stream);
}

int toeplitz_tod32(mm_plan_t pl, const void* y, int y_f64, float* z) {
    auto a = base_args<float>(pl, pl->fft32);
    a.y = y;
    a.y_f64 = y_f64;
    a.mode = y_f64 ? 2 : 3;
    a.z = z;
    return launch<float>(a, pl->fft32, pl->stream);
}

// ------------------------------------------------------------------ FFT length autotuner
//
// Every admissible tile length is built and its map-mode launch (gather + overlap-save,
// the kernel of A x) timed on the plan's own pointing and intervals; the fastest is
// kept.  Choices are cached per process by the interval-length profile, lambda, n_s
// and precision, so plans of the same workload tune once.

namespace {

void swap_tiling(FftTiling& a, FftTiling& b) {
    std::swap(a.logm, b.logm);
    std::swap(a.n_r, b.n_r);
    std::swap(a.n_tiles, b.n_tiles);
    std::swap(a.paired, b.paired);
    a.tiles.swap(b.tiles);
    a.H64.swap(b.H64);
    a.H32.swap(b.H32);
    a.tw64.swap(b.tw64);
    a.tw32.swap(b.tw32);
}

std::mutex g_tune_mu;
std::map<std::vector<int64_t>, int> g_tune_cache;

template <typename T>
int time_map_launch(mm_plan_t pl, FftTiling& ft, T* xp, const double* x, T* z, float* ms) {
    auto a = base_args<T>(pl, ft);
    a.x = x;
    a.xp = xp;
    a.mode = pl->n_s == 3 ? 0 : 1;
    a.z = z;
    hipEvent_t e0, e1;
    MM_HIP(hipEventCreate(&e0));
    MM_HIP(hipEventCreate(&e1));
    int s = launch<T>(a, ft, pl->stream);  // warm-up
    if (s == MM_OK) {
        (void)hipEventRecord(e0, pl->stream);
        for (int r = 0; r < 3 && s == MM_OK; ++r) s = launch<T>(a, ft, pl->stream);
        (void)hipEventRecord(e1, pl->stream);
        (void)hipEventSynchronize(e1);
        (void)hipEventElapsedTime(ms, e0, e1);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return s;
}

}  // namespace

int autotune_tiling(mm_plan_t pl, FftTiling& ft, bool fp64) {
    const int lam = pl->opts.lambda;
    const int maxlogm = fp64 ? kMaxLogM64 : kMaxLogM32;
    std::vector<int64_t> key;
    key.reserve(pl->n_int + 4);
    key.push_back(fp64);
    key.push_back(lam);
    key.push_back(pl->n_s);
    for (int32_t j = 0; j < pl->n_int; ++j) key.push_back(pl->h_off[j + 1] - pl->h_off[j]);
    int cached = 0;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tune_cache.find(key);
        if (it != g_tune_cache.end()) cached = it->second;
    }
    if (cached) return build_tiling(pl, ft, fp64, 2 << cached);
    const int64_t nx = pl->n_obs * pl->n_s;
    DBuf<double> x;
    DBuf<unsigned char> xp, z;
    MM_TRY(x.alloc(nx));
    MM_TRY(xp.alloc((size_t)4 * pl->n_obs * (fp64 ? 8 : 4)));
    MM_TRY(z.alloc((size_t)pl->n_t * (fp64 ? 8 : 4)));
    // a nonzero map (byte pattern 0x3f: 0.747f / 4.8e-4), so no tile takes the zero shortcut
    MM_HIP(hipMemsetAsync(x.p, 0x3f, nx * 8, pl->stream));
    MM_HIP(hipMemsetAsync(xp.p, 0x3f, xp.n, pl->stream));
    int best_l = 0;
    float best_ms = 0.0f;
    for (int l = kMinLogM + 1; l <= maxlogm; ++l) {
        const int64_t nr = (int64_t)2 << l;
        if (nr - 2 * (int64_t)lam < nr / 4) continue;
        FftTiling cand;
        MM_TRY(build_tiling(pl, cand, fp64, (int)nr));
        float ms = 0.0f;
        if (fp64)
            MM_TRY(time_map_launch<double>(pl, cand, (double*)xp.p, x.p, (double*)z.p, &ms));
        else
            MM_TRY(time_map_launch<float>(pl, cand, (float*)xp.p, x.p, (float*)z.p, &ms));
        if (best_l == 0 || ms < best_ms) {
            best_ms = ms;
            best_l = l;
            swap_tiling(ft, cand);
        }
    }
    if (best_l == 0) return build_tiling(pl, ft, fp64, 0);  // reports the error
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune_cache[key] = best_l;
    return MM_OK;
}

}  // namespace mm
