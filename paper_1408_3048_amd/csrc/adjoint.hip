// Adjoint of the GLS map m_hat = A^-1 P^T N^-1 d [Sect. 2.1, eq. glsSol] with respect to
// the time-ordered data and the noise parameters of every stationary interval.
//
// For a loss L(m_hat) with g = dL/dm_hat, mu = A^-1 g (one more PCG solve, A symmetric):
//   dL/dd        = N^-1 P mu
//   dL/dtheta_j  = (P mu)_j^T (dT_j/dtheta_j) (d - P m_hat)_j
//                = sum_k dt_k^(j)/dtheta_j c_j(k),
// where T_j is interval j's symmetric band Toeplitz block with taps t_k [Sect. 4.1.4,
// App. D] and c_j(0) = sum_t u_t v_t, c_j(k) = sum_t (u_t v_{t+k} + u_{t+k} v_t), u = P mu,
// v = d - P m_hat, t and t+k inside interval j.  The lag correlations are a banded
// product of the same shape as N^-1 itself; the tap derivatives are the windowed inverse
// DFTs of the derivatives of the inverse PSD, computed by the taps transform.
#include <algorithm>
#include <cfloat>
#include <cstdint>
#include <vector>

#include "mm_device.h"
#include "mm_fft.h"

namespace mm {
namespace {

constexpr int kLcThreads = 256;
constexpr int kLcR = 4;                       // lags per thread, 256 apart
constexpr int kLcLags = kLcThreads * kLcR;    // lags per block
constexpr int kLcT = 1024;                    // samples per chunk

__device__ __forceinline__ int find_interval(const int64_t* __restrict__ off, int n, int64_t v) {
    int a = 0, b = n - 1;
    while (a < b) {
        const int m = (a + b + 1) >> 1;
        if (off[m] <= v) a = m; else b = m - 1;
    }
    return a;
}

// Lags [kLcLags b, kLcLags (b + 1)) of interval j by direct sums
struct LagItem {
    int32_t j, b;
    int32_t run;  // chunks of kLcT samples per row of partial sums
    int32_t pad;
};

// Partial lag correlations of a run of chunks of one item (rows [roff[i], roff[i + 1]) are item
// i's) into part[row][kLcLags].  Samples past the interval end are zeros, so only pairs inside
// the interval contribute.
__global__ __launch_bounds__(kLcThreads) void k_lag_corr(
    const double* __restrict__ u, const double* __restrict__ v,
    const int64_t* __restrict__ int_lo, const int64_t* __restrict__ int_hi,
    const LagItem* __restrict__ items, const int64_t* __restrict__ roff, int n_items,
    double* __restrict__ part) {
    __shared__ double su[kLcT], sv[kLcT], su2[kLcT + kLcLags], sv2[kLcT + kLcLags];
    const int it = find_interval(roff, n_items, blockIdx.x);
    const LagItem item = items[it];
    const int64_t lo = int_lo[item.j], hi = int_hi[item.j];
    const int64_t k0 = (int64_t)item.b * kLcLags;
    const int64_t c0 = (blockIdx.x - roff[it]) * item.run;
    double acc[kLcR];
#pragma unroll
    for (int r = 0; r < kLcR; ++r) acc[r] = 0.0;
    for (int64_t ch = c0; ch < c0 + item.run; ++ch) {
        // samples that have a partner at the item's first lag
        const int64_t t0 = lo + ch * kLcT;
        const int n = (int)min((int64_t)kLcT, hi - t0 - k0);
        if (n <= 0) break;
        __syncthreads();  // the previous chunk has been read
        for (int i = threadIdx.x; i < kLcT; i += kLcThreads) {
            const int64_t t = t0 + i;
            su[i] = t < hi ? u[t] : 0.0;
            sv[i] = t < hi ? v[t] : 0.0;
        }
        for (int i = threadIdx.x; i < kLcT + kLcLags; i += kLcThreads) {
            const int64_t t = t0 + k0 + i;
            su2[i] = t < hi ? u[t] : 0.0;
            sv2[i] = t < hi ? v[t] : 0.0;
        }
        __syncthreads();
#pragma unroll 4
        for (int i = 0; i < n; ++i) {
            const double a = su[i], b = sv[i];
#pragma unroll
            for (int r = 0; r < kLcR; ++r) {
                const int q = i + threadIdx.x + r * kLcThreads;
                acc[r] = fma(a, sv2[q], acc[r]);
                acc[r] = fma(su2[q], b, acc[r]);
            }
        }
    }
    double* out = part + (int64_t)blockIdx.x * kLcLags;
#pragma unroll
    for (int r = 0; r < kLcR; ++r) out[threadIdx.x + r * kLcThreads] = acc[r];
}

// c[j][k] of an item's lags k <= K_j = the sum over its rows, in order
__global__ void k_lag_item_sum(const double* __restrict__ part, const LagItem* __restrict__ items,
                               const int64_t* __restrict__ roff, const int64_t* __restrict__ int_lo,
                               const int64_t* __restrict__ int_hi, int lam,
                               double* __restrict__ c) {
    const LagItem item = items[blockIdx.x];
    const int64_t K = min((int64_t)lam, int_hi[item.j] - int_lo[item.j] - 1);
    for (int i = threadIdx.x; i < kLcLags; i += blockDim.x) {
        const int64_t k = (int64_t)item.b * kLcLags + i;
        if (k > K) break;
        double s = 0.0;
        for (int64_t r = roff[blockIdx.x]; r < roff[blockIdx.x + 1]; ++r) s += part[r * kLcLags + i];
        c[(int64_t)item.j * (lam + 1) + k] = k == 0 ? 0.5 * s : s;
    }
}

// lag 0 of every chunk: sum u_t v_t over the chunk (lambda = 0, where it is the only lag)
__global__ __launch_bounds__(kLcThreads) void k_lag0(const double* __restrict__ u,
                                                     const double* __restrict__ v,
                                                     const int64_t* __restrict__ int_lo,
                                                     const int64_t* __restrict__ int_hi,
                                                     const int64_t* __restrict__ choff,
                                                     int32_t n_int, double* __restrict__ part) {
    __shared__ double red[kLcThreads];
    const int64_t ch = blockIdx.x;
    const int j = find_interval(choff, n_int, ch);
    const int64_t hi = int_hi[j];
    const int64_t t0 = int_lo[j] + (ch - choff[j]) * kLcT;
    double s = 0.0;
    for (int i = threadIdx.x; i < kLcT; i += kLcThreads) {
        const int64_t t = t0 + i;
        if (t < hi) s = fma(u[t], v[t], s);
    }
    write_partial_at(s, part + ch, 0, red);
}

// c[j] = the sum over the chunks of interval j, in chunk order
__global__ void k_lag0_sum(const double* __restrict__ part, const int64_t* __restrict__ choff,
                           int32_t n_int, double* __restrict__ c) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n_int;
         j += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0;
        for (int64_t ch = choff[j]; ch < choff[j + 1]; ++ch) s += part[ch];
        c[j] = s;
    }
}

// ---- lag correlations by FFT
//
// An interval is cut into blocks of B >= lambda samples.  With U_c, V_c the transforms on
// N = 2B points of block c of u and v (zero-padded), the pairs whose first sample lies in
// block c contribute conj(U_c) (V_c + s V_{c+1}) + conj(V_c) (U_c + s U_{c+1}) to the transform
// of c(k), k <= B, where s = (-1)^f is the shift of block c + 1 by N/2.  Every block is
// transformed once (u and v as one complex sequence u + i v, split by symmetry), a workgroup
// takes kLfRun consecutive blocks (plus the one after them), keeping the spectra of the last
// block and the running sum in registers (less a few that spill) for the frequency pairs
// (f, N - f), and writes its sum; k_lag_inverse adds the sums of an interval in order and
// transforms back.
//
// u and v can differ by many orders of magnitude (u = P mu against the residual v), and the
// split of their common transform would carry the larger one's rounding into the other: each
// workgroup scales both by powers of two to unit norm and scales its product back; where one of
// them is zero it writes the exact zeros.
//
// The transforms' rounding follows the norms, at every lag alike: P_j = sum of ||u|| ||v|| over an
// interval's workgroups.  That of the direct sums follows the terms of a lag, S_j(k) = sum of
// |u_t| |v_{t+k}| + |u_{t+k}| |v_t|, which is far less where the samples are few or far apart
// (bursts, flagged stretches, lags near the interval's length).  The same launches correlate |u|
// and |v|, which gives S_j(k), and blocks of kLcLags lags that hold one with S_j(k) < P_j / 8, or
// one that is not finite, are taken by direct sums: every lag keeps a rounding of its own terms.
// (Gaussian u and v have S_j(k) of about (1 - k / t_j) P_j.)
//
// The transform's length goes by K_j = min(lambda, t_j - 1), so that intervals shorter than the
// band take what they need; lag 0 alone (lambda = 0) and lags past 4096 are direct sums.
//
// The whole call in us, direct sums of everything (bound by one LDS read per product) / this
// (bound by the transforms' LDS passes; two thirds of the time without the magnitudes): 2^22
// samples in 32 intervals, lambda = 2048: 2231 / 231; 2^24 in 256, lambda = 2048: 8202 / 837; 2^24
// in 64, lambda = 4096: 16321 / 824; 2^14 in 32, lambda = 64: 112 / 58; with the last lags left to
// direct sums, 2^22 in 2000, lambda = 2000: 3060 / 1649; 2^20 in 10000 of about 100 samples,
// lambda = 2000: 2652 / 729.  The spectra's registers spill 84-88 bytes a thread.
constexpr int kLfRun = 4;         // blocks per workgroup, at least
constexpr int kLfMaxParts = 128;  // workgroups per interval, at most
constexpr int kLfMaxLogM = 13;    // N = 8192: lags up to 4096
// scratch of one launch, spectra of workgroups or rows of direct sums: more go in turn
constexpr int64_t kLagScratch = (int64_t)256 << 20;
constexpr int64_t kLagMaxRows = 4096;  // rows per item of direct sums, at most

// power of two that brings a largest magnitude m to [0.5, 1) (1 for m = 0, and for infinities
// and NaN, which reach the result unscaled), as an exponent
__device__ __forceinline__ int unit_exponent(double m) {
    int e = 0;
    if (m > 0.0 && m <= DBL_MAX) (void)frexp(m, &e);
    return -e;
}

// Powers of two 2^eu, 2^ev that bring the norms of u and v over the samples [t0, t1) to
// [0.5, 1), and the product of the norms; zero: one of the two is zero throughout.  By the sums
// of squares, after a first scaling by the largest magnitudes where these leave the range.  All
// threads must call.
struct RunScale {
    int eu, ev;
    double norms;
    bool zero;
};
template <int NT>
__device__ __forceinline__ RunScale run_scale(const double* __restrict__ u,
                                              const double* __restrict__ v, int64_t t0, int64_t t1,
                                              double* red) {
    RunScale s{0, 0, 0.0, false};
    double su, sv;
    const auto in_range = [](double x) { return x > 1e-280 && x < 1e280; };
    for (int pass = 0;; ++pass) {
        double a = 0.0, b = 0.0;
        for (int64_t t = t0 + threadIdx.x; t < t1; t += NT) {
            const double x = ldexp(u[t], s.eu), y = ldexp(v[t], s.ev);
            a = fma(x, x, a);
            b = fma(y, y, b);
        }
        su = block_sum(a, red);
        sv = block_sum(b, red);
        if (pass == 1 || (in_range(su) && in_range(sv))) break;
        double mu = 0.0, mv = 0.0;
        for (int64_t t = t0 + threadIdx.x; t < t1; t += NT) {
            mu = fmax(mu, fabs(u[t]));
            mv = fmax(mv, fabs(v[t]));
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            mu = fmax(mu, __shfl_xor(mu, o));
            mv = fmax(mv, __shfl_xor(mv, o));
        }
        if ((threadIdx.x & 63) == 0) {
            red[2 * (threadIdx.x >> 6)] = mu;
            red[2 * (threadIdx.x >> 6) + 1] = mv;
        }
        __syncthreads();
        for (int w = 0; w < NT / 64; ++w) {
            mu = fmax(mu, red[2 * w]);
            mv = fmax(mv, red[2 * w + 1]);
        }
        __syncthreads();
        s.eu = unit_exponent(mu);
        s.ev = unit_exponent(mv);
    }
    s.norms = ldexp(sqrt(su) * sqrt(sv), -s.eu - s.ev);
    s.zero = su == 0.0 || sv == 0.0;
    // (x + 1) >> 1: the exponent of the norm from that of its square
    s.eu -= (1 - unit_exponent(su)) >> 1;
    s.ev -= (1 - unit_exponent(sv)) >> 1;
    return s;
}

struct LagPart {
    int32_t j;       // interval
    int32_t c0, c1;  // its blocks [c0, c1)
};

// blockIdx.y = 0: u and v; 1: their magnitudes, and the products of the norms into norms[part].
// Sums into spec[blockIdx.y][part]
template <int LOGM, int NT>
__global__ __launch_bounds__(NT, 2) void k_lag_spectra(const double* __restrict__ u,
                                                    const double* __restrict__ v,
                                                    const int64_t* __restrict__ int_lo,
                                                    const int64_t* __restrict__ int_hi,
                                                    const LagPart* __restrict__ parts,
                                                    const double* __restrict__ tw,
                                                    double* __restrict__ spec,
                                                    double* __restrict__ norms) {
    constexpr int M = 1 << LOGM, B = M / 2;
    constexpr int NP = (M / 2) / NT;  // frequency pairs (f, M - f), f = 1 .. M/2 - 1, per thread
    __shared__ __align__(16) unsigned char smem[2 * M * sizeof(double)];
    __shared__ double red[2 * (NT / 64)];
    const CBuf<double> buf = make_cbuf<double>(smem, M);
    const LagPart part = parts[blockIdx.x];
    const bool mag = blockIdx.y != 0;
    const int64_t lo = int_lo[part.j], hi = int_hi[part.j];
    const int64_t t0 = lo + (int64_t)part.c0 * B;
    const int64_t t1 = min(hi, lo + ((int64_t)part.c1 + 1) * B);
    // M/2 complex values
    double* out = spec + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * M;
    const RunScale sc = run_scale<NT>(u, v, t0, t1, red);
    if (mag && threadIdx.x == 0) norms[blockIdx.x] = sc.norms;
    if (sc.zero) {
        for (int i = threadIdx.x; i < M; i += NT) out[i] = 0.0;
        return;
    }
    // pair i of the thread: f = tid + i NT; f = 0 carries the real bins 0 and M/2
    double ar[NP], ai[NP];                      // running sum at f (f = 0: bins 0 and M/2)
    double ur[NP], ui[NP], vr[NP], vi[NP];      // U, V of the last block at f (f = 0: bin 0 in
                                                // the real parts, bin M/2 in the imaginary)
#pragma unroll
    for (int i = 0; i < NP; ++i) ar[i] = ai[i] = ur[i] = ui[i] = vr[i] = vi[i] = 0.0;
    for (int c = part.c0; c <= part.c1; ++c) {
        const int64_t b0 = lo + (int64_t)c * B;
        if (b0 >= hi) break;  // uniform: no samples in this block, nothing to add
        const int len = (int)min((int64_t)B, hi - b0);
        for (int i = threadIdx.x; i < M; i += NT) {
            double x = 0.0, y = 0.0;
            if (i < len) {
                x = ldexp(u[b0 + i], sc.eu);
                y = ldexp(v[b0 + i], sc.ev);
                if (mag) {
                    x = fabs(x);
                    y = fabs(y);
                }
            }
            buf.put(i, x, y);
        }
        __syncthreads();
        fwd_passes<double, LOGM, NT, LOGM>(buf, tw);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int f = threadIdx.x + i * NT;
            double pr, pi, qr, qi;  // Z at f and M - f
            buf.get(rev_bits<LOGM>(f), pr, pi);
            buf.get(f == 0 ? rev_bits<LOGM>(M / 2) : rev_bits<LOGM>(M - f), qr, qi);
            double nur, nui, nvr, nvi;
            if (f == 0) {  // U and V are real at bins 0 and M/2
                nur = pr;
                nvr = pi;
                nui = qr;
                nvi = qi;
                // the previous block with this one as its successor, then this block
                ar[i] += 2.0 * (ur[i] * nvr + vr[i] * nur);
                ai[i] += 2.0 * (ui[i] * nvi + vi[i] * nui);  // M/2 is even: s = 1
                if (c < part.c1) {
                    ar[i] += 8.0 * nur * nvr;
                    ai[i] += 8.0 * nui * nvi;
                }
                ur[i] = 2.0 * nur;
                ui[i] = 2.0 * nui;
                vr[i] = 2.0 * nvr;
                vi[i] = 2.0 * nvi;
                continue;
            }
            // 2 U = Z_f + conj(Z_{M-f}), 2 V = -i (Z_f - conj(Z_{M-f}))
            nur = pr + qr;
            nui = pi - qi;
            nvr = pi + qi;
            nvi = qr - pr;
            const double s = (f & 1) ? -1.0 : 1.0;
            // conj(U_prev) V + conj(V_prev) U
            ar[i] += s * (ur[i] * nvr + ui[i] * nvi + vr[i] * nur + vi[i] * nui);
            ai[i] += s * (ur[i] * nvi - ui[i] * nvr + vr[i] * nui - vi[i] * nur);
            if (c < part.c1) ar[i] += 2.0 * (nur * nvr + nui * nvi);  // conj(U) V + conj(V) U
            ur[i] = nur;
            ui[i] = nui;
            vr[i] = nvr;
            vi[i] = nvi;
        }
        __syncthreads();  // the next block overwrites the buffer
    }
    // 4 from the two split factors of 2 in every product
    const int e = -sc.eu - sc.ev - 2;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int f = threadIdx.x + i * NT;
        out[2 * f] = ldexp(ar[i], e);
        out[2 * f + 1] = ldexp(ai[i], e);
    }
}

// Interval j = ids[blockIdx.x], from the sums of its workgroups [poff[i], poff[i + 1]) less p0 of
// n_parts.  blockIdx.y = 0: c[j][k], k <= min(K_j, B), and 0 for k > K_j.  blockIdx.y = 1: from the
// magnitudes, which blocks of kLcLags lags are left to direct sums: flags[j][b], b < nb.
template <int LOGM, int NT>
__global__ __launch_bounds__(NT) void k_lag_inverse(
    const double* __restrict__ spec, const double* __restrict__ norms, int64_t n_parts,
    const int32_t* __restrict__ ids, const int64_t* __restrict__ poff, int64_t p0,
    const int64_t* __restrict__ int_lo, const int64_t* __restrict__ int_hi, int lam,
    const double* __restrict__ tw, int nb, double* __restrict__ c, uint8_t* __restrict__ flags) {
    constexpr int M = 1 << LOGM;
    constexpr int BL = M / 2 / kLcLags + 1;  // blocks of lags that the transform reaches
    __shared__ __align__(16) unsigned char smem[2 * M * sizeof(double)];
    __shared__ int low[BL];
    const CBuf<double> buf = make_cbuf<double>(smem, M);
    const int j = ids[blockIdx.x];
    const int64_t q0 = poff[blockIdx.x] - p0, q1 = poff[blockIdx.x + 1] - p0;
    const double2* s = reinterpret_cast<const double2*>(spec + (int64_t)blockIdx.y * n_parts * M);
    for (int f = threadIdx.x; f < M / 2; f += NT) {
        double re = 0.0, im = 0.0;
#pragma unroll 8
        for (int64_t p = q0; p < q1; ++p) {
            const double2 g = s[p * (M / 2) + f];
            re += g.x;
            im += g.y;
        }
        if (f == 0) {
            buf.put(0, re, 0.0);
            buf.put(rev_bits<LOGM>(M / 2), im, 0.0);
        } else {
            buf.put(rev_bits<LOGM>(f), re, im);
            buf.put(rev_bits<LOGM>(M - f), re, -im);
        }
    }
    if (threadIdx.x < BL) low[threadIdx.x] = 0;
    __syncthreads();
    inv_passes<double, LOGM, NT, LOGM>(buf, tw);
    const int64_t K = min((int64_t)lam, int_hi[j] - int_lo[j] - 1);
    if (blockIdx.y == 0) {
        for (int k = threadIdx.x; k <= lam; k += NT) {
            if (k > K) c[(int64_t)j * (lam + 1) + k] = 0.0;
            if (k > K || k > M / 2) continue;
            const double r = buf.get_part(k, 0) * (1.0 / M);
            c[(int64_t)j * (lam + 1) + k] = k == 0 ? 0.5 * r : r;
        }
        return;
    }
    double norm = 0.0;
    for (int64_t p = q0; p < q1; ++p) norm += norms[p];
    for (int k = threadIdx.x; k <= K && k <= M / 2; k += NT) {
        const double r = buf.get_part(k, 0) * (1.0 / M);
        if (!((k == 0 ? 0.5 * r : r) >= 0.125 * norm && norm <= DBL_MAX)) low[k / kLcLags] = 1;
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += NT)
        flags[(int64_t)j * nb + b] = K > M / 2 && b >= BL - 1 ? (int64_t)b * kLcLags <= K
                                                              : b < BL && low[b];
}

// v = d - v (d FP32 or FP64)
template <typename TD>
__global__ void k_resid_tod(const TD* __restrict__ d, double* __restrict__ v, int64_t n) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x)
        v[t] = (double)d[t] - v[t];
}

__global__ void k_to_f32(const double* __restrict__ a, float* __restrict__ b, int64_t n) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x)
        b[t] = (float)a[t];
}

inline int grid_for(int64_t n) {
    int64_t g = (n + 255) / 256;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, 65536));
}

}  // namespace

namespace {

// Intervals whose K_j takes one transform length, with the tables of their launches
struct LagClass {
    std::vector<int32_t> ids;
    std::vector<LagPart> parts;
    std::vector<int64_t> poff{0};
    DBuf<int32_t> d_ids;
    DBuf<LagPart> d_parts;
    DBuf<int64_t> d_poff;
    DBuf<double> tw, spec, norms;
};

template <int LOGM, int NT>
int lag_fft(mm_plan_t pl, const double* u, const double* v, LagClass& lc, int nb, double* c,
            uint8_t* flags) {
    if (lc.ids.empty()) return MM_OK;
    constexpr int B = 1 << (LOGM - 1);
    constexpr int64_t cap = std::max<int64_t>(kLfMaxParts, kLagScratch / (2 * (8ll << LOGM)));
    hipStream_t st = pl->stream;
    for (int32_t j : lc.ids) {
        const int64_t nblk = (pl->h_off[j + 1] - pl->h_off[j] + B - 1) / B;
        const int64_t run = std::max<int64_t>(kLfRun, (nblk + kLfMaxParts - 1) / kLfMaxParts);
        for (int64_t b = 0; b < nblk; b += run)
            lc.parts.push_back({j, (int32_t)b, (int32_t)std::min(nblk, b + run)});
        lc.poff.push_back((int64_t)lc.parts.size());
    }
    const int64_t n = (int64_t)lc.ids.size();
    const int64_t np = std::min<int64_t>(cap, (int64_t)lc.parts.size());
    MM_TRY(lc.d_ids.alloc(n));
    MM_TRY(lc.d_parts.alloc(lc.parts.size()));
    MM_TRY(lc.d_poff.alloc(n + 1));
    MM_TRY(lc.tw.alloc((size_t)2 << LOGM));
    MM_TRY(lc.spec.alloc((size_t)(2 * np) << LOGM));
    MM_TRY(lc.norms.alloc(np));
    MM_HIP(hipMemcpyAsync(lc.d_ids.p, lc.ids.data(), n * 4, hipMemcpyHostToDevice, st));
    MM_HIP(hipMemcpyAsync(lc.d_parts.p, lc.parts.data(), lc.parts.size() * sizeof(LagPart),
                          hipMemcpyHostToDevice, st));
    MM_HIP(hipMemcpyAsync(lc.d_poff.p, lc.poff.data(), (n + 1) * 8, hipMemcpyHostToDevice, st));
    MM_TRY(fft_twiddles(pl, (int64_t)1 << LOGM, (int64_t)2 << LOGM, lc.tw.p));
    for (int64_t i0 = 0, i1; i0 < n; i0 = i1) {  // as many intervals as the scratch holds
        i1 = i0 + 1;
        while (i1 < n && lc.poff[i1 + 1] - lc.poff[i0] <= np) ++i1;
        const int64_t p0 = lc.poff[i0], k = lc.poff[i1] - p0;
        hipLaunchKernelGGL((k_lag_spectra<LOGM, NT>), dim3((unsigned)k, 2), dim3(NT), 0, st, u, v,
                           pl->int_lo.p, pl->int_hi.p, lc.d_parts.p + p0, lc.tw.p, lc.spec.p,
                           lc.norms.p);
        MM_HIP(hipGetLastError());
        hipLaunchKernelGGL((k_lag_inverse<LOGM, NT>), dim3((unsigned)(i1 - i0), 2), dim3(NT), 0, st,
                           lc.spec.p, lc.norms.p, k, lc.d_ids.p + i0, lc.d_poff.p + i0, p0,
                           pl->int_lo.p, pl->int_hi.p, pl->opts.lambda, lc.tw.p, nb, c, flags);
        MM_HIP(hipGetLastError());
    }
    return MM_OK;
}

// the flagged blocks of lags by direct sums
int lag_direct(mm_plan_t pl, const double* u, const double* v, const std::vector<uint8_t>& flags,
               int nb, double* c) {
    hipStream_t st = pl->stream;
    std::vector<LagItem> items;
    std::vector<int64_t> roff;
    int64_t rows = 0;
    DBuf<LagItem> d_items;
    DBuf<int64_t> d_roff;
    DBuf<double> part;
    auto flush = [&]() -> int {
        if (items.empty()) return MM_OK;
        const int n = (int)items.size();
        roff.push_back(rows);
        MM_TRY(d_items.alloc(n));
        MM_TRY(d_roff.alloc(n + 1));
        MM_TRY(part.alloc((size_t)rows * kLcLags));
        MM_HIP(hipMemcpyAsync(d_items.p, items.data(), n * sizeof(LagItem), hipMemcpyHostToDevice,
                              st));
        MM_HIP(hipMemcpyAsync(d_roff.p, roff.data(), (n + 1) * 8, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(k_lag_corr, dim3((unsigned)rows), dim3(kLcThreads), 0, st, u, v,
                           pl->int_lo.p, pl->int_hi.p, d_items.p, d_roff.p, n, part.p);
        MM_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_lag_item_sum, dim3(n), dim3(256), 0, st, part.p, d_items.p, d_roff.p,
                           pl->int_lo.p, pl->int_hi.p, pl->opts.lambda, c);
        MM_HIP(hipGetLastError());
        MM_HIP(hipStreamSynchronize(st));
        items.clear();
        roff.clear();
        rows = 0;
        return MM_OK;
    };
    for (int32_t j = 0; j < pl->n_int; ++j)
        for (int b = 0; b < nb; ++b) {
            if (!flags[(size_t)j * nb + b]) continue;
            const int64_t n = pl->h_off[j + 1] - pl->h_off[j] - (int64_t)b * kLcLags;
            const int64_t nch = (n + kLcT - 1) / kLcT;
            const int64_t run = (nch + kLagMaxRows - 1) / kLagMaxRows;
            const int64_t add = (nch + run - 1) / run;
            if ((rows + add) * kLcLags * 8 > kLagScratch) MM_TRY(flush());
            items.push_back({j, b, (int32_t)run, 0});
            roff.push_back(rows);
            rows += add;
        }
    return flush();
}

}  // namespace

int lag_correlations(mm_plan_t pl, const double* u, const double* v, double* c) {
    hipStream_t st = pl->stream;
    const int lam = pl->opts.lambda;
    if (lam == 0) {
        std::vector<int64_t> choff(pl->n_int + 1, 0);
        for (int32_t j = 0; j < pl->n_int; ++j)
            choff[j + 1] = choff[j] + (pl->h_off[j + 1] - pl->h_off[j] + kLcT - 1) / kLcT;
        const int64_t nch = choff[pl->n_int];
        DBuf<int64_t> dch;
        DBuf<double> part;
        MM_TRY(dch.alloc(pl->n_int + 1));
        MM_TRY(part.alloc((size_t)nch));
        MM_HIP(hipMemcpyAsync(dch.p, choff.data(), (pl->n_int + 1) * 8, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(k_lag0, dim3(nch), dim3(kLcThreads), 0, st, u, v, pl->int_lo.p,
                           pl->int_hi.p, dch.p, pl->n_int, part.p);
        MM_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_lag0_sum, dim3(grid_for(pl->n_int)), dim3(256), 0, st, part.p, dch.p,
                           pl->n_int, c);
        MM_HIP(hipGetLastError());
        MM_HIP(hipStreamSynchronize(st));  // scratch is released on return
        return MM_OK;
    }
    // the shortest transform whose blocks reach every lag of an interval, but 8192 points also for
    // K_j in (1024, 2048], where one workgroup of 8 waves per CU ran faster than two of 4 with
    // 4096 points (2^24 samples, intervals of 2^16, without the magnitudes: 468 against 549 us)
    LagClass lc[3];
    for (int32_t j = 0; j < pl->n_int; ++j) {
        const int64_t K = std::min<int64_t>(lam, pl->h_off[j + 1] - pl->h_off[j] - 1);
        lc[K <= 512 ? 0 : (K <= 1024 ? 1 : 2)].ids.push_back(j);
    }
    const int nb = lam / kLcLags + 1;
    DBuf<uint8_t> d_flags;
    std::vector<uint8_t> flags((size_t)pl->n_int * nb);
    MM_TRY(d_flags.alloc(flags.size()));
    MM_TRY((lag_fft<10, 64>(pl, u, v, lc[0], nb, c, d_flags.p)));
    MM_TRY((lag_fft<11, 128>(pl, u, v, lc[1], nb, c, d_flags.p)));
    MM_TRY((lag_fft<kLfMaxLogM, 512>(pl, u, v, lc[2], nb, c, d_flags.p)));
    MM_HIP(hipMemcpyAsync(flags.data(), d_flags.p, flags.size(), hipMemcpyDeviceToHost, st));
    MM_HIP(hipStreamSynchronize(st));  // scratch is released on return
    return lag_direct(pl, u, v, flags, nb, c);
}

// dt[j][i][k] (host, [n_int][3][lambda+1], zero past K_j) for every interval
int tap_derivatives(mm_plan_t pl, std::vector<double>& dt) {
    const int lam = pl->opts.lambda;
    dt.assign((size_t)pl->n_int * 3 * (lam + 1), 0.0);
    for (int i = 0; i < 3; ++i) {
        std::vector<double> t;
        std::vector<int64_t> toff, tcnt;
        MM_TRY(kernel_taps(pl, i + 1, t, toff, tcnt));
        for (int32_t j = 0; j < pl->n_int; ++j) {
            const int g = pl->h_int_kern[j];
            double* o = dt.data() + ((size_t)j * 3 + i) * (lam + 1);
            for (int64_t k = 0; k < tcnt[g]; ++k) o[k] = t[toff[g] + k];
        }
    }
    return MM_OK;
}

int adjoint_tod(mm_plan_t pl, const double* m_hat, const double* mu, const void* d, int d_f64,
                void* grad_d, int grad_d_f64, double* grad_psd) {
    hipStream_t st = pl->stream;
    const int64_t n = pl->n_t;
    const int lam = pl->opts.lambda;
    DBuf<double> u, v, c;
    MM_TRY(u.alloc(n));
    MM_TRY(v.alloc(n));
    MM_TRY(depoint(pl, mu, u.p, 1));  // u = P mu
    if (grad_d) {
        if (grad_d_f64) {
            MM_TRY(toeplitz_tod64(pl, u.p, 1, (double*)grad_d));
        } else {
            MM_TRY(toeplitz_tod64(pl, u.p, 1, v.p));
            hipLaunchKernelGGL(k_to_f32, dim3(grid_for(n)), dim3(256), 0, st, (const double*)v.p,
                               (float*)grad_d, n);
            MM_HIP(hipGetLastError());
        }
    }
    if (!grad_psd) return MM_OK;
    MM_TRY(depoint(pl, m_hat, v.p, 1));  // v = d - P m_hat
    if (d_f64)
        hipLaunchKernelGGL(k_resid_tod<double>, dim3(grid_for(n)), dim3(256), 0, st,
                           (const double*)d, v.p, n);
    else
        hipLaunchKernelGGL(k_resid_tod<float>, dim3(grid_for(n)), dim3(256), 0, st,
                           (const float*)d, v.p, n);
    MM_HIP(hipGetLastError());
    MM_TRY(c.alloc((size_t)pl->n_int * (lam + 1)));
    MM_TRY(lag_correlations(pl, u.p, v.p, c.p));
    std::vector<double> hc((size_t)pl->n_int * (lam + 1));
    MM_HIP(hipMemcpyAsync(hc.data(), c.p, hc.size() * 8, hipMemcpyDeviceToHost, st));
    MM_HIP(hipStreamSynchronize(st));
    std::vector<double> dt;
    MM_TRY(tap_derivatives(pl, dt));
    for (int32_t j = 0; j < pl->n_int; ++j)
        for (int i = 0; i < 3; ++i) {
            const double* a = dt.data() + ((size_t)j * 3 + i) * (lam + 1);
            const double* b = hc.data() + (size_t)j * (lam + 1);
            double s = 0.0;
            for (int k = 0; k <= lam; ++k) s += a[k] * b[k];
            grad_psd[3 * j + i] = s;
        }
    return MM_OK;
}

}  // namespace mm
