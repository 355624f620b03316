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

// Partial lag correlations of one chunk of kLcT samples of one interval for the lags
// [kbeg + blockIdx.y * kLcLags, ...) into part[chunk][k], by direct sums: the lags past those
// that the FFT below reaches (lambda > 4096).  Samples past the interval end are zeros, so
// only pairs inside the interval contribute.
__global__ __launch_bounds__(kLcThreads) void k_lag_corr(
    const double* __restrict__ u, const double* __restrict__ v,
    const int64_t* __restrict__ int_lo, const int64_t* __restrict__ int_hi,
    const int64_t* __restrict__ choff, int32_t n_int, int lam, int kbeg,
    double* __restrict__ part) {
    __shared__ double su[kLcT], sv[kLcT], su2[kLcT + kLcLags], sv2[kLcT + kLcLags];
    const int64_t ch = blockIdx.x;
    const int j = find_interval(choff, n_int, ch);
    const int64_t lo = int_lo[j], hi = int_hi[j];
    const int64_t t0 = lo + (ch - choff[j]) * kLcT;
    const int64_t K = min((int64_t)lam, hi - lo - 1);
    const int64_t k0 = kbeg + (int64_t)blockIdx.y * kLcLags;
    if (k0 > K) return;
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
    double acc[kLcR];
#pragma unroll
    for (int r = 0; r < kLcR; ++r) acc[r] = 0.0;
    for (int i = 0; i < kLcT; ++i) {
        const double a = su[i], b = sv[i];
#pragma unroll
        for (int r = 0; r < kLcR; ++r) {
            const int q = i + threadIdx.x + r * kLcThreads;
            acc[r] = fma(a, sv2[q], acc[r]);
            acc[r] = fma(su2[q], b, acc[r]);
        }
    }
    double* out = part + ch * (int64_t)(lam + 1);
#pragma unroll
    for (int r = 0; r < kLcR; ++r) {
        const int64_t k = k0 + threadIdx.x + r * kLcThreads;
        if (k <= K) out[k] = acc[r];
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

// c[j][k] for the lags k >= kbeg = the sum over the chunks of interval j, in chunk order; 0 for
// k > K_j
__global__ void k_lag_reduce(const double* __restrict__ part, const int64_t* __restrict__ choff,
                             const int64_t* __restrict__ int_lo, const int64_t* __restrict__ int_hi,
                             int lam, int kbeg, double* __restrict__ c) {
    const int j = blockIdx.y;
    const int64_t K = min((int64_t)lam, int_hi[j] - int_lo[j] - 1);
    for (int64_t k = kbeg + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k <= lam;
         k += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0;
        if (k <= K)
            for (int64_t ch = choff[j]; ch < choff[j + 1]; ++ch) s += part[ch * (lam + 1) + k];
        c[(int64_t)j * (lam + 1) + k] = s;
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
// block and the running sum in registers for the frequency pairs (f, N - f), and writes its
// sum; k_lag_inverse adds the sums of an interval in order and transforms back.
//
// u and v can differ by many orders of magnitude (u = P mu against the residual v), and the
// split of their common transform would carry the larger one's rounding into the other: each
// workgroup scales both by powers of two to unit size and scales its product back.
//
// The whole call in us, direct sums (bound by one LDS read per product) / FFT (bound by the
// transforms' LDS passes): 2^22 samples in 32 intervals, lambda = 2048: 2202 / 156; 2^24
// in 256, lambda = 2048: 8176 / 468; 2^24 in 64, lambda = 4096: 16258 / 461; 2^14 in 32, lambda =
// 64: 102 / 62.
constexpr int kLfRun = 4;         // blocks per workgroup, at least
constexpr int kLfMaxParts = 128;  // workgroups per interval, at most
constexpr int kLfMaxLogM = 13;    // N = 8192: lags up to 4096

// power of two that brings a largest magnitude m to [0.5, 1) (1 for m = 0, and for infinities
// and NaN, which reach the result unscaled), as an exponent
__device__ __forceinline__ int unit_exponent(double m) {
    int e = 0;
    if (m > 0.0 && m <= DBL_MAX) (void)frexp(m, &e);
    return -e;
}

struct LagPart {
    int32_t j;       // interval
    int32_t c0, c1;  // its blocks [c0, c1)
};

template <int LOGM, int NT>
__global__ __launch_bounds__(NT, 2) void k_lag_spectra(const double* __restrict__ u,
                                                    const double* __restrict__ v,
                                                    const int64_t* __restrict__ int_lo,
                                                    const int64_t* __restrict__ int_hi,
                                                    const LagPart* __restrict__ parts,
                                                    const double* __restrict__ tw,
                                                    double* __restrict__ spec) {
    constexpr int M = 1 << LOGM, B = M / 2;
    constexpr int NP = (M / 2) / NT;  // frequency pairs (f, M - f), f = 1 .. M/2 - 1, per thread
    __shared__ __align__(16) unsigned char smem[2 * M * sizeof(double)];
    __shared__ double red[2 * (NT / 64)];
    const CBuf<double> buf = make_cbuf<double>(smem, M);
    const LagPart part = parts[blockIdx.x];
    const int64_t lo = int_lo[part.j], hi = int_hi[part.j];
    const int64_t t0 = lo + (int64_t)part.c0 * B;
    const int64_t t1 = min(hi, lo + ((int64_t)part.c1 + 1) * B);
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
    const int eu = unit_exponent(mu), ev = unit_exponent(mv);
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
                x = ldexp(u[b0 + i], eu);
                y = ldexp(v[b0 + i], ev);
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
    const int e = -eu - ev - 2;
    double* out = spec + (int64_t)blockIdx.x * M;  // M/2 complex values
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const int f = threadIdx.x + i * NT;
        out[2 * f] = ldexp(ar[i], e);
        out[2 * f + 1] = ldexp(ai[i], e);
    }
}

// c[j][k], k <= min(lambda, B), of interval j = blockIdx.x from the sums of its workgroups
// [poff[j], poff[j + 1]); 0 for k > K_j
template <int LOGM, int NT>
__global__ __launch_bounds__(NT) void k_lag_inverse(const double* __restrict__ spec,
                                                    const int64_t* __restrict__ poff,
                                                    const int64_t* __restrict__ int_lo,
                                                    const int64_t* __restrict__ int_hi, int lam,
                                                    const double* __restrict__ tw,
                                                    double* __restrict__ c) {
    constexpr int M = 1 << LOGM;
    __shared__ __align__(16) unsigned char smem[2 * M * sizeof(double)];
    const CBuf<double> buf = make_cbuf<double>(smem, M);
    const int j = blockIdx.x;
    const double2* s = reinterpret_cast<const double2*>(spec);
    for (int f = threadIdx.x; f < M / 2; f += NT) {
        double re = 0.0, im = 0.0;
#pragma unroll 8
        for (int64_t p = poff[j]; p < poff[j + 1]; ++p) {
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
    __syncthreads();
    inv_passes<double, LOGM, NT, LOGM>(buf, tw);
    const int64_t K = min((int64_t)lam, int_hi[j] - int_lo[j] - 1);
    const int top = min(lam, M / 2);
    for (int k = threadIdx.x; k <= top; k += NT) {
        const double r = buf.get_part(k, 0) * (1.0 / M);
        c[(int64_t)j * (lam + 1) + k] = k > K ? 0.0 : (k == 0 ? 0.5 * r : r);
    }
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

template <int LOGM, int NT>
int lag_fft(mm_plan_t pl, const double* u, const double* v, double* c) {
    constexpr int B = 1 << (LOGM - 1);
    hipStream_t st = pl->stream;
    const int lam = pl->opts.lambda;
    std::vector<LagPart> parts;
    std::vector<int64_t> poff(pl->n_int + 1, 0);
    for (int32_t j = 0; j < pl->n_int; ++j) {
        const int64_t nb = (pl->h_off[j + 1] - pl->h_off[j] + B - 1) / B;
        const int64_t run = std::max<int64_t>(kLfRun, (nb + kLfMaxParts - 1) / kLfMaxParts);
        for (int64_t b = 0; b < nb; b += run)
            parts.push_back({j, (int32_t)b, (int32_t)std::min(nb, b + run)});
        poff[j + 1] = (int64_t)parts.size();
    }
    DBuf<LagPart> d_parts;
    DBuf<int64_t> d_poff;
    DBuf<double> tw, spec;
    MM_TRY(d_parts.alloc(parts.size()));
    MM_TRY(d_poff.alloc(poff.size()));
    MM_TRY(tw.alloc((size_t)2 << LOGM));
    MM_TRY(spec.alloc(parts.size() << LOGM));
    MM_HIP(hipMemcpyAsync(d_parts.p, parts.data(), parts.size() * sizeof(LagPart),
                          hipMemcpyHostToDevice, st));
    MM_HIP(hipMemcpyAsync(d_poff.p, poff.data(), poff.size() * 8, hipMemcpyHostToDevice, st));
    MM_TRY(fft_twiddles(pl, (int64_t)1 << LOGM, (int64_t)2 << LOGM, tw.p));
    hipLaunchKernelGGL((k_lag_spectra<LOGM, NT>), dim3((unsigned)parts.size()), dim3(NT), 0, st, u,
                       v, pl->int_lo.p, pl->int_hi.p, d_parts.p, tw.p, spec.p);
    MM_HIP(hipGetLastError());
    hipLaunchKernelGGL((k_lag_inverse<LOGM, NT>), dim3(pl->n_int), dim3(NT), 0, st, spec.p,
                       d_poff.p, pl->int_lo.p, pl->int_hi.p, lam, tw.p, c);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

}  // namespace

int lag_correlations(mm_plan_t pl, const double* u, const double* v, double* c) {
    hipStream_t st = pl->stream;
    const int lam = pl->opts.lambda;
    // the shortest transform whose blocks reach every lag, but 8192 points also for lambda in
    // (1024, 2048], where one workgroup of 8 waves per CU ran faster than two of 4 with
    // 4096 points (2^24 samples, intervals of 2^16: 468 against 549 us); lag 0 alone and the
    // lags past 4096 by direct sums
    constexpr int kFftLags = 1 << (kLfMaxLogM - 1);
    if (lam > 1024)
        MM_TRY((lag_fft<kLfMaxLogM, 512>(pl, u, v, c)));
    else if (lam > 512)
        MM_TRY((lag_fft<11, 128>(pl, u, v, c)));
    else if (lam > 0)
        MM_TRY((lag_fft<10, 64>(pl, u, v, c)));
    if (lam == 0 || lam > kFftLags) {
        const int kbeg = lam == 0 ? 0 : kFftLags + 1;
        std::vector<int64_t> choff(pl->n_int + 1, 0);
        for (int32_t j = 0; j < pl->n_int; ++j)
            choff[j + 1] = choff[j] + (pl->h_off[j + 1] - pl->h_off[j] + kLcT - 1) / kLcT;
        const int64_t nch = choff[pl->n_int];
        DBuf<int64_t> dch;
        DBuf<double> part;
        MM_TRY(dch.alloc(pl->n_int + 1));
        MM_TRY(part.alloc((size_t)nch * (lam + 1)));
        MM_HIP(hipMemcpyAsync(dch.p, choff.data(), (pl->n_int + 1) * 8, hipMemcpyHostToDevice, st));
        if (lam == 0)
            hipLaunchKernelGGL(k_lag0, dim3(nch), dim3(kLcThreads), 0, st, u, v, pl->int_lo.p,
                               pl->int_hi.p, dch.p, pl->n_int, part.p);
        else
            hipLaunchKernelGGL(k_lag_corr, dim3(nch, (lam - kbeg + kLcLags) / kLcLags),
                               dim3(kLcThreads), 0, st, u, v, pl->int_lo.p, pl->int_hi.p, dch.p,
                               pl->n_int, lam, kbeg, part.p);
        MM_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_lag_reduce, dim3((lam - kbeg + 256) / 256, pl->n_int), dim3(256), 0,
                           st, part.p, dch.p, pl->int_lo.p, pl->int_hi.p, lam, kbeg, c);
        MM_HIP(hipGetLastError());
    }
    MM_HIP(hipStreamSynchronize(st));  // scratch is released on return
    return MM_OK;
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
