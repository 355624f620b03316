// FP64 complex FFT of N = 2^LOGN points (4096 or 8192) held in registers, R = 16 points per
// thread over NT = N / 16 threads, with two exchanges through LDS each way.
//
// Forward (decimation in frequency): radix 16 over the points t + NT i, radix 16 over the
// blocks of NT points, and the remaining blocks of Q2 = NT / 16 points, of which a thread holds
// 16 consecutive positions (bit-reversed order; N = 8192 leaves blocks of 32, whose first stage
// runs between neighbouring lanes).  The inverse (decimation in time) retraces it.  The
// exchanges move the real parts, then the imaginary parts, through one array of N doubles:
// half the LDS of a complex buffer, so that 16 waves fit a CU where 8 did, and 4 exchanges
// instead of a read and a write of every point per pass.
//
// LDS positions (8-byte accesses, served 32 lanes at a time over 32 banks of 8 bytes): the
// first exchange pads the blocks where they are shorter than 32 points apart, the second
// permutes the 16 points of a thread by XOR; every access is without conflicts.
#pragma once

#include "mm_fft.h"

namespace mm {
namespace {

template <int LOGN>
struct RegFft {
    static constexpr int LOGR = 4, N = 1 << LOGN, R = 1 << LOGR, NT = N / R, Q2 = NT / R;
    static_assert(Q2 == 16 || Q2 == 32, "radix 16, radix 16, and blocks of 16 or 32");
    static constexpr bool CROSS = Q2 == 32;
    static constexpr int S1 = NT + (Q2 == 16 ? 16 : 0);  // LDS distance of the NT-point blocks
    static constexpr int ELEMS = R * S1;
    // the twiddle table: exp(-2 pi i 2^b t / N), t < NT, for b = 0 .. LOGR - 1, then
    // exp(-2 pi i 2^b k / NT), k < Q2
    static constexpr int TW = LOGR * (NT + Q2);

    // the compiler keeps the points in registers here, instead of moving loads, selects or
    // butterflies across and spilling
    static __device__ __forceinline__ void pin(double* vr, double* vi) {
#pragma unroll
        for (int i = 0; i < R; ++i) asm volatile("" : "+v"(vr[i]), "+v"(vi[i]));
    }
    // t as a value that the compiler does not know to be t: addresses formed from it are formed
    // again instead of being kept in registers from their first use
    static __device__ __forceinline__ int fresh(int t) {
        asm volatile("" : "+v"(t));
        return t;
    }

    // ---- powers w^e applied to the points of a radix step (INV: their conjugates)
    template <bool INV>
    static __device__ __forceinline__ void mul(double& r, double& i, double pr, double pi) {
        const double t = INV ? r * pr + i * pi : r * pr - i * pi;
        i = INV ? i * pr - r * pi : r * pi + i * pr;
        r = t;
    }
    // the exponents E + (bits below BIT), depth first: at most LOGR powers live
    template <bool INV, int BIT, int E>
    static __device__ __forceinline__ void twiddle_below(double* vr, double* vi, const double* wr,
                                                         const double* wi, double cr, double ci) {
        if constexpr (BIT > 0) {
            constexpr int b = BIT - 1, e = E + (1 << b), i = rev(e);
            const double pr = E ? cr * wr[b] - ci * wi[b] : wr[b];
            const double pi = E ? cr * wi[b] + ci * wr[b] : wi[b];
            mul<INV>(vr[i], vi[i], pr, pi);
            twiddle_below<INV, b, e>(vr, vi, wr, wi, pr, pi);
            twiddle_below<INV, b, E>(vr, vi, wr, wi, cr, ci);
        }
    }
    static constexpr int rev(int e) {
        int r = 0;
        for (int b = 0; b < LOGR; ++b) r |= ((e >> b) & 1) << (LOGR - 1 - b);
        return r;
    }
    // w^(2^b) at w + 2 b n, of a table of n entries per power: rounded once each, where
    // repeated squares would double the error at every step
    template <bool INV>
    static __device__ __forceinline__ void twiddle(double* vr, double* vi,
                                                   const double* __restrict__ w, int n) {
        double wr[LOGR], wi[LOGR];
#pragma unroll
        for (int b = 0; b < LOGR; ++b) {
            wr[b] = w[2 * b * n];
            wi[b] = w[2 * b * n + 1];
        }
        twiddle_below<INV, LOGR, 0>(vr, vi, wr, wi, 1.0, 0.0);
    }

    // ---- LDS positions of point i of thread t
    static __device__ __forceinline__ int first(int t, int i) { return t + i * S1; }
    static __device__ __forceinline__ int second(int t, int i) {  // first exchange, radix step 2
        return (t / Q2) * S1 + (t & (Q2 - 1)) + i * Q2;
    }
    // second exchange: position p of the transform sits at p ^ ((p >> 5) & 15) of its 16
    static __device__ __forceinline__ int second2(int t, int i) {
        const int blk = t / Q2, k = t & (Q2 - 1);
        if constexpr (CROSS) return blk * S1 + (k & 16) + 32 * i + ((k & 15) ^ i);
        else return blk * S1 + 16 * i + (k ^ (((blk & 1) << 3) ^ (i >> 1)));
    }
    static __device__ __forceinline__ int third(int t, int i) {
        return 16 * t + (t / Q2) * (S1 - NT) + (i ^ ((t >> 1) & 15));
    }

    template <class From, class To>
    static __device__ __forceinline__ void move(double* s, double* v, From from, To to) {
#pragma unroll
        for (int i = 0; i < R; ++i) s[from(i)] = v[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = s[to(i)];
        __syncthreads();
    }

    // v of the neighbouring lane (t ^ 1), plus or minus one's own
    static __device__ __forceinline__ double across(double v, double sg) {
        const int2 p = __builtin_bit_cast(int2, v);
        return __builtin_bit_cast(double,
                                  make_int2(__builtin_amdgcn_mov_dpp(p.x, 0xB1, 0xf, 0xf, true),
                                            __builtin_amdgcn_mov_dpp(p.y, 0xB1, 0xf, 0xf, true))) +
               sg * v;
    }

    // natural order (point t + NT i in v[i]) -> bit-reversed order (position 16 t + i)
    static __device__ __forceinline__ void forward(double* vr, double* vi, double* s,
                                                   const double* __restrict__ tw, int t) {
        dif_net<double, R>(vr, vi);
        twiddle<false>(vr, vi, tw + 2 * t, NT);
        move(s, vr, [&](int i) { return first(t, i); }, [&](int i) { return second(t, i); });
        move(s, vi, [&](int i) { return first(t, i); }, [&](int i) { return second(t, i); });
        pin(vr, vi);
        t = fresh(t);
        dif_net<double, R>(vr, vi);
        twiddle<false>(vr, vi, tw + 2 * LOGR * NT + 2 * (t & (Q2 - 1)), Q2);
        move(s, vr, [&](int i) { return second2(t, i); }, [&](int i) { return third(t, i); });
        move(s, vi, [&](int i) { return second2(t, i); }, [&](int i) { return third(t, i); });
        pin(vr, vi);
        if constexpr (CROSS) {
            const double sg = t & 1 ? -1.0 : 1.0;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                vr[i] = across(vr[i], sg);
                vi[i] = across(vi[i], sg);
            }
            if (t & 1) {
#pragma unroll
                for (int i = 1; i < R; ++i) {
                    double c, sn;
                    root32<double>(i, c, sn);
                    mul<false>(vr[i], vi[i], c, sn);
                }
            }
        }
        dif_net<double, R>(vr, vi);
    }

    // the inverse, unscaled: bit-reversed order -> natural order
    static __device__ __forceinline__ void inverse(double* vr, double* vi, double* s,
                                                   const double* __restrict__ tw, int t) {
        dit_net_inv<double, R>(vr, vi);
        if constexpr (CROSS) {
            if (t & 1) {
#pragma unroll
                for (int i = 1; i < R; ++i) {
                    double c, sn;
                    root32<double>(i, c, sn);
                    mul<true>(vr[i], vi[i], c, sn);
                }
            }
            const double sg = t & 1 ? -1.0 : 1.0;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                vr[i] = across(vr[i], sg);
                vi[i] = across(vi[i], sg);
            }
        }
        move(s, vr, [&](int i) { return third(t, i); }, [&](int i) { return second2(t, i); });
        move(s, vi, [&](int i) { return third(t, i); }, [&](int i) { return second2(t, i); });
        pin(vr, vi);
        t = fresh(t);
        twiddle<true>(vr, vi, tw + 2 * LOGR * NT + 2 * (t & (Q2 - 1)), Q2);
        dit_net_inv<double, R>(vr, vi);
        move(s, vr, [&](int i) { return second(t, i); }, [&](int i) { return first(t, i); });
        move(s, vi, [&](int i) { return second(t, i); }, [&](int i) { return first(t, i); });
        pin(vr, vi);
        twiddle<true>(vr, vi, tw + 2 * t, NT);
        dit_net_inv<double, R>(vr, vi);
    }
};

}  // namespace
}  // namespace mm
