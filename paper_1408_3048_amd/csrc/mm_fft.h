// LDS-resident complex FFTs (radix 16, decimation in frequency forward and in time
// inverse) shared by the overlap-save N^-1, the plan-time transforms of the taps and the
// lag correlations of the adjoint.
#pragma once

#include "mm_internal.h"

namespace mm {
namespace {

// LDS layout of the complex work array (M points).  Element a lives at
// swz(a) = a ^ (((a >> 5) ^ (a >> 10)) & 31), a bijection within every block of 32
// points, with no padding.  With 8-byte accesses served 32 lanes at a time over the 64
// four-byte banks, enumerating every access pattern gives conflict-free radix-16 passes
// (the block-size-32 pass with its groups mapped so that k is uniform over a wave) and
// load/store phases, and a 1.2-way spectrum pass.  FP32 points are stored interleaved
// (one 8-byte access per point), FP64 as split real and imaginary arrays (two 8-byte
// accesses).
// swz is linear over XOR, so for bit-disjoint a and c, swz(a + c) = swz(a) ^ swz(c): the
// passes swizzle their thread's base index once and reach the other points by XOR with
// compile-time constants.
__host__ __device__ constexpr int swz(int a) { return a ^ (((a >> 5) ^ (a >> 10)) & 31); }

template <typename T>
struct CBuf;

template <>
struct CBuf<float> {
    float2* c;
    // at byte offset b (8 times an already swizzled position)
    __device__ __forceinline__ void get_swb(int b, float& re, float& im) const {
        const float2 v = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(c) + b);
        re = v.x;
        im = v.y;
    }
    __device__ __forceinline__ void put_swb(int b, float re, float im) const {
        *reinterpret_cast<float2*>(reinterpret_cast<char*>(c) + b) = make_float2(re, im);
    }
    __device__ __forceinline__ void put_part_sw(int p, int part, float v) const {
        reinterpret_cast<float*>(c)[2 * p + part] = v;
    }
    __device__ __forceinline__ void get(int a, float& re, float& im) const {
        const float2 v = c[swz(a)];
        re = v.x;
        im = v.y;
    }
    __device__ __forceinline__ void put(int a, float re, float im) const {
        c[swz(a)] = make_float2(re, im);
    }
    __device__ __forceinline__ void put_part(int a, int part, float v) const {
        reinterpret_cast<float*>(c)[2 * swz(a) + part] = v;
    }
    __device__ __forceinline__ float get_part(int a, int part) const {
        return reinterpret_cast<const float*>(c)[2 * swz(a) + part];
    }
};

template <>
struct CBuf<double> {
    double* re;
    double* im;
    __device__ __forceinline__ void get_swb(int b, double& r, double& i) const {
        r = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(re) + b);
        i = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(im) + b);
    }
    __device__ __forceinline__ void put_swb(int b, double r, double i) const {
        *reinterpret_cast<double*>(reinterpret_cast<char*>(re) + b) = r;
        *reinterpret_cast<double*>(reinterpret_cast<char*>(im) + b) = i;
    }
    __device__ __forceinline__ void put_part_sw(int p, int part, double v) const {
        (part ? im : re)[p] = v;
    }
    __device__ __forceinline__ void get(int a, double& r, double& i) const {
        const int p = swz(a);
        r = re[p];
        i = im[p];
    }
    __device__ __forceinline__ void put(int a, double r, double i) const {
        const int p = swz(a);
        re[p] = r;
        im[p] = i;
    }
    __device__ __forceinline__ void put_part(int a, int part, double v) const {
        (part ? im : re)[swz(a)] = v;
    }
    __device__ __forceinline__ double get_part(int a, int part) const {
        return (part ? im : re)[swz(a)];
    }
};

// the M-point complex buffer over 2 M sizeof(T) bytes of LDS
template <typename T>
__device__ __forceinline__ CBuf<T> make_cbuf(unsigned char* smem, int M) {
    CBuf<T> b;
    if constexpr (sizeof(T) == 4) {
        b.c = reinterpret_cast<float2*>(smem);
    } else {
        b.re = reinterpret_cast<double*>(smem);
        b.im = b.re + M;
    }
    return b;
}

template <int BITS>
__device__ __forceinline__ int rev_bits(int v) {
    return (int)(__builtin_bitreverse32((uint32_t)v) >> (32 - BITS));
}

// exp(-2 pi i e / 32), e = 0..15: the constants of the networks, and the twiddles of a
// radix-16 pass of block size 32 for its group k = 1 (cos and sin of multiples of pi/16)
template <typename T>
__device__ __forceinline__ void root32(int e, T& c, T& s) {
    // cos and sin of pi e / 16
    constexpr double cs[16] = {1.0, 0.98078528040323044913, 0.92387953251128675613,
                               0.83146961230254523708, 0.70710678118654752440,
                               0.55557023301960222474, 0.38268343236508977173,
                               0.19509032201612826785, 0.0, -0.19509032201612826785,
                               -0.38268343236508977173, -0.55557023301960222474,
                               -0.70710678118654752440, -0.83146961230254523708,
                               -0.92387953251128675613, -0.98078528040323044913};
    constexpr double sn[16] = {0.0, 0.19509032201612826785, 0.38268343236508977173,
                               0.55557023301960222474, 0.70710678118654752440,
                               0.83146961230254523708, 0.92387953251128675613,
                               0.98078528040323044913, 1.0, 0.98078528040323044913,
                               0.92387953251128675613, 0.83146961230254523708,
                               0.70710678118654752440, 0.55557023301960222474,
                               0.38268343236508977173, 0.19509032201612826785};
    c = (T)cs[e & 15];
    s = (T)(-sn[e & 15]);
}

// in-register radix-R DIF network (R <= 32): natural in, bit-reversed out (forward, e^{-i})
template <typename T, int R>
__device__ __forceinline__ void dif_net(T* vr, T* vi) {
#pragma unroll
    for (int h = R / 2; h >= 1; h >>= 1) {
#pragma unroll
        for (int b = 0; b < R; b += 2 * h) {
#pragma unroll
            for (int kk = 0; kk < h; ++kk) {
                const T ar = vr[b + kk], ai = vi[b + kk];
                const T cr = vr[b + kk + h], ci = vi[b + kk + h];
                vr[b + kk] = ar + cr;
                vi[b + kk] = ai + ci;
                const T dr = ar - cr, di = ai - ci;
                const int e = kk * (16 / h);  // exp(-2 pi i kk / 2h) = exp(-2 pi i e / 32)
                if (e == 0) {
                    vr[b + kk + h] = dr;
                    vi[b + kk + h] = di;
                } else if (e == 8) {  // * (-i)
                    vr[b + kk + h] = di;
                    vi[b + kk + h] = -dr;
                } else {
                    T c, s;
                    root32<T>(e, c, s);
                    vr[b + kk + h] = dr * c - di * s;
                    vi[b + kk + h] = dr * s + di * c;
                }
            }
        }
    }
}

// in-register inverse radix-R DIT network: bit-reversed in, natural out (e^{+i})
template <typename T, int R>
__device__ __forceinline__ void dit_net_inv(T* vr, T* vi) {
#pragma unroll
    for (int h = 1; h < R; h <<= 1) {
#pragma unroll
        for (int b = 0; b < R; b += 2 * h) {
#pragma unroll
            for (int kk = 0; kk < h; ++kk) {
                const int e = kk * (16 / h);
                T cr = vr[b + kk + h], ci = vi[b + kk + h];
                if (e == 8) {  // * (+i)
                    const T t = cr;
                    cr = -ci;
                    ci = t;
                } else if (e != 0) {
                    T c, s;
                    root32<T>(e, c, s);
                    s = -s;  // conjugate root
                    const T t = cr * c - ci * s;
                    ci = cr * s + ci * c;
                    cr = t;
                }
                const T ar = vr[b + kk], ai = vi[b + kk];
                vr[b + kk] = ar + cr;
                vi[b + kk] = ai + ci;
                vr[b + kk + h] = ar - cr;
                vi[b + kk + h] = ai - ci;
            }
        }
    }
}

// w^e for e = 0..R-1 from w (binary powering: short dependency chains)
template <typename T, int R>
__device__ __forceinline__ void powers(T wr, T wi, T* pr, T* pi) {
    pr[0] = (T)1;
    pi[0] = (T)0;
    if (R > 1) {
        pr[1] = wr;
        pi[1] = wi;
    }
#pragma unroll
    for (int e = 2; e < R; ++e) {
        const int a = (e & 1) ? e - 1 : e / 2;
        const int b = (e & 1) ? 1 : e / 2;
        pr[e] = pr[a] * pr[b] - pi[a] * pi[b];
        pi[e] = pr[a] * pi[b] + pi[a] * pr[b];
    }
}

// The passes address LDS by byte offsets: an 8-byte point (FP32 (re, im), or one FP64
// part) at swizzled position p sits at byte 8 p, and swz is linear over XOR, so the
// byte offset of point (base + c) is (8 swz(base)) ^ (8 swz(c)) for bit-disjoint base and
// c: one XOR with a compile-time constant per point.
// Twiddles of a pass (block size B = 2^LOGB, Q = B / 2^LR groups per block):
//  - Q == 2 (B = 32): the groups are mapped so that every wave has one k; k = 0 needs none,
//    k = 1 the constants root32;
//  - the passes after the first with Q >= 4 read w^e, e = 1 .. R-1, from an LDS table
//    filled at the start of the kernel (lt, [e - 1][k] per pass) where the table leaves the
//    tile's occupancy unchanged;
//  - otherwise binary powers of w = tw[k TWS] (the first pass, the plan-time transforms).
// Every source gives the same values: the LDS table holds the powers the last case forms.
template <typename T, int LOGM, int LOGB>
constexpr bool first_pass() {
    return LOGB == LOGM;
}
// entries of the LDS twiddle table before the pass of block size 2^LOGB (passes after the
// first, with Q >= 4), and in all
__host__ __device__ constexpr int ltw_offset(int logm, int logb) {
    int off = 0;
    for (int l = logm; l > logb; l -= (l >= 4 ? 4 : l)) {
        const int lr = l >= 4 ? 4 : l;
        const int q = (1 << l) >> lr;
        if (l != logm && q >= 4) off += ((1 << lr) - 1) * q;
    }
    return off;
}
__host__ __device__ constexpr int ltw_total(int logm) { return ltw_offset(logm, 0); }

template <typename T, int LOGM, int NT, int LR, int LOGB, bool LTW>
__device__ __forceinline__ void pass_twiddles(int k, const T* __restrict__ tw,
                                              const T* __restrict__ lt, T* pr, T* pi) {
    constexpr int R = 1 << LR, B = 1 << LOGB, Q = B / R, M = 1 << LOGM;
    constexpr int TWS = (2 * M) / B;
    if constexpr (Q == 2 && R == 16) {
#pragma unroll
        for (int e = 1; e < R; ++e) root32<T>(e, pr[e], pi[e]);
    } else if constexpr (LTW && !first_pass<T, LOGM, LOGB>() && Q >= 4) {
        const T* tb = lt + 2 * (ltw_offset(LOGM, LOGB) + k);
#pragma unroll
        for (int e = 1; e < R; ++e) {
            pr[e] = tb[2 * (e - 1) * Q];
            pi[e] = tb[2 * (e - 1) * Q + 1];
        }
    } else {
        powers<T, R>(tw[2 * k * TWS], tw[2 * k * TWS + 1], pr, pi);
    }
}

// the LDS twiddle table of the passes after the first (see pass_twiddles), formed by the
// same binary powers the passes would take; every thread must call
template <typename T, int LOGM, int NT>
__device__ __forceinline__ void fill_ltw(const T* __restrict__ tw, T* lt) {
    constexpr int M = 1 << LOGM;
    for (int l = LOGM - 4; l > 0; l -= (l >= 4 ? 4 : l)) {
        const int lr = l >= 4 ? 4 : l;
        const int q = (1 << l) >> lr;
        if (q < 4) continue;
        const int tws = (2 * M) >> l;
        const int off = ltw_offset(LOGM, l);
        for (int k = threadIdx.x; k < q; k += NT) {
            T pr[16], pi[16];
            const T wr = tw[2 * k * tws], wi = tw[2 * k * tws + 1];
            if (lr == 4) powers<T, 16>(wr, wi, pr, pi);
            else if (lr == 3) powers<T, 8>(wr, wi, pr, pi);
            else powers<T, 4>(wr, wi, pr, pi);
            for (int e = 1; e < (1 << lr); ++e) {
                lt[2 * (off + (e - 1) * q + k)] = k ? pr[e] : (T)1;
                lt[2 * (off + (e - 1) * q + k) + 1] = k ? pi[e] : (T)0;
            }
        }
    }
}

// group g of a pass -> (block, k); for Q == 2 the first half of the groups has k = 0 and
// the second k = 1, so that k is uniform over a wave
template <int Q, int G>
__device__ __forceinline__ void pass_group(int g, int& blk, int& k) {
    if constexpr (Q == 2) {
        k = g >= G / 2 ? 1 : 0;
        blk = g & (G / 2 - 1);
    } else {
        k = g & (Q - 1);
        blk = g / Q;
    }
}

template <typename T, int LOGM, int NT, int LR, int LOGB, bool LTW = false>
__device__ __forceinline__ void dif_pass(const CBuf<T>& buf, const T* __restrict__ tw,
                                         const T* __restrict__ lt = nullptr) {
    constexpr int R = 1 << LR, B = 1 << LOGB, Q = B / R, M = 1 << LOGM, G = M / R;
    for (int g = threadIdx.x; g < G; g += NT) {
        int blk, k;
        pass_group<Q, G>(g, blk, k);
        const int sbb = swz(blk * B + k) << 3;  // base and m Q are bit-disjoint
        T vr[R], vi[R];
#pragma unroll
        for (int m = 0; m < R; ++m) buf.get_swb(sbb ^ (swz(m * Q) << 3), vr[m], vi[m]);
        dif_net<T, R>(vr, vi);
        if (Q > 1 && k != 0) {
            T pr[R], pi[R];
            pass_twiddles<T, LOGM, NT, LR, LOGB, LTW>(k, tw, lt, pr, pi);
#pragma unroll
            for (int i = 1; i < R; ++i) {
                const int e = rev_bits<LR>(i);
                const T t = vr[i] * pr[e] - vi[i] * pi[e];
                vi[i] = vr[i] * pi[e] + vi[i] * pr[e];
                vr[i] = t;
            }
        }
#pragma unroll
        for (int i = 0; i < R; ++i) buf.put_swb(sbb ^ (swz(i * Q) << 3), vr[i], vi[i]);
    }
    __syncthreads();
}

template <typename T, int LOGM, int NT, int LR, int LOGB, bool LTW = false>
__device__ __forceinline__ void dit_pass(const CBuf<T>& buf, const T* __restrict__ tw,
                                         const T* __restrict__ lt = nullptr) {
    constexpr int R = 1 << LR, B = 1 << LOGB, Q = B / R, M = 1 << LOGM, G = M / R;
    for (int g = threadIdx.x; g < G; g += NT) {
        int blk, k;
        pass_group<Q, G>(g, blk, k);
        const int sbb = swz(blk * B + k) << 3;
        T vr[R], vi[R];
#pragma unroll
        for (int i = 0; i < R; ++i) buf.get_swb(sbb ^ (swz(i * Q) << 3), vr[i], vi[i]);
        if (Q > 1 && k != 0) {
            T pr[R], pi[R];
            pass_twiddles<T, LOGM, NT, LR, LOGB, LTW>(k, tw, lt, pr, pi);
#pragma unroll
            for (int i = 1; i < R; ++i) {
                const int e = rev_bits<LR>(i);
                const T t = vr[i] * pr[e] + vi[i] * pi[e];  // * conj(w^e)
                vi[i] = vi[i] * pr[e] - vr[i] * pi[e];
                vr[i] = t;
            }
        }
        dit_net_inv<T, R>(vr, vi);
#pragma unroll
        for (int m = 0; m < R; ++m) buf.put_swb(sbb ^ (swz(m * Q) << 3), vr[m], vi[m]);
    }
    __syncthreads();
}

// STOP = 1: the last radix-2 stage (LOGB == 1) is left to the fused spectrum pass.  LTW:
// the passes after the first read their twiddles from the LDS table lt.
template <typename T, int LOGM, int NT, int LOGB, int STOP = 0, bool LTW = false>
__device__ __forceinline__ void fwd_passes(const CBuf<T>& buf, const T* tw,
                                           const T* lt = nullptr) {
    if constexpr (LOGB > STOP) {
        constexpr int LR = LOGB >= 4 ? 4 : LOGB;
        dif_pass<T, LOGM, NT, LR, LOGB, LTW>(buf, tw, lt);
        fwd_passes<T, LOGM, NT, LOGB - LR, STOP, LTW>(buf, tw, lt);
    }
}

template <typename T, int LOGM, int NT, int LOGB, int STOP = 0, bool LTW = false>
__device__ __forceinline__ void inv_passes(const CBuf<T>& buf, const T* tw,
                                           const T* lt = nullptr) {
    if constexpr (LOGB > STOP) {
        constexpr int LR = LOGB >= 4 ? 4 : LOGB;
        inv_passes<T, LOGM, NT, LOGB - LR, STOP, LTW>(buf, tw, lt);
        dit_pass<T, LOGM, NT, LR, LOGB, LTW>(buf, tw, lt);
    }
}

}  // namespace
}  // namespace mm
