// Pixel-domain kernels of PCG [Sect. 3.1] for a batch of independent problems:
// fused updates with deterministic per-problem partial sums and device-resident
// per-problem scalars, so the host never waits for a dot product, and the small
// control kernels (one block per problem) that take every convergence decision
// on the device.  A plain plan is a batch of one.
#include <algorithm>
#include <vector>

#include "mm_device.h"

namespace mm {
namespace {

__device__ __forceinline__ bool first_thread(const VecBlock& v) {
    return v.k == 0 && threadIdx.x == 0;
}

// partials of a^T b (per problem) into `slot`
__global__ __launch_bounds__(kVecThreads) void k_dot(const double* __restrict__ a,
                                                     const double* __restrict__ b, int slot,
                                                     int ns, PcgCtl c,
                                                     const int64_t* __restrict__ wave_off) {
    __shared__ double red[kVecThreads];
    const VecBlock v = vec_block(c, ns, true);
    if (c.mask && !c.mask[v.b]) return;
    // the problems whose partials P^T has left already
    if (wave_off && wave_off[v.b + 1] - wave_off[v.b] <= kVecBlocks) return;
    double acc = 0.0;
    for (int64_t i = (int64_t)v.k * kVecThreads + threadIdx.x; i < v.n;
         i += v.stride)
        acc += a[v.base + i] * b[v.base + i];
    write_partial_at(acc, slot_part(c, slot, v.b), v.k, red);
}

// the step length alpha = r^T z / p^T q of a block's problem from the partials of p^T q, and
// its bookkeeping; false (for every thread) on a breakdown.  All threads must call.
__device__ __forceinline__ bool step_length(const PcgCtl& c, const VecBlock& v, double* red,
                                            double& alpha) {
    PcgScalars& s = c.sc[v.b];
    const double pq = reduce_partials(slot_part(c, kSlotPQ, v.b), kVecBlocks, red);
    const double rz = c.rz_hist[(int64_t)v.b * c.hstride + s.iter];
    if (!(pq > 0.0 && isfinite(pq) && isfinite(rz))) {
        if (first_thread(v)) {
            s.status = 1;
            s.state = kBreakdown;
            s.pq = pq;
            c.act[v.b] = 0;
        }
        return false;
    }
    alpha = rz / pq;
    if (first_thread(v)) {
        s.alpha = alpha;
        s.pq = pq;
        s.iter_next = s.iter + 1;
        if (c.alpha_hist) c.alpha_hist[(int64_t)v.b * c.hstride + s.iter] = alpha;
    }
    return true;
}

// x += alpha p; r -= alpha q; partials of ||r||^2
__global__ __launch_bounds__(kVecThreads) void k_update_xr(double* __restrict__ x,
                                                           double* __restrict__ r,
                                                           const double* __restrict__ p,
                                                           const double* __restrict__ q, int ns,
                                                           PcgCtl c) {
    __shared__ double red[kVecThreads];
    const VecBlock v = vec_block(c, ns, true);
    if (c.mask && !c.mask[v.b]) return;
    double alpha;
    if (!step_length(c, v, red, alpha)) return;
    double acc = 0.0;
    for (int64_t i = (int64_t)v.k * kVecThreads + threadIdx.x; i < v.n;
         i += v.stride) {
        const int64_t e = v.base + i;
        x[e] += alpha * p[e];
        const double rv = r[e] - alpha * q[e];
        r[e] = rv;
        acc += rv * rv;
    }
    write_partial_at(acc, slot_part(c, kSlotRR, v.b), v.k, red);
}

// k_update_xr and block Jacobi in one pass per pixel: z = M_BD r of the new residual while it
// is in registers, partials of ||r||^2 and r^T z.  One launch and one read of r instead of
// three launches with k_pcg_check between them (each about 2.5-4.5 us when small)
template <int NS>
__global__ __launch_bounds__(kVecThreads) void k_update_xr_bj(
    double* __restrict__ x, double* __restrict__ r, double* __restrict__ z,
    const double* __restrict__ p, const double* __restrict__ q, const double* __restrict__ bj,
    PcgCtl c) {
    __shared__ double red[kVecThreads];
    const VecBlock v = vec_block(c, NS, false);
    if (c.mask && !c.mask[v.b]) return;
    double alpha;
    if (!step_length(c, v, red, alpha)) return;
    double rr = 0.0, rz = 0.0;
    for (int64_t i = (int64_t)v.k * kVecThreads + threadIdx.x; i < v.n; i += v.stride) {
        const int64_t px = v.base + i, e = px * NS;
        double rv[NS], zv[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            x[e + s] += alpha * p[e + s];
            rv[s] = r[e + s] - alpha * q[e + s];
            r[e + s] = rv[s];
            rr += rv[s] * rv[s];
        }
        bj_block<NS>(bj + (NS == 3 ? 6 : 1) * px, rv, zv);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            z[e + s] = zv[s];
            rz += rv[s] * zv[s];
        }
    }
    write_partial_at(rr, slot_part(c, kSlotRR, v.b), v.k, red);
    write_partial_at(rz, slot_part(c, kSlotRZ, v.b), v.k, red);
}

// The convergence test of problem b on its recursive residual (partials of ||r||^2): after an
// iteration (initial = 0) it also counts the iteration and records the history.  Returns the
// problem's new state; thread 0 writes it where `write` is set.  All threads must call.
__device__ __forceinline__ int test_residual(const PcgCtl& c, int b, int initial, bool write,
                                             double* red) {
    const double rr = reduce_partials(slot_part(c, kSlotRR, b), kVecBlocks, red);
    PcgScalars& s = c.sc[b];
    const int iter = initial ? s.iter : s.iter_next;
    const double rel = sqrt(rr) / s.bnorm;
    int st = kActive;
    if (rel <= s.tol) st = (!initial && c.replace) ? kCheck : kDone;
    else if (!initial && c.replace_ratio > 0.0 && rel < c.replace_ratio * s.last_rel) st = kCheck;
    else if (!initial && iter >= c.max_iter) st = kMaxIter;
    if (write && threadIdx.x == 0) {
        s.iter = iter;
        s.rr = rr;
        s.rel = rel;
        if (!initial && c.hist) c.hist[(int64_t)(iter - 1) * c.B + b] = rel;
        if (st != kActive) {
            s.state = st;
            c.act[b] = 0;
        }
    }
    return st;
}

// beta = r_new^T z_new / r^T z; p = z + beta p (p = z on the first call), and p's packed map
// xp for the next A p.  The iteration count it = iter_next is that of the iteration just
// completed (or of the last completed one when resuming after a residual evaluation): r^T z
// of the new residual is stored at rz_hist[it] and divided by rz_hist[it - 1].
// test: the launch first takes the iteration's convergence test; every block of a problem
// takes it from the same partials, its first block writes the outcome (the others read
// neither iter nor state, and where it clears act, none has anything left to do).
// The test and the packing were launches of their own (2.5-4.6 and 1.4-4.7 us each)
template <int NS, typename TP>
__global__ __launch_bounds__(kVecThreads) void k_update_p(double* __restrict__ p,
                                                          const double* __restrict__ z,
                                                          TP* __restrict__ xp, int test,
                                                          PcgCtl c) {
    __shared__ double red[kVecThreads];
    const VecBlock v = vec_block(c, NS, false);
    if (c.mask && !c.mask[v.b]) return;
    PcgScalars& s = c.sc[v.b];
    const int it = s.iter_next;
    if (test && test_residual(c, v.b, 0, v.k == 0, red) != kActive) return;
    const double rz_new = reduce_partials(slot_part(c, kSlotRZ, v.b), kVecBlocks, red);
    double* rh = c.rz_hist + (int64_t)v.b * c.hstride;
    const double beta = c.first ? 0.0 : rz_new / rh[it - 1];
    if (first_thread(v)) {
        rh[it] = rz_new;
        s.beta = beta;
    }
    // Krylov recording: z of this iteration (rewritten when a residual evaluation resumes
    // the same iteration, together with rz_hist[it])
    double* kz = c.krylov && it < c.kcap ? c.krylov + (int64_t)it * c.knv : nullptr;
    for (int64_t i = (int64_t)v.k * kVecThreads + threadIdx.x; i < v.n; i += v.stride) {
        const int64_t px = v.base + i, e = px * NS;
        double pv[NS];
#pragma unroll
        for (int s1 = 0; s1 < NS; ++s1) {
            const double zv = z[e + s1];
            pv[s1] = c.first ? zv : zv + beta * p[e + s1];
            p[e + s1] = pv[s1];
            if (kz) kz[e + s1] = zv;
        }
        if constexpr (NS == 3) {
            xp[4 * px] = (TP)pv[0];
            xp[4 * px + 1] = (TP)pv[1];
            xp[4 * px + 2] = (TP)pv[2];
            xp[4 * px + 3] = (TP)0;
        }
    }
}

// out = b - y; partials of ||out||^2 in the Aux slot
__global__ __launch_bounds__(kVecThreads) void k_residual(const double* __restrict__ b,
                                                          const double* __restrict__ y,
                                                          double* __restrict__ out, int ns,
                                                          PcgCtl c) {
    __shared__ double red[kVecThreads];
    const VecBlock v = vec_block(c, ns, true);
    if (c.mask && !c.mask[v.b]) return;
    double acc = 0.0;
    for (int64_t i = (int64_t)v.k * kVecThreads + threadIdx.x; i < v.n;
         i += v.stride) {
        const int64_t e = v.base + i;
        const double t = b[e] - y[e];
        out[e] = t;
        acc += t * t;
    }
    write_partial_at(acc, slot_part(c, kSlotAux, v.b), v.k, red);
}

__global__ __launch_bounds__(kVecThreads) void k_axpby(double a, const double* __restrict__ x,
                                                       double b, const double* __restrict__ y,
                                                       double* __restrict__ out, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * kVecThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kVecThreads)
        out[i] = a * x[i] + b * y[i];
}

// x_b = 0 for the problems flagged in `flag`
__global__ __launch_bounds__(kVecThreads) void k_zero_flagged(double* __restrict__ x,
                                                              const int* __restrict__ flag,
                                                              int ns, PcgCtl c) {
    const VecBlock v = vec_block(c, ns, true);
    if (!flag[v.b]) return;
    for (int64_t i = (int64_t)v.k * kVecThreads + threadIdx.x; i < v.n;
         i += v.stride)
        x[v.base + i] = 0.0;
}

// ---------------------------------------------------------------- control kernels
// One block per problem b (gridDim.x = B).

// start of a solve: ||b_b|| from the Aux partials; a problem with b_b = 0 is done at
// once (its solution is 0) and flagged in zero_b when zero_b_done is set
__global__ __launch_bounds__(kVecThreads) void k_pcg_init(PcgCtl c, double tol, int zero_b_done,
                                                          int* __restrict__ sel) {
    __shared__ double red[kVecThreads];
    const int b = blockIdx.x;
    const double bb = reduce_partials(slot_part(c, kSlotAux, b), kVecBlocks, red);
    if (threadIdx.x == 0) {
        PcgScalars& s = c.sc[b];
        s.bnorm = sqrt(bb);
        s.tol = tol;
        s.alpha = s.beta = s.pq = s.rr = 0.0;
        s.rel = 1.0;
        s.last_rel = 1.0;
        s.status = 0;
        s.iter = 0;
        s.iter_next = 0;
        s.evals = 0;
        const bool zero = !(bb > 0.0);
        s.state = (zero && zero_b_done) ? kDone : kActive;
        c.act[b] = s.state == kActive;
        sel[b] = zero && zero_b_done;
    }
}

// convergence test of the initial residual (RR partials) of every iterating problem
__global__ __launch_bounds__(kVecThreads) void k_pcg_check(PcgCtl c) {
    __shared__ double red[kVecThreads];
    const int b = blockIdx.x;
    if (!c.act[b]) return;
    test_residual(c, b, 1, true, red);
}

// after b - A x of the problems in c.mask (state kCheck) is in r with its Aux partials:
// done when it meets the tolerance, else resume from it (or stop at max_iter)
__global__ __launch_bounds__(kVecThreads) void k_pcg_decide(PcgCtl c, int* __restrict__ sel) {
    __shared__ double red[kVecThreads];
    const int b = blockIdx.x;
    if (!sel[b]) return;
    const double tt = reduce_partials(slot_part(c, kSlotAux, b), kVecBlocks, red);
    if (threadIdx.x != 0) return;
    PcgScalars& s = c.sc[b];
    const double rel = sqrt(tt) / s.bnorm;
    s.last_rel = rel;
    s.rel = rel;
    if (rel <= s.tol) {
        s.state = kDone;
        sel[b] = 0;
    } else if (s.iter >= c.max_iter) {
        s.state = kMaxIter;
        sel[b] = 0;
    } else {
        s.state = kResume;
        s.evals++;
    }
}

// op 0: sel = (state == kCheck); op 1: resumed problems iterate again, sel cleared
__global__ void k_pcg_states(PcgCtl c, int* __restrict__ sel, int op) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= c.B) return;
    PcgScalars& s = c.sc[b];
    if (op == 0) {
        sel[b] = s.state == kCheck;
    } else {
        if (sel[b] && s.state == kResume) {
            s.state = kActive;
            c.act[b] = 1;
        }
        sel[b] = 0;
    }
}

// final true relative residual of every problem from the Aux partials (stored in rel)
__global__ __launch_bounds__(kVecThreads) void k_pcg_final(PcgCtl c) {
    __shared__ double red[kVecThreads];
    const int b = blockIdx.x;
    const double tt = reduce_partials(slot_part(c, kSlotAux, b), kVecBlocks, red);
    if (threadIdx.x == 0) {
        PcgScalars& s = c.sc[b];
        s.rel = s.bnorm > 0.0 ? sqrt(tt) / s.bnorm : sqrt(tt);
    }
}

}  // namespace

int64_t nvec(mm_plan_t pl) { return pl->n_obs * pl->n_s; }

// block offsets of the per-problem vector kernels
int build_batch_layout(mm_plan_t pl) {
    const int B = pl->n_prob;
    std::vector<int32_t> eb(B + 1, 0), pb(B + 1, 0);
    for (int b = 0; b < B; ++b) {
        const int64_t np = pl->h_ooff[b + 1] - pl->h_ooff[b];
        const int64_t ne = np * pl->n_s;
        // several items per thread: the prologue reductions of every block (over the
        // problem's partials) cost as much as a few items, so small problems of a batch
        // get few blocks; the count depends on the problem alone
        auto blocks = [](int64_t m, int per_thread) {
            const int64_t per_block = (int64_t)kVecThreads * per_thread;
            int64_t g = (m + per_block - 1) / per_block;
            return (int32_t)std::min<int64_t>(kVecBlocks, std::max<int64_t>(1, g));
        };
        eb[b + 1] = eb[b] + blocks(ne, kVecPerThreadE);
        pb[b + 1] = pb[b] + blocks(np, kVecPerThreadP);
    }
    pl->n_eblk = eb[B];
    pl->n_pblk = pb[B];
    hipStream_t st = pl->stream;
    MM_TRY(pl->eblk.alloc(B + 1));
    MM_TRY(pl->pblk.alloc(B + 1));
    MM_HIP(hipMemcpyAsync(pl->eblk.p, eb.data(), (B + 1) * 4, hipMemcpyHostToDevice, st));
    MM_HIP(hipMemcpyAsync(pl->pblk.p, pb.data(), (B + 1) * 4, hipMemcpyHostToDevice, st));
    MM_HIP(hipStreamSynchronize(st));
    return MM_OK;
}

PcgCtl batch_ctl(mm_plan_t pl) {
    PcgCtl c;
    c.part = pl->part.p;
    c.sc = pl->sc.p;
    c.mask = nullptr;
    c.act = pl->act.p;
    c.rz_hist = pl->rz_hist.p;
    c.hist = pl->hist.p;
    c.eblk = pl->eblk.p;
    c.pblk = pl->pblk.p;
    c.ooff = pl->ooff.p;
    c.B = pl->n_prob;
    c.hstride = pl->hstride;
    if (pl->krec.basis) {
        c.krylov = pl->krec.basis;
        c.alpha_hist = pl->krec.alpha;
        c.kcap = pl->krec.cap;
        c.knv = nvec(pl);
    }
    return c;
}

int vec_dot(mm_plan_t pl, const double* a, const double* b, int slot, const PcgCtl& ctl,
            const int64_t* wave_off) {
    hipLaunchKernelGGL(k_dot, dim3(pl->n_eblk), dim3(kVecThreads), 0, pl->stream, a, b, slot,
                       pl->n_s, ctl, wave_off);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int pcg_update_xr(mm_plan_t pl, double* x, double* r, const double* p, const double* q,
                  const PcgCtl& ctl) {
    hipLaunchKernelGGL(k_update_xr, dim3(pl->n_eblk), dim3(kVecThreads), 0, pl->stream, x, r, p,
                       q, pl->n_s, ctl);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int pcg_update_xr_bj(mm_plan_t pl, double* x, double* r, double* z, const double* p,
                     const double* q, const PcgCtl& ctl) {
    const dim3 g(pl->n_pblk), t(kVecThreads);
    if (pl->n_s == 3)
        hipLaunchKernelGGL(k_update_xr_bj<3>, g, t, 0, pl->stream, x, r, z, p, q,
                           (const double*)pl->bj.p, ctl);
    else
        hipLaunchKernelGGL(k_update_xr_bj<1>, g, t, 0, pl->stream, x, r, z, p, q,
                           (const double*)pl->bj.p, ctl);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int pcg_update_p(mm_plan_t pl, double* p, const double* z, bool op32, int test,
                 const PcgCtl& ctl) {
    const dim3 g(pl->n_pblk), t(kVecThreads);
    if (pl->n_s != 3)
        hipLaunchKernelGGL((k_update_p<1, double>), g, t, 0, pl->stream, p, z, (double*)nullptr,
                           test, ctl);
    else if (op32)
        hipLaunchKernelGGL((k_update_p<3, float>), g, t, 0, pl->stream, p, z, pl->xp32.p, test,
                           ctl);
    else
        hipLaunchKernelGGL((k_update_p<3, double>), g, t, 0, pl->stream, p, z, pl->xp64.p, test,
                           ctl);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int vec_residual(mm_plan_t pl, const double* b, const double* y, double* out,
                 const PcgCtl& ctl) {
    hipLaunchKernelGGL(k_residual, dim3(pl->n_eblk), dim3(kVecThreads), 0, pl->stream, b, y, out,
                       pl->n_s, ctl);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int vec_axpby(mm_plan_t pl, double a, const double* x, double b, const double* y, double* out) {
    hipLaunchKernelGGL(k_axpby, dim3(kVecBlocks), dim3(kVecThreads), 0, pl->stream, a, x, b, y, out,
                       nvec(pl));
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int vec_zero_flagged(mm_plan_t pl, double* x, const int* flag, const PcgCtl& ctl) {
    hipLaunchKernelGGL(k_zero_flagged, dim3(pl->n_eblk), dim3(kVecThreads), 0, pl->stream, x, flag,
                       pl->n_s, ctl);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int pcg_init(mm_plan_t pl, const PcgCtl& ctl, double tol, int zero_b_done) {
    hipLaunchKernelGGL(k_pcg_init, dim3(pl->n_prob), dim3(kVecThreads), 0, pl->stream, ctl, tol,
                       zero_b_done, pl->sel.p);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int pcg_check(mm_plan_t pl, const PcgCtl& ctl) {
    hipLaunchKernelGGL(k_pcg_check, dim3(pl->n_prob), dim3(kVecThreads), 0, pl->stream, ctl);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int pcg_decide(mm_plan_t pl, const PcgCtl& ctl) {
    hipLaunchKernelGGL(k_pcg_decide, dim3(pl->n_prob), dim3(kVecThreads), 0, pl->stream, ctl,
                       pl->sel.p);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int pcg_select(mm_plan_t pl, const PcgCtl& ctl) {
    hipLaunchKernelGGL(k_pcg_states, dim3((pl->n_prob + 255) / 256), dim3(256), 0, pl->stream, ctl,
                       pl->sel.p, 0);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int pcg_resume(mm_plan_t pl, const PcgCtl& ctl) {
    hipLaunchKernelGGL(k_pcg_states, dim3((pl->n_prob + 255) / 256), dim3(256), 0, pl->stream, ctl,
                       pl->sel.p, 1);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

int pcg_final(mm_plan_t pl, const PcgCtl& ctl) {
    hipLaunchKernelGGL(k_pcg_final, dim3(pl->n_prob), dim3(kVecThreads), 0, pl->stream, ctl);
    MM_HIP(hipGetLastError());
    return MM_OK;
}

}  // namespace mm
