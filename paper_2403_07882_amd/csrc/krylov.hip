// krylov.hip -- preconditioned BiCGStab and flexible GMRES(m) on the device,
// the AMG V-cycle, and the mixed-precision wrapper.
//
// Solver families of Sec. 2.3 (GMRES, bi-conjugate gradient) with the AMG
// preconditioner.  All Krylov scalars (rho, alpha, omega, Hessenberg, Givens)
// live in device memory, one set per system, so a batch of independent
// systems runs through the same launches; the host only reads the
// per-system "converged" flags every `check_every` iterations.  Reductions
// are two-stage and deterministic: one partial per (system, work item),
// then a per-system sum over its items in a fixed order.
//
// Mixed precision: the hierarchy (level matrices, smoother sweeps, level
// vectors) runs in FP32, while residuals, inner products, D^{-1} and the
// coarsest dense inverse stay FP64 (FP64 -> FP32 casts round to nearest even).
#include "cbs_internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace {

enum { PH_INIT = 0, PH_END, PH_RESTART, PH_TRUE, PH_SNORM };

// flags bits: 1 breakdown; 2 converged at the half step (||s|| met the
// tolerance: the iteration ends with x += alpha ph, r = s); 4 the residual,
// shrinking as in the last iteration, would be within 4x of the tolerance
// after the next one
constexpr int32_t kFlagBreak = 1, kFlagHalf = 2, kFlagNear = 4;
// Slots of partial sums in a BiCGStab iteration: (rhat, v), later (t, s) and
// (t, t) in the first two; (s, s), written with s, read at the half-step test;
// the new (r, r) and (rhat, r), written by the workgroups that still read the
// first three.
constexpr int kSlotSS = 2, kSlotRR = 3, kSlotRhR = 4, kSlots = 5;
constexpr int32_t kDotWgs = 4096;                 // see spmv_dots

__device__ inline double block_sum(double v, double *sh) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) sh[wid] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
    __syncthreads();
    return t;   // valid in thread 0
}

// the block sums of K values at once -> v[0..K) in thread 0 (sh: 4 K doubles)
template <int K>
__device__ inline void block_sums(double (&v)[K], double *sh) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < K; ++q) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o, 64);
        if (lane == 0) sh[wid * K + q] = v[q];
    }
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int q = 0; q < K; ++q) {
            v[q] = 0.0;
            for (int w = 0; w < (int)(blockDim.x >> 6); ++w) v[q] += sh[w * K + q];
        }
}

// up to three dot products of one work item -> partial[q * n_items + item]
__global__ __launch_bounds__(kVecThreads) void k_dots(const Item *__restrict__ items, int32_t n_items,
                                                      const int32_t *__restrict__ done, int K,
                                                      const double *a0, const double *b0, const double *a1,
                                                      const double *b1, const double *a2, const double *b2,
                                                      double *partial) {
    __shared__ double sh[kVecThreads / 64];
    const Item it = items[blockIdx.x];
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    if (!done[it.sys]) {
        for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) {
            s0 += a0[e] * b0[e];
            if (K > 1) s1 += a1[e] * b1[e];
            if (K > 2) s2 += a2[e] * b2[e];
        }
    }
    s0 = block_sum(s0, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = s0;
    if (K > 1) { s1 = block_sum(s1, sh); if (threadIdx.x == 0) partial[n_items + blockIdx.x] = s1; }
    if (K > 2) { s2 = block_sum(s2, sh); if (threadIdx.x == 0) partial[2 * n_items + blockIdx.x] = s2; }
}

// Sums of one system's partials in K slots, by the whole workgroup: thread t
// adds items i0+t, i0+t+256, ... in order, then a fixed tree combines the
// threads, so the result does not depend on timing, nor on the workgroup that
// forms it.  Every thread gets the values.  sh: 4 K doubles.
constexpr int kFinThreads = 256;
static_assert(kFinThreads == kVecThreads, "element-wise workgroups form the sums too");

template <int K>
__device__ inline void sum_items(const double *__restrict__ partial, int32_t n_items, const int (&slot)[K],
                                 int32_t i0, int32_t i1, double *sh, double (&v)[K]) {
#pragma unroll
    for (int q = 0; q < K; ++q) v[q] = 0.0;
#pragma unroll 4
    for (int32_t k = i0 + (int32_t)threadIdx.x; k < i1; k += kFinThreads)
#pragma unroll
        for (int q = 0; q < K; ++q) v[q] += partial[(int64_t)slot[q] * n_items + k];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < K; ++q) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o, 64);
        if (lane == 0) sh[wid * K + q] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < K; ++q) {
        v[q] = 0.0;
        for (int w = 0; w < kFinThreads / 64; ++w) v[q] += sh[w * K + q];
    }
}

#define SC(slot) scal[(slot) * nsys + s]

// Where the scalar kernels leave a system's state for the host (pinned memory;
// see cbs_system::h_state): done, flags and iterations after every change, and
// the scalars that the host reads when a true residual is formed.  From
// kMirrorSystems systems on (state null here) a launch after them does it, whose
// stores are in whole lines: 20,000 systems, k_fin 82 us, with the scalars 274 us,
// and now 28 + 7 and 17 + 17 us; 2,000 systems 11 and 32 us, now 5.6 + 4.1 us.
struct HostMirror {
    int32_t *state;
    double *scal;
};
constexpr int kMirrorSystems = 1024;

__device__ inline void publish_state(const HostMirror &hm, int s, int nsys, const int32_t *done, const int32_t *flags,
                                     const int32_t *iters) {
    if (!hm.state) return;
    hm.state[s] = done[s];
    hm.state[nsys + s] = flags[s];
    hm.state[2 * nsys + s] = iters[s];
}

__device__ inline void publish_scal(const HostMirror &hm, int s, int nsys, const double *scal) {
    if (!hm.state) return;
    constexpr int slot[4] = {S_RR, S_BB, S_RES0, S_RREC};
#pragma unroll
    for (int q = 0; q < 4; ++q) hm.scal[slot[q] * nsys + s] = scal[slot[q] * nsys + s];
}

__global__ __launch_bounds__(256) void k_publish(HostMirror hm, int nsys, const int32_t *__restrict__ done,
                                                 const int32_t *__restrict__ flags, const int32_t *__restrict__ iters,
                                                 const double *__restrict__ scal) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= nsys) return;
    publish_state(hm, s, nsys, done, flags, iters);
    if (scal) publish_scal(hm, s, nsys, scal);
}

// Per-system scalar updates after a reduction.
__global__ __launch_bounds__(kFinThreads) void k_fin(int phase, int32_t nsys, const int32_t *__restrict__ item_off,
                                                      int32_t n_items, const double *__restrict__ partial, double *scal,
                                                      int32_t *done, int32_t *flags, int32_t *iters, double tol2,
                                                      const int32_t *restart_mask, HostMirror hm) {
    const int s = blockIdx.x;
    const int32_t i0 = item_off[s], i1 = item_off[s + 1];
    const bool skip = (phase == PH_RESTART && !restart_mask[s]) ||
                      ((phase == PH_END || phase == PH_SNORM) && (done[s] || (flags[s] & kFlagBreak)));
    if (skip) return;
    __shared__ double sh[2 * kFinThreads / 64];
    double q[2];
    if (phase == PH_INIT || phase == PH_END)
        sum_items<2>(partial, n_items, {phase == PH_END ? kSlotRR : 0, phase == PH_END ? kSlotRhR : 1}, i0, i1, sh, q);
    else
        sum_items<1>(partial, n_items, {phase == PH_SNORM ? kSlotSS : 0}, i0, i1, sh, reinterpret_cast<double(&)[1]>(q));
    const double q0 = q[0], q1 = q[1];
    if (threadIdx.x != 0) return;
    if (phase == PH_INIT) {
        const double rr = q0, bb = q1;
        SC(S_RR) = rr; SC(S_BB) = bb; SC(S_RES0) = bb > 0.0 ? sqrt(rr / bb) : 0.0;
        SC(S_RHO) = rr; SC(S_RHO0) = 1.0; SC(S_ALPHA) = 1.0; SC(S_OMEGA) = 1.0; SC(S_RRPREV) = 0.0;
        done[s] = (bb == 0.0 || rr <= tol2 * bb) ? 1 : 0;
        flags[s] = 0;
        iters[s] = 0;
    } else if (phase == PH_TRUE) {                   // true residual of every system; the
        SC(S_RREC) = SC(S_RR);                       // recurrence's is kept
        SC(S_RR) = q0;
        publish_scal(hm, s, nsys, scal);
        return;
    } else if (phase == PH_RESTART) {                // rhat = r; p = v = 0 done by the caller
        const double rr = q0;
        SC(S_RR) = rr; SC(S_RHO) = rr; SC(S_RHO0) = 1.0; SC(S_ALPHA) = 1.0; SC(S_OMEGA) = 1.0;
        SC(S_RRPREV) = 0.0;
        done[s] = (SC(S_BB) == 0.0 || rr <= tol2 * SC(S_BB)) ? 1 : 0;
        flags[s] = 0;
    } else if (phase == PH_SNORM) {                  // ||s||^2: converged at the half step?
        if (q0 <= tol2 * SC(S_BB)) flags[s] |= kFlagHalf;
    } else if (phase == PH_END) {
        const double rr = q0, rhn = q1;
        SC(S_RR) = rr;
        SC(S_RHO0) = SC(S_RHO);
        SC(S_RHO) = rhn;
        // after a half step r = s has met the tolerance whatever (r, r) rounds to:
        // it may be summed in another order than (s, s) was
        if (rr <= tol2 * SC(S_BB) || (flags[s] & kFlagHalf)) done[s] = 1;
        else if (SC(S_OMEGA) == 0.0 || rhn == 0.0 || !isfinite(rhn) || (flags[s] & kFlagBreak)) flags[s] |= kFlagBreak;
        flags[s] &= ~(kFlagHalf | kFlagNear);
        const double rrp = SC(S_RRPREV);
        if (rrp > 0.0 && rr * (rr / rrp) <= 16.0 * tol2 * SC(S_BB)) flags[s] |= kFlagNear;
        SC(S_RRPREV) = rr;
    }
    publish_state(hm, s, nsys, done, flags, iters);
}

// The preconditioner's zero-guess block-Jacobi sweep x = omega Dinv v, made by
// the kernel that forms the vector v it starts from: one launch less per
// application, and v is not read again.  b keeps v rounded to T (null in FP64,
// where the cycle reads v itself), c = Dinv v if it is wanted; the roundings are
// those of the sweep's own kernels.
template <typename T>
struct SweepOut {
    T *b, *x, *c;
    const double *Dinv;
    double omega;
};

// Work items start at a block row, so a workgroup takes kVecThreads / n whole
// rows at a time.
template <int n> constexpr int kTile = kVecThreads / n * n;

// One item of v and the sweep on it, kTiles tiles at a time so that their loads
// are in flight together: load(e, raw) reads what element e is made of, form(e,
// raw) makes it, stores it and returns it.  sb holds a step's values, others
// from step to step, so that one barrier is enough.
constexpr int kTiles = 2;
template <int n, typename T> using TileLds = T[2][kTiles][kVecThreads];

template <int n, typename T, typename Load, typename Form>
__device__ inline void item_sweep0(const Item &it, const SweepOut<T> &z, TileLds<n, T> &sb, Load load, Form form) {
    const int t = threadIdx.x;
    int turn = 0;
    for (int64_t base = it.beg; base < it.end; base += kTiles * kTile<n>, turn ^= 1) {
        double raw[kTiles][3], di[kTiles][n];
        bool act[kTiles];
#pragma unroll
        for (int u = 0; u < kTiles; ++u) {
            const int64_t e = base + u * kTile<n> + t;
            act[u] = t < kTile<n> && e < it.end;
            if (!act[u]) continue;
            load(e, raw[u]);
            const double *d = z.Dinv + e * n;              // (element e is a row of a block: n values)
#pragma unroll
            for (int k = 0; k < n; ++k) di[u][k] = d[k];
        }
#pragma unroll
        for (int u = 0; u < kTiles; ++u) {
            if (!act[u]) continue;
            const int64_t e = base + u * kTile<n> + t;
            const T bv = (T)form(e, raw[u]);
            sb[turn][u][t] = bv;
            if (z.b) z.b[e] = bv;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kTiles; ++u) {
            if (!act[u]) continue;
            const int64_t e = base + u * kTile<n> + t;
            const T *row = sb[turn][u] + t / n * n;
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < n; ++k) s += di[u][k] * (double)row[k];
            z.x[e] = (T)((T)0 + (T)(z.omega * s));
            if (z.c) z.c[e] = (T)s;
        }
    }
}

// p = r + beta (p - omega v),  beta = (rho / rho0) (alpha / omega), and the
// zero-guess sweep on p (on the old p for a system that is through)
template <int n, typename T>
__global__ __launch_bounds__(kVecThreads) void k_p_update_sweep(const Item *__restrict__ items, int32_t nsys,
                                                                const int32_t *__restrict__ done,
                                                                const double *__restrict__ scal,
                                                                const int32_t *__restrict__ flags,
                                                                const double *__restrict__ r, double *__restrict__ p,
                                                                const double *__restrict__ v, SweepOut<T> z) {
    __shared__ TileLds<n, T> sb;
    const Item it = items[blockIdx.x];
    const int s = it.sys;
    const bool on = !(done[s] || (flags[s] & kFlagBreak));
    const double omega = SC(S_OMEGA);
    const double beta = (SC(S_RHO) / SC(S_RHO0)) * (SC(S_ALPHA) / omega);
    item_sweep0<n, T>(
        it, z, sb,
        [&](int64_t e, double (&raw)[3]) {
            raw[0] = p[e];
            raw[1] = r[e];
            raw[2] = v[e];
        },
        [&](int64_t e, const double (&raw)[3]) {
            if (!on) return raw[0];
            const double pe = raw[1] + beta * (raw[0] - omega * raw[2]);
            p[e] = pe;
            return pe;
        });
}

// p alone, for the other preconditioners
__global__ __launch_bounds__(kVecThreads) void k_p_update(const Item *__restrict__ items, int32_t nsys,
                                                          const int32_t *__restrict__ done,
                                                          const double *__restrict__ scal,
                                                          const int32_t *__restrict__ flags, const double *r,
                                                          double *p, const double *v) {
    const Item it = items[blockIdx.x];
    const int s = it.sys;
    if (done[s] || (flags[s] & kFlagBreak)) return;
    const double omega = SC(S_OMEGA);
    const double beta = (SC(S_RHO) / SC(S_RHO0)) * (SC(S_ALPHA) / omega);
    for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) p[e] = r[e] + beta * (p[e] - omega * v[e]);
}

// The two updates that follow a reduction form its sums themselves, every
// workgroup those of its own system in the same order, instead of waiting for
// a launch that does nothing else (two of three such launches an iteration).
// BiCGStab of 960 rows: the three took 177 us of 15 iterations, solve and setup
// now 6.8% faster; 8,000 rows 6.3%, 55,000 rows 5.6%; 1M rows (977 partials)
// 0.2%.  The first workgroup of a system leaves the scalars.
// Every workgroup reading every partial grows with the square of the system: from
// kFoldItems items of a system on, a launch sums them first (k_fold_sums, the
// same sums) and the workgroups read its result.  5x5, 8M rows (9,769 items), FP64:
// k_xr_update 542 -> 516 us, k_s_update 193 -> 173 us, a BiCGStab iteration with
// block Jacobi 6.65 -> 6.63 ms, an FGMRES step with the V-cycle 23.5 -> 23.1 ms;
// 4M rows 3.33 and 3.33 ms, 11.54 -> 11.45 ms; 2M rows (2,443) 1.685 and 1.685
// ms, 5.865 -> 5.845 ms; 1M rows 0.867 and 0.869 ms, 3.048 -> 3.041 ms.

// Where the two products that follow A x are: partials of the work items in
// the first slots (k_dots), or of the product's own workgroups (count of them,
// one system).
struct DotSrc {
    const double *p;
    int32_t stride, count;                        // count 0: the system's items
};

// the items of every system; folded: the place of a system's first item in a
// slot of partials holds their sum (after k_fold_sums, or because it is the only
// one: no reductions in 20,000 workgroups of a system each)
struct ItemRange {
    const int32_t *off;
    bool folded;
};

// the sums of system s in K slots, by the whole workgroup; sh: 4 K doubles
template <int K>
__device__ inline void range_sums(const double *__restrict__ partial, int32_t n_items, const int (&slot)[K],
                                  const ItemRange &r, int s, double *sh, double (&v)[K]) {
    const int32_t i0 = r.off[s];
    if (!r.folded) {
        sum_items<K>(partial, n_items, slot, i0, r.off[s + 1], sh, v);
        return;
    }
#pragma unroll
    for (int q = 0; q < K; ++q) v[q] = partial[(int64_t)slot[q] * n_items + i0];
}
// the same where a product may have left its own partials
template <int K>
__device__ inline void dot_sums(const DotSrc &d, const int (&slot)[K], const ItemRange &r, int s, double *sh,
                                double (&v)[K]) {
    if (d.count) sum_items<K>(d.p, d.stride, slot, 0, d.count, sh, v);
    else range_sums<K>(d.p, d.stride, slot, r, s, sh, v);
}

// Sums of the slots slot0 + blockIdx.y, into the place of the system's first item
__global__ __launch_bounds__(kFinThreads) void k_fold_sums(const int32_t *__restrict__ item_off, int32_t n_items,
                                                            int slot0, double *partial) {
    __shared__ double sh[kFinThreads / 64];
    const int s = blockIdx.x, slot = slot0 + (int)blockIdx.y;
    double v[1];
    sum_items<1>(partial, n_items, {slot}, item_off[s], item_off[s + 1], sh, v);
    if (threadIdx.x == 0) partial[(int64_t)slot * n_items + item_off[s]] = v[0];
}

// alpha = rho / (rhat, v);  s = r - alpha v, and partials of (s, s) for the
// half-step test.  A breakdown ends the iteration's later parts, so it is
// published here.
struct AlphaStep {
    ItemRange items;
    const int32_t *done;
    double *scal;
    int32_t *flags, *iters;
    DotSrc ds;
    HostMirror hm;
};

// alpha of system s, or false at a breakdown (the whole workgroup); sh: 4 doubles.
// The system's first workgroup may set the breakdown flag while others read it,
// so the barriers of the sum lie before any branch on it: a wavefront that sees
// the flag then decides as the others do from the sum.
__device__ inline bool alpha_step(const AlphaStep &a, int s, int nsys, double *sh, double &alpha) {
    double *scal = a.scal;
    const int32_t i0 = a.items.off[s];
    const double rho = SC(S_RHO), rr = SC(S_RR);
    double rv[1];
    dot_sums<1>(a.ds, {0}, a.items, s, sh, rv);
    const bool broken = a.flags[s] & kFlagBreak;
    const bool bad = rv[0] == 0.0 || !isfinite(rv[0]) || fabs(rv[0]) < 1e-300 * fmax(rr, 1e-300);
    alpha = bad ? 0.0 : rho / rv[0];
    if (!broken && (int32_t)blockIdx.x == i0 && threadIdx.x == 0) {
        SC(S_RV) = rv[0];
        SC(S_ALPHA) = alpha;
        a.iters[s] += 1;
        if (bad) {
            a.flags[s] |= kFlagBreak;
            publish_state(a.hm, s, nsys, a.done, a.flags, a.iters);
        }
    }
    return !bad && !broken;
}

__global__ __launch_bounds__(kVecThreads) void k_s_update(const Item *__restrict__ items, int32_t n_items,
                                                          int32_t nsys, AlphaStep a, const double *__restrict__ r,
                                                          const double *__restrict__ v, double *__restrict__ sv,
                                                          double *__restrict__ partial) {
    __shared__ double red[kVecThreads / 64], sh[kFinThreads / 64];
    const Item it = items[blockIdx.x];
    const int s = it.sys;
    double s0 = 0.0;
    if (!a.done[s]) {
        int64_t e = it.beg + threadIdx.x;
        const bool have = e < it.end;
        double re = have ? r[e] : 0.0, ve = have ? v[e] : 0.0;       // (with the partials)
        double alpha;
        if (alpha_step(a, s, nsys, sh, alpha) && have)
            for (;;) {
                const double se = re - alpha * ve;
                sv[e] = se;
                s0 += se * se;
                e += kVecThreads;
                if (e >= it.end) break;
                re = r[e];
                ve = v[e];
            }
    }
    s0 = block_sum(s0, red);
    if (threadIdx.x == 0) partial[(int64_t)kSlotSS * n_items + blockIdx.x] = s0;
}

// the same and the zero-guess sweep on s
template <int n, typename T>
__global__ __launch_bounds__(kVecThreads) void k_s_update_sweep(const Item *__restrict__ items, int32_t n_items,
                                                                int32_t nsys, AlphaStep a,
                                                                const double *__restrict__ r,
                                                                const double *__restrict__ v, double *__restrict__ sv,
                                                                double *__restrict__ partial, SweepOut<T> z) {
    __shared__ double red[kVecThreads / 64], sh[kFinThreads / 64];
    __shared__ TileLds<n, T> sb;
    const Item it = items[blockIdx.x];
    const int s = it.sys;
    double alpha = 0.0, s0 = 0.0;
    const bool on = !a.done[s] && alpha_step(a, s, nsys, sh, alpha);
    item_sweep0<n, T>(
        it, z, sb,
        [&](int64_t e, double (&raw)[3]) {
            raw[0] = on ? r[e] : sv[e];
            raw[1] = v[e];
        },
        [&](int64_t e, const double (&raw)[3]) {
            if (!on) return raw[0];
            const double se = raw[0] - alpha * raw[1];
            sv[e] = se;
            s0 += se * se;
            return se;
        });
    s0 = block_sum(s0, red);
    if (threadIdx.x == 0) partial[(int64_t)kSlotSS * n_items + blockIdx.x] = s0;
}

// omega = (t, s) / (t, t);  x += alpha ph + omega sh;  r = s - omega t;
// partials (r,r), (rhat,r).  A system converged at the half step takes
// x += alpha ph, r = s.
__global__ __launch_bounds__(kVecThreads) void k_xr_update(const Item *__restrict__ items, ItemRange range,
                                                           int32_t n_items, int32_t nsys,
                                                           const int32_t *__restrict__ done, double *scal,
                                                           int32_t *flags, double tol2, double *__restrict__ x,
                                                           const double *__restrict__ ph, const double *__restrict__ sh,
                                                           double *__restrict__ r, const double *__restrict__ sv,
                                                           const double *__restrict__ t, const double *__restrict__ rh,
                                                           double *partial, DotSrc ds) {
    __shared__ double red[kVecThreads / 64], sums[3 * kFinThreads / 64];
    const Item it = items[blockIdx.x];
    const int s = it.sys;
    double s0 = 0.0, s1 = 0.0;
    const int32_t fl = flags[s];
    if (!done[s] && !(fl & kFlagBreak)) {
        const int32_t i0 = range.off[s];
        const double alpha = SC(S_ALPHA), bb = SC(S_BB);
        double q[2], ss[1];
        dot_sums<2>(ds, {0, 1}, range, s, sums, q);
        range_sums<1>(partial, n_items, {kSlotSS}, range, s, sums + 2 * kFinThreads / 64, ss);
        const bool half = (fl & kFlagHalf) || ss[0] <= tol2 * bb;
        const double omega = half ? 0.0 : (q[1] > 0.0 ? q[0] / q[1] : 0.0);
        if ((int32_t)blockIdx.x == i0 && threadIdx.x == 0) {
            SC(S_TS) = q[0];
            SC(S_TT) = q[1];
            SC(S_OMEGA) = omega;
            if (half) flags[s] = fl | kFlagHalf;
        }
        if (half) {
            for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) {
                x[e] += alpha * ph[e];
                const double re = sv[e];
                r[e] = re;
                s0 += re * re;
                s1 += rh[e] * re;
            }
        } else {
#pragma unroll 2
            for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) {
                x[e] += alpha * ph[e] + omega * sh[e];
                const double re = sv[e] - omega * t[e];
                r[e] = re;
                s0 += re * re;
                s1 += rh[e] * re;
            }
        }
    }
    s0 = block_sum(s0, red);
    if (threadIdx.x == 0) partial[(int64_t)kSlotRR * n_items + blockIdx.x] = s0;
    s1 = block_sum(s1, red);
    if (threadIdx.x == 0) partial[(int64_t)kSlotRhR * n_items + blockIdx.x] = s1;
}

// masked vector ops: y = a (copy), y = 0, x = 0 where b = 0 systems
__global__ void k_mask_copy(const Item *__restrict__ items, const int32_t *__restrict__ mask, int want,
                            const double *a, double *y) {
    const Item it = items[blockIdx.x];
    if ((mask[it.sys] != 0) != (want != 0)) return;
    for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) y[e] = a ? a[e] : 0.0;
}

__global__ void k_zero_if_bzero(const Item *__restrict__ items, int32_t nsys, const double *__restrict__ scal,
                                double *x) {
    const Item it = items[blockIdx.x];
    const int s = it.sys;
    if (SC(S_BB) != 0.0) return;
    for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) x[e] = 0.0;
}

// x += z (every element; a system that did not move contributes z = 0)
__global__ void k_gm_add(const Item *__restrict__ items, const double *__restrict__ z, double *x) {
    const Item it = items[blockIdx.x];
    for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) x[e] += z[e];
}

// ------------------------------------------------------------------ FGMRES
// The Gram-Schmidt kernels are bound by reading the basis.  A workgroup takes
// one item and kBasisGroup basis vectors at a time: the vector w is read once
// per group instead of once per basis vector, the group's loads are in flight
// together, and their sums are reduced in one pass.  59,319 cells, 5x5,
// GMRES(30), mean of 15 vectors and of both passes, the second mostly skipped:
// one vector at a time with a reduction each took 43 us for k_mdot and 28 us
// for k_maxpy, this form 8.1 us and 5.4 us.
constexpr int kBasisGroup = 8;

// One item's partials of (V_i, w) for the basis vectors i0 .. i0 + kBasisGroup - 1;
// past the basis (i > j) the slot up to K - 1 takes (w, w)
__device__ inline void item_dots(const Item &it, int item, int32_t n_items, int i0, int j, int K, int64_t ld,
                                 const double *__restrict__ V, const double *w, double *__restrict__ partial,
                                 double *red) {
    const double *vp[kBasisGroup];
    double acc[kBasisGroup];
#pragma unroll
    for (int q = 0; q < kBasisGroup; ++q) {
        vp[q] = i0 + q <= j ? V + (i0 + q) * ld : w;
        acc[q] = 0.0;
    }
#pragma unroll 2
    for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) {
        const double we = w[e];
#pragma unroll
        for (int q = 0; q < kBasisGroup; ++q) acc[q] += we * vp[q][e];
    }
    block_sums<kBasisGroup>(acc, red);
    if (threadIdx.x == 0)
#pragma unroll
        for (int q = 0; q < kBasisGroup; ++q)
            if (i0 + q < K) partial[(int64_t)(i0 + q) * n_items + item] = acc[q];
}

// partials of (V_i, w), i = 0..j, and (w, w) in slot j + 1; blockIdx.y picks
// the group of basis vectors
__global__ __launch_bounds__(kVecThreads) void k_mdot(const Item *__restrict__ items, int32_t n_items,
                                                      const int32_t *__restrict__ done, int j, int64_t ld,
                                                      const double *__restrict__ V, const double *__restrict__ w,
                                                      double *__restrict__ partial) {
    __shared__ double red[kBasisGroup * (kVecThreads / 64)];
    const Item it = items[blockIdx.x];
    if (done[it.sys]) return;                     // its partials are not read
    item_dots(it, blockIdx.x, n_items, (int)blockIdx.y * kBasisGroup, j, j + 2, ld, V, w, partial, red);
}

// Sums over one system's items of K slots of partials -> out[0..K) (LDS), one
// wavefront per slot, so that the slots' sums run side by side.  The caller
// waits (a barrier) before it reads them.
template <int THREADS>
__device__ inline void slot_sums(const double *__restrict__ partial, int32_t n_items, int K, int32_t i0, int32_t i1,
                                 double *out) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int i = wid; i < K; i += THREADS / 64) {
        const double *pi = partial + (int64_t)i * n_items;
        double t = 0.0;
#pragma unroll 4
        for (int32_t k = i0 + lane; k < i1; k += 64) t += pi[k];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
        if (lane == 0) out[i] = t;
    }
}

// First pass: h_i (per system) = sum of partials, into H(:, j) and coef, one
// wavefront per basis vector (one after the other by the whole workgroup:
// 7.9 us, now 3.2 us).  A system whose w keeps more than a tenth of its norm,
// ||w - sum h_i V_i||^2 = ||w||^2 - sum h_i^2 > 0.01 ||w||^2 ((w, w) in slot
// j + 1), skips the second (re-orthogonalising) pass: skip[s] = 1 (also for a
// finished system).
constexpr int kMdotFinThreads = 1024;
constexpr int kMaxRestart = 200;                  // cbs_setup refuses larger ones

__global__ __launch_bounds__(kMdotFinThreads) void k_mdot_fin(int j, int m, const int32_t *__restrict__ item_off,
                                                               int32_t n_items, const double *__restrict__ partial,
                                                               const int32_t *__restrict__ done, double *H,
                                                               double *coef, int32_t *skip) {
    __shared__ double sh[kMaxRestart + 2];
    const int s = blockIdx.x;
    if (done[s]) {
        if (threadIdx.x == 0) skip[s] = 1;
        return;
    }
    slot_sums<kMdotFinThreads>(partial, n_items, j + 2, item_off[s], item_off[s + 1], sh);
    __syncthreads();
    if ((int)threadIdx.x <= j) {
        const int i = threadIdx.x;
        H[(int64_t)s * (m + 1) * m + (int64_t)i * m + j] = sh[i];
        coef[(int64_t)s * (m + 1) + i] = sh[i];
    }
    if (threadIdx.x == 0) {
        double hh = 0.0;
        for (int i = 0; i <= j; ++i) hh += sh[i] * sh[i];
        skip[s] = (sh[j + 1] - hh > 0.01 * sh[j + 1]) ? 1 : 0;
    }
}

// base + sum of sgn c_i V_i at element e, i = 0..K-1 in order, kBasisGroup
// loads in flight
template <int SGN>
__device__ inline double basis_sum(double base, int K, const double *__restrict__ c, int64_t ld,
                                   const double *__restrict__ V, int64_t e) {
    double acc = base;
    int i = 0;
    for (; i + kBasisGroup <= K; i += kBasisGroup) {
        double v[kBasisGroup];
#pragma unroll
        for (int q = 0; q < kBasisGroup; ++q) v[q] = V[(i + q) * ld + e];
#pragma unroll
        for (int q = 0; q < kBasisGroup; ++q) acc += SGN * c[i + q] * v[q];
    }
    for (; i < K; ++i) acc += SGN * c[i] * V[i * ld + e];
    return acc;
}

// w -= sum_i c_i V_i over one item; returns this thread's part of the new (w, w)
__device__ inline double item_axpy(const Item &it, int j, int64_t ld, const double *__restrict__ V, const double *c,
                                   double *w) {
    double s0 = 0.0;
#pragma unroll 2
    for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) {
        const double we = basis_sum<-1>(w[e], j + 1, c, ld, V, e);
        w[e] = we;
        s0 += we * we;
    }
    return s0;
}

// End of the first pass: w -= sum_i coef_i V_i, and the partials of the new
// (w, w) in slot `slot`.  For a system that takes the second pass, also that
// pass's partials (V_i, w): a workgroup's item of w, just written by the
// threads that read it again, is all they need.
__global__ __launch_bounds__(kVecThreads) void k_maxpy(const Item *__restrict__ items, int32_t n_items,
                                                       const int32_t *__restrict__ done,
                                                       const int32_t *__restrict__ skip, int j, int m, int64_t ld,
                                                       const double *__restrict__ V, const double *__restrict__ coef,
                                                       double *w, double *__restrict__ partial, int slot) {
    __shared__ double red[kBasisGroup * (kVecThreads / 64)];
    const Item it = items[blockIdx.x];
    if (done[it.sys]) return;
    double s0 = block_sum(item_axpy(it, j, ld, V, coef + (int64_t)it.sys * (m + 1), w), red);
    if (threadIdx.x == 0) partial[(int64_t)slot * n_items + blockIdx.x] = s0;
    if (skip[it.sys]) return;
    for (int i0 = 0; i0 <= j; i0 += kBasisGroup) {
        item_dots(it, blockIdx.x, n_items, i0, j, j + 1, ld, V, w, partial, red);
        __syncthreads();                          // red is used again
    }
}

// The second pass, for the systems that take it: every workgroup sums the
// partials for its coefficients, the system's first one adds them to H(:, j).
// Most steps skip it, and a launch that does nothing costs 4 us: this is the
// only one (with products, sums and V_{j+1} in launches of their own a step had
// eight; 59,319 cells, 5x5, GMRES(30) of 86 steps: 10.93 -> 10.52 ms).
__global__ __launch_bounds__(kVecThreads) void k_maxpy_again(const Item *__restrict__ items, ItemRange range,
                                                             int32_t n_items,
                                                             const int32_t *__restrict__ skip, int j, int m,
                                                             int64_t ld, const double *__restrict__ V, double *H,
                                                             double *w, double *partial, int slot) {
    __shared__ double c[kMaxRestart + 1], red[kVecThreads / 64];
    const Item it = items[blockIdx.x];
    const int s = it.sys;
    if (skip[s]) return;
    const int32_t i0 = range.off[s];
    slot_sums<kVecThreads>(partial, n_items, j + 1, i0, range.folded ? i0 + 1 : range.off[s + 1], c);
    __syncthreads();
    if ((int32_t)blockIdx.x == i0)
        for (int i = threadIdx.x; i <= j; i += kVecThreads) H[(int64_t)s * (m + 1) * m + (int64_t)i * m + j] += c[i];
    const double s0 = block_sum(item_axpy(it, j, ld, V, c, w), red);
    if (threadIdx.x == 0) partial[(int64_t)slot * n_items + blockIdx.x] = s0;
}

// y = a / d over one item
__device__ inline void item_scale(const Item &it, double d, const double *__restrict__ a, double *__restrict__ y) {
    const double f = d > 0.0 ? 1.0 / d : 0.0;
    for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) y[e] = a[e] * f;
}

// V_0 = r / beta
__global__ __launch_bounds__(kVecThreads) void k_scale(const Item *__restrict__ items, const int32_t *__restrict__ done,
                                                       const double *__restrict__ nrm, const double *__restrict__ a,
                                                       double *__restrict__ y) {
    const Item it = items[blockIdx.x];
    if (!done[it.sys]) item_scale(it, nrm[it.sys], a, y);
}

// Restart start: beta = ||r||, g = (beta, 0, ...), converged check.
__global__ __launch_bounds__(kFinThreads) void k_gm_start(int32_t nsys, int m, const int32_t *__restrict__ item_off,
                                                           int32_t n_items, const double *__restrict__ partial,
                                                           double *scal, double *g, int32_t *done, int32_t *jlen,
                                                           double tol2, int first, const int32_t *flags,
                                                           const int32_t *iters, HostMirror hm) {
    const int s = blockIdx.x;
    __shared__ double sh[2 * kFinThreads / 64];
    double q[2];                                       // (r, r), (b, b)
    sum_items<2>(partial, n_items, {0, 1}, item_off[s], item_off[s + 1], sh, q);
    if (threadIdx.x != 0) return;
    const double rr = q[0], bbs = q[1];
    // the least-squares residual of the last cycle (first cycle: the initial
    // true residual) before the restart replaces it
    SC(S_RREC) = first ? rr : SC(S_RR);
    SC(S_RR) = rr;
    if (first) {
        const double bb = bbs;
        SC(S_BB) = bb;
        SC(S_RES0) = bb > 0.0 ? sqrt(rr / bb) : 0.0;
    }
    const double beta = sqrt(rr);
    SC(S_RHO) = beta;            // ||r|| of this cycle
    double *gs = g + (int64_t)s * (m + 1);
    for (int i = 0; i <= m; ++i) gs[i] = 0.0;
    gs[0] = beta;
    jlen[s] = 0;
    done[s] = (SC(S_BB) == 0.0 || rr <= tol2 * SC(S_BB)) ? 1 : 0;
    publish_state(hm, s, nsys, done, flags, iters);
    publish_scal(hm, s, nsys, scal);
}

// After the orthogonalisation of column j: H(j+1,j) = ||w|| (partials in slot
// `slot`), and in two kinds of workgroups side by side:
// the first nsys, one per system, apply the previous rotations, make rotation
// j, update g, and test |g(j+1)|.  The column and the rotations pass through
// LDS: the rotations are applied one after the other, which from memory cost a
// load each.
// The others, one per item, form V_{j+1} = w / ||w|| (a system that finishes in
// this step may leave its items undone: they are not read again; the sum, with
// its barrier, comes before any look at `done`, which the first workgroups set).
__global__ __launch_bounds__(kFinThreads) void k_gm_givens(int32_t nsys, int j, int m, const Item *__restrict__ items,
                                                            ItemRange range, int32_t n_items,
                                                            const double *__restrict__ partial, int slot, double *scal,
                                                            double *H, double *cs, double *sn, double *g, int32_t *done,
                                                            int32_t *jlen, int32_t *iters, double tol2,
                                                            const int32_t *flags, HostMirror hm,
                                                            const double *__restrict__ w, double *__restrict__ vnext) {
    __shared__ double sH[kMaxRestart + 1], sc[kMaxRestart + 1], ss[kMaxRestart + 1];
    __shared__ double sh[kFinThreads / 64];
    double ww[1];
    if ((int)blockIdx.x >= nsys) {
        const Item it = items[blockIdx.x - nsys];
        range_sums<1>(partial, n_items, {slot}, range, it.sys, sh, ww);
        if (!done[it.sys]) item_scale(it, sqrt(ww[0]), w, vnext);
        return;
    }
    const int s = blockIdx.x;
    if (done[s]) return;
    double *Hs = H + (int64_t)s * (m + 1) * m;
    double *c = cs + (int64_t)s * (m + 1), *sv = sn + (int64_t)s * (m + 1), *gs = g + (int64_t)s * (m + 1);
    for (int i = threadIdx.x; i <= j; i += kFinThreads) {
        sH[i] = Hs[i * m + j];
        sc[i] = i < j ? c[i] : 0.0;
        ss[i] = i < j ? sv[i] : 0.0;
    }
    range_sums<1>(partial, n_items, {slot}, range, s, sh, ww);
    __syncthreads();
    const double hn = sqrt(ww[0]);
    if (threadIdx.x == 0) {
        double a = sH[0];
        for (int i = 0; i < j; ++i) {
            const double b = sH[i + 1];
            sH[i] = sc[i] * a + ss[i] * b;
            a = -ss[i] * a + sc[i] * b;
        }
        const double den = sqrt(a * a + hn * hn);
        const double cj = den > 0.0 ? a / den : 1.0, sj = den > 0.0 ? hn / den : 0.0;
        c[j] = cj;
        sv[j] = sj;
        sH[j] = den;
        Hs[(j + 1) * m + j] = 0.0;
        const double gj = gs[j], gn = -sj * gj;
        gs[j + 1] = gn;
        gs[j] = cj * gj;
        jlen[s] = j + 1;
        iters[s] += 1;
        const double est = gn * gn;
        SC(S_RR) = est;
        if (est <= tol2 * SC(S_BB) || hn == 0.0) done[s] = 1;
        publish_state(hm, s, nsys, done, flags, iters);
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= j; i += kFinThreads) Hs[i * m + j] = sH[i];
}

// y = H^{-1} g on the jlen x jlen upper triangle, one wavefront per system:
// from the last column back, each y_i leaves every earlier row's right side.
// The triangle of up to kTriLds columns is staged in LDS first.
constexpr int kTriLds = 64;

__global__ __launch_bounds__(64) void k_gm_solve(int m, const double *__restrict__ H, const double *__restrict__ g,
                                                 const int32_t *__restrict__ jlen, double *__restrict__ y) {
    __shared__ double sR[kTriLds * kTriLds], sg[kMaxRestart + 1];
    const int s = blockIdx.x, t = threadIdx.x;
    const int j = jlen[s];
    const double *Hs = H + (int64_t)s * (m + 1) * m;
    const double *gs = g + (int64_t)s * (m + 1);
    double *ys = y + (int64_t)s * (m + 1);
    const bool lds = j <= kTriLds;
    if (lds)
        for (int e = t; e < j * j; e += 64) sR[e] = Hs[(e / j) * m + e % j];
    for (int i = t; i <= m; i += 64) {
        sg[i] = i < j ? gs[i] : 0.0;
        if (i >= j) ys[i] = 0.0;
    }
    __syncthreads();
    for (int i = j - 1; i >= 0; --i) {
        const double d = lds ? sR[i * j + i] : Hs[i * m + i];
        const double yi = d != 0.0 ? sg[i] / d : 0.0;
        if (t == 0) ys[i] = yi;
        for (int k = t; k < i; k += 64) sg[k] -= (lds ? sR[k * j + i] : Hs[k * m + i]) * yi;
        __syncthreads();
    }
}

// x += sum_i y_i Z_i (all systems; y = 0 beyond jlen)
__global__ __launch_bounds__(kVecThreads) void k_gm_update(const Item *__restrict__ items, int m, int jmax, int64_t ld,
                                                           const double *__restrict__ Z, const double *__restrict__ y,
                                                           const int32_t *__restrict__ jlen, double *__restrict__ x) {
    const Item it = items[blockIdx.x];
    const double *ys = y + (int64_t)it.sys * (m + 1);
    const int js = min(jmax, jlen[it.sys]);      // columns this system built in the cycle
#pragma unroll 2
    for (int64_t e = it.beg + threadIdx.x; e < it.end; e += kVecThreads) x[e] = basis_sum<1>(x[e], js, ys, ld, Z, e);
}

#undef SC

// ------------------------------------------------------------------ helpers
inline const int32_t *done_none(cbs_system *h) { return h->flags.get() + h->n_sys; }   // all-zero mask

void dots(cbs_system *h, int K, const double *a0, const double *b0, const double *a1 = nullptr,
          const double *b1 = nullptr, const double *a2 = nullptr, const double *b2 = nullptr,
          const int32_t *mask = nullptr) {
    hipLaunchKernelGGL(k_dots, dim3(h->n_items), dim3(kVecThreads), 0, h->stream, h->items.get(), h->n_items,
                       mask ? mask : h->done.get(), K, a0, b0, a1, b1, a2, b2, h->partial.get());
    LAUNCHCHK();
}

ItemRange item_range(const cbs_system *h) {
    return ItemRange{h->item_off.get(), h->fold_sums || h->n_items == h->n_sys};
}

// K slots of partials from slot0 on, ready for kernels whose workgroups all sum them
void fold(cbs_system *h, int slot0, int K) {
    if (!h->fold_sums) return;
    hipLaunchKernelGGL(k_fold_sums, dim3(h->n_sys, K), dim3(kFinThreads), 0, h->stream, h->item_off.get(), h->n_items,
                       slot0, h->partial.get());
    LAUNCHCHK();
}

int32_t *iters_ptr(cbs_system *h) { return h->done.get() + 2 * h->n_sys; }

HostMirror mirror(cbs_system *h) {
    return h->n_sys < kMirrorSystems ? HostMirror{h->h_state, h->h_scal} : HostMirror{nullptr, nullptr};
}

// after a kernel that was given mirror(h)
void publish(cbs_system *h, bool with_scal) {
    if (h->n_sys < kMirrorSystems) return;
    hipLaunchKernelGGL(k_publish, dim3(cdiv(h->n_sys, 256)), dim3(256), 0, h->stream, HostMirror{h->h_state, h->h_scal},
                       h->n_sys, h->done.get(), h->flags.get(), iters_ptr(h), with_scal ? h->scal.get() : nullptr);
    LAUNCHCHK();
}

void fin(cbs_system *h, int phase, double tol2, const int32_t *restart_mask = nullptr) {
    hipLaunchKernelGGL(k_fin, dim3(h->n_sys), dim3(kFinThreads), 0, h->stream, phase, h->n_sys, h->item_off.get(),
                       h->n_items, h->partial.get(), h->scal.get(), h->done.get(), h->flags.get(),
                       h->done.get() + 2 * h->n_sys, tol2, restart_mask, mirror(h));
    LAUNCHCHK();
    publish(h, phase == PH_TRUE);
}

// ------------------------------------------------------------------ V-cycle
template <typename T> T *vptr(DArr<char> &a) { return reinterpret_cast<T *>(a.get()); }

template <typename T>
const T *level_vals(Level &L, bool tr);
template <>
const double *level_vals<double>(Level &L, bool tr) { return tr ? L.sell.v64T.get() : L.sell.v64.get(); }
template <>
const float *level_vals<float>(Level &L, bool tr) { return tr ? L.sell.v32T.get() : L.sell.v32.get(); }

template <typename T>
const T *ilu_vals(Level &L, bool tr);
template <>
const double *ilu_vals<double>(Level &L, bool tr) { return tr ? L.iluS64T.get() : L.iluS64.get(); }
template <>
const float *ilu_vals<float>(Level &L, bool tr) { return tr ? L.iluS32T.get() : L.iluS32.get(); }

// One DILU or block ILU(0) smoothing step x <- x + M^{-1}(b - A x)
// (zero_guess: x <- M^{-1} b).  Both have M = (E + L) E^{-1} (E + U): DILU
// with A's own off-diagonal blocks, ILU(0) with those of its factor.
template <typename T>
void dilu_smooth(cbs_system *h, Level &L, bool tr, const T *b, T *x, bool zero_guess) {
    const T *val = level_vals<T>(L, tr);
    const T *fv = L.ilu ? ilu_vals<T>(L, tr) : nullptr;
    const double *Einv = tr ? L.EinvT.get() : L.Einv.get();
    T *y = vptr<T>(L.vt);
    const int ncol = (int)L.colour_off.size() - 1;
    const SellView S = L.sell.view(sizeof(T) == 4);
    auto cnt = [&](int c) { return L.colour_off[c + 1] - L.colour_off[c]; };
    // with two colours the kernels know every neighbour's colour without
    // reading it: the other one
    const int32_t *colour = ncol <= 2 ? nullptr : L.colour.get();
    for (int c = 0; c < ncol; ++c)
        launch_dilu_fwd<T>(h->n, S, val, fv, colour, c, L.sell.cpos[c], cnt(c), Einv, b, x, y, zero_guess,
                           c == ncol - 1, h->stream);
    // the last colour's backward step changes nothing; its forward launch
    // already made its update
    for (int c = ncol - 2; c >= 0; --c)
        launch_dilu_bwd<T>(h->n, S, fv ? fv : val, colour, c, L.sell.cpos[c], cnt(c), Einv, y, x, zero_guess,
                           h->stream);
}

// One symmetric block Gauss-Seidel step in place: the colour classes in
// order, then in reverse (the oracle's order: colour first, then row).  The
// last colour's second pass is left out: nothing it reads changed since its
// first, so it would recompute the same values.
template <typename T>
void sgs_smooth(cbs_system *h, Level &L, bool tr, const T *b, T *x) {
    const T *val = level_vals<T>(L, tr);
    const double *Dinv = tr ? L.DinvT.get() : L.Dinv.get();
    const int ncol = (int)L.colour_off.size() - 1;
    const SellView S = L.sell.view(sizeof(T) == 4);
    auto colour = [&](int c) {
        launch_gs_colour<T>(h->n, S, val, L.sell.cpos[c], L.colour_off[c + 1] - L.colour_off[c], Dinv, b, x,
                            h->stream);
    };
    for (int c = 0; c < ncol; ++c) colour(c);
    for (int c = ncol - 2; c >= 0; --c) colour(c);
}

// Levels whose colouring has two classes (hex meshes are bipartite).  Colour
// 0 has no earlier neighbours, so its DILU / ILU(0) pivot is its diagonal
// block, and with two colours the ILU(0) factor keeps A's off-diagonal
// blocks.  One DILU or ILU(0) step from x, y_0 = E_0^{-1} r_0, y_1 = E_1^{-1}
// (r_1 - A_10 y_0), z_0 = y_0 - E_0^{-1} A_01 y_1, is then the same as
//   x_0 = E_0^{-1} (b_0 - A_01 x_1);  x_1 += E_1^{-1} (b_1 - A_1. x);
//   x_0 = E_0^{-1} (b_0 - A_01 x_1)
// and a symmetric Gauss-Seidel step is the same with D for E and the
// replacement x_1 = D_1^{-1} (b_1 - A_10 x_0).  Both give the same update up
// to rounding order.  A step's first colour-0 update repeats the last one of
// the step before (x_1 has not changed since), so `steps` steps take one
// colour-0 launch more than colour-1 launches.  After them the residual of
// colour 0 is zero; rz, when given, gets those zeros.
template <typename T>
void smooth_two_colour(cbs_system *h, Level &L, bool tr, const T *b, T *x, int steps, bool zero_guess, T *rz) {
    if (steps <= 0) return;
    const T *val = level_vals<T>(L, tr);
    const double *P = L.dilu ? (tr ? L.EinvT.get() : L.Einv.get()) : (tr ? L.DinvT.get() : L.Dinv.get());
    const SellView S = L.sell.view(sizeof(T) == 4);
    const int32_t n0 = L.colour_off[1] - L.colour_off[0], n1 = L.colour_off[2] - L.colour_off[1];
    auto c0 = [&](int form, T *z) { launch_gs_colour<T>(h->n, S, val, L.sell.cpos[0], n0, P, b, x, h->stream, form, z); };
    auto c1 = [&](int form) { launch_gs_colour<T>(h->n, S, val, L.sell.cpos[1], n1, P, b, x, h->stream, form); };
    c0(zero_guess ? 2 : 0, nullptr);                 // from zero: every x_1 is still zero
    for (int s = 0; s < steps; ++s) {
        // DILU's colour-1 update is a correction of x_1, except from zero
        c1(L.dilu && !(zero_guess && s == 0) ? 1 : 0);
        c0(0, s == steps - 1 ? rz : nullptr);
    }
}

// the positions [p0, p1) of a colour-ordered copy as a copy of their own
// (p0 a whole number of slices)
SellView position_range(SellView S, int32_t p0, int32_t p1) {
    if (p0 & ((1 << S.lc) - 1)) cbs_throw(CBS_ERR_ARG, "colour range not slice-aligned");
    const int32_t s0 = p0 >> S.lc;
    S.N = p1 - p0;
    S.soff += s0;
    S.sw += s0;
    S.prow += p0;
    return S;
}

// x = V(b) with zero initial guess on level l; the result lands in x.  When
// rfine is given, b is not yet formed: it is the restriction of the finer
// level's residual rfine, which the first kernel of this level computes and
// stores into b (fused into the zero-guess sweep when there is one).  On
// level 0 of a mixed-precision cycle, b64 is the FP64 right side (rounded
// into b by the first kernel) and the result goes widened to x64 instead.
//
// zero = false (levels below the finest only, rfine null): x holds a start
// and b the level's right side, both left by an earlier cycle on this level,
// whose zero-guess sweep also left c = D^{-1} b behind.  This is the second
// run of a W-cycle's coarse correction.
//
// begun: the zero-guess sweep has been made (x of it in cycle_start, b and c =
// D^{-1} b as this level keeps them), fused into the launch that formed b.
template <typename T>
T *cycle_start(cbs_system *h, int l, T *x) {
    const int nu1 = std::max(0, h->opt.pre_sweeps), nu2 = std::max(0, h->opt.post_sweeps);
    const int switches = (nu1 >= 1 ? nu1 - 1 : 0) + nu2;
    return switches % 2 == 0 ? x : vptr<T>(h->lev[l].vt);
}

// a level that starts with a zero-guess block-Jacobi sweep
bool starts_with_sweep0(const cbs_system *h, int l) {
    const Level &L = h->lev[l];
    return l < (int)h->lev.size() - 1 && !(l > 0 && l == h->tail.level) && !L.dilu && !L.sgs && h->opt.pre_sweeps >= 1;
}

// FP32 sweeps run on the row-scaled values Dinv A (D^{-T} A^T in the transposed
// solve) against c = Dinv b, which the zero-guess sweep leaves behind
template <typename T>
bool scaled_sweeps(const Level &L, bool tr) { return sizeof(T) == sizeof(float) && (tr ? L.scaledT : L.scaled); }

template <typename T>
void vcycle(cbs_system *h, bool tr, int l, T *b, T *x, const T *rfine, const double *b64 = nullptr,
            double *x64 = nullptr, bool zero = true, bool begun = false) {
    hipStream_t st = h->stream;
    const cbs_options &o = h->opt;
    const int n = h->n;
    const int nlev = (int)h->lev.size();
    Level &L = h->lev[l];
    const int64_t m = (int64_t)L.N * n;
    const int nu1 = std::max(0, o.pre_sweeps), nu2 = std::max(0, o.post_sweeps);
    const double om = level_omega(o, l);
    constexpr bool fp32 = sizeof(T) == sizeof(float);
    const bool bj = l < nlev - 1 && !L.dilu && !L.sgs;
    const bool fuse_in = fp32 && b64 && bj && nu1 >= 1 && !begun;
    const bool fuse_out = fp32 && x64 && bj && nu2 >= 1;
    if (b64 && !fuse_in && !begun) launch_cast<double, T>(m, b64, b, st);
    auto finish = [&] {
        if (x64 && !fuse_out) launch_cast<T, double>(m, x, x64, st);
    };
    auto restrict_into_b = [&] {
        const Level &F = h->lev[l - 1];
        launch_restrict<T>(n, L.N, F.agg_ptr.get(), F.agg_mem.get(), rfine, b, st);
    };
    if (!zero && (rfine || b64 || l == 0 || l == nlev - 1 || l == h->tail.level))
        cbs_throw(CBS_ERR_ARG, "V-cycle from a start: not on this level");
    // the coarse correction: the next level's cycle, twice on the w_levels
    // finest levels (the second run from the first one's result), once where
    // the next level is the coarsest (solved exactly)
    auto coarse = [&](T *bc, T *xc, const T *r) {
        vcycle<T>(h, tr, l + 1, bc, xc, r);
        if (l < o.w_levels && l + 2 < nlev) vcycle<T>(h, tr, l + 1, bc, xc, nullptr, nullptr, nullptr, false);
    };
    if (rfine && l == h->tail.level) {                       // the rest of the cycle at once
        launch_tail<T>(h, tr, rfine, x);
        return;
    }
    if (l == nlev - 1) {
        if (rfine) restrict_into_b();
        launch_coarse_solve(h, tr, b, x, fp32);
        finish();
        return;
    }
    const T *val = level_vals<T>(L, tr);
    const double *Dinv = tr ? L.DinvT.get() : L.Dinv.get();
    T *tmp = vptr<T>(L.vt);
    T *r = vptr<T>(L.vr);
    Level &C = h->lev[l + 1];
    T *bc = vptr<T>(C.vb), *xc = vptr<T>(C.vx);
    if (L.dilu || L.sgs) {
        if (rfine) restrict_into_b();
        const bool two = L.colour_off.size() == 3 && L.sell.cpos.size() == 3;
        if (two && nu1 >= 1) {
            // colour 0's residual is zero after the steps: only colour 1's is formed
            smooth_two_colour<T>(h, L, tr, b, x, nu1, zero, r);
            launch_rows<T, T>(1, n, position_range(L.sell.view(fp32), L.sell.cpos[1], L.sell.cpos[2]), val, x, b, r,
                              nullptr, 0.0, st);
        } else {
            if (zero && (L.sgs || nu1 == 0)) launch_fill<T>(m, x, st);    // Gauss-Seidel starts from x = 0
            for (int s = 0; s < nu1; ++s) {
                if (L.dilu) dilu_smooth<T>(h, L, tr, b, x, zero && s == 0);
                else sgs_smooth<T>(h, L, tr, b, x);
            }
            launch_rows<T, T>(1, n, L.sell.view(fp32), val, x, b, r, nullptr, 0.0, st);
        }
        coarse(bc, xc, r);
        launch_prolong<T>(n, L.N, L.agg.get(), xc, x, x, st);
        if (two) {
            smooth_two_colour<T>(h, L, tr, b, x, nu2, false, nullptr);
        } else {
            for (int s = 0; s < nu2; ++s) {
                if (L.dilu) dilu_smooth<T>(h, L, tr, b, x, false);
                else sgs_smooth<T>(h, L, tr, b, x);
            }
        }
        finish();
        return;
    }
    // On large levels the extra aggregate-map gathers cost more than the
    // separate prolongation pass; on small ones the saved launch wins.
    const bool fuse_pro = nu2 > 0 && L.N < kSmallLevelRows;
    // From a start in x the cycle returns there after an even number of sweeps.
    // After an odd one the separate prolongation changes over too (FP32 4x4,
    // 213,888 rows: a copy of the start took 5.8 us); fused, the start is copied.
    const bool change_over = !zero && (nu1 + nu2) % 2 != 0 && !fuse_pro;
    T *cur = zero ? cycle_start<T>(h, l, x) : (nu1 + nu2) % 2 == 0 || change_over ? x : tmp;
    T *oth = (cur == x) ? tmp : x;
    if (!zero && cur != x) launch_cast<T, T>(m, x, cur, st);
    const bool scaled = scaled_sweeps<T>(L, tr);
    const T *sval = scaled ? reinterpret_cast<const T *>(tr ? L.sod.v32T.get() : L.sod.v32.get()) : nullptr;
    T *c = scaled ? vptr<T>(L.vc) : nullptr;
    // pagg/pe: sweep from x + P e (the prolongation fused into the sweep);
    // y64: write the result widened to FP64 there instead of into `to`
    auto sweep = [&](T *from, T *to, const int32_t *pagg, const T *pe, double *y64) {
        if (scaled)
            launch_rows<T, T>(4, n, L.sod.view(true), sval, from, c, to, nullptr, om, st, nullptr, pagg, pe,
                              y64);
        else
            launch_rows<T, T>(2, n, L.sell.view(fp32), val, from, b, to, Dinv, om, st, nullptr, pagg, pe, y64);
    };
    if (!zero) {
        for (int s = 0; s < nu1; ++s) {
            sweep(cur, oth, nullptr, nullptr, nullptr);
            std::swap(cur, oth);
        }
    } else if (nu1 >= 1) {
        if (begun) {
        } else if (fuse_in) {
            if constexpr (fp32)
                launch_cast_sweep0(n, L.N, b64, b, Dinv, om, cur, c, st);
        } else if (rfine) {
            launch_restrict_sweep0<T>(n, L.N, h->lev[l - 1].agg_ptr.get(), h->lev[l - 1].agg_mem.get(), rfine, b,
                                      Dinv, om, cur, c, st);
        } else {
            launch_rows<T, T>(3, n, L.sell.view(fp32), val, cur, b, cur, Dinv, om, st, c);
        }
        for (int s = 1; s < nu1; ++s) {
            sweep(cur, oth, nullptr, nullptr, nullptr);
            std::swap(cur, oth);
        }
    } else {
        if (rfine) restrict_into_b();
        if (scaled && nu2 > 0)   // c only; oth is scratch here
            launch_rows<T, T>(3, n, L.sell.view(true), val, oth, b, oth, Dinv, om, st, c);
        launch_fill<T>(m, cur, st);
    }
    launch_rows<T, T>(1, n, L.sell.view(fp32), val, cur, b, r, Dinv, om, st);
    coarse(bc, xc, r);
    if (!fuse_pro) {
        T *to = change_over ? oth : cur;
        launch_prolong<T>(n, L.N, L.agg.get(), xc, cur, to, st);
        if (change_over) std::swap(cur, oth);
    }
    for (int s = 0; s < nu2; ++s) {
        const bool first = s == 0 && fuse_pro, last = s == nu2 - 1 && fuse_out;
        sweep(cur, oth, first ? L.agg.get() : nullptr, first ? xc : nullptr, last ? x64 : nullptr);
        std::swap(cur, oth);
    }
    finish();
}

}  // namespace

// FP64 operator of the Krylov loop: level 0 in the internal numbering
void spmv64(cbs_system *h, const double *x, double *y, bool transposed) {
    Level &L0 = h->lev[0];
    const double *val = transposed ? L0.sell.v64T.get() : L0.sell.v64.get();
    launch_rows<double, double>(0, h->n, L0.sell.view(), val, x, nullptr, y, nullptr, 0.0, h->stream);
}

static void residual64(cbs_system *h, const double *b, const double *x, double *r, bool transposed) {
    Level &L0 = h->lev[0];
    const double *val = transposed ? L0.sell.v64T.get() : L0.sell.v64.get();
    launch_rows<double, double>(1, h->n, L0.sell.view(), val, x, b, r, nullptr, 0.0, h->stream);
}

void precond_apply(cbs_system *h, const double *r, double *z, bool tr, bool begun) {
    const int n = h->n;
    const int64_t m = (int64_t)h->N * n;
    hipStream_t st = h->stream;
    switch (h->opt.precond) {
        case CBS_PREC_NONE:
            launch_copy(m, r, z, st);
            return;
        case CBS_PREC_BJACOBI:
            launch_block_apply(n, h->N, tr ? h->lev[0].DinvT.get() : h->lev[0].Dinv.get(), r, z, st);
            return;
        case CBS_PREC_SGS: {
            Level &L0 = h->lev[0];
            const int steps = std::max(1, h->opt.pre_sweeps);
            if (L0.colour_off.size() == 3 && L0.sell.cpos.size() == 3) {
                smooth_two_colour<double>(h, L0, tr, r, z, steps, true, nullptr);
                return;
            }
            launch_fill<double>(m, z, st);
            for (int s = 0; s < steps; ++s) sgs_smooth<double>(h, L0, tr, r, z);
            return;
        }
        default:
            break;
    }
    if (h->opt.precision == CBS_PRECISION_MIXED) {
        Level &L0 = h->lev[0];
        float *b32 = vptr<float>(L0.vb), *x32 = vptr<float>(L0.vx);
        vcycle<float>(h, tr, 0, b32, x32, nullptr, r, z, true, begun);
    } else {
        vcycle<double>(h, tr, 0, const_cast<double *>(r), z, nullptr, nullptr, nullptr, true, begun);
    }
}

// The sweep with which precond_apply(., z) begins on T, for the kernel that
// forms its argument; see SweepOut.
template <typename T>
static SweepOut<T> sweep_out(cbs_system *h, double *z, bool tr) {
    Level &L0 = h->lev[0];
    constexpr bool fp32 = sizeof(T) == sizeof(float);
    T *x = fp32 ? vptr<T>(L0.vx) : reinterpret_cast<T *>(z);
    return SweepOut<T>{fp32 ? vptr<T>(L0.vb) : nullptr, cycle_start<T>(h, 0, x),
                       scaled_sweeps<T>(L0, tr) ? vptr<T>(L0.vc) : nullptr, tr ? L0.DinvT.get() : L0.Dinv.get(),
                       level_omega(h->opt, 0)};
}

// f(n, SweepOut) with the block size as a constant where the preconditioner's
// application to z begins with a zero-guess sweep; false where it does not, and
// for vectors of kSweepUpdateElems values on, where the update in steps with a
// barrier each falls behind by more than the launch.  960 rows: 2,440 -> 2,380
// us a step, 8,000: 3,280 -> 3,240, 55k: 8,590 -> 8,535, 219k (1.1M values):
// 11.97 -> 11.98 ms, 24 systems of 355k rows together (1.8M): 24.55 -> 24.18;
// 1M rows (4M values) would go from 59.53 to 59.79.
constexpr int64_t kSweepUpdateElems = 2 << 20;

template <typename F>
static bool with_sweep0(cbs_system *h, double *z, bool tr, F f) {
    if (h->opt.precond != CBS_PREC_AMG || !starts_with_sweep0(h, 0) || (int64_t)h->N * h->n >= kSweepUpdateElems)
        return false;
    auto run = [&](auto out) {
        switch (h->n) {
            case 1: f(std::integral_constant<int, 1>(), out); break;
            case 2: f(std::integral_constant<int, 2>(), out); break;
            case 3: f(std::integral_constant<int, 3>(), out); break;
            case 4: f(std::integral_constant<int, 4>(), out); break;
            case 5: f(std::integral_constant<int, 5>(), out); break;
        }
    };
    if (h->opt.precision == CBS_PRECISION_MIXED) run(sweep_out<float>(h, z, tr));
    else run(sweep_out<double>(h, z, tr));
    return true;
}

// ------------------------------------------------------------------ drivers
namespace {

struct HostView {
    std::vector<double> scal;
    std::vector<int32_t> state;     // done | flags | iters
};

// what the scalar kernels left in the pinned mirrors, copied: launches to come
// write there again (the scalars are those of the last true residual)
void read_state(cbs_system *h, HostView &hv, bool with_scal) {
    HIPCHK(hipStreamSynchronize(h->stream));
    hv.state.assign(h->h_state, h->h_state + 3 * h->n_sys);
    if (with_scal) hv.scal.assign(h->h_scal, h->h_scal + S_NSCAL * h->n_sys);
}

// true residual r = b - A x of every system -> S_RR
// (the recurrence's goes to S_RREC)
void true_residual(cbs_system *h, const double *b, const double *x, bool tr) {
    residual64(h, b, x, h->r.get(), tr);
    dots(h, 1, h->r.get(), h->r.get(), nullptr, nullptr, nullptr, nullptr, done_none(h));
    fin(h, PH_TRUE, 0.0);
}

DotSrc items_dots(cbs_system *h) { return DotSrc{h->partial.get(), h->n_items, 0}; }

// y = A x with (a, y) and, if c is given (c = y), (c, y) left as partials.  One
// system whose product takes at most kDotWgs workgroups forms them in the
// product itself: two launches less an iteration, while every workgroup of the
// next update sums that many partials.  960 rows: 2,510 -> 2,430 us a step,
// 55,000 rows (875 workgroups): 8,690 -> 8,580, 219k (3,423): 12,210 -> 12,090;
// 1M (15,625) would go from 59,320 to 59,490.  Batches share workgroups between
// systems and take the launch over their items.
DotSrc spmv_dots(cbs_system *h, const double *x, double *y, const double *a, const double *c, bool tr) {
    Level &L0 = h->lev[0];
    const SellView S = L0.sell.view();
    const int32_t wgs = rows_workgroups(S);
    if (h->n_sys > 1 || wgs > kDotWgs) {
        spmv64(h, x, y, tr);
        dots(h, c ? 2 : 1, a, y, c, y);
        return items_dots(h);
    }
    launch_rows<double, double>(5, h->n, S, tr ? L0.sell.v64T.get() : L0.sell.v64.get(), x, a, y, nullptr, 0.0,
                                h->stream, nullptr, nullptr, nullptr, h->dpart.get());
    return DotSrc{h->dpart.get(), wgs, wgs};
}

// One right-preconditioned BiCGStab iteration for every unfinished system,
// in two halves: the first ends with s = r - alpha v and the half-step test
// on ||s||, the second applies the preconditioner to s and finishes.  Only
// kernel launches on h->stream (no memset/memcpy, no host sync), so each
// part can be captured once and replayed as a graph.
void bicg_half1(cbs_system *h, bool tr) {
    hipStream_t st = h->stream;
    const int nsys = h->n_sys;
    double *r = h->r.get(), *rh = h->rh.get(), *p = h->p.get(), *v = h->v.get();
    double *ph = h->ph.get(), *sv = h->s.get();
    const Item *items = h->items.get();
    const dim3 G(h->n_items), B(kVecThreads);
    const bool begun = with_sweep0(h, ph, tr, [&](auto nc, auto z) {
        hipLaunchKernelGGL((k_p_update_sweep<nc, std::remove_pointer_t<decltype(z.x)>>), G, B, 0, st, items, nsys,
                           h->done.get(), h->scal.get(), h->flags.get(), r, p, v, z);
    });
    if (!begun)
        hipLaunchKernelGGL(k_p_update, G, B, 0, st, items, nsys, h->done.get(), h->scal.get(), h->flags.get(), r, p, v);
    precond_apply(h, p, ph, tr, begun);
    const DotSrc ds = spmv_dots(h, ph, v, rh, nullptr, tr);
    if (!ds.count) fold(h, 0, 1);
    const AlphaStep a{item_range(h), h->done.get(), h->scal.get(), h->flags.get(), iters_ptr(h), ds, mirror(h)};
    if (!with_sweep0(h, h->sh.get(), tr, [&](auto nc, auto z) {
            hipLaunchKernelGGL((k_s_update_sweep<nc, std::remove_pointer_t<decltype(z.x)>>), G, B, 0, st, items,
                               h->n_items, nsys, a, r, v, sv, h->partial.get(), z);
        }))
        hipLaunchKernelGGL(k_s_update, G, B, 0, st, items, h->n_items, nsys, a, r, v, sv, h->partial.get());
    LAUNCHCHK();
}

// x and r updates and the end-of-iteration scalars
void bicg_finish(cbs_system *h, double *x, const DotSrc &ds) {
    hipStream_t st = h->stream;
    const double tol2 = h->opt.tol * h->opt.tol;
    const dim3 G(h->n_items), B(kVecThreads);
    if (ds.count) fold(h, kSlotSS, 1);
    else fold(h, 0, kSlotSS + 1);
    hipLaunchKernelGGL(k_xr_update, G, B, 0, st, h->items.get(), item_range(h), h->n_items, h->n_sys, h->done.get(),
                       h->scal.get(), h->flags.get(), tol2, x, h->ph.get(), h->sh.get(), h->r.get(), h->s.get(),
                       h->t.get(), h->rh.get(), h->partial.get(), ds);
    fin(h, PH_END, tol2);
    LAUNCHCHK();
}

void bicg_half2(cbs_system *h, double *x, bool tr) {
    double *sv = h->s.get(), *sh = h->sh.get(), *t = h->t.get();
    // (the first half began it, and nothing has used the cycle's vectors since)
    precond_apply(h, sv, sh, tr, with_sweep0(h, sh, tr, [](auto, auto) {}));
    bicg_finish(h, x, spmv_dots(h, sh, t, sv, t, tr));
}

enum { PART_FULL = 0, PART_HALF1, PART_HALF2 };

// The whole iteration tests ||s|| with omega (the result of a half-step
// convergence is then exact, only nothing is skipped); the first half alone
// ends with the test so that the host can skip the second.
void bicg_part(cbs_system *h, double *x, bool tr, int part) {
    if (part != PART_HALF2) bicg_half1(h, tr);
    if (part == PART_HALF1) fin(h, PH_SNORM, h->opt.tol * h->opt.tol);
    if (part != PART_HALF1) bicg_half2(h, x, tr);
}

// Replay a captured part of the iteration (captured on first use).
void bicg_part_graph(cbs_system *h, double *xw, bool tr, int part) {
    hipGraphExec_t &ex = h->g_iter[part][tr ? 1 : 0];
    if (!ex) {
        if (!h->cap_stream) HIPCHK(hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking));
        hipStream_t saved = h->stream;
        h->stream = h->cap_stream;
        hipGraph_t g = nullptr;
        try {
            HIPCHK(hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeRelaxed));
            bicg_part(h, xw, tr, part);
            HIPCHK(hipStreamEndCapture(h->cap_stream, &g));
        } catch (...) {
            hipGraph_t junk = nullptr;
            (void)hipStreamEndCapture(h->cap_stream, &junk);
            if (junk) (void)hipGraphDestroy(junk);
            h->stream = saved;
            throw;
        }
        h->stream = saved;
        const hipError_t e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e != hipSuccess) { ex = nullptr; cbs_throw(CBS_ERR_HIP, "hipGraphInstantiate failed"); }
    }
    HIPCHK(hipGraphLaunch(ex, h->stream));
}

int bicgstab(cbs_system *h, const double *b, double *x, bool tr, std::vector<int> &status) {
    hipStream_t st = h->stream;
    const cbs_options &o = h->opt;
    const double tol2 = o.tol * o.tol;
    const int nsys = h->n_sys;
    double *r = h->r.get(), *rh = h->rh.get(), *p = h->p.get(), *v = h->v.get();
    double *ph = h->ph.get(), *sv = h->s.get(), *sh = h->sh.get(), *t = h->t.get();
    const Item *items = h->items.get();
    const dim3 G(h->n_items), B(kVecThreads);
    int32_t *rmask = h->flags.get() + 2 * nsys;     // restart mask scratch
    (void)sv; (void)sh; (void)t; (void)ph;

    residual64(h, b, x, r, tr);
    dots(h, 2, r, r, b, b, nullptr, nullptr, done_none(h));
    fin(h, PH_INIT, tol2);
    hipLaunchKernelGGL(k_zero_if_bzero, G, B, 0, st, items, nsys, h->scal.get(), x);
    HIPCHK(hipMemcpyAsync(rh, r, sizeof(double) * (size_t)h->N * h->n, hipMemcpyDeviceToDevice, st));
    HIPCHK(hipMemsetAsync(p, 0, sizeof(double) * (size_t)h->N * h->n, st));
    HIPCHK(hipMemsetAsync(v, 0, sizeof(double) * (size_t)h->N * h->n, st));

    std::vector<int> bd_restarts(nsys, 0), tr_restarts(nsys, 0);
    status.assign(nsys, CBS_NOT_CONVERGED);
    HostView hv;
    int it = 0;
    const int every = std::max(1, o.check_every);
    const bool graphs = x == h->xw.get();
    bool split = false;          // next iteration in two halves with a check between
    for (;;) {
        bool check = (it % every == 0) || it >= o.max_iter;
        if (check) {
            read_state(h, hv, false);
            const int32_t *dn = hv.state.data(), *fl = dn + nsys;
            bool all_done = true, any_bd = false;
            for (int s = 0; s < nsys; ++s) {
                if (status[s] == CBS_ERR_BREAKDOWN) continue;
                if (!dn[s]) all_done = false;
                if (fl[s] & 1) any_bd = true;
            }
            if (any_bd) {
                // restart broken systems once from the true residual
                std::vector<int32_t> mask(nsys, 0);
                for (int s = 0; s < nsys; ++s) {
                    if (status[s] == CBS_ERR_BREAKDOWN || !(fl[s] & 1)) continue;
                    if (bd_restarts[s]++ >= 1) { status[s] = CBS_ERR_BREAKDOWN; mask[s] = 0; }
                    else mask[s] = 1;
                }
                HIPCHK(hipMemcpyAsync(rmask, mask.data(), sizeof(int32_t) * nsys, hipMemcpyHostToDevice, st));
                residual64(h, b, x, h->w.get(), tr);
                hipLaunchKernelGGL(k_mask_copy, G, B, 0, st, items, rmask, 1, h->w.get(), r);
                hipLaunchKernelGGL(k_mask_copy, G, B, 0, st, items, rmask, 1, h->w.get(), rh);
                hipLaunchKernelGGL(k_mask_copy, G, B, 0, st, items, rmask, 1, nullptr, p);
                hipLaunchKernelGGL(k_mask_copy, G, B, 0, st, items, rmask, 1, nullptr, v);
                dots(h, 1, r, r, nullptr, nullptr, nullptr, nullptr, done_none(h));
                fin(h, PH_RESTART, tol2, rmask);
                // systems out of restarts stay frozen: mark them done
                for (int s = 0; s < nsys; ++s)
                    if (status[s] == CBS_ERR_BREAKDOWN) {
                        int32_t one = 1;
                        HIPCHK(hipMemcpyAsync(h->done.get() + s, &one, sizeof(int32_t), hipMemcpyHostToDevice, st));
                        HIPCHK(hipStreamSynchronize(st));
                        h->h_state[s] = 1;
                    }
                continue;
            }
            if (all_done) {
                // verify with the true residual; restart systems that fall short
                true_residual(h, b, x, tr);
                read_state(h, hv, true);
                std::vector<int32_t> mask(nsys, 0);
                bool any = false;
                for (int s = 0; s < nsys; ++s) {
                    if (status[s] == CBS_ERR_BREAKDOWN) continue;
                    const double bb = hv.scal[S_BB * nsys + s], rr = hv.scal[S_RR * nsys + s];
                    if (bb == 0.0 || rr <= tol2 * bb) status[s] = CBS_OK;
                    else if (it < o.max_iter && tr_restarts[s]++ < 50) { mask[s] = 1; any = true; }
                }
                if (!any) return it;             // S_RR holds the true residuals
                HIPCHK(hipMemcpyAsync(rmask, mask.data(), sizeof(int32_t) * nsys, hipMemcpyHostToDevice, st));
                hipLaunchKernelGGL(k_mask_copy, G, B, 0, st, items, rmask, 1, r, rh);
                hipLaunchKernelGGL(k_mask_copy, G, B, 0, st, items, rmask, 1, nullptr, p);
                hipLaunchKernelGGL(k_mask_copy, G, B, 0, st, items, rmask, 1, nullptr, v);
                dots(h, 1, r, r, nullptr, nullptr, nullptr, nullptr, done_none(h));
                fin(h, PH_RESTART, tol2, rmask);
                continue;
            }
        }
        if (it >= o.max_iter) break;
        if (check) {
            // Near convergence (every unfinished system flagged by the end of
            // the last iteration) run the iteration in halves: if every
            // unfinished system already meets the tolerance with s, the second
            // preconditioner application and product are skipped.
            const int32_t *dn = hv.state.data(), *fl = dn + nsys;
            split = true;
            for (int s = 0; s < nsys && split; ++s)
                if (!dn[s] && !(fl[s] & kFlagBreak) && !(fl[s] & kFlagNear)) split = false;
        }
        if (!split) {
            if (graphs) bicg_part_graph(h, x, tr, PART_FULL);
            else bicg_part(h, x, tr, PART_FULL);
        } else {
            if (graphs) bicg_part_graph(h, x, tr, PART_HALF1);
            else bicg_part(h, x, tr, PART_HALF1);
            read_state(h, hv, false);
            const int32_t *dn = hv.state.data(), *fl = dn + nsys;
            bool all_half = true;
            for (int s = 0; s < nsys && all_half; ++s)
                if (!dn[s] && !(fl[s] & kFlagBreak) && !(fl[s] & kFlagHalf)) all_half = false;
            if (all_half) bicg_finish(h, x, items_dots(h));        // (no second product: omega is not formed)
            else if (graphs) bicg_part_graph(h, x, tr, PART_HALF2);
            else bicg_part(h, x, tr, PART_HALF2);
        }
        ++it;
    }
    true_residual(h, b, x, tr);            // for the statistics
    return it;
}

// Flexible GMRES(m) (Z_j = M^{-1} V_j kept, x += Z y), or with flexible ==
// false right-preconditioned GMRES(m): only V is kept, the preconditioned
// vector is formed for the product and dropped, and each cycle ends with
// x += M^{-1} (V y) -- one more preconditioner application per cycle and m
// fewer stored vectors.
int fgmres(cbs_system *h, const double *b, double *x, bool tr, std::vector<int> &status) {
    hipStream_t st = h->stream;
    const cbs_options &o = h->opt;
    const bool flexible = o.solver == CBS_SOLVER_FGMRES;
    const double tol2 = o.tol * o.tol;
    const int nsys = h->n_sys;
    const int m = std::max(1, o.restart);
    const int64_t ld = (int64_t)h->N * h->n;
    double *r = h->r.get(), *w = h->w.get();
    double *V = h->V.get(), *Z = h->Z.get();
    const Item *items = h->items.get();
    const dim3 G(h->n_items), B(kVecThreads), GS(nsys), BS(kFinThreads);
    const int wslot = m + 1;                      // partials of (w, w) after the orthogonalisation
    double *coef = h->yv.get() + (int64_t)nsys * (m + 1);       // (m+1) per system
    status.assign(nsys, CBS_NOT_CONVERGED);
    HostView hv;
    int it = 0;
    bool first = true;
    const int every = std::max(1, o.check_every);
    int32_t *iters = iters_ptr(h);
    const HostMirror hm = mirror(h);
    HIPCHK(hipMemsetAsync(iters, 0, sizeof(int32_t) * nsys, st));
    for (;;) {
        residual64(h, b, x, r, tr);
        dots(h, 2, r, r, b, b, nullptr, nullptr, done_none(h));
        hipLaunchKernelGGL(k_gm_start, GS, BS, 0, st, nsys, m, h->item_off.get(), h->n_items, h->partial.get(),
                           h->scal.get(), h->gvec.get(), h->done.get(), h->flags.get() + 3 * nsys, tol2, first ? 1 : 0,
                           h->flags.get(), iters, hm);
        publish(h, true);
        if (first) hipLaunchKernelGGL(k_zero_if_bzero, G, B, 0, st, items, nsys, h->scal.get(), x);
        first = false;
        read_state(h, hv, false);
        bool all_done = true;
        for (int s = 0; s < nsys; ++s) {
            if (hv.state[s]) status[s] = CBS_OK; else all_done = false;
        }
        if (all_done || it >= o.max_iter) break;
        hipLaunchKernelGGL(k_scale, G, B, 0, st, items, h->done.get(), h->scal.get() + S_RHO * nsys, r, V);
        int j = 0;
        for (; j < m && it < o.max_iter; ++j) {
            double *vj = V + j * ld, *zj = flexible ? Z + j * ld : h->ph.get();
            precond_apply(h, vj, zj, tr);
            spmv64(h, zj, w, tr);
            // classical Gram-Schmidt; a second pass re-orthogonalises the
            // systems whose w lost more than 90% of its norm in the first
            int32_t *skip = h->flags.get() + 4 * nsys;
            hipLaunchKernelGGL(k_mdot, dim3(h->n_items, cdiv(j + 2, kBasisGroup)), B, 0, st, items, h->n_items,
                               h->done.get(), j, ld, V, w, h->partial.get());
            hipLaunchKernelGGL(k_mdot_fin, GS, dim3(kMdotFinThreads), 0, st, j, m, h->item_off.get(), h->n_items,
                               h->partial.get(), h->done.get(), h->H.get(), coef, skip);
            hipLaunchKernelGGL(k_maxpy, G, B, 0, st, items, h->n_items, h->done.get(), skip, j, m, ld, V, coef, w,
                               h->partial.get(), wslot);
            fold(h, 0, j + 1);
            hipLaunchKernelGGL(k_maxpy_again, G, B, 0, st, items, item_range(h), h->n_items, skip, j, m, ld, V,
                               h->H.get(), w, h->partial.get(), wslot);
            fold(h, wslot, 1);
            hipLaunchKernelGGL(k_gm_givens, dim3(nsys + h->n_items), BS, 0, st, nsys, j, m, items, item_range(h),
                               h->n_items, h->partial.get(), wslot, h->scal.get(), h->H.get(), h->cs.get(),
                               h->sn.get(), h->gvec.get(), h->done.get(), h->flags.get() + 3 * nsys, iters, tol2,
                               h->flags.get(), hm, w, V + (j + 1) * ld);
            LAUNCHCHK();
            publish(h, false);
            ++it;
            if ((it % every) == 0) {
                read_state(h, hv, false);
                bool ad = true;
                for (int s = 0; s < nsys; ++s) ad = ad && hv.state[s];
                if (ad) { ++j; break; }
            }
        }
        const int jmax = std::min(j, m);
        hipLaunchKernelGGL(k_gm_solve, GS, dim3(64), 0, st, m, h->H.get(), h->gvec.get(), h->flags.get() + 3 * nsys,
                           h->yv.get());
        if (flexible) {
            hipLaunchKernelGGL(k_gm_update, G, B, 0, st, items, m, jmax, ld, Z, h->yv.get(), h->flags.get() + 3 * nsys,
                               x);
        } else {
            double *u = h->sh.get(), *z = h->ph.get();
            launch_fill<double>(ld, u, st);
            hipLaunchKernelGGL(k_gm_update, G, B, 0, st, items, m, jmax, ld, V, h->yv.get(), h->flags.get() + 3 * nsys,
                               u);
            precond_apply(h, u, z, tr);
            hipLaunchKernelGGL(k_gm_add, G, B, 0, st, items, z, x);
        }
        LAUNCHCHK();
        // next cycle re-evaluates every system from its true residual
        HIPCHK(hipMemsetAsync(h->done.get(), 0, sizeof(int32_t) * nsys, st));
    }
    return it;                                   // S_RR holds the true residuals: the last cycle's start
}

}  // namespace

void invalidate_graphs(cbs_system *h) {
    for (auto &part : h->g_iter)
        for (auto &g : part)
            if (g) { (void)hipGraphExecDestroy(g); g = nullptr; }
}

void alloc_krylov(cbs_system *h) {
    // any reallocation below would leave the captured graphs pointing at freed buffers
    const void *before[5] = {h->r.get(), h->partial.get(), h->V.get(), h->yv.get(), h->dpart.get()};
    struct Check {
        cbs_system *h;
        const void *const *b;
        ~Check() {
            const void *after[5] = {h->r.get(), h->partial.get(), h->V.get(), h->yv.get(), h->dpart.get()};
            for (int i = 0; i < 5; ++i)
                if (after[i] != b[i]) { invalidate_graphs(h); break; }
        }
    } check{h, before};
    const int64_t m = (int64_t)h->N * h->n;
    const int nsys = h->n_sys;
    for (DArr<double> *a : {&h->r, &h->rh, &h->p, &h->v, &h->ph, &h->s, &h->sh, &h->t, &h->w}) a->ensure(m);
    if (h->opt.solver != CBS_SOLVER_BICGSTAB) {
        const int mr = std::max(1, h->opt.restart);
        h->V.ensure((size_t)(mr + 1) * m);
        if (h->opt.solver == CBS_SOLVER_FGMRES) h->Z.ensure((size_t)mr * m);
        h->H.ensure((size_t)nsys * (mr + 1) * mr);
        h->gvec.ensure((size_t)nsys * (mr + 1));
        h->cs.ensure((size_t)nsys * (mr + 1));
        h->sn.ensure((size_t)nsys * (mr + 1));
        h->yv.ensure((size_t)nsys * (mr + 1) * 2);
    }
    if (!h->h_scal) {
        // written by the scalar kernels, read after a synchronisation; one
        // allocation, so that both are there or neither
        const unsigned how = hipHostMallocMapped | hipHostMallocCoherent | hipHostMallocPortable;
        void *p = nullptr;
        HIPCHK(hipHostMalloc(&p, (sizeof(double) * S_NSCAL + sizeof(int32_t) * 3) * nsys, how));
        h->h_scal = static_cast<double *>(p);
        h->h_state = reinterpret_cast<int32_t *>(h->h_scal + (size_t)S_NSCAL * nsys);
    }
    const int K = std::max(kSlots, h->opt.solver != CBS_SOLVER_BICGSTAB ? h->opt.restart + 2 : 0);
    h->partial.ensure((size_t)K * h->n_items);
    if (h->opt.solver == CBS_SOLVER_BICGSTAB && nsys == 1) h->dpart.ensure(2 * kDotWgs);
}

int krylov_solve(cbs_system *h, const double *b, double *x, cbs_stats *stv, bool tr) {
    hipStream_t st = h->stream;
    const int nsys = h->n_sys;
    if (tr) amg_build_transposed(h);
    alloc_krylov(h);
    HIPCHK(hipMemsetAsync(h->flags.get(), 0, sizeof(int32_t) * 5 * nsys, st));
    HIPCHK(hipMemsetAsync(h->done.get(), 0, sizeof(int32_t) * 3 * nsys, st));
    std::fill(h->h_state, h->h_state + 3 * nsys, 0);             // (the stream was synchronised by the last read)
    HIPCHK(hipEventRecord(h->ev0, st));
    std::vector<int> status;
    // the solvers run on work copies in the internal numbering (the captured
    // iteration graph points at xw)
    const int64_t m = (int64_t)h->N * h->n;
    h->xw.ensure(m);
    h->bw.ensure(m);
    const double *bi = b;
    if (h->renumbered) {
        permute_vec(h, b, h->bw.get(), true);
        permute_vec(h, x, h->xw.get(), true);
        bi = h->bw.get();
    } else {
        launch_copy(m, x, h->xw.get(), st);
    }
    if (h->opt.solver != CBS_SOLVER_BICGSTAB) fgmres(h, bi, h->xw.get(), tr, status);
    else bicgstab(h, bi, h->xw.get(), tr, status);
    if (h->renumbered) permute_vec(h, h->xw.get(), x, false);
    else launch_copy(m, h->xw.get(), x, st);
    HIPCHK(hipEventRecord(h->ev1, st));
    // statistics: both solvers leave the true residuals of x in S_RR
    HostView hv;
    read_state(h, hv, true);
    float ms = 0.f;
    HIPCHK(hipEventElapsedTime(&ms, h->ev0, h->ev1));
    int worst = CBS_OK;
    const double tol2 = h->opt.tol * h->opt.tol;
    for (int s = 0; s < nsys; ++s) {
        const double bb = hv.scal[S_BB * nsys + s], rr = hv.scal[S_RR * nsys + s];
        int stt = status[s];
        if (stt != CBS_ERR_BREAKDOWN) stt = (bb == 0.0 || rr <= tol2 * bb) ? CBS_OK : CBS_NOT_CONVERGED;
        if (stt < 0) worst = std::min(worst, stt);
        else if (worst >= 0) worst = std::max(worst, stt);
        if (stv) {
            cbs_stats &S = stv[s];
            S.iterations = hv.state[2 * nsys + s];
            S.status = stt;
            S.levels = (int32_t)h->lev.size();
            S.precision_fallback = 0;
            S.rel_res_true = bb > 0.0 ? std::sqrt(rr / bb) : 0.0;
            S.rel_res_recursive = bb > 0.0 ? std::sqrt(std::max(hv.scal[S_RREC * nsys + s], 0.0) / bb) : 0.0;
            S.rel_res_initial = hv.scal[S_RES0 * nsys + s];
            S.t_convert_ms = h->t_convert_ms;
            S.t_setup_ms = h->t_setup_ms;
            S.t_solve_ms = ms;
            S.op_complexity = h->op_complexity;
        }
    }
    return worst;
}
