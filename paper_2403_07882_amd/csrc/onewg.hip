// onewg.hip -- steps of the AMG setup (Sec. 2.3) on small levels, each in one
// workgroup.
//
// On a level of up to kOneWgRows block rows a setup kernel has a few
// microseconds of work at most, but every step of the matching, the member
// lists, the renumbering and the sliced patterns was a kernel of its own: some
// 90 launches per level, 0.4 ms, whatever its size.  Here one workgroup of 1024
// threads runs a whole step, its arrays in LDS and barriers where the launches
// were.  Every choice and every order is that of the kernels for large levels,
// so the hierarchy is the same.  MI355X, with the Galerkin kernel's one-pass
// ordering: setup of the 960-cell 4x4 system (4 levels) 1.46 -> 0.81 ms, of the
// 55,965-cell one (7 levels) 3.17 -> 2.28 ms.  The line lies at kOneWgRows
// because that many rows (two per thread) match in at most 58 us, about what
// the separate launches take; beyond it one CU's loads would set the time.
#include "cbs_internal.h"

namespace {

constexpr int kOneThreads = 1024;
constexpr int kOneCache = 8192;            // graph entries kept in LDS (10 bytes each)

// exclusive scan of v[0 .. n), n <= 2 * kOneThreads, in place in LDS; returns
// the total in every thread
__device__ inline int32_t scan_lds(int32_t *v, int32_t n) {
    __shared__ int32_t wsum[kOneThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int32_t a = 2 * t < n ? v[2 * t] : 0, b = 2 * t + 1 < n ? v[2 * t + 1] : 0;
    int32_t inc = a + b;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t u = __shfl_up(inc, o, 64);
        if (lane >= o) inc += u;
    }
    if (lane == 63) wsum[wid] = inc;
    __syncthreads();
    int32_t off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kOneThreads / 64; ++w) {
        off += w < wid ? wsum[w] : 0;
        tot += wsum[w];
    }
    const int32_t ex = off + inc - (a + b);
    if (2 * t < n) v[2 * t] = ex;
    if (2 * t + 1 < n) v[2 * t + 1] = ex + a;
    __syncthreads();                       // also frees wsum for the next scan
    return tot;
}

// One pass of handshake matching: the rounds of k_match_pick and
// k_match_confirm, then k_match_rep and the numbering of the aggregates, and
// (rs_c given) each aggregate's system.
__global__ __launch_bounds__(kOneThreads) void k_match_one(int32_t N, int rounds, const int32_t *__restrict__ rp,
                                                           const int32_t *__restrict__ col,
                                                           const double *__restrict__ w,
                                                           const int32_t *__restrict__ row_sys,
                                                           const int32_t *__restrict__ sys_frozen,
                                                           int32_t *__restrict__ agg, int32_t *__restrict__ nc,
                                                           int32_t *__restrict__ rs_c) {
    __shared__ int32_t partner[kOneWgRows], cand[kOneWgRows];
    extern __shared__ double cache_w[];                       // kOneCache weights, then columns
    uint16_t *cache_c = reinterpret_cast<uint16_t *>(cache_w + kOneCache);
    constexpr int R = kOneWgRows / kOneThreads;
    const int t = threadIdx.x;
    const int32_t nnz = rp[N];
    const bool cached = nnz <= kOneCache;
    if (cached)
        for (int32_t k = t; k < nnz; k += kOneThreads) {
            cache_w[k] = w[k];
            cache_c[k] = (uint16_t)col[k];
        }
    int32_t r0[R], r1[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int32_t i = t + q * kOneThreads;
        r0[q] = i < N ? rp[i] : 0;
        r1[q] = i < N ? rp[i + 1] : 0;
        if (i < N) partner[i] = sys_frozen[row_sys[i]] ? -2 : -1;
    }
    __syncthreads();
    // the strongest neighbour of row i that is still free (FREE) or matched:
    // the largest weight, of equal ones the smallest column
    auto best_of = [&](int32_t i, int32_t k0, int32_t k1, bool free_ones) {
        int32_t best = -1;
        double bw = 0.0;
        auto look = [&](int32_t j, double wk) {
            const bool ok = free_ones ? partner[j] == -1 : partner[j] >= 0;
            if (j != i && ok && wk > 0.0 && (wk > bw || (wk == bw && j < best))) { bw = wk; best = j; }
        };
        if (cached) {
            for (int32_t k = k0; k < k1; ++k) look(cache_c[k], cache_w[k]);
        } else {
            constexpr int U = 8;
            for (int32_t k = k0; k < k1; k += U) {
                int32_t j[U];
                double wk[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    j[u] = k + u < k1 ? col[k + u] : i;
                    wk[u] = k + u < k1 ? w[k + u] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) look(j[u], wk[u]);
            }
        }
        return best;
    };
    for (int round = 0; round < rounds; ++round) {
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int32_t i = t + q * kOneThreads;
            if (i < N) cand[i] = partner[i] == -1 ? best_of(i, r0[q], r1[q], true) : -1;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int32_t i = t + q * kOneThreads;
            if (i < N) {
                const int32_t j = cand[i];
                if (j >= 0 && cand[j] == i) partner[i] = j;
            }
        }
        __syncthreads();
    }
    int32_t rep[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int32_t i = t + q * kOneThreads;
        rep[q] = i;
        if (i >= N) continue;
        const int32_t p = partner[i];
        if (p >= 0) {
            rep[q] = min(i, p);
        } else if (p == -1) {              // unmatched: join the strongest matched neighbour's pair
            const int32_t b = best_of(i, r0[q], r1[q], false);
            if (b >= 0) rep[q] = min(b, partner[b]);
        }
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int32_t i = t + q * kOneThreads;
        if (i < N) cand[i] = rep[q] == i ? 1 : 0;
    }
    __syncthreads();
    const int32_t total = scan_lds(cand, N);
    if (t == 0) *nc = total;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int32_t i = t + q * kOneThreads;
        if (i >= N) continue;
        const int32_t a = cand[rep[q]];
        agg[i] = a;
        if (rs_c) rs_c[a] = row_sys[i];    // every member writes the same value
    }
}

// Member lists (ascending) of a map of N rows, first composed with a2 when
// given (agg = a2[agg]); past the last aggregate every aptr entry holds N.
// *maxc: the largest sum of row lengths (of the graph rp) over an aggregate.
__global__ __launch_bounds__(kOneThreads) void k_members_one(int32_t N, int32_t *__restrict__ agg,
                                                             const int32_t *__restrict__ a2,
                                                             const int32_t *__restrict__ rp,
                                                             int32_t *__restrict__ aptr, int32_t *__restrict__ amem,
                                                             int32_t *__restrict__ maxc) {
    __shared__ int32_t cnt[kOneWgRows], len[kOneWgRows], fill[kOneWgRows], mem[kOneWgRows], ag[kOneWgRows], mx;
    const int t = threadIdx.x;
    if (t == 0) mx = 0;
    for (int32_t i = t; i < N; i += kOneThreads) {
        int32_t a = agg[i];
        if (a2) {
            a = a2[a];
            agg[i] = a;
        }
        ag[i] = a;
        cnt[i] = len[i] = 0;
    }
    __syncthreads();
    for (int32_t i = t; i < N; i += kOneThreads) {
        atomicAdd(&cnt[ag[i]], 1);
        atomicAdd(&len[ag[i]], rp[i + 1] - rp[i]);
    }
    __syncthreads();
    int32_t m = 0;
    for (int32_t i = t; i < N; i += kOneThreads) m = max(m, len[i]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
    if ((t & 63) == 0) atomicMax(&mx, m);
    scan_lds(cnt, N);
    for (int32_t i = t; i < N; i += kOneThreads) {
        fill[i] = cnt[i];
        aptr[i] = cnt[i];
    }
    if (t == 0) {
        aptr[N] = N;
        *maxc = mx;
    }
    __syncthreads();
    for (int32_t i = t; i < N; i += kOneThreads) mem[atomicAdd(&fill[ag[i]], 1)] = i;
    __syncthreads();
    for (int32_t I = t; I < N; I += kOneThreads) {
        const int32_t b = cnt[I], e = I + 1 < N ? cnt[I + 1] : N;
        for (int32_t a = b + 1; a < e; ++a) {
            const int32_t v = mem[a];
            int32_t q = a - 1;
            while (q >= b && mem[q] > v) { mem[q + 1] = mem[q]; --q; }
            mem[q + 1] = v;
        }
    }
    __syncthreads();
    for (int32_t i = t; i < N; i += kOneThreads) amem[i] = mem[i];
}

// Internal numbering of a level from that of the next coarser one (pos_c):
// start of each aggregate's rows (new_aptr), the rows' positions, and the
// level's arrays at their new positions (see k_pos_assign).
__global__ __launch_bounds__(kOneThreads) void k_positions_one(int32_t N, int32_t nc, const int32_t *__restrict__ aptr,
                                                               const int32_t *__restrict__ amem,
                                                               const int32_t *__restrict__ pos_c,
                                                               const int32_t *__restrict__ rp,
                                                               const int32_t *__restrict__ row_sys,
                                                               int32_t *__restrict__ new_aptr, PosArrays out) {
    __shared__ int32_t start[kOneWgRows], len[kOneWgRows];
    const int t = threadIdx.x;
    for (int32_t I = t; I < nc; I += kOneThreads) start[pos_c[I]] = aptr[I + 1] - aptr[I];
    __syncthreads();
    const int32_t rows = scan_lds(start, nc);
    for (int32_t I = t; I < nc; I += kOneThreads) new_aptr[I] = start[I];
    if (t == 0) new_aptr[nc] = rows;
    for (int32_t I = t; I < nc; I += kOneThreads) {
        const int32_t pc = pos_c[I];
        int32_t p = start[pc];
        for (int32_t q = aptr[I]; q < aptr[I + 1]; ++q, ++p) {
            const int32_t i = amem[q];
            out.pos[i] = p;
            out.ip[p] = i;
            out.agg[p] = pc;
            out.mem[p] = p;
            out.row_sys[p] = row_sys[i];
            len[p] = rp[i + 1] - rp[i];
        }
    }
    __syncthreads();
    const int32_t nnz = scan_lds(len, N);
    for (int32_t i = t; i < N; i += kOneThreads) out.rp[i] = len[i];
    if (t == 0) out.rp[N] = nnz;
}

// Slice widths and offsets of several sliced patterns, a workgroup each.
__global__ __launch_bounds__(kOneThreads) void k_sell_widths_one(SellJobs jobs) {
    __shared__ int32_t off[kOneWgRows];
    const SellJob j = jobs.j[blockIdx.x];
    const int t = threadIdx.x, C = 1 << j.lc;
    const int32_t ns = (j.N + C - 1) >> j.lc;          // <= N <= kOneWgRows
    for (int32_t p = t; p < ((ns << j.lc) + 63) / 64 * 64; p += kOneThreads) {
        int32_t len = 0;
        if (p < j.N) {
            len = j.rp[p + 1] - j.rp[p];
            if (j.offdiag)
                for (int32_t k = j.rp[p]; k < j.rp[p + 1]; ++k) len -= j.col[k] == p ? 1 : 0;
        }
        for (int o = C >> 1; o > 0; o >>= 1) len = max(len, __shfl_xor(len, o, 64));
        const int32_t sl = p >> j.lc;
        if ((p & (C - 1)) == 0 && sl < ns) {
            j.sw[sl] = len;
            off[sl] = len * C;
        }
    }
    __syncthreads();
    const int32_t tot = scan_lds(off, ns);
    for (int32_t sl = t; sl < ns; sl += kOneThreads) j.soff[sl] = off[sl];
    if (t == 0) j.soff[ns] = tot;
}

}  // namespace

void one_wg_match(int32_t N, int rounds, const int32_t *rp, const int32_t *col, const double *w,
                  const int32_t *row_sys, const int32_t *sys_frozen, int32_t *agg, int32_t *nc, int32_t *rs_c,
                  hipStream_t st) {
    constexpr size_t lds = kOneCache * (sizeof(double) + sizeof(uint16_t));
    HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_match_one), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds));
    hipLaunchKernelGGL(k_match_one, dim3(1), dim3(kOneThreads), lds, st, N, rounds, rp, col, w, row_sys, sys_frozen,
                       agg, nc, rs_c);
    LAUNCHCHK();
}

void one_wg_members(int32_t N, int32_t *agg, const int32_t *a2, const int32_t *rp, int32_t *aptr, int32_t *amem,
                    int32_t *maxc, hipStream_t st) {
    hipLaunchKernelGGL(k_members_one, dim3(1), dim3(kOneThreads), 0, st, N, agg, a2, rp, aptr, amem, maxc);
    LAUNCHCHK();
}

void one_wg_positions(int32_t N, int32_t nc, const int32_t *aptr, const int32_t *amem, const int32_t *pos_c,
                      const int32_t *rp, const int32_t *row_sys, int32_t *new_aptr, const PosArrays &out,
                      hipStream_t st) {
    hipLaunchKernelGGL(k_positions_one, dim3(1), dim3(kOneThreads), 0, st, N, nc, aptr, amem, pos_c, rp, row_sys,
                       new_aptr, out);
    LAUNCHCHK();
}

void one_wg_sell_widths(const SellJobs &jobs, int count, hipStream_t st) {
    if (count > 0) hipLaunchKernelGGL(k_sell_widths_one, dim3(count), dim3(kOneThreads), 0, st, jobs);
    LAUNCHCHK();
}
