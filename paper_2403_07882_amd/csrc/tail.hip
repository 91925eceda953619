// tail.hip -- the coarse end of the AMG V-cycle (Sec. 2.2: the
// aggregation-AMG preconditioner) as one dense operator per system.
//
// Below a few hundred block rows a level's kernels are too small to fill the
// chip, and every step of the cycle there (restriction, each smoothing sweep,
// the residual, the prolongation, the coarsest solve) waits on launches and
// chains of dependent loads: about 4.5 us per launch inside a captured graph,
// and 27-45 us for all of it run by one workgroup with its vectors in LDS.
// From the first such level down to the coarsest and back the cycle is a
// fixed linear map of that level's right side, though, and the map changes
// only with the matrix.  cbs_setup therefore forms it once per system by
// running the cycle on the columns of the identity, in FP64 whatever the
// precision of the hierarchy (k_tail_operator), and a V-cycle applies it with
// one launch (k_tail_apply: the restriction and a dense product).  The result
// is the cycle's up to rounding; in mixed precision it is closer to the exact
// cycle than FP32 sweeps are.
//
// MI355X, FP32 hierarchy of the 41x39x35-cell 4x4 system (tail of 107, 27 and
// 6 rows): one workgroup 31.7 us per cycle, the operator 5.9 us, formed in
// 67 us per setup; FP64, 960 cells (241, 62 and 16 rows): 34.9 ->
// 6.6 us, formed in 71 us.
#include "cbs_internal.h"

#include <algorithm>
#include <cstring>

namespace {

constexpr int kTailThreads = 1024;         // threads of the workgroups that form the operator
constexpr int kTailRowsPerWg = 16;         // scalar rows per workgroup of the product: one 128-byte
                                           // line of a column of the operator
constexpr int kTailApplyThreads = 512;
constexpr int64_t kTailLdsReserve = 1024;
// A tail of the coarsest level alone saves one launch of two, and only up to this
// many workgroups is that more than its operators cost.  5x5, product against
// restriction and dense solve, and the forming: 64 systems of 20 unknowns 4.0,
// 6.0 and 10 us, 128 systems 4.0, 6.1 and 16 us (256 workgroups); 256 systems of
// 35 unknowns 7.1, 6.9 and 47 us, 512 of 20 6.9, 6.6 and 50 us, 2,048 of 20 36,
// 13 and 353 us.
constexpr int64_t kTailCoarseBlocks = 256;

// one level of the tail
struct TailLvl {
    const double *val, *Dinv;              // sliced FP64 values, inverses of the diagonal blocks
    const int32_t *soff, *sw, *scol;       // sliced pattern
    const int32_t *aptr, *amem, *agg;      // rows of the finer level per row here; row of the coarser level
    int32_t lc;
};

struct TailArgs {
    TailLvl lv[kTailMax];                  // smoothed levels, coarsest last (lv[nl])
    const int32_t *roff;                   // first row of system s on tail level k: roff[k * (nsys + 1) + s]
    const double *cinv;                    // coarsest: per-system dense inverses
    const int64_t *coff;
    const int32_t *cm;
    const int64_t *opoff;                  // first value of each system's operator
    const int32_t *wgoff;                  // first workgroup of each system
    double *op;
    double omega;
    int32_t nl, nu1, nu2, nsys;
};
static_assert(sizeof(TailArgs) <= 4096, "V-cycle tail arguments exceed the kernel-argument limit");

// leading dimension of an operator of order m (its columns start on 128-byte lines)
__host__ __device__ inline int64_t tail_ld(int64_t m) { return (m + kTailRowsPerWg - 1) / kTailRowsPerWg * kTailRowsPerWg; }

// row r of one block: n contiguous values (16-byte loads for n = 4)
template <int n>
__device__ inline void tail_load_row(const double *__restrict__ p, double (&v)[n]) {
    if constexpr (n == 4) {
        typedef double d2 __attribute__((ext_vector_type(2)));
        const d2 a = *reinterpret_cast<const d2 *>(p), b = *(reinterpret_cast<const d2 *>(p) + 1);
        v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
    } else {
#pragma unroll
        for (int c = 0; c < n; ++c) v[c] = p[c];
    }
}

// Doubles that one block row of a vector takes in LDS.  The residual gathers
// rows of x, the correction reads rows of r, in 16-byte pieces; at a distance of a multiple of 32 bytes the
// pieces of a wavefront's 16 rows fall on few of the banks (n = 4, NC = 4: on
// one eighth), at an odd multiple of 16 bytes on all of them: 960 cells 4x4 108
// -> 71 us, 24 systems 5x5 328 -> 282 us.
__host__ __device__ constexpr int tail_row(int n, int NC) {
    return n * NC >= 8 && n * NC % 4 == 0 ? n * NC + 2 : n * NC;
}

// one system's rows of a level, and where its vectors (doubles, NC columns side
// by side) and staged index lists (integers) start in LDS
struct TailRows {
    int32_t row0, N, sl0;                  // first row, rows, first slice
    int32_t b, x, r;
    int32_t soff, sw, aptr, amem, agg;
};

// r = b - A x over one system's rows of a level.  sp adjacent lanes share a
// scalar row and take its blocks kk, kk + sp, ... (four loaded before they
// are summed); their partial sums meet by shuffles.
template <int n, int NC>
__device__ __forceinline__ void tail_residual(const TailLvl &L, const TailRows &S, double *vs, const int32_t *is) {
    constexpr int nn = n * n, U = 4;
    const double *x = vs + S.x, *b = vs + S.b;
    double *r = vs + S.r;
    const int32_t *soff = is + S.soff, *sw = is + S.sw;
    int sp = 1;
    while (sp < 16 && S.N * n * sp * 2 <= kTailThreads) sp *= 2;
    const int lane_row = threadIdx.x / sp, kk = threadIdx.x & (sp - 1), R = kTailThreads / sp;
    const int32_t m = S.N * n;
    for (int32_t o0 = 0; o0 < m; o0 += R) {
        const int32_t o = o0 + lane_row;
        double acc[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = 0.0;
        const int32_t i = o / n, rr = o - i * n, gi = S.row0 + i;
        if (o < m) {
            const int32_t sl = gi >> L.lc, base = soff[sl - S.sl0] + (gi - (sl << L.lc)), w = sw[sl - S.sl0];
            for (int32_t k = kk; k < w; k += sp * U) {
                int32_t j[U];
                double bv[U][n];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t kq = k + u * sp;
                    const int64_t e = base + ((int64_t)(kq < w ? kq : kk) << L.lc);
                    j[u] = L.scol[e];
                    if (kq >= w) j[u] = -1;
                    tail_load_row<n>(L.val + e * nn + rr * n, bv[u]);
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (j[u] >= 0) {
                        const double *xj = x + (j[u] - S.row0) * tail_row(n, NC);
#pragma unroll
                        for (int q = 0; q < n; ++q)
#pragma unroll
                            for (int c = 0; c < NC; ++c) acc[c] += bv[u][q] * xj[q * NC + c];
                    }
            }
        }
        for (int s = sp >> 1; s > 0; s >>= 1)
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[c] += __shfl_xor(acc[c], s, 64);
        if (o < m && kk == 0)
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int32_t e = i * tail_row(n, NC) + rr * NC + c;
                r[e] = b[e] - acc[c];
            }
    }
    __syncthreads();
}

// x += omega Dinv r, or from a zero guess (ZERO) x = omega Dinv b
template <int n, int NC, bool ZERO>
__device__ __forceinline__ void tail_correct(const TailLvl &L, const TailRows &S, double *vs, double omega) {
    const double *v = vs + (ZERO ? S.b : S.r);
    double *x = vs + S.x;
    for (int32_t o = threadIdx.x; o < S.N * n; o += kTailThreads) {
        const int32_t i = o / n, rr = o - i * n;
        double d[n];
        tail_load_row<n>(L.Dinv + ((int64_t)(S.row0 + i) * n + rr) * n, d);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            double z = 0.0;
#pragma unroll
            for (int q = 0; q < n; ++q) z += d[q] * v[i * tail_row(n, NC) + q * NC + c];
            double &xo = x[i * tail_row(n, NC) + rr * NC + c];
            xo = (ZERO ? 0.0 : xo) + omega * z;
        }
    }
    __syncthreads();
}

// Columns q0 .. q0 + NC of one system's operator: the cycle of the tail on
// unit right sides.  The level vectors and index lists of the system are in
// LDS; matrix values and columns are read from L2, each block row once for
// the NC columns.  Bound by those reads, by the gathers from LDS (see tail_row)
// and by the barriers between steps.
template <int n, int NC>
__global__ __launch_bounds__(kTailThreads) void k_tail_operator(const TailArgs a) {
    extern __shared__ __align__(16) char smem[];
    __shared__ TailRows sS[kTailMax];
    double *vs = reinterpret_cast<double *>(smem);
    const int nl = a.nl, t = threadIdx.x;
    // the workgroup's system (the last whose first workgroup is not past it) and columns
    int s = 0;
    for (int hi = a.nsys - 1; s < hi;) {
        const int mid = (s + hi + 1) >> 1;
        if (a.wgoff[mid] <= (int32_t)blockIdx.x) s = mid;
        else hi = mid - 1;
    }
    const int32_t q0 = ((int32_t)blockIdx.x - a.wgoff[s]) * NC;
    int32_t nv = 0;                                  // doubles of the vectors
    for (int k = 0; k <= nl; ++k) {
        const int32_t *ro = a.roff + k * (a.nsys + 1) + s;
        nv += (k < nl ? 3 : 2) * (ro[1] - ro[0]) * tail_row(n, NC);
    }
    int32_t *is = reinterpret_cast<int32_t *>(vs + nv);
    if (t == 0) {
        int32_t v = 0, p = 0;
        for (int k = 0; k <= nl; ++k) {
            const int32_t *ro = a.roff + k * (a.nsys + 1) + s;
            TailRows S{};
            S.row0 = ro[0];
            S.N = ro[1] - ro[0];
            S.sl0 = S.row0 >> a.lv[k].lc;
            S.b = v; v += S.N * tail_row(n, NC);
            S.x = v; v += S.N * tail_row(n, NC);
            S.r = v; v += k < nl ? S.N * tail_row(n, NC) : 0;
            if (k < nl) {
                const int32_t ns = ((S.row0 + S.N - 1) >> a.lv[k].lc) - S.sl0 + 1;
                S.soff = p; p += ns;
                S.sw = p; p += ns;
                S.agg = p; p += S.N;
            }
            if (k > 0) {
                S.aptr = p; p += S.N + 1;
                S.amem = p; p += sS[k - 1].N;
            }
            sS[k] = S;
        }
    }
    __syncthreads();
    for (int k = 0; k <= nl; ++k) {
        const TailRows S = sS[k];
        const TailLvl &L = a.lv[k];
        if (k < nl) {
            const int32_t ns = ((S.row0 + S.N - 1) >> L.lc) - S.sl0 + 1, c0 = sS[k + 1].row0;
            for (int32_t e = t; e < ns; e += kTailThreads) {
                is[S.soff + e] = L.soff[S.sl0 + e];
                is[S.sw + e] = L.sw[S.sl0 + e];
            }
            for (int32_t e = t; e < S.N; e += kTailThreads) is[S.agg + e] = L.agg[S.row0 + e] - c0;
        }
        if (k > 0) {
            const int32_t p0 = L.aptr[S.row0], f0 = sS[k - 1].row0, nf = sS[k - 1].N;
            for (int32_t e = t; e <= S.N; e += kTailThreads) is[S.aptr + e] = L.aptr[S.row0 + e] - p0;
            for (int32_t e = t; e < nf; e += kTailThreads) is[S.amem + e] = L.amem[p0 + e] - f0;
        }
    }
    const int32_t m = sS[0].N * n;
    for (int32_t e = t; e < m * NC; e += kTailThreads)
        vs[sS[0].b + e / (n * NC) * tail_row(n, NC) + e % (n * NC)] = e / NC == q0 + e % NC ? 1.0 : 0.0;
    __syncthreads();
    for (int k = 0; k < nl; ++k) {
        const TailRows S = sS[k], C = sS[k + 1];
        const TailLvl &L = a.lv[k];
        if (a.nu1 >= 1) {
            tail_correct<n, NC, true>(L, S, vs, a.omega);
            for (int q = 1; q < a.nu1; ++q) {
                tail_residual<n, NC>(L, S, vs, is);
                tail_correct<n, NC, false>(L, S, vs, a.omega);
            }
            tail_residual<n, NC>(L, S, vs, is);
        } else {
            for (int32_t e = t; e < S.N * tail_row(n, NC); e += kTailThreads) {
                vs[S.x + e] = 0.0;
                vs[S.r + e] = vs[S.b + e];
            }
            __syncthreads();
        }
        // b of the next level: the residual summed over each aggregate
        for (int32_t e = t; e < C.N * n * NC; e += kTailThreads) {
            const int32_t I = e / (n * NC), q = e - I * n * NC;
            double v = 0.0;
            for (int32_t p = is[C.aptr + I]; p < is[C.aptr + I + 1]; ++p)
                v += vs[S.r + is[C.amem + p] * tail_row(n, NC) + q];
            vs[C.b + I * tail_row(n, NC) + q] = v;
        }
        __syncthreads();
    }
    {   // coarsest: the dense inverse
        const TailRows S = sS[nl];
        const int mc = a.cm[s];
        const double *M = a.cinv + a.coff[s];
        // 16 adjacent lanes share a row, which they read in one run
        for (int32_t o0 = 0; o0 < mc; o0 += kTailThreads / 16) {
            const int32_t o = o0 + t / 16, kk = t & 15;
            double acc[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[c] = 0.0;
            if (o < mc)
#pragma unroll 4
                for (int q = kk; q < mc; q += 16) {
                    const double v = M[(int64_t)o * mc + q];
#pragma unroll
                    for (int c = 0; c < NC; ++c) acc[c] += v * vs[S.b + q / n * tail_row(n, NC) + q % n * NC + c];
                }
#pragma unroll
            for (int w = 8; w > 0; w >>= 1)
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c] += __shfl_xor(acc[c], w, 64);
            if (o < mc && kk == 0)
#pragma unroll
                for (int c = 0; c < NC; ++c) vs[S.x + o / n * tail_row(n, NC) + o % n * NC + c] = acc[c];
        }
        __syncthreads();
    }
    for (int k = nl - 1; k >= 0; --k) {
        const TailRows S = sS[k];
        const int32_t xc = sS[k + 1].x;
        for (int32_t e = t; e < S.N * n * NC; e += kTailThreads) {
            const int32_t i = e / (n * NC), q = e - i * n * NC;
            vs[S.x + i * tail_row(n, NC) + q] += vs[xc + is[S.agg + i] * tail_row(n, NC) + q];
        }
        __syncthreads();
        for (int q = 0; q < a.nu2; ++q) {
            tail_residual<n, NC>(a.lv[k], S, vs, is);
            tail_correct<n, NC, false>(a.lv[k], S, vs, a.omega);
        }
    }
    const int64_t ld = tail_ld(m);
    double *op = a.op + a.opoff[s];
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (q0 + c < m)
            for (int32_t o = t; o < m; o += kTailThreads)
                op[(q0 + c) * ld + o] = vs[sS[0].x + o / n * tail_row(n, NC) + o % n * NC + c];
}

// kTailRowsPerWg scalar rows of one system's operator times the restricted
// residual of the finer level.  Every workgroup forms the whole right side of
// its system (a few KB of gathers); its 16 lanes per column read one line of
// the operator each step.
template <int n, typename T>
__global__ __launch_bounds__(kTailApplyThreads) void k_tail_apply(const TailBlk *__restrict__ blk,
                                                                  const double *__restrict__ op,
                                                                  const int32_t *__restrict__ aptr,
                                                                  const int32_t *__restrict__ amem,
                                                                  const T *__restrict__ rf, T *__restrict__ x) {
    extern __shared__ __align__(16) char smem[];
    double *b = reinterpret_cast<double *>(smem);
    __shared__ double red[kTailApplyThreads / 64][kTailRowsPerWg];
    constexpr int J = kTailApplyThreads / kTailRowsPerWg, U = 4;
    const TailBlk d = blk[blockIdx.x];
    const int t = threadIdx.x, i = t & (kTailRowsPerWg - 1), jj = t / kTailRowsPerWg;
    const int64_t ld = tail_ld(d.m);
    const double *Ti = op + d.off + d.o0 + i;
    // Up to kTailApplyThreads unknowns, whose right side is formed in one round,
    // the operator's values are on their way meanwhile (32 workgroups of m = 512
    // FP32: 7.8 -> 5.6 us a cycle; 416, 5x5: 7.3 -> 6.0).  Loads come back in
    // order, so a second round would wait for them (m = 860: 6.1 -> 7.7 us).
    constexpr int P = kTailApplyThreads / J;
    const bool early = d.m <= kTailApplyThreads;
    double pre[P];
    if (early)
#pragma unroll
        for (int u = 0; u < P; ++u) pre[u] = jj + u * J < d.m ? Ti[(jj + u * J) * ld] : 0.0;
    for (int32_t g = t; g < d.m; g += kTailApplyThreads) {
        const int32_t I = d.row0 + g / n, q = g % n, p0 = aptr[I], p1 = aptr[I + 1];
        // members are summed in order, U rows in flight
        T s = 0;
        for (int32_t p = p0; p < p1; p += U) {
            T v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = rf[(int64_t)amem[min(p + u, p1 - 1)] * n + q];
#pragma unroll
            for (int u = 0; u < U; ++u) s += p + u < p1 ? v[u] : (T)0;
        }
        b[g] = (double)s;
    }
    __syncthreads();
    double acc = 0.0;
    if (early) {
#pragma unroll
        for (int u = 0; u < P; ++u)
            if (jj + u * J < d.m) acc += pre[u] * b[jj + u * J];
    } else {
#pragma unroll 8
        for (int32_t j = jj; j < d.m; j += J) acc += Ti[j * ld] * b[j];
    }
    acc += __shfl_xor(acc, 16, 64);
    acc += __shfl_xor(acc, 32, 64);
    if ((t & 63) < kTailRowsPerWg) red[t >> 6][i] = acc;
    __syncthreads();
    if (t < kTailRowsPerWg && d.o0 + t < d.m) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < kTailApplyThreads / 64; ++w) v += red[w][t];
        x[(int64_t)d.row0 * n + d.o0 + t] = (T)v;
    }
}

// LDS of k_tail_operator for the largest system when the tail starts at l0
// and NC columns run together
int64_t tail_lds(const cbs_system *h, int l0, int NC) {
    const int nlev = (int)h->lev.size();
    int64_t most = 0;
    for (int s = 0; s < h->n_sys; ++s) {
        int64_t dbl = 0, ints = 0, finer = 0;
        for (int l = l0; l < nlev; ++l) {
            const Level &L = h->lev[l];
            const int64_t N = L.sys_off[s + 1] - L.sys_off[s];
            dbl += (l + 1 < nlev ? 3 : 2) * N * tail_row(h->n, NC);
            if (l + 1 < nlev) ints += 2 * ((N >> L.sell.lc) + 2) + N;
            if (l > l0) ints += N + 1 + finer;
            finer = N;
        }
        most = std::max(most, dbl * 8 + ints * 4);
    }
    return most;
}

int64_t tail_lds_budget(const cbs_system *h) {
    return (int64_t)h->lds_max - (int64_t)sizeof(TailRows) * kTailMax - kTailLdsReserve;
}

// the first level (>= 1) that starts the tail, or -1
int tail_level(const cbs_system *h) {
    const int nlev = (int)h->lev.size();
    if (nlev < 2 || h->opt.precond != CBS_PREC_AMG) return -1;
    const int32_t lim = h->opt.tail_rows == 0 ? kTailRowsDefault : h->opt.tail_rows;
    if (lim < 0) return -1;
    // a level whose cycle runs twice (W-cycle) keeps its per-step kernels
    for (int l = std::max(1, h->opt.w_levels + 1); l < nlev; ++l) {
        if (nlev - l > kTailMax) continue;
        const Level &L = h->lev[l];
        int64_t rows = 0, vals = 0, m_max = 0, blocks = 0;
        for (int s = 0; s < h->n_sys; ++s) {
            const int64_t N = L.sys_off[s + 1] - L.sys_off[s], m = N * h->n;
            rows = std::max(rows, N);
            m_max = std::max(m_max, m);
            vals += m * tail_ld(m);
            blocks += cdiv(m, kTailRowsPerWg);
        }
        if (l + 1 == nlev && blocks > kTailCoarseBlocks) continue;
        if (rows > lim || vals * 8 > kTailOpBytes || m_max * 8 > 64 * 1024) continue;
        // DILU and Gauss-Seidel levels keep their own kernels, and so do levels
        // whose copy is window-ordered (kSplitLevelRows rows and more of all
        // systems together, which fill the chip): k_tail_operator takes a
        // system's rows in order, and the rows of a window change places
        // across systems
        bool own = false;
        for (int q = l; q + 1 < nlev; ++q) own = own || h->lev[q].dilu || h->lev[q].sgs || h->lev[q].sell.win;
        if (!own && tail_lds(h, l, 1) <= tail_lds_budget(h)) return l;
    }
    return -1;
}

template <int n, int NC>
void operator_launch(const TailArgs &a, unsigned wgs, size_t lds, hipStream_t st) {
    // more than 64 KB of dynamic LDS is requested explicitly
    if (lds > 64 * 1024)
        HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_tail_operator<n, NC>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL((k_tail_operator<n, NC>), dim3(wgs), dim3(kTailThreads), lds, st, a);
    LAUNCHCHK();
}

template <int n>
void operator_nc(int NC, const TailArgs &a, unsigned wgs, size_t lds, hipStream_t st) {
    if (NC == 4) operator_launch<n, 4>(a, wgs, lds, st);
    else if (NC == 2) operator_launch<n, 2>(a, wgs, lds, st);
    else operator_launch<n, 1>(a, wgs, lds, st);
}

}  // namespace

void tail_plan(cbs_system *h, bool kept) {
    Tail &T = h->tail;
    const int was = T.level, nsys = h->n_sys, nlev = (int)h->lev.size();
    T.level = tail_level(h);
    // a setup that keeps its aggregates appends levels all the same where the
    // last one ended on a stalled level that the new values let go on
    if (T.level < 0 || (kept && T.level == was && T.nlev == nlev)) return;
    T.nlev = nlev;
    T.max_m = 0;
    const int nl = nlev - 1 - T.level;
    std::vector<TailBlk> blk;
    std::vector<int64_t> off(nsys + 1, 0);
    std::vector<int32_t> roff;
    for (int k = 0; k <= nl; ++k)
        for (int64_t o : h->lev[T.level + k].sys_off) roff.push_back((int32_t)o);
    for (int s = 0; s < nsys; ++s) {
        const int32_t row0 = roff[s], m = (roff[s + 1] - row0) * h->n;
        for (int32_t o = 0; o < m; o += kTailRowsPerWg) blk.push_back(TailBlk{row0, m, o, 0, off[s]});
        off[s + 1] = off[s] + m * tail_ld(m);
        T.max_m = std::max(T.max_m, m);
    }
    // columns per workgroup of k_tail_operator: as many as LDS holds, since
    // they share the reads of the matrix, but no fewer workgroups than half
    // the chip's CUs
    std::vector<int32_t> wg(nsys + 1, 0);
    for (T.ncols = 4;; T.ncols /= 2) {
        for (int s = 0; s < nsys; ++s) wg[s + 1] = wg[s] + (int32_t)cdiv((int64_t)(roff[s + 1] - roff[s]) * h->n, T.ncols);
        if (T.ncols == 1 || (wg[nsys] >= 128 && tail_lds(h, T.level, T.ncols) <= tail_lds_budget(h))) break;
    }
    T.wgs = wg[nsys];
    roff.insert(roff.end(), wg.begin(), wg.end());
    T.nblk = (int32_t)blk.size();
    T.vals = off[nsys];
    // one array: the operators' offsets, the workgroups of the product, the rows
    const size_t nb = sizeof(TailBlk) * blk.size(), no = sizeof(int64_t) * off.size(), nr = sizeof(int32_t) * roff.size();
    std::vector<char> plan(no + nb + nr);
    memcpy(plan.data(), off.data(), no);
    memcpy(plan.data() + no, blk.data(), nb);
    memcpy(plan.data() + no + nb, roff.data(), nr);
    T.plan.ensure(plan.size());
    T.off = reinterpret_cast<int64_t *>(T.plan.get());
    T.blk = reinterpret_cast<TailBlk *>(T.plan.get() + no);
    T.roff = reinterpret_cast<int32_t *>(T.plan.get() + no + nb);
    HIPCHK(hipMemcpyAsync(T.plan.get(), plan.data(), plan.size(), hipMemcpyHostToDevice, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));         // the host array ends here
}

void tail_form(cbs_system *h, bool tr) {
    Tail &T = h->tail;
    if (T.level < 0) return;
    const int nlev = (int)h->lev.size(), nl = nlev - 1 - T.level, n = h->n;
    DArr<double> &op = tr ? T.opT : T.op;
    op.ensure(T.vals);
    TailArgs a{};
    for (int k = 0; k <= nl; ++k) {
        Level &L = h->lev[T.level + k];
        TailLvl &d = a.lv[k];
        const Level &F = h->lev[T.level + k - 1];
        d.aptr = F.agg_ptr.get();
        d.amem = F.agg_mem.get();
        if (k == nl) break;                          // the coarsest needs no more
        if (L.sell.prow.get()) cbs_throw(CBS_ERR_ARG, "V-cycle tail: a level whose rows are not in order");
        d.val = tr ? L.sell.v64T.get() : L.sell.v64.get();
        d.Dinv = tr ? L.DinvT.get() : L.Dinv.get();
        d.soff = L.sell.soff.get();
        d.sw = L.sell.sw.get();
        d.scol = L.sell.scol.get();
        d.lc = L.sell.lc;
        d.agg = L.agg.get();
    }
    a.roff = T.roff;
    a.cinv = tr ? h->coarse.invT.get() : h->coarse.inv.get();
    a.coff = h->coarse.off;
    a.cm = h->coarse.m;
    a.opoff = T.off;
    a.op = op.get();
    a.omega = level_omega(h->opt, T.level);          // every tail level is below level 0
    a.nl = nl;
    a.nu1 = std::max(0, h->opt.pre_sweeps);
    a.nu2 = std::max(0, h->opt.post_sweeps);
    a.nsys = h->n_sys;
    a.wgoff = T.roff + (size_t)(nl + 1) * (h->n_sys + 1);
    const int NC = T.ncols;
    const unsigned g = (unsigned)T.wgs;
    const size_t lds = (size_t)tail_lds(h, T.level, NC);
    switch (n) {
        case 1: operator_nc<1>(NC, a, g, lds, h->stream); break;
        case 2: operator_nc<2>(NC, a, g, lds, h->stream); break;
        case 3: operator_nc<3>(NC, a, g, lds, h->stream); break;
        case 4: operator_nc<4>(NC, a, g, lds, h->stream); break;
        case 5: operator_nc<5>(NC, a, g, lds, h->stream); break;
        default: cbs_throw(CBS_ERR_ARG, "bdim must be 1..5");
    }
}

template <typename T>
void launch_tail(cbs_system *h, bool tr, const T *rfine, T *x) {
    const Tail &Tl = h->tail;
    if (Tl.level < 1) cbs_throw(CBS_ERR_ARG, "V-cycle tail: bad level");
    const Level &F = h->lev[Tl.level - 1];
    const dim3 g(Tl.nblk), b(kTailApplyThreads);
    const size_t shm = sizeof(double) * (size_t)Tl.max_m;
#define TAIL_N(NN)                                                                                              \
    hipLaunchKernelGGL((k_tail_apply<NN, T>), g, b, shm, h->stream, Tl.blk, tr ? Tl.opT.get() : Tl.op.get(), \
                       F.agg_ptr.get(), F.agg_mem.get(), rfine, x)
    switch (h->n) {
        case 1: TAIL_N(1); break;
        case 2: TAIL_N(2); break;
        case 3: TAIL_N(3); break;
        case 4: TAIL_N(4); break;
        case 5: TAIL_N(5); break;
        default: cbs_throw(CBS_ERR_ARG, "bdim must be 1..5");
    }
#undef TAIL_N
    LAUNCHCHK();
}
template void launch_tail<float>(cbs_system *, bool, const float *, float *);
template void launch_tail<double>(cbs_system *, bool, const double *, double *);
