// The streaming kernels beside the step: global averaging T_u (Sec. 2; Sec. 4, Eq. 13), the consensus distance
// (Sec. 3), the synthetic delayed gradient of the delay-by-one workload (Sec. 4, Eq. 13/14), the reference streams
// used for measurement, and the device-side builder of the ring tables (Sec. 3, Eq. 3 and Eq. 8).  Included by
// psgd_kernels.hip only.
#ifndef PSGD_STREAMS_H
#define PSGD_STREAMS_H

#include "psgd_pace.h"

namespace psgd {
namespace {

// ---------------------------------------------------------------------------------------
// Global averaging, T_u = (1/n) 1 1^T (Sec. 2: S-PSGD; Sec. 4, Eq. 13: D1D-PSGD's allreduce / L):
//     X_out[i,:] = mean_j X[j,:] - lr * G[i,:].
// A lane owns a column group: first sweep sums its n rows (fp64, so the mean carries one
// fp32 rounding whatever n is), second sweep reads G and writes the n outputs.  All of the
// lane's X loads precede its first store, so X_out may alias X.  Same bytes as the ring step.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void add_to(double* s, f32x4 x) {
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] += (double)x[k];
}
__device__ __forceinline__ f32x4 mean_of(const double* s, double inv_n) {
    return (f32x4){(float)(s[0] * inv_n), (float)(s[1] * inv_n), (float)(s[2] * inv_n), (float)(s[3] * inv_n)};
}

// T = workgroup size, chosen as for the ring step: on long rows a large workgroup whose wavefronts
// sweep the rows in lockstep (a barrier per batch), so each row sees one long contiguous burst.
// RAGGED: 4 does not divide d.
template <typename GT, bool CD, int T, bool RAGGED>
__global__ __launch_bounds__(T) void mix_full_kernel(const float* X, float* Xout, const GT* __restrict__ G, int n,
                                                     int64_t d, Pitch ld, float neg_lr, Sweeps sweeps,
                                                     Gather gather) {
    typedef f32x4 V;
    __shared__ double lds_waves[T / 64];
    const int64_t ncg = (d + kVec - 1) / kVec;
    const double inv_n = 1.0 / (double)n;
    double total = 0.0;
    for (int64_t sw = 0; sw < sweeps.count; ++sw) {
        const int64_t base = sweeps.base(sw), cg = base + threadIdx.x;
        if (base >= ncg) break;                                  // nothing left for this workgroup (uniform)
        const int64_t end = base + sweeps.chunk < ncg ? base + sweeps.chunk : ncg;   // uniform
        const ColGroup c = col_group_of<RAGGED>(cg < end ? cg : ncg, ncg, d);   // an idle lane owns nothing and shadows another
        const float* xc = X + c.col;
        const GT* gc = G + c.col;
        float* oc = Xout + c.col;
        double sum[kVec];
#pragma unroll
        for (int k = 0; k < kVec; ++k) sum[k] = 0.0;
        int r = 0;
        for (; r + kUnroll <= n; r += kUnroll) {
            lockstep_barrier();
            V xs[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) xs[u] = ld_x(xc + (int64_t)(r + u) * ld.x);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) add_to(sum, xs[u]);
        }
        for (; r < n; ++r) add_to(sum, ld_x(xc + (int64_t)r * ld.x));
        const V mean = mean_of(sum, inv_n);
        ColStats<RAGGED> stats;
        if (CD) stats.reset();
        r = 0;
        for (; r + kUnroll <= n; r += kUnroll) {
            lockstep_barrier();
            V gs[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) gs[u] = ld_g(gc + (int64_t)(r + u) * ld.g);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const V out = vfma(neg_lr, gs[u], mean);
                st_cols_of<RAGGED>(oc + (int64_t)(r + u) * ld.o, out, c);
                if (CD) stats.add(out);
            }
        }
        for (; r < n; ++r) {
            const V out = vfma(neg_lr, ld_g(gc + (int64_t)r * ld.g), mean);
            st_cols_of<RAGGED>(oc + (int64_t)r * ld.o, out, c);
            if (CD) stats.add(out);
        }
        if (CD) total += stats.result(inv_n, c);
    }
    if (CD) last_sum(gather, block_sum(total, lds_waves, blockDim.x));
}

// The same on long rows, paced as the ring walk is (psgd_pace.h): a sweep is n items that add an X row and n items that read a
// gradient row and write an output row; loads are D items ahead, the first gradients travelling under the last X rows and the next
// sweep's first X rows under the last outputs.  Rows beyond n (where D does not divide it) repeat the last one; they add nothing and
// their stores are dropped.  All X loads of a lane's columns precede its first store, so X_out may alias X.
// us, dense (lockstep batches of eight rows before): 64 x 25.6 M fp32 with the distance 3703 -> 3313, 64 x 1 M bf16 122 -> 112, 64 x 600 k
// 97 -> 80, 512 x 310 k 390 -> 331.
template <typename GT, bool CD, int D>
__device__ __forceinline__ double full_walk(const float* X, float* Xout, const GT* __restrict__ G, int n, int64_t d, Pitch ld,
                                            float neg_lr, const Sweeps& sweeps, int64_t my_sweeps, Pace* pace) {
    typedef typename RawG<GT>::T GR;
    const int64_t ncg = (d + kVec - 1) / kVec;
    const double inv_n = 1.0 / (double)n;
    WalkCols now = walk_cols<true>(sweeps, 0, ncg, d);
    double total = 0.0;
    int items = 0;
    bool paced = true;
    f32x4 x[D];
    GR g[D];
#pragma unroll
    for (int u = 0; u < D; ++u) x[u] = ld_x(lane_at(X + ((int64_t)row_or_last(u, n) * ld.x + now.col), now.at));
    auto done = [&]() __attribute__((always_inline)) {
        ++items;
        if (threadIdx.x == 0) lds_poke(&pace->done, items);
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int64_t sw = 0; sw < my_sweeps; ++sw) {
        const WalkCols nxt = walk_cols<true>(sweeps, sw + 1 < my_sweeps ? sw + 1 : sw, ncg, d);
        double sum[kVec] = {0.0, 0.0, 0.0, 0.0};
        int r = 0;
        for (; r + D < n; r += D) {
#pragma unroll
            for (int u = 0; u < D; ++u) {
                wait_for_pace(pace, items, paced);
                __builtin_amdgcn_sched_barrier(0);
                const f32x4 in = set_apart(x[u]);
                x[u] = ld_x(lane_at(X + ((int64_t)row_or_last(r + u + D, n) * ld.x + now.col), now.at));
                done();
                add_to(sum, in);
            }
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            wait_for_pace(pace, items, paced);
            __builtin_amdgcn_sched_barrier(0);
            const f32x4 in = set_apart(x[u]);
            g[u] = ld_g_raw(lane_at(G + ((int64_t)row_or_last(u, n) * ld.g + now.col), now.at));
            done();
            if (r + u < n) add_to(sum, in);
        }
        const f32x4 mean = mean_of(sum, inv_n);
        ColStats<true> stats;
        if (CD) stats.reset();
        auto put = [&](int row, GR grad) __attribute__((always_inline)) {
            const f32x4 out = vfma(neg_lr, widen_g(grad), mean);
            float* to = Xout + ((int64_t)row_or_last(row, n) * ld.o + now.col);
            st_row(to, row < n ? now.to : kDropStore, out);
            if (now.lo > 0 && now.lo < 4 && row < n) {           // one lane of the launch
#pragma unroll
                for (int k = 1; k < 4; ++k)
                    if (k >= now.lo) __builtin_nontemporal_store(out[k], to + now.at + k);
            }
            if (CD && row < n) stats.add(out);
        };
        auto mid = [&](int at) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < D; ++u) {
                wait_for_pace(pace, items, paced);
                __builtin_amdgcn_sched_barrier(0);
                const GR grad = set_apart(g[u]);
                g[u] = ld_g_raw(lane_at(G + ((int64_t)row_or_last(at + u + D, n) * ld.g + now.col), now.at));
                done();
                put(at + u, grad);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        mid(0);                                                  // apart: its waits count no stores yet (n > D)
        for (r = D; r + D < n; r += D) mid(r);
#pragma unroll
        for (int u = 0; u < D; ++u) {
            wait_for_pace(pace, items, paced);
            __builtin_amdgcn_sched_barrier(0);
            const GR grad = set_apart(g[u]);
            x[u] = ld_x(lane_at(X + ((int64_t)row_or_last(u, n) * ld.x + nxt.col), nxt.at));
            done();
            put(r + u, grad);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (CD) total += stats.result(inv_n, ColGroup{0, now.lo, 4});
        now = nxt;
    }
    return total;
}
template <typename GT, bool CD, int D>
__global__ __launch_bounds__(plan::kRingThreadsMost) void mix_full_walk_kernel(const float* X, float* Xout, const GT* __restrict__ G,
                                                                               int n, int64_t d, Pitch ld, float neg_lr,
                                                                               Sweeps sweeps, int lanes, int slot, int lead,
                                                                               Gather gather) {
    __shared__ double lds_waves[plan::kRingThreadsMost / 64];
    __shared__ Pace pace;
    const int tid = threadIdx.x;
    if (tid == 0) pace = Pace{0, lead};
    __syncthreads();
    const int64_t my_sweeps = sweeps_of(sweeps, (d + kVec - 1) / kVec);
    const int items = 2 * ((n + D - 1) / D) * D;                 // of a sweep
    double total = 0.0;
    if (my_sweeps > 0) {
        if (tid >= lanes) keep_pace(&pace, slot, lead, (int)my_sweeps * items, items);
        else total = full_walk<GT, CD, D>(X, Xout, G, n, d, ld, neg_lr, sweeps, my_sweeps, &pace);
    }
    if (CD) last_sum(gather, block_sum(total, lds_waves, lanes + 64));
}

// The same where the columns alone do not fill the chip: a tile is all n rows x C column groups on nrg row groups of C
// lanes, as in the short-row kernel; a lane sums rows rg, rg + nrg, ... of its column group, the row groups' sums meet
// in LDS and the mean comes back through it.  The first eight gradient rows travel beside the first X rows.  Every X
// row of the tile has been read before its first output is stored, so X_out may alias X.
// FEW: rows of fewer than four columns.
template <typename GT, bool CD, bool FEW>
__global__ __launch_bounds__(plan::kShortThreads, 4) void mix_full_rows_kernel(const float* X, float* Xout,
                                                                               const GT* __restrict__ G, int n, int64_t d,
                                                                               Pitch ld, float neg_lr, int logc, int nrg,
                                                                               Gather gather) {
    typedef typename RawG<GT>::T GR;
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    __shared__ double lds_waves[plan::kShortThreads / 64];
    const int T = nrg << logc, C = 1 << logc, tid = threadIdx.x, lane = tid & (C - 1);
    int rg = tid >> logc;
    double* sums = reinterpret_cast<double*>(lds_raw);             // [4][nrg][C]
    float* means = reinterpret_cast<float*>(sums + 4 * T);         // [4][C]
    float* pivots = means + 4 * C;                                 // [4][nrg][C], CD only
    const double inv_n = 1.0 / (double)n;
    const int64_t ntiles = (((d + 3) >> 2) + C - 1) >> logc;
    double total = 0.0;
    for (int64_t t = plan::die_contiguous_slot(blockIdx.x, gridDim.x, kXcds); t < ntiles; t += gridDim.x) {
        asm volatile("" : "+v"(rg));                             // row offsets are computed again, not kept in registers
        const ColGroup c = col_group(t * C + lane, d);
        const float* xc = X + c.col;
        const GT* gc = G + c.col;
        float* oc = Xout + c.col;
        f32x4 xs[kUnroll];
        GR gs[kUnroll];
        double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) xs[u] = ld_cols<FEW>(xc + (int64_t)row_or_last(rg + u * nrg, n) * ld.x, d);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) gs[u] = ld_cols_raw<FEW>(gc + (int64_t)row_or_last(rg + u * nrg, n) * ld.g, d);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            if (rg + u * nrg < n) add_to(sum, xs[u]);
        for (int r = rg + kUnroll * nrg; r < n; r += kUnroll * nrg) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) xs[u] = ld_cols<FEW>(xc + (int64_t)row_or_last(r + u * nrg, n) * ld.x, d);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (r + u * nrg < n) add_to(sum, xs[u]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) sums[((k * nrg + rg) << logc) + lane] = sum[k];
        lds_barrier();                                           // also: every X row of the tile has arrived
        row_group_columns(logc, nrg, T, [&](int k, int l, int first, int step, int reach) {
            double at = 0.0;
#pragma unroll 4
            for (int q = first; q < nrg; q += step) at += sums[((k * nrg + q) << logc) + l];
            for (int off = reach; off < 64; off <<= 1) at += __shfl_xor(at, off, 64);
            if (first == 0) means[(k << logc) + l] = (float)(at * inv_n);
        });
        lds_barrier();
        const f32x4 mean = {means[lane], means[C + lane], means[2 * C + lane], means[3 * C + lane]};
        asm volatile("" : "+v"(rg));
        f32x4 pv;
        double a[4] = {0.0, 0.0, 0.0, 0.0}, sq[4] = {0.0, 0.0, 0.0, 0.0};
        auto put = [&](int r, GR g, bool first) __attribute__((always_inline)) {
            const f32x4 out = vfma(neg_lr, widen_g(g), mean);
            if (CD && first) pv = out;
            if (r < n) {
                st_cols(oc + (int64_t)r * ld.o, out, c);
                if (CD && !first) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const double df = (double)out[k] - (double)pv[k];
                        a[k] += df;
                        sq[k] = fma(df, df, sq[k]);
                    }
                }
            }
        };
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) put(rg + u * nrg, gs[u], u == 0);
        for (int r = rg + kUnroll * nrg; r < n; r += kUnroll * nrg) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) gs[u] = ld_cols_raw<FEW>(gc + (int64_t)row_or_last(r + u * nrg, n) * ld.g, d);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) put(r + u * nrg, gs[u], false);
        }
        if (CD) total += row_group_distance(sums, pivots, logc, nrg, n, T, rg, lane, inv_n, a, sq, pv, c, t * C, d);
        lds_barrier();                                           // the merge slots are free again
    }
    if (CD) last_sum(gather, block_sum(total, lds_waves, T));
}

// Consensus-distance kernels (the per-column arithmetic is defined above the ring walk).
template <bool RAGGED>
__global__ __launch_bounds__(kThreads) void consensus_partial_kernel(const float* __restrict__ X, int n,
                                                                     int64_t d, int64_t ldx, int chunk,
                                                                     Gather gather) {
    typedef f32x4 V;
    __shared__ double lds4[4];
    const int64_t ncg = (d + kVec - 1) / kVec;
    const int64_t stride = (int64_t)gridDim.x * chunk;
    const double inv_n = 1.0 / (double)n;
    double total = 0.0;
    for (int64_t cg = (int)threadIdx.x < chunk ? (int64_t)blockIdx.x * chunk + threadIdx.x : ncg; cg < ncg; cg += stride) {
        const ColGroup c = col_group_of<RAGGED>(cg, ncg, d);
        const float* xc = X + c.col;
        double s[kVec], a[kVec], b[kVec];
        pivot_of(ld_x(xc), s);
#pragma unroll
        for (int k = 0; k < kVec; ++k) a[k] = b[k] = 0.0;
        int r = 1;
        for (; r + kUnroll <= n; r += kUnroll) {
            V xs[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) xs[u] = ld_x(xc + (int64_t)(r + u) * ldx);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) acc_diff(a, b, xs[u], s);
        }
        if (r < n) {
            V xs[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (r + u < n) xs[u] = ld_x(xc + (int64_t)(r + u) * ldx);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (r + u < n) acc_diff(a, b, xs[u], s);
        }
#pragma unroll
        for (int k = 0; k < kVec; ++k)
            if (!RAGGED || k >= c.lo) total += b[k] - a[k] * a[k] * inv_n;
    }
    last_sum_or_none(gather, block_sum(total, lds4, blockDim.x));
}

// The same where the columns alone do not fill the chip: rows spread over row groups of lanes as in the short-row kernel.
template <bool FEW>
__global__ __launch_bounds__(plan::kShortThreads, 4) void consensus_rows_kernel(const float* __restrict__ X, int n, int64_t d,
                                                                                int64_t ldx, int logc, int nrg,
                                                                                Gather gather) {
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    __shared__ double lds_waves[plan::kShortThreads / 64];
    const int T = nrg << logc, C = 1 << logc, tid = threadIdx.x, lane = tid & (C - 1), rg = tid >> logc;
    double* sums = reinterpret_cast<double*>(lds_raw);             // [4][nrg][C]
    float* pivots = reinterpret_cast<float*>(sums + 4 * T);        // the same
    const double inv_n = 1.0 / (double)n;
    const int64_t ntiles = (((d + 3) >> 2) + C - 1) >> logc;
    double total = 0.0;
    for (int64_t t = plan::die_contiguous_slot(blockIdx.x, gridDim.x, kXcds); t < ntiles; t += gridDim.x) {
        const ColGroup c = col_group(t * C + lane, d);
        const float* xc = X + c.col;
        f32x4 pv;
        double s[4], a[4] = {0.0, 0.0, 0.0, 0.0}, sq[4] = {0.0, 0.0, 0.0, 0.0};
        for (int r = rg; r == rg || r < n; r += kUnroll * nrg) {   // a row group without rows still has a pivot
            f32x4 xs[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) xs[u] = ld_cols<FEW>(xc + (int64_t)row_or_last(r + u * nrg, n) * ldx, d);
            if (r == rg) {
                pv = xs[0];
                pivot_of(pv, s);
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                if (r + u * nrg < n) acc_diff(a, sq, xs[u], s);
        }
        total += row_group_distance(sums, pivots, logc, nrg, n, T, rg, lane, inv_n, a, sq, pv, c, t * C, d);
        lds_barrier();                                           // the merge slots are free again
    }
    last_sum(gather, block_sum(total, lds_waves, T));
}

// The same distance for long rows, in the form of the step kernels: one large workgroup per compute unit whose
// wavefronts sweep the rows in lockstep batches, the column groups split evenly and die-contiguously over the
// persistent grid.  A lane owns one column group per sweep.
template <int T, bool RAGGED>
__global__ __launch_bounds__(T) void consensus_sweep_kernel(const float* __restrict__ X, int n, int64_t d, int64_t ldx,
                                                            Sweeps sweeps, Gather gather) {
    typedef f32x4 V;
    __shared__ double lds_waves[T / 64];
    const int64_t ncg = (d + kVec - 1) / kVec;
    const double inv_n = 1.0 / (double)n;
    double total = 0.0;
    for (int64_t sw = 0; sw < sweeps.count; ++sw) {
        const int64_t base = sweeps.base(sw), cg = base + threadIdx.x;
        if (base >= ncg) break;                                  // nothing left for this workgroup (uniform)
        const int64_t end = base + sweeps.chunk < ncg ? base + sweeps.chunk : ncg;   // uniform
        const ColGroup c = col_group_of<RAGGED>(cg < end ? cg : ncg, ncg, d);   // an idle lane owns nothing and shadows another
        const float* xc = X + c.col;
        double s[kVec], a[kVec], b[kVec];
        pivot_of(ld_x(xc), s);
#pragma unroll
        for (int k = 0; k < kVec; ++k) a[k] = b[k] = 0.0;
        int r = 1;
        for (; r + kUnroll <= n; r += kUnroll) {
            lockstep_barrier();
            V xs[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) xs[u] = ld_x(xc + (int64_t)(r + u) * ldx);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) acc_diff(a, b, xs[u], s);
        }
        if (r < n) {
            V xs[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll - 1; ++u)
                if (r + u < n) xs[u] = ld_x(xc + (int64_t)(r + u) * ldx);
#pragma unroll
            for (int u = 0; u < kUnroll - 1; ++u)
                if (r + u < n) acc_diff(a, b, xs[u], s);
        }
#pragma unroll
        for (int k = 0; k < kVec; ++k)
            if (RAGGED ? k >= c.lo && k < c.hi : c.lo == 0) total += b[k] - a[k] * a[k] * inv_n;
    }
    last_sum(gather, block_sum(total, lds_waves, blockDim.x));
}

// The distance's last sum where the workgroups leave it (plan::distance_summed_apart), in a fixed order.
__global__ __launch_bounds__(kThreads) void sum_partials_kernel(const double* __restrict__ partials, int count, double* __restrict__ out) {
    __shared__ double lds_waves[kThreads / 64];
    double v = 0.0;
    for (int i = threadIdx.x; i < count; i += kThreads) v += partials[i];
    v = block_sum(v, lds_waves, kThreads);
    if (threadIdx.x == 0) *out = v;
}

// The distance of rows without columns.
__global__ void no_distance_kernel(double* out) { *out = 0.0; }

// The stand-in gradient producer: row blockIdx.y, a lane per column group.  FEW: rows of fewer than four columns.
template <bool FEW>
__global__ __launch_bounds__(kThreads) void synth_grad_kernel(const float* __restrict__ xp, int64_t ldx,
                                                              const float* __restrict__ noise, int64_t ldn,
                                                              float* __restrict__ g, int64_t ldg, int64_t d, float c) {
    const int64_t ncg = (d + kVec - 1) / kVec;
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    xp += (int64_t)blockIdx.y * ldx;
    noise += (int64_t)blockIdx.y * ldn;
    g += (int64_t)blockIdx.y * ldg;
    for (int64_t cg = (int64_t)blockIdx.x * kThreads + threadIdx.x; cg < ncg; cg += stride) {
        const ColGroup at = col_group(cg, d);
        st_cols(g + at.col, vfma(c, ld_cols<FEW>(xp + at.col, d), ld_cols<FEW>(noise + at.col, d)), at);
    }
}

// ---------------------------------------------------------------------------------------
// Reference streams (measurement support, not a step of the method): the memory traffic of the step with the
// mixing taken out, as a walk that nothing keeps in step issues it -- a lane owns one 128-bit column group and
// walks the n rows, the workgroup's wavefronts sweep the rows in lockstep batches, the column groups are split
// evenly over a persistent grid.  KIND 0 only reads X and G, KIND 1 only writes X_out, KIND 2 is
// X_out = X + a * G (the step's 4 + 2 + 4 or 4 + 4 + 4 bytes per element, no neighbours).  The rate these
// reach is what the chip's memory system gives that access pattern; the paced walks are ahead of KIND 2 (psgd_pace.h).
// ---------------------------------------------------------------------------------------
enum { kRefRead = 0, kRefWrite = 1, kRefAxpy = 2 };

template <int KIND, typename GT, int T>
__global__ __launch_bounds__(T) void reference_stream_kernel(const float* X, float* Xout, const GT* __restrict__ G,
                                                             int n, int64_t d, Pitch ld, float a, Sweeps sweeps) {
    const int64_t ncg = d / 4;
    f32x4 keep = splat4(0.0f);
    for (int64_t sw = 0; sw < sweeps.count; ++sw) {
        const int64_t base = sweeps.base(sw), cg = base + threadIdx.x;
        if (base >= ncg) break;                                  // nothing left for this workgroup (uniform)
        const int64_t end = base + sweeps.chunk < ncg ? base + sweeps.chunk : ncg;   // uniform
        const bool act = cg < end;                               // an idle lane shadows column group 0
        const int64_t col = (act ? cg : 0) * 4;
        const float* xc = X + col;
        const GT* gc = G + col;
        float* oc = Xout + col;
        int r = 0;
        for (; r + kUnroll <= n; r += kUnroll) {
            lockstep_barrier();
            f32x4 xs[kUnroll], gs[kUnroll];
            if (KIND != kRefWrite) {
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    xs[u] = ld_x(xc + (int64_t)(r + u) * ld.x);
                    gs[u] = ld_g(gc + (int64_t)(r + u) * ld.g);
                }
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (KIND == kRefRead) keep += xs[u] + gs[u];
                if (KIND == kRefWrite && act) st_x(oc + (int64_t)(r + u) * ld.o, splat4(a));
                if (KIND == kRefAxpy && act) st_x(oc + (int64_t)(r + u) * ld.o, vfma(a, gs[u], xs[u]));
            }
        }
        for (; r < n; ++r) {
            if (KIND == kRefRead) keep += ld_x(xc + (int64_t)r * ld.x) + ld_g(gc + (int64_t)r * ld.g);
            if (KIND == kRefWrite && act) st_x(oc + (int64_t)r * ld.o, splat4(a));
            if (KIND == kRefAxpy && act)
                st_x(oc + (int64_t)r * ld.o, vfma(a, ld_g(gc + (int64_t)r * ld.g), ld_x(xc + (int64_t)r * ld.x)));
        }
    }
    // The loads of the read-only stream must have an observer: a store that the data never triggers.
    if (KIND == kRefRead && __float_as_uint(keep.x + keep.y + keep.z + keep.w) == 0x7FC0BEEFu) Xout[0] = keep.x;
}

// ---------------------------------------------------------------------------------------
// Mixing table of one iteration, built on the device (Sec. 4: all learners derive the same
// ring from a shared seed, so the table is a function of (n, seed, step) only).  One
// workgroup, a lane per ring position, no serial part: the kernel is pure latency, and the
// Durstenfeld shuffle's n - 1 swaps, run by one lane in LDS, were nearly all of it.
//
// The SplitMix64 draws are counter-based (state of draw t = state0 + (t + 1) * increment), so
// all swap partners j(i) are computed at once.  The shuffle runs i = n-1 .. 1 and swaps
// positions i and j(i) <= i, so position i is final after its own step and what it then holds
// is what stood at j(i) just before.  A position p is written before that only by steps i' > i
// with j(i') = p, and each puts there what stood at i' before step i'.  Hence, with
//     W(p)    what stands at position p before step p:  W(next(p)) if next(p) = min{i' : j(i') = p, i' > p} exists, else p
//     same(i) min{i' > i : j(i') = j(i)}
// the result is sigma(i) = W(i) where j(i) = i, else W(same(i)) where that exists, else j(i);
// sigma(0) = W(0).  The positions that share a partner are linked in LDS (in any order: only the
// smallest index above one's own is asked for); such a list, and the strictly increasing chain
// along next that W follows, are about ln n long.
// Kernel time for 8 / 64 / 128 / 512 learners: 1.8 / 2.2 / 2.3 / 3.0 us, by serial swaps 2.0 / 4.0 / 6.4 / 21.0.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(PSGD_MAX_N) void build_mixing_kernel(int randomize, int n, uint64_t seed,
                                                                  uint64_t* step_dev, uint64_t step_offset,
                                                                  uint64_t advance, int32_t* __restrict__ nbr,
                                                                  float* __restrict__ w) {
    __shared__ int sigma[PSGD_MAX_N];
    __shared__ int head[PSGD_MAX_N], link[PSGD_MAX_N];   // per partner: the positions that share it
    __shared__ int next[PSGD_MAX_N];
    const int p = threadIdx.x;                            // the launch has a lane for every position below n
    const uint64_t base = step_dev ? *static_cast<volatile uint64_t*>(step_dev) : 0ull;
    const uint64_t step = base + step_offset;
    if (randomize) {
        constexpr uint64_t kWeyl = 0x9E3779B97F4A7C15ull;
        const uint64_t state0 = seed ^ ((step + 1ull) * kWeyl);
        int mine = -1;                                    // position 0 and lanes beyond n take part in no swap
        if (p >= 1 && p < n) {
            const int t = n - 1 - p;                      // draw t serves position n - 1 - t
            uint64_t z = state0 + (uint64_t)(t + 1) * kWeyl;
            z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
            z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
            z ^= z >> 31;
            mine = (int)__umul64hi(z, (uint64_t)(p + 1));
        }
        head[p] = -1;
        next[p] = PSGD_MAX_N;                             // none
        __syncthreads();
        if (mine >= 0) {
            link[p] = atomicExch(&head[mine], p);
            if (mine != p) atomicMin(&next[mine], p);
        }
        __syncthreads();
        if (p < n) {
            int at = p;
            if (p != 0 && mine != p) {
                at = PSGD_MAX_N;
                for (int i = head[mine]; i >= 0; i = link[i])
                    if (i > p && i < at) at = i;
            }
            if (at == PSGD_MAX_N) {
                at = mine;
            } else {
                for (int up = next[at]; up < PSGD_MAX_N; up = next[at]) at = up;
            }
            sigma[p] = at;
        }
    } else {
        sigma[p] = p;
    }
    __syncthreads();
    const float third = 1.0f / 3.0f;
    if (p < n) {
        const int me = sigma[p];
        nbr[3 * me + 0] = me;
        nbr[3 * me + 1] = sigma[p == 0 ? n - 1 : p - 1];
        nbr[3 * me + 2] = sigma[p == n - 1 ? 0 : p + 1];
        w[3 * me + 0] = third;
        w[3 * me + 1] = third;
        w[3 * me + 2] = third;
    }
    if (p == 0 && step_dev && advance) *step_dev = base + advance;
}

}  // namespace
}  // namespace psgd

#endif
