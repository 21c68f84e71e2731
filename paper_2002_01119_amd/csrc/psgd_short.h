// The model-averaging step (Sec. 2, Eq. 2) on short rows, for any mixing table: mix_short_kernel.  Included by
// psgd_kernels.hip only.
#ifndef PSGD_SHORT_H
#define PSGD_SHORT_H

#include "psgd_device.h"

#include <type_traits>

namespace psgd {
namespace {

// ---------------------------------------------------------------------------------------
// One tile = all n rows x C column groups.  The workgroup's lanes form nrg row groups of C lanes; lane (rg, lane)
// loads, produces and stores rows rg, rg + nrg, ... of column group `lane`, R of them, all in registers.  The X rows
// pass through LDS once, where the other row groups read their neighbours; any table is served alike, so nothing is
// classified.  The tile is complete in LDS before its first output is stored and tiles own their columns, so X_out
// may alias X.
//
// Launches of this size are bound by latency and by how many bytes are in flight, not by the HBM's rate.  Rows are
// spread over lanes as well as columns, so that few columns (many learners of a small model) still fill the chip;
// every load of the first tile is issued at once, behind the loads of the table that they do not depend on; and where
// a workgroup has several tiles the next one's X rows are loaded as soon as the registers have gone to LDS, its
// gradients as each row is finished.
//
// Measured (step with the distance and its final sum unless noted, MI355X; before: the ring walk or the tiled kernel in
// small workgroups, a lane walking all rows): 512 learners x 60 k 171 -> 77 us (4.8 TB/s), 16 x 1 M with 5 slots 49.8 -> 38.6,
// 8 x 1 M 25.6 -> 18.5, 100 x 50 k without the distance 34.7 -> 10.8, 32 x 786 433 at odd addresses, no distance, 77 -> 58.
//
// Inside the loop every load and store is unconditional (the waits then count operations instead of waiting for all
// of them): a lane without a row repeats the last one, loads and stores alike.  The one tile at the ragged end of the
// rows comes after the loop.
//
// The distance (CD): every lane measures its outputs against its first one, in fp64, and the row groups' sums meet in
// LDS, where they are brought to row group 0's pivot exactly (row_group_merge).
// ---------------------------------------------------------------------------------------
// The next gradients alone, where the table is invalid: the workgroup's tiles, row by row.
__device__ __forceinline__ void produce_tiles(int tid, const float* X, int n, int64_t d, int64_t ldx, int logc, int nrg, const Produce& prod) {
    const int C = 1 << logc, lane = tid & (C - 1);
    const int64_t ntiles = (((d + 3) >> 2) + C - 1) >> logc;
    for (int64_t t = plan::die_contiguous_slot(blockIdx.x, gridDim.x, kXcds); t < ntiles; t += gridDim.x) {
        const ColGroup c = col_group(t * C + lane, d);
        for (int r = tid >> logc; r < n; r += nrg)
            st_cols(prod.g + (int64_t)r * prod.ldg + c.col,
                    vfma(prod.c, ld_x(X + (int64_t)r * ldx + c.col), ld_x(prod.noise + (int64_t)r * prod.ldn + c.col)), c);
    }
}

// DEG: slots per table row, 3 or 0 (any).  ONE: a tile per workgroup (two or up to eight rows per lane: nothing is
// loaded ahead, so those registers hold rows).  CACHED: which accesses go without the non-temporal hint (plan::cached_accesses).
// FEW: rows of fewer than four columns.  PROD: also the next gradients of the delay-by-one schedule, of the rows as they were.  WALK: in the kernel
// of the ring walk.
// Run by nrg << logc lanes of the workgroup, lane `tid` of them, the others having ended.
struct ShortLds {
    char* dynamic;                           // plan::ShortPlan::lds bytes
    double* waves;                           // one per wavefront
    int* bad;                                // the same
};
template <typename GT, bool CD, int DEG, int R, bool ONE, int CACHED, bool FEW, bool PROD, bool WALK>
__device__ __forceinline__ void short_tiles(int tid, const float* X, float* Xout, const GT* __restrict__ G,
                                            const int32_t* __restrict__ nbr, const float* __restrict__ w, int deg_any, int n, int64_t d, Pitch ld, float neg_lr,
                                            int logc, int nrg, int tab_bytes, int tile_bytes, const Gather& gather,
                                            const ShortLds& lds, const Produce& prod) {
    typedef typename RawG<GT>::T GR;
    char* lds_raw = lds.dynamic;
    double* lds_waves = lds.waves;
    int* lds_bad = lds.bad;
    const int deg = DEG ? DEG : deg_any;
    const int T = nrg << logc, C = 1 << logc, lane = tid & (C - 1), lane16 = lane * 16;
    int rg = tid >> logc;
    TileSlot* tab = reinterpret_cast<TileSlot*>(lds_raw);       // slot: byte offset of the source row in the tile, weight
    char* tile = lds_raw + tab_bytes;
    // the distance's merge slots, [4][nrg][C]: where there is one tile they take its place once it has been read
    double* sums = reinterpret_cast<double*>(tile + (ONE ? 0 : tile_bytes));
    float* pivots = reinterpret_cast<float*>(sums + 4 * T);
    const int entries = n * deg;
    const int64_t nfull = (d >> 2) >> logc, ntiles = (((d + 3) >> 2) + C - 1) >> logc;
    const int64_t step = gridDim.x;
    int64_t t = plan::die_contiguous_slot(blockIdx.x, gridDim.x, kXcds);
    const double inv_n = 1.0 / (double)n;
    double total = 0.0;

    // The table's loads go first, the first tile's behind them; a lane's share of a larger table follows.
    constexpr int TE = 2;
    int32_t tv[TE];
    float tw[TE];
#pragma unroll
    for (int i = 0; i < TE; ++i) {
        const int e = tid + i * T < entries ? tid + i * T : entries - 1;
        tv[i] = nbr[e];
        tw[i] = w[e];
    }
    f32x4 x[R];
    GR g[R];
    auto row_of = [&](int u) {
        const int r = rg + u * nrg;
        return r < n ? r : n - 1;
    };
    ColGroup cg = col_group(t * C + lane, d);
    constexpr bool CL = (CACHED & plan::kCachedLoads) != 0, CS = (CACHED & plan::kCachedStores) != 0;
#pragma unroll
    for (int u = 0; u < R; ++u) x[u] = ld_cols<FEW, CL>(X + (int64_t)row_of(u) * ld.x + cg.col, d);
#pragma unroll
    for (int u = 0; u < R; ++u) g[u] = ld_cols_raw<FEW, CL>(G + (int64_t)row_of(u) * ld.g + cg.col, d);
    // The noise of the next gradients travels with them where registers allow (few rows per lane: the launches whose latency shows).
    // More rows take the registers of the first few in turn.
    constexpr bool EARLY = PROD && R <= 4;
    constexpr int NR = !PROD ? 1 : R <= 4 ? R : CD && R == 8 ? 2 : 4;
    f32x4 noise[NR];
    auto load_noise = [&](int u, const ColGroup& at) __attribute__((always_inline)) {
        noise[u % NR] = ld_x<CL>(prod.noise + (int64_t)row_of(u) * prod.ldn + at.col);
    };
    auto own_row = [&](int u) __attribute__((always_inline)) {
        return *reinterpret_cast<const f32x4*>(tile + ((row_of(u) << (logc + 4)) + lane16));
    };
    if (EARLY) {
#pragma unroll
        for (int u = 0; u < NR; ++u) load_noise(u, cg);
    }
    int bad = 0;
#pragma unroll
    for (int i = 0; i < TE; ++i) {
        const int e = tid + i * T;
        if (e < entries) {
            bad |= (unsigned)tv[i] >= (unsigned)n;
            tab[e] = TileSlot{(uint32_t)tv[i] << (logc + 4), tw[i]};
        }
    }
    for (int e = tid + TE * T; e < entries; e += T) {
        const int v = nbr[e];
        bad |= (unsigned)v >= (unsigned)n;
        tab[e] = TileSlot{(uint32_t)v << (logc + 4), w[e]};
    }
    const bool wave_bad = __any(bad);
    if ((tid & 63) == 0) lds_bad[tid >> 6] = wave_bad;
    lds_barrier();
    {
        int any = 0;
        for (int i = 0; i < T / 64; ++i) any |= lds_bad[i];
        if (any) {                                              // nothing of the step is written
            if (blockIdx.x == 0 && tid == 0) atomicOr(&g_status_word, 1);
            if (PROD) produce_tiles(tid, X, n, d, ld.x, logc, nrg, prod);
            if (CD) last_sum(gather, __builtin_nan(""));
            return;
        }
    }

    // One tile, its X rows in x and its gradients in g; the next one's, columns `next`, take their places.
    auto one_tile = [&](auto full, const ColGroup& next) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full)::value;
        // Row offsets are cheap to compute again and would take two registers per row and array if kept from tile to tile.
        asm volatile("" : "+v"(rg));
#pragma unroll
        for (int u = 0; u < R; ++u) *reinterpret_cast<f32x4*>(tile + ((row_of(u) << (logc + 4)) + lane16)) = x[u];
        lds_barrier();
        if (FULL) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < R; ++u) x[u] = ld_cols<FEW, CL>(X + (int64_t)row_of(u) * ld.x + next.col, d);
        }
        if (PROD && !EARLY) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < NR; ++u) load_noise(u, cg);
        }
        // SB rows' slot chains advance together (a table read, then a tile read that depends on it, per slot).
        constexpr int SB = PROD && !ONE ? 2 : R < 4 ? R : 4;           // two where registers go to the noise too
        // The next gradients' loads behind the outputs' stores: with two rows the compiler puts them in front beside the ring walk, and with bf16 gradients,
        // and a tile then waits for its gradients where it needs its rows (with the distance, 5 x 14.5 M off the lines bf16 159 / 147 us, 5 x 11.2 M 132 / 125,
        // 6 slots 5 x 14.9 M bf16 160 / 149; fp32 gradients in the short-row kernel are in that order anyway, and pinning it loses off the lines, 6 x 24.5 M
        // with 4 slots 316 / 331).
        constexpr bool LOADS_LAST = R == 2 && !PROD && !ONE && (WALK || sizeof(GT) == 2);
        // The last place of a lane may have no row: without the distance, where registers allow it, its output is not stored a second time (7 x
        // 31.3 M 499 / 463 us, 11 x 2.1 M off the lines 55.4 / 52.7, 34 x 475 741 bf16 38.7 / 37.6).
        constexpr bool CHECKED = R == 4 && !CD && !PROD;
        double a[4] = {0.0, 0.0, 0.0, 0.0}, sq[4] = {0.0, 0.0, 0.0, 0.0};
        f32x4 pv;
        auto to_distance = [&](int u, const f32x4& o) __attribute__((always_inline)) {
            if (CD && u == 0) pv = o;
            if (CD && u > 0 && rg + u * nrg < n) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double df = (double)o[k] - (double)pv[k];
                    a[k] += df;
                    sq[k] = fma(df, df, sq[k]);
                }
            }
        };
#pragma unroll
        for (int j = 0; j < R; j += SB) {
            __builtin_amdgcn_sched_barrier(0);
            if (PROD) asm volatile("" : "+v"(rg));
            const TileSlot* tp[SB];
            f32x4 out[SB];
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                if (j + i >= R) break;
                tp[i] = tab + row_of(j + i) * deg;
                const TileSlot e = tp[i][0];
                out[i] = *reinterpret_cast<const f32x4*>(tile + (e.off + lane16)) * e.w;
            }
            auto slot = [&](int s) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < SB; ++i) {
                    if (j + i >= R) break;
                    const TileSlot e = tp[i][s];
                    out[i] = vfma(e.w, *reinterpret_cast<const f32x4*>(tile + (e.off + lane16)), out[i]);
                }
            };
            if (DEG) {
#pragma unroll
                for (int s = 1; s < DEG; ++s) slot(s);
            } else {
#pragma unroll 2
                for (int s = 1; s < deg; ++s) slot(s);
            }
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                const int u = j + i;
                if (u >= R) break;
                const f32x4 o = vfma(neg_lr, widen_g(g[u]), out[i]);
                if (PROD && !EARLY) asm volatile("" : "+v"(rg));
                float* to = Xout + (int64_t)row_of(u) * ld.o + cg.col;
                if (FULL) {
                    if (!CHECKED || u + 1 < R || rg + u * nrg < n) st_x<CS>(to, o);
                    if (PROD) {
                        st_x<CS>(prod.g + (int64_t)row_of(u) * prod.ldg + cg.col, vfma(prod.c, own_row(u), noise[u % NR]));
                        load_noise(u, next);
                    }
                    if (!LOADS_LAST) g[u] = ld_cols_raw<FEW, CL>(G + (int64_t)row_of(u) * ld.g + next.col, d);
                } else if (rg + u * nrg < n) {
                    st_cols<CS>(to, o, cg);
                    if (PROD) st_cols<CS>(prod.g + (int64_t)row_of(u) * prod.ldg + cg.col, vfma(prod.c, own_row(u), noise[u % NR]), cg);
                }
                if (PROD && u + NR < R) load_noise(u + NR, cg);
                if (LOADS_LAST) out[i] = o;
                else to_distance(u, o);
            }
            if (LOADS_LAST) {
                if (FULL) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < R; ++u) g[u] = ld_cols_raw<FEW, CL>(G + (int64_t)row_of(u) * ld.g + next.col, d);
                }
#pragma unroll
                for (int u = 0; u < R; ++u) to_distance(u, out[u]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (CD && nrg == 1) {                                   // few learners: the lane has seen all rows of its columns
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (FULL || (k >= cg.lo && k < cg.hi)) total += sq[k] - a[k] * a[k] * inv_n;
        } else if (CD) {
            if (ONE) lds_barrier();                             // every row of the tile has been read
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                sums[((k * nrg + rg) << logc) + lane] = a[k];
                pivots[((k * nrg + rg) << logc) + lane] = pv[k];
                if (FULL || (k >= cg.lo && k < cg.hi)) total += sq[k];   // the column exists and is this lane's
            }
        }
        lds_barrier();                                          // the tile is free again; the sums are complete
        if (CD && nrg > 1)                                      // t is already the next tile's in the loop
            total += row_group_merge<FULL>(sums, pivots, logc, nrg, n, T, inv_n, (t - (FULL ? step : 0)) * C, d);
    };
    while (!ONE && t < nfull) {
        t += step;
        const ColGroup next = col_group(t * C + lane, d);
        one_tile(std::true_type{}, next);
        cg = next;
    }
    if (t < ntiles) one_tile(std::false_type{}, cg);
    if (CD) last_sum(gather, block_sum(total, lds_waves, T));
}

template <typename GT, bool CD, int DEG, int R, bool ONE, int CACHED, bool FEW, bool PROD>
__global__ __launch_bounds__(plan::kShortThreads, plan::kShortThreads / 256) void mix_short_kernel(
    const float* X, float* Xout, const GT* __restrict__ G, const int32_t* __restrict__ nbr, const float* __restrict__ w,
    int deg_any, int n, int64_t d, Pitch ld, float neg_lr, int logc, int nrg, int tab_bytes, int tile_bytes,
    Gather gather, Produce prod) {
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    __shared__ double lds_waves[plan::kShortThreads / 64];
    __shared__ int lds_bad[plan::kShortThreads / 64];
    short_tiles<GT, CD, DEG, R, ONE, CACHED, FEW, PROD, false>(threadIdx.x, X, Xout, G, nbr, w, deg_any, n, d, ld, neg_lr, logc, nrg, tab_bytes,
                                                  tile_bytes, gather, ShortLds{lds_raw, lds_waves, lds_bad}, prod);
}

}  // namespace
}  // namespace psgd

#endif
