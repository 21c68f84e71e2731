// The ring walk, the register-only form of the model-averaging step (Sec. 2, Eq. 2) for the ring tables of
// Sec. 3 (Eq. 3, Eq. 8), and its kernel mix_step_kernel.  Included by psgd_kernels.hip only.
#ifndef PSGD_RING_WALK_H
#define PSGD_RING_WALK_H

#include "psgd_pace.h"
#include "psgd_short.h"

namespace psgd {
namespace {

// ---------------------------------------------------------------------------------------
// Ring walk: one lane, one column group, all n rows, registers only.
// Rows are visited in ring order p = 0..n-1.  `first` and `last` (positions 0 and n-1) stay
// in registers for the wrap-around, so every X element is loaded exactly once and, when
// X_out aliases X, always before the store that replaces it.
// ---------------------------------------------------------------------------------------
// All rows of the workgroup's column groups, sweep by sweep, as one stream of items: item q is position q mod n of sweep q / n.
// The X rows arrive in the order 0, n-1, 1, 2, .. n-2 of every sweep, so that at item q the stream stands at q + 2; loads, X and
// gradient, are issued D items ahead, and across sweeps nothing drains.  Loads and stores are unconditional (the waits
// then count operations instead of waiting for all of them); the stores of lanes that own nothing are dropped by the buffer's
// bounds check.  An item's addresses and weights are worked out behind the item before it, so that a row's place is free for the
// next load as soon as it has arrived: with them in between (LDS reads, 64-bit products) two rows took 2.3 us, not 1.6.
// PROD: also the next gradients; noise travels with the gradients.
template <typename GT, bool CD, bool RAGGED, int D, bool PROD>
__device__ __forceinline__ double ring_walk(const float* X, float* Xout, const GT* __restrict__ G, const RingEnt* ring, int n,
                                            int64_t d, Pitch ld, float neg_lr, const Sweeps& sweeps, int64_t my_sweeps, Pace* pace,
                                            double inv_n, const Produce& prod) {
    typedef typename RawG<GT>::T GR;
    const int64_t ncg = (d + kVec - 1) / kVec;
    int64_t sw = 0;
    WalkCols now = walk_cols<RAGGED>(sweeps, 0, ncg, d), nxt = walk_cols<RAGGED>(sweeps, my_sweeps > 1 ? 1 : 0, ncg, d);
    double total = 0.0;
    ColStats<RAGGED> stats;
    if (CD) stats.reset();
    // Position s of the X stream and position p of the gradients, of this sweep or (from n on) the next: the row's place and the lane's
    // in it.
    auto x_at = [&](int s) __attribute__((always_inline)) {
        const int64_t col = now.col, next_col = nxt.col;
        const bool over = s >= n;
        if (over) s -= n;
        if (s < 2) s = s ? n : 1;
        return X + ((uint64_t)(uint32_t)ring_row(ring + s - 1) * (uint64_t)ld.x + (uint64_t)(over ? next_col : col));
    };
    auto g_at = [&](int p) __attribute__((always_inline)) {
        const int64_t col = now.col, next_col = nxt.col;
        const bool over = p >= n;
        return G + ((uint64_t)(uint32_t)ring_row(ring + (over ? p - n : p)) * (uint64_t)ld.g + (uint64_t)(over ? next_col : col));
    };
    auto noise_at = [&](int p) __attribute__((always_inline)) {
        const int64_t col = now.col, next_col = nxt.col;
        const bool over = p >= n;
        return prod.noise + ((uint64_t)(uint32_t)ring_row(ring + (over ? p - n : p)) * (uint64_t)prod.ldn + (uint64_t)(over ? next_col : col));
    };
    auto lane_of = [&](int p) __attribute__((always_inline)) {
        const uint32_t at = now.at, next_at = nxt.at;
        return p >= n ? next_at : at;
    };
    f32x4 first = ld_x(lane_at(x_at(0), now.at)), last = ld_x(lane_at(x_at(1), now.at)), prev = last, cur = first, ahead = first;
    f32x4 x[D], noise[PROD ? D : 1];
    GR g[D];
#pragma unroll
    for (int u = 0; u < D; ++u) {
        x[u] = ld_x(lane_at(x_at(u + 2), lane_of(u + 2)));
        g[u] = ld_g_raw(lane_at(g_at(u), now.at));
        if (PROD) noise[u] = ld_x(lane_at(noise_at(u), now.at));
    }
    // The next item: where its loads come from, where its output goes, its weights.
    const float* from_x;
    const GT* from_g;
    const float* from_noise = nullptr;
    float *to, *to_g = nullptr;
    RingEnt e;
    int p = 0, items = 0;
    auto prepare = [&]() __attribute__((always_inline)) {
        e = ring_ent(ring + p);
        to = Xout + ((uint64_t)(uint32_t)e.row * (uint64_t)ld.o + (uint64_t)now.col);
        from_x = x_at(p + 2 + D);
        from_g = g_at(p + D);
        if (PROD) {
            from_noise = noise_at(p + D);
            to_g = prod.g + ((uint64_t)(uint32_t)e.row * (uint64_t)prod.ldg + (uint64_t)now.col);
        }
    };
    prepare();
    bool paced = true;
    auto item = [&](f32x4& xu, GR& gu, f32x4& nu) __attribute__((always_inline)) {
        wait_for_pace(pace, items, paced);
        __builtin_amdgcn_sched_barrier(0);
        const f32x4 in = set_apart(xu);
        const GR grad = set_apart(gu);
        f32x4 next_g;
        if (PROD) next_g = vfma(prod.c, cur, nu);
        xu = ld_x(lane_at(from_x, lane_of(p + 2 + D)));
        gu = ld_g_raw(lane_at(from_g, lane_of(p + D)));
        if (PROD) nu = ld_x(lane_at(from_noise, lane_of(p + D)));
        ++items;
        if (threadIdx.x == 0) lds_poke(&pace->done, items);
        __builtin_amdgcn_sched_barrier(0);
        f32x4 right = in;
        if (p >= n - 2) right = pick(p == n - 2, last, first);
        const f32x4 out = mix_one(e.w0, e.w1, e.w2, cur, prev, right, widen_g(grad), neg_lr);
        st_row(to, now.to, out);
        if (PROD) st_row(to_g, now.to, next_g);
        if (RAGGED && now.lo > 0 && now.lo < 4) {                  // one lane of the launch
#pragma unroll
            for (int k = 1; k < 4; ++k)
                if (k >= now.lo) {
                    __builtin_nontemporal_store(out[k], to + now.at + k);
                    if (PROD) __builtin_nontemporal_store(next_g[k], to_g + now.at + k);
                }
        }
        if (CD) stats.add(out);
        prev = cur;
        cur = right;
        if (p == n - 2) ahead = in;                                 // position 0 of the next sweep
        if (++p == n) {
            if (CD) {
                total += stats.result(inv_n, ColGroup{0, now.lo, 4});
                stats.reset();
            }
            first = cur = ahead;
            last = prev = in;                                       // its position n - 1
            p = 0;
            ++sw;
            now = nxt;
            nxt = walk_cols<RAGGED>(sweeps, sw + 1 < my_sweeps ? sw + 1 : my_sweeps - 1, ncg, d);
        }
        prepare();
        __builtin_amdgcn_sched_barrier(0);
    };
    // The first D items apart: a wait that they shared with the loop would count the operations since the start, which are fewer.
    const int64_t all = my_sweeps * n;
#pragma unroll
    for (int u = 0; u < D; ++u) item(x[u], g[u], noise[PROD ? u : 0]);
    for (int64_t i = D; i + D <= all; i += D)
#pragma unroll
        for (int u = 0; u < D; ++u) item(x[u], g[u], noise[PROD ? u : 0]);
    const int more = (int)(all % D);
#pragma unroll
    for (int u = 0; u + 1 < D; ++u)
        if (u < more) item(x[u], g[u], noise[PROD ? u : 0]);
    return total;
}


// The next gradients alone, for tables that are not walked: the same columns, row by row.
template <bool RAGGED>
__device__ __forceinline__ void produce_rows(const float* X, int n, int64_t d, int64_t ldx, const Sweeps& sweeps, int64_t my_sweeps,
                                             const Produce& prod) {
    const int64_t ncg = (d + kVec - 1) / kVec;
    for (int64_t sw = 0; sw < my_sweeps; ++sw) {
        const WalkCols c = walk_cols<RAGGED>(sweeps, sw, ncg, d);
        const ColGroup own{0, c.lo, 4};
        const int64_t at = c.col + c.at;
        for (int r0 = 0; r0 < n; r0 += 4) {
            f32x4 x[4], z[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t r = row_or_last(r0 + u, n);
                x[u] = ld_x(X + r * ldx + at);
                z[u] = ld_x(prod.noise + r * prod.ldn + at);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (r0 + u < n) st_cols(prod.g + (int64_t)(r0 + u) * prod.ldg + at, vfma(prod.c, x[u], z[u]), own);
        }
    }
}

// The step on long rows for any 3-slot table, one launch.  The workgroups stage and classify the table alike; one ring is walked, any
// other table goes through tiles (short_tiles; Tiles: how), an invalid one raises the flag and nothing is written.  A
// kernel of its own behind this one for the other tables, which for a ring classified the table once more and ended, took 4.5 to 7 us
// of every launch.
// CD = also reduce the consensus distance of the outputs into *gather.out.
// The column groups are split evenly over the persistent grid (plan::sweep_plan): every workgroup makes the
// same number of sweeps; the wavefronts that neither a sweep nor the tiles need are not launched.
// RAGGED: 4 may not divide d.  D: rows on their way per lane.  PROD: the next gradients too, whatever the table; APART: in front of the tiles,
// not with them (plan::tiles_produce).
struct Tiles {
    int form;                                                     // rows | cached << 4 | logc << 8: few scalar registers
    int nrg;
};
template <typename GT, bool CD, bool RAGGED, int D, bool PROD, bool APART>
__global__ __launch_bounds__(plan::kRingLanes + 64) void mix_step_kernel(const float* X, float* Xout, const GT* __restrict__ G,
                                                                         const int32_t* __restrict__ nbr,
                                                                         const float* __restrict__ w, int n, int64_t d, Pitch ld,
                                                                         float neg_lr, Sweeps sweeps, int lanes, int slot, int lead,
                                                                         Tiles tiles, Produce prod, Gather gather) {
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    __shared__ double lds_waves[(plan::kRingLanes + 64) / 64];
    __shared__ int lds_bad[(plan::kRingLanes + 64) / 64];
    __shared__ Pace pace;
    __shared__ int found;
    const int tid = threadIdx.x;
    RingEnt* ring = reinterpret_cast<RingEnt*>(lds_raw);
    if (tid == 0) pace = Pace{0, lead};
    // Uniform, but the compiler is told so only for bf16 gradients with the distance: it lays the walk out otherwise then (us, told / not:
    // 24 x 3 M 126.6 / 129.4, 16 x 4 100 003 117.8 / 119.6, 28 x 1.5 M 77.6 / 79.8; without the distance 24 x 3 M 126.1 / 121.8, fp32 128 x 8 M
    // with the next gradients 3476 / 3415).
    if (tid < 64) {
        const int k = n <= 64 ? stage_table<1>(nbr, w, n, lds_raw, tid) : stage_table<8>(nbr, w, n, lds_raw, tid);
        if (tid == 0) found = k;
    }
    lds_barrier();
    const int staged = found;
    const int kind = CD && sizeof(GT) == 2 ? __builtin_amdgcn_readfirstlane(staged) : staged;
    const int64_t ncg = (d + kVec - 1) / kVec;
    const int64_t my_sweeps = sweeps_of(sweeps, ncg);            // uniform
    constexpr bool BESIDE = PROD && !APART;
    if (APART && kind != kTableRing && tid < lanes) produce_rows<RAGGED>(X, n, d, ld.x, sweeps, my_sweeps, prod);
    if (kind == kTableRing) {
        if (tid >= lanes + 64) return;                           // whole wavefronts
        double total = 0.0;
        if (my_sweeps > 0) {
            if (tid >= lanes) keep_pace(&pace, slot, lead, (int)(my_sweeps * n), n);
            else total = ring_walk<GT, CD, RAGGED, D, PROD>(X, Xout, G, ring, n, d, ld, neg_lr, sweeps, my_sweeps, &pace, 1.0 / (double)n, prod);
        }
        if (CD) last_sum(gather, block_sum(total, lds_waves, lanes + 64));
        return;
    }
    const int tile_rows = tiles.form & 15, cached = tiles.form >> 4 & 15, logc_all = tiles.form >> 8;
    if (kind == kTableBad) {
        if (blockIdx.x == 0 && tid == 0) atomicOr(&g_status_word, 1);
        if (BESIDE && tid < tiles.nrg << logc_all) produce_tiles(tid, X, n, d, ld.x, logc_all, tiles.nrg, prod);
        if (CD) last_sum(gather, __builtin_nan(""));
        return;
    }
    if (tid >= tiles.nrg << logc_all) return;                     // whole wavefronts
    lds_barrier();                                               // the staged table has been read
    // Every form starts from values of its own.  With common ones the compiler hoists what the forms share to the front of the
    // choice and holds it through all of them: up to 27 vector registers spilled, in the tiles' loop too (us, so / now, fp32: 16 x 2 M
    // with the distance 80.3 / 75.6, 40 x 700 k 73.3 / 70.8, 24 x 6 M without 319 / 314, 32 x 1.4 M 109.4 / 105.3).
#define PSGD_TILES(R, CACHED)                                                                                              \
    do {                                                                                                                   \
        int t = tid, rows = n, logc = logc_all, nrg = tiles.nrg;                                                         \
        asm volatile("; tiles of %4 rows per lane, accesses %5" : "+v"(t), "+s"(rows), "+s"(logc), "+s"(nrg) : "n"(R), "n"(CACHED)); \
        short_tiles<GT, CD, 3, R, false, CACHED, false, BESIDE, true>(t, X, Xout, G, nbr, w, 3, rows, d, ld, neg_lr, logc, nrg,          \
                                                        plan::short_table_bytes(rows, 3), rows << (logc + 4), gather,            \
                                                        ShortLds{lds_raw, lds_waves, lds_bad}, prod);                      \
    } while (0)
    constexpr int kBoth = plan::kCachedLoads | plan::kCachedStores;
    if (tile_rows <= 2) {
        if (cached == kBoth) PSGD_TILES(2, kBoth);
        else PSGD_TILES(2, 0);
    } else if (tile_rows == 3) {
        if (cached == kBoth) PSGD_TILES(3, kBoth);
        else PSGD_TILES(3, 0);
    } else if constexpr (!BESIDE) {                              // with the noise four rows are more than the registers hold
        if (cached == kBoth) PSGD_TILES(4, kBoth);
        else if (sizeof(GT) == 2 && cached) PSGD_TILES(4, plan::kCachedLoads);
        else PSGD_TILES(4, 0);
    }
#undef PSGD_TILES
}

}  // namespace
}  // namespace psgd

#endif
