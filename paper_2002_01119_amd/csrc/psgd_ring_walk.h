// The ring walk, the register-only form of the model-averaging step (Sec. 2, Eq. 2) for the ring tables of
// Sec. 3 (Eq. 3, Eq. 8), and its kernel mix_step_kernel.  Included by psgd_kernels.hip only.
#ifndef PSGD_RING_WALK_H
#define PSGD_RING_WALK_H

#include "psgd_device.h"
#include "psgd_short.h"

namespace psgd {
namespace {

// ---------------------------------------------------------------------------------------
// Ring walk: one lane, one column group, all n rows, registers only.
// Rows are visited in ring order p = 0..n-1.  `first` and `last` (positions 0 and n-1) stay
// in registers for the wrap-around, so every X element is loaded exactly once and, when
// X_out aliases X, always before the store that replaces it.
//
// What bounds it is how the rows in flight lie in memory.  Left alone, the workgroups of one launch drift apart by whole sweeps;
// at any moment the chip then reads and writes all n rows of three arrays in 8 KB pieces, and plain dense arrays run at
// 5.1-5.4 TB/s whatever the batch, the workgroup or the order of the rows.  Kept on the same row, the 32 workgroups of one
// accelerator die, which take neighbouring column ranges, read and write one stretch of 230 KB of a row at a time, and the same
// traffic runs at 6.1-6.2 TB/s (x + a g over 64 x 25.6 M fp32: 3740 -> 3240 us; one linear pass over the arrays: 2950-3080).  Two
// conditions: no more in flight than the memory needs (448 lanes with two rows of each array on their way; with eight rows the
// gain is gone), and workgroups no more than about one and a half steps of two rows ahead of the mean (half a step: 5.6; four: 5.7).
//
// Pacing: the last wavefront of every workgroup adds the workgroup's progress to one word per die (in that die's L2, hence cheap)
// and hands the mean progress of the die's workgroups back through LDS; a wavefront that is too far ahead of it waits.
// The wait decides nothing but when the loads go out: it is bounded, and after one that ran out the wavefront walks on unpaced (a
// workgroup that shares the chip with other kernels, or whose neighbours have not started).
// ---------------------------------------------------------------------------------------
// One word per launch slot and die, in a line of its own: the progress of the workgroups under way (upper 40 bits), those started and
// those done (12 bits each).  The last one done puts it back to zero.
__device__ unsigned long long g_pace[plan::kPaceSlots][kXcds][16];

// The operations are performed by the L2 of the die the workgroup runs on, which is what they are meant to reach: no more than
// workgroup scope is asked for (a wider one would go past the L2 to memory and back).
__device__ __forceinline__ unsigned long long pace_add(unsigned long long* word, unsigned long long v) {
    return __hip_atomic_fetch_add(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) + v;
}
__device__ __forceinline__ int lds_peek(int* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ void lds_poke(int* p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }

// What the workers and the pacing wavefront of a workgroup exchange: items done by the first wavefront, and how far the
// workgroup may be, in quarter items.
struct Pace {
    int done, allowed;
};

// The pacing wavefront: ends when the workers have made all `total` items; `sweep` items are one sweep.
__device__ __forceinline__ void keep_pace(Pace* pace, int slot, int lead, int total, int sweep) {
    constexpr unsigned long long kStarted = 1ull << 12, kProgress = 1ull << 24;
    const int die = __builtin_amdgcn_s_getreg(20 | 31 << 11) & (kXcds - 1);   // hwreg XCC_ID: which die this is
    if ((threadIdx.x & 63) != 0) return;
    unsigned long long* word = g_pace[slot][die];
    unsigned long long v = pace_add(word, kStarted);
    auto started = [&] { return (unsigned)(v >> 12) & 0xFFFu; };
    auto done = [&] { return (unsigned)v & 0xFFFu; };
    // A workgroup that starts late counts from the sweep the others are in, so that it neither holds them up nor falls out of step.
    const unsigned before = started() - 1 - done();
    const int from = before ? (int)((unsigned)(v >> 24) / before) / sweep * sweep : 0;
    int at = 0;
    for (int now = from;;) {
        v = pace_add(word, (unsigned long long)(now - at) * kProgress);   // one operation whether there is progress or not: a plain
        at = now;                                                        // load might be served by the compute unit's own cache
        if (now - from >= total) break;
        const unsigned under_way = started() - done();
        if (under_way) lds_poke(&pace->allowed, (int)(4u * (unsigned)(v >> 24) / under_way) - 4 * from + lead);
        __builtin_amdgcn_s_sleep(1);
        now = from + lds_peek(&pace->done);
    }
    v = pace_add(word, 1 - (unsigned long long)at * kProgress);            // out of the mean
    if (started() == done()) {
        unsigned long long seen = v;
        __hip_atomic_compare_exchange_strong(word, &seen, 0ull, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// Where a lane is in one sweep: the workgroup's first column (uniform), the lane's distance from it in elements for loads, the same
// in bytes for stores (beyond the buffer where the lane owns no whole group: such a store is dropped), and what it owns.
constexpr uint32_t kDropStore = 0x80000000u;
struct WalkCols {
    int64_t col;
    uint32_t at, to;
    int lo, hi;
};
template <bool RAGGED>
__device__ __forceinline__ WalkCols walk_cols(const Sweeps& sweeps, int64_t sw, int64_t ncg, int64_t d) {
    const int64_t base = sweeps.base(sw), end = base + sweeps.chunk < ncg ? base + sweeps.chunk : ncg;   // uniform
    const int64_t mine = base + (int64_t)threadIdx.x, cg = mine < end ? mine : end - 1;   // a lane without a group shadows the last one
    const ColGroup g = col_group(cg, d);
    WalkCols c;
    c.col = RAGGED && base * 4 > d - 4 ? d - 4 : base * 4;
    c.at = (uint32_t)(g.col - c.col);
    c.lo = mine < end ? g.lo : 4;
    c.hi = 4;
    c.to = c.lo == 0 ? c.at * 4 : kDropStore;
    return c;
}

// 128 bits at a lane's byte offset from a uniform address; an offset beyond the 1 GiB that the buffer is said to have is dropped.
__device__ __forceinline__ void st_row(float* row, uint32_t bytes, f32x4 v) {
    constexpr int kNonTemporal = 2, kRaw32 = 4 << 15;   // cache policy bit; descriptor: plain 32-bit data, no swizzle
    const __amdgpu_buffer_rsrc_t buf = __builtin_amdgcn_make_buffer_rsrc(row, 0, 1 << 30, kRaw32);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), buf, (int)bytes, 0, kNonTemporal);
}
// A loaded value in registers of its own, so that the next load goes where this one arrived.  Left to the compiler, the value stays
// there as the next item's neighbour and the load under way is what gets moved at the end of the loop, which waits for it.
template <typename V> __device__ __forceinline__ V set_apart(V v) {
    V o;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(V) / 4); ++k) {
        uint32_t t;
        asm volatile("v_mov_b32 %0, %1" : "=v"(t) : "v"(v[k]));
        o[k] = __builtin_bit_cast(decltype(+v[k]), t);
    }
    return o;
}
__device__ __forceinline__ f32x4 pick(bool a, f32x4 x, f32x4 y) { return a ? x : y; }
// A uniform address and the lane's distance from it in elements, kept in 32 bits.
template <typename T> __device__ __forceinline__ const T* lane_at(const T* base, uint32_t elements) {
    return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + (uint32_t)(elements * sizeof(T)));
}

// The gradient producer of the delay-by-one schedule beside the step (Sec. 4, Eq. 14; the stand-in G_next = c X + noise): the walk holds
// every row of X in registers at the moment its output is made, so the pair moves 20 bytes per element instead of 24.
struct Produce {
    const float* noise;
    float* g;
    int64_t ldn, ldg;
    float c;
};

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
        if (paced) {
            int spin = 0;
            while (lds_peek(&pace->allowed) < 4 * items && ++spin < plan::kPaceSpins) __builtin_amdgcn_s_sleep(1);
            paced = spin < plan::kPaceSpins;
        }
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
// CD = also reduce the consensus distance of the outputs into partials[blockIdx.x].
// The column groups are split evenly over the persistent grid (plan::sweep_plan): every workgroup makes the
// same number of sweeps; the wavefronts that neither a sweep nor the tiles need are not launched.
// RAGGED: 4 may not divide d.  D: rows on their way per lane.  PROD: the next gradients too, whatever the table.
struct Tiles {
    int rows, cached, logc, nrg, tab_bytes, tile_bytes;
};
template <typename GT, bool CD, bool RAGGED, int D, bool PROD>
__global__ __launch_bounds__(plan::kRingLanes + 64) void mix_step_kernel(const float* X, float* Xout, const GT* __restrict__ G,
                                                                         const int32_t* __restrict__ nbr,
                                                                         const float* __restrict__ w, int n, int64_t d, Pitch ld,
                                                                         float neg_lr, Sweeps sweeps, int lanes, int slot, int lead,
                                                                         Tiles tiles, Produce prod, double* __restrict__ partials) {
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    __shared__ double lds_waves[(plan::kRingLanes + 64) / 64];
    __shared__ int lds_bad[(plan::kRingLanes + 64) / 64];
    __shared__ Pace pace;
    const int tid = threadIdx.x;
    const Lds l = carve(lds_raw, n);
    if (tid == 0) pace = Pace{0, lead};
    const int kind = stage_table(nbr, w, n, l, blockDim.x);      // contains barriers
    const int64_t ncg = (d + kVec - 1) / kVec;
    int64_t my_sweeps = sweeps.count;
    while (my_sweeps > 0 && sweeps.base(my_sweeps - 1) >= ncg) --my_sweeps;   // uniform
    if (PROD && kind != kTableRing && tid < lanes) produce_rows<RAGGED>(X, n, d, ld.x, sweeps, my_sweeps, prod);
    if (kind == kTableBad) {
        if (blockIdx.x == 0 && tid == 0) atomicOr(&g_status_word, 1);
        if (CD && tid == 0) partials[blockIdx.x] = __builtin_nan("");
        return;
    }
    if (kind == kTableGeneral) {
        if (tid >= tiles.nrg << tiles.logc) return;              // whole wavefronts
        lds_barrier();                                           // the staged table has been read
#define PSGD_TILES(R, CACHED)                                                                                              \
    short_tiles<GT, CD, 3, R, false, CACHED, false>(X, Xout, G, nbr, w, 3, n, d, ld, neg_lr, tiles.logc, tiles.nrg,        \
                                                    tiles.tab_bytes, tiles.tile_bytes, partials,                          \
                                                    ShortLds{lds_raw, lds_waves, lds_bad})
        constexpr int kBoth = plan::kCachedLoads | plan::kCachedStores;
        if (tiles.rows <= 2) {
            if (tiles.cached == kBoth) PSGD_TILES(2, kBoth);
            else PSGD_TILES(2, 0);
        } else if (tiles.rows == 3) {
            if (tiles.cached == kBoth) PSGD_TILES(3, kBoth);
            else PSGD_TILES(3, 0);
        } else {
            if (tiles.cached == kBoth) PSGD_TILES(4, kBoth);
            else if (sizeof(GT) == 2 && tiles.cached) PSGD_TILES(4, plan::kCachedLoads);
            else PSGD_TILES(4, 0);
        }
#undef PSGD_TILES
        return;
    }
    if (tid >= lanes + 64) return;                               // whole wavefronts
    double total = 0.0;
    if (my_sweeps > 0) {
        if (tid >= lanes) keep_pace(&pace, slot, lead, (int)(my_sweeps * n), n);
        else total = ring_walk<GT, CD, RAGGED, D, PROD>(X, Xout, G, l.ring, n, d, ld, neg_lr, sweeps, my_sweeps, &pace, 1.0 / (double)n, prod);
    }
    if (CD) {
        const double bs = block_sum_any(total, lds_waves, lanes + 64);
        if (tid == 0) partials[blockIdx.x] = bs;
    }
}

}  // namespace
}  // namespace psgd

#endif
