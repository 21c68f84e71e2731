// What the kernels share whose lanes walk the rows of long arrays, one column group each: how the workgroups of a die keep pace,
// where a lane stands in a sweep, and loads and stores from uniform addresses.  Included by psgd_kernels.hip only.
#ifndef PSGD_PACE_H
#define PSGD_PACE_H

#include "psgd_device.h"

namespace psgd {
namespace {

// ---------------------------------------------------------------------------------------
// What bounds a kernel whose lanes walk the rows is how the rows in flight lie in memory.  Left alone, the workgroups of one
// launch drift apart by whole sweeps; at any moment the chip then reads and writes all n rows of three arrays in 8 to 16 KB pieces,
// and plain dense arrays run at 5.1-5.4 TB/s whatever the batch, the workgroup or the order of the rows.  Kept on the same row,
// the 32 workgroups of one accelerator die, which take neighbouring column ranges, read and write one stretch of up to 480 KB of a
// row at a time, and the same traffic runs at 6.1-6.3 TB/s (one linear pass over the arrays: 6.4-6.7).  Two conditions: no more in
// flight than the memory needs (960 lanes with one row of each array on their way; with eight times that the gain is gone), and
// workgroups no more than about one and a half rows ahead of the mean (64 x 25.6 M fp32, us: 3130; two rows ahead 3290; unpaced 3800).
//
// Pacing: the last wavefront of every workgroup adds the workgroup's progress to one word per die (in that die's L2, hence cheap)
// and hands the mean progress of the die's workgroups back through LDS; a wavefront that is too far ahead of it waits.
// The wait decides nothing but when the loads go out: it is bounded, and after one that ran out the wavefront walks on unpaced (a
// workgroup that shares the chip with other kernels, or whose neighbours have not started).
// ---------------------------------------------------------------------------------------
// One word per launch slot and die, in a line of its own: the progress of the workgroups under way (upper 32 bits), those started and
// those done (16 bits each).  The last one done puts it back to zero; only launches on one slot that overlapped without a gap 2000
// times over would run out of the counts, and then lose the pace, not a result.
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
    constexpr unsigned long long kStarted = 1ull << 16, kProgress = 1ull << 32;
    const int die = __builtin_amdgcn_s_getreg(20 | 31 << 11) & (kXcds - 1);   // hwreg XCC_ID: which die this is
    if ((threadIdx.x & 63) != 0) return;
    unsigned long long* word = g_pace[slot][die];
    unsigned long long v = pace_add(word, kStarted);
    auto started = [&] { return (unsigned)(v >> 16) & 0xFFFFu; };
    auto done = [&] { return (unsigned)v & 0xFFFFu; };
    // A workgroup that starts late counts from the sweep the others are in, so that it neither holds them up nor falls out of step.
    const unsigned before = started() - 1 - done();
    const int from = before ? (int)((unsigned)(v >> 32) / before) / sweep * sweep : 0;
    int at = 0;
    for (int now = from;;) {
        v = pace_add(word, (unsigned long long)(now - at) * kProgress);   // one operation whether there is progress or not: a plain
        at = now;                                                        // load might be served by the compute unit's own cache
        if (now - from >= total) break;
        const unsigned under_way = started() - done();
        if (under_way) lds_poke(&pace->allowed, (int)(4u * (unsigned)(v >> 32) / under_way) - 4 * from + lead);
        __builtin_amdgcn_s_sleep(1);
        now = from + lds_peek(&pace->done);
    }
    v = pace_add(word, 1 - (unsigned long long)at * kProgress);            // out of the mean
    if (started() == done()) {
        unsigned long long seen = v;
        __hip_atomic_compare_exchange_strong(word, &seen, 0ull, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// A wavefront in front of its item number `items`: waits while the workgroup is too far ahead, unless a wait has run out before.
__device__ __forceinline__ void wait_for_pace(Pace* pace, int items, bool& paced) {
    if (!paced) return;
    int spin = 0;
    while (lds_peek(&pace->allowed) < 4 * items && ++spin < plan::kPaceSpins) __builtin_amdgcn_s_sleep(1);
    paced = spin < plan::kPaceSpins;
}
// Sweeps in which this workgroup has columns.
__device__ __forceinline__ int64_t sweeps_of(const Sweeps& sweeps, int64_t ncg) {
    int64_t mine = sweeps.count;
    while (mine > 0 && sweeps.base(mine - 1) >= ncg) --mine;
    return mine;
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

}  // namespace
}  // namespace psgd

#endif
