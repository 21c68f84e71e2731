// Device-side building blocks shared by the kernels of libpsgd (gfx950 / CDNA4): launch constants, column-group
// value types and their loads and stores, the LDS layout of the staged mixing table and its classification
// (one ring or not), workgroup sums, the running sums of the consensus distance (Sec. 3), and the even split of
// the column groups over a persistent grid.  Included by psgd_kernels.hip only (one translation unit).
#ifndef PSGD_DEVICE_H
#define PSGD_DEVICE_H

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "psgd.h"
#include "psgd_internal.h"

namespace psgd {
namespace {

constexpr int kThreads = 256;        // 4 wavefronts of 64 lanes
constexpr int kRingThreads = 768;    // workgroup of the streaming kernels on long rows (12 wavefronts in lockstep, one per CU)
constexpr int kDeepThreads = 1024;   // workgroup of the tiled kernel: 16 wavefronts, four per SIMD, which is what keeps the slot
                                     // loop's LDS round trips and arithmetic hidden
constexpr int kTileThreads = 512;    // the same with the distance: 8 wavefronts with up to 256 registers
constexpr int kUnroll = 8;           // rows whose loads are in flight together per lane
using plan::kMaxGrid;                // upper bound on persistent workgroups (partials buffer sizing)
constexpr int kGridPerCu = 4;        // persistent workgroups per compute unit (16 waves per CU)
constexpr int kXcds = 8;             // accelerator dies of an MI355X: consecutive workgroups go to consecutive dies
// LDS a workgroup may ask for: a compute unit has 160 KB.  The large workgroups are alone on their CU.
constexpr size_t kLdsCapLarge = 160 * 1024 - 1024;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ int g_status_word = 0;

// ---------------------------------------------------------------------------------------
// A lane owns a group of kVec adjacent columns: one 128-bit access per row (64-bit for bf16 gradients).
//
// Rows may start at any element and hold any number of columns: gfx950 takes such accesses at any element alignment
// (the compiler's default for this target, unaligned-access-mode), so alignment decides nothing; the types below only
// tell the compiler.  A row of d columns has (d + 3) / 4 groups.  If 4 does not divide d the last one covers columns
// d-4 .. d-1, of which the first few belong to the group before: they are loaded and computed but not stored (in place
// they may be read after that group has replaced them; the values are dropped), [lo, hi) is what the lane owns.  Rows
// of fewer than four columns are one group, loaded element by element.
// Measured on rows at odd addresses, before (a column per lane wherever d, a pitch or a base was odd) and now: step with
// bf16 gradients on 16 x 4 100 003 227 -> 144 us, fp32 on 16 x 32 000 003 1406 -> 1264 (aligned 1141), 5 slots on
// 64 x 8 000 001 2032 -> 1230, distance of 64 x 25 600 001 1738 -> 988 (aligned 981); aligned rows unchanged.
// ---------------------------------------------------------------------------------------
constexpr int kVec = 4;
typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));

__device__ __forceinline__ f32x4 splat4(float v) { return (f32x4){v, v, v, v}; }
__device__ __forceinline__ float vfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ f32x4 vfma(float a, f32x4 b, f32x4 c) {
    return __builtin_elementwise_fma(splat4(a), b, c);
}

// X, G and X_out are each touched once per step: mark the accesses non-temporal so they
// stream through the caches instead of displacing one another.  CACHED: without the hint, for launches where a line is
// wanted again soon, by the neighbouring tile or by the next call (plan::cached_accesses).
template <bool CACHED = false> __device__ __forceinline__ f32x4 ld_x(const float* p) {
    if (CACHED) return *reinterpret_cast<const f32x4_any*>(p);
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(p));
}
template <bool CACHED = false> __device__ __forceinline__ void st_x(float* p, f32x4 v) {
    if (CACHED) *reinterpret_cast<f32x4_any*>(p) = v;
    else __builtin_nontemporal_store(v, reinterpret_cast<f32x4_any*>(p));
}

// A gradient group as it arrives from memory, widened only where it is used: a value that is converted right
// after its load would make the wavefront wait for that load (and every earlier one) on the spot, which defeats
// loads that are issued early to travel during other work; bf16 groups also take half the registers this way.
// bfloat16 is the upper half of an fp32, so widening is a 16-bit shift and exact.
template <typename GT> struct RawG;
template <> struct RawG<float> { typedef f32x4 T; };
template <> struct RawG<uint16_t> { typedef u32x2 T; };
template <bool CACHED = false> __device__ __forceinline__ f32x4 ld_g_raw(const float* p) { return ld_x<CACHED>(p); }
template <bool CACHED = false> __device__ __forceinline__ u32x2 ld_g_raw(const uint16_t* p) {
    if (CACHED) return *reinterpret_cast<const u32x2_any*>(p);
    return __builtin_nontemporal_load(reinterpret_cast<const u32x2_any*>(p));
}
__device__ __forceinline__ f32x4 widen_g(f32x4 v) { return v; }
__device__ __forceinline__ f32x4 widen_g(u32x2 b) {
    return (f32x4){__uint_as_float(b.x << 16), __uint_as_float(b.x & 0xFFFF0000u),
                   __uint_as_float(b.y << 16), __uint_as_float(b.y & 0xFFFF0000u)};
}
template <typename GT> __device__ __forceinline__ f32x4 ld_g(const GT* p) { return widen_g(ld_g_raw(p)); }
__device__ __forceinline__ float widen_1(float v) { return v; }
__device__ __forceinline__ float widen_1(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

struct ColGroup {
    int64_t col;   // first column
    int lo, hi;    // the lane's columns are col + lo .. col + hi - 1; lo == hi: no group of its own
};
__device__ __forceinline__ ColGroup col_group(int64_t cg, int64_t d) {
    ColGroup c;
    const int64_t full = d >> 2;
    c.col = cg * 4;
    c.lo = 0;
    c.hi = 4;
    if (cg >= full) {
        const int rem = (int)(d & 3);
        c.col = d >= 4 ? d - 4 : 0;
        c.hi = d >= 4 ? 4 : rem;
        c.lo = cg == full && rem ? c.hi - rem : c.hi;
    }
    return c;
}
// FEW: rows of fewer than four columns (d of them).
template <bool FEW, bool CACHED = false> __device__ __forceinline__ f32x4 ld_cols(const float* p, int64_t d) {
    if (!FEW) return ld_x<CACHED>(p);
    return (f32x4){p[0], d > 1 ? p[1] : 0.0f, d > 2 ? p[2] : 0.0f, 0.0f};
}
template <bool FEW, bool CACHED = false> __device__ __forceinline__ f32x4 ld_cols_raw(const float* p, int64_t d) {
    return ld_cols<FEW, CACHED>(p, d);
}
template <bool FEW, bool CACHED = false> __device__ __forceinline__ u32x2 ld_cols_raw(const uint16_t* p, int64_t d) {
    if (!FEW) return ld_g_raw<CACHED>(p);
    return (u32x2){(uint32_t)p[0] | (d > 1 ? (uint32_t)p[1] << 16 : 0u), d > 2 ? (uint32_t)p[2] : 0u};
}
// The same for kernels that are built apart for rows that 4 divides (RAGGED false), where a group is whole or none.
template <bool RAGGED> __device__ __forceinline__ ColGroup col_group_of(int64_t cg, int64_t ncg, int64_t d) {
    if (RAGGED) return col_group(cg, d);
    return cg < ncg ? ColGroup{cg * 4, 0, 4} : ColGroup{0, 4, 4};
}
template <bool CACHED = false> __device__ __forceinline__ void st_cols(float* p, f32x4 v, const ColGroup& c) {
    if (c.lo == 0 && c.hi == 4) {
        st_x<CACHED>(p, v);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k >= c.lo && k < c.hi) __builtin_nontemporal_store(v[k], p + k);
    }
}

template <bool RAGGED> __device__ __forceinline__ void st_cols_of(float* p, f32x4 v, const ColGroup& c) {
    if (RAGGED) st_cols(p, v, c);
    else if (c.lo == 0) st_x(p, v);
}

// Two barriers that are lighter than __syncthreads(), which also waits until every global load and store the
// wavefront has issued is complete.  That wait is exactly what the step kernels must avoid: their loads are
// issued early to travel during other work, and their stores need never be waited for.
//   lockstep_barrier: keeps the workgroup's wavefronts on the same batch of rows; no data passes between them.
//   lds_barrier: the wavefront's own LDS reads and writes are complete (its global ones may still travel), then
//   the barrier: LDS written before it by any wavefront is read after it by any other.
__device__ __forceinline__ void lockstep_barrier() { __builtin_amdgcn_s_barrier(); }
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One output group.  The operation order is part of the boundary's contract.
__device__ __forceinline__ f32x4 mix_one(float w0, float w1, float w2, f32x4 self, f32x4 left, f32x4 right,
                                         f32x4 g, float neg_lr) {
    f32x4 acc = self * w0;
    acc = vfma(w1, left, acc);
    acc = vfma(w2, right, acc);
    return vfma(neg_lr, g, acc);
}

// Row pitches in elements: row i of X starts at X + i * x, of X_out at X_out + i * o, of G at
// G + i * g.  Dense arrays have all three equal to d; larger pitches let a caller interleave
// the rows of several arrays across the whole HBM (see the note on placement in the header).
struct Pitch {
    int64_t x, o, g;
};

// The gradient producer of the delay-by-one schedule beside the step (Sec. 4, Eq. 14; the stand-in G_next = c X + noise): the step has
// every row of X at hand when its output is made, so the pair moves 20 bytes per element instead of 24.
struct Produce {
    const float* noise;
    float* g;
    int64_t ldn, ldg;
    float c;
};

// One ring position, packed so the walk fetches it with a single 128-bit LDS read.
struct __attribute__((aligned(16))) RingEnt {
    int row;
    float w0, w1, w2;
};

// One slot of a table row as the tiled and the short-row kernel keep it in LDS: where the source row starts inside the tile
// (nbr * lanes-per-row, in column groups) and its weight.
struct __attribute__((aligned(8))) TileSlot {
    uint32_t off;
    float w;
};

// LDS of the 3-slot step kernel (dynamic, sized by the launcher): RingEnt ring[n], entries[n] | uint32_t words[n], the latter two for the
// classification.
__host__ __device__ inline size_t lds_classify_bytes(int n) { return (size_t)n * (2 * sizeof(RingEnt) + sizeof(uint32_t)); }

// Ring entries are the same for every lane; moving them to scalar registers keeps the row
// offsets and weights out of the vector register file.
__device__ __forceinline__ int ring_row(const RingEnt* e) { return __builtin_amdgcn_readfirstlane(e->row); }
__device__ __forceinline__ RingEnt ring_ent(const RingEnt* e) {
    RingEnt r;
    r.row = __builtin_amdgcn_readfirstlane(e->row);
    r.w0 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(e->w0)));
    r.w1 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(e->w1)));
    r.w2 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(e->w2)));
    return r;
}

// Row `r` of n, or the last one for a lane without a row (which then repeats that row's loads).
__device__ __forceinline__ int row_or_last(int r, int n) { return r < n ? r : n - 1; }

enum TableKind { kTableBad = 0, kTableRing = 1, kTableGeneral = 2 };

// Check the table, decide whether it is a single ring, and if so put its entries into `ring` in walk order.  By one wavefront, K
// learners to a lane at a time: its LDS accesses need no barriers, and the workgroup's others do not take turns with it.
//
// A ring here means: slot 0 of row i is i itself, and the left/right slots are mutually
// consistent (the right neighbour's left is i and vice versa), which makes "right" a
// bijection, and following it from learner 0 visits all n learners.  The last property is
// decided by parallel list ranking (pointer doubling) toward learner 0's left neighbour;
// the resulting distances are the ring positions.
// From the kernel's start to here 1.0 us for up to 64 learners; by all 16 wavefronts, with a barrier for each step, 2.6: 24 x 1 M 54.0 / 52.0 us,
// 64 x 430 k with bf16 gradients 54.8 / 52.9, 32 x 786 433 54.5 / 52.8.
template <int K>
__device__ __forceinline__ int stage_table(const int32_t* __restrict__ nbr, const float* __restrict__ w, int n, char* lds, int lane) {
    RingEnt* ring = reinterpret_cast<RingEnt*>(lds);
    RingEnt* entries = ring + n;                                  // by learner
    uint32_t* words = reinterpret_cast<uint32_t*>(entries + n);
    unsigned most = 0, odd = 0;
    for (int from = 0; from < n; from += 64 * K) {
        int self[K], left[K], right[K];
        RingEnt e[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            e[k].row = row_or_last(from + 64 * k + lane, n);
            self[k] = nbr[3 * e[k].row];
            left[k] = nbr[3 * e[k].row + 1];
            right[k] = nbr[3 * e[k].row + 2];
            e[k].w0 = w[3 * e[k].row];
            e[k].w1 = w[3 * e[k].row + 1];
            e[k].w2 = w[3 * e[k].row + 2];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            for (unsigned v : {(unsigned)self[k], (unsigned)left[k], (unsigned)right[k]}) most = v > most ? v : most;
            odd |= (unsigned)(self[k] ^ e[k].row);
            words[e[k].row] = (unsigned)left[k] | (unsigned)right[k] << 16;
            entries[e[k].row] = e[k];
        }
    }
    if (__any(most >= (unsigned)n)) return kTableBad;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const unsigned tail = words[0] & 0xFFFFu;
    // K learners at a time, so that their reads travel together; a lane without one repeats the last.
    for (int from = lane; from < n + lane; from += 64 * K) {
        unsigned both[K], l[K], r[K];
#pragma unroll
        for (int k = 0; k < K; ++k) both[k] = words[row_or_last(from + 64 * k, n)];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            l[k] = words[both[k] & 0xFFFFu];
            r[k] = words[both[k] >> 16];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const unsigned i = (unsigned)row_or_last(from + 64 * k, n);
            odd |= ((r[k] & 0xFFFFu) ^ i) | ((l[k] >> 16) ^ i);
        }
    }
    if (__any(odd != 0)) return kTableGeneral;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // From here per learner: one that is to the right of it (lower half), not beyond the tail, and how many steps that is.
    for (int i = lane; i < n; i += 64) words[i] = (unsigned)i == tail ? tail : (words[i] >> 16) | 1u << 16;
    for (int span = 1; span < n; span <<= 1) {
        for (int from = lane; from < n + lane; from += 64 * K) {  // of some the new word is read already, which is further along
            unsigned far[K], then[K];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int k = 0; k < K; ++k) far[k] = words[row_or_last(from + 64 * k, n)];
#pragma unroll
            for (int k = 0; k < K; ++k) then[k] = words[far[k] & 0xFFFFu];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int k = 0; k < K; ++k) words[row_or_last(from + 64 * k, n)] = (far[k] & 0xFFFF0000u) + then[k];
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int i = lane; i < n; i += 64) odd |= (words[i] & 0xFFFFu) ^ tail;
    if (__any(odd != 0)) return kTableGeneral;
#pragma unroll 4
    for (int i = lane; i < n; i += 64) ring[n - 1 - (int)(words[i] >> 16)] = entries[i];
    return kTableRing;
}

// ---------------------------------------------------------------------------------------
// Consensus distance.  Per column: with pivot s = X[0, j],
//   sum_i (x_i - xbar)^2 = sum_i (x_i - s)^2 - (sum_i (x_i - s))^2 / n,
// one pass, differences and sums in fp64 (the difference of two fp32 values is exact in
// fp64 unless their exponents are more than 29 apart, and because the pivot is one of the
// points the subtraction cancels at most a factor n).
// ---------------------------------------------------------------------------------------
// Sum over a wavefront, all of whose lanes take part; every lane gets it.  Lane to lane through the vector unit's own shifts (a row of 16
// lanes, then row to row): through LDS (64-bit shuffles) the six steps were 0.3 us of every small launch with a distance.
template <int CTRL, int ROWS> __device__ __forceinline__ double add_shifted(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xF, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xF, true);
    return v + __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);   // lanes without a source add zero
}
__device__ __forceinline__ double row_sum(double v) {           // of 16 lanes, in the last of them
    v = add_shifted<0x111, 0xF>(v);
    v = add_shifted<0x112, 0xF>(v);
    v = add_shifted<0x114, 0xF>(v);
    return add_shifted<0x118, 0xF>(v);
}
__device__ __forceinline__ double from_lane(double v, int lane) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)b, lane), hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = row_sum(v);
    v = add_shifted<0x142, 0xA>(v);                              // lane 15 to row 1, lane 47 to row 3
    v = add_shifted<0x143, 0xC>(v);                              // lane 31 to rows 2 and 3
    return from_lane(v, 63);
}

// Sum over the workgroup's T lanes (whole wavefronts, at most 16 of them), valid in its first wavefront; the per-wavefront sums are
// added in a fixed order.
__device__ __forceinline__ double block_sum(double v, double* lds_waves, int T) {
    v = wave_sum(v);
    const int tid = threadIdx.x;
    if ((tid & 63) == 0) lds_waves[tid >> 6] = v;
    lds_barrier();
    return tid < 64 ? from_lane(row_sum(tid < T / 64 ? lds_waves[tid] : 0.0), 15) : 0.0;
}

// ---------------------------------------------------------------------------------------
// The distance's last sum, over the workgroups, by the workgroup that is done last.  Every workgroup writes its partial sum past the caches and then
// draws a ticket: from one counter, or where many workgroups would queue at it (16 ns each) from one of plan::kTicketLeaves first, whose
// last one goes on to it.  The last of all reads the partial sums and adds them in a fixed order whichever workgroup it is.  Nobody waits,
// and every counter ends at zero (plan::Ticket).
// Against the second kernel (us of a launch of 256 lanes a workgroup and little work): 64 workgroups 4.3 / 4.3, 157 4.1 / 4.2, 256 of 8 us 9.3 / 8.8, 512
// 6.8 / 6.6: as long on the device, but a launch less, which is 2.6 us of host time on calls that are bound by it.
// ---------------------------------------------------------------------------------------
__device__ unsigned g_tickets[2][plan::kTicketCounters][32];   // for each array of partial sums; a counter in each 128-byte line
struct Gather {
    double* partials;
    double* out;
    int array;
};
__device__ __forceinline__ void last_sum(const Gather& g, double mine) {       // `mine`: of the workgroup, in its first wavefront
    const int tid = threadIdx.x;
    if (tid >= 64) return;
    const unsigned count = gridDim.x;
    unsigned (*counters)[32] = g_tickets[g.array];                // not named in the lambda, which would take its address from a table in memory
    auto draw = [&](plan::Ticket t) {                             // whether this is the last of t.of to come
        return atomicInc(&counters[t.at][0], (unsigned)t.of - 1) == (unsigned)t.of - 1;
    };
    int last = 0;
    if (tid == 0) {
        __hip_atomic_store(g.partials + blockIdx.x, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // written before the ticket is drawn
        last = (!plan::ticket_leaves(count) || draw(plan::ticket_leaf(blockIdx.x, count))) && draw(plan::ticket_root(count));
    }
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    asm volatile("" ::: "memory");
    double sum = 0.0;
    for (unsigned from = 0; from < count; from += 512) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const unsigned at = from + 64 * k + tid;
            v[k] = at < count ? __hip_atomic_load(g.partials + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += v[k];
    }
    sum = wave_sum(sum);
    if (tid == 0) *g.out = sum;
}
// The same, or left to sum_partials_kernel behind this one.
__device__ __forceinline__ void last_sum_or_none(const Gather& g, double mine) {
    if (g.out)
        last_sum(g, mine);
    else if (threadIdx.x == 0)
        g.partials[blockIdx.x] = mine;
}
__device__ __forceinline__ void acc_diff(double* a, double* b, f32x4 x, const double* s) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double df = (double)x[k] - s[k];
        a[k] += df;
        b[k] = fma(df, df, b[k]);
    }
}
__device__ __forceinline__ void pivot_of(f32x4 x, double* s) {
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = (double)x[k];
}
__device__ __forceinline__ void floats_of(f32x4 x, float* f) {
#pragma unroll
    for (int k = 0; k < 4; ++k) f[k] = x[k];
}

// Running sums of one lane's column group; the first value it is given becomes the pivot (kept as
// the fp32 value it is).  Unless the group may be owned in part (RAGGED) the squares of its columns share one
// accumulator: only their total is needed, and three fp64 accumulators less are five to seven registers less in the ring walk
// (without the tiles beside it 103 against 110 with four rows on their way, 121 against 126 with six).
template <bool RAGGED>
struct ColStats {
    f32x4 s;
    double a[4], sq[RAGGED ? 4 : 1];
    int have;
    __device__ __forceinline__ void reset() {
        have = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) a[k] = sq[RAGGED ? k : 0] = 0.0;
    }
    __device__ __forceinline__ void add(f32x4 x) {
        if (!have) {
            s = x;
            have = 1;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double df = (double)x[k] - (double)s[k];
                a[k] += df;
                sq[RAGGED ? k : 0] = fma(df, df, sq[RAGGED ? k : 0]);
            }
        }
    }
    // over the columns the lane owns
    __device__ __forceinline__ double result(double inv_n, const ColGroup& c) const {
        double t = RAGGED ? 0.0 : sq[0];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (!RAGGED || (k >= c.lo && k < c.hi)) t += (RAGGED ? sq[RAGGED ? k : 0] : 0.0) - a[k] * a[k] * inv_n;
        return RAGGED || c.lo == 0 ? t : 0.0;
    }
};

// ---------------------------------------------------------------------------------------
// Tiles whose rows are spread over row groups: T = nrg * C lanes, C = 1 << logc column groups wide, lane (rg, lane) sees
// rows rg, rg + nrg, ... of column group `lane`.  What follows combines the row groups' values per column through LDS
// arrays laid out [4][nrg][C].
// ---------------------------------------------------------------------------------------
// Calls f(k, l, first, step, reach) with every lane: column k of lane l is the lane's, which takes row groups first,
// first + step, ...; the lanes that share a column differ in the bits reach, 2 reach, .. 32 of their number, and first = 0
// in one of them.  The lanes of a wavefront read L neighbouring columns of 64 / L row groups, so that the few columns of
// a tile with many rows still occupy many lanes.
template <typename F>
__device__ __forceinline__ void row_group_columns(int logc, int nrg, int T, const F& f) {
    const int C = 1 << logc, most = nrg >= 8 ? 4 : 6;
    const int logl = logc < most ? logc : most, parts = 64 >> logl;
    for (int idx = threadIdx.x; idx < 4 * C * parts; idx += T) {   // whole wavefronts
        const int col = (idx >> 6 << logl) + (idx & ((1 << logl) - 1));
        f(col >> logc, col & (C - 1), (idx >> logl) & (parts - 1), parts, 1 << logl);
    }
}

// The column sums a_q of the row groups, each against its own pivot p_q, to the squares about the column's mean: with
// P = p_0, D_q = p_q - P and m_q rows in group q,
//     sum_i (o_i - P)   = sum_q (a_q + m_q D_q)
//     sum_i (o_i - P)^2 = sum_q (sq_q + 2 D_q a_q + m_q D_q^2)
// exactly; in fp64 the corrections are of the size of the sums themselves, as every pivot is one of the values, and
// equal values give exactly 0.  Returns this lane's part of what is to be added to the sum of all sq_q.
// FULL: every column of the tile, which starts at column group `first`, exists.
template <bool FULL>
__device__ __forceinline__ double row_group_merge(const double* sums, const float* pivots, int logc, int nrg, int n, int T,
                                                  double inv_n, int64_t first, int64_t d) {
    const int each = n / nrg, more = n % nrg;                   // rows of group q: each, one more if q < more
    double total = 0.0;
    row_group_columns(logc, nrg, T, [&](int k, int l, int q0, int step, int reach) {
        const int at0 = ((k * nrg) << logc) + l;
        const double p0 = (double)pivots[at0];
        double at = 0.0, corr = 0.0;
#pragma unroll 4
        for (int q = q0; q < nrg; q += step) {
            const double aq = sums[at0 + (q << logc)];
            const double dq = (double)pivots[at0 + (q << logc)] - p0;
            const double tq = fma((double)(each + (q < more ? 1 : 0)), dq, aq);
            at += tq;
            corr = fma(dq, tq + aq, corr);
        }
        for (int off = reach; off < 64; off <<= 1) {
            at += __shfl_xor(at, off, 64);
            corr += __shfl_xor(corr, off, 64);
        }
        const ColGroup c = col_group(FULL ? 0 : first + l, d);
        if (q0 == 0 && (FULL || (k >= c.lo && k < c.hi))) total += corr - at * at * inv_n;
    });
    return total;
}

// A tile's whole distance from every lane's sums against its pivot.  Contains a barrier; the LDS arrays must be free
// when it is called and are being read when it returns.
__device__ __forceinline__ double row_group_distance(double* sums, float* pivots, int logc, int nrg, int n, int T, int rg,
                                                     int lane, double inv_n, const double (&a)[4], const double (&sq)[4],
                                                     f32x4 pv, const ColGroup& c, int64_t first, int64_t d) {
    double total = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        sums[((k * nrg + rg) << logc) + lane] = a[k];
        pivots[((k * nrg + rg) << logc) + lane] = pv[k];
        if (k >= c.lo && k < c.hi) total += sq[k];
    }
    lds_barrier();
    return total + row_group_merge<false>(sums, pivots, logc, nrg, n, T, inv_n, first, d);
}

// The column groups are split evenly over the persistent grid (plan::sweep_plan): every workgroup makes the
// same number of sweeps, lanes beyond the chunk idle.
struct Sweeps {
    int64_t count, chunk;
    // first column group of this workgroup in sweep sw
    __device__ __forceinline__ int64_t base(int64_t sw) const {
        return (sw * gridDim.x + plan::die_contiguous_slot(blockIdx.x, gridDim.x, kXcds)) * chunk;
    }
};
// Computed by the launcher (the device would pay two 64-bit divisions per lane for it).
inline Sweeps make_sweeps(int64_t ncg, int grid, int threads, bool even = true) {
    const plan::SweepPlan p = plan::sweep_plan(ncg, grid, threads, even);
    return Sweeps{p.count, p.chunk};
}

}  // namespace
}  // namespace psgd

#endif
