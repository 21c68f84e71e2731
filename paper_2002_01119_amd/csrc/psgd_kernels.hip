// libpsgd's HIP translation unit (gfx950 / CDNA4): the launchers and C entry points for the model-averaging step
//     X_out[i,:] = sum_s w[i,s] * X[nbr[i,s],:] - lr * G[i,:]            (Sec. 2, Eq. 2)
// and for the consensus distance sum_i ||x_i - xbar||^2 (Sec. 3).  The kernels live in the headers included
// below: psgd_device.h (shared building blocks), psgd_pace.h (workgroups of a die in step), psgd_short.h (any table: short rows, few
// learners, most tables of other than three slots), psgd_ring_walk.h (3-slot tables on long rows, rings in registers only),
// psgd_tiled.h (long rows, other slot counts, numbers of learners that fill its LDS tiles), psgd_streams.h (global averaging, distance,
// gradient producer, reference streams, table builder).
//
// The step is bound by HBM traffic (about 7 flops against 10-12 bytes per element), so the
// design goal is to touch every X, G and X_out byte exactly once:
//   * the update is separable by column, so a lane owns a group of 4 adjacent columns
//     (one 128-bit access per row) and sees all n rows of it;
//   * when the table describes a single ring (every table of Sec. 3 does), the lane walks
//     the ring in position order holding three consecutive rows in registers, so each
//     neighbour read is a register move, not a memory access, and the update may run in
//     place because a row is only written after its old value is in registers;
//   * any other table goes through [n x columns] tiles in LDS (a neighbour read is an LDS read), with the
//     next tiles travelling from HBM through registers while the current one is computed; a tile is
//     complete in LDS before its first output is stored, so this path too may run in place.
// Short rows, where a launch is bound by latency, take tiles for every table (psgd_short.h).
// Tables live in device memory and are validated and, on long rows, classified (one ring or not) by the kernels.
// Workgroups are persistent, so table staging is paid once per launch.  On long rows there is one large workgroup per compute
// unit (up to 1024 lanes for the ring walk, 512 or 1024 for the tiled kernel, 768 for the kernels in psgd_streams.h).  What the
// HBM delivers then depends on the order the chip visits the rows in: the ring walk keeps the workgroups of a die on the same
// row (psgd_ring_walk.h), which is worth 15-20 % on plain dense arrays.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdint>
#include <mutex>

#include "psgd.h"
#include "psgd_internal.h"

// Partial sums of psgd_mix_step_cd_static, the entry point for callers that cannot allocate: one double
// per persistent workgroup.  Every GPU holds its own copy of this array at its own address; host code
// never uses the name as a pointer, only the address hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) double scratch[PSGD_STATIC_SLOTS];

#include "psgd_device.h"
#include "psgd_pace.h"
#include "psgd_short.h"
#include "psgd_tiled.h"
#include "psgd_ring_walk.h"
#include "psgd_streams.h"

namespace psgd {
namespace {

// ---------------------------------------------------------------------------------------
// Host helpers.
// ---------------------------------------------------------------------------------------
struct DeviceInfo {
    int cus = 0;
    double* partials = nullptr;        // hipMalloc'ed on first use: kMaxGrid partials
    hipEvent_t partials_idle = nullptr;     // recorded on the previous user's stream when another stream takes over
    hipStream_t partials_stream = nullptr;  // the stream (not under capture) that used `partials` last
    bool partials_used = false;
    std::mutex partials_mutex;         // held from acquire_partials until the caller has launched
    double* static_partials = nullptr;  // device address of ::scratch on this GPU (psgd_mix_step_cd_static)
    double* host_result = nullptr;      // pinned host memory, hipHostMalloc'ed on first use (psgd_consensus_dist),
    double* host_result_dev = nullptr;  // and its address on the device
    std::mutex host_result_mutex;       // held from the launch until the word has been read
};
constexpr int kMaxDevices = 64;
DeviceInfo g_dev[kMaxDevices];
std::mutex g_dev_mutex;

int hip_fail(hipError_t e, const char* what) {
    return fail(PSGD_EHIP, "%s: %s", what, hipGetErrorString(e));
}

// Looks up (and caches) the current device's compute-unit count.
int device_info(DeviceInfo** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(PSGD_EHIP, "device index %d unsupported", dev);
    std::lock_guard<std::mutex> lock(g_dev_mutex);
    DeviceInfo& di = g_dev[dev];
    if (di.cus == 0) {
        int cus = 0;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
        di.cus = cus > 0 ? cus : 1;
    }
    *out = &di;
    return PSGD_OK;
}

bool stream_is_capturing(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st != hipStreamCaptureStatusNone;
}

// The per-device partials buffer of the fused-distance and consensus calls, handed to work that is about
// to be enqueued on `s`.  It is allocated on the first call on a device; allocation is not allowed while a
// stream is being captured, so a first call made under capture is refused with an explanation instead of
// invalidating the capture.  All calls on a device share the buffer.  As long as they come on one stream the
// stream orders them and nothing is done here (no runtime call at all: short launches are bound by host time).
// When a call arrives on another stream than the previous one, an event is recorded behind everything enqueued
// so far on the previous stream and the new stream is made to wait for it (on the device, not on the host), so
// two streams that both gather a distance are serialised instead of racing.  Streams under capture are left
// alone: the order of graph launches is the caller's.
// `use` holds the buffer until the caller has launched: a thread that came in between would make its stream wait for what stood on this one
// before the launch.
int acquire_partials(DeviceInfo* di, hipStream_t s, double** out, std::unique_lock<std::mutex>* use) {
    *use = std::unique_lock<std::mutex>(di->partials_mutex);
    if (di->partials && di->partials_used && di->partials_stream == s) {
        *out = di->partials;
        return PSGD_OK;
    }
    const bool capturing = stream_is_capturing(s);
    if (!di->partials) {
        if (capturing)
            return fail(PSGD_EHIP, "the per-device partials buffer is allocated on first use, which stream capture "
                                   "forbids: make one fused-distance or consensus call on this device before capturing");
        hipError_t e = hipMalloc(reinterpret_cast<void**>(&di->partials), sizeof(double) * kMaxGrid);
        if (e != hipSuccess) return hip_fail(e, "hipMalloc(partials)");
        e = hipEventCreateWithFlags(&di->partials_idle, hipEventDisableTiming);
        if (e != hipSuccess) {
            (void)hipFree(di->partials);
            di->partials = nullptr;
            return hip_fail(e, "hipEventCreateWithFlags");
        }
    }
    *out = di->partials;
    if (capturing) return PSGD_OK;                // captured work: ordered by whoever launches the graphs
    if (di->partials_used && !stream_is_capturing(di->partials_stream)) {
        // another stream used the buffer last: wait for all it has been given so far.  If that stream no longer
        // exists the record fails; its work may still be running, so the whole device is waited for instead.
        hipError_t e = hipEventRecord(di->partials_idle, di->partials_stream);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, di->partials_idle, 0);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            e = hipDeviceSynchronize();
            if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize(partials)");
        }
    }
    di->partials_stream = s;
    di->partials_used = true;
    return PSGD_OK;
}

// Device address of the static scratch array on the current GPU, looked up once per device.
int static_partials(DeviceInfo* di, double** out) {
    std::lock_guard<std::mutex> lock(g_dev_mutex);
    if (!di->static_partials) {
        double* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!ptr) return fail(PSGD_EHIP, "hipGetSymbolAddress(scratch) returned a null address");
        di->static_partials = ptr;
    }
    *out = di->static_partials;
    return PSGD_OK;
}

inline bool aligned_to(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

inline bool overlaps(const void* a, size_t abytes, const void* b, size_t bbytes) {
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return a0 < b0 + bbytes && b0 < a0 + abytes;
}

inline int persistent_grid(const DeviceInfo& di, int64_t work_items, int per_cu, int threads = kThreads) {
    return plan::persistent_grid(di.cus, work_items, per_cu, threads);
}

using plan::deg_grid;

// True if any row of A ([n] rows of ra bytes, lda bytes apart) shares a byte with any row of B.
bool rows_overlap(const void* A, int64_t lda, size_t ra, const void* B, int64_t ldb, size_t rb, int n) {
    if (ra == 0 || rb == 0) return false;
    const size_t span_a = (size_t)(n - 1) * (size_t)lda + ra, span_b = (size_t)(n - 1) * (size_t)ldb + rb;
    if (!overlaps(A, span_a, B, span_b)) return false;
    if ((size_t)lda == ra && (size_t)ldb == rb) return true;  // both dense: the spans are the arrays
    if (lda == ldb) {
        // Equal pitches P: row i of A meets row j of B iff  D - ra < (i - j) P < D + rb  with D = B - A.
        // Take the largest k = i - j (|k| <= n - 1) below the upper bound; smaller k only move away
        // from the lower one.
        const int64_t P = lda;
        const int64_t D = (int64_t)(reinterpret_cast<uintptr_t>(B) - reinterpret_cast<uintptr_t>(A));
        const int64_t t = D + (int64_t)rb - 1;
        int64_t k = t >= 0 ? t / P : -((-t + P - 1) / P);       // floor(t / P)
        if (k > n - 1) k = n - 1;
        if (k < -(int64_t)(n - 1)) return false;
        return k * P > D - (int64_t)ra;
    }
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(A), b0 = reinterpret_cast<uintptr_t>(B);
    for (int i = 0; i < n; ++i) {
        const uintptr_t ai = a0 + (uintptr_t)i * (uintptr_t)lda;
        for (int j = 0; j < n; ++j) {
            const uintptr_t bj = b0 + (uintptr_t)j * (uintptr_t)ldb;
            if (ai < bj + rb && bj < ai + ra) return true;
        }
    }
    return false;
}

// Workgroups of `fn` (256 threads, `lds_bytes` of dynamic LDS) that fit one compute unit, as the
// runtime computes it from the kernel's registers and LDS; remembered per (kernel, LDS size).
int resident_per_cu(const void* fn, size_t lds_bytes, int threads = kThreads) {
    struct Entry {
        const void* fn;
        size_t lds;
        int occ;
    };
    static std::mutex mu;
    static Entry cache[128];
    static int used = 0;
    std::lock_guard<std::mutex> lock(mu);
    for (int i = 0; i < used; ++i)
        if (cache[i].fn == fn && cache[i].lds == lds_bytes) return cache[i].occ;
    int q = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&q, fn, threads, lds_bytes) != hipSuccess || q < 1) q = 1;
    if (used < 128) cache[used++] = Entry{fn, lds_bytes, q};
    return q;
}

// True if the double at p shares a byte with any row of B.
bool scalar_overlaps(const double* p, const void* B, int64_t ldb, size_t rb, int n) {
    const uintptr_t p0 = reinterpret_cast<uintptr_t>(p), b0 = reinterpret_cast<uintptr_t>(B);
    for (int j = 0; j < n; ++j) {
        const uintptr_t bj = b0 + (uintptr_t)j * (uintptr_t)ldb;
        if (p0 < bj + rb && bj < p0 + sizeof(double)) return true;
    }
    return false;
}

// A workgroup gets 64 KB of dynamic LDS by default; a kernel that is to be launched with more is opted in.
// Once per kernel and device (the attribute belongs to the kernel's code object on that device).
int allow_lds(const void* fn, size_t lds_bytes) {
    if (lds_bytes <= 64 * 1024 - 256) return PSGD_OK;
    struct Entry {
        const void* fn;
        int device;
    };
    static std::mutex mu;
    static Entry done[512];
    static int used = 0;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    std::lock_guard<std::mutex> lock(mu);
    for (int i = 0; i < used; ++i)
        if (done[i].fn == fn && done[i].device == device) return PSGD_OK;
    // the most this library ever asks for (the kernels' few hundred bytes of static LDS come on top of it)
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsCapLarge);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(MaxDynamicSharedMemorySize)");
    if (used < 512) done[used++] = Entry{fn, device};
    return PSGD_OK;
}

// Long rows take the large lockstep workgroup: at least `sweeps` column groups per lane of one such
// workgroup per CU.
inline bool long_rows(const DeviceInfo& di, int64_t column_groups, int sweeps = 2) {
    return column_groups >= (int64_t)di.cus * kRingThreads * sweeps;
}

// Lanes of a workgroup that takes `sw.chunk` column groups at a time, without a wavefront that has none.
inline int sweep_threads(const Sweeps& sw) { return ((int)sw.chunk + 63) / 64 * 64; }

// Every row of X and X_out starts on `bytes` (a power of two): a 128-byte line, or a lane's 16 bytes.
inline bool rows_start_on(int bytes, const float* X, const float* X_out, const Pitch& ld) {
    return aligned_to(X, bytes) && aligned_to(X_out, bytes) && ld.x % (bytes / 4) == 0 && ld.o % (bytes / 4) == 0;
}
inline bool rows_on_lines(const float* X, const float* X_out, const Pitch& ld) { return rows_start_on(128, X, X_out, ld); }

// Short rows: one launch of the short-row kernel.
template <typename GT, bool CD, int DEG, int R, bool ONE, int CACHED, bool FEW, bool PROD = false>
int launch_short_t(const DeviceInfo& di, const plan::ShortPlan& p, hipStream_t s, const float* X, float* X_out, const GT* G,
                   const int32_t* nbr, const float* w, int deg, int n, int64_t d, Pitch ld, float neg_lr, const Gather& gather,
                   const Produce& prod = {}) {
    const void* fn = reinterpret_cast<const void*>(mix_short_kernel<GT, CD, DEG, R, ONE, CACHED, FEW, PROD>);
    if (int rc = allow_lds(fn, p.lds)) return rc;
    const int grid = ONE ? (int)p.tiles : plan::short_grid(p, di.cus, CD ? plan::kShortSlots : INT32_MAX);
    hipLaunchKernelGGL((mix_short_kernel<GT, CD, DEG, R, ONE, CACHED, FEW, PROD>), dim3(grid), dim3(p.threads), p.lds, s, X,
                       X_out, G, nbr, w, deg, n, d, ld, neg_lr, p.logc, p.nrg, p.tab_bytes, p.tile_bytes, gather, prod);
    return PSGD_OK;
}

template <typename GT, bool CD, int DEG>
int launch_short(const DeviceInfo& di, const plan::ShortPlan& p, hipStream_t s, const float* X, float* X_out, const GT* G,
                 const int32_t* nbr, const float* w, int deg, int n, int64_t d, Pitch ld, float neg_lr, const Gather& gather,
                 const Produce* prod) {
    static_assert(plan::kShortSlots <= PSGD_STATIC_SLOTS && plan::kShortSlots <= kMaxGrid, "one partial per workgroup");
    const bool on_lines = rows_on_lines(X, X_out, ld);
    const int cached = plan::cached_accesses(p, plan::counted_bytes(n * d, sizeof(GT), prod != nullptr, on_lines), on_lines, sizeof(GT) == 2);
    constexpr int kBoth = plan::kCachedLoads | plan::kCachedStores;
#define PSGD_SHORT(DEG, R, ONE, CACHED, FEW)                                                                              \
    return launch_short_t<GT, CD, DEG, R, ONE, CACHED, FEW>(di, p, s, X, X_out, G, nbr, w, deg, n, d, ld, neg_lr, gather)
    // Only what the plan asks for is built: four rows and one tile are three or four learners on wide tiles, one row and
    // several tiles a single learner; without a variant the accesses keep their hints.
#define PSGD_SHORT_ONE(R)                                                                                                 \
    case R:                                                                                                               \
        if constexpr (R != 4)                                                                                             \
            if (cached) PSGD_SHORT(DEG, R, true, kBoth, false);                                                           \
        PSGD_SHORT(DEG, R, true, 0, false)
#define PSGD_SHORT_LOOP(R)                                                                                                \
    case R:                                                                                                               \
        if constexpr (R != 1)                                                                                             \
            if (cached == kBoth) PSGD_SHORT(DEG, R, false, kBoth, false);                                                 \
        if constexpr (R != 1 || CD)                                                                                       \
            if (cached == plan::kCachedLoads) PSGD_SHORT(DEG, R, false, plan::kCachedLoads, false);                       \
        PSGD_SHORT(DEG, R, false, 0, false)
    if constexpr (sizeof(GT) == 4 && DEG == 3) {
        if (prod) {
#define PSGD_SHORT_PROD(R, ONE, CACHED)                                                                                   \
    return launch_short_t<GT, CD, 3, R, ONE, CACHED, false, true>(di, p, s, X, X_out, G, nbr, w, deg, n, d, ld, neg_lr, gather, *prod)
#define PSGD_SHORT_PROD_ONE(R)                                                                                            \
    case R:                                                                                                               \
        if constexpr (R != 4)                                                                                             \
            if (cached) PSGD_SHORT_PROD(R, true, kBoth);                                                                  \
        PSGD_SHORT_PROD(R, true, 0)
#define PSGD_SHORT_PROD_LOOP(R)                                                                                           \
    case R:                                                                                                               \
        if (cached == kBoth) PSGD_SHORT_PROD(R, false, kBoth);                                                            \
        if (cached == plan::kCachedLoads) PSGD_SHORT_PROD(R, false, plan::kCachedLoads);                                  \
        PSGD_SHORT_PROD(R, false, 0)
            if (p.one) {
                switch (p.rows) {
                    PSGD_SHORT_PROD_ONE(2);
                    PSGD_SHORT_PROD_ONE(4);
                    PSGD_SHORT_PROD_ONE(6);
                    PSGD_SHORT_PROD_ONE(8);
                }
            } else {
                switch (p.rows) {
                    PSGD_SHORT_PROD_LOOP(2);
                    PSGD_SHORT_PROD_LOOP(3);
                    PSGD_SHORT_PROD_LOOP(4);
                }
            }
            return fail(PSGD_EINVAL, "no short-row kernel of %d rows per lane with the next gradients", p.rows);
#undef PSGD_SHORT_PROD_LOOP
#undef PSGD_SHORT_PROD_ONE
#undef PSGD_SHORT_PROD
        }
    }
    if (d < kVec) PSGD_SHORT(0, 2, true, 0, true);
    if (p.one) {
        switch (p.rows) {
            PSGD_SHORT_ONE(2);
            PSGD_SHORT_ONE(4);
            PSGD_SHORT_ONE(6);
            PSGD_SHORT_ONE(8);
        }
    } else {
        switch (p.rows) {
            PSGD_SHORT_LOOP(1);
            PSGD_SHORT_LOOP(2);
            PSGD_SHORT_LOOP(3);
            PSGD_SHORT_LOOP(4);
        }
    }
#undef PSGD_SHORT_LOOP
#undef PSGD_SHORT_ONE
#undef PSGD_SHORT
    return fail(PSGD_EINVAL, "no short-row kernel of %d rows per lane", p.rows);
}

// Long rows, 3-slot tables: one launch of mix_step_kernel, one workgroup per compute unit.
std::atomic<unsigned> g_paced_launches{0};   // each takes the next of the pace words
int next_pace_slot() { return (int)(g_paced_launches.fetch_add(1, std::memory_order_relaxed) % plan::kPaceSlots); }
template <typename GT, bool CD, bool RAGGED, int D, bool PROD, bool APART = false>
int launch_ring_t(const plan::SweepPlan& sp, int grid, const plan::ShortPlan& tp, int cached, hipStream_t s, const float* X, float* X_out,
                  const GT* G, const int32_t* nbr, const float* w, int n, int64_t d, Pitch ld, float neg_lr, const Gather& gather,
                  const Produce& prod) {
    size_t lds = tp.lds > plan::kRingLds ? tp.lds : plan::kRingLds;
    if (lds < lds_classify_bytes(n)) lds = lds_classify_bytes(n);
    const int lanes = plan::ring_threads({1, sp.chunk}, plan::kRingLanes);
    const int threads = lanes + 64 > tp.threads ? lanes + 64 : tp.threads;
    if (int rc = allow_lds(reinterpret_cast<const void*>(mix_step_kernel<GT, CD, RAGGED, D, PROD, APART>), lds)) return rc;
    hipLaunchKernelGGL((mix_step_kernel<GT, CD, RAGGED, D, PROD, APART>), dim3(grid), dim3(threads), lds, s, X, X_out, G, nbr, w, n, d, ld, neg_lr,
                       Sweeps{sp.count, sp.chunk}, lanes,
                       next_pace_slot(), plan::pace_lead(D, PROD),
                       Tiles{tp.rows | cached << 4 | tp.logc << 8, tp.nrg}, prod, gather);
    return PSGD_OK;
}
template <typename GT, bool CD>
int launch_ring(const DeviceInfo& di, const char* name, hipStream_t s, const float* X, float* X_out, const GT* G, const int32_t* nbr,
                const float* w, int n, int64_t d, Pitch ld, float neg_lr, const Gather& gather, const Produce* prod) {
    const int64_t ncg = (d + kVec - 1) / kVec;
    const int grid = di.cus < kMaxGrid ? di.cus : kMaxGrid;   // the sweeps split any row evenly
    if (CD && grid > plan::kShortSlots)                       // one partial per workgroup must fit the smallest buffer
        return fail(PSGD_EINVAL, "%s: this launch needs %d partial sums, the buffer holds %d", name, grid, (int)plan::kShortSlots);
    const plan::SweepPlan sp = plan::sweep_plan(ncg, grid, plan::kRingLanes);
    const bool on_lines = rows_on_lines(X, X_out, ld);
    const plan::ShortPlan tp = plan::ring_tiles(n, ncg, CD, prod != nullptr, sizeof(GT) == 4 && !on_lines);
    const int cached = plan::cached_accesses(tp, (int64_t)n * d * (int64_t)(8 + sizeof(GT)), on_lines, sizeof(GT) == 2);
#define PSGD_RING(RAGGED, D, ...)                                                                                         \
    launch_ring_t<GT, CD, RAGGED, D, __VA_ARGS__>(sp, grid, tp, cached, s, X, X_out, G, nbr, w, n, d, ld, neg_lr, gather, \
                                                  prod ? *prod : Produce{})
    const int depth = plan::ring_depth(sp, n);
    // With one or two rows on their way the ragged form costs nothing (64 x 25.6 M 3137 / 3129 us); with more, a lane's own work shows
    // (512 x 205 k with six rows, in one run: whole groups 246, the ragged form 265).
    if constexpr (sizeof(GT) == 4) {
        if (prod) {
            const bool one = plan::ring_depth_produce(sp) == 1;
            if (plan::tiles_produce(n)) return one ? PSGD_RING(true, 1, true) : PSGD_RING(true, 2, true);
            return one ? PSGD_RING(true, 1, true, true) : PSGD_RING(true, 2, true, true);
        }
    }
    switch (depth) {
        case 1: return PSGD_RING(true, 1, false);
        case 2: return PSGD_RING(true, 2, false);
        case 4: return d % kVec ? PSGD_RING(true, 4, false) : PSGD_RING(false, 4, false);
        case 6: return d % kVec ? PSGD_RING(true, 6, false) : PSGD_RING(false, 6, false);
    }
#undef PSGD_RING
    return fail(PSGD_EINVAL, "%s: no ring walk of this depth", name);
}

// Enqueues G = c X_prev + noise on n rows of d columns, in dispatch order, one 128-bit access per lane and array: what is in flight
// stays a narrow window that moves through the arrays, which the HBM serves at 6.4 TB/s; lanes that walk the rows, or 4096 persistent
// workgroups that stride over the array, reach 4.9-5.4 (128 x 8 M dense 2460 -> 1930 us).  A launch counts its lanes in 32 bits: beyond
// kShortMostTiles workgroups a row they stride.
int enqueue_producer(const char* name, const float* xp, int64_t ldx, const float* noise, int64_t ldn, float* g, int64_t ldg, int n,
                     int64_t d, float c, hipStream_t s) {
    if (n > 1 && ldx == d && ldn == d && ldg == d) {           // dense: one row
        d *= n;
        n = 1;
    }
    const int64_t need = ((d + kVec - 1) / kVec + kThreads - 1) / kThreads;
    const dim3 grid((unsigned)(need < plan::kShortMostTiles ? need : plan::kShortMostTiles), (unsigned)n);
    if (d < kVec) hipLaunchKernelGGL(synth_grad_kernel<true>, grid, dim3(kThreads), 0, s, xp, ldx, noise, ldn, g, ldg, d, c);
    else hipLaunchKernelGGL(synth_grad_kernel<false>, grid, dim3(kThreads), 0, s, xp, ldx, noise, ldn, g, ldg, d, c);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? PSGD_OK : hip_fail(e, name);
}

// Pitches are in elements of the array they belong to.
template <typename GT>
int mix_step_impl(const char* name, const float* X, int64_t ldx, float* X_out, int64_t ldo, const GT* G, int64_t ldg,
                  const int32_t* nbr, const float* w, int n, int64_t d, float lr, int delay_mode, bool want_cd,
                  double* cd_out, void* stream, int deg = 3, bool no_alloc = false, const Produce* prod = nullptr) {
    clear_error();
    if (!X || !X_out || !G || !nbr || !w || (want_cd && !cd_out)) return fail(PSGD_EINVAL, "%s: null pointer", name);
    if (n < 1 || n > PSGD_MAX_N) return fail(PSGD_EINVAL, "%s: n=%d outside 1..%d", name, n, (int)PSGD_MAX_N);
    if (deg < 1 || deg > PSGD_MAX_DEG || (int64_t)n * deg > PSGD_MAX_TABLE)
        return fail(PSGD_EINVAL, "%s: deg=%d outside 1..%d or n*deg > %d", name, deg, (int)PSGD_MAX_DEG,
                    (int)PSGD_MAX_TABLE);
    if (d < 0) return fail(PSGD_EINVAL, "%s: d=%lld is negative", name, (long long)d);
    if (delay_mode != 0 && delay_mode != 1) return fail(PSGD_EINVAL, "%s: delay_mode=%d", name, delay_mode);
    if (n > 1 && (ldx < d || ldo < d || ldg < d))
        return fail(PSGD_EINVAL, "%s: a row pitch is smaller than d=%lld", name, (long long)d);
    if (n == 1) ldx = ldo = ldg = d;
    if (!aligned_to(X, 4) || !aligned_to(X_out, 4) || !aligned_to(G, sizeof(GT)) || !aligned_to(nbr, 4) ||
        !aligned_to(w, 4) || (want_cd && !aligned_to(cd_out, 8)))
        return fail(PSGD_EALIGN, "%s: pointer not aligned to its element size", name);
    const int64_t ldmax = ldx > ldo ? (ldx > ldg ? ldx : ldg) : (ldo > ldg ? ldo : ldg);
    if (ldmax > 0 && (int64_t)n > INT64_MAX / 8 / ldmax) return fail(PSGD_EINVAL, "%s: n * pitch overflows", name);
    const size_t xrow = (size_t)d * sizeof(float), grow = (size_t)d * sizeof(GT);
    const int64_t bx = ldx * (int64_t)sizeof(float), bo = ldo * (int64_t)sizeof(float), bg = ldg * (int64_t)sizeof(GT);
    if (static_cast<const void*>(X) == static_cast<const void*>(X_out) && ldx == ldo) {
        if (delay_mode == 1)
            return fail(PSGD_EALIAS, "%s: delay-by-one keeps X read-only, X_out must be another buffer", name);
    } else if (rows_overlap(X, bx, xrow, X_out, bo, xrow, n)) {
        return fail(PSGD_EALIAS, "%s: X_out partially overlaps X", name);
    }
    if (rows_overlap(G, bg, grow, X_out, bo, xrow, n)) return fail(PSGD_EALIAS, "%s: X_out overlaps G", name);
    if (want_cd && (scalar_overlaps(cd_out, X_out, bo, xrow, n) || scalar_overlaps(cd_out, X, bx, xrow, n) ||
                    scalar_overlaps(cd_out, G, bg, grow, n)))
        return fail(PSGD_EALIAS, "%s: the distance output overlaps a data buffer", name);
    hipStream_t s = static_cast<hipStream_t>(stream);
    DeviceInfo* di = nullptr;
    if (d == 0 && !want_cd) return PSGD_OK;
    if (int rc = device_info(&di)) return rc;
    // Where the per-workgroup partial sums of the distance go: the library's own buffer (allocated on first
    // use, shared by every call on the device, streams serialised), or the static array of the entry point
    // that may not allocate (no serialisation: that would need an event).
    double* partials = nullptr;
    std::unique_lock<std::mutex> use;
    if (want_cd) {
        if (no_alloc) {
            if (int rc = static_partials(di, &partials)) return rc;
        } else if (int rc = acquire_partials(di, s, &partials, &use)) {
            return rc;
        }
    }
    if (d == 0) {
        hipLaunchKernelGGL(no_distance_kernel, dim3(1), dim3(1), 0, s, cd_out);
        const hipError_t e0 = hipGetLastError();
        if (e0 != hipSuccess) return hip_fail(e0, "no_distance_kernel");
        return PSGD_OK;
    }
    const float neg_lr = -lr;
    const Pitch ld{ldx, ldo, ldg};
    const Gather gather{partials, cd_out, no_alloc ? 1 : 0};
    const int64_t ncg = (d + kVec - 1) / kVec;
    // 3-slot tables: where plan::walk_rows says so mix_step_kernel, which walks one ring (every table of Sec. 3) and takes any other table
    // through tiles; below it the short-row kernel.
    // Tables of other slot counts: the short-row kernel, but for long rows where plan::tiled_rows says so.
    const bool quads = d % kVec == 0 && rows_start_on(16, X, X_out, ld);
    const int room = !long_rows(*di, ncg) ? 0 : rows_on_lines(X, X_out, ld) ? 2 : quads && long_rows(*di, ncg, 4) ? 1 : 0;
    const bool ring = deg == 3 && plan::walk_rows(n, ncg, di->cus, want_cd, prod != nullptr);
    const bool tiled = deg != 3 && long_rows(*di, ncg) && plan::tiled_rows(n, deg, want_cd, room);
    bool produced = ring;                                        // the next gradients, by the same kernel
    if (ring) {
        if (int rc = want_cd ? launch_ring<GT, true>(*di, name, s, X, X_out, G, nbr, w, n, d, ld, neg_lr, gather, prod)
                             : launch_ring<GT, false>(*di, name, s, X, X_out, G, nbr, w, n, d, ld, neg_lr, gather, prod))
            return rc;
    } else if (!tiled) {
        const plan::ShortPlan sp = d < 4 ? plan::short_shape(n, deg, 1, want_cd, true, 0, 2)
                                         : plan::short_plan(n, deg, ncg, di->cus, want_cd, quads);
        const Produce* beside = prod && deg == 3 && d >= kVec && plan::short_produces(sp, n * d, rows_on_lines(X, X_out, ld)) ? prod : nullptr;
        produced = beside != nullptr;
        int rc;
        if (want_cd && deg == 3) rc = launch_short<GT, true, 3>(*di, sp, s, X, X_out, G, nbr, w, deg, n, d, ld, neg_lr, gather, beside);
        else if (want_cd) rc = launch_short<GT, true, 0>(*di, sp, s, X, X_out, G, nbr, w, deg, n, d, ld, neg_lr, gather, beside);
        else if (deg == 3) rc = launch_short<GT, false, 3>(*di, sp, s, X, X_out, G, nbr, w, deg, n, d, ld, neg_lr, gather, beside);
        else rc = launch_short<GT, false, 0>(*di, sp, s, X, X_out, G, nbr, w, deg, n, d, ld, neg_lr, gather, beside);
        if (rc) return rc;
    } else {
        // 1024 lanes without the distance, 512 with it.
        const int threads = want_cd ? kTileThreads : kDeepThreads;
        const plan::TilePlan tp = plan::tile_plan(n, deg, threads, want_cd, kLdsCapLarge,
                                                  want_cd ? TileShape<kTileThreads>::RB : TileShape<kDeepThreads>::RB);
        if (tp.lpr == 0)
            return fail(PSGD_EINVAL, "%s: n=%d, deg=%d does not fit the tiled kernel's LDS", name, n, deg);
        size_t lds_bytes = tp.total;
        const size_t remainder = (size_t)n * (d % kVec) * 2 * sizeof(float);
        if (lds_bytes < tp.tab_bytes + remainder) lds_bytes = tp.tab_bytes + remainder;
        const int64_t ntiles = (d / kVec + tp.lpr - 1) / tp.lpr;
#define PSGD_DEG_LAUNCH(CD, UQ)                                                                                           \
    do {                                                                                                                  \
        constexpr int T = CD ? kTileThreads : kDeepThreads;                                                               \
        const void* fn = reinterpret_cast<const void*>(mix_deg_kernel<GT, CD, T, UQ>);                                    \
        if (int rc = allow_lds(fn, lds_bytes)) return rc;                                                                 \
        int per_cu = resident_per_cu(fn, lds_bytes, T);                                                                   \
        if (per_cu > 2 * kGridPerCu) per_cu = 2 * kGridPerCu;                                                             \
        int grid = deg_grid(ntiles, di->cus, per_cu);                                                                       \
        /* one partial per workgroup: a smaller persistent grid still covers every tile */                                \
        if (CD && grid > (int)plan::kShortSlots) grid = (int)plan::kShortSlots;                                           \
        hipLaunchKernelGGL((mix_deg_kernel<GT, CD, T, UQ>), dim3(grid), dim3(T), lds_bytes, s, X, X_out, G, nbr, w, deg,  \
                           n, d, ld, neg_lr, tp.lpr, tp.comb_in_tile ? 1 : 0, gather);                                    \
    } while (0)
        if (want_cd && tp.lpr >= 64) PSGD_DEG_LAUNCH(true, true);
        else if (want_cd) PSGD_DEG_LAUNCH(true, false);
        else if (tp.lpr >= 64) PSGD_DEG_LAUNCH(false, true);
        else PSGD_DEG_LAUNCH(false, false);
#undef PSGD_DEG_LAUNCH
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, name);
    if (prod && !produced)
        if (int rc = enqueue_producer(name, X, ldx, prod->noise, prod->ldn, prod->g, prod->ldg, n, d, prod->c, s)) return rc;
    return PSGD_OK;
}

template <typename GT>
int mix_full_impl(const char* name, const float* X, int64_t ldx, float* X_out, int64_t ldo, const GT* G, int64_t ldg,
                  int n, int64_t d, float lr, int delay_mode, double* cd_out, void* stream) {
    clear_error();
    const bool want_cd = cd_out != nullptr;
    if (!X || !X_out || !G) return fail(PSGD_EINVAL, "%s: null pointer", name);
    if (n < 1 || n > PSGD_MAX_N) return fail(PSGD_EINVAL, "%s: n=%d outside 1..%d", name, n, (int)PSGD_MAX_N);
    if (d < 0) return fail(PSGD_EINVAL, "%s: d=%lld is negative", name, (long long)d);
    if (delay_mode != 0 && delay_mode != 1) return fail(PSGD_EINVAL, "%s: delay_mode=%d", name, delay_mode);
    if (n > 1 && (ldx < d || ldo < d || ldg < d))
        return fail(PSGD_EINVAL, "%s: a row pitch is smaller than d=%lld", name, (long long)d);
    if (n == 1) ldx = ldo = ldg = d;
    if (!aligned_to(X, 4) || !aligned_to(X_out, 4) || !aligned_to(G, sizeof(GT)) || (want_cd && !aligned_to(cd_out, 8)))
        return fail(PSGD_EALIGN, "%s: pointer not aligned to its element size", name);
    const int64_t ldmax = ldx > ldo ? (ldx > ldg ? ldx : ldg) : (ldo > ldg ? ldo : ldg);
    if (ldmax > 0 && (int64_t)n > INT64_MAX / 8 / ldmax) return fail(PSGD_EINVAL, "%s: n * pitch overflows", name);
    const size_t xrow = (size_t)d * sizeof(float), grow = (size_t)d * sizeof(GT);
    const int64_t bx = ldx * (int64_t)sizeof(float), bo = ldo * (int64_t)sizeof(float), bg = ldg * (int64_t)sizeof(GT);
    if (static_cast<const void*>(X) == static_cast<const void*>(X_out) && ldx == ldo) {
        if (delay_mode == 1)
            return fail(PSGD_EALIAS, "%s: delay-by-one keeps X read-only, X_out must be another buffer", name);
    } else if (rows_overlap(X, bx, xrow, X_out, bo, xrow, n)) {
        return fail(PSGD_EALIAS, "%s: X_out partially overlaps X", name);
    }
    if (rows_overlap(G, bg, grow, X_out, bo, xrow, n)) return fail(PSGD_EALIAS, "%s: X_out overlaps G", name);
    if (want_cd && (scalar_overlaps(cd_out, X_out, bo, xrow, n) || scalar_overlaps(cd_out, X, bx, xrow, n) ||
                    scalar_overlaps(cd_out, G, bg, grow, n)))
        return fail(PSGD_EALIAS, "%s: the distance output overlaps a data buffer", name);
    hipStream_t s = static_cast<hipStream_t>(stream);
    DeviceInfo* di = nullptr;
    if (d == 0 && !want_cd) return PSGD_OK;
    if (int rc = device_info(&di)) return rc;
    double* partials = nullptr;
    std::unique_lock<std::mutex> use;
    if (want_cd)
        if (int rc = acquire_partials(di, s, &partials, &use)) return rc;
    if (d == 0) {
        hipLaunchKernelGGL(no_distance_kernel, dim3(1), dim3(1), 0, s, cd_out);
        const hipError_t e0 = hipGetLastError();
        if (e0 != hipSuccess) return hip_fail(e0, "no_distance_kernel");
        return PSGD_OK;
    }
    const int64_t ncg = (d + kVec - 1) / kVec;
    const Pitch ld{ldx, ldo, ldg};
    const float neg_lr = -lr;
    const bool big = long_rows(*di, ncg, 2);
    const plan::RowsPlan rp = plan::full_rows_plan(n, d, di->cus, want_cd);
    const bool walk = plan::walk_full_rows(n, ncg, di->cus);
    const bool split = !walk && !big && rp.threads != 0;
    const Gather gather{partials, cd_out, 0};
    int grid = 0;
    if (walk) {
        grid = di->cus < kMaxGrid ? di->cus : kMaxGrid;
        const plan::SweepPlan sp = plan::sweep_plan(ncg, grid, plan::kRingLanes);
        const int lanes = plan::ring_threads({1, sp.chunk}, plan::kRingLanes);
#define PSGD_LAUNCH_WALK(CD, D)                                                                                            \
    do {                                                                                                                   \
        if (int rc = allow_lds(reinterpret_cast<const void*>(mix_full_walk_kernel<GT, CD, D>), plan::kRingLds)) return rc;  \
        hipLaunchKernelGGL((mix_full_walk_kernel<GT, CD, D>), dim3(grid), dim3(lanes + 64), plan::kRingLds, s, X, X_out, G, \
                           n, d, ld, neg_lr, Sweeps{sp.count, sp.chunk}, lanes, next_pace_slot(), plan::full_lead(D),       \
                           gather);                                                                                        \
    } while (0)
        const bool two = plan::full_depth(sp, n) == 2;
        if (two && want_cd) PSGD_LAUNCH_WALK(true, 2);
        else if (two) PSGD_LAUNCH_WALK(false, 2);
        else if (want_cd) PSGD_LAUNCH_WALK(true, 4);
        else PSGD_LAUNCH_WALK(false, 4);
#undef PSGD_LAUNCH_WALK
    } else if (split) {
        grid = (int)(rp.tiles < kMaxGrid ? rp.tiles : kMaxGrid);
        const size_t lds = (size_t)rp.threads * (want_cd ? 48 : 32) + (16 << rp.logc);
#define PSGD_LAUNCH_ROWS(CD, FEW)                                                                                          \
    hipLaunchKernelGGL((mix_full_rows_kernel<GT, CD, FEW>), dim3(grid), dim3(rp.threads), lds, s, X, X_out, G, n, d, ld,    \
                       neg_lr, rp.logc, rp.nrg, gather)
        if (d < kVec && want_cd) PSGD_LAUNCH_ROWS(true, true);
        else if (d < kVec) PSGD_LAUNCH_ROWS(false, true);
        else if (want_cd) PSGD_LAUNCH_ROWS(true, false);
        else PSGD_LAUNCH_ROWS(false, false);
#undef PSGD_LAUNCH_ROWS
    } else {
        grid = big ? persistent_grid(*di, ncg, 1, kRingThreads) : plan::full_grid(n, ncg, di->cus, kGridPerCu, kThreads);
#define PSGD_LAUNCH_FULL(CD, T)                                                                                            \
    do {                                                                                                                   \
        const Sweeps sw = make_sweeps(ncg, grid, T, n > 8);                                                                \
        if (d % kVec)                                                                                                      \
            hipLaunchKernelGGL((mix_full_kernel<GT, CD, T, true>), dim3(grid), dim3(sweep_threads(sw)), 0, s, X, X_out, G,  \
                               n, d, ld, neg_lr, sw, gather);                                                              \
        else                                                                                                               \
            hipLaunchKernelGGL((mix_full_kernel<GT, CD, T, false>), dim3(grid), dim3(sweep_threads(sw)), 0, s, X, X_out, G, \
                               n, d, ld, neg_lr, sw, gather);                                                              \
    } while (0)
        if (big && want_cd) PSGD_LAUNCH_FULL(true, kRingThreads);
        else if (big) PSGD_LAUNCH_FULL(false, kRingThreads);
        else if (want_cd) PSGD_LAUNCH_FULL(true, kThreads);
        else PSGD_LAUNCH_FULL(false, kThreads);
    }
#undef PSGD_LAUNCH_FULL
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, name);
    return PSGD_OK;
}

int consensus_enqueue(const float* X, int64_t ldx, int n, int64_t d, double* out_dev, hipStream_t s) {
    DeviceInfo* di = nullptr;
    if (int rc = device_info(&di)) return rc;
    double* partials = nullptr;
    std::unique_lock<std::mutex> use;
    if (int rc = acquire_partials(di, s, &partials, &use)) return rc;
    Gather gather{partials, out_dev, 0};
    if (d > 0) {
        const int64_t ncg = (d + kVec - 1) / kVec;
        if (long_rows(*di, ncg) && !plan::distance_alone(n, ncg, di->cus)) {
            const int grid = persistent_grid(*di, ncg, 1, kRingThreads);
            const Sweeps sw = make_sweeps(ncg, grid, kRingThreads);
            if (d % kVec)
                hipLaunchKernelGGL((consensus_sweep_kernel<kRingThreads, true>), dim3(grid), dim3(sweep_threads(sw)), 0, s, X, n, d,
                                   ldx, sw, gather);
            else
                hipLaunchKernelGGL((consensus_sweep_kernel<kRingThreads, false>), dim3(grid), dim3(sweep_threads(sw)), 0, s, X, n, d,
                                   ldx, sw, gather);
        } else {
            const plan::RowsPlan rp = plan::distance_rows_plan(n, d, di->cus);
            if (rp.threads != 0) {
                const int grid = (int)(rp.tiles < kMaxGrid ? rp.tiles : kMaxGrid);
                const size_t lds = (size_t)rp.threads * 48;
                if (d < kVec)
                    hipLaunchKernelGGL(consensus_rows_kernel<true>, dim3(grid), dim3(rp.threads), lds, s, X, n, d, ldx, rp.logc,
                                       rp.nrg, gather);
                else
                    hipLaunchKernelGGL(consensus_rows_kernel<false>, dim3(grid), dim3(rp.threads), lds, s, X, n, d, ldx, rp.logc,
                                       rp.nrg, gather);
            } else {
                const int grid = plan::distance_grid(n, ncg, di->cus, 8, kThreads);  // light kernel: 32 waves per CU
                const Sweeps sw = make_sweeps(ncg, grid, kThreads);
                const bool apart = plan::distance_summed_apart(grid, n, d, di->cus);
                if (apart) gather.out = nullptr;
                if (d % kVec)
                    hipLaunchKernelGGL(consensus_partial_kernel<true>, dim3(grid), dim3(sweep_threads(sw)), 0, s, X, n, d, ldx, (int)sw.chunk,
                                       gather);
                else
                    hipLaunchKernelGGL(consensus_partial_kernel<false>, dim3(grid), dim3(sweep_threads(sw)), 0, s, X, n, d, ldx, (int)sw.chunk,
                                       gather);
                if (apart) hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(kThreads), 0, s, partials, grid, out_dev);
            }
        }
    } else {
        hipLaunchKernelGGL(no_distance_kernel, dim3(1), dim3(1), 0, s, out_dev);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "consensus_partial_kernel");
    return PSGD_OK;
}

int consensus_check(const char* name, const float* X, int64_t ldx, int n, int64_t d) {
    if (!X) return fail(PSGD_EINVAL, "%s: null pointer", name);
    if (n < 1 || n > PSGD_MAX_N) return fail(PSGD_EINVAL, "%s: n=%d outside 1..%d", name, n, (int)PSGD_MAX_N);
    if (d < 0) return fail(PSGD_EINVAL, "%s: d=%lld is negative", name, (long long)d);
    if (n > 1 && ldx < d) return fail(PSGD_EINVAL, "%s: row pitch smaller than d", name);
    if (!aligned_to(X, 4)) return fail(PSGD_EALIGN, "%s: X not 4-byte aligned", name);
    if (ldx > 0 && (int64_t)n > INT64_MAX / 8 / ldx) return fail(PSGD_EINVAL, "%s: n * pitch overflows", name);
    return PSGD_OK;
}

int consensus_async_impl(const char* name, const float* X, int64_t ldx, int n, int64_t d, double* out_dev,
                         void* stream) {
    clear_error();
    if (!out_dev) return fail(PSGD_EINVAL, "%s: null output pointer", name);
    if (!aligned_to(out_dev, 8)) return fail(PSGD_EALIGN, "%s: out_dev not 8-byte aligned", name);
    if (int rc = consensus_check(name, X, ldx, n, d)) return rc;
    return consensus_enqueue(X, n == 1 ? d : ldx, n, d, out_dev, static_cast<hipStream_t>(stream));
}

}  // namespace
}  // namespace psgd

extern "C" {

int psgd_mix_step(const float* X, float* X_out, const float* G, const int32_t* nbr, const float* w, int n, int64_t d,
                  float lr, int delay_mode, void* stream) {
    return psgd::mix_step_impl<float>("psgd_mix_step", X, d, X_out, d, G, d, nbr, w, n, d, lr, delay_mode, false,
                                      nullptr, stream);
}

int psgd_mix_step_bf16g(const float* X, float* X_out, const uint16_t* G_bf16, const int32_t* nbr, const float* w,
                        int n, int64_t d, float lr, int delay_mode, void* stream) {
    return psgd::mix_step_impl<uint16_t>("psgd_mix_step_bf16g", X, d, X_out, d, G_bf16, d, nbr, w, n, d, lr,
                                         delay_mode, false, nullptr, stream);
}

int psgd_mix_step_cd(const float* X, float* X_out, const float* G, const int32_t* nbr, const float* w, int n,
                     int64_t d, float lr, int delay_mode, double* cdist_out, void* stream) {
    return psgd::mix_step_impl<float>("psgd_mix_step_cd", X, d, X_out, d, G, d, nbr, w, n, d, lr, delay_mode, true,
                                      cdist_out, stream);
}

int psgd_mix_step_cd_bf16g(const float* X, float* X_out, const uint16_t* G_bf16, const int32_t* nbr, const float* w,
                           int n, int64_t d, float lr, int delay_mode, double* cdist_out, void* stream) {
    return psgd::mix_step_impl<uint16_t>("psgd_mix_step_cd_bf16g", X, d, X_out, d, G_bf16, d, nbr, w, n, d, lr,
                                         delay_mode, true, cdist_out, stream);
}

int psgd_mix_step_ex(const float* X, int64_t ldx, float* X_out, int64_t ldo, const void* G, int64_t ldg, int g_is_bf16,
                     const int32_t* nbr, const float* w, int n, int64_t d, float lr, int delay_mode,
                     double* cdist_out, void* stream) {
    if (g_is_bf16 != 0 && g_is_bf16 != 1) {
        psgd::clear_error();
        return psgd::fail(PSGD_EINVAL, "psgd_mix_step_ex: g_is_bf16=%d", g_is_bf16);
    }
    if (g_is_bf16)
        return psgd::mix_step_impl<uint16_t>("psgd_mix_step_ex", X, ldx, X_out, ldo, static_cast<const uint16_t*>(G),
                                             ldg, nbr, w, n, d, lr, delay_mode, cdist_out != nullptr, cdist_out,
                                             stream);
    return psgd::mix_step_impl<float>("psgd_mix_step_ex", X, ldx, X_out, ldo, static_cast<const float*>(G), ldg, nbr,
                                      w, n, d, lr, delay_mode, cdist_out != nullptr, cdist_out, stream);
}

int psgd_mix_step_cd_static(const float* X, int64_t ldx, float* X_out, int64_t ldo, const void* G, int64_t ldg,
                            int g_is_bf16, const int32_t* nbr, const float* w, int n, int64_t d, float lr,
                            int delay_mode, double* cdist_out, void* stream) {
    if (g_is_bf16 != 0 && g_is_bf16 != 1) {
        psgd::clear_error();
        return psgd::fail(PSGD_EINVAL, "psgd_mix_step_cd_static: g_is_bf16=%d", g_is_bf16);
    }
    if (g_is_bf16)
        return psgd::mix_step_impl<uint16_t>("psgd_mix_step_cd_static", X, ldx, X_out, ldo,
                                             static_cast<const uint16_t*>(G), ldg, nbr, w, n, d, lr, delay_mode, true,
                                             cdist_out, stream, 3, true);
    return psgd::mix_step_impl<float>("psgd_mix_step_cd_static", X, ldx, X_out, ldo, static_cast<const float*>(G), ldg,
                                      nbr, w, n, d, lr, delay_mode, true, cdist_out, stream, 3, true);
}

int psgd_mix_step_deg(const float* X, int64_t ldx, float* X_out, int64_t ldo, const void* G, int64_t ldg, int g_is_bf16,
                      const int32_t* nbr, const float* w, int deg, int n, int64_t d, float lr, int delay_mode,
                      double* cdist_out, void* stream) {
    if (g_is_bf16 != 0 && g_is_bf16 != 1) {
        psgd::clear_error();
        return psgd::fail(PSGD_EINVAL, "psgd_mix_step_deg: g_is_bf16=%d", g_is_bf16);
    }
    if (g_is_bf16)
        return psgd::mix_step_impl<uint16_t>("psgd_mix_step_deg", X, ldx, X_out, ldo, static_cast<const uint16_t*>(G),
                                             ldg, nbr, w, n, d, lr, delay_mode, cdist_out != nullptr, cdist_out,
                                             stream, deg);
    return psgd::mix_step_impl<float>("psgd_mix_step_deg", X, ldx, X_out, ldo, static_cast<const float*>(G), ldg, nbr,
                                      w, n, d, lr, delay_mode, cdist_out != nullptr, cdist_out, stream, deg);
}

int psgd_mix_step_d1d(const float* X, int64_t ldx, float* X_out, int64_t ldo, const float* G, int64_t ldg, const int32_t* nbr,
                      const float* w, int deg, int n, int64_t d, float lr, const float* noise, int64_t ldn, float* G_next, int64_t ldgn,
                      float c, double* cdist_out, void* stream) {
    using namespace psgd;
    const char* name = "psgd_mix_step_d1d";
    clear_error();
    if (!X || !X_out || !G || !noise || !G_next) return fail(PSGD_EINVAL, "%s: null pointer", name);
    if (n < 1 || n > PSGD_MAX_N || d < 0) return fail(PSGD_EINVAL, "%s: n=%d d=%lld", name, n, (long long)d);
    if (n > 1 && (ldx < d || ldo < d || ldg < d || ldn < d || ldgn < d)) return fail(PSGD_EINVAL, "%s: a row pitch is smaller than d", name);
    if (n == 1) ldx = ldo = ldg = ldn = ldgn = d;
    if (!aligned_to(noise, 4) || !aligned_to(G_next, 4)) return fail(PSGD_EALIGN, "%s: pointer not 4-byte aligned", name);
    int64_t ldmax = ldn > ldgn ? ldn : ldgn;
    for (int64_t l : {ldx, ldo, ldg}) ldmax = l > ldmax ? l : ldmax;
    if (ldmax > 0 && (int64_t)n > INT64_MAX / 8 / ldmax) return fail(PSGD_EINVAL, "%s: n * pitch overflows", name);
    const size_t row = (size_t)d * sizeof(float);
    // what is written here and read there, or written twice, at the same time
    if (rows_overlap(G_next, ldgn * 4, row, X, ldx * 4, row, n) || rows_overlap(G_next, ldgn * 4, row, noise, ldn * 4, row, n) ||
        rows_overlap(G_next, ldgn * 4, row, G, ldg * 4, row, n) || rows_overlap(G_next, ldgn * 4, row, X_out, ldo * 4, row, n) ||
        rows_overlap(noise, ldn * 4, row, X_out, ldo * 4, row, n))
        return fail(PSGD_EALIAS, "%s: an output overlaps another array", name);
    if (cdist_out && (scalar_overlaps(cdist_out, G_next, ldgn * 4, row, n) || scalar_overlaps(cdist_out, noise, ldn * 4, row, n)))
        return fail(PSGD_EALIAS, "%s: the distance output overlaps a data buffer", name);
    const Produce prod{noise, G_next, ldn, ldgn, c};
    return mix_step_impl<float>(name, X, ldx, X_out, ldo, G, ldg, nbr, w, n, d, lr, 1, cdist_out != nullptr, cdist_out, stream, deg, false,
                                &prod);
}

int psgd_mix_full(const float* X, int64_t ldx, float* X_out, int64_t ldo, const void* G, int64_t ldg, int g_is_bf16,
                  int n, int64_t d, float lr, int delay_mode, double* cdist_out, void* stream) {
    if (g_is_bf16 != 0 && g_is_bf16 != 1) {
        psgd::clear_error();
        return psgd::fail(PSGD_EINVAL, "psgd_mix_full: g_is_bf16=%d", g_is_bf16);
    }
    if (g_is_bf16)
        return psgd::mix_full_impl<uint16_t>("psgd_mix_full", X, ldx, X_out, ldo, static_cast<const uint16_t*>(G), ldg,
                                             n, d, lr, delay_mode, cdist_out, stream);
    return psgd::mix_full_impl<float>("psgd_mix_full", X, ldx, X_out, ldo, static_cast<const float*>(G), ldg, n, d, lr,
                                      delay_mode, cdist_out, stream);
}

int psgd_build_mixing_device(int topology, int n, uint64_t seed, uint64_t* step_dev, uint64_t step_offset, int advance,
                             int32_t* nbr, float* w, void* stream) {
    using namespace psgd;
    clear_error();
    if (!nbr || !w) return fail(PSGD_EINVAL, "psgd_build_mixing_device: null output pointer");
    if (n < 1 || n > PSGD_MAX_N)
        return fail(PSGD_EINVAL, "psgd_build_mixing_device: n=%d outside 1..%d", n, (int)PSGD_MAX_N);
    if (topology == PSGD_TOPO_FULL)
        return fail(PSGD_EINVAL, "psgd_build_mixing_device: the uniform topology has no 3-slot table, use psgd_mix_full");
    if (topology != PSGD_TOPO_RING && topology != PSGD_TOPO_RAND_RING)
        return fail(PSGD_EINVAL, "psgd_build_mixing_device: unknown topology %d", topology);
    if (advance < 0) return fail(PSGD_EINVAL, "psgd_build_mixing_device: advance=%d is negative", advance);
    if (!aligned_to(nbr, 4) || !aligned_to(w, 4) || (step_dev && !aligned_to(step_dev, 8)))
        return fail(PSGD_EALIGN, "psgd_build_mixing_device: pointer not aligned to its element size");
    const size_t tb = (size_t)n * 3 * 4;
    if (overlaps(nbr, tb, w, tb) || (step_dev && (overlaps(step_dev, 8, nbr, tb) || overlaps(step_dev, 8, w, tb))))
        return fail(PSGD_EALIAS, "psgd_build_mixing_device: nbr, w and step_dev overlap");
    hipLaunchKernelGGL(build_mixing_kernel, dim3(1), dim3((n + 63) / 64 * 64), 0, static_cast<hipStream_t>(stream),
                       topology == PSGD_TOPO_RAND_RING ? 1 : 0, n, seed, step_dev, step_offset, (uint64_t)advance, nbr, w);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "build_mixing_kernel");
    return PSGD_OK;
}

double psgd_consensus_dist(const float* X, int n, int64_t d) {
    using namespace psgd;
    clear_error();
    if (consensus_check("psgd_consensus_dist", X, d, n, d) != PSGD_OK) return NAN;
    if (d == 0 || n == 1) return 0.0;
    hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) { hip_fail(e, "hipDeviceSynchronize"); return NAN; }
    // The final sum goes straight to pinned host memory, one word and one call at a time per device: a copy of eight bytes
    // after the kernels cost more host time than both launches (27 us a call on a small array, now 16).
    DeviceInfo* di = nullptr;
    if (device_info(&di) != PSGD_OK) return NAN;
    std::lock_guard<std::mutex> lock(di->host_result_mutex);
    if (!di->host_result) {
        e = hipHostMalloc(reinterpret_cast<void**>(&di->host_result), sizeof(double), hipHostMallocDefault);
        if (e != hipSuccess) {
            di->host_result = nullptr;
            hip_fail(e, "hipHostMalloc(result)");
            return NAN;
        }
    }
    if (!di->host_result_dev) {
        e = hipHostGetDevicePointer(reinterpret_cast<void**>(&di->host_result_dev), di->host_result, 0);
        if (e != hipSuccess) { di->host_result_dev = nullptr; hip_fail(e, "hipHostGetDevicePointer(result)"); return NAN; }
    }
    *di->host_result = NAN;
    if (consensus_enqueue(X, d, n, d, di->host_result_dev, nullptr) != PSGD_OK) return NAN;
    e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) { hip_fail(e, "hipStreamSynchronize"); return NAN; }
    return *static_cast<volatile double*>(di->host_result);
}

int psgd_consensus_dist_async(const float* X, int n, int64_t d, double* out_dev, void* stream) {
    return psgd::consensus_async_impl("psgd_consensus_dist_async", X, d, n, d, out_dev, stream);
}

int psgd_consensus_dist_ex(const float* X, int64_t ldx, int n, int64_t d, double* out_dev, void* stream) {
    return psgd::consensus_async_impl("psgd_consensus_dist_ex", X, ldx, n, d, out_dev, stream);
}

int psgd_synth_grad(const float* X_prev, const float* noise, float* G, int64_t count, float c, void* stream) {
    using namespace psgd;
    clear_error();
    if (!X_prev || !noise || !G) return fail(PSGD_EINVAL, "psgd_synth_grad: null pointer");
    if (count < 0) return fail(PSGD_EINVAL, "psgd_synth_grad: negative count");
    if (!aligned_to(X_prev, 4) || !aligned_to(noise, 4) || !aligned_to(G, 4))
        return fail(PSGD_EALIGN, "psgd_synth_grad: pointer not 4-byte aligned");
    const size_t bytes = (size_t)count * sizeof(float);
    if (overlaps(G, bytes, X_prev, bytes) || overlaps(G, bytes, noise, bytes))
        return fail(PSGD_EALIAS, "psgd_synth_grad: G overlaps an input");
    if (count == 0) return PSGD_OK;
    return enqueue_producer("synth_grad_kernel", X_prev, count, noise, count, G, count, 1, count, c, static_cast<hipStream_t>(stream));
}

int psgd_synth_grad_ex(const float* X_prev, int64_t ldx, const float* noise, int64_t ldn, float* G, int64_t ldg,
                       int n, int64_t d, float c, void* stream) {
    using namespace psgd;
    clear_error();
    if (!X_prev || !noise || !G) return fail(PSGD_EINVAL, "psgd_synth_grad_ex: null pointer");
    if (n < 1 || n > PSGD_MAX_N || d < 0) return fail(PSGD_EINVAL, "psgd_synth_grad_ex: n=%d d=%lld", n, (long long)d);
    if (n > 1 && (ldx < d || ldn < d || ldg < d)) return fail(PSGD_EINVAL, "psgd_synth_grad_ex: a row pitch is smaller than d");
    if (n == 1) ldx = ldn = ldg = d;
    if (!aligned_to(X_prev, 4) || !aligned_to(noise, 4) || !aligned_to(G, 4))
        return fail(PSGD_EALIGN, "psgd_synth_grad_ex: pointer not 4-byte aligned");
    const int64_t ldmax = ldx > ldn ? (ldx > ldg ? ldx : ldg) : (ldn > ldg ? ldn : ldg);
    if (ldmax > 0 && (int64_t)n > INT64_MAX / 8 / ldmax) return fail(PSGD_EINVAL, "psgd_synth_grad_ex: n * pitch overflows");
    const size_t row = (size_t)d * sizeof(float);
    if (rows_overlap(G, ldg * 4, row, X_prev, ldx * 4, row, n) || rows_overlap(G, ldg * 4, row, noise, ldn * 4, row, n))
        return fail(PSGD_EALIAS, "psgd_synth_grad_ex: G overlaps an input");
    if (d == 0) return PSGD_OK;
    return enqueue_producer("synth_grad_kernel", X_prev, ldx, noise, ldn, G, ldg, n, d, c, static_cast<hipStream_t>(stream));
}

int psgd_reference_stream(int kind, const float* X, int64_t ldx, float* X_out, int64_t ldo, const void* G, int64_t ldg,
                          int g_is_bf16, int n, int64_t d, float a, void* stream) {
    using namespace psgd;
    clear_error();
    if (kind != kRefRead && kind != kRefWrite && kind != kRefAxpy)
        return fail(PSGD_EINVAL, "psgd_reference_stream: kind=%d", kind);
    if (g_is_bf16 != 0 && g_is_bf16 != 1) return fail(PSGD_EINVAL, "psgd_reference_stream: g_is_bf16=%d", g_is_bf16);
    if (!X || !X_out || !G) return fail(PSGD_EINVAL, "psgd_reference_stream: null pointer");
    if (n < 1 || n > PSGD_MAX_N || d < 0) return fail(PSGD_EINVAL, "psgd_reference_stream: n=%d d=%lld", n, (long long)d);
    if (n > 1 && (ldx < d || ldo < d || ldg < d))
        return fail(PSGD_EINVAL, "psgd_reference_stream: a row pitch is smaller than d");
    if (n == 1) ldx = ldo = ldg = d;
    const size_t gsz = g_is_bf16 ? 2 : 4;
    if (d % 4 || ldx % 4 || ldo % 4 || ldg % 4 || !aligned_to(X, 16) || !aligned_to(X_out, 16) || !aligned_to(G, 4 * gsz))
        return fail(PSGD_EALIGN, "psgd_reference_stream: needs d and the pitches in multiples of 4 and 128-bit aligned rows");
    const int64_t ldmax = ldx > ldo ? (ldx > ldg ? ldx : ldg) : (ldo > ldg ? ldo : ldg);
    if (ldmax > 0 && (int64_t)n > INT64_MAX / 8 / ldmax) return fail(PSGD_EINVAL, "psgd_reference_stream: n * pitch overflows");
    const size_t xrow = (size_t)d * 4, grow = (size_t)d * gsz;
    if (kind != kRefRead && (rows_overlap(X, ldx * 4, xrow, X_out, ldo * 4, xrow, n) ||
                             rows_overlap(G, ldg * (int64_t)gsz, grow, X_out, ldo * 4, xrow, n)))
        return fail(PSGD_EALIAS, "psgd_reference_stream: X_out overlaps an input");
    if (d == 0) return PSGD_OK;
    DeviceInfo* di = nullptr;
    if (int rc = device_info(&di)) return rc;
    const bool big = long_rows(*di, d / 4);
    const int threads = big ? kRingThreads : kThreads;
    const int grid = persistent_grid(*di, d / 4, big ? 1 : kGridPerCu, threads);
    const Sweeps sw = make_sweeps(d / 4, grid, threads);
    const Pitch ld{ldx, ldo, ldg};
    hipStream_t s = static_cast<hipStream_t>(stream);
#define PSGD_REF_LAUNCH(KIND, GT, T)                                                                                    \
    hipLaunchKernelGGL((reference_stream_kernel<KIND, GT, T>), dim3(grid), dim3(T), 0, s, X, X_out,                      \
                       static_cast<const GT*>(G), n, d, ld, a, sw)
#define PSGD_REF_KIND(KIND)                                                                                             \
    do {                                                                                                                \
        if (g_is_bf16 && big) PSGD_REF_LAUNCH(KIND, uint16_t, kRingThreads);                                            \
        else if (g_is_bf16) PSGD_REF_LAUNCH(KIND, uint16_t, kThreads);                                                  \
        else if (big) PSGD_REF_LAUNCH(KIND, float, kRingThreads);                                                       \
        else PSGD_REF_LAUNCH(KIND, float, kThreads);                                                                    \
    } while (0)
    if (kind == kRefRead) PSGD_REF_KIND(kRefRead);
    else if (kind == kRefWrite) PSGD_REF_KIND(kRefWrite);
    else PSGD_REF_KIND(kRefAxpy);
#undef PSGD_REF_KIND
#undef PSGD_REF_LAUNCH
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "reference_stream_kernel");
    return PSGD_OK;
}

int psgd_device_status(int clear) {
    using namespace psgd;
    clear_error();
    hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize");
    int word = 0;
    e = hipMemcpyFromSymbol(&word, HIP_SYMBOL(g_status_word), sizeof(int));
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyFromSymbol");
    if (clear && word) {
        const int zero = 0;
        e = hipMemcpyToSymbol(HIP_SYMBOL(g_status_word), &zero, sizeof(int));
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyToSymbol");
    }
    return word;
}

}  // extern "C"
