// Declarations shared by the library's own translation units (not part of the C boundary).
#ifndef PSGD_INTERNAL_H
#define PSGD_INTERNAL_H

#include <cstddef>
#include <cstdint>

namespace psgd {

// Records a printf-style message for psgd_last_error() on this thread and returns `code`.
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

// Launch arithmetic of the persistent grids: plain host functions, kept apart from the kernels so that a CPU
// build can check them (every column group covered once, grids within the partials buffer).
namespace plan {

constexpr int kMaxGrid = 4096;    // upper bound on persistent workgroups = slots of the partials buffer
constexpr int kChunkAlign = 16;   // column groups (256 bytes): ranges that start at an odd 16 bytes cost 7 %

// Workgroups of `threads` lanes for `work_items` lane-sized items: one per item batch, at most `per_cu`
// per compute unit, never more than kMaxGrid.
inline int persistent_grid(int cus, int64_t work_items, int per_cu, int threads) {
    const int64_t need = (work_items + threads - 1) / threads;
    int64_t cap = (int64_t)cus * per_cu;
    if (cap > kMaxGrid) cap = kMaxGrid;
    const int64_t g = need < cap ? need : cap;
    return (int)(g < 1 ? 1 : g);
}

// The same with as many workgroups on each compute unit, of fewer lanes: `g` workgroups short of a whole round leave compute units idle, or
// waiting for the few that have one more.
inline int even_grid(int g, int cus) { return (g + cus - 1) / cus * cus; }
// Global averaging: from 16 learners on, where under 3/4 of the even grid would be there, from 96 learners on 85 %; beyond two on each compute
// unit, where half a round is missing.  us, workgroups of 256 lanes / even: 29 x 298 099 26.9 / 23.9, 120 x 299 507 with the distance 81.2 % of the time, 320 x 140 877 85.8 %,
// 39 x 529 933 88.4 %; not 33 x 198 253 19.4 / 20.3, 52 x 242 112 29.6 / 30.8, 23 x 414 464 + 4.5 %, nor few learners (4 x 458 912 7.5 / 8.3, 6 x
// 266 400 8.9 / 10.0, 7 x 475 009 with the distance 13.8 / 14.8, 9 x 475 584 10.9 / 11.9), whose lanes wait for one row after the other.
inline int full_grid(int n, int64_t work_items, int cus, int per_cu, int threads) {
    const int g = persistent_grid(cus, work_items, per_cu, threads), even = even_grid(g, cus);
    if (n < 16 || g <= cus / 2 || even > kMaxGrid) return g;
    if (g > 2 * cus) return even - g > cus / 2 ? even : g;
    return 4 * g < 3 * even || (n >= 96 && 20 * g < 17 * even) ? even : g;
}
// The distance: from 25 learners on, for more than one on each compute unit.  77 x 271 744 85.9 % of the time, 131 x 294 771 82.7, 70 x 326 464 91.4, 104 x
// 393 203 96.5, 124 x 792 365 90.8; fewer learners 102 to 112 % (11 x 147 227, 5 x 554 592, 7 x 1 049 335), one on each 101 to 105 (23 x 154 816, 74 x 164 288).
inline int distance_grid(int n, int64_t work_items, int cus, int per_cu, int threads) {
    const int g = persistent_grid(cus, work_items, per_cu, threads), even = even_grid(g, cus);
    if (n < 25 || g <= cus || even > kMaxGrid) return g;
    return even - g > (g > 2 * cus ? cus / 3 : cus / 8) ? even : g;
}

// Grid of the degree-K kernel: one workgroup per tile up to what is resident, within the same bound.
inline int deg_grid(int64_t ntiles, int cus, int per_cu) {
    int64_t cap = (int64_t)cus * per_cu;
    if (cap > kMaxGrid) cap = kMaxGrid;
    const int64_t g = ntiles < cap ? ntiles : cap;
    return (int)(g < 1 ? 1 : g);
}

// Which range of a sweep workgroup `b` of `grid` takes.  The hardware deals consecutive workgroups out to the
// chip's `xcds` accelerator dies in turn (each with its own L2), so taking range b would hand every die every
// xcds-th range of the row; with this mapping the workgroups that share a die (b, b + xcds, ...) take
// neighbouring ranges, and each L2 sees one contiguous stretch of every row in flight.  Measured on MI355X
// (8 dies) with the step's traffic pattern: 78.4 against 78.0 % of the HBM peak.  A bijection on 0..grid-1 when
// xcds divides grid, the identity otherwise.
#if defined(__HIPCC__)
#define PSGD_HOST_DEVICE __host__ __device__
#else
#define PSGD_HOST_DEVICE
#endif
PSGD_HOST_DEVICE inline int64_t die_contiguous_slot(int64_t b, int64_t grid, int xcds) {
    if (xcds <= 1 || grid % xcds != 0) return b;
    return (b % xcds) * (grid / xcds) + b / xcds;
}

// Even split of `ncg` column groups over a persistent grid: every workgroup makes `count` sweeps and takes
// `chunk` <= threads consecutive groups in each; workgroup b's range in sweep sw starts at
// (sw * grid + die_contiguous_slot(b)) * chunk.  With a fixed chunk of `threads` the last, partly filled sweep costs as
// much as a full one (11 instead of 10.2 on rows of 2 M groups with 256 workgroups of 768 lanes; three instead of 2.03
// on 400 000: ring step of 512 learners 2185 us, split evenly 1939); the kernels are bound by bytes, so a sweep is as
// much faster as it is smaller.  The chunk stays a multiple of kChunkAlign.
struct SweepPlan {
    int64_t count, chunk;
};
// even = false: fewer than four sweeps in full chunks after all, for kernels whose sweep is short (few rows): a sweep more is
// then a round of latency more for every workgroup, not for the few that reach it (global averaging of 3 x 1.1 M 11.0 us split
// evenly, 9.6 in full chunks).
inline SweepPlan sweep_plan(int64_t ncg, int grid, int threads, bool even = true) {
    SweepPlan s;
    const int64_t per = (int64_t)grid * threads;
    s.count = (ncg + per - 1) / per;
    if (!even && s.count > 1 && s.count < 4) {
        s.chunk = threads;
        return s;
    }
    const int64_t parts = s.count * grid;
    s.chunk = parts > 0 ? (ncg + parts - 1) / parts : 1;
    s.chunk = (s.chunk + kChunkAlign - 1) / kChunkAlign * kChunkAlign;
    return s;
}

// The counters that the workgroups of a launch with a distance draw tickets from (last_sum): the one that draws the last ticket adds the partial
// sums up.  A draw adds one to its counter, or puts it back to zero at the last of `of`, in one access.  Every counter is used with one
// `of` only, whatever the launch: then any number of launches, in order or by a caller's mistake at the same time, ends with the
// counter at zero, and what such a mistake spoils are the distances of those launches, not of a later one.
// Up to 64 workgroups draw at one counter, its `of` being its place; more draw at one of 16 leaves each, of a size of its own, and the last of
// each leaf at the counter of 16.
constexpr int kTicketLeaves = 16, kTicketQueue = 64;
constexpr int kTicketCounters = kTicketQueue + 1 + kTicketLeaves * (kMaxGrid / kTicketLeaves);
struct Ticket {
    int at, of;
};
PSGD_HOST_DEVICE inline bool ticket_leaves(int grid) { return grid > kTicketQueue; }
PSGD_HOST_DEVICE inline Ticket ticket_leaf(int block, int grid) {
    const int leaf = block % kTicketLeaves, of = (grid - leaf + kTicketLeaves - 1) / kTicketLeaves;
    return Ticket{kTicketQueue + 1 + leaf + kTicketLeaves * (of - 1), of};
}
PSGD_HOST_DEVICE inline Ticket ticket_root(int grid) {
    const int of = ticket_leaves(grid) ? kTicketLeaves : grid;
    return Ticket{of, of};
}

// The ring walk: most lanes that have columns (one more wavefront keeps the pace), words to keep it with (launches under way at a
// time that do not share one), and how often a wavefront asks before it walks on by itself (about 30 us).
constexpr int kRingLanes = 960;
constexpr int kPaceSlots = 64;
constexpr int kPaceSpins = 400;
// Rows on their way per lane, and how far ahead of the mean a workgroup may be, in quarter rows.  The narrower the chunk, the more rows: about 900 lanes times rows keep the memory busy, and
// what is beyond that costs more in order than it gains (us; one row each 64 x 1.2 M 154, two 153; 128 x 500 k 138 / 129; two / four
// 130 x 200 k with a distance 79 / 68, 256 x 280 k with bf16 gradients 154 / 135; four / six 512 x 205 k 244.7 / 237.0, without the distance 222.8 /
// 212.9, 300 x 210 k 147.9 / 143.3, 256 x 220 001 bf16 143.8 / 141.1, 512 x 240 k bf16 226.0 / 207.8, 200 x 260 k bf16 94.8 / 92.1; from 240 to 260 fp32
// alone would stay at four: 512 x 240 k 252.1 / 258.1, 256 x 260 k 138.5 / 142.6).  Lead: one row 1.25 / 1.5 / 1.75 / 2 rows 64 x 25.6 M
// 3134 / 3136 / 3186 / 3289; four rows of lead or none for a depth of one: 3500 / 3800.
inline int ring_depth(const SweepPlan& s, int n) { return s.chunk >= 576 || n < 4 ? 1 : s.chunk >= 400 || n < 16 ? 2 : s.chunk >= 260 ? 4 : 6; }
constexpr int kRingThreadsMost = kRingLanes + 64;   // of the workgroup
// With the producer of the next gradients in the walk five arrays are on their way, not three: fewer rows, less lead (pairs, us: one row
// of lead 5, 6 and 7 quarters 128 x 8 M 3414 / 3494 / 3674; one row or two of depth 128 x 520 k 223 / 235, two or four 113 x 328 k 134 / 171,
// 421 x 301 k 445 / 576).
inline int ring_depth_produce(const SweepPlan& s) { return s.chunk >= 450 ? 1 : 2; }
inline int pace_lead(int depth, bool produce = false) { return depth == 1 ? (produce ? 5 : 6) : 5 * depth; }
// More than half of a compute unit's LDS: the workgroups then take a compute unit each.  Two on one fall behind the others, which wait.
constexpr size_t kRingLds = 82 * 1024;

// Lanes that a plan's workgroups need: all of `threads`, but no wavefront without columns where the row takes one sweep.  The ring
// walk asks for one sweep's worth whatever their number: a wavefront without columns shadows another's loads (paced, 256 x 1 M with
// bf16 gradients in two sweeps of 496 lanes: 532 us on 960 lanes, 429 on 512).
inline int ring_threads(const SweepPlan& s, int threads) {
    return s.count > 1 ? threads : (int)((s.chunk + 63) / 64 * 64);
}

// Whether a 3-slot table on n rows of `ncg` column groups takes mix_step_kernel (the ring walk, tiles for any other table) instead
// of the short-row kernel; in column groups per compute unit.  The walk takes 0.45 us a row and sweep however
// few columns there are, and stages and classifies the table first; the short-row kernel reads and writes all rows of a tile at once,
// which holds its rate to 5.0-5.3 TB/s once the arrays do not fit the last-level cache.  us, short-row kernel / ring walk, fp32 with the
// distance: 9 x 2.5 M 52.5 / 51 (bf16 gradients 43 / 45), 12 x 1.5 M 42.6 / 44.7, 16 x 1.5 M 56.0 / 56.1, x 2.9 M 106 / 95, 24 x 0.66 M 37.5 / 39.2, x 0.82 M 48.1 / 46.8,
// 32 x 0.51 M 41.3 / 41.2, x 0.82 M 66 / 59, 64 x 0.33 M 51 / 54, x 0.41 M 64 / 60, x 0.66 M 97 / 88, 128 x 0.26 M 78 / 75 (bf16 gradients, no
// distance, 0.19 M 53 / 66; with it 0.33 M 94.8 / 86.8), x 0.32 M 103.9 / 92.3, 96 x 0.33 M bf16, no distance, 69.3 / 58.9, 199 x 325 001 174 / 150, 200 x 0.26 M
// 135 / 113, 256 x 0.2 M 139.8 / 122.9, 512 x 0.2 M 266.8 / 236.5, x 230 001 331 / 273 (300 x 0.2 M with bf16 gradients 133.6 / 142.9).
inline bool ring_rows(int n, int64_t ncg, int cus) {
    const int64_t from = n < 12 ? 3600 : n < 16 ? 2500 : n < 24 ? 1600 : n < 32 ? 800 : n < 48 ? 560 : n < 96 ? 400 : n < 200 ? 307 : n < 256 ? 230 : 192;
    return n > 8 && ncg >= from * cus;
}
// The same for all calls of a 3-slot table.
//   - Three to eight learners, whose rows the short-row kernel holds in one lane, or with the distance spreads over two: by the column groups
//     of all learners together (us, short-row kernel / ring walk, fp32 with the distance 3 x 12 M 76.0 / 73.2, 4 x 8 M 69.0 / 66.3, 5 x 6 M 68.9 / 62.9,
//     7 x 4 M 63.4 / 59.6, 8 x 3.1 M 57.1 / 53.7, 8 x 12 M 201 / 184, bf16 gradients 6 x 5 M 56.5 / 55.9, 7 x 32 M 424 / 361; 3 x 3 M 20.5 / 24.6, 8 x 1 M 17.8 / 22).
//     Without the distance later, and not for the fewest: 8 x 24 M 412 / 362, bf16 338 / 307, 6 x 24 M 304 / 273; 7 x 7 M 97.3 / 95.9, where other tables'
//     tiles lose more than rings gain; 5 x 12 M 117.1 / 116.8, 3 x 32 M 182 / 183.
//   - With the next gradients of the delay-by-one schedule, five arrays: earlier (32 x 500 k 62.8 / 58.9, 64 x 250 k 67.6 / 61.1, 128 x 250 k 132.9 / 116.6,
//     16 x 1 M 61.2 / 58.7, 12 x 2 M 90.7 / 83.3; 9 x 1 M 35.8 / 36.6, 24 x 500 k 46.1 / 45.9, 64 x 160 k 43.3 / 51.0); 5 x 6 M 119 / 103, 8 x 3 M 87.6 / 83.5, without the
//     distance 4 x 6 M 78.9 / 81.1.
inline bool walk_rows(int n, int64_t ncg, int cus, bool cd, bool produce) {
    if (n > 8 && !produce) return ring_rows(n, ncg, cus);
    if (n > 8) return ncg >= (n < 12 ? 1500 : n < 16 ? 1200 : n < 24 ? 900 : n < 48 ? 440 : n < 256 ? 220 : 192) * (int64_t)cus;
    const int64_t all = n * ncg;
    if (produce) return n >= (cd ? 4 : 5) && all >= 24000 * (int64_t)cus;
    return cd ? n > 2 && all >= 24000 * (int64_t)cus : n > 5 && all >= 100000 * (int64_t)cus;
}

// Global averaging with the workgroups of a die in step, in column groups per compute unit, and how far ahead of the mean a workgroup
// may be, in quarter rows: more than in the ring walk, as half of the rows are only read.  us, lanes walking alone or rows spread over
// lanes / in step: 9 x 1.5 M 32.4 / 32.9 (bf16 gradients, no distance 25.2 / 27.5), x 3 M 63.8 / 59.3, 16 x 0.82 M 33.7 / 31.1, x 0.4 M bf16
// 11.7 / 14.8, 32 x 0.5 M 34.9 / 36.4, 64 x 0.22 M 34.6 / 37.8, x 0.31 M 51 / 46, x 0.6 M 97 / 80, 512 x 0.31 M 390 / 331.  Lead with two rows on
// their way, 64 x 25.6 M: 10 quarters 3326, 14 3306, 16 3313, 20 3441.
inline bool full_rows_paced(int n, int64_t ncg, int cus) {
    const int64_t from = n < 16 ? 2400 : n < 32 ? 800 : n < 48 ? 560 : 300;
    return n > 8 && ncg >= from * cus;
}
// Three to eight learners by the column groups of all of them (us, fp32 / bf16 gradients with the distance: 5 x 2.5 M 32.1 / 29.1, 35.1 / 28.1, 7 x 1.8 M
// 34.4 / 29.1, 36.0 / 27.3, 8 x 30 M 529 / 474, 437 / 403, 3 x 30 M 195 / 182, 191 / 159; 3 x 3 M 22.1 / 22.7, 23.9 / 23.0).
inline bool walk_full_rows(int n, int64_t ncg, int cus) {
    return n > 8 ? full_rows_paced(n, ncg, cus) : n > 2 && n * ncg >= 12000 * (int64_t)cus;
}
// The distance of two or three learners on long rows: small workgroups by themselves, not swept in batches of eight rows that they do not
// have (us, swept / alone, over three buffers in turn: 2 x 12 M 26.0 / 22.7, 2 x 24 M 45.8 / 39.4, 3 x 12 M 29.3 / 27.2, 3 x 30 M 65.8 / 57.6; 2 x 8.4 M, a fifth
// sweep that is nearly empty, 19.2 / 19.9, 3 x 8.4 M 21.9 / 22.6; 4 x 8 M 24.3 / 24.4, 5 x 8 M 27.6 / 28.9).
inline bool distance_alone(int n, int64_t ncg, int cus) { return n < 4 && ncg >= 10000 * (int64_t)cus; }
// Whether the partial sums of the distance's small workgroups are added up by a kernel of its own, not by the workgroup that is done last:
// from 192 MB of X on, where its launch is hidden behind the reading, and for more workgroups than three on each compute unit, which queue longer at
// the tickets.  us, last workgroup / kernel of its own: 117 x 1 320 544 98.6 / 93.9, 31 x 1 552 672 33.7 / 32.6, 42 x 1 383 552 40.1 / 39.2, 262 x 1 111 648
// 176.7 / 173.1, 202 x 860 489 113.6 / 112.4; the synchronous call 40 x 1 420 419 55.0 / 52.6, 75 x 1 126 016 70.4 / 67.6, 64 x 1 M 53.6 / 53.2.  Even at the line: 62 x
// 864 096 35.7 / 35.9, 59 x 996 255 41.4 / 41.9.  Below it: 27 x 786 464 16.7 / 17.7, 30 x 1 089 152 23.8 / 24.6, 66 x 603 168 (590 workgroups) 28.2 / 28.8.
// More than five on each from 120 MB on: 25 x 1 454 523 28.0 / 26.6, 32 x 1 363 200 31.1 / 30.2, 22 x 1 484 000 23.9 / 23.9.
inline bool distance_summed_apart(int grid, int n, int64_t d, int cus) { return grid > 3 * cus && n * d >= (grid > 5 * cus ? 30000000 : 48000000); }
// Rows on their way per lane in global averaging's walk, which needs more rows than that.
inline int full_depth(const SweepPlan& s, int n) { return n < 6 || s.chunk >= 576 ? 2 : 4; }
inline int full_lead(int depth) { return depth == 2 ? 16 : 7 * depth; }

// LDS of the tiled kernel (long rows, tables of other than three slots): the slot table (8 bytes per slot), TWO tile
// buffers of n rows x lpr lanes x 16 bytes (the next tile is staged while the current one is read), and, when the
// consensus distance is gathered in the same pass, the merge slots of the column sums: a double and a float (the row
// group's own pivot) per column and row group.  They go into the buffer that has just been read (one more barrier per tile)
// when they do not fit beside the two tiles.
// `lpr`, the lanes that share a row, is the largest power of two <= threads for which all of it fits `cap` and every row
// of a tile is in one batch, at most rows_per_batch rows per lane; at least 16 (256-byte row segments; also what keeps the
// lanes that share a column in the merge inside one wavefront).  lpr = 0 if there is none.
constexpr int kTileMinLpr = 16;
struct TilePlan {
    int lpr;
    bool comb_in_tile;
    size_t tab_bytes, tile_bytes, comb_bytes, total;
};
inline TilePlan tile_plan(int n, int deg, int threads, bool cd, size_t cap, int rows_per_batch) {
    TilePlan p;
    p.comb_in_tile = false;
    p.tab_bytes = (((size_t)n * deg * 8) + 15) & ~(size_t)15;
    for (p.lpr = threads; p.lpr >= kTileMinLpr; p.lpr >>= 1) {
        const int nrg = threads / p.lpr;
        if ((n + nrg - 1) / nrg > rows_per_batch) continue;
        p.tile_bytes = (size_t)n * p.lpr * 16;
        p.comb_bytes = cd ? (size_t)nrg * p.lpr * 48 : 0;
        p.total = p.tab_bytes + 2 * p.tile_bytes + p.comb_bytes;
        if (p.total <= cap) return p;
        if (cd && p.comb_bytes <= p.tile_bytes && p.total - p.comb_bytes <= cap) {
            p.comb_in_tile = true;
            p.total -= p.comb_bytes;
            return p;
        }
    }
    p.lpr = 0;
    return p;
}

// Whether long rows (two column groups for every lane of 768 per compute unit) of a table of other than three slots take the tiled
// kernel.  `room`: 2, every row of X and X_out starts on a 128-byte line; 1, on 16 bytes, and there are twice as many columns; 0, neither.
// Its tiles are a power of two of column groups wide, and as deep as a power of two of row groups: learners that fill them, 13 to 16, 29 to 32,
// 49 to 64 and 105 to 128, are as well off there or better, tables of many slots with the distance most (us, short-row / tiled: 64 x 2 M with 16
// slots and the distance 296 / 270, 30 x 3.2 M with 20 and bf16 gradients 303 / 215); the others leave places empty (on lines, with the distance, tiled /
// short-row: 9 x 6 M with 5 slots 156 / 119, with 32 264 / 190, 12 x 4 M 123 / 108, 20 x 4 M 204 / 178, 24 x 4 M 226 / 214, 33 x 3 M 276 / 225, 40 x 2 M 202 / 178, 48 x 2 M
// 225 / 213; off them, 16 slots and more, in times: 10 x 8 M 1.1 to 1.5, 24 x 4 M 1.02 to 1.2, 40 x 4 M 1.03 to 1.35).  13 to 16 learners on lines: only
// with the distance and 16 slots (14 x 6 M with 4 slots and none 193 / 180, with 16 and the distance 205 / 206).  Nearly filled, and without
// the distance: on lines 25 to 28 with 14 to 23 slots, 23 and 24 from 16, 43 to 48 from 18 (27 x 2.2 M with 23 slots 69 % of the short-row kernel's time, 28 x
// 2 003 296 bf16 with 21 86.7, 24 x 1 687 520 bf16 with 22 91.7, 27 x 2 890 912 bf16 with 14 83.4, 43 x 2 105 728 bf16 with 19 91.3, 47 x 1 981 024 bf16 with 21 87.7;
// with 24 a tile per workgroup is ahead, 44 x 2.4 M 253 / 298; 45 x 5 M with 17 103.5, 22 bf16 with 19 and 22 110); off the lines 25 to 28 from 16 on, the others from
// 20 (27 x 8 M with 22 79, 28 x 5.5 M bf16 with 25 84, 23 x 7 M with 23 95, 47 x 3.4 M bf16 with 24 90).
// 65 to 104: from 16 slots (with fewer the tiles take
// 97 to 114 % of the time, 103.5 on average over 60 shapes).  The largest tables halve the tile (128 x 1.6 M with 32 slots 1.6 to 1.8 times).  Off the lines few slots
// keep to it with 29 to 32 learners only (32 x 3 M with 13, short-row / tiled 236 / 220).
inline bool tiled_rows(int n, int deg, bool cd, int room) {
    if ((n > 22 && n < 29) || (n > 42 && n < 49)) {              // nearly filled
        const int from = n < 25 ? 16 : n < 29 ? 14 : 18;
        return !cd && (room == 2 ? deg >= from && deg < 24 : room == 1 && deg >= (n > 24 && n < 29 ? 16 : 20));
    }
    if (n < 13 || (n > 16 && n < 29) || (n > 32 && n < 49) || n > 128 || n * deg > 3840) return false;
    if (room < 2) return (n > 28 && n < 33) || (room == 1 && n <= 64 && deg >= 16);
    return n < 17 ? cd && deg >= 16 : n < 65 || n > 104 || deg >= 16;
}

// The short-row kernel's tile: all n rows x `1 << logc` column groups on `nrg` row groups of as many lanes (a multiple
// of 64 lanes in all), `rows` rows per lane, and its LDS: slot table (8 bytes per slot), the tile, and with the distance
// the merge slots (48 bytes per lane).
constexpr int kShortThreads = 1024;      // most lanes of its workgroups
constexpr int kShortRows = 4;            // most rows per lane where the next tile's rows are loaded ahead,
constexpr int kShortRowsOne = 8;         // and where a workgroup has one tile: what 128 registers hold in flight
constexpr size_t kShortLds = 160 * 1024 - 2048;
// A launch counts its lanes in 32 bits: one row of 2^34 columns at a tile per workgroup would be more than that (and would
// still fit the device).  Beyond these tiles the looping form, whose grid does not grow with the row.
constexpr int64_t kShortMostTiles = (int64_t)1 << 22;   // times up to 256 lanes
// With the distance, a workgroup has one partial sum: no more workgroups than the smallest buffer of them holds, whichever
// buffer the call uses, so that the form and with it the order of the sums do not depend on the entry point.
constexpr int64_t kShortSlots = 2048;
struct ShortPlan {
    bool one;                            // a tile per workgroup
    int threads, rows, logc, nrg;
    int tab_bytes, tile_bytes;
    int64_t tiles;
    size_t lds;
};
PSGD_HOST_DEVICE inline int short_table_bytes(int n, int deg) { return (n * deg * 8 + 15) & ~15; }
inline ShortPlan short_shape(int n, int deg, int64_t ncg, bool cd, bool one, int logc, int rows) {
    ShortPlan p;
    p.one = one;
    p.logc = logc;
    const int c = 1 << logc, whole = c < 64 ? 64 / c : 1;
    p.nrg = ((n + rows - 1) / rows + whole - 1) / whole * whole;
    p.rows = (n + p.nrg - 1) / p.nrg;
    if (one) p.rows = (p.rows + 1) & ~1;
    p.threads = p.nrg * c;
    p.tab_bytes = short_table_bytes(n, deg);
    p.tile_bytes = n * c * 16;
    p.tiles = (ncg + c - 1) >> logc;
    const int merge = cd && p.nrg > 1 ? p.threads * 48 : 0;
    if (one && p.tile_bytes < merge) p.tile_bytes = merge;
    p.lds = (size_t)p.tab_bytes + p.tile_bytes + (one ? 0 : merge);
    return p;
}
// The widest tile of at most `threads` lanes whose LDS fits.
inline ShortPlan short_widest(int n, int deg, int64_t ncg, bool cd, bool one, int threads, int rows) {
    ShortPlan p;
    for (int logc = 10; logc >= 0; --logc) {
        p = short_shape(n, deg, ncg, cd, one, logc, rows);
        if (p.threads <= threads && p.lds <= kShortLds) break;
    }
    return p;
}
// Which accesses of the short-row kernel go without the non-temporal hint.  `bytes`: X, G and X_out together;
// `on_lines`: every row of X and X_out starts on a 128-byte line.  (us, with the hint / without.)
//   - Loads where all arrays together take up to half of the 256 MB last-level cache and a workgroup has several tiles:
//     120 x 66 656 28.4 / 23.2, 24 x 333 312 23.1 / 20.5, 120 x 66 669 29.8 / 24.2 (stores too: 28.4); not beyond (192 MB, 16 x 1 M:
//     35.2 / 36.2), nor with one tile each (64 x 100 k with bf16 gradients 11.2 / 11.6).
//   - Loads and stores where rows are off the lines: neighbouring tiles share a line at every row's end, and a hinted line
//     travels twice.  Up to 128 column groups wide: 512 x 78 125 166 / 117, 200 x 200 013 131 / 110, 64 x 1 874 989 325 / 301,
//     24 x 5 000 013 287 / 280; wider tiles lose (16 x 2 500 013 94 / 97), as do rows on lines (512 x 78 112 97 / 103); one tile each, up
//     to 16 wide: 512 x 15 629 30.2 / 25.7 (128 wide, 64 x 125 005: 22.9 / 23.6).
//   - Loads where bf16 gradients come in segments of half a line (8 column groups): neighbouring tiles share that line too.
//     512 x 800 k without the distance 979 / 887, 300 x 800 k 570 / 502, with it 512 x 200 k 237 / 208.
enum { kCachedLoads = 1, kCachedStores = 2 };
inline int cached_accesses(const ShortPlan& p, int64_t bytes, bool on_lines, bool bf16) {
    if (!p.one && bytes <= (int64_t)128 << 20) return kCachedLoads;
    if (!on_lines && p.logc <= (p.one ? 4 : 7)) return kCachedLoads | kCachedStores;
    return bf16 && !p.one && p.logc <= 3 ? kCachedLoads : 0;
}
// Workgroups of the looping form: one per tile up to what is resident together (128 registers per lane at four rows:
// 1024 lanes per compute unit), at most `most`.
inline int short_grid(const ShortPlan& p, int cus, int64_t most) {
    int64_t per_cu = kShortThreads / p.threads;
    if (per_cu > (int64_t)(kShortLds / p.lds)) per_cu = kShortLds / p.lds;
    int64_t g = cus * per_cu;
    if (g > p.tiles) g = p.tiles;
    if (g > most) g = most;
    return (int)(g < 1 ? 1 : g);
}
// Tiles of global averaging and of the distance with rows spread over row groups of lanes: at most `rows` rows per lane,
// the widest tile of at most `threads` lanes.  threads == 0: the columns alone fill the chip, a lane walks all rows.
struct RowsPlan {
    int threads, logc, nrg;
    int64_t tiles;
};
inline RowsPlan rows_shape(int n, int64_t ncg, int threads, int rows) {
    RowsPlan p;
    for (p.logc = 10; p.logc >= 0; --p.logc) {
        const int c = 1 << p.logc, whole = c < 64 ? 64 / c : 1;
        p.nrg = ((n + rows - 1) / rows + whole - 1) / whole * whole;
        p.threads = p.nrg * c;
        p.tiles = (ncg + c - 1) >> p.logc;
        if (p.threads <= threads) break;
    }
    return p;
}
// As for the short-row kernel, one round of at most one workgroup per compute unit where that holds everything (the
// widest workgroup that occupies more than half of them), on eight rows per lane, or up to `most_rows`; many learners
// beyond it take more rows per lane, up to where the columns alone do as well.  us, lane per column group / rows spread:
// global averaging with the distance 512 x 6 k 175 / 13.4, 64 x 100 k 28.8 / 19.5, 512 x 60 k 187 / 69, 82 x 90 k 38 / 22, 128 x 200 k
// 61.6 / 60.8, 64 x 300 k 49.4 / 49.7; distance alone 512 x 6 k 52 / 8.5, 64 x 100 k 11.4 / 9.2, 512 x 60 k 54 / 23, 127 x 90 k 18 / 12,
// 128 x 200 k 20.2 / 22.3.
// `least`: the fewest learners.
inline RowsPlan rows_plan(int n, int64_t ncg, int cus, int most_threads, int most_rows, int least) {
    if (ncg == 1) return rows_shape(n, ncg, 256, 8);             // also the only form for fewer than four columns
    if (n >= least) {
        for (int rows = 8; rows <= most_rows; rows *= 2) {
            for (int threads = most_threads; threads >= 256; threads /= 2) {
                const RowsPlan p = rows_shape(n, ncg, threads, rows);
                if (p.tiles > cus) break;
                if (p.tiles > cus / 2 || threads == 256) return p;
            }
        }
        if (n > 64 && ncg < (int64_t)cus * 128)
            return most_threads > 512 && n < 128 ? rows_shape(n, ncg, most_threads, 16) : rows_shape(n, ncg, 512, 32);
    }
    return RowsPlan{0, 0, 0, 0};
}
// Global averaging passes twice over the rows: from 17 learners on, a lane walking all of them is behind on few columns, from
// 10 on at 4000 columns and more (us, lane / spread: 12 x 50 k 9.2 / 8.5, with bf16 gradients and no distance 5.3 / 4.7; 12 x 1000 6.5 / 7.7; 9 x
// 200 k 9.1 / 10.2), ragged rows earlier (13 x 1599 5.2 / 4.4); with the distance and whole column groups not for ten (10 x 164 k
// 7.0 / 9.0), for 16, whole batches of eight, from 160 000 (16 x 50 k 8.4 / 8.9, 16 x 200 k 11.3 / 11.0).
inline RowsPlan full_rows_plan(int n, int64_t d, int cus, bool cd) {
    const int64_t ncg = (d + 3) / 4;
    const int64_t from = d % 4 ? 230 : cd && n == 16 ? 40000 : cd && n == 10 ? INT64_MAX : 1000;
    return rows_plan(n, ncg, cus, kShortThreads, 8, ncg < from ? 17 : 10);
}
// The distance passes once: from 48 learners on, from 30 where rows are ragged and not the shortest (42 x 50 001 8.3 / 6.3; 36 x
// 20 k 5.9 / 6.0; 33 x 566 4.9 / 5.7).
inline RowsPlan distance_rows_plan(int n, int64_t d, int cus) {
    return rows_plan(n, (d + 3) / 4, cus, 512, 16, d % 4 && d >= 4000 ? 30 : 48);
}

// Most lanes per compute unit, over the whole launch, at which two rows per lane are the better form (short_plan): 384
// where a row has few slots, or few and the distance's merge, more the wider the table; fewer where row segments are a
// line or less.  us, eight rows per lane / two, on the far side of the lines: 25 x 38 k 8.2 / 9.4, 30 x 68 k with 5 slots
// 11.0 / 13.9 (both with the distance), 85 x 21.7 k with 5 slots and none 7.6 / 8.8 (128-byte segments).
inline int two_rows_lanes(int n, int deg, bool cd, int logc) {
    if (cd && n < 5) return 256;
    int most = deg <= 3 || (cd && deg < 8) ? 384 : 960;
    if (!cd && deg > 3) {
        if (deg < 8) most = logc > 4 ? 1024 : logc == 4 ? 640 : 512;
        else most = logc <= 3 ? 1024 : deg < 16 ? 1280 : 1536;
    }
    if (logc < 3 && most > 512) most = 512;
    return cd && n < 8 && most > 768 ? 768 : most;
}
// The looping form: 1024 lanes, up to four rows each.
inline ShortPlan short_loop_plan(int n, int deg, int64_t ncg, bool cd) {
    // A lane without a row of its own repeats the last one, loads and stores alike: fewer rows per lane where that leaves
    // fewer such places, unless the tile then narrows below a wavefront's 64 column groups (13 x 3.9 M, 16 places at four
    // rows, 14 at two: 131 and 119 us; 200 x 250 k, 208 at four, 204 at three on half the width: 131 and 143), or from 128 with
    // the distance and 20 to 28 learners (28 places, 26 on half the width: 26 x 2 M 126 / 134, with 13 slots 131 / 156).
    ShortPlan best = short_widest(n, deg, ncg, cd, false, kShortThreads, kShortRows);
    for (int rows = kShortRows - 1; rows >= 2; --rows) {
        const ShortPlan p = short_widest(n, deg, ncg, cd, false, kShortThreads, rows);
        if (p.nrg * p.rows < best.nrg * best.rows && (p.logc == best.logc || (p.logc >= 6 && (!cd || n < 20 || n > 28))))
            best = p;
    }
    return best;
}
// The tiles of a table that is not one ring, on rows that the ring walk would take.  Up to eight learners: 512 lanes of four rows, with the distance
// and five to seven of them 1024 lanes of two (us, short_plan's, which it was / 512 lanes of four / 1024 of two: 3 x 9 M 58.7 / 56.8 / 74.4, 4 x 6 M 54.2 / 52.1
// / 56.5, 8 x 24 M 408 / 391 / 413; with the distance 5 x 11.1 M 126.1 / 131.5 / 124.2, bf16 gradients 5 x 24.6 M 230 / 240 / 229, 6 x 21.3 M 232 / 243 / 233, fp32 6 x 6.2 M 79.9 / 80.9
// / 80.3, off the lines 7 x 15.6 M 254 / 259 / 254; not six of fp32 off the lines, 24.3 M 315 / 305 / 320, nor eight, 14.2 M 242 / 235 / 242; seven without it stay behind, 7 x 31.3 M 451 / 463, bf16 7 x 20 M 239 / 252, where one ring is ahead,
// 484 / 431).
// With the next gradients at most three rows: more than that the registers do not hold.  Beyond
// 384 learners that would leave segments of 64 bytes: the next gradients are made in front of the tiles, which keep four rows (436 x 257 984 620 with them,
// 523 apart, 446 x 297 344 806 / 668, 470 x 196 608 599 / 512, off the lines 507 x 244 161 705 / 659).
inline bool tiles_produce(int n) { return n <= 384; }
inline ShortPlan ring_tiles(int n, int64_t ncg, bool cd, bool produce, bool fp32_off_lines) {
    const bool two = cd && (n == 5 || n == 7 || (n == 6 && !fp32_off_lines));
    if (n < 9) return produce || two ? short_widest(n, 3, ncg, cd, false, kShortThreads, 2) : short_widest(n, 3, ncg, cd, false, 512, 4);
    const ShortPlan p = short_loop_plan(n, 3, ncg, cd);
    return produce && tiles_produce(n) && p.rows > 3 ? short_widest(n, 3, ncg, cd, false, kShortThreads, 3) : p;
}
// Which tile a launch takes (fp32 gradients, with the distance unless said otherwise, kernel + final sum):
//   - few columns: two rows per lane, on as few lanes as leave a row segment of a 128-byte line.  A lane reads its rows'
//     slots from LDS one after the other; with eight rows each on a few workgroups that chain is the launch.  Eight rows /
//     two, without the distance: 8 x 20 k with 5 slots 5.1 / 3.8, with 32 12.6 / 4.4; 64 x 20 k with 13 8.3 / 4.9; ring of 8 x 61 k
//     with it 7.1 / 6.1;
//   - wide tables on rows that start on 16 bytes (`quads`), where LDS reads are the bound: two rows per lane, a tile per
//     workgroup of 512 lanes.  Without the distance, bf16 gradients: 8 x 700 k with 13 slots 15.7 / 12.1, 16 x 1.4 M with 32
//     71 / 49; fp32 32 x 410 k with 32 54 / 34; with it 8 x 700 k with 32 29.5 / 23.9.  On other rows it loses (20 x 941 559 with 20 slots
//     55 / 64), as with fewer slots (45 x 1.2 M with 16 119 / 138);
//   - everything in one round of at most one workgroup per compute unit, eight rows per lane: the whole chip's loads
//     are in flight at once.  8 learners x 1 M without the distance 15.7 us, looping over narrower tiles 18.9; 64 x 100 k
//     17.9 against 21.2.  The widest workgroup that still occupies more than half of the compute units: 16 x 250 k at
//     512 lanes (245 tiles) 12.4, at 1024 (123 tiles) 15.2;
//   - up to 8 learners beyond that: a lane holds all rows of its columns, nothing is exchanged and small independent
//     workgroups hide each other's latency: 8 x 1.5 M 30.3, looping 32.2; up to kShortMostTiles of them, with the distance
//     kShortSlots, of twice the lanes from five learners on (5 x 4 M 47, looping 54; 7 x 4 M 64 / 72; 2 x 2.5 M 15.8 / 14.4; wide
//     tables loop);
//   - five to eight learners of longer rows, with the distance: looping, two rows per lane (5 x 30 M with bf16 gradients 307
//     on three rows, 289 on two; 7 x 8 M 135 / 124);
//   - all else: 1024 lanes, four rows each, the next tile's loads ahead: 512 x 60 k 77.6 us, at 512 lanes 107;
//     64 x 1 M with bf16 gradients 126 against 130.
inline ShortPlan short_plan(int n, int deg, int64_t ncg, int cus, bool cd, bool quads) {
    if (n > 2 && (!cd || n > 5 || deg >= (n > 4 ? 4 : 9))) {
        for (int threads = 256; threads <= kShortThreads; threads *= 2) {
            const ShortPlan p = short_widest(n, deg, ncg, cd, true, threads, 2);
            if (p.threads > threads || (p.logc < 3 && threads < kShortThreads)) continue;
            if (p.tiles * p.threads <= (int64_t)cus * two_rows_lanes(n, deg, cd, p.logc) && (!cd || p.tiles <= kShortSlots)) return p;
        }
    }
    if (quads && n > 4 && (cd ? n <= 8 && deg >= 20 : n <= 8 ? deg >= 7 : n <= 16 ? deg >= 16 : n <= 48 && deg >= 24)) {
        const ShortPlan p = short_widest(n, deg, ncg, cd, true, 512, 2);
        if (p.tiles <= (cd ? kShortSlots : kShortMostTiles)) return p;
    }
    for (int threads = kShortThreads; threads >= 256; threads /= 2) {
        const ShortPlan p = short_widest(n, deg, ncg, cd, true, threads, kShortRowsOne);
        if (p.threads > threads || p.tiles > cus) break;
        if (p.tiles > cus / 2 || threads == 256) return p;
    }
    if (n <= kShortRowsOne) {
        for (int threads = 256; threads <= (cd && n > 4 && deg < 16 ? 512 : 256); threads *= 2) {
            const ShortPlan p = short_widest(n, deg, ncg, cd, true, threads, kShortRowsOne);
            if (p.tiles <= (cd ? kShortSlots : kShortMostTiles)) return p;
        }
        if (n > 4) return short_widest(n, deg, ncg, cd, false, kShortThreads, 2);
    }
    return short_loop_plan(n, deg, ncg, cd);
}

// Whether the short-row kernel also makes the next gradients of the delay-by-one schedule, or a producer behind it does: not on one round of
// large workgroups whose row segments are 256 bytes or less, five arrays of which lie badly (us, 512 x 15 000 in one pass / two launches 41.1 / 39.4,
// without the distance 39.6 / 35.5; 400 x 15 000 30.6 / 33.5, 29.1 / 28.8; 300 x 10 000, smaller workgroups, 15.0 / 21.8); nor off the lines in loops over
// segments as short, from where five arrays are more than the last-level cache holds (on the arrays of the schedule, in turn: 498 x 43 411 108.7 / 94.2,
// 257 x 61 035 76.7 / 69.0, 463 x 51 433 125.6 / 112.7, 142 x 130 547 88.5 / 81.2, 306 x 145 227 209 / 206; below it 381 x 33 063 51.1 / 58.4, 173 x 67 547 44.1 / 52.0; on the
// lines 393 x 80 736 131 / 141, 439 x 86 240 157 / 167).
inline bool short_produces(const ShortPlan& p, int64_t elements, bool on_lines) {
    return p.one ? p.threads <= 768 || p.logc > 4 : p.rows > 1 && (on_lines || p.logc > 4 || elements <= 13500000);
}
// Bytes that the choice of cached_accesses goes by: X, G and X_out; with the next gradients off the lines noise and G_next too.  With three counted
// the loads alone were kept from 7 to 11 M elements, where both are better (on the arrays of the schedule, in turn, loads / both: 393 x 24 927 53.2 / 36.0,
// 148 x 67 855 45.6 / 33.9, 67 x 138 907 41.6 / 35.2; on the lines neither matters, 92 x 93 152 30.0 / 29.9).
inline int64_t counted_bytes(int64_t elements, int gradient, bool next_gradients, bool on_lines) {
    return elements * (8 + gradient + (next_gradients && !on_lines ? 8 : 0));
}

}  // namespace plan
}  // namespace psgd

#endif
