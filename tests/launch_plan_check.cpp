// CPU check of the launch arithmetic in psgd_internal.h (built and run by tests/test_library_host.py).
// Every column group must be owned by exactly one (sweep, workgroup) range, ranges must start on a
// 256-byte boundary, every workgroup must make the same number of sweeps, and no grid may exceed the
// partials buffer, whatever the device reports.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <vector>

#include "psgd_internal.h"

using namespace psgd::plan;

static int failures = 0;
#define CHECK(cond, ...)                       \
    do {                                       \
        if (!(cond)) {                         \
            std::printf("FAIL: " __VA_ARGS__); \
            std::printf("\n");                 \
            ++failures;                        \
        }                                      \
    } while (0)

static void check_cover(int64_t ncg, int grid, int threads, bool even = true) {
    const SweepPlan p = sweep_plan(ncg, grid, threads, even);
    CHECK(p.chunk >= 1 && p.chunk <= threads, "ncg=%lld grid=%d: chunk %lld", (long long)ncg, grid, (long long)p.chunk);
    CHECK(p.count < 4 || p.chunk % kChunkAlign == 0, "ncg=%lld grid=%d: chunk %lld unaligned", (long long)ncg, grid,
          (long long)p.chunk);
    // ranges are consecutive in (sw * grid + b): they tile [0, count * grid * chunk), which must reach ncg,
    // and the range before the last sweep must not already have reached it (no sweep without work at all)
    const int64_t covered = p.count * grid * p.chunk;
    CHECK(covered >= ncg, "ncg=%lld grid=%d T=%d: only %lld covered", (long long)ncg, grid, threads, (long long)covered);
    CHECK(p.count == 0 || (p.count - 1) * grid * p.chunk < ncg, "ncg=%lld grid=%d T=%d: an empty sweep", (long long)ncg,
          grid, threads);
    // walk the ranges the way the kernel does and count owners of a few thousand probe groups
    const int64_t probes[] = {0, 1, p.chunk - 1, p.chunk, p.chunk + 1, ncg / 2, ncg - p.chunk, ncg - 2, ncg - 1};
    for (int64_t g : probes) {
        if (g < 0 || g >= ncg) continue;
        int owners = 0;
        const int64_t slot = g / p.chunk;           // the only range that can hold it
        for (int64_t s = slot > 0 ? slot - 1 : 0; s <= slot + 1; ++s) {
            const int64_t sw = s / grid, b = s % grid;
            if (sw >= p.count) continue;
            const int64_t base = (sw * grid + b) * p.chunk;
            if (base >= ncg) continue;
            const int64_t end = base + p.chunk < ncg ? base + p.chunk : ncg;
            if (g >= base && g < end && g - base < threads) ++owners;
        }
        CHECK(owners == 1, "ncg=%lld grid=%d T=%d: group %lld has %d owners", (long long)ncg, grid, threads,
              (long long)g, owners);
    }
}

// The counters of the distance's last sum as the kernels use them: a draw adds one, or puts back to zero at the last of `of`.
struct Counters {
    std::vector<int> value = std::vector<int>(kTicketCounters, 0), of = std::vector<int>(kTicketCounters, 0);
    bool draw(Ticket t) {
        CHECK(t.at >= 0 && t.at < kTicketCounters && t.of >= 1 && (of[t.at] == 0 || of[t.at] == t.of), "counter %d drawn from as of %d and of %d", t.at, of[t.at], t.of);
        if (t.at < 0 || t.at >= kTicketCounters) return false;
        of[t.at] = t.of;
        const int old = value[t.at];
        value[t.at] = old >= t.of - 1 ? 0 : old + 1;
        return old == t.of - 1;
    }
    bool last(int block, int grid) { return (!ticket_leaves(grid) || draw(ticket_leaf(block, grid))) && draw(ticket_root(grid)); }
};
static void check_tickets() {
    std::srand(1);
    Counters c;
    // launches that a caller let overlap, their workgroups interleaved, and behind them launches in order: every one of these has one last
    // workgroup, and it is the one that came last
    for (int round = 0; round < 400; ++round) {
        std::vector<int> grids, blocks;
        for (int k = 0; k < 2 + round % 3; ++k) {
            const int g = round % 5 == 4 ? kMaxGrid - k : 1 + std::rand() % (round % 2 ? 80 : 700);
            grids.push_back(k && round % 4 == 0 ? grids[0] : g);
            blocks.push_back(0);
        }
        for (;;) {
            std::vector<int> open;
            for (size_t k = 0; k < grids.size(); ++k)
                if (blocks[k] < grids[k]) open.push_back((int)k);
            if (open.empty()) break;
            const int k = open[std::rand() % open.size()];
            (void)c.last(blocks[k]++, grids[k]);
        }
        for (int g : {grids[0], grids[1], 1 + std::rand() % kMaxGrid, 16, 64, 65, 66, 80, 512}) {
            int lasts = 0, where = -1;
            const int first = std::rand() % g;                  // in any order
            for (int b = 0; b < g; ++b)
                if (c.last((first + b) % g, g)) { ++lasts; where = b; }
            CHECK(lasts == 1 && where == g - 1, "%d workgroups: %d of them the last, place %d", g, lasts, where);
        }
    }
    for (int g = 1; g <= kMaxGrid; ++g)
        for (int b = 0; b < g; ++b) (void)c.last(b, g);
    for (int k = 0; k < kTicketCounters; ++k) CHECK(c.value[k] == 0, "counter %d ends at %d", k, c.value[k]);
}

int main() {
    check_tickets();
    // the five workloads' rows in 128-bit column groups, the grids an MI355X gives them, and odd neighbours
    const int64_t rows[] = {250000, 8000000, 6400000, 2000000, 25000000, 1, 15, 16, 17, 767, 768, 769, 196608, 196609,
                            786431, 786432, 786433, 123456789, (1ll << 31) + 257, (1ll << 33) + 5};
    const int grids[] = {1, 2, 7, 255, 256, 304, 1024, 4096};
    const int threads[] = {256, 768};
    for (int64_t ncg : rows)
        for (int g : grids)
            for (int t : threads) {
                check_cover(ncg, g, t);
                check_cover(ncg, g, t, false);
            }
    // the die-contiguous mapping permutes the ranges of a sweep among the workgroups: a bijection, and the
    // workgroups of one die (b, b + 8, ...) take neighbouring ranges
    for (int grid : {1, 7, 8, 16, 255, 256, 304, 1024}) {
        std::vector<int> seen(grid, 0);
        for (int b = 0; b < grid; ++b) {
            const int64_t s = die_contiguous_slot(b, grid, 8);
            CHECK(s >= 0 && s < grid, "grid %d: slot %lld of workgroup %d", grid, (long long)s, b);
            if (s >= 0 && s < grid) ++seen[s];
        }
        for (int i = 0; i < grid; ++i) CHECK(seen[i] == 1, "grid %d: range %d taken %d times", grid, i, seen[i]);
        if (grid % 8 == 0 && grid >= 16)
            CHECK(die_contiguous_slot(8, grid, 8) == die_contiguous_slot(0, grid, 8) + 1, "grid %d: die neighbours", grid);
        else if (grid % 8 != 0)
            CHECK(die_contiguous_slot(grid - 1, grid, 8) == grid - 1, "grid %d: identity expected", grid);
    }
    // workload 5 on 256 compute units: 128 sweeps of 768-group chunks, the last range 64 groups long
    const SweepPlan w5 = sweep_plan(25000000, 256, 768);
    CHECK(w5.count == 128 && w5.chunk == 768, "workload 5 plan %lld x %lld", (long long)w5.count, (long long)w5.chunk);
    // workload 4: 10.2 sweeps' worth of groups take 11 sweeps of 720-group chunks (not 11 of 768)
    const SweepPlan w4 = sweep_plan(2000000, 256, 768);
    CHECK(w4.count == 11 && w4.chunk == 720, "workload 4 plan %lld x %lld", (long long)w4.count, (long long)w4.chunk);

    CHECK(sweep_plan(275000, 1024, 256, false).chunk == 256 && sweep_plan(275000, 1024, 256).chunk == 144, "full chunks where sweeps are short");
    // the ring walk's workgroups: every column group has a lane, and no wavefront of a single sweep is without one
    for (int64_t ncg : {(int64_t)1, (int64_t)49152, (int64_t)52500, (int64_t)88474, (int64_t)196608, (int64_t)196609, (int64_t)25000000}) {
        const SweepPlan p = sweep_plan(ncg, 256, 768);
        const int t = ring_threads(p, 768);
        CHECK(t % 64 == 0 && t <= 768 && t >= p.chunk && (p.count > 1 ? t == 768 : t < p.chunk + 64), "ring walk: %d lanes for chunks of %lld",
              t, (long long)p.chunk);
    }

    // the ring walk at every length of row: its workgroups are no larger than the depth's kernel is built for, and no load is issued
    // further ahead than the end of the next sweep
    for (int cus : {1, 64, 256, 304})
        for (int64_t ncg = 1; ncg < (int64_t)1 << 34; ncg += ncg / 7 + 16)
            for (int n : {3, 4, 5, 6, 8, 9, 10, 15, 16, 17, 64, 512}) {
                const SweepPlan p = sweep_plan(ncg, cus, kRingLanes);
                const int depth = ring_depth(p, n), t = ring_threads({1, p.chunk}, kRingLanes) + 64;
                CHECK(t <= kRingThreadsMost && t - 64 >= p.chunk && t % 64 == 0, "ring walk: %d lanes, depth %d, chunk %lld", t, depth,
                      (long long)p.chunk);
                CHECK((depth == 1 || depth == 2 || depth == 4 || depth == 6) && n - 1 + 2 + depth < 2 * n, "ring walk: depth %d, n %d", depth, n);
                CHECK(pace_lead(depth) >= 4 * depth && kPaceSpins > 0, "ring walk: a lead that the loads on their way need");
            }

    // grids never exceed the partials buffer, however many compute units a device reports
    for (int cus : {1, 64, 256, 304, 512, 513, 1024, 100000})
        for (int per_cu : {1, 4, 8}) {
            for (int64_t items : {(int64_t)0, (int64_t)1, (int64_t)255, (int64_t)256, (int64_t)1 << 20, (int64_t)1 << 40}) {
                const int g = persistent_grid(cus, items, per_cu, 256);
                CHECK(g >= 1 && g <= kMaxGrid, "persistent_grid(%d, %lld, %d) = %d", cus, (long long)items, per_cu, g);
                CHECK((int64_t)g <= (int64_t)cus * per_cu || g == 1, "persistent_grid above residency");
                const int dg = deg_grid(items, cus, per_cu);
                CHECK(dg >= 1 && dg <= kMaxGrid, "deg_grid(%lld, %d, %d) = %d", (long long)items, cus, per_cu, dg);
                CHECK(items < 1 || dg <= items, "deg_grid above the tile count");
            }
        }
    CHECK(persistent_grid(256, 25000000, 1, 768) == 256, "workload 5 grid");
    // global averaging and the distance with the columns spread over workgroups: within the buffer, every column group once, evened out
    // only where measured to gain
    for (int cus : {1, 64, 256, 304, 1024})
        for (int n : {1, 2, 9, 15, 16, 24, 25, 64, 95, 96, 512})
            for (int64_t ncg : {1, 257, 16384, 33000, 50704, 68560, 99999, 118750, 140000, 199999, 262144, 393215})
                for (int g : {full_grid(n, ncg, cus, 4, 256), distance_grid(n, ncg, cus, 8, 256)}) {
                    CHECK(g >= 1 && g <= kMaxGrid, "n=%d ncg=%lld: grid %d", n, (long long)ncg, g);
                    check_cover(ncg, g, 256);
                    check_cover(ncg, g, 256, false);
                }
    const struct { int n; int64_t d; bool apart; } summed[] = {{27, 786464, false}, {30, 1089152, false}, {40, 1149088, false}, {31, 1552672, true}, {66, 603168, false},
                                                               {178, 671232, false}, {64, 1000000, true}, {117, 1320544, true}, {16, 1000000, false},
                                                               {25, 1454523, true}, {20, 1474931, false}, {30, 1262304, false}};
    for (const auto& e : summed)
        CHECK(distance_summed_apart(distance_grid(e.n, (e.d + 3) / 4, 256, 8, 256), e.n, e.d, 256) == e.apart, "n=%d d=%lld: last sum", e.n, (long long)e.d);
    const struct { int n; int64_t d; int full, distance; } evened[] = {
        {4, 458912, 449, 449}, {6, 266400, 261, 261}, {9, 475584, 465, 465}, {15, 299507, 293, 293}, {16, 299507, 512, 293}, {17, 402112, 393, 393},
        {23, 414464, 405, 405}, {25, 299507, 512, 512}, {33, 198253, 194, 194}, {33, 160000, 256, 157}, {52, 242112, 237, 237}, {39, 529933, 768, 768},
        {28, 690496, 675, 768}, {144, 209472, 256, 205}, {192, 226815, 222, 222}, {64, 1000000, 977, 977}, {77, 271744, 512, 512}, {74, 164288, 256, 161}};
    for (const auto& e : evened)
        CHECK(full_grid(e.n, (e.d + 3) / 4, 256, 4, 256) == e.full && distance_grid(e.n, (e.d + 3) / 4, 256, 8, 256) == e.distance, "n=%d d=%lld: %d and %d workgroups",
              e.n, (long long)e.d, full_grid(e.n, (e.d + 3) / 4, 256, 4, 256), distance_grid(e.n, (e.d + 3) / 4, 256, 8, 256));
    CHECK(persistent_grid(256, 1000, 4, 256) == 4, "short rows take one workgroup per 256 items");
    CHECK(deg_grid(1 << 30, 1024, 8) == kMaxGrid, "deg_grid clamp");
    // LDS plan of the tiled path: the widest power-of-two lane count whose slot table, two tile buffers and merge slots
    // fit, every row of a tile in one batch; the merge slots (48 KB at 1024 lanes) inside the consumed tile buffer when they
    // do not fit beside the two tiles.  Every table of the learners it serves (9 to 128) has a plan.
    const size_t large = 160 * 1024 - 1024;
    for (int n : {1, 2, 3, 5, 8, 9, 16, 20, 32, 48, 64, 65, 70, 128, 200, 256, 257, 512})
        for (int deg : {1, 3, 5, 13, 32})
            for (int threads : {512, 1024})
                for (bool cd : {false, true}) {
                    if ((long)n * deg > 4096) continue;
                    const int rpb = threads == 1024 ? 4 : 8;
                    const TilePlan p = tile_plan(n, deg, threads, cd, large, rpb);
                    if (p.lpr == 0) {
                        CHECK(n > 128, "n=%d deg=%d cd=%d has no tile", n, deg, (int)cd);
                        continue;
                    }
                    const int nrg = threads / p.lpr;
                    CHECK(p.lpr >= 16 && (p.lpr & (p.lpr - 1)) == 0 && (n + nrg - 1) / nrg <= rpb, "tile shape: lpr %d", p.lpr);
                    CHECK(nrg <= 64, "n=%d: %d row groups, the lanes of a column would not fit a wavefront", n, nrg);
                    CHECK(p.tab_bytes >= (size_t)n * deg * 8 && p.tab_bytes % 16 == 0, "slot table size");
                    CHECK(p.tile_bytes >= (size_t)n * p.lpr * 16 && p.tile_bytes % 16 == 0, "tile size");
                    CHECK(p.comb_bytes == (cd ? (size_t)nrg * p.lpr * 48 : 0), "merge slots");
                    CHECK(p.total == p.tab_bytes + 2 * p.tile_bytes + (p.comb_in_tile ? 0 : p.comb_bytes) && p.total <= large, "total");
                    CHECK(!p.comb_in_tile || (cd && p.comb_bytes <= p.tile_bytes), "merge slots inside a tile buffer must fit it");
                }
    {
        const TilePlan p = tile_plan(64, 13, 1024, true, large, 4);
        CHECK(p.lpr == 64 && p.comb_in_tile, "n = 64, 13 slots, distance: 1 KB row segments, merge slots in the tile");
        CHECK(tile_plan(64, 3, 1024, false, large, 4).lpr == 64, "n = 64 without the distance");
        CHECK(tile_plan(64, 13, 512, true, large, 8).lpr == 64 && !tile_plan(64, 13, 512, true, large, 8).comb_in_tile,
              "n = 64 with the distance at 512 lanes: merge slots beside the tiles");
        CHECK(tile_plan(64, 32, 512, true, large, 8).lpr == 64 && tile_plan(64, 32, 512, true, large, 8).comb_in_tile,
              "n = 64, 32 slots, distance: merge slots in the tile");
        CHECK(tile_plan(16, 3, 1024, true, large, 4).lpr == 256, "n = 16: 4 KB row segments, 4 rows per lane");
        CHECK(tile_plan(8, 3, 1024, true, large, 4).lpr == 512, "n = 8: 8 KB row segments");
        CHECK(tile_plan(128, 3, 1024, false, large, 4).lpr == 32, "n = 128: 512-byte row segments, 32 row groups of 4 rows");
        CHECK(tile_plan(128, 3, 512, true, large, 8).lpr == 32, "n = 128 with the distance: 16 row groups of 8 rows");
        CHECK(tile_plan(256, 3, 1024, false, large, 4).lpr == 16, "n = 256: 256-byte row segments");
        CHECK(tile_plan(257, 3, 1024, false, large, 4).lpr == 0, "n = 257: no plan");
    }
    // which tables of other than three slots on long rows take the tiled kernel; every one of them has a plan at both sizes of its workgroups
    const struct { int n, deg; bool cd; int room; bool tiled; } tables[] = {
        {12, 16, true, 2, false}, {13, 16, true, 2, true}, {14, 15, true, 2, false}, {16, 32, true, 2, true}, {16, 32, false, 2, false}, {16, 5, true, 2, false},
        {17, 20, true, 2, false}, {22, 20, false, 2, false}, {23, 16, false, 2, true}, {24, 15, false, 2, false}, {25, 14, false, 2, true}, {27, 23, false, 2, true}, {28, 24, false, 2, false}, {28, 20, true, 2, false},
        {28, 20, false, 1, true}, {28, 32, false, 1, true}, {24, 20, false, 1, true}, {24, 19, false, 1, false}, {44, 20, false, 1, true}, {44, 20, true, 1, false}, {27, 20, false, 0, false}, {29, 4, false, 0, true}, {30, 13, true, 2, true}, {32, 32, true, 1, true}, {33, 20, false, 2, false}, {42, 20, false, 2, false},
        {43, 18, false, 2, true}, {43, 17, false, 2, false}, {48, 23, false, 2, true}, {48, 24, false, 2, false}, {49, 4, true, 2, true}, {60, 16, true, 1, true}, {60, 15, true, 1, false}, {60, 16, true, 0, false},
        {64, 13, false, 2, true}, {65, 15, true, 2, false}, {70, 13, false, 2, false}, {100, 16, true, 2, true}, {104, 5, false, 2, false}, {105, 5, true, 2, true}, {113, 5, false, 2, true},
        {113, 16, false, 1, false}, {120, 32, false, 2, true}, {128, 30, true, 2, true}, {128, 32, false, 2, false}, {129, 5, true, 2, false}};
    for (const auto& e : tables) CHECK(tiled_rows(e.n, e.deg, e.cd, e.room) == e.tiled, "n=%d deg=%d cd=%d room=%d: tiled kernel", e.n, e.deg, (int)e.cd, e.room);
    for (int n = 1; n <= 512; ++n)
        for (int deg = 1; deg <= 32 && n * deg <= 4096; ++deg)
            for (int form = 0; form < 6; ++form) {
                const bool cd = form & 1;
                if (!tiled_rows(n, deg, cd, form >> 1)) continue;
                const TilePlan p = tile_plan(n, deg, cd ? 512 : 1024, cd, large, cd ? 8 : 4);
                CHECK(p.lpr >= 16 && p.total <= large, "n=%d deg=%d cd=%d: no tile", n, deg, (int)cd);
            }
    // where the ring walk and the paced global averaging run: each band of learners from its line on (column groups per compute unit)
    const struct { int lo, hi; int64_t line; } bands[] = {{9, 11, 3600}, {12, 15, 2500}, {16, 23, 1600}, {24, 31, 800}, {32, 47, 560},
                                                          {48, 95, 400}, {96, 199, 307}, {200, 255, 230}, {256, 512, 192}};
    const struct { int lo, hi; int64_t line; } full_bands[] = {{9, 15, 2400}, {16, 31, 800}, {32, 47, 560}, {48, 512, 300}};
    for (int cus : {64, 256, 304})
        for (const auto& b : bands)
            for (int n = b.lo; n <= b.hi; ++n)
                for (int64_t ncg : {b.line * cus - 1, b.line * cus, b.line * cus + 1, b.line * cus * 3 + 7, b.line * cus * 40 + 1}) {
                    CHECK(ring_rows(n, ncg, cus) == (ncg >= b.line * cus), "ring walk: n=%d, %lld column groups", n, (long long)ncg);
                    if (!ring_rows(n, ncg, cus)) continue;
                    const SweepPlan p = sweep_plan(ncg, cus, kRingLanes);
                    const int depth = ring_depth(p, n), produce = ring_depth_produce(p);
                    CHECK(p.chunk <= kRingLanes && depth <= n - 2 && (produce == 1 || produce == 2) && produce <= n - 2,
                          "ring walk: n=%d, depths %d and %d", n, depth, produce);
                    CHECK(pace_lead(produce, true) >= 4 * produce, "with the next gradients: a lead that the loads on their way need");
                    CHECK(p.count * n < (int64_t)1 << 29, "ring walk: %lld items, counted in quarters in 32 bits", (long long)(p.count * n));
                    // any other table in the same launch: looping tiles of two to four rows per lane on the same workgroups, one partial
                    // sum and at least one tile each
                    for (bool cd : {false, true}) {
                        const ShortPlan t = ring_tiles(n, ncg, cd, false, ncg & 1);
                        CHECK(!t.one && t.rows >= 2 && t.rows <= 4 && t.nrg * t.rows >= n && t.threads == t.nrg << t.logc &&
                                  t.threads % 64 == 0 && t.threads <= kRingThreadsMost && t.lds <= kShortLds,
                              "n=%d: tiles of %d rows per lane, %d lanes, %zu bytes of LDS", n, t.rows, t.threads, t.lds);
                        CHECK(t.tiles >= cus && t.tiles << t.logc >= ncg, "n=%d, %lld column groups: %lld tiles", n, (long long)ncg, (long long)t.tiles);
                    }
                }
    for (int n = 3; n < 9; ++n) {
        const ShortPlan with = ring_tiles(n, 3000000, true, false, false), without = ring_tiles(n, 30000000, false, false, true);
        CHECK(ring_tiles(6, 3000000, true, false, true).rows == 3, "six learners off the lines");
        CHECK(with.rows == (n == 3 ? 3 : n == 4 || n == 8 ? 4 : 2) && without.rows == (n < 4 || n == 5 || n == 6 ? 3 : 4), "n=%d: tiles of %d and %d rows", n, with.rows, without.rows);
    }
    // with the next gradients beside the tiles three rows at most (no kernel has more), on segments no narrower than without them but for
    // half of them; in front of the tiles the same tiles as without
    for (int cus : {64, 256, 304})
        for (int n = 3; n <= 512; ++n)
            for (int64_t ncg : {192 * (int64_t)cus, 3600 * (int64_t)cus + 1, 30000 * (int64_t)cus + 5})
                for (bool cd : {false, true}) {
                    const ShortPlan t = ring_tiles(n, ncg, cd, true, ncg & 1), u = ring_tiles(n, ncg, cd, false, ncg & 1);
                    CHECK(!t.one && t.rows >= 1 && t.rows <= (tiles_produce(n) ? 3 : 4) && t.nrg * t.rows >= n && t.threads % 64 == 0 && t.threads <= kRingThreadsMost &&
                              t.lds <= kShortLds && t.tiles << t.logc >= ncg, "n=%d: tiles of %d rows beside the next gradients", n, t.rows);
                    CHECK(u.rows <= 4 && u.nrg * u.rows >= n && u.threads <= kRingThreadsMost && u.lds <= kShortLds && u.tiles << u.logc >= ncg, "n=%d: tiles of %d rows", n, u.rows);
                    CHECK(n < 9 || (tiles_produce(n) ? t.logc >= 3 && t.logc + 1 >= u.logc : t.logc == u.logc), "n=%d: segments of 2^%d groups with the next gradients, 2^%d without",
                          n, t.logc, u.logc);
                }
    for (int cus : {64, 256, 304})
        for (const auto& b : full_bands)
            for (int n = b.lo; n <= b.hi; ++n)
                for (int64_t ncg : {b.line * cus - 1, b.line * cus, b.line * cus + 1, b.line * cus * 40 + 1})
                    CHECK(full_rows_paced(n, ncg, cus) == (ncg >= b.line * cus), "global averaging in step: n=%d, %lld column groups", n, (long long)ncg);
    // where the launches walk: three to eight learners too, by the column groups of all of them (per compute unit; 0: never)
    const struct { int n; int64_t without, with, pair_without, pair_with, full; } few[] = {
        {1, 0, 0, 0, 0, 0}, {2, 0, 0, 0, 0, 0}, {3, 0, 24000, 0, 0, 12000}, {4, 0, 24000, 0, 24000, 12000}, {5, 0, 24000, 24000, 24000, 12000},
        {6, 100000, 24000, 24000, 24000, 12000}, {8, 100000, 24000, 24000, 24000, 12000}};
    for (const auto& f : few)
        for (int cus : {64, 256})
            for (int form = 0; form < 5; ++form) {
                const int64_t lines[] = {f.without, f.with, f.pair_without, f.pair_with, f.full}, at = lines[form] ? (lines[form] * cus + f.n - 1) / f.n : (int64_t)1 << 34;
                auto walks = [&](int64_t ncg) { return form == 4 ? walk_full_rows(f.n, ncg, cus) : walk_rows(f.n, ncg, cus, form & 1, form & 2); };
                CHECK(!walks(at - 1) && walks(at) == (lines[form] != 0), "n=%d: walked in form %d around %lld column groups", f.n, form, (long long)at);
            }
    // whatever is walked: lanes for every chunk, no load further ahead than the rows allow, and workgroups that keep pace
    for (int cus : {1, 64, 256, 304})
        for (int n = 1; n <= 512; ++n)
            for (int64_t per_cu : {1, 192, 220, 307, 440, 576, 800, 961, 1500, 2400, 3600, 4001, 8001, 33334, 100001})
                for (int form = 0; form < 5; ++form) {
                    const int64_t ncg = per_cu * cus - 1;
                    const bool full = form == 4, produce = !full && form & 2;
                    if (full ? !walk_full_rows(n, ncg, cus) : !walk_rows(n, ncg, cus, form & 1, produce)) continue;
                    const SweepPlan p = sweep_plan(ncg, cus, kRingLanes);
                    const int depth = full ? full_depth(p, n) : produce ? ring_depth_produce(p) : ring_depth(p, n);
                    CHECK(full ? (depth == 2 || depth == 4) && depth < n : depth <= n - 2 && (depth == 1 || depth == 2 || (!produce && (depth == 4 || depth == 6))),
                          "n=%d, %lld column groups, form %d: depth %d", n, (long long)ncg, form, depth);
                    CHECK((full ? full_lead(depth) : pace_lead(depth, produce)) >= 4 * depth, "n=%d, depth %d: a lead that the loads on their way need", n, depth);
                    CHECK(p.chunk <= kRingLanes && ring_threads({1, p.chunk}, kRingLanes) + 64 <= kRingThreadsMost, "n=%d, %lld column groups: chunks of %lld", n,
                          (long long)ncg, (long long)p.chunk);
                    CHECK(2 * p.count * n < (int64_t)1 << 29, "n=%d: %lld items, counted in quarters in 32 bits", n, (long long)(2 * p.count * n));
                }
    // distances by small workgroups: two or three learners on long rows only
    CHECK(distance_alone(2, 2560000, 256) && distance_alone(3, 2560000, 256) && !distance_alone(3, 2559999, 256) && !distance_alone(4, (int64_t)1 << 32, 256),
          "the distance of two and three learners");
    // short rows: whole wavefronts, the rows covered, the LDS within a compute unit's, the grid within the buffer
    for (int n : {1, 2, 3, 5, 8, 9, 16, 17, 33, 64, 65, 100, 128, 200, 256, 257, 300, 511, 512})
        for (int deg : {1, 3, 8, 13, 32})
            for (int64_t ncg : {1, 2, 63, 64, 65, 1000, 16384, 65536, 65537, 250000, 393215})
                for (int cus : {1, 64, 256, 304})
                    for (int form = 0; form < 4; ++form) {
                        if ((long)n * deg > 4096) continue;
                        const bool cd = form & 1, quads = form & 2;
                        const int64_t slots = kShortSlots;
                        const ShortPlan p = short_plan(n, deg, ncg, cus, cd, quads);
                        CHECK(p.threads % 64 == 0 && p.threads >= 64 && p.threads <= kShortThreads && p.threads == p.nrg << p.logc,
                              "short rows n=%d deg=%d ncg=%lld: %d lanes", n, deg, (long long)ncg, p.threads);
                        CHECK(p.rows * p.nrg >= n && p.rows >= 1 && p.rows <= (p.one ? kShortRowsOne : kShortRows) &&
                                  (!p.one || p.rows % 2 == 0), "short rows n=%d: %d rows on %d row groups", n, p.rows, p.nrg);
                        CHECK(p.tiles << p.logc >= ncg && (p.tiles - 1) << p.logc < ncg, "short rows: %lld tiles", (long long)p.tiles);
                        const size_t merge = cd && p.nrg > 1 ? (size_t)p.threads * 48 : 0;
                        CHECK(p.tab_bytes >= n * deg * 8 && p.tab_bytes % 16 == 0 && p.tile_bytes >= n * (16 << p.logc) &&
                                  p.lds <= kShortLds && p.lds >= (size_t)p.tab_bytes + p.tile_bytes + (p.one ? 0 : merge) &&
                                  (!p.one || (size_t)p.tile_bytes >= merge), "short rows n=%d deg=%d: LDS %zu", n, deg, p.lds);
                        const int64_t grid = p.one ? p.tiles : short_grid(p, cus, cd ? slots : INT32_MAX);
                        CHECK(grid >= 1 && grid <= p.tiles && (!cd || grid <= slots), "short rows: grid %lld", (long long)grid);
                    }
    // the next gradients beside the step or by a producer behind it, and what the cache hints go by then
    const struct { int n; int64_t d; bool cd, lines, beside; } next[] = {
        {498, 43411, false, false, false}, {257, 61035, false, false, false}, {306, 145227, true, false, false}, {142, 130547, true, false, false},
        {381, 33063, false, false, true}, {173, 67547, false, false, true}, {393, 24927, false, false, true}, {393, 80736, true, true, true},
        {439, 86240, true, true, true}, {107, 205493, true, false, true}, {45, 278507, false, false, true}, {512, 15000, true, true, false}, {300, 10000, true, true, true}};
    for (const auto& e : next)
        CHECK(short_produces(short_plan(e.n, 3, (e.d + 3) / 4, 256, e.cd, e.d % 4 == 0), e.n * e.d, e.lines) == e.beside, "n=%d d=%lld: next gradients", e.n, (long long)e.d);
    for (int n : {1, 2, 3, 7, 16, 100, 300, 385, 512})
        for (int64_t d : {4, 5, 1000, 20003, 100001, 300000, 3000001})
            for (int form = 0; form < 4; ++form) {
                const bool cd = form & 1, lines = form & 2;
                const ShortPlan p = short_plan(n, 3, (d + 3) / 4, 256, cd, d % 4 == 0);
                if (short_produces(p, n * d, lines))
                    CHECK(p.rows >= 2 && p.rows <= (p.one ? 8 : 4), "n=%d d=%lld: no kernel of %d rows with the next gradients", n, (long long)d, p.rows);
            }
    {
        const ShortPlan p = short_plan(393, 3, 6232, 256, false, false);
        CHECK(cached_accesses(p, counted_bytes(393 * 24927, 4, true, false), false, false) == (kCachedLoads | kCachedStores) &&
                  cached_accesses(p, counted_bytes(393 * 24927, 4, false, false), false, false) == kCachedLoads, "cache hints with the next gradients off the lines");
    }
    // few columns: two rows per lane, so that a table's slot chain is short and the workgroups are many; wide tables the same
    // on longer rows; row segments stay a 128-byte line wide where the workgroup has room for it
    for (int n : {3, 8, 16, 40, 64, 105, 200})
        for (int deg : {5, 13, 20}) {
            const ShortPlan p = short_plan(n, deg, 250, 256, false, true);
            CHECK(p.one && p.rows == 2 && (p.logc >= 3 || n > 128), "n=%d deg=%d on few columns: %d rows per lane, 2^%d groups wide", n,
                  deg, p.rows, p.logc);
        }
    CHECK(short_plan(8, 3, 15000, 256, true, true).rows == 2 && short_plan(8, 3, 40000, 256, true, true).rows == 8, "8 learners: two rows up to 24 576 column groups");
    CHECK(short_plan(8, 13, 175000, 256, false, true).rows == 2 && short_plan(8, 13, 175000, 256, false, false).rows == 8, "wide tables on 16 bytes");
    CHECK(short_plan(4, 13, 700000, 256, false, true).rows == 4 && short_plan(64, 20, 300000, 256, false, true).rows == 4, "wide tables, other counts");
    // five to eight learners of long rows with the distance loop on two rows; 26 learners keep the wide tile with it
    for (int n : {5, 6, 7, 8})
        CHECK(short_plan(n, 3, 7500000, 256, true, true).rows == 2 && !short_plan(n, 3, 7500000, 256, true, true).one, "n=%d loops on two rows", n);
    CHECK(short_plan(26, 5, 500000, 256, true, true).logc == 7 && short_plan(26, 5, 500000, 256, false, true).logc == 6, "26 learners");

    // a launch holds fewer than 2^32 lanes, also on the longest rows that fit a device (one learner of 18e9 columns and more)
    for (int n : {1, 2, 3, 8, 9, 64})
        for (int64_t ncg : {(int64_t)1 << 22, (int64_t)1 << 30, ((int64_t)1 << 32) + 3, (int64_t)4500000001, (int64_t)1 << 34})
            for (bool cd : {false, true}) {
                const ShortPlan p = short_plan(n, 3, ncg, 256, cd, true);
                const int64_t grid = p.one ? p.tiles : short_grid(p, 256, cd ? kShortSlots : INT32_MAX);
                CHECK(grid >= 1 && grid * p.threads < (int64_t)1 << 32, "short rows n=%d ncg=%lld: %lld workgroups of %d lanes", n,
                      (long long)ncg, (long long)grid, p.threads);
            }
    // global averaging and the distance with rows spread over lanes
    for (int n : {1, 2, 9, 10, 14, 16, 17, 30, 33, 48, 64, 65, 82, 127, 128, 300, 512})
        for (int64_t d : {1, 4, 5, 8, 252, 257, 260, 3999, 4000, 6000, 60000, 131068, 131069, 131072, 1000000})
            for (int cus : {1, 256})
                for (int form = 0; form < 3; ++form) {
                    const int64_t ncg = (d + 3) / 4;
                    const RowsPlan p = form == 2 ? distance_rows_plan(n, d, cus) : full_rows_plan(n, d, cus, form);
                    if (p.threads == 0) {
                        CHECK(ncg > 1, "one column group has no lane-per-column form");
                        continue;
                    }
                    CHECK(p.threads % 64 == 0 && p.threads >= 64 && p.threads <= 1024 && p.threads == p.nrg << p.logc && p.nrg >= 1,
                          "rows n=%d ncg=%lld: %d lanes", n, (long long)ncg, p.threads);
                    CHECK(p.tiles << p.logc >= ncg && (p.tiles - 1) << p.logc < ncg, "rows: %lld tiles", (long long)p.tiles);
                    CHECK(p.threads * 48 + (16 << p.logc) <= 65280, "rows: LDS");
                }
    CHECK(full_rows_plan(9, 200000, 256, false).threads == 0 && full_rows_plan(16, 20000, 256, true).threads == 0 &&
              full_rows_plan(16, 20000, 256, false).threads != 0 && full_rows_plan(16, 20001, 256, true).threads != 0 &&
              full_rows_plan(12, 20000, 256, true).threads != 0 && full_rows_plan(12, 3000, 256, false).threads == 0 &&
              full_rows_plan(17, 3000, 256, true).threads != 0, "global averaging: where rows are spread over lanes");
    CHECK(full_rows_plan(82, 89641, 256, true).threads != 0 && full_rows_plan(82, 131072, 256, true).threads == 0 &&
              distance_rows_plan(82, 89641, 256).threads != 0 && distance_rows_plan(42, 50001, 256).threads != 0 &&
              distance_rows_plan(42, 50000, 256).threads == 0, "65 learners and more; ragged rows");
    if (failures) return 1;
    std::printf("launch plan ok\n");
    return 0;
}
