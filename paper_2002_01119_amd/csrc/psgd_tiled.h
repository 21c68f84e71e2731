// The LDS-tiled form of the model-averaging step (Sec. 2, Eq. 2) on long rows, for mixing tables of other than three slots and numbers of learners
// that fill its tiles (plan::tiled_rows), and its kernel mix_deg_kernel.  Included by psgd_kernels.hip only.
#ifndef PSGD_TILED_H
#define PSGD_TILED_H

#include "psgd_device.h"

namespace psgd {
namespace {

// ---------------------------------------------------------------------------------------
// Tiled path (any number of slots per row).
//
// The workgroup's T lanes form T / lpr row groups of lpr lanes; a tile is n rows by lpr column groups and lives
// in LDS, so a neighbour read is an LDS read and every X element crosses the HBM interface once.  Lane (rg,
// lane) produces rows rg, rg + nrg, ... of column group `lane` of the tile.  Two tile buffers alternate: while
// the rows of tile t are computed from one, the X rows of the workgroup's next tile are written into the
// other.  A barrier per tile separates "everyone has finished reading this buffer and writing the other" from
// the next tile.  A tile is complete in LDS before its first output is stored, and different tiles own
// different columns, so X_out may alias X.
//
// The tile's rows are one batch, every memory operation is unconditional, and a lane reloads each of its registers
// the moment its value has been used (tile_path).
//
// Per output the slots are taken in table order, acc = w0 * x0, one fma per further slot, then the gradient
// term (for 3 slots exactly mix_one's order).  The slot loop is the latency-critical part (a table read, then
// a tile read that depends on it, per slot): SB rows advance together and two slots per trip, so SB * 2
// independent chains hide each other's LDS round trips.
//
// With CD the distance of the outputs is gathered in the same pass.  The rows of one column group are spread
// over the row groups; every row group measures against its own first output and the merge brings the sums to row
// group 0's pivot exactly (tile_finish).
// ---------------------------------------------------------------------------------------
// The value of the lane whose number differs in bit 0 (CTRL 0xB1: quad order 1,0,3,2) or bit 1 (0x4E: 2,3,0,1),
// moved inside the vector unit (no LDS round trip).  All four lanes of a quad must be active.
template <int CTRL>
__device__ __forceinline__ double lane_xor_quad(double v) {
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(bits & 0xFFFFFFFFll), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(bits >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The workgroups are alone on their compute unit: 512 lanes with up to 256 registers per lane (8
// wavefronts x 8 rows cover n = 64 at once), or 1024 lanes with up to 128 (16 x 4).
template <int T> struct TileShape {
    static constexpr int RB = T > 512 ? 4 : 8;   // rows per lane and batch
    static constexpr int SB = T == 512 ? 3 : 2;   // rows whose slot chains advance together (two slots per trip each);
                                                 // more rows at once cost registers and ran slower (4: -1 to -6 %)
};

// Per-lane state of the tiled path that does not change from tile to tile.
struct TileCtx {
    const TileSlot* tab;
    int n, deg, lpr, lane, rg, nrg;
    int rows_each, rows_more;   // n = rows_each * nrg + rows_more: row group q has rows_each (+ 1 if q < rows_more) rows
    int tlane;   // the lane's column inside the tile (lane, or the last valid one for a lane beyond the ragged end)
    float neg_lr;
};

// Running sums of the distance for one lane and one tile.
struct TileStats {
    double a[kVec], sq;
    float pivot[kVec];   // the pivot as the fp32 output it is
    __device__ __forceinline__ void reset() {
        sq = 0.0;
#pragma unroll
        for (int k = 0; k < kVec; ++k) {
            a[k] = 0.0;
            pivot[k] = 0.0f;
        }
    }
};

// Rows rg + u nrg, u < RB, of the tile in `cur`: mix, subtract the gradient, store, gather.
//
// Nothing here is conditional except the arithmetic of the distance.  A lane without a row (or without a
// column group: the caller then points it at the last valid one) repeats the work of the lane that owns the
// clamped row and column and stores the same bits to the same place.  This is what lets loads that were issued
// early stay in flight: the compiler counts outstanding memory operations to wait for exactly the ones it
// needs, and a load or store that may or may not have been issued makes that count unknown, upon which it
// waits for all of them.
//
// `feed(j0)` runs in front of every group of SB rows and `refill(j0)` behind it (its gradients have been used,
// its outputs stored): the caller's places for the loads of the next tiles, so that they enter the memory
// pipeline a few at a time between the rows' arithmetic instead of in one burst.
template <bool CD, int RB, int SB, typename GR, typename FEED, typename REFILL>
__device__ __forceinline__ void tile_rows(const TileCtx& c, const f32x4* cur, const GR (&g)[RB], bool active, float* out_col,
                                          int64_t ldo, TileStats& st, const FEED& feed, const REFILL& refill) {
    typedef f32x4 V;
#pragma unroll
    for (int j0 = 0; j0 < RB; j0 += SB) {
        feed(j0);
        const TileSlot* tp[SB];
        bool ok[SB];
        int row[SB];
        V acc[SB];
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            row[i] = c.rg + (j0 + i) * c.nrg;
            ok[i] = active && row[i] < c.n;
            if (row[i] > c.n - 1) row[i] = c.n - 1;
            tp[i] = c.tab + row[i] * c.deg;
        }
        {
            TileSlot e[SB];
#pragma unroll
            for (int i = 0; i < SB; ++i) e[i] = tp[i][0];
#pragma unroll
            for (int i = 0; i < SB; ++i) acc[i] = cur[e[i].off + c.tlane] * e[i].w;
        }
        // two slots per trip; where four wavefronts share a SIMD they hide each other's round trips and the
        // registers are worth more than a longer unrolled trip
        auto trip = [&](int s) {
            TileSlot e0[SB], e1[SB];
            V x0[SB], x1[SB];
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                e0[i] = tp[i][s];
                e1[i] = tp[i][s + 1];
            }
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                x0[i] = cur[e0[i].off + c.tlane];
                x1[i] = cur[e1[i].off + c.tlane];
            }
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                acc[i] = vfma(e0[i].w, x0[i], acc[i]);
                acc[i] = vfma(e1[i].w, x1[i], acc[i]);
            }
        };
        int s = 1;
        if (RB == 4 || (CD && sizeof(GR) > 8)) {
#pragma unroll 1
            for (; s + 1 < c.deg; s += 2) trip(s);
        } else {
            for (; s + 1 < c.deg; s += 2) trip(s);
        }
        if (s < c.deg) {
            TileSlot e[SB];
#pragma unroll
            for (int i = 0; i < SB; ++i) e[i] = tp[i][s];
#pragma unroll
            for (int i = 0; i < SB; ++i) acc[i] = vfma(e[i].w, cur[e[i].off + c.tlane], acc[i]);
        }
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            const int j = j0 + i;
            if (j < RB) {
                const V out = vfma(c.neg_lr, widen_g(g[j]), acc[i]);
                st_x(out_col + (int64_t)row[i] * ldo, out);
                if (CD && j == 0) floats_of(out, st.pivot);
                if (CD && ok[i]) {
                    double o[kVec];
                    pivot_of(out, o);      // widen
#pragma unroll
                    for (int k = 0; k < kVec; ++k) {
                        const double df = o[k] - (double)st.pivot[k];
                        st.a[k] += df;
                        st.sq = fma(df, df, st.sq);
                    }
                }
            }
        }
        refill(j0);
    }
}

// Merge of the column sums at the end of a tile (CD only), brought from each row group's own pivot p_q (its first
// output) to a common one: with P = p_0, D_q = p_q - P and m_q rows in group q,
//     sum_i (o_i - P)   = sum_q (a_q + m_q D_q)
//     sum_i (o_i - P)^2 = sum_q (sq_q + 2 D_q a_q + m_q D_q^2)
// exactly; in fp64 the corrections are of the size of the sums themselves (every pivot is one of the outputs).
// If all outputs of a column are equal every D_q is 0 and the distance comes out exactly 0.  One slot per row
// group and column: a double for the sum and a float for the pivot.  Contains the tile's barriers: when it returns every
// read of the current buffer and every write of the other one is done.
template <int T>
__device__ __forceinline__ void tile_finish(const TileCtx& c, double* comb, float* combp, int live_cols,
                                            TileStats& st, double inv_n, double& total) {
    // live_cols: the lanes of the tile that own a column group (all of them except in the ragged last tile)
    // slot of row group q, column k of lane l: (q kVec + k) lpr + l, so that the lanes of a wavefront write
    // neighbouring words (no bank conflicts); the merge below numbers the tile's columns in the same order
    const int cols = c.lpr * kVec;
    const size_t mine = (size_t)c.rg * cols + c.lane;
#pragma unroll
    for (int k = 0; k < kVec; ++k) {
        comb[mine + k * c.lpr] = st.a[k];
        combp[mine + k * c.lpr] = st.pivot[k];
    }
    total += st.sq;
    lds_barrier();
    // The tile has lpr * kVec columns and nrg partial sums per column.  Where there are more lanes than columns
    // (1 KB row segments: four times as many) `parts` adjacent lanes share a column, each takes nrg / parts of its
    // row groups and a symmetric exchange adds the shares up, the same bits in every lane of the column.  (Left
    // to one lane per column the loop over the row groups is a chain of LDS round trips on a quarter of the
    // wavefronts while the others wait at the barrier below.)
    // Nothing here branches on data: every lane reads kVec slots (clamped to slot 0 where it has fewer), all
    // reads are issued before the first is used, and a slot that does not count enters with weight 0.
    const int parts = c.nrg >= kVec ? c.nrg / kVec : 1;        // a power of two; the lanes of a column sit side by side in one wavefront
    const int each = c.nrg / parts;                          // row groups per lane: min(nrg, kVec)
    for (int idx = threadIdx.x; idx < cols * parts; idx += T) {
        const int col = idx / parts, part = idx % parts;
        const bool live = (col & (c.lpr - 1)) < live_cols;   // a column of a lane beyond the ragged end counts for nothing
        double aq[kVec], md[kVec];
        float pq[kVec];
        const float p0f = combp[col];                        // row group 0 owns row 0: its pivot is the common one
#pragma unroll
        for (int k = 0; k < kVec; ++k) {
            const bool on = k < each;                        // uniform
            const int q = on ? part * each + k : 0;
            const size_t at_q = (size_t)q * cols + col;
            aq[k] = comb[at_q];
            pq[k] = combp[at_q];
            md[k] = on ? (double)(c.rows_each + (q < c.rows_more ? 1 : 0)) : -1.0;   // rows q, q + nrg, ... below n
        }
        const double p0 = (double)p0f;
        double at = 0.0, corr = 0.0;
#pragma unroll
        for (int k = 0; k < kVec; ++k) {
            const double dq = (double)pq[k] - p0;
            const double tq = fma(md[k], dq, aq[k]);         // a row group without rows has a = 0 and weight 0: no share
            const double cq = dq * (tq + aq[k]);
            at += md[k] >= 0.0 ? tq : 0.0;
            corr += md[k] >= 0.0 ? cq : 0.0;
        }
        if (parts > 1) {
            at += lane_xor_quad<0xB1>(at);                   // lanes 1 apart
            corr += lane_xor_quad<0xB1>(corr);
        }
        if (parts > 2) {
            at += lane_xor_quad<0x4E>(at);                   // lanes 2 apart
            corr += lane_xor_quad<0x4E>(corr);
        }
        for (int off = 4; off < parts; off <<= 1) {
            at += __shfl_xor(at, off, 64);
            corr += __shfl_xor(corr, off, 64);
        }
        if (part == 0 && live) total += corr - at * at * inv_n;
    }
    lds_barrier();                                     // the merge slots are free again
}

// The tiled path of the large workgroup (1024 lanes without the distance, 512 with it; alone on its compute
// unit) for tables whose tile is ONE batch of rows: at most TileShape<T>::RB rows per lane (n = 64 with 1 KB row
// segments, fewer learners with wider ones, up to 256 learners with narrower ones).  The launcher picks the
// shape (plan::tile_plan).
// With `comb_in_tile` the merge slots of the distance are the tile buffer that has just been consumed.
//
// UQ: a row group is whole wavefronts (lpr >= 64), so its number is the same in every lane of a wavefront and is
// kept in a scalar register: row offsets and table addresses then cost no vector registers.  Narrower rows
// (n > 64 at 16 B per lane: two or four row groups share a wavefront) keep it per lane.
template <typename GT, bool CD, int T, bool UQ>
__device__ double tile_path(const float* X, float* Xout, const GT* __restrict__ G, const TileSlot* tab, char* tiles, int n,
                            int deg, Pitch ld, int64_t ncg, float neg_lr, int lpr, double inv_n, bool comb_in_tile) {
    typedef f32x4 V;
    typedef typename RawG<GT>::T GR;
    constexpr int RB = TileShape<T>::RB, SB = TileShape<T>::SB;
    TileCtx c;
    c.tab = tab;
    c.n = n;
    c.deg = deg;
    c.lpr = lpr;
    c.lane = c.tlane = threadIdx.x % lpr;
    c.nrg = T / lpr;
    c.rows_each = n / c.nrg;
    c.rows_more = n % c.nrg;
    c.neg_lr = neg_lr;
    const int lane = c.lane, nrg = c.nrg;
    const size_t tile_bytes = (((size_t)n * lpr * sizeof(V)) + 15) & ~(size_t)15;
    V* cur = reinterpret_cast<V*>(tiles);
    V* nxt = reinterpret_cast<V*>(tiles + tile_bytes);
    double* comb = reinterpret_cast<double*>(tiles + 2 * tile_bytes);   // [nrg][lpr][kVec] sums, then as many float pivots
    const int64_t ntiles = (ncg + lpr - 1) / lpr;
    const int64_t step = gridDim.x;
    int64_t t = plan::die_contiguous_slot(blockIdx.x, gridDim.x, kXcds);   // the first of tiles t, t + step, ...
    if (t >= ntiles) return 0.0;                             // uniform: the whole workgroup has nothing to do
    double total = 0.0;
    TileStats st;
    // A tile is one batch of whole-wavefront rows (n <= 64 with 1 KB row segments, fewer learners with wider
    // ones).  A lane keeps ONE register per row for X and one for the gradients, each reloaded the moment
    // its value has been used, so every load has a whole tile's time to arrive:
    //   in front of a group of rows: X of tile t + step (loaded one tile ago) goes into the other LDS buffer,
    //       which nobody reads during this tile, and the same registers are loaded with tile t + 2 step;
    //   behind it: its gradients (tile t) have been used, the registers are loaded with tile t + step.
    // The loads thus enter the memory pipeline a few at a time between the arithmetic.  (Issued in one burst
    // at the start of the tile they hold the wavefront at the issue stage until the pipeline has taken them,
    // and the arithmetic starts only then: the two times add up instead of overlapping.)  Every load and
    // store here is unconditional (see tile_rows): rows, columns and tiles beyond the end are clamped to the
    // last valid one.
    const int q = UQ ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x / lpr)) : (int)(threadIdx.x / lpr);
    c.rg = q;
    const int last_row = n - 1;
    auto cge_of = [&](int64_t tile) {                       // the lane's column group in `tile`, clamped
        const int64_t cg = tile * lpr + lane;
        return cg < ncg ? cg : ncg - 1;
    };
    auto row_of = [&](int u) {
        const int r = q + u * nrg;
        return r < last_row ? r : last_row;
    };
    V x[RB];
    GR g[RB];
    if (t * lpr + lane < ncg) {                              // the first tile: straight into `cur`
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            const int r = q + u * nrg;
            if (r < n) cur[r * lpr + lane] = ld_x(X + (int64_t)r * ld.x + (t * lpr + lane) * kVec);
        }
    }
    {
        const int64_t colx = cge_of(t + step) * kVec, colg = cge_of(t) * kVec;
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            x[u] = ld_x(X + (int64_t)row_of(u) * ld.x + colx);
            g[u] = ld_g_raw(G + (int64_t)row_of(u) * ld.g + colg);
        }
    }
    lds_barrier();
    // One tile.  It runs once in front of the loop and then inside it: the waits for the loads of the tile before
    // are counted per place in the program, and a place that both the start and the loop reach waits for the
    // smaller count, the start's, where fewer operations have been issued since.
    auto one_tile = [&]() __attribute__((always_inline)) {
        const int64_t colx = cge_of(t + 2 * step) * kVec, colg = cge_of(t + step) * kVec;
        // where tile t + step goes in the other buffer: the lane's own slot, the last valid lane's at the ragged
        // end (the same value twice), and beyond the last tile anywhere (nobody will read it) - never a branch
        const int lane_to = (int)(cge_of(t + step) - (t + step) * lpr);
        const int lane_n = lane_to >= 0 ? lane_to : lane;
        auto feed = [&](int j0) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                const int u = j0 + i;
                if (u < RB) {
                    const int r = row_of(u);
                    nxt[r * lpr + lane_n] = x[u];
                    x[u] = ld_x(X + (int64_t)r * ld.x + colx);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto refill = [&](int j0) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                const int u = j0 + i;
                if (u < RB) g[u] = ld_g_raw(G + (int64_t)row_of(u) * ld.g + colg);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        const int64_t cge = cge_of(t);
        const bool active = t * lpr + lane < ncg;
        c.tlane = (int)(cge - t * lpr);
        if (CD) st.reset();
        tile_rows<CD, RB, SB>(c, cur, g, active, Xout + cge * kVec, ld.o, st, feed, refill);
        if (CD) {
            const int64_t left = ncg - t * lpr;                       // column groups of this tile (uniform)
            double* sums = comb;
            if (comb_in_tile) {                                       // uniform
                lds_barrier();                                        // every row of `cur` has been read
                sums = reinterpret_cast<double*>(cur);
            }
            tile_finish<T>(c, sums, reinterpret_cast<float*>(sums + (size_t)nrg * lpr * kVec),
                           (int)(left < lpr ? left : lpr), st, inv_n, total);
        } else {
            lds_barrier();
        }
        V* sw = cur;
        cur = nxt;
        nxt = sw;
        t += step;
    };
    one_tile();
    while (t < ntiles) one_tile();
    return total;
}


// The d mod 4 columns behind the last whole column group, one element per lane, by one workgroup: they pass through
// LDS (`lds`: two floats per element, free when this is called) as a tile does.  Returns their part of the distance.
template <typename GT, bool CD, int T>
__device__ double tile_remainder(const float* X, float* Xout, const GT* __restrict__ G, const int32_t* __restrict__ nbr,
                                 const float* __restrict__ w, float* lds, int n, int deg, Pitch ld, int64_t d, float neg_lr,
                                 double inv_n) {
    const int rem = (int)(d & 3), count = n * rem;
    const int64_t col = d - rem;
    float* out = lds + count;
    __syncthreads();                                             // the LDS is free
    for (int e = threadIdx.x; e < count; e += T) lds[e] = X[(int64_t)(e / rem) * ld.x + col + e % rem];
    __syncthreads();
    for (int e = threadIdx.x; e < count; e += T) {
        const int r = e / rem, c = e % rem;
        float acc = lds[nbr[r * deg] * rem + c] * w[r * deg];
        for (int s = 1; s < deg; ++s) acc = vfma(w[r * deg + s], lds[nbr[r * deg + s] * rem + c], acc);
        acc = vfma(neg_lr, widen_1(G[(int64_t)r * ld.g + col + c]), acc);
        Xout[(int64_t)r * ld.o + col + c] = acc;
        out[e] = acc;
    }
    if (!CD) return 0.0;
    __syncthreads();
    double a = 0.0, sq = 0.0;
    if ((int)threadIdx.x < rem) {
        for (int r = 1; r < n; ++r) {
            const double df = (double)out[r * rem + threadIdx.x] - (double)out[threadIdx.x];
            a += df;
            sq = fma(df, df, sq);
        }
    }
    return sq - a * a * inv_n;
}

// Any table with `deg` slots per row (sparse doubly stochastic matrices beyond the ring: more neighbours, lazy
// walks, products of several mixing rounds).
// LDS: TileSlot tab[deg n] | two tile buffers | merge slots (plan::tile_plan).
//
// UQ: a row group is whole wavefronts (lpr >= 64).
template <typename GT, bool CD, int T, bool UQ>
__global__ __launch_bounds__(T) void mix_deg_kernel(const float* X, float* Xout, const GT* __restrict__ G,
                                                    const int32_t* __restrict__ nbr, const float* __restrict__ w,
                                                    int deg, int n, int64_t d, Pitch ld, float neg_lr, int lpr,
                                                    int comb_in_tile, Gather gather) {
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    __shared__ double lds_waves[T / 64];
    const size_t tab_bytes = (((size_t)n * deg * sizeof(TileSlot)) + 15) & ~(size_t)15;
    TileSlot* tab = reinterpret_cast<TileSlot*>(lds_raw);
    int ok = 1;
    for (int e = threadIdx.x; e < deg * n; e += T) {
        const int v = nbr[e];
        tab[e] = TileSlot{(uint32_t)(v * lpr), w[e]};
        ok &= (unsigned)v < (unsigned)n;
    }
    if (!__syncthreads_and(ok)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(&g_status_word, 1);
        if (CD) last_sum(gather, __builtin_nan(""));
        return;
    }
    const double inv_n = 1.0 / (double)n;
    double total = tile_path<GT, CD, T, UQ>(X, Xout, G, tab, lds_raw + tab_bytes, n, deg, ld, d / kVec, neg_lr, lpr, inv_n,
                                            comb_in_tile != 0);
    if (d % kVec != 0 && blockIdx.x == 0)
        total += tile_remainder<GT, CD, T>(X, Xout, G, nbr, w, reinterpret_cast<float*>(lds_raw + tab_bytes), n, deg, ld, d,
                                           neg_lr, inv_n);
    if (CD) {
        last_sum(gather, block_sum(total, lds_waves, T));
    }
}

}  // namespace
}  // namespace psgd

#endif
