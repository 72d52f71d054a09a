// Host-side planner of libcce: how one call is tiled over the GPU and laid out in the caller's
// workspace -- vocabulary splits of the forward, [row block x vocabulary chunk] of the backward,
// contraction tile, form of the dHidden running sum -- ranked with a small time model whose
// constants were measured on MI355X.  No device code; included by cce_kernels.hip only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <string.h>
#include <atomic>

#include "../../include/cce.h"
#include "gemm_core.h"
#include "host_util.h"

#ifndef CCE_PLAN_PRICED
#define CCE_PLAN_PRICED() ((void)0)     // a makespan was searched for: counted by the host tests
#endif

namespace cce {

// Row skipping: a row block's row map lives in an LDS table behind everything else the
// contraction kernel uses, which bounds the block to this many 256-row tiles.
constexpr int kCompactMaxRowTiles = 16;
constexpr int kRowTableBytes = kCompactMaxRowTiles * 256 * 4;

// Compute units of the CURRENT device (looked up once per device ordinal; 256 if the query fails,
// e.g. on a host without a GPU).
static int device_cu_count() {
    static std::atomic<int> cached[64];
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    const int have = cached[dev].load(std::memory_order_relaxed);
    if (have > 0) return have;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
    cached[dev].store(n, std::memory_order_relaxed);
    return n;
}


// Logit tiles of 128 x 128 instead of 256 x 256 (TileBig's loop): where a launch has so few of the large ones that four
// times as many small ones are at most two rounds of the compute units.  One round: 322 x 1856 x 1015
// (8 large tiles) 102.8 -> 58.2 us a step; two: forward / backward of 500 x 2048 x 10000 (80) 47 / 101 ->
// 42 / 93 us, of 3399 x 1088 x 1802 (112) 33 / 76 -> 31 / 72.  Beyond, the large tiles move half the bytes.
static bool use_small_tiles(int64_t row_tiles, int64_t vocab_tiles) {
    return row_tiles * vocab_tiles * 2 <= device_cu_count();
}

struct Plan {
    int TT, VT, S;              // forward: token tiles, vocabulary tiles, vocabulary splits
    int64_t Nb, Vc;             // backward: rows per row block, vocabulary columns per chunk (multiples of 256)
    int gemm_kind;              // backward: output tile of the contractions, 0 = 256 x 256, 1 = 256 x 128
    int split_acc;              // backward: dH running sum as two 16-bit planes (see GemmJob)
    bool small_tiles;           // forward: 128 x 128 tiles, one per workgroup (fwd_vt() splits; FP8 keeps 256 x 256)
    int64_t rows, cols;         // N, V
    int fwd_tt() const { return (int)((rows + 127) / 128); }
    int fwd_vt() const { return (int)((cols + 127) / 128); }
    size_t off_status, off_partials, off_sumz, off_dhacc, off_g, total;
    size_t budget;              // what `total` may grow to (see room_for_planes)
    bool forced;                // a knob was set: the layout and order are exactly those
    // row skipping only (budget_rows != 0): compact-row bookkeeping
    int64_t rows_pad;           // compact rows rounded up to 256
    size_t off_count, off_perm, off_labels_c, off_fa_c, off_fb_c;
    size_t off_zero_row;        // D zeros (bf16): what the dW contraction reads for a k-row that maps to no row
};

// Workspace budget: 1 % of the materialised fp32 logits, but never below a floor that
// keeps the backward chunks large enough to fill the GPU.
static constexpr size_t kBudgetFloor = 48000000;

// Output tiles of the two gradient contractions: 256 x 256, or 256 x 128 with two K groups.
// The planner picks per shape: the narrow tile costs about 10 % more per flop (more operand
// bytes per MFMA) but gives twice as many tiles, which matters when a chunk's outputs are too
// few to fill the GPU (D = 1024: 124 big tiles per 4096 x 4096 chunk against 248 narrow ones)
// or when D is not a multiple of 256 (D = 896 = 7 x 128).  (A 128 x 224 tile, which would give
// D = 896 exactly 256 equal tiles per chunk, was measured 3 % slower: its 32 x 224 wavefront
// tiles need 1.14 LDS fragment reads per MFMA instead of 0.75.)
struct GemmTile { int kind, bm, bn; double us_per_slice; };
static GemmTile gemm_tile_of_kind(int kind) {
    if (kind == 0) return {0, TileBig::BM, TileBig::BN, 2.0};
    if (kind == 1) return {1, TileNarrow::BM, TileNarrow::BN, 1.1};
    if (kind == 2) return {2, TileSmall::BM, TileSmall::BN, 0.6};              // chosen per launch, see contraction_kind
    return {3, TileDuo::BM, TileDuo::BN, 1.1};                  // likewise
}

// Process-wide tuning / testing knobs (0 = automatic).  Atomics: a knob may be set from any host
// thread; every plan reads each knob once (Knobs::read) and the plan cache is keyed by what it read,
// so a change between two calls can never mix two settings inside one plan.  (A caller that sizes
// its workspace under one setting and computes under another still gets CCE_ERR_INVALID if the
// workspace is too small: the knobs are aids for tests and measurements, not a per-call option.)
static std::atomic<int> g_force_tiling{0};           // cce_set_backward_tiling: (row_tiles << 16) | vocab_tiles
static std::atomic<int> g_force_gemm_cols{0};        // cce_set_backward_gemm_tile: 128 or 256
static std::atomic<int> g_force_split_acc{0};        // cce_set_backward_accumulator: 1 = fp32, 2 = split
static std::atomic<int> g_force_row_skipping{0};     // cce_set_row_skipping: 1 = never, 2 = whenever a bound on the valid rows is below N
struct Knobs {
    int row_tiles, vocab_tiles, gemm_cols, split_acc;
    static Knobs read() {
        const int t = g_force_tiling.load(std::memory_order_relaxed);
        return {t >> 16, t & 0xffff, g_force_gemm_cols.load(std::memory_order_relaxed),
                g_force_split_acc.load(std::memory_order_relaxed)};
    }
};

// Completion time of n1 jobs of length c1 followed by n2 jobs of length c2 <= c1, handed in that
// order to `cus` units, each taking the next job when it becomes free.  A plan asks this thousands of
// times, so the searches start where no unit would be idle, which is a lower bound of every answer
// behind the last long job; short jobs that all fit beside it are answered first.
static double two_class_makespan(int64_t cus, int64_t n1, double c1, int64_t n2, double c2) {
    CCE_PLAN_PRICED();
    const int64_t full = n1 / cus, rem = n1 % cus;
    const double tA = (double)full * c1;                     // units without a long job in the last round
    const double tB = (double)(rem ? full + 1 : full) * c1;
    const int64_t nA = cus - rem, nB = rem;
    if (n2 == 0 || nA * (int64_t)((tB - tA) / c2) >= n2) return tB;
    const double t0 = ((double)n2 * c2 + (double)nA * tA + (double)nB * tB) / (double)cus;
    auto first_k = [&](double from) { const int64_t k = (int64_t)((t0 - from) / c2) - 1; return k > 1 ? k : (int64_t)1; };
    // smallest t with nA * floor((t - tA) / c2) + nB * floor((t - tB) / c2) >= n2
    double best = 1e300;
    for (int64_t k = first_k(tA); k <= n2; ++k) {            // t = tA + k c2
        const double t = tA + (double)k * c2;
        const int64_t fromB = t > tB ? (int64_t)((t - tB) / c2) : 0;
        if (nA * k + nB * fromB >= n2) { best = t; break; }
    }
    if (nB > 0) {
        for (int64_t k = first_k(tB); k <= n2; ++k) {        // t = tB + k c2
            const double t = tB + (double)k * c2;
            if (t >= best) break;
            if (nA * (int64_t)((t - tA) / c2) + nB * k >= n2) { best = t; break; }
        }
    }
    return best;
}

// The same of two jobs in either order, longer items first.
static double makespan(int64_t cus, int64_t n1, double c1, int64_t n2, double c2) {
    return c1 >= c2 ? two_class_makespan(cus, n1, c1, n2, c2) : two_class_makespan(cus, n2, c2, n1, c1);
}
// A bound that it never falls below, without the search: all work spread evenly, the rounds of the longer job.
// TIGHT: also the items of the unit with most of them (k = items / units, rounded up): k short ones, and one more or one of them long
// where the units with fewer than k cannot hold all long ones.  It takes as long as a search does, so only tilings that the first bound leaves
// and what would be searched are asked for it (asked for all: plans of twelve shapes 1.2 ms for 0.87, orders 3.6 for 3.1).
enum Floor { kPrice = 0, kFloor = 1, kTightFloor = 2 };      // of a step: its time, or one of the two bounds
template <bool TIGHT = false>
static double makespan_floor(int64_t cus, int64_t n1, double c1, int64_t n2, double c2) {
    double most = ((double)n1 * c1 + (double)n2 * c2) / (double)cus;
    const double rounds = c1 >= c2 ? (double)((n1 + cus - 1) / cus) * c1 : (double)((n2 + cus - 1) / cus) * c2;
    most = rounds > most ? rounds : most;
    if (!TIGHT) return most;
    const int64_t n = n1 + n2, k = (n + cus - 1) / cus, n_long = c1 >= c2 ? n1 : n2;
    const double c_long = c1 >= c2 ? c1 : c2, c_short = n1 == 0 ? c2 : n2 == 0 ? c1 : c1 < c2 ? c1 : c2;
    const double each = (double)k * c_short + (n_long > (k * cus - n) * (k - 1) ? (c_long < 2.0 * c_short ? c_long - c_short : c_short) : 0.0);
    return each > most ? each : most;
}
// Floors and times are sums in different orders: what lies above by less than this is not passed over.
constexpr double kAbove = 1.0 + 1e-9;

// Time of a launch of 256 x 128 tiles two to a compute unit (TileDuo), microseconds: n1 items that take c1 beside
// another one of their unit, n2 that take c2.  An item alone on its unit takes 0.6 of that time (96 slices: 181 us
// beside another, 100 alone), so what counts beside the even share of the work is when the slots run empty and how
// many of them the last items keep.  FLOOR: a bound it never falls below.
template <bool FLOOR = false>
static double duo_makespan(int64_t cus, int64_t n1, double c1, int64_t n2, double c2) {
    if (c2 > c1) { const int64_t n = n1; n1 = n2; n2 = n; const double c = c1; c1 = c2; c2 = c; }
    if (n1 == 0) { n1 = n2; c1 = c2; n2 = 0; }
    const int64_t units = 2 * cus, rounds = (n1 + units - 1) / units;
    const double even = ((double)n1 * c1 + (double)n2 * c2) / (double)units, last = (double)rounds * c1;
    if (n1 + n2 <= cus) return 0.6 * c1 + 1.0;
    const double spread = even + 0.5 * (n2 ? c2 : c1);
    if (FLOOR) return even > 0.6 * last ? even : 0.6 * last;
    if (spread >= last || n2 == 0) {
        const double end = spread > last ? spread : last, start = 2.0 * even - end;      // slots run empty one by one
        return start > 0.0 ? start + 0.75 * (end - start) : 0.75 * end;
    }
    const double f = (double)(n1 - (rounds - 1) * units) / (double)units;                 // the long items' share of the slots
    const double start = f < 1.0 ? (even - last * f) / (1.0 - f) : 0.0;
    const double alone = f <= 0.5 ? 0.6 : 0.2 + 0.8 * f;
    return start > 0.0 ? start + alone * (last - start) : alone * last;
}

// Tile of one contraction launch: 128 x 128 where the planned 256 x 128 tiles would leave half of the
// compute units without work (an item then costs about half as much, and all of them still start at
// once).  A forced tile stays.  Backward of 256 x 64 x 1000: 23 -> 16 us, 322 x 1856 x 1015: 36 -> 28,
// 2269 x 896 x 2131: 58 -> 50, 2500 x 64 x 1300: 33 -> 25.
static bool small_contractions(int kind, int64_t items, const Knobs& knobs) {
    return kind == 1 && knobs.gemm_cols == 0 && items * 2 <= device_cu_count();
}

// Rough time model of the backward pipeline, in microseconds, used only to rank tilings.
// One compute unit runs one workgroup at a time.  Measured on MI355X with random bf16 data:
// a 256 x 256 x 64 slice of the main loop takes about 2 us, a 256 x 128 x 64 one about 1.1 us;
// a gradient-tile workgroup adds about 9 us (pipeline fill, softmax epilogue, store of the
// tile), a contraction workgroup about 4 us.  (bf16 gradient tiles of two wavefront groups take less: see ScheduleModel::logit_tile.)
struct BackwardModel {
    int cus; int64_t D; GemmTile tile;
    double t_tile() const { return (double)(D / 64) * 2.0 + 9.0; }
    double t_gemm(int k_tiles) const { return (double)(k_tiles * 4) * tile.us_per_slice + 4.0; }
    int d_tiles() const { return (int)((D + tile.bn - 1) / tile.bn); }

    // One step = the gradient tiles, then the contractions, of an [a x b] block of 256 x 256
    // tiles: two launches that follow each other on the caller's stream.  FLOOR: with makespan_floor.
    template <int FLOOR = kPrice>
    double step(int a, int b, bool dw_beta) const {
        const int dt = d_tiles(), per256 = 256 / tile.bm;
        const int n_dh = a * per256 * dt, n_dw = b * per256 * dt;
        const double c_dh = t_gemm(b), c_dw = t_gemm(a);
        const double mk = FLOOR ? makespan_floor<FLOOR == kTightFloor>(cus, n_dh, c_dh, n_dw, c_dw) : makespan(cus, n_dh, c_dh, n_dw, c_dw);
        // fp32 accumulator traffic of the step at ~3 TB/s
        const double bytes = (double)a * 256 * D * 8.0 + (dw_beta ? (double)b * 256 * D * 8.0 : (double)b * 256 * D * 4.0);
        return ((a * b + cus - 1) / cus) * t_tile() + mk + bytes / 3.0e6 + 4.0;
    }
    // All work of TT x VT tiles spread evenly, and a bound made of it for a backward in blocks of a x b.
    double even(int TT, int VT) const {
        return (double)TT * VT * (t_tile() + 8.0 * d_tiles() * (256 / tile.bm) * tile.us_per_slice) / cus;
    }
    double quick_floor(double even_us, int TT, int VT, int nblk, int nch) const {
        return even_us + (double)(nblk * nch) * 4.0 + (double)(256 * D) / 3.0e6 * (8.0 * (double)TT * nch + (double)VT * (8.0 * nblk - 4.0));
    }
    // The whole backward of TT x VT tiles in blocks of a x b.
    template <int FLOOR = kPrice>
    double backward(int TT, int VT, int a, int b) const {
        const int nblk = (TT + a - 1) / a, a_last = TT - (nblk - 1) * a;
        const int nch = (VT + b - 1) / b, b_last = VT - (nch - 1) * b;
        // the first row block overwrites dW, later ones add to it
        auto block_cost = [&](int aa, bool beta) {
            return (nch > 1 ? (nch - 1) * step<FLOOR>(aa, b, beta) : 0.0) + step<FLOOR>(aa, b_last, beta);
        };
        return nblk == 1 ? block_cost(a_last, false)
                         : block_cost(a, false) + (nblk > 2 ? (nblk - 2) * block_cost(a, true) : 0.0) + block_cost(a_last, true);
    }
};

// budget_rows != 0 selects row skipping: the plan is made for N compact rows while the workspace
// budget (1 % of the materialised logits) is that of the budget_rows original rows, and the
// workspace also holds the compact-row bookkeeping (row map and per-row scalars).
static bool make_plan(int64_t N, int64_t D, int64_t V, Plan* p, int64_t budget_rows = 0) {
    if (N <= 0 || D <= 0 || V <= 0) return false;
    const Knobs knobs = Knobs::read();
    const int cus = device_cu_count();
    // A row-skipping call asks for two plans (all rows, the valid ones) in its forward and again in its
    // backward, so the cache holds several; the oldest entry goes first.
    struct Key { int64_t N, D, V, B; int cus, fa, fb, fc, fs; Plan plan; bool valid; };
    constexpr int kCached = 32;
    static thread_local Key cache[kCached] = {};
    static thread_local int cache_next = 0;
    for (const Key& k : cache)
        if (k.valid && k.N == N && k.D == D && k.V == V && k.B == budget_rows && k.cus == cus && k.fa == knobs.row_tiles &&
            k.fb == knobs.vocab_tiles && k.fc == knobs.gemm_cols && k.fs == knobs.split_acc) { *p = k.plan; return true; }
    const bool compact = budget_rows != 0;

    const int64_t Np = round_up(N, 256), Vp = round_up(V, 256);
    p->TT = (int)(Np / 256);
    p->VT = (int)(Vp / 256);
    // Vocabulary splits of the forward: TT x S workgroups run in rounds of `cus`, each walking
    // ceil(VT / S) vocabulary tiles; take the S with the least time (the smallest on a tie).  A
    // workgroup costs about a quarter of a tile by itself (fill, merge): counted without it, 27 token
    // tiles x 586 vocabulary tiles went to S = 293 to save 1.6 % of the tile times, and the pairs
    // of 293 splits took half of the workspace from the backward.
    {
        int best_s = 1;
        int64_t best_cost = INT64_MAX;
        const int s_max = p->VT < 2 * cus ? p->VT : 2 * cus;
        for (int s = 1; s <= s_max; ++s) {
            const int64_t rounds = ((int64_t)p->TT * s + cus - 1) / cus;
            const int64_t cost = rounds * (4 * (int64_t)((p->VT + s - 1) / s) + 1);
            if (cost < best_cost) { best_cost = cost; best_s = s; }
        }
        p->S = best_s;
    }
    p->rows = N; p->cols = V;
    p->small_tiles = use_small_tiles(p->TT, p->VT);
    const int S = p->small_tiles && p->fwd_vt() > p->S ? p->fwd_vt() : p->S;       // pairs per token that the workspace holds

    // per (token, split): (max, sum-exp) pair + the logit sum that label smoothing needs
    const size_t md_bytes = (size_t)round_up((int64_t)N * S * 8, 256);
    const size_t partial_bytes = md_bytes + (size_t)round_up((int64_t)N * S * 4, 256);
    size_t budget = (size_t)((double)(compact ? budget_rows : N) * (double)V * 4.0 * 0.01);
    if (budget < kBudgetFloor) budget = kBudgetFloor;
    const size_t scalar_bytes = compact ? (size_t)round_up(Np * 4, 256) : 0;      // one per-row int32 / fp32 array
    const size_t zero_row_bytes = compact ? (size_t)round_up(D * 2, 256) : 0;
    const size_t fixed = 256 + partial_bytes + (compact ? 256 + 4 * scalar_bytes + zero_row_bytes : 0);

    // Row block of a tiles, vocabulary chunk of b tiles.
    int acc_bytes = 4;          // per element of the dH running sum: 4 (fp32) or 2 (split planes)
    auto bytes_needed = [&](int64_t a, int64_t b) {
        return (double)fixed + (double)round_up(a * 256 * D * acc_bytes, 256) + (double)(a * 256) * (double)(b * 256) * 2.0;
    };
    // Tiling for a given contraction tile: the (a, b) with the smallest modelled time (the smallest of
    // equal ones).  The widest blocks are tried first, they are usually the best, and a tiling whose floor
    // is above the best so far is passed over: of 5504 makespans for 16000 x 64 x 2000 26 are left, of 31158
    // for 30000 x 3584 x 151936 1866.  Where nothing is below `bound` the result is `bound` or more.
    auto plan_for_kind = [&](int kind, double bound, int* a_out, int* b_out) -> double {
        BackwardModel model{cus, D, gemm_tile_of_kind(kind)};
        if (knobs.row_tiles > 0 && knobs.vocab_tiles > 0) {
            *a_out = knobs.row_tiles < p->TT ? knobs.row_tiles : p->TT;
            if (compact && *a_out > kCompactMaxRowTiles) *a_out = kCompactMaxRowTiles;
            *b_out = knobs.vocab_tiles < p->VT ? knobs.vocab_tiles : p->VT;
            return 0.0;
        }
        double best_cost = bound;
        const double even_us = model.even(p->TT, p->VT);
        // (row skipping: a row block's row map must fit its LDS table)
        const int a_cap = compact ? kCompactMaxRowTiles : 64;
        const int a_max = p->TT < a_cap ? p->TT : a_cap, b_max = p->VT < 128 ? p->VT : 128;
        *a_out = 1; *b_out = 1;
        for (int a = a_max; a >= 1; --a) {
            const double left = (double)budget - bytes_needed(a, 0);
            int b_fits = left < 0.0 ? 0 : left >= (double)a * 131072.0 * b_max ? b_max : (int)(left / ((double)a * 131072.0));
            if (a == 1 && b_fits < 1) b_fits = 1;           // one tile is always allowed
            for (int b = b_fits; b >= 1; --b) {
                // measured per contraction launch: the split running sum costs 2 us, 9 us when its
                // upper-half plane is also reached through the row map of the compact row space
                const int nblk = (p->TT + a - 1) / a, nch = (p->VT + b - 1) / b;
                const double split_us = acc_bytes == 2 ? (double)nblk * nch * (compact ? 9.0 : 2.0) : 0.0;
                if (model.quick_floor(even_us, p->TT, p->VT, nblk, nch) + split_us > best_cost * kAbove) continue;
                if (model.backward<kFloor>(p->TT, p->VT, a, b) + split_us > best_cost * kAbove) continue;
                if (model.backward<kTightFloor>(p->TT, p->VT, a, b) + split_us > best_cost * kAbove) continue;
                const double cost = model.backward(p->TT, p->VT, a, b) + split_us;
                if (cost <= best_cost) { best_cost = cost; *a_out = a; *b_out = b; }
            }
        }
        return best_cost;
    };
    // 256 x 256 tiles when D is a multiple of 256 and they fill the rounds of `cus` workgroups
    // of a contraction launch to at least 70 %; else 256 x 128.  (The cost model ranks tilings
    // of one tile shape well but is off by ~15 % between the shapes, so the shape is decided
    // by occupancy: measured, D = 1024 and 2048 gain 17 % with the narrow tile, D = 1536 with
    // 77 % occupancy loses 6 %.)
    auto plan_for_acc = [&](int bytes, double bound, int* a_out, int* b_out, int* kind_out) -> double {
        acc_bytes = bytes;
        double cost = 0.0;
        *kind_out = 1;
        if (knobs.gemm_cols != 0) {
            *kind_out = knobs.gemm_cols == 256 ? 0 : 1;
            if (*kind_out == 0) cost = plan_for_kind(0, bound, a_out, b_out);
        } else if (D % 256 == 0) {
            cost = plan_for_kind(0, 1e300, a_out, b_out);      // (the tile follows from its tiling, below the bound or not)
            const int64_t tiles = (int64_t)(*a_out + *b_out) * (D / 256);
            const int64_t rounds = (tiles + cus - 1) / cus;
            *kind_out = (double)tiles >= 0.7 * (double)(rounds * cus) ? 0 : 1;
        }
        if (*kind_out == 1) cost = plan_for_kind(1, bound, a_out, b_out);
        return cost;
    };
    // The dH running sum: plain fp32 unless the split form (half the workspace, a little slower
    // per launch) buys a tiling that the model rates at least 3 % faster.
    int best_a = 1, best_b = 1, best_kind = 1, sa = 1, sb = 1, skind = 1;
    const double cost_f32 = plan_for_acc(4, 1e300, &best_a, &best_b, &best_kind);
    const double cost_split = plan_for_acc(2, knobs.split_acc == 0 ? 0.97 * cost_f32 : 1e300, &sa, &sb, &skind);
    p->split_acc = 0;
    if (knobs.split_acc == 2 || (knobs.split_acc == 0 && cost_split < 0.97 * cost_f32)) {
        best_a = sa; best_b = sb; best_kind = skind; p->split_acc = 1;
    }
    acc_bytes = p->split_acc ? 2 : 4;
    p->gemm_kind = best_kind;
    p->Nb = (int64_t)best_a * 256;
    p->Vc = (int64_t)best_b * 256;
    p->off_status = 0;
    p->off_partials = 256;
    p->off_sumz = p->off_partials + md_bytes;
    p->off_dhacc = p->off_partials + partial_bytes;
    p->off_g = p->off_dhacc + (size_t)round_up(p->Nb * D * acc_bytes, 256);
    p->total = p->off_g + (size_t)(p->Nb * p->Vc * 2);
    p->rows_pad = Np;
    p->off_count = p->off_perm = p->off_labels_c = p->off_fa_c = p->off_fb_c = p->off_zero_row = 0;
    if (compact) {
        p->off_count = round_up((int64_t)p->total, 256);
        p->off_perm = p->off_count + 256;
        p->off_labels_c = p->off_perm + scalar_bytes;
        p->off_fa_c = p->off_labels_c + scalar_bytes;
        p->off_fb_c = p->off_fa_c + scalar_bytes;
        p->off_zero_row = p->off_fb_c + scalar_bytes;
        p->total = p->off_zero_row + zero_row_bytes;
    }
    p->budget = budget;
    p->forced = knobs.row_tiles || knobs.vocab_tiles || knobs.gemm_cols || knobs.split_acc;
    // the gradient chunk is addressed with 32-bit byte offsets (only a forced tiling can get here)
    if (p->Nb * p->Vc * 2 >= ((int64_t)1 << 32)) return false;
    cache[cache_next] = {N, D, V, budget_rows, cus, knobs.row_tiles, knobs.vocab_tiles, knobs.gemm_cols, knobs.split_acc, *p, true};
    cache_next = (cache_next + 1) % kCached;
    return true;
}

// All rows in one block and budget to spare: the Plan itself has no use for more, but a schedule that cuts
// dH's serial reduction into parts wants room for their planes (up to 16 parts) beside a wide chunk.  *q
// is that layout.  A call takes it only where its workspace holds it, so what a call NEEDS stays p.total.
static bool room_for_planes(const Plan& p, int64_t D, Plan* q) {
    if (p.forced || p.Nb != (int64_t)p.TT * 256 || p.TT > 16) return false;
    const int64_t slack = (int64_t)p.budget - (int64_t)p.total, b = p.Vc / 256;
    const int64_t tile = (int64_t)p.TT * 131072, planes = 15 * (int64_t)round_up(p.rows * D * 4, 256);
    const int64_t room = b < p.VT ? slack / 2 : slack;
    const int64_t spare = (planes < room ? planes : room) / 256 * 256;
    if (spare < planes / 15) return false;
    int64_t wide = b + (slack - spare) / tile;
    wide = wide < p.VT ? wide : p.VT;
    const size_t more = (size_t)(spare + (wide - b) * tile);
    *q = p;
    q->Vc = wide * 256;
    q->off_g += (size_t)spare;
    q->total += more;
    if (q->off_count) {
        q->off_count += more; q->off_perm += more; q->off_labels_c += more;
        q->off_fa_c += more; q->off_fb_c += more; q->off_zero_row += more;
    }
    return true;
}

// ------------------------------------------------------------------------------------------
// Schedules of the backward.  A Plan walks [row block x vocabulary chunk] steps whose gradient
// chunk and dH sums share 1 % of the logits' size.  Two things make other orders faster where they
// fit the same workspace:
//   * When dW is overwritten, the rows of dW behind the current vocabulary chunk hold nothing yet.
//     A step over ALL rows can keep its gradient chunk there: far larger chunks, hence fewer
//     launches, and dW is written once instead of being added to by every row block.  The chunks
//     shrink with the rest of dW, and a step over all rows of a narrow chunk has few dW tiles with a
//     long reduction: below a width the chunk is taken in row_parts steps over part of the rows
//     each, whose chunks are that much wider.  The last ones use the workspace.
//   * The rows of dHidden in front of the current row block are final only once their own block has
//     run.  With the blocks taken from the last to the first, a block may keep its gradient chunk or
//     its dH sums there -- also under row skipping, where compact row r goes to a row >= r.
//   * A contraction with few output tiles (few rows, or a small vocabulary) leaves most of the
//     GPU idle for the length of its reduction; its K range is split into parts that write planes
//     of their own, summed by a small launch.
// ------------------------------------------------------------------------------------------
// One row block of an order with dHidden as scratch: a row tiles, chunks of b vocabulary tiles.
struct RowBlock {
    int r0, a, b, kind, split_acc;      // r0: first row tile
    bool acc_in_dh, g_in_dh;            // dH sums / gradient chunk in the front rows of dHidden
    size_t off_acc, off_g;              // from the workspace or from dHidden
};
constexpr int kMaxRowBlocks = 48;

struct ScheduleSteps {
    bool use;                   // false: the Plan's row blocks and chunks, or blocks[]
    int kind;                   // contraction tile
    int a;                      // row tiles per block (all of them: one row block)
    int b;                      // vocabulary tiles per chunk, at most
    int split_h, split_w;       // K parts of the dH / dW contraction, at most
    bool tail;                  // gradient chunks in the unwritten rows of dW where they fit
    int row_parts, b_min;       // chunks of fewer than b_min tiles are taken in row_parts steps
    int split_acc;              // dH running sum as two 16-bit planes (see GemmJob); split_h = 1
    int64_t plane_h, plane_w;   // fp32 elements per plane
    size_t off_acc, off_part_w, off_hc, off_g;      // workspace: dH planes, dW planes, gathered rows, gradient chunk
    size_t g_bytes;
    double us;                  // modelled time of the backward
    double plan_us;             // ... and of the Plan's order, same model
};
struct Schedule : ScheduleSteps {
    int n_blocks;               // > 0: blocks[], in execution order
    RowBlock blocks[kMaxRowBlocks];
};

// The chunk that starts `rest` columns before the end of the vocabulary: b tiles wide, in steps over
// `rows` row tiles each.
struct ScheduleChunk { int64_t b; int rows; bool in_tail; };
static inline ScheduleChunk schedule_chunk(const ScheduleSteps& sc, int64_t D, int64_t rest) {
    const int64_t rest_tiles = (rest + 255) / 256;
    ScheduleChunk c = {0, 0, false};
    for (int parts = 1; ; parts = sc.row_parts) {
        const int rows = (sc.a + parts - 1) / parts;
        const int64_t row_bytes = (int64_t)rows * 256 * 2;           // of one vocabulary column of the chunk
        const int64_t in_ws = (int64_t)sc.g_bytes / (row_bytes * 256);
        // the chunk's b x 256 columns lie behind dW's own b x 256 rows (256 B for the alignment)
        const int64_t behind = sc.tail ? (rest * D * 4 - 256) / (256 * (row_bytes + D * 4)) : 0;
        int64_t b = in_ws > behind ? in_ws : behind;
        b = b < sc.b ? b : sc.b;
        b = b < rest_tiles ? b : rest_tiles;
        c = {b, rows, b > in_ws};
        if (parts == sc.row_parts || b >= sc.b_min || b == rest_tiles) return c;
    }
}

// Contractions on tiles of two wavefront groups (TurnTile), microseconds: a 256 x 256 x 64 slice 1.38, 13 beside the slices (first
// slice, epilogue), 6 more where the item adds to its output.  A last column tile whose second half lies behind the matrix takes 0.66
// of that, which is counted on in launches of four rounds and more: items go out in the order of their rows, not the short ones last
// (19 x 14 tiles at D = 3456, 266 items, rated as if the 19 halves filled in: 248 -> 267 us a step).
// Rated / measured: 1008 items of 32 x 40 tiles at D = 3584 859 / 866, 768 of 64 x 32 at D = 2048 758 / 789, 1120 of 16 x 64 at D = 3584
// 741 / 720, 512 of 16 x 16 at D = 4096 212 / 228, 256 of 32 x 32 at D = 896 196 / 181.
struct TurnModel {
    int64_t cus, D;
    // Launches of fewer items leave too many compute units idle (128 items where 256 x 128 tiles are 256: 105 us for 77): not rated.
    bool enough(int64_t tiles) const { return 5 * tiles * ((D + 255) / 256) >= 3 * cus; }
    static double item(double slices, bool beta) { return slices * 1.38 + 13.0 + (beta ? 6.0 : 0.0); }
    // a x b tiles of 256, reductions of s_dh and s_dw slices in parts_h and parts_w parts.  FLOOR: a bound it never falls below.
    template <int FLOOR = kPrice>
    double us(int64_t a, int64_t parts_h, int64_t s_dh, bool dh_beta, int64_t b, int64_t parts_w, int64_t s_dw, bool dw_beta) const {
        const int64_t across = (D + 255) / 256, n_dh = a * parts_h * across, n_dw = b * parts_w * across;
        const double c_dh = item((double)s_dh, dh_beta), c_dw = item((double)s_dw, dw_beta);
        const double whole = FLOOR ? makespan_floor<FLOOR == kTightFloor>(cus, n_dh, c_dh, n_dw, c_dw) : makespan(cus, n_dh, c_dh, n_dw, c_dw);
        return halves(a * parts_h + b * parts_w) ? whole * half_columns() : whole;
    }
    // Whether a last column tile whose second half lies behind the matrix is counted on, and what is left of the launch then.
    bool halves(int64_t tiles) const { return D % 256 != 0 && D % 256 <= 128 && tiles * ((D + 255) / 256) >= 4 * cus; }
    double half_columns() const { const double across = (double)((D + 255) / 256); return (across - 0.34) / across; }
};

// Time model of the schedules, microseconds, from launches timed on MI355X with random data: a
// 256 x 256 x 64 slice 1.58, a 256 x 128 x 64 one 0.79; a gradient tile adds 7 to its slices, a
// contraction tile 13 / 9 (first slice, epilogue) and 2 more where it adds to its output; a
// launch boundary 4; HBM 4.5 TB/s where a step moves more than it computes.  (Checked against forced tilings: 8192 x
// 896 x 151936 in steps of 16 x 16 tiles 7.47 ms modelled, 7.33 measured; of 32 x 32 6.3 and 6.45.)
struct ScheduleModel {
    int cus; int64_t D; GemmTile tile;
    bool mapped;                // the dW job reads hidden rows through the row map: priced at 0.11 of a slice more, what the lookup
                                // took with its bounds checks (0.85 us against 0.76); byte offsets take less, see OperandTile
    int64_t dt;                 // output tiles across D
    bool one_to_unit = false;   // 256 x 128 tiles: not two to a compute unit
    bool turns = false;         // tiles of two wavefront groups (256 x 256) where those are faster
    bool duo() const { return tile.kind == 1 && !mapped && !one_to_unit; }
    ScheduleModel() = default;
    ScheduleModel(int cus_, int64_t D_, GemmTile tile_, bool mapped_ = false)
        : cus(cus_), D(D_), tile(tile_), mapped(mapped_), dt((D_ + tile_.bn - 1) / tile_.bn) {}
    ScheduleModel with_turns(bool on) const { ScheduleModel m = *this; m.turns = on; return m; }
    // (32-bit divisions: a search makes tens of thousands of them, and 64-bit ones take twice as long)
    static int64_t ceil_div(int64_t a, int64_t b) { return (int64_t)(((uint32_t)a + (uint32_t)b - 1u) / (uint32_t)b); }
    double slice() const { return tile.kind == 0 ? 1.58 : 0.79; }
    double item(int64_t slices, bool beta) const { return (double)slices * slice() + (tile.kind == 0 ? 13.0 : 9.0) + (beta ? 2.0 : 0.0); }
    double duo_item(int64_t slices, bool beta, bool split) const { return (double)slices * 1.53 + 10.0 + (beta ? 6.0 : 0.0) + (split ? 8.0 : 0.0); }
    int64_t d_tiles() const { return dt; }
    // Whether launches of at most a x b tiles may be on tiles of two wavefront groups, and the least part of their time that such a launch
    // is rated with.
    struct MayTurn { bool on; double part; };
    MayTurn may_turn(int64_t a, int64_t b, int split_h, int split_w) const {
        const TurnModel turn{cus, D};
        const int64_t tiles = a * split_h + b * split_w;
        const bool on = turns && turn.enough(tiles);
        return {on, on && turn.halves(tiles) ? turn.half_columns() : 1.0};
    }
    // What an item costs at least, of either form: a slice and what is beside the slices of the work spread evenly, and a slice of one
    // item's reduction.  (Tiles of two wavefront groups are 256 columns wide, two of these at 256 x 128.)
    double least_slice(MayTurn turn) const { return turn.on ? (tile.kind == 0 ? 1.38 * turn.part : 0.69) : duo() ? 0.765 : slice(); }
    double least_item(MayTurn turn) const { return duo() ? 5.0 : turn.on ? (tile.kind == 0 ? 13.0 * turn.part : 6.0) : item(0, false); }
    double least_chain(MayTurn turn) const { return turn.on && tile.kind == 0 ? 1.38 * turn.part : slice(); }
    // Both contractions of a step; *kind becomes the tile they take.  (Narrow tiles are searched for only where they could win.)
    template <int FLOOR = kPrice>
    double contractions(int64_t n_dh, int64_t s_dh, bool dh_beta, bool split, int64_t n_dw, int64_t s_dw, bool dw_beta, int* kind = nullptr) const {
        const double c_dh = item(s_dh, dh_beta), c_dw = item(s_dw, dw_beta) + (mapped ? (double)s_dw * 0.11 * slice() : 0.0);
        const double least = makespan_floor<FLOOR != kFloor>(cus, n_dh, c_dh, n_dw, c_dw);
        double duo_us = 1e300;
        if (duo()) {
            duo_us = duo_makespan<FLOOR != kPrice>(cus, n_dh, duo_item(s_dh, dh_beta, split), n_dw, duo_item(s_dw, dw_beta, false));
            if (kind) *kind = 3;
            if (duo_us <= least) return duo_us;
        }
        const double us = FLOOR ? least : makespan(cus, n_dh, c_dh, n_dw, c_dw);
        if (duo_us < us) return duo_us;
        if (kind) *kind = tile.kind;
        return us;
    }
    // The same of a x b tiles in parts_h and parts_w parts where tiles of two wavefront groups may be taken: the faster ones.  The form
    // with the lower floor is priced first, the other one only if its floor is 7 % below that.
    template <int FLOOR>
    double with_turns_us(int64_t a, int64_t parts_h, int64_t s_dh, bool dh_beta, bool split, int64_t b, int64_t parts_w, int64_t s_dw, bool dw_beta) const {
        const TurnModel turn{cus, D};
        if (!turn.enough(a * parts_h + b * parts_w))
            return contractions<FLOOR>(a * dt * parts_h, s_dh, dh_beta, split, b * dt * parts_w, s_dw, dw_beta);
        const int64_t n_dh = a * dt * parts_h, n_dw = b * dt * parts_w;
        const double f_turn = turn.template us<FLOOR ? FLOOR : kTightFloor>(a, parts_h, s_dh, dh_beta, b, parts_w, s_dw, dw_beta);
        const double f_other = contractions<FLOOR ? FLOOR : kTightFloor>(n_dh, s_dh, dh_beta, split, n_dw, s_dw, dw_beta);
        const bool first = f_turn <= f_other;
        double us = first ? f_turn : f_other;
        if (FLOOR) return us;
        us = first ? turn.us(a, parts_h, s_dh, dh_beta, b, parts_w, s_dw, dw_beta) : contractions(n_dh, s_dh, dh_beta, split, n_dw, s_dw, dw_beta);
        if ((first ? f_other : f_turn) * 1.07 >= us) return us;
        const double other = first ? contractions(n_dh, s_dh, dh_beta, split, n_dw, s_dw, dw_beta) : turn.us(a, parts_h, s_dh, dh_beta, b, parts_w, s_dw, dw_beta);
        return other < us ? other : us;
    }
    // (The loop of FP8 tiles and of bf16 ones before those of two wavefront groups, which take 5 - 15 % less, up to 30 % where the taller
    // ones fill the rounds better, see tall_grad_tiles: the orders stay those that were measured with it.)
    double logit_tile() const { return (double)(D / 64) * 1.55 + 7.0; }
    // One step over a x b tiles.  FLOOR: with makespan_floor.
    template <int FLOOR = kPrice>
    double step(int64_t a, int64_t b, int split_h, int split_w, bool dh_beta, bool dw_beta, bool split = false) const {
        const int64_t kh = ceil_div(b, split_h), kw = ceil_div(a, split_w);       // K tiles per part
        const int64_t n_dh = a * dt * ceil_div(b, kh), n_dw = b * dt * ceil_div(a, kw);
        const double mk = turns ? with_turns_us<FLOOR>(a, ceil_div(b, kh), kh * 4, dh_beta, split, b, ceil_div(a, kw), kw * 4, dw_beta)
                                : contractions<FLOOR>(n_dh, kh * 4, dh_beta, split, n_dw, kw * 4, dw_beta);
        const double g = (double)(a * b) * 131072.0, w = (double)b * 512.0 * (double)D;
        const double tiles_us = (double)((a * b + cus - 1) / cus) * logit_tile();
        const double tiles_mem = (g + w) / 4.5e6;
        const double gemm_mem = (g * 2.0 + w * (dw_beta ? 5.0 : 3.0)) / 4.5e6;
        double t = (tiles_us > tiles_mem ? tiles_us : tiles_mem) + (mk > gemm_mem ? mk : gemm_mem) + 8.0;
        if (split_w > 1) t += 4.0 + w * 2.0 * (double)(split_w + 1) / 4.0e6;
        return t;
    }
    // A bound that no sequence of steps over `a` row tiles and `b` vocabulary tiles falls below, in chunks of
    // at most `b_max`: all work spread evenly, the serial reduction of one item per step or all bytes at the rate
    // of HBM, and what each step costs by itself.
    double floor_us(int64_t a, int64_t b, int64_t b_max, int split_h, int split_w) const {
        const MayTurn turn = may_turn(a, b_max < b ? b_max : b, split_h, split_w);
        const double ab = (double)(a * b), per_item = least_item(turn);
        const double steps = (double)ceil_div(b, b_max);
        const int64_t kh = ceil_div(b, split_h), kw = ceil_div(a, split_w);
        double even = (8.0 * ab * (double)dt * least_slice(turn) + ((double)(b * ceil_div(a, kw)) + (double)a * steps) * (double)dt * per_item) / (double)cus;
        const double chain = least_chain(turn);
        const double dh_item = (double)(kh * 4) * chain + steps * per_item, dw_item = steps * ((double)(kw * 4) * chain + per_item);
        if (dh_item > even) even = dh_item;
        if (dw_item > even) even = dw_item;
        const double tiles_us = ab * logit_tile() / (double)cus;
        const double w = (double)b * 512.0 * (double)D;
        const double tiles_mem = (ab * 131072.0 + w) / 4.5e6, gemm_mem = (ab * 262144.0 + w * 3.0) / 4.5e6;
        return (tiles_us > tiles_mem ? tiles_us : tiles_mem) + (even > gemm_mem ? even : gemm_mem) + 8.0 * steps +
               (split_w > 1 ? 4.0 * steps + w * 2.0 * (double)(split_w + 1) / 4.0e6 : 0.0);
    }
    // The part of it that grows with the width, per vocabulary tile.
    double floor_per_tile(int64_t a, int64_t b_max, int split_h, int split_w) const {
        const MayTurn turn = may_turn(a, b_max, split_h, split_w);
        const double per_item = least_item(turn), steps = 1.0 / (double)b_max;
        return (double)a * logit_tile() / (double)cus + 8.0 * steps +
               (8.0 * (double)a * (double)dt * least_slice(turn) + (1.0 + (double)a * steps) * (double)dt * per_item) / (double)cus;
    }
};

// Tile of one launch of n_dh and n_dw work items of `kind` with reductions of s_dh and s_dw slices: the forms that a
// plan or schedule leaves open.  row_map: the dW job reads its rows through a map (256 x 128 tiles one to a unit).
static int contraction_kind(int kind, int64_t D, int64_t n_dh, int64_t s_dh, bool dh_beta, bool split, int64_t n_dw, int64_t s_dw,
                            bool dw_beta, bool row_map, const Knobs& knobs) {
    if (small_contractions(kind, n_dh + n_dw, knobs)) return 2;
    if (kind != 1 || knobs.gemm_cols != 0 || row_map) return kind;
    const ScheduleModel m{device_cu_count(), D, gemm_tile_of_kind(kind)};
    m.contractions(n_dh, s_dh, dh_beta, split, n_dw, s_dw, dw_beta, &kind);
    return kind;
}

// The same of a launch whose rows are counted on the device (a x b tiles, no K parts, dH sums in planes): the tile that it takes
// over all rows, so that a call without ignored rows has the sums and the time of one that does not look for them -- but tiles two
// to a unit only where they are rated no slower over launches with one to four eighths of the rows left out, and at none of them a
// sixth slower: dH's long items, on units that they share, bound what is left of a launch (without that, 3000 x 2048 x 151936 with
// 40 % ignored 3.74 -> 4.02 ms, 7000 x 640 x 151936 with 25 % 3.87 -> 3.96, 8001 x 576 x 150001 with 40 % 3.66 -> 3.71).
static int counted_contraction_kind(int kind, int64_t D, int64_t a, int64_t b, int64_t d_tiles, bool dh_beta, bool dw_beta, const Knobs& knobs) {
    const int taken = contraction_kind(kind, D, a * d_tiles, b * 4, dh_beta, true, b * d_tiles, a * 4, dw_beta, false, knobs);
    if (taken != 3) return taken;
    ScheduleModel m{device_cu_count(), D, gemm_tile_of_kind(kind)};
    m.one_to_unit = true;
    double paired = 0.0, single = 0.0;
    for (int64_t eighths = 7; eighths >= 4; --eighths) {
        const int64_t left = (eighths * a + 4) / 8;
        const double two = duo_makespan(m.cus, left * d_tiles, m.duo_item(b * 4, dh_beta, true), b * d_tiles, m.duo_item(left * 4, dw_beta, false));
        const double one = m.contractions(left * d_tiles, b * 4, dh_beta, true, b * d_tiles, left * 4, dw_beta);
        if (6.0 * two > 7.0 * one) return kind;
        paired += two;
        single += one;
    }
    return paired <= single ? 3 : kind;
}

// Whether a launch over e_h x e_w tiles takes tiles of two wavefront groups instead of `kind` (contraction_kind); parts_h / parts_w parts of s_h and s_w
// slices each.  From the shape of the launch alone, so that calls that count their rows and calls that compute all of them agree.
static bool turn_contractions(int kind, int64_t D, int64_t e_h, int64_t parts_h, int64_t s_h, bool beta_h, int64_t e_w, int64_t parts_w, int64_t s_w,
                              bool beta_w, bool row_map, const Knobs& knobs) {
    const int cus = device_cu_count();
    if (kind == 2 || knobs.gemm_cols != 0 || !TurnModel{cus, D}.enough(e_h * parts_h + e_w * parts_w)) return false;
    const ScheduleModel m{cus, D, gemm_tile_of_kind(kind == 0 ? 0 : 1), row_map};
    const int64_t per256 = 256 / m.tile.bm;
    const double other = m.contractions(e_h * parts_h * per256 * m.d_tiles(), s_h, beta_h, false, e_w * parts_w * per256 * m.d_tiles(), s_w, beta_w);
    const double us = TurnModel{cus, D}.us(e_h, parts_h, s_h, beta_h, e_w, parts_w, s_w, beta_w);
    return us < other;
}

// One contraction launch of a backward: row_tiles x v_tiles tiles of 256, the reductions of dH over the columns and of dW over the rows in parts
// of at most kh and kw tiles; whether the jobs add to their outputs.
struct LaunchShape { int row_tiles, v_tiles, kh, parts_h, kw, parts_w; bool dh_beta, dw_beta; };
static LaunchShape launch_shape(int row_tiles, int v_tiles, int split_h, int split_w, bool dh_beta, bool dw_beta) {
    const int kh = (v_tiles + split_h - 1) / split_h, kw = (row_tiles + split_w - 1) / split_w;
    return {row_tiles, v_tiles, kh, (v_tiles + kh - 1) / kh, kw, (row_tiles + kw - 1) / kw, dh_beta, dw_beta};
}
// Its tiles: `kind` is the order's; row_map: the dW job reads its rows through a map; counted: rows counted on the device.
struct LaunchTiles { int kind; bool turn; };
static LaunchTiles launch_tiles(const LaunchShape& s, int64_t D, int kind, bool split_acc, bool row_map, bool counted, const Knobs& knobs) {
    const int64_t d_tiles = (D + gemm_tile_of_kind(kind).bn - 1) / gemm_tile_of_kind(kind).bn;
    const int taken = counted ? counted_contraction_kind(kind, D, s.row_tiles, s.v_tiles, d_tiles, s.dh_beta, s.dw_beta, knobs)
                              : contraction_kind(kind, D, (int64_t)s.row_tiles * s.parts_h * d_tiles, s.kh * 4, s.dh_beta, split_acc,
                                                 (int64_t)s.v_tiles * s.parts_w * d_tiles, s.kw * 4, s.dw_beta, row_map, knobs);
    return {taken, turn_contractions(taken, D, s.row_tiles, s.parts_h, s.kh * 4, s.dh_beta, s.v_tiles, s.parts_w, s.kw * 4, s.dw_beta, row_map, knobs)};
}

// The forward under the same constants, to compare calls with and without row skipping (what its tiles take: forward_tile): rounds of workgroups that walk their vocabulary tiles, or of one
// small tile each (500 x 2048 x 10000, two rounds of 32 slices: 42 us).
struct ForwardCost {
    int cus; int64_t D;
    double us(const Plan& p) const {
        if (p.small_tiles) {
            const int64_t tiles = (int64_t)p.fwd_tt() * p.fwd_vt();
            return (double)((tiles + cus - 1) / cus) * ((double)(D / 64) * 0.55 + 4.0);
        }
        const int64_t rounds = ((int64_t)p.TT * p.S + cus - 1) / cus;
        return (double)(rounds * ((p.VT + p.S - 1) / p.S)) * ((double)(D / 64) * 1.55 + 4.0);
    }
};

// Tiles of a bf16 forward beyond the 128 x 128 ones: TileBig's 256 x 256 loop, or 256 x 256 or 384 x 256 outputs by two
// groups of wavefronts (PingTile), whichever is rated fastest.  A workgroup walks a split of the vocabulary, of whole tiles (TileBig)
// or cut at half tiles, whose last half tile brings fewer products but the loads and the epilogue of a whole one: 0.65 of its slices.
// Fitted to 399 forwards of 200 to 32768 rows, D 64 to 4096, V 1000 to 151936, in each of the three forms (3.7 % standard
// deviation): a slice takes longer the more of the compute units are busy, TileBig's most (power), and an epilogue costs about two
// slices.  So TileBig has launches that leave units idle and those of few slices and tiles to a workgroup, the taller tiles long
// ones; TileBig's 1.5 % are the error of the rating (640 other forwards: 1.9 - 2.7 % faster than on TileBig on average and up to
// 2.5 % slower; without them up to 7 %).  us of TileBig / square / tall: 13265 x 64 x 10636 44.8 / 48.2 / 48.7,
// 903 x 768 x 9581 (152 workgroups of one tile) 22.1 / 24.0 / 31.3, 4606 x 1664 x 6680 90.1 / 84.7 / 97.6, 16384 x 2048 x 151936
// 7983 / 7576 / 6977.  (Rows that are counted on the device: by the splits of all rows; those calls are long, and the taller
// tiles theirs.)
enum ForwardTile { kForwardSmall, kForwardBig, kForwardSquare, kForwardTall };
static ForwardTile forward_tile(const Plan& p, int64_t D) {
    if (p.small_tiles) return kForwardSmall;
    const int cus = device_cu_count();
    const int64_t work = (int64_t)p.TT * p.S, rounds = (work + cus - 1) / cus;
    const double busy = (double)work / (double)(rounds * cus), slices = (double)(D / 64);
    auto halves = [&](int64_t unit) { return ((p.cols + unit - 1) / unit + p.S - 1) / p.S; };       // half tiles of the longest split
    auto us = [&](double launch, double round, double tile, double slice, double slice_busy, int64_t half) {
        const double products = (double)(half / 2) + 0.65 * (double)(half % 2);
        return launch + (double)rounds * (round + (double)((half + 1) / 2) * tile + products * slices * (slice + slice_busy * busy));
    };
    const double big = 0.985 * us(5.1, 1.8, 2.33, 0.56, 0.89, 2 * ((p.VT + p.S - 1) / p.S));
    const double square = us(5.2, 2.4, 2.5, 0.75, 0.63, halves(128)), tall = us(6.7, 2.5, 3.7, 1.12, 0.78, halves(192));
    return tall <= square && tall <= big ? kForwardTall : square < big ? kForwardSquare : kForwardBig;
}

// Row blocks from the last to the first with dHidden's front rows as scratch: the partition of the
// row tiles with the least modelled time (f(R) = min over a of [block of rows R - a .. R] + f(R - a)).
struct RowBlockPlanner {
    ScheduleModel m[2];
    int TT, VT; int64_t D; size_t region, off0; bool compact, dw_free;
    // Rows 0 .. R: their least time and the last block of that order once `exact`, else it is `us` or more.
    struct State { double us; RowBlock block; bool exact; };
    State states[1 + 256];
    struct Priced { int b; bool beta; double us; };
    Priced priced[1 + 64][2][2][3];
    static constexpr double kNone = 1e300;

    template <int FLOOR = kPrice>
    double block_us(const RowBlock& k, bool beta) const {
        const int64_t nch = (VT + k.b - 1) / k.b;
        const ScheduleModel& mm = m[k.kind];
        double t = nch > 1 ? (double)(nch - 1) * mm.template step<FLOOR>(k.a, k.b, 1, 1, true, beta, k.split_acc != 0) : 0.0;
        t += mm.template step<FLOOR>(k.a, VT - (nch - 1) * k.b, 1, 1, nch > 1, beta, k.split_acc != 0);
        if (k.split_acc) t += (double)nch * (compact ? 9.0 : 2.0);
        return t;
    }
    void prepare() {
        for (int a = 0; a <= 64 && a <= TT; ++a)
            for (int i = 0; i < 12; ++i) priced[a][i / 6][i / 3 % 2][i % 3].b = 0;
        states[0].us = 0.0;
        states[0].exact = true;
        for (int R = 1; R <= TT; ++R) {
            const double f0 = m[0].floor_us(R, VT, VT, 1, 1), f1 = m[1].floor_us(R, VT, VT, 1, 1);
            states[R].us = f0 < f1 ? f0 : f1;
            states[R].exact = false;
        }
    }
    // The least time of the first R row tiles if it is below `bound`, else kNone.
    double best(int R, double bound) {
        State& st = states[R];
        if (st.exact) return st.us;
        if (st.us > bound * kAbove) return kNone;
        double least = bound;
        bool found = false;
        const int sizes[] = {R, (R + 1) / 2, (R + 2) / 3, 4, 6, 8, 10, 12, 14, 16, 20, 24, 32};
        for (int i = 0; i < 13; ++i) {
            const int a = sizes[i];
            if (a > R || a > 64 || (compact && a > kCompactMaxRowTiles)) continue;
            const int64_t front = (int64_t)(R - a) * 256 * D * 2, ws = (int64_t)region, tile = (int64_t)a * 131072;
            for (int split = 0; split < 2; ++split) {
                const int64_t acc = round_up((int64_t)a * 256 * D * (split ? 2 : 4), 256);
                // where the chunk gets widest: sums in front of the block, chunk in front of it, both in the workspace
                RowBlock k = {R - a, a, 0, 0, split, false, false, off0, off0};
                int64_t cap = 0;
                if (acc <= front && ws / tile > cap) { cap = ws / tile; k.acc_in_dh = true; k.g_in_dh = false; k.off_acc = 0; k.off_g = off0; }
                if (acc <= ws && front / tile > cap) { cap = front / tile; k.acc_in_dh = false; k.g_in_dh = true; k.off_acc = off0; k.off_g = 0; }
                if (acc < ws && (ws - acc) / tile > cap) { cap = (ws - acc) / tile; k.acc_in_dh = k.g_in_dh = false; k.off_acc = off0; k.off_g = off0 + (size_t)acc; }
                if (cap > VT) cap = VT;
                if (cap > 30000 / a) cap = 30000 / a;                    // 32-bit chunk offsets
                if (cap < 1) continue;
                const int64_t nch = (VT + cap - 1) / cap;
                const int64_t rounds = a * cap / m[0].cus;
                const int64_t bs[3] = {cap, (VT + nch - 1) / nch, rounds ? rounds * m[0].cus / a : cap};
                for (int kind = 0; kind < 2; ++kind) {
                    if (kind == 0 && m[0].d_tiles() * 256 * 7 > D * 8) continue;
                    k.kind = kind;
                    for (int j = 0; j < 3; ++j) {
                        if (j > 0 && bs[j] == bs[j - 1]) continue;
                        k.b = (int)bs[j];
                        if (k.b < 1 || k.b > cap) continue;
                        const bool beta = R < TT || !dw_free;
                        Priced& known = priced[a][split][kind][j];           // chunks in the workspace are alike for every R
                        const bool hit = known.b == k.b && known.beta == beta;
                        if (!hit && block_us<kFloor>(k, beta) + states[R - a].us > least * kAbove) continue;
                        const double us = hit ? known.us : block_us(k, beta);
                        known = {k.b, beta, us};
                        if (us + states[R - a].us > least * kAbove) continue;
                        const double rest = best(R - a, kNone);
                        if (us + rest < least) { least = us + rest; st.block = k; found = true; }
                    }
                }
            }
        }
        if (!found) { st.us = st.us > bound ? st.us : bound; return kNone; }
        st.us = least;
        st.exact = true;
        return least;
    }
};

// A forward over all rows that leaves the ignored ones out: their number is found on the device, so the launch has the
// workgroups of all rows and those beyond the rows that take part return at once; from the plan's partials on (the plan's own
// are not needed then) lie the row map, the counts, FP8 scales in the order of those rows, and the partials: 256 per workgroup.
// Taken from about 1 ms of forward on (1.15 PFLOP/s, what 256 x 256 tiles of one loop reach; the taller tiles 5 - 13 % more): 8192 x 896 x 151936 with 15 % ignored 1.87 -> 1.63 ms, 4099 x 2048 x 128256
// with 5 % 1.76 -> 1.68, 3000 x 2048 x 151936 with 25 % 1.59 -> 1.23, none ignored 1.591 -> 1.599.
// The label scan is one workgroup: 4 us and 0.4 ns a row (131072 rows 55 us, a million 406), paid also where nothing is ignored.
// It may take a fiftieth of the forward, whose products run at a rate that falls with D (2 N V (0.75 D + 72) fs: 131072 x 64 x 70000
// 2.19 ms, 8192 x 896 x 80000 0.94), up to twice that with FP8 logits: 0.2 to 1.2 % on 8192 to 65536 rows without ignored ones;
// calls that it leaves out lost 2.5 % (131072 x 256 x 32000) to 16 % (1000000 x 64 x 9100) there.
// Below 1 ms, and for few row tiles, a launch of one round hardly gets shorter by the rows that real padding leaves out.
// Whether it is taken decides the order of the fp32 sums, so it follows from the shape alone and not from the workspace of a
// call: the layout has to fit the smallest one that the shape's calls accept, the static array's included.
struct ForwardSkip { bool use; int s_max, workgroups; size_t off_perm, off_found, off_scales, off_partials, off_sumz, end; };
static ForwardSkip forward_skip(const Plan& p, int64_t D, bool fp8) {
    ForwardSkip f = {};
    if ((p.small_tiles && !fp8) || p.TT < 8 || g_force_row_skipping.load(std::memory_order_relaxed) == 1) return f;
    if (2.0 * (double)p.rows * (double)p.cols * (double)D < 1.15e12) return f;
    const double scan_ns = 4000.0 + 0.4 * (double)p.rows, forward_ns = 2e-6 * (double)p.rows * (double)p.cols * (0.75 * (double)D + 72.0);
    if (50.0 * scan_ns > forward_ns) return f;
    const int cus = device_cu_count(), most = 2 * p.S + 8;
    f.s_max = most < p.VT ? most : p.VT;
    if (f.s_max > 1024) f.s_max = 1024;
    if (f.s_max < p.S) return f;
    f.workgroups = (p.TT * p.S + cus - 1) / cus * cus;
    f.off_perm = p.off_partials;
    f.off_found = f.off_perm + (size_t)p.TT * 1024;
    f.off_scales = f.off_found + 256;                          // FP8: the scale bytes of the rows that take part
    f.off_partials = f.off_scales + (fp8 ? (size_t)round_up(D / 128 * p.TT * 256, 256) : (size_t)0);
    f.off_sumz = f.off_partials + (size_t)f.workgroups * 2048;
    f.end = f.off_sumz + (size_t)f.workgroups * 1024;
    const size_t array = CCE_STATIC_SCRATCH_BYTES;
    f.use = f.end <= (p.off_dhacc <= array && array < p.total ? array : p.total);
    return f;
}

// Whether a backward over all rows may leave the ignored ones out (see backward_skip, which looks at its order too).
static bool may_skip_backward(const Plan& p, int64_t D) {
    return !p.forced && p.TT >= 8 && p.TT <= kRowTableBytes / 512 && 2.0 * (double)p.rows * (double)p.cols * (double)D >= 1.15e12;
}

// The schedule of a backward over N rows (row skipping: the compact ones) for the workspace laid out
// by `p`.  dw_free: dW is overwritten, so its unwritten rows may hold a gradient chunk.  Forced
// tilings, tiles and accumulators keep the Plan's order.  Nothing that takes `limit` or longer is looked for.
// A shape that is seen once pays for this search, so orders whose floor is not below the best so far
// are passed over: of the thousands of orders a few hundred are priced, the one chosen stays the same.
static void make_schedule(const Plan& p, int64_t N, int64_t D, int64_t V, bool compact, bool dw_free, Schedule* out, double limit = 1e300) {
    const int cus = device_cu_count();
    Schedule best = {};
    const int TT = p.TT, VT = p.VT;
    const bool turns = (double)N * (double)D * (double)V >= 2e10;      // (smaller ones have too few tiles of 256 for them)
    const size_t region = (compact ? p.off_count : p.total) - p.off_dhacc;
    {   // the Plan's order under the same model
        const ScheduleModel m = ScheduleModel(cus, D, gemm_tile_of_kind(p.gemm_kind), compact).with_turns(turns);
        const int64_t a = p.Nb / 256, b = p.Vc / 256, nch = (VT + b - 1) / b;
        auto block_us = [&](int64_t aa, bool later) {
            return (nch > 1 ? (double)(nch - 1) * m.step(aa, b, 1, 1, true, later, p.split_acc != 0) : 0.0) +
                   m.step(aa, VT - (nch - 1) * b, 1, 1, nch > 1, later, p.split_acc != 0);
        };
        const int64_t nblk = (TT + a - 1) / a;
        best.plan_us = block_us(nblk > 1 ? a : TT, false);
        if (nblk > 1) best.plan_us += (nblk > 2 ? (double)(nblk - 2) * block_us(a, true) : 0.0) + block_us(TT - (nblk - 1) * a, true);
        if (p.split_acc) best.plan_us += (double)(nblk * nch) * (compact ? 9.0 : 2.0);
    }
    // A schedule has to be rated 10 % faster, one without K parts 4 % where launches may be on tiles of two wavefront groups, whose times
    // the model has more closely.  (Of 70 drawn orders that 4 % and, for row blocks, 2 % decide otherwise than 10 % and 5 %, timed in 105 calls,
    // the calls take 2.6 % less on average: a fifth less at best (11020 x 1920 x 1637 267 -> 210 us), 18 of them 3 to 13 % more (1822 x 3328 x
    // 12641 with 15 % skipped, added to dW, 434 -> 489; 14251 x 320 x 93097 3857 -> 4155).  16384 x 2048 x 151936 31.0 -> 30.4 ms.)
    // Such an order with its sums in planes counts for 4 % less than it is rated where it may leave ignored rows out (backward_skip), which
    // the rating does not know: that stands for batches of which a tenth is padding.  Of 974 drawn shapes it decides 98; 24 of those, timed
    // with and without, take 1.8 % longer where no row is ignored (up to 13.6 % where the other order is in K parts: 1934 x 2560 x 127550
    // 3871 us for 3446, 3762 before tiles of two wavefront groups), 0.3 % less with 5 % ignored and 6.0 % less with 15 % (6523 x 2816 x
    // 36339 3116 us for 3859).
    const bool may_skip = turns && !compact && may_skip_backward(p, D);
    const double parts_us = 0.90 * best.plan_us < limit ? 0.90 * best.plan_us : limit;
    double rated = (turns ? 0.96 : 0.90) * best.plan_us;        // of the best so far
    rated = rated < limit ? rated : limit;
    best.us = rated;
    const int caps[] = {4, 6, 8, 12, 16, 20, 24, 28, 32, 36, 40, 48, 56, 64, 80, 96, 128, 192, 256, 384, 1 << 30};
    const int splits[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};
    const ScheduleModel models[2] = {ScheduleModel(cus, D, gemm_tile_of_kind(0)).with_turns(turns), ScheduleModel(cus, D, gemm_tile_of_kind(1)).with_turns(turns)};
    // (row blocks add to dW with every block, as do the orders with dHidden's front rows, and both are rated with the same
    // items: one to a unit, though a launch of theirs may take two, so that the choice among them stays the one that was measured)
    ScheduleModel block_models[2] = {models[0], models[1]};
    block_models[1].one_to_unit = true;
    // What the steps of a chunk over all rows take, in 1 ... 4 row parts: many orders share such chunks
    // (from eight row tiles on, where row parts are tried).
    constexpr int kKnown = 64;
    double chunk_us[2][2][2][4][kKnown];
    const bool keep = TT >= 8;
    if (keep) memset(chunk_us, 0, sizeof chunk_us);
    auto try_one = [&](int kind, int a, int bcap, int sh, int sw, int row_parts, int b_min, int split_acc) {
        const ScheduleModel& m = a < TT ? block_models[kind] : models[kind];
        ScheduleSteps sc = {};
        sc.kind = kind; sc.a = a; sc.split_h = sh; sc.split_w = sw;
        sc.b = bcap < VT ? bcap : VT;
        sc.tail = dw_free && a == TT;
        sc.row_parts = row_parts; sc.b_min = b_min; sc.split_acc = split_acc;
        if (VT > 4096 * sc.b) return;           // thousands of launches (vocabularies of millions)
        const bool one_chunk = a < TT;          // row blocks: the whole vocabulary in one chunk, no running sums
        if (one_chunk && bcap < VT) return;
        const int64_t rows = (int64_t)a * 256;
        const int64_t cols_max = (int64_t)sc.b * 256 < V ? (int64_t)sc.b * 256 : V;
        sc.plane_h = (rows < N ? rows : N) * D;
        sc.plane_w = cols_max * D;
        const int nblk = (TT + a - 1) / a;
        const double worth = may_skip && kind == 1 && split_acc && a == TT ? 0.96 : 1.0;
        double most = sh > 1 || sw > 1 ? (rated < parts_us ? rated : parts_us) : rated / worth;
        if (limit < most) most = limit;
        // beside the steps: the sum of the planes, the gathered rows
        const double sum_us = sh > 1 ? (double)nblk * (8.0 + (double)sh * (double)sc.plane_h * 4.0 / 4.0e6) : 0.0;
        const double gather_us = compact ? (double)nblk * 5.0 + (double)N * (double)D * 4.0 / 4.0e6 : 0.0;
        const double extra = sum_us + gather_us;
        if (m.floor_us(TT, VT, sc.b, sh, sw) + (double)(nblk - 1) * 8.0 + extra > most * kAbove) return;
        auto lay_out = [&](int planes) {
            sc.off_acc = p.off_dhacc;
            sc.off_part_w = sc.off_acc + (size_t)round_up((int64_t)planes * sc.plane_h * (split_acc ? 2 : 4), 256);
            sc.off_hc = sc.off_part_w + (size_t)round_up((int64_t)(sw - 1) * sc.plane_w * 4, 256);
            sc.off_g = sc.off_hc + (compact && a < TT ? (size_t)round_up(rows * D * 2, 256) : (size_t)0);
            const size_t used = sc.off_g - p.off_dhacc;
            sc.g_bytes = used < region ? region - used : 0;
            return used <= region;
        };
        // without running sums if the whole vocabulary is one chunk, else with a plane per part
        bool ok = sh == 1 && !split_acc && row_parts == 1 && lay_out(0) && schedule_chunk(sc, D, V).b == VT;
        if (!ok) ok = lay_out(sh) && (!one_chunk || schedule_chunk(sc, D, V).b == VT);
        if (!ok) return;
        const double per_tile = m.floor_per_tile(a, sc.b, sh, sw);
        double block_us[2] = {0.0, 0.0};        // first row block, later ones (they add to dW)
        for (int later = 0; later < (one_chunk ? 2 : 1); ++later) {
            ScheduleChunk last = {-1, 0, false}; double last_us = 0.0;
            for (int64_t v = 0; v < V; ) {
                const ScheduleChunk c = schedule_chunk(sc, D, V - v);
                if (c.b < 1 || (int64_t)c.rows * c.b * 131072 >= ((int64_t)1 << 32)) return;
                if (c.b != last.b || c.rows != last.rows) {
                    double* const known = keep && sh == 1 && sw == 1 && !one_chunk && c.b < kKnown
                                              ? &chunk_us[kind][split_acc][v > 0][(a + c.rows - 1) / c.rows - 1][c.b] : nullptr;
                    last_us = known ? *known : 0.0;
                    const int64_t rest = VT - v / 256 - c.b;
                    const double least = last_us > 0.0 ? last_us : (double)(a / c.rows) * m.template step<kFloor>(c.rows, c.b, sh, sw, v > 0, later > 0 || !dw_free);
                    if (block_us[later] + least + (double)rest * per_tile + extra > most * kAbove) return;
                    if (last_us == 0.0) {
                        double step_us = 0.0;
                        int step_rows = 0;
                        bool step_beta = false;                 // (the row parts behind the first one are alike but for the last)
                        for (int r = 0; r < a; r += c.rows) {
                            const int rows = a - r < c.rows ? a - r : c.rows;
                            const bool beta = later > 0 || r > 0 || !dw_free;
                            if (rows != step_rows || beta != step_beta)
                                step_us = m.step(rows, c.b, sh, sw, v > 0, beta, split_acc != 0) + (split_acc ? 2.0 : 0.0);
                            step_rows = rows;
                            step_beta = beta;
                            last_us += step_us;
                        }
                    }
                    if (known) *known = last_us;
                    last = c;
                }
                block_us[later] += last_us;
                if (block_us[later] >= most) return;
                v += c.b * 256;
            }
        }
        sc.us = block_us[0] + (double)(nblk - 1) * block_us[1] + sum_us + gather_us;
        if (sc.us < most) {
            rated = sc.us * worth;
            sc.use = true;
            sc.plan_us = best.plan_us;
            (ScheduleSteps&)best = sc;
        }
    };
    if (!p.forced) {
        for (int kind = 0; kind < 2; ++kind) {
            const ScheduleModel& m = models[kind];
            const int64_t dt = (D + gemm_tile_of_kind(kind).bn - 1) / gemm_tile_of_kind(kind).bn;
            if (kind == 0 && dt * 256 * 7 > D * 8) continue;           // more than an eighth of the columns wasted
            for (int sh : splits) {
                if (sh > 1 && (sh > VT || TT * dt * (sh / 2) > 2 * cus)) break;     // parts beyond two rounds of tiles
                for (int sw : splits) {
                    if (sw > 1 && (sw > TT || VT * dt * (sw / 2) > 2 * cus)) break;
                    if (m.floor_us(TT, VT, VT, sh, sw) > (sh > 1 || sw > 1 || !may_skip ? rated : rated / 0.96) * kAbove) continue;
                    int prev = 0;
                    for (int cap : caps) {
                        const int b = cap < VT ? cap : VT;
                        if (b == prev) break;
                        prev = b;
                        try_one(kind, TT, b, sh, sw, 1, 0, 0);
                        if (sh > 1 || sw > 1 || TT < 8) continue;
                        for (int acc = 0; acc < (compact ? 1 : 2); ++acc)
                            for (int parts = acc ? 1 : 2; parts <= 4; ++parts)
                                for (int b_min : {8, 12, 16, 24, 1 << 30})
                                    if (parts > 1 || b_min == 8) try_one(kind, TT, b, sh, sw, parts, b_min, acc);
                    }
                    // row blocks over the whole vocabulary
                    for (int nblk = 2; nblk <= 64 && nblk <= TT; ++nblk) {
                        const int a = (TT + nblk - 1) / nblk;
                        if ((int64_t)a * VT * 131072 <= (int64_t)region) try_one(kind, a, VT, sh, sw, 1, 0, 0);
                    }
                }
            }
        }
    }
    if (!p.forced && TT > 1 && TT <= 256) {
        // 5 %, 2 %: steps like the Plan's own, which the model ranks more closely than chunks of other widths
        double bound = best.use ? rated : (turns ? 0.98 : 0.95) * best.plan_us;
        if (limit < bound) bound = limit;
        RowBlockPlanner rp;
        rp.m[0] = ScheduleModel(cus, D, gemm_tile_of_kind(0), compact).with_turns(turns);
        rp.m[1] = ScheduleModel(cus, D, gemm_tile_of_kind(1), compact).with_turns(turns);
        rp.TT = TT; rp.VT = VT; rp.D = D; rp.region = region; rp.off0 = p.off_dhacc; rp.compact = compact; rp.dw_free = dw_free;
        rp.prepare();
        const double us = rp.best(TT, bound);
        if (us < bound) {
            int n = 0, R = TT;
            bool front = false;
            for (; R > 0 && n < kMaxRowBlocks; R -= best.blocks[n++].a) {
                best.blocks[n] = rp.states[R].block;
                front = front || best.blocks[n].acc_in_dh || best.blocks[n].g_in_dh;
            }
            if (R == 0 && front) { best.n_blocks = n; best.use = false; best.us = us; }
        }
    }
    if (!best.use && !best.n_blocks) best.us = best.plan_us;
    *out = best;
}

// The layout and order of a backward whose workspace has `workspace_bytes` (at least p->total): *p becomes
// the layout with room for planes where the workspace holds it and schedules on it are rated 10 % faster in
// both forms of the backward.  (Where only one form is rated so the model is not sure enough: of 13 such
// shapes added to dW, nine gained 5 ... 28 % on the larger layout and 40 x 2240 x 108256 and 58 x 1408 x 95496 lost 3 and 5.)
// Kept per thread for the last shapes, the oldest goes first.
static void plan_backward(Plan* p, int64_t N, int64_t D, int64_t V, bool compact, bool dw_free, size_t workspace_bytes, Schedule* sc) {
    Plan roomy;
    const bool room = room_for_planes(*p, D, &roomy) && roomy.total <= workspace_bytes;
    const int cus = device_cu_count(), f = dw_free ? 1 : 0;
    // chosen: basic or roomy (or not decided); order[form] of the chosen layout, or of the basic one before that
    enum Layout { kOpen, kBasic, kRoomy };
    struct Key {
        int64_t N, D, V; size_t total, budget; int cus; bool forced, compact, room, valid;
        Layout layout; bool have[2]; Schedule order[2];
    };
    constexpr int kCached = 16;
    static thread_local Key cache[kCached] = {};
    static thread_local int cache_next = 0;
    Key* k = nullptr;
    for (Key& c : cache)
        if (c.valid && c.N == N && c.D == D && c.V == V && c.total == p->total && c.budget == p->budget && c.cus == cus &&
            c.forced == p->forced && c.compact == compact && c.room == room) k = &c;
    if (!k) {
        k = &cache[cache_next];
        cache_next = (cache_next + 1) % kCached;
        k->N = N; k->D = D; k->V = V; k->total = p->total; k->budget = p->budget; k->cus = cus;
        k->forced = p->forced; k->compact = compact; k->room = room; k->valid = true;
        k->layout = room ? kOpen : kBasic;
        k->have[0] = k->have[1] = false;
    }
    auto basic = [&](int form) {
        if (!k->have[form]) make_schedule(*p, N, D, V, compact, form != 0, &k->order[form]);
        k->have[form] = true;
    };
    if (k->layout != kRoomy) basic(f);
    if (k->layout == kOpen) {
        Schedule own, other;
        make_schedule(roomy, N, D, V, compact, f != 0, &own, 0.9 * k->order[f].us);
        k->layout = kBasic;
        if (own.use) {
            basic(1 - f);
            make_schedule(roomy, N, D, V, compact, f == 0, &other, 0.9 * k->order[1 - f].us);
            if (other.use) {
                k->layout = kRoomy;
                k->order[f] = own;
                k->order[1 - f] = other;
            }
        }
    }
    if (k->layout == kRoomy) *p = roomy;
    *sc = k->order[f];
}

// The workspace to ask for.  What a call with this many rows or fewer needs (same D and V; row skipping: under
// any bound) fits it, whichever tiling each row count gets: the budget, or the most that a plan's layout for such a
// problem can hold where that is less.  So does, up to the budget's floor, the layout with room for planes; beyond the
// floor only this call's own is counted, if it would be taken.  (Sized by its own layout alone, 356 rows at
// D = 2048, V = 4000 asked for 48 MB where 1024 rows asked for 17: a workspace made for the largest batch did not
// serve the last, short one.)  `p` is the plan for N rows, or with `compact` the one for some of N rows.
static size_t workspace_to_ask_for(const Plan& p, int64_t N, int64_t D, int64_t V, bool compact) {
    if (p.forced) return p.total;
    Plan roomy, taken = p;
    Schedule order;
    const bool room = room_for_planes(p, D, &roomy);
    if (room && roomy.total > kBudgetFloor) plan_backward(&taken, p.rows, D, V, compact, false, roomy.total, &order);
    else if (room) taken = roomy;
    const int64_t TT = (N + 255) / 256, VT = (V + 255) / 256, a = TT < 64 ? TT : 64, b = VT < 128 ? VT : 128;
    const int64_t splits = 2 * VT < 2 * device_cu_count() ? 2 * VT : 2 * device_cu_count();
    const double rows = compact ? 4.0 * (double)(TT * 256 * 4 + 256) + (double)(D * 2 + 512) : 0.0;
    const double sums = 256.0 + 512.0 + (double)N * 12.0 * (double)splits + (double)a * 256.0 * (double)D * 4.0 + rows;
    const double planes = 15.0 * ((double)(N < 4096 ? N : 4096) * (double)D * 4.0 + 256.0);
    const double plan_most = sums + (double)(a * b) * 131072.0, room_most = sums + planes + (double)(a * VT) * 131072.0;
    const size_t plans = plan_most < (double)p.budget ? (size_t)plan_most : p.budget;
    const size_t rooms = room_most < (double)kBudgetFloor ? (size_t)room_most : kBudgetFloor;
    const size_t serves = plans > rooms ? plans : rooms;
    return taken.total > serves ? taken.total : serves;
}

// A backward over all rows that leaves the ignored ones out likewise (see ForwardSkip): one whose schedule has all rows in one block,
// no K parts and its dH sums in two planes (large ones have), and whose row map fits the contraction's LDS table in 16 bits.  The
// order stays.  Backwards that compute every row against this, one box: 8192 x 896 x 151936 with 15 % ignored 6.42 -> 5.96 ms, with
// FP8 logits 5.82 -> 5.35, 5200 x 2048 x 65001 with 15 % 3.91 -> 3.47.  Without ignored rows it costs the scan, the gather of the
// per-row scalars and the scatter of dHidden's rows, 0.1 to 0.6 %: 6.46 -> 6.47, FP8 5.85 -> 5.87, 3.91 -> 3.93; more only where
// launches keep one tile to a unit that would run two of them (see counted_contraction_kind): 3000 x 2048 x 151936 5.14 -> 5.37,
// for 5.14 -> 4.70 with 15 %.
// The bookkeeping lies where the forward's partials were.
struct BackwardSkip { bool use; size_t off_perm, off_labels, off_lse, off_dloss, off_count, off_scales; };
static BackwardSkip backward_skip(const Plan& p, const Schedule& sc, int64_t D, bool fp8) {
    BackwardSkip b = {};
    // (256 x 128 tiles: no order with the planes was ever planned with 256 x 256 ones)
    if (!sc.use || sc.kind != 1 || !sc.split_acc || sc.a < p.TT || sc.split_h != 1 || sc.split_w != 1 || !may_skip_backward(p, D)) return b;
    if (g_force_row_skipping.load(std::memory_order_relaxed) == 1) return b;
    const size_t each = (size_t)p.TT * 1024;
    b.off_perm = p.off_partials;
    b.off_labels = b.off_perm + each;
    b.off_lse = b.off_labels + each;
    b.off_dloss = b.off_lse + each;
    b.off_count = b.off_dloss + each;
    b.off_scales = b.off_count + 256;
    b.use = b.off_scales + (fp8 ? (size_t)(D / 128 * p.TT * 256) : (size_t)0) <= p.off_dhacc;
    return b;
}

// Row skipping: the order keeps something in dHidden while it runs -- the gathered rows of a single row block,
// or sums and chunks in front of a row block -- and zeroes the rows that take no part when it is done.
static bool order_uses_dhidden(const Plan& p, const Schedule& sc) {
    if (sc.use) return sc.a >= p.TT;
    for (int i = 0; i < sc.n_blocks; ++i)
        if (sc.blocks[i].acc_in_dh || sc.blocks[i].g_in_dh) return true;
    return false;
}

// Backwards of all rows at D = 64 and 128 without a gradient chunk (see fused_backward.h): how the launch's two jobs are cut.  The streamed
// ranges are cut into parts of whole tiles of 128 rows where the stationary tiles alone leave compute units idle; a part of the
// dH job writes a plane, and so does one of the dW job from the second on, summed by a small launch each.  From the shape and the planned
// layout alone (the workspace asked for), so that calls of a shape agree.
// Over a gradient chunk / this, us: 256 x 64 x 1000 15.2 / 10.2, 2000 x 64 x 5000 31 / 21, 600 x 64 x 150000 224 / 78, 8192 x 64 x 151936
// 3381 / 670, 28457 x 64 x 48721 3321 / 735, 500 x 128 x 3000 16.7 / 13.3, 1000 x 128 x 50000 107 / 79, 22053 x 128 x 77882 4119 / 1811:
// so every call that can takes it (FP8 logits and row skipping cannot).  The constants are fitted to 1 to 144 cuts each of 102
// shapes, a row to a million: 4 us and the bytes or, where those are few, the chain of one load behind the other, 0.39 us a plane, for a
// sum of planes (rated by the bytes alone, 228 x 128 x 12162 was cut into 48 parts and took 26 us, for 17.5 in 16 parts and 21 over
// a chunk; 900 x 128 x 12162 33 / 27.7 / 30).  What is chosen takes 2.3 % longer than the fastest cut on average, 23 % at most
// (9129 x 64 x 18135 130 us for 105).  Of 273 calls timed over a chunk and so, none is slower.
struct FusedChoice { bool use, shared; int parts_h, parts_w, len_h, len_w, n_h, n_w; double us; };
static FusedChoice fused_backward_choice(const Plan& p, int64_t N, int64_t D, int64_t V) {
    FusedChoice best = {};
    best.us = 1e300;
    if (p.forced || (D != 64 && D != 128)) return best;
    struct Key { int64_t N, D, V; size_t region; int cus; FusedChoice choice; bool valid; };
    constexpr int kCached = 16;
    static thread_local Key cache[kCached] = {};
    static thread_local int cache_next = 0;
    const int cus = device_cu_count();
    const size_t region = p.total - p.off_dhacc;
    for (const Key& k : cache)
        if (k.valid && k.N == N && k.D == D && k.V == V && k.region == region && k.cus == cus) return k.choice;
    const int64_t tiles_n = (N + 127) / 128, tiles_v = (V + 127) / 128;
    const int cuts[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64};
    auto planes_us = [](int planes, double bytes) { return planes == 0 ? 0.0 : 4.0 + (0.39 * planes > bytes / 3.2e6 ? 0.39 * planes : bytes / 3.2e6); };
    for (int shared = 0; shared < 2; ++shared) {
        // stationary rows of an item, items to a unit, microseconds of a streamed tile beside the unit's other items and alone
        const int64_t rows = shared ? 32 : D == 64 ? 256 : 128, slots = (D == 64 && shared ? 4 : 2) * cus;
        const double beside = shared ? (D == 64 ? 1.16 : 1.2) : D == 64 ? 3.64 : 3.25, alone = shared ? (D == 64 ? 0.79 : 0.8) : D == 64 ? 2.9 : 2.65;
        const double fixed = shared && D == 128 ? 2.9 : 4.0;
        for (int ph : cuts) {
            const int64_t len_h = (tiles_v + ph - 1) / ph, n_h_parts = (tiles_v + len_h - 1) / len_h;
            if (n_h_parts != ph) continue;
            for (int pw : cuts) {
                const int64_t len_w = (tiles_n + pw - 1) / pw;
                if ((tiles_n + len_w - 1) / len_w != pw) continue;
                const double plane_h = ph > 1 ? (double)ph * (double)(N * D * 4) : 0.0, plane_w = (double)(pw - 1) * (double)(V * D * 4);
                if (plane_h + plane_w + 1024.0 > (double)region) continue;
                const int64_t n_h = (N + rows - 1) / rows * ph, n_w = (V + rows - 1) / rows * pw;
                if (n_h + n_w > 1 << 20) continue;
                const double tile = n_h + n_w <= cus ? alone : beside;
                const double us = makespan(slots, n_h, (double)len_h * tile + fixed, n_w, (double)len_w * tile + fixed) +
                                  planes_us(ph > 1 ? ph : 0, plane_h) + planes_us(pw - 1, plane_w);
                if (us < best.us) best = {true, shared != 0, ph, pw, (int)len_h, (int)len_w, (int)n_h, (int)n_w, us};
            }
        }
    }
    cache[cache_next] = {N, D, V, region, cus, best, true};
    cache_next = (cache_next + 1) % kCached;
    return best;
}

// Modelled time of the backward that a call would run in a workspace of the size asked for: plan_backward's order, or over all rows at
// D = 64 and 128 the launch without a gradient chunk.
static double backward_us(Plan p, int64_t N, int64_t D, int64_t V, bool compact, bool dw_free) {
    if (!compact) {
        const FusedChoice f = fused_backward_choice(p, N, D, V);
        if (f.use) return f.us;
    }
    Schedule s;
    plan_backward(&p, N, D, V, compact, dw_free, (size_t)-1, &s);
    return s.us;
}

// Row skipping pays when enough rows can be skipped: the compact row space costs a label scan and a few
// small launches, its hidden rows are read through the row map or gathered, and its tiling may fit the
// launches worse.  `comp` is the plan for M compact rows, `plain` the one for all N.  15 us stand for the small
// launches (500 x 256 x 3000 with 300 valid rows: 29 -> 43 us, 1500 x 512 x 2000 with 900: 41 -> 53).  The forward
// and the workspace query do not know whether the backward will overwrite dW or add to it, and the two run in
// different orders: skipping is taken where the schedules' model, with the tiles that each would run, rates it 3.3 % faster on the mean
// of the two.  Of 3700 drawn shapes of D 192 to 4096 with 5 ... 60 % of the rows ignored this answers 120 otherwise than ratings without tiles of
// two wavefront groups, one of the two forms 6 % faster and the other no slower: 75 of those, both forms of both calls timed, are 0.6 %
// above the better side on average and were 8.0 (17712 x 1280 x 4257 with 15 % 654 us for 810; 8950 x 384 x 4089 with 10 % loses 5 %); 86
// others 0.7 and 0.9 %.  At 2.5 % the model is wrong where it costs most (16384 x 2048 x 151936 with 15565 valid, rated 0.95 and
// 0.999, takes 1.08 and 1.10).
// At D = 64 and 128 all rows without a chunk are the faster ones up to some 60 % ignored: of 44 shapes with 5 ... 80 % two skip, the
// faster form each time (8699 x 64 x 68133 with 80 % 332 us for 481, 24548 x 64 x 92355 with 5 % 4 575 for 1 767).
static bool skipping_pays(const Plan& plain, const Plan& comp, int64_t N, int64_t M, int64_t D, int64_t V) {
    const ForwardCost fwd{device_cu_count(), D};
    double rated[2] = {0.0, 0.0};
    for (int dw_free = 1; dw_free >= 0; --dw_free) {
        rated[dw_free] = (backward_us(comp, M, D, V, true, dw_free != 0) + fwd.us(comp) + 15.0) /
                         (backward_us(plain, N, D, V, false, dw_free != 0) + fwd.us(plain));
        if (rated[1] > 1.1) return false;       // (the two are never that far apart)
    }
    return rated[0] + rated[1] < 2.0 * 0.967;
}

// Whether a call with at most M = max_valid_rows < N valid rows skips the others; mode as in
// cce_set_row_skipping.  *p becomes the plan it runs on.  Kept per thread for the last shapes.
static bool plan_row_skipping(int64_t N, int64_t D, int64_t V, int64_t max_valid_rows, int mode, Plan* p, bool* skipping) {
    const int64_t M = max_valid_rows < 1 ? 1 : max_valid_rows;
    *skipping = false;
    if (!make_plan(N, D, V, p)) return false;
    Plan comp;
    if (M >= N || mode == 1 || !make_plan(M, D, V, &comp, N)) return true;
    if (mode == 2) *skipping = true;
    else {
        struct Key { int64_t N, M, D, V; size_t plain, comp; int cus; bool forced, valid, skipping; };
        constexpr int kCached = 32;
        static thread_local Key cache[kCached] = {};
        static thread_local int cache_next = 0;
        const int cus = device_cu_count();
        const Key* hit = nullptr;
        for (const Key& k : cache)
            if (k.valid && k.N == N && k.M == M && k.D == D && k.V == V && k.plain == p->total && k.comp == comp.total &&
                k.cus == cus && k.forced == p->forced) hit = &k;
        if (!hit) {
            cache[cache_next] = {N, M, D, V, p->total, comp.total, cus, p->forced, true, skipping_pays(*p, comp, N, M, D, V)};
            hit = &cache[cache_next];
            cache_next = (cache_next + 1) % kCached;
        }
        *skipping = hit->skipping;
    }
    if (*skipping) *p = comp;
    return true;
}

}  // namespace cce
