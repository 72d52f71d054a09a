// Host-only check of the backward's schedules (csrc/plan.h), built and run by tests/test_schedule_host.py
// with AddressSanitizer and UndefinedBehaviorSanitizer on the host side: over seeded shapes every step
// of a schedule covers the vocabulary once, keeps its gradient chunk inside the workspace or behind the
// rows of dW that are written by then, and gives its K parts whole, non-empty ranges.  The time model's
// makespan is compared with a hand-out of the jobs.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <functional>
#include <queue>
#include <vector>

namespace cce { thread_local int g_last_hip_error = 0; }
static long priced = 0;
#define CCE_PLAN_PRICED() ((void)++priced)
#include "../../paper_2601_02609_amd/csrc/plan.h"
#include "../../paper_2601_02609_amd/csrc/wg_map.h"

using namespace cce;

static uint64_t state = 0x2545F4914F6CDD1Dull;
static int64_t pick(int64_t lo, int64_t hi) {
    state ^= state << 13; state ^= state >> 7; state ^= state << 17;
    return lo + (int64_t)(state % (uint64_t)(hi - lo + 1));
}
static int failures = 0, used = 0, in_tails = 0, split_hs = 0, split_ws = 0, blocks = 0, parts = 0, split_accs = 0, fronts = 0, fwd_skips = 0, bwd_skips = 0;
#define CHECK(cond) do { if (!(cond)) { ++failures; fprintf(stderr, "FAIL %d: %s | N=%lld D=%lld V=%lld B=%lld free=%d\n", __LINE__, #cond, \
    (long long)N, (long long)D, (long long)V, (long long)B, (int)dw_free); } } while (0)

// A backward that leaves ignored rows out: its bookkeeping lies in the partials' area, its row map fits the table.
static void check_backward_skip(const Plan& p, const Schedule& s, int64_t N, int64_t D, int64_t V, bool dw_free) {
    const int64_t B = 0;
    for (int fp8 = 0; fp8 < (D % 128 ? 1 : 2); ++fp8) {
        const BackwardSkip b = backward_skip(p, s, D, fp8 != 0);
        if (!b.use) continue;
        ++bwd_skips;
        const size_t each = (size_t)p.TT * 256 * 4;
        CHECK(s.use && s.kind == 1 && s.a == p.TT && s.split_acc && s.split_h == 1 && s.split_w == 1);
        CHECK(p.TT * 256 * 2 <= kRowTableBytes && N <= 65536);
        CHECK(b.off_perm >= p.off_partials && b.off_labels - b.off_perm >= each && b.off_lse - b.off_labels >= each);
        CHECK(b.off_dloss - b.off_lse >= each && b.off_count - b.off_dloss >= each && b.off_scales - b.off_count >= 8);
        CHECK(b.off_scales + (fp8 ? (size_t)(D / 128 * p.TT * 256) : (size_t)0) <= p.off_dhacc && p.off_dhacc <= s.off_acc);
        CHECK(((b.off_perm | b.off_labels | b.off_lse | b.off_dloss | b.off_count | b.off_scales) & 255) == 0);
    }
}

static bool check_layout(const Plan& p, int64_t N, int64_t D, int64_t V, int64_t B, bool dw_free) {
    Schedule s;
    make_schedule(p, N, D, V, B != 0, dw_free, &s);
    if (s.n_blocks) {
        ++fronts;
        CHECK(!s.use && s.us < s.plan_us);
        const size_t end = B ? p.off_count : p.total;
        int R = p.TT;
        for (int i = 0; i < s.n_blocks; ++i) {
            const RowBlock& k = s.blocks[i];
            CHECK(k.a >= 1 && k.r0 == R - k.a && k.b >= 1 && k.b <= p.VT && (!B || k.a <= kCompactMaxRowTiles));
            R -= k.a;
            // dHidden's rows in front of the block are free; sums and chunk never share an area
            const size_t front = (size_t)k.r0 * 256 * (size_t)D * 2;
            const size_t acc = (size_t)k.a * 256 * (size_t)D * (k.split_acc ? 2 : 4), g = (size_t)k.a * (size_t)k.b * 131072;
            CHECK(g < ((size_t)1 << 32) && !(k.acc_in_dh && k.g_in_dh));
            CHECK(((k.off_acc | k.off_g) & 255) == 0);
            if (k.acc_in_dh) CHECK(k.off_acc + acc <= front); else CHECK(k.off_acc >= p.off_dhacc && k.off_acc + acc <= end);
            if (k.g_in_dh) CHECK(k.off_g + g <= front); else CHECK(k.off_g >= p.off_dhacc && k.off_g + g <= end);
            if (!k.acc_in_dh && !k.g_in_dh) CHECK(k.off_g >= k.off_acc + acc);
        }
        CHECK(R == 0);
    }
    if (B) CHECK(order_uses_dhidden(p, s) == (s.use ? (int64_t)s.a * 256 >= N : s.n_blocks > 0));
    if (!B) check_backward_skip(p, s, N, D, V, dw_free);
    if (!s.use) return false;
    ++used;
    const int64_t block = (int64_t)s.a * 256;
    const size_t ws_end = B ? p.off_count : p.total;
    CHECK(s.us < s.plan_us);
    CHECK(s.a >= 1 && s.a <= p.TT && s.b >= 1 && s.b <= p.VT);
    CHECK(s.off_acc >= p.off_dhacc && s.off_part_w >= s.off_acc && s.off_hc >= s.off_part_w && s.off_g >= s.off_hc);
    CHECK(s.off_g + s.g_bytes <= ws_end);
    CHECK(((s.off_acc | s.off_part_w | s.off_hc | s.off_g) & 255) == 0);
    if (s.a < p.TT) { ++blocks; CHECK(!s.tail); if (B) CHECK(s.off_g - s.off_hc >= (size_t)(block * D * 2)); }
    CHECK(s.row_parts >= 1 && (!s.split_acc || (s.split_h == 1 && !B)));
    for (int64_t r0 = 0; r0 < N; r0 += block) {
        const int64_t rows = N - r0 < block ? N - r0 : block;
        int steps = 0, planes = 0;
        for (int64_t v0 = 0; v0 < V; ) {
            const ScheduleChunk c = schedule_chunk(s, D, V - v0);
            const int64_t t = c.b;
            CHECK(t >= 1 && c.rows >= 1 && c.rows <= s.a);
            if (t < 1 || c.rows < 1) return true;
            const int64_t cols = V - v0 < t * 256 ? V - v0 : t * 256;
            const int64_t kh = (t + s.split_h - 1) / s.split_h, nh = (t + kh - 1) / kh;
            for (int64_t s0 = 0; s0 < rows; s0 += (int64_t)c.rows * 256, ++steps) {
                const int64_t srows = rows - s0 < (int64_t)c.rows * 256 ? rows - s0 : (int64_t)c.rows * 256, row_tiles = (srows + 255) / 256;
                const int64_t g = row_tiles * 256 * t * 512;
                CHECK(g < ((int64_t)1 << 32));
                if (c.in_tail) {
                    ++in_tails;
                    CHECK(dw_free && s.a == p.TT);
                    const int64_t at = (V * D * 4 - g) & ~(int64_t)255;
                    CHECK(at >= (v0 + cols) * D * 4 && at + g <= V * D * 4);
                } else {
                    CHECK((size_t)g <= s.g_bytes);
                }
                const int64_t kw = (row_tiles + s.split_w - 1) / s.split_w, nw = (row_tiles + kw - 1) / kw;
                CHECK(nh >= 1 && nh <= s.split_h && (nh - 1) * kh < t && nw >= 1 && nw <= s.split_w && (nw - 1) * kw < row_tiles);
                // an operand's last part starts inside its valid extent
                CHECK((nh - 1) * kh * 256 < cols && (nw - 1) * kw * 256 < srows);
                if (nw > 1) { ++split_ws; CHECK(s.off_hc - s.off_part_w >= (size_t)((nw - 1) * s.plane_w * 4) && s.plane_w >= cols * D); }
                if (c.rows < s.a) ++parts;
            }
            planes = planes > nh ? planes : (int)nh;
            v0 += cols;
        }
        // one step and one part need no running sum: the result is final at once
        if (steps > 1 || s.split_h > 1) CHECK(s.off_part_w - s.off_acc >= (size_t)(planes * s.plane_h * (s.split_acc ? 2 : 4)) && s.plane_h >= rows * D);
        if (s.split_h > 1) ++split_hs;
        if (s.split_acc) ++split_accs;
    }
    return true;
}

// A forward that leaves ignored rows out: its layout fits every workspace that the shape's calls accept, the static array
// included where cce_forward_static takes the shape, and holds the partials of any number of rows.
static void check_forward_skip(const Plan& p, int64_t N, int64_t D, int64_t V) {
    const int64_t B = 0; const bool dw_free = false;
    for (int fp8 = 0; fp8 < (D % 128 ? 1 : 2); ++fp8) {
        const ForwardSkip f = forward_skip(p, D, fp8 != 0);
        if (!f.use) continue;
        ++fwd_skips;
        CHECK(f.end <= p.total && (p.off_dhacc > CCE_STATIC_SCRATCH_BYTES || f.end <= CCE_STATIC_SCRATCH_BYTES));
        CHECK(f.off_perm >= p.off_partials && f.off_found - f.off_perm >= (size_t)p.TT * 256 * 4 && f.off_scales - f.off_found >= 16);
        CHECK(f.off_partials - f.off_scales >= (fp8 ? (size_t)(D / 128 * p.TT * 256) : (size_t)0));
        CHECK(((f.off_perm | f.off_found | f.off_scales | f.off_partials | f.off_sumz) & 255) == 0);
        CHECK(p.S <= f.s_max && f.s_max <= p.VT && p.TT * p.S <= f.workgroups);
        for (int tiles = 1; tiles <= p.TT; ++tiles) {
            int s = f.workgroups / tiles;                        // as many splits as the label scan may take
            s = s < f.s_max ? s : f.s_max;
            CHECK(s >= 1 && tiles <= f.workgroups);
            const size_t pairs = (size_t)(tiles * 256 < N ? tiles * 256 : N) * s;
            CHECK(f.off_sumz - f.off_partials >= pairs * 8 && f.end - f.off_sumz >= pairs * 4);
        }
    }
}

// The plan's own layout, and the one with room for planes that a call takes where its workspace holds it.
static bool check(int64_t N, int64_t D, int64_t V, int64_t B, bool dw_free) {
    Plan p, roomy;
    if (!make_plan(N, D, V, &p, B)) return false;
    bool used = check_layout(p, N, D, V, B, dw_free);
    if (!B) check_forward_skip(p, N, D, V);
    const size_t ask = workspace_to_ask_for(p, B ? B : N, D, V, B != 0);
    CHECK(p.total <= ask);
    for (int i = 0; i < 3; ++i) {            // any smaller call's own layout fits, and up to the floor its room for planes
        const int64_t b = B ? pick(1, B) : 0, n = pick(1, B ? b : N);
        Plan less, less_roomy;
        CHECK(make_plan(n, D, V, &less, b) && less.total <= ask);
        if (room_for_planes(less, D, &less_roomy)) CHECK(less_roomy.total <= ask || less_roomy.total > kBudgetFloor);
    }
    if (room_for_planes(p, D, &roomy)) {
        CHECK(roomy.total <= ask || roomy.total > kBudgetFloor);
        CHECK(roomy.total > p.total && roomy.off_dhacc == p.off_dhacc);
        CHECK((roomy.off_g & 255) == 0 && (roomy.off_perm & 255) == 0 && (!B || roomy.off_count - p.off_count == roomy.total - p.total));
        used = check_layout(roomy, N, D, V, B, dw_free) || used;
    }
    return used;
}

// two_class_makespan against the hand-out itself: every job goes to the unit that is free first.
// (Whole lengths: sums and quotients are exact.)
static void check_makespan() {
    for (int it = 0; it < 4000; ++it) {
        const int cus = it % 3 ? 256 : (int)pick(1, 300);
        const int64_t n1 = it % 2 ? pick(1, 40) : pick(1, 1200), n2 = it % 4 < 2 ? pick(0, 20) : pick(0, 1200);
        const int64_t c2 = pick(1, 60), c1 = c2 + (it % 5 ? pick(0, 60) : pick(0, 3000));
        std::priority_queue<int64_t, std::vector<int64_t>, std::greater<int64_t>> free_at;
        for (int u = 0; u < cus; ++u) free_at.push(0);
        int64_t end = 0;
        for (int64_t i = 0; i < n1 + n2; ++i) {
            const int64_t t = free_at.top() + (i < n1 ? c1 : c2);
            free_at.pop();
            free_at.push(t);
            end = end > t ? end : t;
        }
        const double got = two_class_makespan(cus, n1, (double)c1, n2, (double)c2);
        if (got != (double)end) {
            ++failures;
            fprintf(stderr, "FAIL makespan of %lld x %lld, %lld x %lld on %d: %.0f instead of %lld\n", (long long)n1, (long long)c1,
                    (long long)n2, (long long)c2, cus, got, (long long)end);
        }
    }
}

// The bounds that pass orders over against the priced time of orders: steps over all rows, or over a part of them, in chunks of any width
// up to the widest.
static void check_floors() {
    int bad = 0;
    for (int it = 0; it < 40000; ++it) {
        const int64_t D = 64 * (it % 2 ? pick(1, 16) : pick(1, 64)), a = it % 3 ? pick(1, 40) : pick(1, 128), vt = pick(1, 300), widest = pick(1, it % 4 ? 64 : 300);
        const int kind = (int)pick(0, 1), sh = (int)(it % 5 ? 1 : pick(1, 8)), sw = (int)(it % 7 ? 1 : pick(1, 8));
        const bool turns = pick(0, 3) > 0, mapped = pick(0, 7) == 0, split = sh == 1 && pick(0, 1), dw_free = pick(0, 1);
        const int parts = (int)(it % 11 ? 1 : pick(1, 4));
        const ScheduleModel m = ScheduleModel(256, D, gemm_tile_of_kind(kind), mapped).with_turns(turns);
        const int64_t rows = (a + parts - 1) / parts;
        double us = 0.0;
        for (int64_t v = 0; v < vt; ) {
            int64_t b = pick(1, widest);
            b = it % 2 ? widest : b;
            b = b < vt - v ? b : vt - v;
            for (int64_t r = 0; r < a; r += rows) {
                const int64_t t = a - r < rows ? a - r : rows;
                const double s = m.step(t, b, sh, sw, v > 0, r > 0 || !dw_free, split);
                if (m.step<kFloor>(t, b, sh, sw, v > 0, r > 0 || !dw_free, split) > s * kAbove) bad |= 1;
                if (m.step<kTightFloor>(t, b, sh, sw, v > 0, r > 0 || !dw_free, split) > s * kAbove) bad |= 2;
                us += s;
            }
            v += b;
        }
        const int64_t most = widest < vt ? widest : vt;
        if (m.floor_us(a, vt, most, sh, sw) > us * kAbove) bad |= 4;
        if ((double)vt * m.floor_per_tile(a, most, sh, sw) > us * kAbove) bad |= 8;
        if (bad) {
            ++failures;
            fprintf(stderr, "FAIL floor %d: D=%lld %lld x %lld in %lld, parts %d %d, row parts %d, kind %d turns %d mapped %d split %d: %.1f, %.1f per tile, %.1f\n", bad, (long long)D,
                    (long long)a, (long long)vt, (long long)widest, sh, sw, parts, kind, (int)turns, (int)mapped, (int)split, m.floor_us(a, vt, most, sh, sw),
                    (double)vt * m.floor_per_tile(a, most, sh, sw), us);
            if (failures > 12) return;
            bad = 0;
        }
    }
}

// What planning a backward for a shape seen once may cost: callers whose row count changes with every
// batch pay it in front of their launches.  Counted in makespans searched for, which is what pricing an order
// costs (the bounds that pass orders over are a few products each); limits a quarter above today's.
static void check_planning_cost() {
    const struct { int64_t N, D, V; long limit; } shapes[] = {
        {256, 64, 1000, 10}, {900, 256, 12000, 620}, {2000, 512, 5000, 40}, {16000, 64, 2000, 220}, {30000, 64, 2000, 450},
        {509, 896, 151936, 600}, {8192, 896, 151936, 3000}, {3001, 1024, 50257, 400}, {12000, 4096, 32000, 1100},
        {30000, 3584, 151936, 4400}};
    for (auto& s : shapes)
        for (int dw_free = 0; dw_free < 2; ++dw_free) {
            Plan p; Schedule sc;
            const long before = priced;
            const int64_t N = s.N + dw_free;                     // a shape of its own: nothing is kept from the other form
            if (!make_plan(N, s.D, s.V, &p)) { ++failures; return; }
            plan_backward(&p, N, s.D, s.V, false, dw_free != 0, workspace_to_ask_for(p, N, s.D, s.V, false), &sc);
            printf("planning %lld x %lld x %lld, dW %s: %ld makespans\n", (long long)N, (long long)s.D, (long long)s.V,
                   dw_free ? "overwritten" : "added to", priced - before);
            if (priced - before > s.limit) { ++failures; fprintf(stderr, "FAIL planning: %ld makespans, limit %ld\n", priced - before, s.limit); }
        }
}

// The gradient tiles of a call, launch by launch: 384 x 256 ones, 256 x 256 ones, and of the taller ones those whose last
// tile crosses the end of the vocabulary or lies wholly behind it.
struct TileCounts {
    int tall = 0, square = 0, crossing = 0, behind = 0;
    void launch(int64_t row_tiles, int64_t v0, int64_t v_tiles, int64_t D, int64_t V) {
        if (use_small_tiles(row_tiles, v_tiles)) return;
        if (!tall_grad_tiles((int)row_tiles, (int)v_tiles, (int)D, device_cu_count())) { ++square; return; }
        const int64_t last = v0 + ((v_tiles * 256 + 383) / 384 - 1) * 384;       // first column of the last tile
        ++tall;
        crossing += last < V && last + 384 > V;
        behind += last >= V;
    }
};

// What a call runs, as one line of "word=number": rows N of which B = 0 (all) or M take part.
static void print_form(int64_t N, int64_t D, int64_t V, int64_t M, bool dw_free) {
    Plan p; Schedule s;
    const bool compact = M > 0;
    const int64_t rows = compact ? M : N;
    if (!make_plan(rows, D, V, &p, compact ? N : 0)) { printf("refused\n"); return; }
    Plan asked = p;
    if (compact && M < N) { bool skip; plan_row_skipping(N, D, V, M, 2, &asked, &skip); }
    plan_backward(&p, rows, D, V, compact, dw_free, workspace_to_ask_for(asked, N, D, V, compact), &s);
    int chunks = 0, in_dw = 0, part_steps = 0, least_h = 1 << 30, most_h = 0, most_w = 0, sums_dh = 0, chunks_dh = 0, small = 0, steps = 0, same_tiles = 0, paired = 0, most_rows = 0;
    const int64_t dt = (D + gemm_tile_of_kind(s.kind).bn - 1) / gemm_tile_of_kind(s.kind).bn;
    TileCounts tiles;
    if (s.use) {
        for (int64_t v = 0; v < V; ++chunks) {
            const ScheduleChunk c = schedule_chunk(s, D, V - v);
            const int kh = (int)((c.b + s.split_h - 1) / s.split_h), nh = (int)((c.b + kh - 1) / kh);
            const int kw = (c.rows + s.split_w - 1) / s.split_w, nw = (c.rows + kw - 1) / kw;
            least_h = nh < least_h ? nh : least_h; most_h = nh > most_h ? nh : most_h; most_w = nw > most_w ? nw : most_w;
            in_dw += c.in_tail ? 1 : 0;
            part_steps += c.rows < s.a ? 1 : 0;
            for (int64_t r = 0; r < p.TT; r += c.rows) {            // (steps of the first block's sizes)
                const int64_t t = p.TT - r < c.rows ? p.TT - r : c.rows, tw = (t + s.split_w - 1) / s.split_w;
                if (r < s.a) tiles.launch(t, v, c.b, D, V);
                const int plain = contraction_kind(s.kind, D, t * nh * dt, kh * 4, v > 0, s.split_acc != 0, c.b * ((t + tw - 1) / tw) * dt, tw * 4,
                                                   r > 0 || !dw_free, false, Knobs::read());
                const int kind = counted_contraction_kind(s.kind, D, t, c.b, dt, v > 0, r > 0 || !dw_free, Knobs::read());
                small += kind == 2;
                same_tiles += kind == plain;
                ++steps;
                if (kind != 3) continue;
                ++paired;
                most_rows = (int)t > most_rows ? (int)t : most_rows;
            }
            v += c.b * 256;
        }
    } else {
        least_h = most_h = most_w = 1;
        for (int i = 0; i < s.n_blocks; ++i) { sums_dh += s.blocks[i].acc_in_dh; chunks_dh += s.blocks[i].g_in_dh; }
        const int n = s.n_blocks ? s.n_blocks : 1;
        for (int i = 0; i < n; ++i) {
            const int64_t a = s.n_blocks ? s.blocks[i].a : p.Nb / 256 < p.TT ? p.Nb / 256 : p.TT, b = s.n_blocks ? s.blocks[i].b : p.Vc / 256;
            for (int64_t v = 0; v < p.VT; v += b) tiles.launch(a, v * 256, p.VT - v < b ? p.VT - v : b, D, V);
        }
    }
    // All rows of bf16 calls at D = 64 and 128 run without a gradient chunk: nothing of the order above.
    const bool fused = !compact && fused_backward_choice(p, N, D, V).use;
    if (fused) {
        s = Schedule{};
        chunks = in_dw = part_steps = least_h = most_h = most_w = sums_dh = chunks_dh = small = steps = same_tiles = paired = most_rows = 0;
        tiles = TileCounts();
    }
    const ForwardTile fwd = forward_tile(p, D);
    const int64_t unit = fwd == kForwardTall ? 192 : 128, units = (V + unit - 1) / unit;
    int halves = 0;                          // splits that end in a half tile
    for (int64_t i = 0; (fwd == kForwardTall || fwd == kForwardSquare) && i < p.S; ++i) halves += (int)(((i + 1) * units / p.S - i * units / p.S) % 2);
    printf("schedule=%d chunks=%d in_dw=%d row_parts=%d parts_h=%d least_parts_h=%d parts_w=%d split_sums=%d row_blocks=%d "
           "dhidden_blocks=%d sums_in_dhidden=%d chunks_in_dhidden=%d small_tiles=%d paired=%d paired_row_tiles=%d forward_skip=%d forward_skip_fp8=%d "
           "backward_skip=%d backward_skip_fp8=%d same_tiles=%d forward_big=%d forward_square=%d forward_tall=%d forward_halves=%d "
           "tall=%d square=%d tall_crossing=%d tall_behind=%d tall_mapped=%d fused=%d\n",
           (int)s.use, chunks, in_dw, part_steps, most_h, least_h, most_w, s.use ? s.split_acc : 0, s.use ? (p.TT + s.a - 1) / s.a : 0,
           s.n_blocks, sums_dh, chunks_dh, small, paired, most_rows, (int)forward_skip(p, D, false).use, (int)(D % 128 == 0 && forward_skip(p, D, true).use),
           (int)(!compact && backward_skip(p, s, D, false).use), (int)(!compact && D % 128 == 0 && backward_skip(p, s, D, true).use),
           (int)(steps > 0 && same_tiles == steps), (int)(fwd == kForwardBig), (int)(fwd == kForwardSquare), (int)(fwd == kForwardTall), halves,
           tiles.tall, tiles.square, tiles.crossing, tiles.behind, compact && !s.use ? tiles.tall : 0, (int)fused);    // (a schedule gathers the rows)
}

// The label scan in front of a forward that leaves ignored rows out is one workgroup, 0.4 ns a row: it has to be small beside the forward.
static void check_scan_is_priced() {
    const struct { int64_t N, D, V; bool use; } shapes[] = {
        {8192, 896, 151936, true}, {16384, 512, 70001, true}, {32768, 128, 140001, true}, {32768, 4096, 4400, true}, {131072, 896, 151936, true},
        {131072, 256, 32000, false}, {131072, 64, 70000, false}, {262144, 64, 35000, false}, {1000000, 64, 9100, false}, {2000000, 64, 5000, false}};
    for (auto& s : shapes) {
        Plan p;
        if (make_plan(s.N, s.D, s.V, &p) && forward_skip(p, s.D, false).use == s.use) continue;
        ++failures;
        fprintf(stderr, "FAIL scan in front of %lld x %lld x %lld\n", (long long)s.N, (long long)s.D, (long long)s.V);
    }
}

// cce_set_row_skipping: 1 switches every route that leaves rows out off, 2 none.
static void check_row_skipping_modes() {
    for (int mode = 0; mode < 3; ++mode) {
        const int64_t N = 8192, D = 896, V = 151936;
        Plan p; Schedule s;
        g_force_row_skipping.store(mode);
        if (make_plan(N, D, V, &p)) plan_backward(&p, N, D, V, false, true, workspace_to_ask_for(p, N, D, V, false), &s);
        if (forward_skip(p, D, false).use != (mode != 1) || backward_skip(p, s, D, false).use != (mode != 1)) {
            ++failures;
            fprintf(stderr, "FAIL row skipping, mode %d\n", mode);
        }
    }
    g_force_row_skipping.store(0);
}

// Row skipping is rated with the launches that run: over all rows at D = 64 and 128 the one without a gradient chunk, tiles of two
// wavefront groups elsewhere.
static void check_skipping_is_rated() {
    const struct { int64_t N, D, V, M; bool skip; } calls[] = {
        {8192, 64, 151936, 6963, false}, {8192, 128, 151936, 6963, false}, {22053, 128, 77882, 18745, false}, {2000, 64, 50000, 1500, false},
        {4000, 128, 20000, 2400, false}, {30884, 64, 23325, 23163, false}, {8699, 64, 68133, 1740, true}, {4791, 128, 54305, 958, true},
        {8192, 896, 151936, 6963, true}, {32768, 3584, 151936, 31130, false}, {16384, 2048, 151936, 15565, false},
        {17712, 1280, 4257, 15055, true}, {4300, 1344, 11822, 3870, true}, {19587, 1472, 12343, 16649, true}, {9452, 3136, 13619, 8034, true}};
    for (auto& c : calls) {
        Plan p;
        bool skip = !c.skip;
        if (plan_row_skipping(c.N, c.D, c.V, c.M, 0, &p, &skip) && skip == c.skip) continue;
        ++failures;
        fprintf(stderr, "FAIL row skipping %lld x %lld x %lld with %lld valid rows: %d\n", (long long)c.N, (long long)c.D, (long long)c.V, (long long)c.M, (int)skip);
    }
}

int main(int argc, char** argv) {
    if (argc > 2) {                          // N D V M dw_free, any number of times
        for (int i = 1; i + 4 < argc; i += 5) print_form(atoll(argv[i]), atoll(argv[i + 1]), atoll(argv[i + 2]), atoll(argv[i + 3]), atoi(argv[i + 4]) != 0);
        return 0;
    }
    const int iters = argc > 1 ? atoi(argv[1]) : 2000;
    check_makespan();
    check_floors();
    check_planning_cost();
    check_scan_is_priced();
    check_row_skipping_modes();
    check_skipping_is_rated();
    // shapes the schedules exist for: few rows against a full vocabulary; a small vocabulary
    bool dw_free = true; int64_t N = 509, D = 896, V = 151936, B = 0;
    CHECK(check(N, D, V, B, dw_free));
    N = 19823; D = 64; V = 1136;
    CHECK(check(N, D, V, B, dw_free));
    for (int it = 0; it < iters; ++it) {
        const int64_t n = it % 2 ? pick(1, 3000) : pick(1, 40000), d = 64 * (it % 3 ? pick(1, 16) : pick(1, 64));
        const int64_t v = it % 4 == 0 ? pick(1, 3000) : pick(1, 160000);
        if (v * d * 2 >= ((int64_t)1 << 32) || n * d * 2 >= ((int64_t)1 << 32)) continue;
        check(n, d, v, 0, true);
        check(n, d, v, 0, false);
        check(pick(1, n), d, v, n, it % 5 != 0);
    }
    printf("used %d, chunks in dW %d, split dH %d, split dW %d, row blocks %d, row parts %d, split sums %d, orders with dHidden %d, forwards that skip %d, backwards %d\n", used, in_tails, split_hs, split_ws, blocks, parts, split_accs, fronts, fwd_skips, bwd_skips);
    if (!in_tails || !split_hs || !split_ws || !parts || !split_accs || !fronts || !fwd_skips || !bwd_skips) { fprintf(stderr, "a form was never taken\n"); return 1; }
    if (failures) { fprintf(stderr, "%d failures\n", failures); return 1; }
    printf("schedule_fuzz: %d iterations ok\n", iters);
    return 0;
}
