// Which contraction launches of a backward take tiles of two wavefront groups (TurnTile): for each call N D V M F on the command line
// (M valid rows under row skipping or 0, F = 1: dW overwritten) a line of "word=number".  Host code only, no GPU.
#include <stdio.h>
#include <stdlib.h>

#include "../../paper_2601_02609_amd/csrc/plan.h"

using namespace cce;

int main(int argc, char** argv) {
    for (int i = 1; i + 4 < argc; i += 5) {
        const int64_t N = atoll(argv[i]), D = atoll(argv[i + 1]), V = atoll(argv[i + 2]), M = atoll(argv[i + 3]);
        const bool compact = M > 0, dw_free = atoi(argv[i + 4]) != 0;
        const int64_t rows = compact ? M : N;
        Plan p; Schedule s;
        if (!make_plan(rows, D, V, &p, compact ? N : 0)) return 1;
        Plan asked = p;
        if (compact && M < N) { bool skip; plan_row_skipping(N, D, V, M, 2, &asked, &skip); }
        plan_backward(&p, rows, D, V, compact, dw_free, workspace_to_ask_for(asked, N, D, V, compact), &s);
        const Knobs knobs = Knobs::read();
        const bool counted = !compact && backward_skip(p, s, D, false).use;
        int launches = 0, turn = 0, planes = 0, sums = 0, adds = 0, parts = 0, mapped = 0;
        auto count = [&](int kind, bool split, int64_t e_h, int64_t nh, int64_t s_h, bool beta_h, int64_t e_w, int64_t nw, int64_t s_w, bool beta_w, bool map) {
            ++launches;
            if (!turn_contractions(kind, D, e_h, nh, s_h, beta_h, e_w, nw, s_w, beta_w, map, knobs)) return;
            ++turn;
            planes += split; sums += !split; adds += beta_w; parts += nh > 1 || nw > 1; mapped += map;
        };
        if (s.use) {
            const int64_t dt = (D + gemm_tile_of_kind(s.kind).bn - 1) / gemm_tile_of_kind(s.kind).bn;
            for (int64_t v = 0; v < V; ) {
                const ScheduleChunk c = schedule_chunk(s, D, V - v);
                const int64_t kh = (c.b + s.split_h - 1) / s.split_h, nh = (c.b + kh - 1) / kh;
                for (int64_t r = 0; r < s.a; r += c.rows) {
                    const int64_t t = s.a - r < c.rows ? s.a - r : c.rows, kw = (t + s.split_w - 1) / s.split_w, nw = (t + kw - 1) / kw;
                    const int kind = counted ? counted_contraction_kind(s.kind, D, t, c.b, dt, v > 0 || r > 0, r > 0 || !dw_free, knobs)
                                             : contraction_kind(s.kind, D, t * nh * dt, kh * 4, v > 0, s.split_acc != 0, c.b * nw * dt, kw * 4, r > 0 || !dw_free, false, knobs);
                    count(kind, s.split_acc != 0, t, nh, kh * 4, v > 0, c.b, nw, kw * 4, r > 0 || !dw_free, false);
                }
                v += c.b * 256;
            }
        } else {
            const int n = s.n_blocks ? s.n_blocks : (int)((p.TT * 256 + p.Nb - 1) / p.Nb);
            for (int q = 0; q < n; ++q) {
                RowBlock k = s.n_blocks ? s.blocks[q] : RowBlock{(int)(q * (p.Nb / 256)), (int)(p.Nb / 256), (int)(p.Vc / 256), p.gemm_kind, p.split_acc, false, false, 0, 0};
                const int64_t a = p.TT - k.r0 < k.a ? p.TT - k.r0 : k.a, dt = (D + gemm_tile_of_kind(k.kind).bn - 1) / gemm_tile_of_kind(k.kind).bn;
                for (int64_t v = 0; v < p.VT; v += k.b) {
                    const int64_t b = p.VT - v < k.b ? p.VT - v : k.b;
                    const bool beta_w = q > 0 || !dw_free;
                    count(contraction_kind(k.kind, D, a * dt, b * 4, v > 0, k.split_acc != 0, b * dt, a * 4, beta_w, compact, knobs), k.split_acc != 0, a, 1, b * 4, v > 0,
                          b, 1, a * 4, beta_w, compact);
                }
            }
        }
        printf("launches=%d turn=%d planes=%d sums=%d adds=%d parts=%d mapped=%d counted=%d gathered=%d half=%d\n", launches, turn, planes, sums, adds, parts, mapped,
               (int)(counted && turn > 0), (int)(compact && s.use && turn > 0), (int)(turn > 0 && D % 256 != 0 && D % 256 <= 128));
    }
    return 0;
}
