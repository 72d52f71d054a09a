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
        int launches = 0, turn = 0, planes = 0, sums = 0, adds = 0, parts_h = 0, parts_w = 0, mapped = 0;
        auto count = [&](const LaunchShape& l, int kind, bool split, bool map) {
            ++launches;
            if (!launch_tiles(l, D, kind, split, map, counted, knobs).turn) return;
            ++turn;
            planes += split; sums += !split; adds += l.dw_beta; parts_h += l.parts_h > 1; parts_w += l.parts_w > 1; mapped += map;
        };
        if (s.use) {
            for (int64_t v = 0; v < V; ) {
                const ScheduleChunk c = schedule_chunk(s, D, V - v);
                for (int r = 0; r < s.a; r += c.rows)
                    count(launch_shape(s.a - r < c.rows ? s.a - r : c.rows, (int)c.b, s.split_h, s.split_w, v > 0, r > 0 || !dw_free), s.kind, s.split_acc != 0, false);
                v += c.b * 256;
            }
        } else {
            const int n = s.n_blocks ? s.n_blocks : (int)((p.TT * 256 + p.Nb - 1) / p.Nb);
            for (int q = 0; q < n; ++q) {
                RowBlock k = s.n_blocks ? s.blocks[q] : RowBlock{(int)(q * (p.Nb / 256)), (int)(p.Nb / 256), (int)(p.Vc / 256), p.gemm_kind, p.split_acc, false, false, 0, 0};
                const int a = p.TT - k.r0 < k.a ? p.TT - k.r0 : k.a;
                for (int v = 0; v < p.VT; v += k.b)
                    count(launch_shape(a, p.VT - v < k.b ? p.VT - v : k.b, 1, 1, v > 0, q > 0 || !dw_free), k.kind, k.split_acc != 0, compact);
            }
        }
        // (a call over all rows at D = 64 and 128 has no such launches)
        const bool fused = !compact && fused_backward_choice(p, N, D, V).use;
        printf("launches=%d turn=%d planes=%d sums=%d adds=%d parts=%d parts_w=%d mapped=%d counted=%d gathered=%d half=%d fused=%d\n", launches, fused ? 0 : turn, planes, sums,
               adds, parts_h + parts_w, parts_w, mapped, (int)(counted && turn > 0), (int)(compact && s.use && turn > 0),
               (int)(turn > 0 && D % 256 != 0 && D % 256 <= 128), (int)fused);
    }
    return 0;
}
