// How backwards at D = 64 and 128 cut their two jobs (fused_backward_choice): over seeded shapes, every streamed tile lies in exactly one
// part, no part is empty, the items cover the stationary rows, and the planes of the parts fit the planned layout.  Host code, no GPU.
#include <stdio.h>
#include <stdlib.h>
#include <math.h>

#include "../../paper_2601_02609_amd/csrc/plan.h"

using namespace cce;

static int check(int64_t N, int64_t D, int64_t V) {
    Plan p;
    if (!make_plan(N, D, V, &p)) return 1;
    const FusedChoice f = fused_backward_choice(p, N, D, V);
    if (!f.use) return D == 64 || D == 128;
    const int64_t tiles_n = (N + 127) / 128, tiles_v = (V + 127) / 128, rows = f.shared ? 32 : D == 64 ? 256 : 128;
    bool ok = D == 64 || D == 128;
    ok = ok && (int64_t)f.len_h * f.parts_h >= tiles_v && (int64_t)f.len_h * (f.parts_h - 1) < tiles_v;
    ok = ok && (int64_t)f.len_w * f.parts_w >= tiles_n && (int64_t)f.len_w * (f.parts_w - 1) < tiles_n;
    ok = ok && f.n_h == (N + rows - 1) / rows * f.parts_h && f.n_w == (V + rows - 1) / rows * f.parts_w;
    const double planes = ((f.parts_h > 1 ? f.parts_h : 0) * (double)(N * D) + (f.parts_w - 1) * (double)(V * D)) * 4.0;
    ok = ok && (double)p.off_dhacc + planes <= (double)p.total;
    if (!ok) fprintf(stderr, "FAIL %lld x %lld x %lld: parts %d x %d, %d x %d\n", (long long)N, (long long)D, (long long)V, f.parts_h, f.len_h, f.parts_w, f.len_w);
    return ok ? 0 : 1;
}

// The sum of few rows' planes takes 0.39 us a plane: ranges of few tiles (96 here) are not cut into 48 parts because they can be.
static int few_parts(int64_t N, int64_t D, int64_t V, int most) {
    Plan p;
    const FusedChoice f = make_plan(N, D, V, &p) ? fused_backward_choice(p, N, D, V) : FusedChoice{};
    if (f.use && f.parts_h <= most && f.parts_w <= most) return 0;
    fprintf(stderr, "FAIL %lld x %lld x %lld: parts %d, %d\n", (long long)N, (long long)D, (long long)V, f.parts_h, f.parts_w);
    return 1;
}

int main(int argc, char** argv) {
    if (argc > 1) {                          // N D V, any number of times: how the launch is cut
        for (int i = 1; i + 2 < argc; i += 3) {
            const int64_t N = atoll(argv[i]), D = atoll(argv[i + 1]), V = atoll(argv[i + 2]);
            Plan p;
            const FusedChoice f = make_plan(N, D, V, &p) ? fused_backward_choice(p, N, D, V) : FusedChoice{};
            printf("%d %d %d %d\n", (int)f.use, (int)f.shared, (int)(f.parts_h > 1), (int)(f.parts_w > 1));
        }
        return 0;
    }
    int bad = 0, n = 0;
    bad += few_parts(228, 128, 12162, 24) + few_parts(228, 64, 12162, 24) + few_parts(900, 128, 12162, 8) + few_parts(160, 64, 12162, 24);
    srand(11);
    const int64_t edges[] = {1, 31, 32, 33, 127, 128, 129, 255, 257, 1000, 32768, 151936};
    for (int64_t N : edges)
        for (int64_t V : edges)
            for (int64_t D : {64, 128, 192}) { bad += check(N, D, V); ++n; }
    auto draw = [](double lo, double hi) { return (int64_t)exp(log(lo) + (log(hi) - log(lo)) * rand() / RAND_MAX); };
    for (int i = 0; i < 3000; ++i, ++n) bad += check(draw(1, 200000), 64 * (1 + rand() % 2), draw(1, 400000));
    printf("%d shapes, %d failures\n", n, bad);
    return bad != 0;
}
