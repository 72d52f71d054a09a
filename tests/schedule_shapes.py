"""Shapes whose backward runs in an order of its own (csrc/plan.h), and what that order has to contain: read
by test_schedule_gpu.py, which runs them, and by test_schedule_host.py, which asks the planner whether they
still take those orders.  "rows": dW overwritten, "accumulate": added to, "compact": row skipping with the
exact count of valid rows, one in five ignored (one in seven in AGAINST_FORCED).

Words (least values): chunks of the vocabulary, in_dw of them in unwritten rows of dW, row_parts chunks taken in steps over
part of the rows, parts_h / parts_w K parts of dH / dW, varied (a chunk with fewer dH parts than another),
split_sums (dH sums in two planes), row_blocks, dhidden_blocks (row blocks from the last to the first) with
sums_in_dhidden / chunks_in_dhidden; fused: all rows at D = 64 and 128 without a gradient chunk, where the other words are zero."""

# against the fp64 oracle
AGAINST_ORACLE = {
    (300, 64, 30011): dict(rows=dict(fused=1), accumulate=dict(fused=1), compact=dict(parts_h=8)),
    (300, 192, 30011): dict(rows=dict(parts_h=8), accumulate=dict(parts_h=8), compact=dict(parts_h=8)),
    (80, 512, 30000): dict(rows=dict(parts_h=8), accumulate=dict(parts_h=8), compact=dict(parts_h=8)),       # one row tile
    (900, 1088, 9001): dict(rows=dict(parts_h=2), accumulate=dict(parts_h=2), compact=dict(parts_h=2)),      # D not a multiple of the tile
    (3000, 64, 1100): dict(rows=dict(fused=1), accumulate=dict(fused=1), compact=dict(parts_w=2)),       # ragged last part
    (3000, 320, 1100): dict(rows=dict(parts_w=2), accumulate=dict(parts_w=2), compact=dict(parts_w=2)),
    (9000, 64, 300): dict(rows=dict(fused=1), accumulate=dict(fused=1), compact=dict(parts_w=2, row_blocks=2)),
    (9000, 192, 300): dict(rows=dict(parts_w=8), accumulate=dict(parts_w=8)),
    (5000, 128, 700): dict(rows=dict(fused=1), accumulate=dict(fused=1), compact=dict(parts_w=4)),
    (5000, 256, 700): dict(rows=dict(parts_w=4), accumulate=dict(parts_w=4), compact=dict(parts_w=4)),
    (2445, 256, 8265): dict(rows=dict(row_blocks=2, parts_h=2)),
    (3712, 64, 28036): dict(rows=dict(fused=1)),
    (2224, 192, 9419): dict(rows=dict(chunks=2, parts_h=4, parts_w=2, varied=1), accumulate=dict(chunks=2, parts_h=4, parts_w=2, varied=1)),
    (522, 192, 41956): dict(rows=dict(chunks=3, parts_h=4, varied=1)),
    (323, 896, 54016): dict(rows=dict(chunks=2, in_dw=1, parts_h=2)),
    (707, 384, 30095): dict(compact=dict(chunks=2, parts_h=4, varied=1)),
}

# against the same call with forced 16 x 16 tiles
AGAINST_FORCED = {
    (509, 896, 151936): dict(rows=dict(chunks=3, in_dw=2, parts_h=4), accumulate=dict(chunks=3, parts_h=4), compact=dict(chunks=3, in_dw=2, parts_h=4)),
    (8001, 896, 150001): dict(rows=dict(chunks=10, in_dw=8, row_parts=2, split_sums=1), compact=dict(chunks=10, in_dw=8, row_parts=2)),
    (7500, 640, 90001): dict(rows=dict(chunks=10, in_dw=8, row_parts=2, split_sums=1), compact=dict(chunks=10, in_dw=8, row_parts=2)),
    (12001, 4096, 8001): dict(rows=dict(dhidden_blocks=2, sums_in_dhidden=1, chunks_in_dhidden=1),
                              accumulate=dict(dhidden_blocks=2, sums_in_dhidden=1, chunks_in_dhidden=1),
                              compact=dict(dhidden_blocks=2, sums_in_dhidden=1, chunks_in_dhidden=1)),
}

# all-rows calls that find their ignored rows on the device: forward_skip, backward_skip (with _fp8: on E4M3 operands), small_tiles /
# paired contraction launches of 128 x 128 tiles / 256 x 128 ones two to a unit, paired_row_tiles of the longest of those, same_tiles:
# every launch has the tile of the call that computes all rows.
# "forward": the forward alone is tested (test_forward_skip_gpu.py)
COUNTED = {
    (8001, 512, 150001): dict(rows=dict(forward_skip=1, backward_skip=1, small_tiles=1, row_parts=1, same_tiles=1),
                              fp8=dict(forward_skip_fp8=1, backward_skip_fp8=1, small_tiles=1, row_parts=1, same_tiles=1)),
    (6001, 2048, 52001): dict(rows=dict(forward_skip=1, backward_skip=1, paired=1, paired_row_tiles=17, row_parts=1, same_tiles=1)),
    (5000, 1536, 110001): dict(accumulate=dict(backward_skip=1, paired=1, paired_row_tiles=17, same_tiles=1)),
    (5130, 1536, 80001): dict(accumulate=dict(backward_skip=1, row_parts=1)),
    (2527, 3584, 68330): dict(rows=dict(backward_skip=1, paired=1, in_dw=1, same_tiles=1), accumulate=dict(backward_skip=1, paired=1, same_tiles=1),
                              fp8=dict(forward_skip_fp8=1, backward_skip_fp8=1, paired=1, same_tiles=1)),
    (4500, 896, 150001): dict(rows=dict(forward_skip=1, backward_skip=1), fp8=dict(forward_skip_fp8=1, backward_skip_fp8=1)),
    (6000, 640, 150001): dict(rows=dict(forward_skip=1, backward_skip=1, row_parts=1)),
    (5001, 960, 121003): dict(rows=dict(forward_skip=1, backward_skip=1)),
    (2100, 4096, 67001): dict(forward=dict(forward_skip=1)),
    (26694, 960, 28747): dict(forward=dict(forward_skip=1)),
    (28063, 128, 167142): dict(forward=dict(forward_skip=1)),
    (2100, 4096, 70001): dict(forward=dict(forward_skip=1)),
}

# logit tiles: forward_big / forward_square / forward_tall (the loop of 256 x 256 tiles, 256 x 256 and 384 x 256 tiles of two groups of
# wavefronts), forward_halves splits that end in half a tile; tall / square launches of gradient tiles of 384 / 256 columns, tall_crossing /
# tall_behind those whose last tile crosses / lies behind the end of the vocabulary, tall_mapped through a row map.  A quarter of the rows ignored
LOGIT_TILES = {
    (924, 320, 95232): dict(rows=dict(forward_tall=1, tall=2)),                            # 248 tiles of 384
    (1180, 256, 74497): dict(rows=dict(forward_tall=1, forward_halves=3)),                 # one column behind 194
    (257, 640, 92736): dict(rows=dict(forward_tall=1, forward_halves=1)),                  # half a tile behind 241
    (924, 256, 95999): dict(rows=dict(forward_tall=1, forward_halves=4, tall=1)),          # one column short of 250
    (4865, 128, 34176): dict(rows=dict(forward_tall=1, forward_halves=10)),                # two K slices
    (4352, 128, 147584): dict(compact=dict(forward_tall=1, forward_halves=11, tall=18, tall_behind=1)),
    (4352, 320, 23552): dict(rows=dict(forward_tall=1, forward_halves=11, tall=5, tall_crossing=1)),
    (4865, 320, 28031): dict(rows=dict(forward_tall=1, forward_halves=2, tall=7, tall_behind=1)),
    (412, 64, 34049): dict(rows=dict(forward_big=1, fused=1), compact=dict(tall_behind=1)),                       # one K slice
    (3484, 512, 6401): dict(compact=dict(tall_mapped=1, tall_behind=1)),
    (7425, 704, 6272): dict(compact=dict(tall_mapped=1, tall_crossing=1)),
    (668, 896, 42752): dict(rows=dict(forward_square=1, forward_halves=2, square=2)),      # 167 tiles of 256
    (412, 2112, 30721): dict(rows=dict(forward_square=1, forward_halves=1, square=1),      # one column behind 120
                             compact=dict(forward_square=1, forward_halves=1, square=1)),
    (257, 1856, 32640): dict(rows=dict(forward_square=1, forward_halves=1, square=1)),     # half a tile behind 127
    (257, 1408, 32511): dict(rows=dict(forward_square=1, square=1)),                       # one column short of that
    (903, 768, 9581): dict(rows=dict(forward_big=1)),                                      # one tile to a workgroup, units idle
    (1281, 192, 11713): dict(rows=dict(forward_big=1, tall=1, tall_crossing=1), compact=dict(forward_big=1)),
}


def n_ignored(N, against_forced=False):
    return N // 7 if against_forced else int(round(0.2 * N))


def drawn(case):
    """One of the seeded calls of test_random_schedules: sizes at which the planner leaves its own tiling, the loss
    variants, both forms of the backward; nothing forced."""
    import numpy as np
    rng = np.random.default_rng(6100 + case)
    while True:
        N, V = (int(np.exp(rng.uniform(np.log(lo), np.log(hi)))) for lo, hi in ((40, 9000), (300, 90000)))
        D = 64 * int(rng.integers(1, 17))
        if 2e8 <= N * D * V <= 1.6e10:
            break
    return dict(N=N, D=D, V=V, frac=float(rng.choice([0.0, 0.1, 0.4])), skip=bool(rng.integers(0, 2)), slack=int(rng.integers(0, 3)),
                eps=float(rng.choice([0.0, 0.1])), lam=float(rng.choice([0.0, 1e-3])), mean=bool(rng.integers(0, 2)),
                accumulate=bool(rng.integers(0, 2)))


N_DRAWN = 36
