"""The C-ABI shared library loads and exports every symbol include/*.h declares (no GPU needed),
and its host-only entry points behave as documented."""
import os
import re

import pytest

from paper_2601_02609_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    if not build.is_built():
        build.build(verbose=False)
    return binding.lib()


def declared_symbols():
    names = set()
    inc = os.path.join(ROOT, "include")
    for fn in sorted(os.listdir(inc)):
        if not fn.endswith(".h"):
            continue
        text = open(os.path.join(inc, fn)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(cce_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_header_and_binding_agree():
    assert declared_symbols() == sorted(binding.EXPORTED_SYMBOLS)


def test_every_declared_symbol_is_exported(L):
    for name in declared_symbols():
        assert hasattr(L, name), name


def test_host_only_entry_points(L):
    assert re.fullmatch(r"\d+\.\d+\.\d+", binding.version())
    assert L.cce_strerror(0) == b"ok"
    assert b"multiple of 64" in L.cce_strerror(binding.CCE_ERR_UNSUPPORTED)
    # the paper's memory equation: 8 x 1024 tokens x 151,936 x 4 bytes = 4.97 GB
    assert binding.materialised_logit_bytes(8192, 151936) == 8192 * 151936 * 4
    assert binding.materialised_logit_bytes(0, 5) == 0
    # auxiliary entry points: workspace sizes are pure host functions
    assert L.cce_rmsnorm_workspace_bytes(8192, 896) > 0 and L.cce_rmsnorm_workspace_bytes(8192, 100) == 0
    assert L.cce_rmsnorm_workspace_bytes(8192, 16384) == 0          # beyond the row a wavefront holds
    assert L.cce_sumsq_workspace_bytes() >= 8


def test_workspace_is_small_and_independent_of_NV(L):
    N, D, V = 8192, 896, 151936
    ws = binding.workspace_bytes(N, D, V)
    assert 0 < ws <= 0.01 * binding.materialised_logit_bytes(N, V)
    # invalid shapes
    assert binding.workspace_bytes(N, 100, V) == 0
    assert binding.workspace_bytes(0, D, V) == 0
    # O(N*D + tile): doubling V must not double the workspace beyond the 1 % budget rule
    for (n, d, v) in [(16384, 2048, 151936), (32768, 3584, 151936)]:
        assert binding.workspace_bytes(n, d, v) <= 0.01 * binding.materialised_logit_bytes(n, v)


def test_workspace_serves_fewer_rows(L):
    """A workspace sized for the largest batch serves every smaller one, and any bound under row skipping."""
    for d, v in [(2048, 4000), (64, 1000), (896, 151936), (512, 32000), (256, 128256)]:
        rows = [1, 63, 100, 356, 500, 1024, 1500, 2048, 4096, 6000, 8192, 16384]
        ask = [binding.workspace_bytes(n, d, v) for n in rows]
        assert ask == sorted(ask), (d, v, ask)
        compact = [[binding.compact_workspace_bytes(n, d, v, m) for m in (1, n // 2, n * 9 // 10, n)] for n in rows]
        for small, large in zip(compact, compact[1:]):
            assert max(small) <= min(large), (d, v, compact)


def test_workspace_stays_near_what_layouts_hold(L):
    """1 % of the logits is a bound and not the answer where no layout comes near it: a chunk has at most 64 x 128
    tiles (1.07 GB) in a plan's layout, whatever the vocabulary."""
    assert binding.workspace_bytes(5000, 64, 30_000_000) < 0.4e9          # 1 %: 6.0 GB
    assert binding.workspace_bytes(30000, 64, 1 << 24) < 1.4e9            # 1 %: 20 GB
    assert binding.workspace_bytes(4096, 64, 33_000_000) < 0.4e9          # at most 16 row tiles: no room for planes is taken here


@pytest.mark.parametrize("shape,skips", [
    ((8192, 896, 151936, 6963), True), ((16384, 4096, 32000, 12288), True), ((16384, 2048, 151936, 15565), False),
    ((500, 256, 3000, 300), False), ((8385, 192, 2434, 5031), False),
    # faster when skipped by 12 % in both forms of the backward, by 7 and 14 %
    ((1402, 2432, 112762, 1191), True), ((4800, 3008, 37936, 4080), True),
    # only one form of the two gains much: overwriting 9 %, 8 % and 7 %, adding to dW 6 %, nothing and 4 %
    ((4974, 384, 124212, 4477), True), ((6675, 256, 59907, 6341), True), ((1998, 1280, 122224, 1698), True),
    # 0.77 of the time when skipped: the forward of all rows is a round of small tiles longer
    ((2003, 2240, 2596, 1202), True)])
def test_row_skipping_choice(L, shape, skips):
    """The choice on shapes timed both ways (256 compute units; dW overwritten and added to)."""
    assert binding.get_row_skipping(*shape) == skips


def test_forced_tiling_is_bounded(L):
    """A forced tiling whose gradient chunk would need more than 32-bit byte offsets is refused."""
    try:
        binding.set_backward_tiling(128, 594)
        assert binding.workspace_bytes(32768, 3584, 151936) == 0
        binding.set_backward_tiling(2, 3)
        assert binding.get_backward_tiling(8192, 896, 151936) == (2, 3)
        assert binding.workspace_bytes(8192, 896, 151936) > 0
    finally:
        binding.set_backward_tiling(0, 0)
    assert binding.get_backward_tiling(8192, 896, 151936) == (16, 16)
    with pytest.raises(binding.CCEError):
        binding.set_backward_tiling(3, 0)


def test_contraction_tile_choice(L):
    """256 x 128 tiles when D is not a multiple of 256 or when 256 x 256 tiles would fill less than
    70 % of the workgroup rounds of a launch; the override wins over both."""
    assert binding.get_backward_gemm_tile(8192, 896, 151936) == (256, 128)
    assert binding.get_backward_gemm_tile(32768, 3584, 151936) == (256, 256)
    assert binding.get_backward_gemm_tile(16384, 2048, 128256) == (256, 256)
    assert binding.get_backward_gemm_tile(16384, 1024, 50257) == (256, 128)
    try:
        binding.set_backward_gemm_tile(256)
        assert binding.get_backward_gemm_tile(8192, 896, 151936) == (256, 256)
        binding.set_backward_gemm_tile(128)
        assert binding.get_backward_gemm_tile(32768, 3584, 151936) == (256, 128)
    finally:
        binding.set_backward_gemm_tile(0)


def test_accumulator_choice(L):
    """fp32 running sum at the headline shape (it fits the budget with the best tiling), split
    planes where D is large against the budget."""
    assert binding.get_backward_accumulator(8192, 896, 151936) == 1
    assert binding.get_backward_accumulator(16384, 4096, 32000) == 2
    with pytest.raises(binding.CCEError):
        binding.set_backward_accumulator(3)


def test_row_skipping_tiling_query(L):
    """Host-only: where rows are not skipped the row-skipping calls run the all-rows tiling; at the
    headline shape with 15 % of the rows ignored they skip and fit the 28 row tiles into two blocks."""
    assert binding.get_compact_tiling(8192, 896, 151936, 8192) == binding.get_backward_tiling(8192, 896, 151936)
    assert binding.get_row_skipping(8192, 896, 151936, 6963)
    a, b = binding.get_compact_tiling(8192, 896, 151936, 6963)
    assert a == 14 and b >= 16
    with pytest.raises(binding.CCEError):
        binding.get_compact_tiling(8192, 100, 151936, 10)
