"""GPU test of gradient tiles whose shape (384 x 256 or 256 x 256) is picked on the device from the rows that take part: counts
on both sides of the pick, on and around whole row tiles, against the call that computes every row.  The two differ by the
order of the fp32 sums alone (bf16 gradient tiles are the same numbers); bound as in test_parity_gpu.py."""
import pytest
import torch

from tests.gpu_util import GRAD_RTOL
from tests.test_counted_rows_gpu import backward, inputs

pytestmark = pytest.mark.gpu
IGN = -100


@pytest.mark.parametrize("valid", [4500, 4353, 4097, 4096, 3585, 3072, 2049, 257, 256])
@pytest.mark.parametrize("shape", [(4500, 896, 150001), (5001, 960, 121003)])
def test_counts_around_the_pick(shape, valid):
    from paper_2601_02609_amd import binding as B
    N, D, V = shape
    g, H, W, y, dl = inputs(N, D, V)
    y[torch.randperm(N, device="cuda", generator=g)[: N - min(valid, N)]] = IGN
    ws = B.alloc_workspace(N, D, V)
    got = {}
    for mode in (1, 0):
        print(f"[counted tiles] {shape} valid={valid} mode={mode}", flush=True)
        B.set_row_skipping(mode)
        try:
            ws.fill_(0xff)
            got[mode] = backward(B, H, W, y, dl, "rows", None, ws)
            torch.cuda.synchronize()
        finally:
            B.set_row_skipping(0)
    for a, b in zip(got[0][1:], got[1][1:]):
        assert float((a.double() - b.double()).norm() / b.double().norm()) <= GRAD_RTOL
