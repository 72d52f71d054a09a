"""GPU test of gradient tiles whose shape (384 x 256 or 256 x 256) is picked on the device from the rows that take part: counts
on both sides of the pick, on and around whole row tiles, against the call that computes every row.  With the same lse the bf16
gradient tiles are the same numbers (both forms sum a logit's products in the same order), so the two differ by the order of the
fp32 sums alone: at most 5001 terms of dW and 150001 of dHidden, by chance sqrt(terms) 2^-24 of their norm (4e-6, 2.3e-5), here in
every block of 64 columns of the vocabulary and every row; dHidden by its rounding to bf16 too (a value on the other side of a
tie: 2^-7 of it at most)."""
import pytest
import torch

from tests.test_counted_rows_gpu import inputs

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
    lse, dH, dW = {}, {}, {}
    for mode in (1, 0):
        print(f"[counted tiles] {shape} valid={valid} mode={mode}", flush=True)
        B.set_row_skipping(mode)
        try:
            ws.fill_(0xff)
            _, lse[mode] = B.cce_forward(H, W, y, IGN, workspace=ws)
            dH[mode], dW[mode] = B.cce_backward(H, W, y, lse[1], dl, IGN, workspace=ws)
            torch.cuda.synchronize()
        finally:
            B.set_row_skipping(0)
    assert (lse[0].double() - lse[1].double()).abs().max() <= 2e-5      # (fp32 sums of exponentials in other splits; lse of about 15)
    worst = 0.0
    for v0 in range(0, V, 64 * 512):
        a, b = (torch.nn.functional.pad(dW[m][v0:v0 + 64 * 512].double(), (0, 0, 0, -(min(V, v0 + 64 * 512) - v0) % 64)) for m in (0, 1))
        worst = max(worst, float(((a - b).view(-1, 64 * D).norm(dim=1) / b.view(-1, 64 * D).norm(dim=1)).max()))
    a, b = dH[0].double(), dH[1].double()
    rms = b.square().mean(dim=1, keepdim=True).sqrt()
    over = float((((a - b).abs() - b.abs() * 2.0 ** -7) / rms.clamp_min(1e-30)).max())
    print(f"    dW {worst:.1e} dH beyond a rounding {over:.1e}, differing {float((a != b).double().mean()):.1e}", flush=True)
    assert worst <= 2e-5 and over <= 1e-4
