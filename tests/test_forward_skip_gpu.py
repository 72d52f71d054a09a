"""GPU test of forwards that leave ignored rows out without being told their number (all-rows calls of about 1 ms and
more): none ignored, scattered ones, a whole last part, one valid row, none at all; label smoothing and mean; NaN in
ignored rows; a bad label.  Reference: fp32 logits by torch, in blocks of the vocabulary, log-sum-exp in fp64 (the
library's fp32 sums over D = 4096: about 1e-5 on a logit of size 15; tolerance as in test_parity_gpu.py)."""
import pytest
import torch

from tests.gpu_util import LOSS_ATOL

pytestmark = pytest.mark.gpu
IGN = -100
N, D, V = 2100, 4096, 67001             # 8.2 row tiles, 261.7 vocabulary tiles


@pytest.fixture(scope="module")
def operands():
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    parts, total = [], torch.zeros(N, dtype=torch.float64, device="cuda")
    zy = torch.zeros(N, dtype=torch.float64, device="cuda")
    for v0 in range(0, V, 8192):
        z = (H.float() @ W[v0:v0 + 8192].float().t()).double()
        parts.append(torch.logsumexp(z, dim=1))
        total += z.sum(dim=1)
        here = (y >= v0) & (y < v0 + z.shape[1])
        zy[here] = z[here, (y[here] - v0).long()]
    return H, W, y, torch.logsumexp(torch.stack(parts), dim=0), zy, total / V


@pytest.mark.parametrize("keep", ["all", "scattered", "front", "one", "none"])
@pytest.mark.parametrize("eps", [0.0, 0.1])
def test_forward_without_known_count(operands, keep, eps):
    from paper_2601_02609_amd import binding as B
    H, W, y0, lse_ref, zy, zmean = operands
    valid = torch.zeros(N, dtype=torch.bool, device="cuda")
    if keep == "all":
        valid[:] = True
    elif keep == "scattered":
        valid[torch.randperm(N, device="cuda")[:1700]] = True
    elif keep == "front":
        valid[:1024] = True             # whole tiles, the last valid row at an edge
    elif keep == "one":
        valid[1999] = True
    y = torch.where(valid, y0, torch.full_like(y0, IGN))
    Hn = torch.where(valid[:, None], H, torch.full_like(H, float("nan")))
    ws = B.alloc_workspace(N, D, V)
    ws.fill_(0xff)
    print(f"[forward skip] {keep} eps={eps}", flush=True)
    for _ in range(2):
        loss, lse, mean = B.cce_forward_ex(Hn, W, y, IGN, label_smoothing=eps, want_mean=True, workspace=ws)
    torch.cuda.synchronize()
    assert B.read_status(ws) == 0
    want = (1 - eps) * (lse_ref - zy) + eps * (lse_ref - zmean)
    assert torch.all(loss[~valid] == 0) and torch.all(lse[~valid] == 0)
    if keep != "none":
        assert (lse.double() - lse_ref)[valid].abs().max() <= LOSS_ATOL and (loss.double() - want)[valid].abs().max() <= LOSS_ATOL
        assert abs(float(mean) - float(want[valid].mean())) <= LOSS_ATOL
    else:
        assert float(mean) == 0.0


def test_bad_label_is_flagged_and_ignored(operands):
    from paper_2601_02609_amd import binding as B
    H, W, y0, lse_ref, zy, _ = operands
    y = y0.clone()
    y[77], y[900] = V, IGN
    ws = B.alloc_workspace(N, D, V)
    loss, lse = B.cce_forward(H, W, y, IGN, workspace=ws)
    torch.cuda.synchronize()
    assert B.read_status(ws) != 0
    ok = (y >= 0) & (y < V)
    assert torch.all(loss[~ok] == 0) and (loss.double() - (lse_ref - zy))[ok].abs().max() <= LOSS_ATOL


@pytest.mark.parametrize("N,D,V", [(26694, 960, 28747), (28063, 128, 167142), (2100, 4096, 70001)])
def test_static_forward_has_the_bits_of_the_forward(N, D, V):
    """Also where ignored rows are left out, and whatever the workspace holds beyond what the call needs."""
    from paper_2601_02609_amd import binding as B
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    y[torch.randperm(N, device="cuda", generator=g)[:N * 3 // 10]] = IGN
    y[7] = V
    ws = B.alloc_workspace(N, D, V)
    more = torch.empty(2 * ws.numel(), dtype=torch.uint8, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = [(torch.empty(N, device="cuda"), torch.empty(N, device="cuda")) for _ in range(3)]
    print(f"[static] {N}x{D}x{V}", flush=True)
    B.cce_forward_static(H, W, y, IGN, *out[0], status)
    B.cce_forward(H, W, y, IGN, workspace=ws, loss=out[1][0], lse=out[1][1])
    B.cce_forward(H, W, y, IGN, workspace=more, loss=out[2][0], lse=out[2][1])
    torch.cuda.synchronize()
    assert int(status) == 1 == B.read_status(ws)
    for loss, lse in out[1:]:
        assert torch.equal(loss, out[0][0]) and torch.equal(lse, out[0][1])
