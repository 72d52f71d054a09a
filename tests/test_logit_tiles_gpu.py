"""GPU test of the logit tiles at their edges, every column of the vocabulary by itself (shapes of schedule_shapes.LOGIT_TILES,
whose tiles test_schedule_host.py asks the planner for): forwards in each of their forms, splits that end in half a tile,
gradient tiles of 384 columns that end on, cross and lie behind the end of the vocabulary, one K slice, row maps, label
smoothing, z-loss, mean reduction, vocabulary shares, logits that are not finite.

Column v of the vocabulary is the one that row v % N answers to: a logit of 14, the V / N of them sharing the row's probability.
A column left out, counted twice or taken for another moves a row's lse by N / V at least (3e-3 here) and its own row of dW
wholly.  Reference: float64 by torch.  Bounds: a logit sums D products of bf16 in fp32, whose roundings (2^-24 of partial sums
of at most 20) come to 1.2e-6 sqrt(D) = 5e-5 by chance at D = 2112: 2e-4 on lse; G in bf16 (2^-9 of each term) and dHidden too:
GRAD_RTOL on every row of dW and dHidden."""
import pytest
import torch

from tests.gpu_util import GRAD_RTOL
from tests.schedule_shapes import LOGIT_TILES

pytestmark = pytest.mark.gpu
IGN = -100
LSE_ATOL = 2e-4
CASES = [(shape, form) for shape, forms in LOGIT_TILES.items() for form in forms]


def inputs(N, D, V, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(N + D + V + seed)
    H = torch.randn(N, D, device="cuda", generator=g)
    H = (H * (D ** 0.5 / H.norm(dim=1, keepdim=True))).bfloat16()
    W = torch.randn(V, D, device="cuda", generator=g) * (0.3 / D ** 0.5)
    W += H[torch.arange(V, device="cuda") % N].float() * (14.0 / D)
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    y[torch.randperm(N, device="cuda", generator=g)[:N // 4]] = IGN
    dl = (0.5 + torch.rand(N, device="cuda", generator=g)) / N
    return H, W.bfloat16(), y, dl


def reference(H, W, y, dl, eps, lam):
    """loss, lse (float64), dH, dW of the valid rows; dl: per row, None: mean reduction."""
    V, rows = W.shape[0], torch.nonzero(y != IGN).flatten()
    Hv, yv, at = H[rows].double(), y[rows].long(), torch.arange(len(rows), device="cuda")
    blocks = range(0, V, 8192)
    lse = torch.full((len(rows),), -float("inf"), dtype=torch.float64, device="cuda")
    zy, zsum = torch.zeros_like(lse), torch.zeros_like(lse)
    for v0 in blocks:
        z = Hv @ W[v0:v0 + 8192].double().t()
        lse = torch.logaddexp(lse, torch.logsumexp(z, dim=1))
        here = (yv >= v0) & (yv < v0 + z.shape[1])
        zy[here] = z[at[here], yv[here] - v0]
        zsum += z.sum(dim=1)
    loss = (1 - eps) * (lse - zy) + eps * (lse - zsum / V) + lam * lse * lse
    up = dl[rows].double() if dl is not None else torch.full_like(lse, 1.0 / len(rows))
    dH, dW = torch.zeros_like(Hv), torch.empty(V, H.shape[1], dtype=torch.float64, device="cuda")
    for v0 in blocks:
        w = W[v0:v0 + 8192].double()
        G = torch.exp(Hv @ w.t() - lse[:, None]) * (1 + 2 * lam * lse)[:, None] - eps / V
        here = (yv >= v0) & (yv < v0 + len(w))
        G[at[here], yv[here] - v0] -= 1 - eps
        G *= up[:, None]
        dH += G @ w
        dW[v0:v0 + 8192] = G.t() @ Hv
    return rows, loss, lse, dH, dW


def row_errors(got, want):
    return float(((got.double() - want).norm(dim=1) / want.norm(dim=1)).max())


def check(name, y, rows, out, want):
    loss, lse, dH, dW = out
    errs = (float((loss.double()[rows] - want[0]).abs().max()), float((lse.double()[rows] - want[1]).abs().max()),
            row_errors(dH[rows], want[2]), row_errors(dW, want[3]))
    print(f"    {name}: loss {errs[0]:.1e} lse {errs[1]:.1e} dH {errs[2]:.1e} dW {errs[3]:.1e}", flush=True)
    assert torch.all(loss[y == IGN] == 0) and torch.all(lse[y == IGN] == 0) and torch.all(dH[y == IGN] == 0)
    assert errs[0] <= LSE_ATOL and errs[1] <= LSE_ATOL and errs[2] <= GRAD_RTOL and errs[3] <= GRAD_RTOL


@pytest.mark.parametrize("shape,form", CASES)
def test_every_column_takes_part_once(shape, form):
    from paper_2601_02609_amd import binding as B
    N, D, V = shape
    H, W, y, dl = inputs(*shape)
    n_valid = N - N // 4
    for eps, lam, d in ((0.0, 0.0, dl), (0.1, 1e-3, None)):
        print(f"[logit tiles] {shape} {form} eps={eps}", flush=True)
        rows, *want = reference(H, W, y, d, eps, lam)
        B.set_row_skipping(2 if form == "compact" else 0)
        try:
            if form == "compact":
                ws = B.alloc_compact_workspace(N, D, V, n_valid)
                ws.fill_(0xff)
                loss, lse, _ = B.cce_forward_compact_ex(H, W, y, n_valid, IGN, label_smoothing=eps, z_loss=lam, workspace=ws)
                dH, dW = B.cce_backward_compact_ex(H, W, y, lse, d, n_valid, IGN, label_smoothing=eps, z_loss=lam, workspace=ws)
            else:
                ws = B.alloc_workspace(N, D, V)
                ws.fill_(0xff)
                loss, lse, _ = B.cce_forward_ex(H, W, y, IGN, label_smoothing=eps, z_loss=lam, workspace=ws)
                dH, dW = B.cce_backward_ex(H, W, y, lse, d, IGN, label_smoothing=eps, z_loss=lam, workspace=ws)
            torch.cuda.synchronize()
            assert B.read_status(ws) == 0
        finally:
            B.set_row_skipping(0)
        check(f"eps={eps}", y, rows, (loss, lse, dH, dW), want)


@pytest.mark.parametrize("shape", [(4352, 320, 23552), (257, 640, 92736)])
def test_shares_of_the_vocabulary(shape):
    """Two shares, the shape's vocabulary and an odd rest, each with its own tiles."""
    from paper_2601_02609_amd import binding as B
    N, D, Vs = shape
    V, eps, lam = Vs + 30001, 0.1, 1e-3
    H, W, y, dl = inputs(N, D, V)
    print(f"[logit tiles] shares of {shape}", flush=True)
    rows, *want = reference(H, W, y, dl, eps, lam)
    shares = [(0, W[:Vs].contiguous()), (Vs, W[Vs:].contiguous())]
    stats = torch.empty(2, N, 4, device="cuda")
    for i, (off, w) in enumerate(shares):
        B.cce_shard_forward(H, w, y, off, want_sumz=True, stats=stats[i])
    loss, lse, _ = B.cce_shard_merge(stats, y, V, IGN, label_smoothing=eps, z_loss=lam)
    grads = [B.cce_shard_backward(H, w, y, lse, dl, off, V, IGN, label_smoothing=eps, z_loss=lam) for off, w in shares]
    torch.cuda.synchronize()
    # (each share's dHidden is rounded to bf16 by itself: their sum has the rounding of both)
    check("shares", y, rows, (loss, lse, grads[0][0].float() + grads[1][0].float(), torch.cat([g[1] for g in grads])), want)


@pytest.mark.parametrize("shape", [(924, 320, 95232), (257, 1408, 32511), (1281, 192, 11713)])
def test_logits_that_are_not_finite(shape):
    """A NaN row of hidden reaches its own row alone; a column whose logits are minus infinity counts nothing; plus infinity
    and NaN in a column reach every row's loss."""
    from paper_2601_02609_amd import binding as B
    N, D, V = shape
    H, W, y, dl = inputs(*shape)
    H[:, 0] = 4.0
    bad, column = torch.nonzero(y != IGN).flatten()[5], V - 1
    y[y == column] = 0
    print(f"[logit tiles] {shape} not finite", flush=True)

    def forward(h, w):
        return B.cce_forward(h, w, y, IGN)

    loss, lse = forward(H, W)
    dH, _ = B.cce_backward(H, W, y, lse, dl, IGN)
    Hn = H.clone()
    Hn[bad, D - 1] = float("nan")
    loss_n, lse_n = forward(Hn, W)
    dH_n, _ = B.cce_backward(Hn, W, y, lse_n, dl, IGN)
    others = torch.arange(N, device="cuda") != bad
    assert torch.isnan(loss_n[bad]) and torch.isnan(lse_n[bad]) and torch.isnan(dH_n[bad].float()).all()
    assert torch.equal(loss_n[others], loss[others]) and torch.equal(lse_n[others], lse[others]) and torch.equal(dH_n[others], dH[others])
    Wm, valid = W.clone(), y != IGN
    for value in (-3.0e38, 3.0e38, float("nan")):
        Wm[column, 0] = value                                        # times 4: beyond the range of fp32
        loss_w, lse_w = forward(H, Wm)
        if value < 0:
            want = torch.logsumexp(H.double() @ W[:column].double().t(), dim=1)
            assert float((lse_w.double() - want)[valid].abs().max()) <= LSE_ATOL
        else:
            assert not torch.isfinite(loss_w[valid]).any() and not torch.isfinite(lse_w[valid]).any()
    torch.cuda.synchronize()
