"""GPU test of backwards that leave ignored rows out by a count found on the device (large calls whose schedule has all
rows in one block): against the same call with every row computed (row skipping forced off).  The fp32 sums
run in other orders (zero terms left out of dW; launches of the other call that take tiles two to a compute unit, K groups): at
most 6000 and 256 terms at a time, 1e-5 of the norm; a bf16 result of dHidden then differs by one unit (2^-8) where the two
sums round apart, for at most one value in 15: 1e-3 of its norm.  NaN in ignored rows must change nothing."""
import pytest
import torch

pytestmark = pytest.mark.gpu
IGN = -100


@pytest.mark.parametrize("N,D,V", [(4500, 896, 150001), (6000, 640, 150001), (5001, 960, 121003)])     # one column tile cut off; row parts
def test_backward_without_known_count(N, D, V):
    from paper_2601_02609_amd import binding as B
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y0 = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    dl = torch.rand(N, device="cuda", generator=g) / N
    ws = B.alloc_workspace(N, D, V)
    for keep in ("all", "scattered", "front", "one", "none"):
        valid = torch.zeros(N, dtype=torch.bool, device="cuda")
        if keep == "all":
            valid[:] = True
        elif keep == "scattered":
            valid[torch.randperm(N, device="cuda", generator=g)[:N * 4 // 5]] = True
        elif keep == "front":
            valid[:1024] = True
        elif keep == "one":
            valid[N - 3] = True
        y = torch.where(valid, y0, torch.full_like(y0, IGN))
        Hn = torch.where(valid[:, None], H, torch.full_like(H, float("nan")))
        got = {}
        for mode in (1, 0):
            print(f"[backward skip] {N}x{D}x{V} {keep} mode={mode}", flush=True)
            B.set_row_skipping(mode)
            try:
                ws.fill_(0xff)
                x = H if mode == 1 else Hn
                _, lse, _ = B.cce_forward_ex(H, W, y, IGN, workspace=ws)
                for _ in range(2):
                    dH, dW = B.cce_backward_ex(x, W, y, lse, dl if keep != "front" else None, IGN, label_smoothing=0.1, z_loss=1e-4, workspace=ws,
                                               d_hidden=torch.full((N, D), float("nan"), dtype=torch.bfloat16, device="cuda"),
                                               d_weight=torch.full((V, D), float("nan"), device="cuda"))
                torch.cuda.synchronize()
                assert B.read_status(ws) == 0
            finally:
                B.set_row_skipping(0)
            got[mode] = dH, dW
        assert torch.all(got[0][0][~valid] == 0)
        if keep == "none":
            assert torch.all(got[0][0] == 0) and torch.all(got[0][1] == 0)
            continue
        err = (got[0][1] - got[1][1]).double().norm() / got[1][1].double().norm()
        rows = (got[0][0].double() - got[1][0].double()).norm() / got[1][0].double().norm()
        print(f"    dW {float(err):.1e} dH {float(rows):.1e}", flush=True)
        assert err <= 1e-5 and rows <= 1e-3


def test_fp8_without_known_count():
    """Forward and backward on E4M3 operands; codes of ignored rows are NaN where they are left out."""
    from paper_2601_02609_amd import binding as B
    N, D, V = 4500, 896, 150001
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    H *= torch.exp2(torch.randint(-3, 4, (N, 1), device="cuda", generator=g).float()).bfloat16() * 0.25      # scales that differ from row to row
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    dl = torch.rand(N, device="cuda", generator=g) / N
    hq, hs = B.cce_quantize_e4m3(H)
    wq, wsc = B.cce_quantize_e4m3(W)
    ws = B.alloc_workspace(N, D, V)
    for n_ignored in (0, 900):
        y[torch.randperm(N, device="cuda", generator=g)[:n_ignored]] = IGN
        valid = y != IGN
        got = {}
        for mode in (1, 0):
            print(f"[fp8 skip] ignored={n_ignored} mode={mode}", flush=True)
            B.set_row_skipping(mode)
            try:
                ws.fill_(0xff)
                codes = hq.clone()
                if mode == 0:
                    codes.view(torch.uint8)[~valid] = 0x7f
                loss, lse = B.cce_fp8_forward(codes, hs, wq, wsc, y, IGN, workspace=ws)
                dH, dW = B.cce_fp8_backward(codes, hs, wq, wsc, H, W, y, lse, dl, IGN, workspace=ws)
                torch.cuda.synchronize()
                assert B.read_status(ws) == 0
            finally:
                B.set_row_skipping(0)
            got[mode] = [t.double() for t in (loss, lse, dH, dW)]
        for a, b, tol in zip(got[0], got[1], (1e-6, 1e-6, 1e-3, 1e-5)):       # fp32 sums over the vocabulary in other splits
            assert (a - b).norm() <= tol * b.norm()
        assert torch.all(got[0][0][~valid] == 0) and torch.all(got[0][2][~valid] == 0)


def test_status_word_is_the_forwards():
    """A backward over all rows leaves the status word as it is, also where it scans the labels."""
    from paper_2601_02609_amd import binding as B
    N, D, V = 6000, 640, 150001
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    dl = torch.rand(N, device="cuda", generator=g) / N
    ws = B.alloc_workspace(N, D, V)
    bad = y.clone()
    bad[5] = V
    for first, then, want in ((bad, y, 1), (y, bad, 0)):        # 1: CCE_STATUS_BAD_LABEL
        print(f"[status] {want}", flush=True)
        _, lse = B.cce_forward(H, W, first, IGN, workspace=ws)
        B.cce_backward(H, W, then, lse, dl, IGN, workspace=ws)
        assert B.read_status(ws) == want
