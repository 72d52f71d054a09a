"""GPU parity of the backward's schedules (csrc/plan.h): gradient chunks in the unwritten rows of dW, K parts of
either contraction, row parts, row blocks over the whole vocabulary or with dHidden as scratch -- all rows, row skipping
(tight, loose and too small bounds, NaN in the skipped rows), accumulation, FP8 logits, a share of the
vocabulary.  The shapes and the orders they take are in schedule_shapes.py, which test_schedule_host.py checks
against the planner.  Oracle and tolerances as in test_parity_gpu.py."""
import numpy as np
import pytest
import torch

from oracle import cce_oracle as O
from paper_2601_02609_amd import inputs as I
from tests import schedule_shapes as S
from tests.gpu_util import GRAD_RTOL, LOSS_ATOL, bf16_host, dev_inputs, rel_fro

pytestmark = pytest.mark.gpu
IGN = -100
ROW_BOUND = 2          # CCE_STATUS_ROW_BOUND


@pytest.mark.parametrize("shape", list(S.AGAINST_ORACLE))
def test_schedule_matches_oracle(shape):
    from paper_2601_02609_amd import binding as B
    N, D, V = shape
    w = I.make_workload(I.custom_spec(N, D, V, seed=77, ignore_frac=0.2))
    o_loss, o_lse = O.forward(w.hidden, w.weight, w.labels, IGN)
    o_dH, o_dW = O.backward(w.hidden, w.weight, w.labels, w.dloss_var, IGN)
    ign = w.labels == IGN
    H, W, y = dev_inputs(w)
    dl = torch.from_numpy(w.dloss_var).cuda()
    Hn = H.clone()
    Hn[torch.from_numpy(ign).cuda()] = float("nan")
    valid = np.nonzero(~ign)[0]
    dropped = valid[-23:]                                # by the bound of "compact_dropped"
    lab = w.labels.copy()
    lab[dropped] = IGN
    for form in ("rows", "accumulate", "compact", "compact_loose", "compact_dropped"):
        if form == "compact_dropped":
            ign = lab == IGN
            o_loss, o_lse = O.forward(w.hidden, w.weight, lab, IGN)
            o_dH, o_dW = O.backward(w.hidden, w.weight, lab, w.dloss_var, IGN)
        print(f"[schedule] {form}: N={N} D={D} V={V}", flush=True)
        dH = torch.full((N, D), 3.0, dtype=torch.bfloat16, device="cuda")
        dW = torch.full((V, D), 0.5 if form == "accumulate" else float("nan"), device="cuda")
        if form.startswith("compact"):
            B.set_row_skipping(2)
            try:
                # (a bound of N or more skips nothing, and the all-rows calls want finite hidden rows)
                bound = min(w.n_valid + 37, N - 1) if form.endswith("loose") else w.n_valid - (dropped.size if form.endswith("dropped") else 0)
                ws = B.alloc_compact_workspace(N, D, V, bound)
                loss, lse = B.cce_forward_compact(Hn, W, y, bound, IGN, workspace=ws)
                B.cce_backward_compact(Hn, W, y, lse, dl, bound, IGN, workspace=ws, d_hidden=dH, d_weight=dW)
            finally:
                B.set_row_skipping(0)
        else:
            ws = B.alloc_workspace(N, D, V)
            loss, lse = B.cce_forward(H, W, y, IGN, workspace=ws)
            B.cce_backward(H, W, y, lse, dl, IGN, workspace=ws, d_hidden=dH, d_weight=dW, accumulate_dw=form == "accumulate")
        torch.cuda.synchronize()
        assert B.read_status(ws) == (ROW_BOUND if form == "compact_dropped" else 0)
        gH, gW = bf16_host(dH), dW.cpu().numpy().astype(np.float64)
        if form == "accumulate":
            gW -= 0.5          # exact to an fp32 unit of 0.5 (3e-8), below the gradients' bf16 rounding
        assert np.all(gH[ign] == 0.0)
        assert np.abs(loss.cpu().numpy() - o_loss).max() <= LOSS_ATOL and np.abs(lse.cpu().numpy() - o_lse).max() <= LOSS_ATOL
        e = rel_fro(gH, o_dH), rel_fro(gW, o_dW)
        print(f"[schedule] {form}: relF(dH)={e[0]:.2e} relF(dW)={e[1]:.2e}", flush=True)
        assert e[0] <= GRAD_RTOL and e[1] <= GRAD_RTOL


@pytest.mark.parametrize("shape,form", [(shape, form) for shape, forms in S.AGAINST_FORCED.items() for form in forms])
def test_schedule_matches_forced_tiling(shape, form):
    """Wide chunks in dW, then row parts, then the workspace; row blocks from the last to the first with
    sums and chunks in dHidden (the orders large shapes run in) against the
    same backward with a forced 16 x 16 tiling.  Both round the same gradient tiles, so dW differs by
    the order of fp32 sums over at most 12001 terms (sqrt(12001) 2^-24 = 7e-6; 2e-5 allowed) and dHidden
    by the values whose rounding to bf16 flips (each within 2^-8, two roundings 2^-9 apart: 2e-3)."""
    from paper_2601_02609_amd import binding as B
    N, D, V = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    y[torch.randperm(N, device="cuda", generator=g)[:N // 7]] = IGN
    n = N - N // 7
    dl = torch.rand(N, device="cuda", generator=g) / n
    before = torch.randn(V, D, device="cuda", generator=g) * 1e-5 if form == "accumulate" else None
    got = []
    for forced in (False, True):
        try:
            if forced:
                B.set_backward_tiling(16, 16)
            dW = before.clone() if form == "accumulate" else torch.full((V, D), float("nan"), device="cuda")
            if form != "compact":
                ws = B.alloc_workspace(N, D, V)
                _, lse = B.cce_forward(H, W, y, IGN, workspace=ws)
                dH, dW = B.cce_backward(H, W, y, lse, dl, IGN, workspace=ws, d_weight=dW, accumulate_dw=form == "accumulate")
            else:
                B.set_row_skipping(2)
                ws = B.alloc_compact_workspace(N, D, V, n)
                _, lse = B.cce_forward_compact(H, W, y, n, IGN, workspace=ws)
                dH, dW = B.cce_backward_compact(H, W, y, lse, dl, n, IGN, workspace=ws, d_weight=dW)
            torch.cuda.synchronize()
            assert B.read_status(ws) == 0
            got.append((dH.double(), dW.double()))
        finally:
            B.set_row_skipping(0)
            B.set_backward_tiling(0, 0)
    (h0, w0), (h1, w1) = got
    assert float((h0[y == IGN]).abs().max()) == 0.0
    e = float((h0 - h1).norm() / h1.norm()), float((w0 - w1).norm() / w1.norm())
    print(f"[schedule] {form} N={N} D={D} V={V}: relF(dH)={e[0]:.2e} relF(dW)={e[1]:.2e}", flush=True)
    assert e[0] <= 2e-3 and e[1] <= 2e-5


def test_workspace_of_the_largest_batch_serves_shorter_ones():
    """One workspace for 1024 rows, then batches of fewer: accepted, and right whichever order fits it."""
    from paper_2601_02609_amd import binding as B
    D, V = 2048, 4000
    ws = B.alloc_workspace(1024, D, V)
    for N in (1024, 356, 100, 1):
        print(f"[schedule] N={N} in the workspace of 1024 rows", flush=True)
        w = I.make_workload(I.custom_spec(N, D, V, seed=78, ignore_frac=0.2 if N > 1 else 0.0))
        H, W, y = dev_inputs(w)
        loss, lse = B.cce_forward(H, W, y, IGN, workspace=ws)
        dH, dW = B.cce_backward(H, W, y, lse, torch.from_numpy(w.dloss_var).cuda(), IGN, workspace=ws)
        torch.cuda.synchronize()
        assert B.read_status(ws) == 0
        o_loss, _ = O.forward(w.hidden, w.weight, w.labels, IGN)
        o_dH, o_dW = O.backward(w.hidden, w.weight, w.labels, w.dloss_var, IGN)
        assert np.abs(loss.cpu().numpy() - o_loss).max() <= LOSS_ATOL
        assert rel_fro(bf16_host(dH), o_dH) <= GRAD_RTOL and rel_fro(dW.cpu().numpy().astype(np.float64), o_dW) <= GRAD_RTOL


def relative(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


@pytest.mark.parametrize("shape", [(8001, 896, 150001), (12001, 4096, 8001)])
def test_fp8_schedule_matches_forced_tiling(shape):
    """FP8 logits in the same orders (row parts start at a row that is not the first, and the FP8 tiles take the
    whole tensor with a row offset; dHidden as scratch), overwriting and adding to dW: bounds as above."""
    from paper_2601_02609_amd import binding as B
    N, D, V = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    y[torch.randperm(N, device="cuda", generator=g)[:N // 7]] = IGN
    dl = torch.rand(N, device="cuda", generator=g) / N
    hq, hs = B.cce_quantize_e4m3(H)
    wq, wsc = B.cce_quantize_e4m3(W)
    before = torch.randn(V, D, device="cuda", generator=g) * 1e-5
    for accumulate in (False, True):
        got = []
        for forced in (False, True):
            try:
                if forced:
                    B.set_backward_tiling(16, 16)
                ws = B.alloc_workspace(N, D, V)
                dW = before.clone() if accumulate else torch.full((V, D), float("nan"), device="cuda")
                _, lse = B.cce_fp8_forward(hq, hs, wq, wsc, y, IGN, workspace=ws)
                got.append(B.cce_fp8_backward(hq, hs, wq, wsc, H, W, y, lse, dl, IGN, workspace=ws, d_weight=dW, accumulate_dw=accumulate))
                torch.cuda.synchronize()
            finally:
                B.set_backward_tiling(0, 0)
        (h0, w0), (h1, w1) = got
        e = relative(h0, h1), relative(w0, w1)
        print(f"[schedule] fp8 N={N} D={D} V={V} accumulate={accumulate}: relF(dH)={e[0]:.2e} relF(dW)={e[1]:.2e}", flush=True)
        assert float(h0[y == IGN].float().abs().max()) == 0.0 and e[0] <= 2e-3 and e[1] <= 2e-5


@pytest.mark.parametrize("shape", [(7500, 640, 90001), (12001, 4096, 8001), (509, 896, 151936), (3712, 64, 28036), (2224, 192, 9419)])
def test_shard_schedule_matches_forced_tiling(shape):
    """A share of the vocabulary that starts at row 20000 of a larger one, with label smoothing, z-loss and the mean
    reduction, in the orders of its own rows: against the forced tiling, bounds as above.  (Labels of other shares are valid and
    meet no column here.)"""
    from paper_2601_02609_amd import binding as B
    N, D, V = shape
    off, total = 20000, V + 30000
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, total, (N,), device="cuda", generator=g, dtype=torch.int32)
    y[torch.randperm(N, device="cuda", generator=g)[:N // 7]] = IGN
    st = B.cce_shard_forward(H, W, y, off, want_sumz=True)
    lse = torch.where(y == IGN, torch.zeros_like(st[:, 0]), st[:, 0] + st[:, 1].log() + 0.3)      # as if others had added a third
    got = []
    for forced in (False, True):
        try:
            if forced:
                B.set_backward_tiling(16, 16)
            dW = torch.full((V, D), float("nan"), device="cuda")
            got.append(B.cce_shard_backward(H, W, y, lse, None, off, total, IGN, label_smoothing=0.1, z_loss=1e-3, d_weight=dW))
            torch.cuda.synchronize()
        finally:
            B.set_backward_tiling(0, 0)
    (h0, w0), (h1, w1) = got
    e = relative(h0, h1), relative(w0, w1)
    print(f"[schedule] shard N={N} D={D} V={V} of {total}: relF(dH)={e[0]:.2e} relF(dW)={e[1]:.2e}", flush=True)
    assert float(h0[y == IGN].float().abs().max()) == 0.0 and e[0] <= 2e-3 and e[1] <= 2e-5


@pytest.mark.parametrize("cuts", [[30011], [9001, 39012]])
@pytest.mark.parametrize("D", [64, 192])
def test_shards_in_schedules_match_the_undivided_oracle(cuts, D):
    """Shares whose backwards run in K parts (D = 192) or parts of the vocabulary (D = 64), summed and concatenated against the undivided oracle."""
    from paper_2601_02609_amd import binding as B
    from tests.test_shard_gpu import parts_of, run_sharded
    N, V = 300, 60022
    w = I.make_workload(I.custom_spec(N, D, V, seed=79, ignore_frac=0.15))
    _, loss, lse, dH, dW, _, status = run_sharded(B, w, parts_of(V, cuts), w.dloss_var, 0.1, 1e-3)
    o_loss, o_lse = O.forward(w.hidden, w.weight, w.labels, IGN, label_smoothing=0.1, z_loss=1e-3)
    o_dH, o_dW = O.backward(w.hidden, w.weight, w.labels, w.dloss_var, IGN, label_smoothing=0.1, z_loss=1e-3)
    assert status == 0 and np.abs(loss - o_loss).max() <= LOSS_ATOL and np.abs(lse - o_lse).max() <= LOSS_ATOL
    assert rel_fro(dH, o_dH) <= GRAD_RTOL and rel_fro(dW, o_dW) <= GRAD_RTOL


@pytest.mark.parametrize("case", range(S.N_DRAWN))
def test_random_schedules(case):
    """Drawn calls with nothing forced (the sweep of test_random_shapes_gpu.py forces tilings, tiles or accumulators,
    which keeps the plan's own order): every loss variant, either form of the backward, all rows or the valid ones."""
    from paper_2601_02609_amd import binding as B
    c = S.drawn(case)
    print(f"[schedule] drawn {case}: {c}", flush=True)
    N, D, V, eps, lam = c["N"], c["D"], c["V"], c["eps"], c["lam"]
    w = I.make_workload(I.custom_spec(N, D, V, seed=6200 + case, ignore_frac=c["frac"]))
    H, W, y = dev_inputs(w)
    dl_np = np.full(N, 1.0 / max(w.n_valid, 1), dtype=np.float32) if c["mean"] else w.dloss_var
    dl = None if c["mean"] else torch.from_numpy(dl_np).cuda()
    o_loss, o_lse = O.forward(w.hidden, w.weight, w.labels, IGN, label_smoothing=eps, z_loss=lam)
    o_dH, o_dW = O.backward(w.hidden, w.weight, w.labels, dl_np, IGN, label_smoothing=eps, z_loss=lam)
    dH = torch.full((N, D), 3.0, dtype=torch.bfloat16, device="cuda")
    # (added to a dW of ones the sums would lose what lies below 6e-8: something as small as the gradients)
    base = np.random.default_rng(case).standard_normal((V, D)).astype(np.float32) * np.float32(np.abs(o_dW).mean())
    dW = torch.from_numpy(base).cuda() if c["accumulate"] else torch.full((V, D), float("nan"), device="cuda")
    bound = int(w.n_valid) + c["slack"]
    try:
        if c["skip"]:
            B.set_row_skipping(2)
            ws = B.alloc_compact_workspace(N, D, V, bound)
            loss, lse, _ = B.cce_forward_compact_ex(H, W, y, bound, IGN, label_smoothing=eps, z_loss=lam, workspace=ws)
            B.cce_backward_compact_ex(H, W, y, lse, dl, bound, IGN, label_smoothing=eps, z_loss=lam, workspace=ws,
                                      d_hidden=dH, d_weight=dW, accumulate_dw=c["accumulate"])
        else:
            ws = B.alloc_workspace(N, D, V)
            loss, lse, _ = B.cce_forward_ex(H, W, y, IGN, label_smoothing=eps, z_loss=lam, workspace=ws)
            B.cce_backward_ex(H, W, y, lse, dl, IGN, label_smoothing=eps, z_loss=lam, workspace=ws, d_hidden=dH, d_weight=dW,
                              accumulate_dw=c["accumulate"])
        torch.cuda.synchronize()
        assert B.read_status(ws) == 0
    finally:
        B.set_row_skipping(0)
    ign = w.labels == IGN
    gH, gW = bf16_host(dH), dW.cpu().numpy().astype(np.float64)
    if c["accumulate"]:
        gW -= base
    assert np.abs(loss.cpu().numpy() - o_loss).max() <= LOSS_ATOL and np.abs(lse.cpu().numpy() - o_lse).max() <= LOSS_ATOL
    assert np.all(gH[ign] == 0.0)
    assert rel_fro(gH, o_dH) <= GRAD_RTOL and rel_fro(gW, o_dW) <= GRAD_RTOL
