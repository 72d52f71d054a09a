"""GPU parity of the backward's schedules (csrc/plan.h; tests/host/schedule_fuzz.hip checks that such
shapes take them): gradient chunks in the unwritten rows of dW, K parts of either contraction, row
blocks over the whole vocabulary -- all rows, row skipping (tight and loose bound, NaN in the skipped
rows), accumulation.  Oracle and tolerances as in test_parity_gpu.py."""
import numpy as np
import pytest
import torch

from oracle import cce_oracle as O
from paper_2601_02609_amd import inputs as I
from tests.gpu_util import GRAD_RTOL, LOSS_ATOL, bf16_host, dev_inputs, rel_fro

pytestmark = pytest.mark.gpu
IGN = -100


@pytest.mark.parametrize("shape", [
    (300, 64, 30011),       # K parts of dH, two row tiles, ragged last chunk
    (80, 512, 30000),       # one row tile
    (900, 1088, 9001),      # chunks in dW, D not a multiple of the tile
    (3000, 64, 1100),       # K parts of dW, ragged last part
    (9000, 64, 300),        # many parts; row skipping in row blocks
    (5000, 128, 700),
])
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
    for form in ("rows", "accumulate", "compact", "compact_loose"):
        print(f"[schedule] {form}: N={N} D={D} V={V}", flush=True)
        dH = torch.full((N, D), 3.0, dtype=torch.bfloat16, device="cuda")
        dW = torch.full((V, D), 0.5 if form == "accumulate" else float("nan"), device="cuda")
        if form.startswith("compact"):
            B.set_row_skipping(2)
            try:
                # (a bound of N or more skips nothing, and the all-rows calls want finite hidden rows)
                bound = min(w.n_valid + 37, N - 1) if form.endswith("loose") else w.n_valid
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
        assert B.read_status(ws) == 0
        gH, gW = bf16_host(dH), dW.cpu().numpy().astype(np.float64)
        if form == "accumulate":
            gW -= 0.5          # exact to an fp32 unit of 0.5 (3e-8), below the gradients' bf16 rounding
        assert np.all(gH[ign] == 0.0)
        assert np.abs(loss.cpu().numpy() - o_loss).max() <= LOSS_ATOL and np.abs(lse.cpu().numpy() - o_lse).max() <= LOSS_ATOL
        e = rel_fro(gH, o_dH), rel_fro(gW, o_dW)
        print(f"[schedule] {form}: relF(dH)={e[0]:.2e} relF(dW)={e[1]:.2e}", flush=True)
        assert e[0] <= GRAD_RTOL and e[1] <= GRAD_RTOL
