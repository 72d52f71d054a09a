"""GPU parity with the oracle where vocabularies end on, in front of and behind a tile, half a tile and a chunk's last tile, row
counts around a tile, one K slice, with and without label smoothing and row skipping.  Launches this small run their forwards on
the loop of 256 x 256 tiles and nearly all of their gradient tiles on 256 x 256 ones of two groups of wavefronts (see PingTile in
csrc/gemm_core.h), at D = 64 and 128 under row skipping only; the edges of the 384 x 256 ones, and of forwards on either: test_logit_tiles_gpu.py.  Oracle and tolerances as in
test_parity_gpu.py."""
import numpy as np
import pytest
import torch

from oracle import cce_oracle as O
from paper_2601_02609_amd import inputs as I
from tests.gpu_util import GRAD_RTOL, LOSS_ATOL, bf16_host, dev_inputs, rel_fro

pytestmark = pytest.mark.gpu
IGN = -100

# (rows, D, V): at least 129 tiles of 256 x 256, below which the 128 x 128 ones run
SHAPES = [(1281, 64, 384 * 30), (1280, 64, 384 * 30 + 1), (1279, 128, 384 * 30 + 192), (1281, 192, 384 * 30 + 193), (1500, 64, 384 * 30 + 383),
          (1000, 64, 256 * 50), (1025, 128, 256 * 50 + 1), (1024, 64, 256 * 50 + 128), (900, 320, 256 * 50 + 129),
          (4097, 64, 256 * 9 + 255), (7500, 64, 1537), (33, 256, 40001),
          (1281, 192, 384 * 30), (1280, 192, 384 * 30 + 1), (1000, 192, 256 * 50), (1025, 192, 256 * 50 + 1), (4097, 192, 256 * 9 + 255)]


@pytest.mark.parametrize("eps", [0.0, 0.1])
@pytest.mark.parametrize("shape", SHAPES)
def test_ping_tiles_match_oracle(shape, eps):
    from paper_2601_02609_amd import binding as B
    N, D, V = shape
    w = I.make_workload(I.custom_spec(N, D, V, seed=92, ignore_frac=0.25))
    o_loss, o_lse = O.forward(w.hidden, w.weight, w.labels, IGN, label_smoothing=eps)
    o_dH, o_dW = O.backward(w.hidden, w.weight, w.labels, w.dloss_var, IGN, label_smoothing=eps)
    H, W, y = dev_inputs(w)
    dl = torch.from_numpy(w.dloss_var).cuda()
    for skip in (False, True):
        print(f"[ping] N={N} D={D} V={V} eps={eps} skip={skip}", flush=True)
        B.set_row_skipping(2 if skip else 0)
        try:
            if skip:
                ws = B.alloc_compact_workspace(N, D, V, w.n_valid)
                loss, lse, _ = B.cce_forward_compact_ex(H, W, y, w.n_valid, IGN, label_smoothing=eps, workspace=ws)
                dH, dW = B.cce_backward_compact_ex(H, W, y, lse, dl, w.n_valid, IGN, label_smoothing=eps, workspace=ws)
            else:
                ws = B.alloc_workspace(N, D, V)
                loss, lse, _ = B.cce_forward_ex(H, W, y, IGN, label_smoothing=eps, workspace=ws)
                dH, dW = B.cce_backward_ex(H, W, y, lse, dl, IGN, label_smoothing=eps, workspace=ws)
            torch.cuda.synchronize()
            assert B.read_status(ws) == 0
        finally:
            B.set_row_skipping(0)
        assert np.abs(loss.cpu().numpy() - o_loss).max() <= LOSS_ATOL and np.abs(lse.cpu().numpy() - o_lse).max() <= LOSS_ATOL
        gH, gW = bf16_host(dH), dW.cpu().numpy().astype(np.float64)
        assert np.all(gH[w.labels == IGN] == 0.0)
        assert rel_fro(gH, o_dH) <= GRAD_RTOL and rel_fro(gW, o_dW) <= GRAD_RTOL
