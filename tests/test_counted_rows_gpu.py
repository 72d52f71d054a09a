"""GPU test of backwards whose number of rows is counted on the device, in every form that they run in (the shapes of
schedule_shapes.COUNTED, whose routes test_schedule_host.py checks): tiles of 128 x 128 and two to a unit, row maps longer than
their table, adds to dW, row parts, FP8 logits.

Nothing ignored, and every launch with the tile of the call that computes every row: the results have its bits.  Rows ignored:
against the gradients of the valid rows by torch in fp32, in blocks of the vocabulary (tolerance as in test_parity_gpu.py: the
library's gradients pass through bf16 on their way into the contractions)."""
import pytest
import torch

from tests.gpu_util import GRAD_RTOL
from tests.schedule_shapes import COUNTED

pytestmark = pytest.mark.gpu
IGN = -100
CASES = [(shape, form) for shape, forms in COUNTED.items() for form in forms if form != "forward"]


def inputs(N, D, V):
    g = torch.Generator(device="cuda")
    g.manual_seed(N + D)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    dl = torch.rand(N, device="cuda", generator=g) / N
    return g, H, W, y, dl


def e4m3_values(x):
    """What block-wise E4M3 keeps of a bf16 matrix: blocks of 128 columns, the scale amax / 448 rounded up to a power of two."""
    b = x.float().view(x.shape[0], -1, 128)
    amax = b.abs().amax(dim=2, keepdim=True)
    scale = torch.exp2(torch.where(amax > 0, torch.ceil(torch.log2(amax.double() / 448.0)).float(), torch.zeros_like(amax)))
    return ((b / scale).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).float() * scale).view(x.shape)


def backward(B, H, W, y, dl, form, old, ws, codes=None):
    """lse, dH, dW; `codes`: hidden rows of the logits where they are not H's."""
    if form == "fp8":
        wq, wsc = B.cce_quantize_e4m3(W)
        _, lse = B.cce_fp8_forward(*codes, wq, wsc, y, IGN, workspace=ws)
        return (lse, *B.cce_fp8_backward(*codes, wq, wsc, H, W, y, lse, dl, IGN, workspace=ws))
    _, lse = B.cce_forward(H, W, y, IGN, workspace=ws)
    dW = old.clone() if form == "accumulate" else torch.full(W.shape, float("nan"), device="cuda")
    dH = torch.full(H.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    return (lse, *B.cce_backward(H, W, y, lse, dl, IGN, workspace=ws, d_hidden=dH, d_weight=dW, accumulate_dw=form == "accumulate"))


@pytest.mark.parametrize("shape,form", [c for c in CASES if "same_tiles" in COUNTED[c[0]][c[1]]])
def test_nothing_ignored_has_the_bits_of_every_row_computed(shape, form):
    from paper_2601_02609_amd import binding as B
    g, H, W, y, dl = inputs(*shape)
    ws = B.alloc_workspace(*shape)
    old = torch.randn(W.shape, device="cuda", generator=g) * 1e-3 if form == "accumulate" else None
    codes = B.cce_quantize_e4m3(H) if form == "fp8" else None
    got = {}
    for mode in (1, 0):
        print(f"[counted] {shape} {form} mode={mode}", flush=True)
        B.set_row_skipping(mode)
        try:
            ws.fill_(0xff)
            got[mode] = backward(B, H, W, y, dl, form, old, ws, codes)
            torch.cuda.synchronize()
        finally:
            B.set_row_skipping(0)
    for a, b in zip(got[0][1:], got[1][1:]):
        assert torch.equal(a, b)


@pytest.mark.parametrize("keep", ["scattered", "one", "none"])
@pytest.mark.parametrize("shape,form", CASES)
def test_ignored_rows_take_no_part(shape, form, keep):
    from paper_2601_02609_amd import binding as B
    N, D, V = shape
    g, H, W, y, dl = inputs(N, D, V)
    valid = torch.zeros(N, dtype=torch.bool, device="cuda")
    if keep == "scattered":
        valid[torch.randperm(N, device="cuda", generator=g)[:N * 4 // 5]] = True
    elif keep == "one":
        valid[N - 3] = True
    y = torch.where(valid, y, torch.full_like(y, IGN))
    ws = B.alloc_workspace(N, D, V)
    ws.fill_(0xff)
    old = torch.randn(V, D, device="cuda", generator=g) * 1e-3 if form == "accumulate" else torch.zeros(V, D, device="cuda")
    codes = None
    Hz, Wz = H.float(), W.float()
    if form == "fp8":                            # the logits are those of the codes
        codes = B.cce_quantize_e4m3(H)
        Hz, Wz = e4m3_values(H), e4m3_values(W)
        codes[0].view(torch.uint8)[~valid] = 0x7f
    Hn = torch.where(valid[:, None], H, torch.full_like(H, float("nan")))
    print(f"[counted] {shape} {form} {keep}", flush=True)
    lse, dH, dW = backward(B, Hn, W, y, dl, form, old, ws, codes)
    torch.cuda.synchronize()
    assert torch.all(dH[~valid] == 0)
    if keep == "none":
        assert torch.equal(dW, old)
        return
    rows = torch.nonzero(valid).flatten()
    Hv, zv, at = H[rows].float(), Hz[rows], torch.arange(len(rows), device="cuda")
    want_dH = torch.zeros(len(rows), D, device="cuda")
    off = norm = 0.0
    for v0 in range(0, V, 8192):
        p = torch.exp(zv @ Wz[v0:v0 + 8192].t() - lse[rows, None])
        here = (y[rows] >= v0) & (y[rows] < v0 + p.shape[1])
        p[at[here], (y[rows][here] - v0).long()] -= 1
        p *= dl[rows, None]
        want_dH += p @ W[v0:v0 + 8192].float()
        want = p.t() @ Hv
        off += float((dW[v0:v0 + 8192] - old[v0:v0 + 8192] - want).double().square().sum())
        norm += float(want.double().square().sum())
    dh_err = float((dH[rows].double() - want_dH).norm() / want_dH.double().norm())
    print(f"    dW {(off / norm) ** 0.5:.1e} dH {dh_err:.1e}", flush=True)
    assert (off / norm) ** 0.5 <= GRAD_RTOL and dh_err <= GRAD_RTOL
