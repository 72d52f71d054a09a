"""GPU parity where contractions run on 256 x 256 tiles of two wavefront groups: every form of their result (fp32 sums, added to or
not, planes, K parts, rows through a map, gathered, counted on the device), last column tiles of 64, 128 and 192 columns, ragged rows and
vocabularies.  Against gradients by torch in fp32 (the tolerance of test_parity_gpu.py: bf16 gradient tiles and dHidden), and
against the same call with its tile forced to another one, whose fp32 sums run in another order: at most 9000 terms of random sign, so
1e-5 of dW's norm; a bf16 result then differs by one unit (2^-8) where the two sums round apart, for at most one value in 15: 1e-3."""
import pytest
import torch

pytestmark = pytest.mark.gpu
IGN = -100

# N, D, V, form, words that turn_routes.hip has to give
SHAPES = [
    (3138, 2048, 2657, "rows", ("sums",)),
    (2895, 2432, 2699, "accumulate", ("sums", "adds", "half")),              # 128 columns behind 9 x 256
    (3674, 1856, 7519, "rows", ("planes", "half")),                          # 64 behind 7 x 256
    (3547, 1728, 3547, "accumulate", ("planes", "adds")),                    # 192 behind 6 x 256
    (286, 2048, 9128, "rows", ("parts", "sums")),
    (406, 1728, 11339, "accumulate", ("parts", "adds")),
    (5728, 1408, 1459, "rows", ("parts_w", "sums", "half")),
    (11340, 960, 1406, "accumulate", ("parts_w", "sums", "adds")),
    (3459, 1920, 2253, "compact", ("mapped", "sums", "half")),
    (5041, 1728, 3179, "compact", ("mapped", "planes")),
    (6151, 2816, 2893, "compact", ("gathered", "sums")),
    (8001, 896, 150001, "rows", ("counted", "planes", "half")),
    (6001, 2048, 52001, "rows", ("counted", "planes")),
]


def reference(H, W, y, dl):
    """lse and gradients of sum_i dl_i loss_i over the rows that are not ignored, fp32, in blocks of the vocabulary."""
    valid = y != IGN
    h, V = H.float(), W.shape[0]
    m = torch.full((H.shape[0],), -torch.inf, device="cuda")
    d = torch.zeros_like(m)
    for v in range(0, V, 8192):
        z = h @ W[v:v + 8192].float().t()
        mn = torch.maximum(m, z.amax(1))
        d = d * torch.exp(m - mn) + torch.exp(z - mn[:, None]).sum(1)
        m = mn
    lse = m + torch.log(d)
    scale = torch.where(valid, dl, torch.zeros_like(dl))
    dH, dW, rows = torch.zeros_like(h), torch.empty(W.shape, device="cuda"), torch.arange(H.shape[0], device="cuda")
    for v in range(0, V, 8192):
        w = W[v:v + 8192].float()
        g = torch.exp(h @ w.t() - lse[:, None])
        here = valid & (y >= v) & (y < v + w.shape[0])
        g[rows[here], (y[here] - v).long()] -= 1.0
        g *= scale[:, None]
        dH += g @ w
        dW[v:v + w.shape[0]] = g.t() @ h
    return torch.where(valid, lse, torch.zeros_like(lse)), dH, dW


def rel(a, b):
    return float(torch.linalg.vector_norm(a.double() - b.double()) / torch.linalg.vector_norm(b.double()))


@pytest.mark.parametrize("N,D,V,form,words", SHAPES)
def test_turn_tiles_match_torch_and_other_tiles(N, D, V, form, words):
    from paper_2601_02609_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(N + D)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    n_ignored = N // 5
    y[torch.randperm(N, device="cuda", generator=g)[:n_ignored]] = IGN
    dl = (0.5 + torch.rand(N, device="cuda", generator=g)) / (N - n_ignored)
    lse, r_dH, r_dW = reference(H, W, y, dl)
    before = torch.randn(V, D, device="cuda", generator=g) * (0.1 * float(r_dW.square().mean().sqrt()))
    got = {}
    for cols in (0, 128):
        print(f"[turn] N={N} D={D} V={V} {form} cols={cols}", flush=True)
        B.set_backward_gemm_tile(cols)
        try:
            if form == "compact":
                B.set_row_skipping(2)
                ws = B.alloc_compact_workspace(N, D, V, N - n_ignored)
                dH, dW = B.cce_backward_compact(H, W, y, lse, dl, N - n_ignored, IGN, workspace=ws)
            else:
                ws = B.alloc_workspace(N, D, V)
                into = before.clone() if form == "accumulate" else None
                dH, dW = B.cce_backward(H, W, y, lse, dl, IGN, workspace=ws, d_weight=into, accumulate_dw=form == "accumulate")
            torch.cuda.synchronize()
        finally:
            B.set_backward_gemm_tile(0)
            B.set_row_skipping(0)
        got[cols] = dH, dW - before if form == "accumulate" else dW
        assert rel(dH, r_dH) <= 1e-2 and rel(got[cols][1], r_dW) <= 1e-2
        assert not dH[y == IGN].any()
    assert rel(got[0][1], got[128][1]) <= 1e-5 and rel(got[0][0], got[128][0]) <= 1e-3
