"""GPU parity of the backward that keeps its gradient chunk in registers (D = 64 and 128): one and several parts of either streamed range,
wavefronts that share their rows, ragged rows and vocabularies, loss variants, mean reduction, a share of the vocabulary.  Against
gradients by torch in fp32 (the tolerance of test_parity_gpu.py), and against the same call with a forced tiling, which runs over a
gradient chunk in memory: the same bf16 gradients in another order of fp32 sums, 1e-5 of dW's norm; a bf16 result then differs by one
unit (2^-8) where the two sums round apart, for at most one value in 15: 1e-3 of dHidden's norm."""
import pytest
import torch

pytestmark = pytest.mark.gpu
IGN = -100


# N, D, V, form, what the launch is cut into: (wavefronts share their rows, several parts of the vocabulary, of the tokens)
FORMS = [
    (60513, 64, 1203, "accumulate", (0, 0, 1)), (59621, 64, 2309, "mean", (0, 0, 1)),
    (1199, 64, 61313, "variants", (0, 1, 0)), (1893, 64, 65361, "accumulate", (0, 1, 0)),
    (3529, 64, 9829, "shard", (0, 1, 1)), (3573, 64, 9895, "variants", (0, 1, 1)), (3575, 64, 9981, "mean", (0, 1, 1)),
    (1177, 64, 105, "shard", (1, 0, 1)), (101, 64, 2503, "variants", (1, 1, 0)), (1799, 64, 2621, "mean", (1, 1, 1)),
    (22455, 128, 22417, "accumulate", (0, 0, 0)),
    (33001, 128, 2050, "accumulate", (0, 0, 1)), (40007, 128, 1283, "variants", (0, 0, 1)),
    (617, 128, 30573, "mean", (0, 1, 0)), (3001, 128, 33001, "shard", (0, 1, 0)),
    (4100, 128, 9001, "shard", (0, 1, 1)), (1715, 128, 9687, "accumulate", (0, 1, 1)),
    (1025, 128, 101, "shard", (1, 0, 1)), (101, 128, 1187, "variants", (1, 1, 0)), (2259, 128, 3655, "accumulate", (1, 1, 1)),
]


def reference(H, W, y, dl, eps, lam, v_off, v_total, lse):
    """Gradients of this share of the vocabulary for the given lse of all of it, fp32."""
    valid = (y != IGN) & (y >= 0) & (y < v_total)
    h = H.float()
    g = torch.exp(h @ W.float().t() - lse[:, None]) * (1 + 2 * lam * lse)[:, None] - eps / v_total
    here = valid & (y >= v_off) & (y < v_off + W.shape[0])
    rows = torch.arange(H.shape[0], device="cuda")
    g[rows[here], (y[here] - v_off).long()] -= 1 - eps
    g = torch.where(valid[:, None], g * dl[:, None], torch.zeros_like(g))
    return g @ W.float(), g.t() @ h


def rel(a, b):
    return float(torch.linalg.vector_norm(a.double() - b.double()) / torch.linalg.vector_norm(b.double()).clamp_min(1e-30))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,V,form", [
    (1, 2, "rows"), (1, 130, "rows"), (127, 31, "accumulate"), (256, 1000, "rows"), (129, 4099, "variants"), (1023, 259, "mean"),
    (3001, 2050, "accumulate"), (517, 20011, "shard"), (9001, 1283, "variants"), (4100, 9001, "rows"), (20011, 515, "shard"),
])
def test_fused_backward_matches_torch_and_chunks(N, V, form, D):
    check(N, D, V, form)


@pytest.mark.parametrize("N,D,V,form", [f[:4] for f in FORMS])
def test_every_cut_of_the_fused_backward(N, D, V, form):
    """The forms that large calls take; test_fused_cuts_host.py asks the planner whether these shapes still take them."""
    check(N, D, V, form)


def check(N, D, V, form):
    from paper_2601_02609_amd import binding as B
    print(f"[fused] N={N} D={D} V={V} {form}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + D + V)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    v_off, v_total = (V // 2, 2 * V) if form == "shard" else (0, V)
    y = torch.randint(0, v_total, (N,), device="cuda", generator=g, dtype=torch.int32)
    y[torch.rand(N, device="cuda", generator=g) < 0.2] = IGN
    valid = y != IGN
    eps, lam = (0.1, 1e-3) if form in ("variants", "mean", "shard") else (0.0, 0.0)
    lse = torch.logsumexp(H.float() @ W.float().t(), 1) + (0.7 if form == "shard" else 0.0)
    lse = torch.where(valid, lse, torch.full_like(lse, float("nan")))            # (what an ignored row holds is not looked at)
    dl = torch.rand(N, device="cuda", generator=g) + 0.5
    dl = torch.where(valid, dl, torch.full_like(dl, float("nan")))
    mean = form == "mean"
    used = torch.full_like(dl, 1.0 / max(int(valid.sum()), 1)) if mean else dl
    r_dH, r_dW = reference(H, W, y, used, eps, lam, v_off, v_total, lse)
    before = torch.randn(V, D, device="cuda", generator=g) * (0.1 * float(r_dW.square().mean().sqrt()))
    got = []
    for forced in (False, True):
        ws = B.alloc_workspace(N, D, V)
        if forced:
            B.set_backward_tiling(4, 4)
            ws = B.alloc_workspace(N, D, V)
        into = before.clone() if form == "accumulate" else torch.full((V, D), float("nan"), device="cuda")
        try:
            if form == "shard":
                dH, dW = B.cce_shard_backward(H, W, y, lse, dl, v_off, v_total, IGN, label_smoothing=eps, z_loss=lam, workspace=ws, d_weight=into)
            else:
                dH, dW = B.cce_backward_ex(H, W, y, lse, None if mean else dl, IGN, label_smoothing=eps, z_loss=lam, workspace=ws, d_weight=into,
                                           accumulate_dw=form == "accumulate")
            torch.cuda.synchronize()
        finally:
            B.set_backward_tiling(0, 0)
        if form == "accumulate":
            dW = dW - before
        got.append((dH, dW))
        assert not dH[~valid].any()
        if valid.any():
            assert rel(dH, r_dH) <= 1e-2 and rel(dW, r_dW) <= 1e-2, (forced, rel(dH, r_dH), rel(dW, r_dW))
    assert rel(got[0][1], got[1][1]) <= 1e-5 and rel(got[0][0], got[1][0]) <= 1e-3, (rel(got[0][1], got[1][1]), rel(got[0][0], got[1][0]))


@pytest.mark.parametrize("D", [64, 128])
def test_ignored_rows_of_nan_have_zero_gradients(D):
    """dHidden alone: such rows meet dW's contraction, as they do over a chunk."""
    from paper_2601_02609_amd import binding as B
    N, V = 300, 700
    g = torch.Generator(device="cuda").manual_seed(D)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    y[::3] = IGN
    lse = torch.logsumexp(H.float() @ W.float().t(), 1)
    dl = torch.full((N,), 1.0 / N, device="cuda")
    ws = B.alloc_workspace(N, D, V)
    clean, _ = B.cce_backward(H, W, y, lse, dl, IGN, workspace=ws)
    H[::3] = float("nan")
    dH, _ = B.cce_backward(H, W, y, lse, dl, IGN, workspace=ws)
    torch.cuda.synchronize()
    assert not dH[::3].any() and torch.equal(dH, clean)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,V,mean,eps", [(301, 701, False, 0.0), (301, 701, False, 0.1), (1023, 259, True, 0.0), (9001, 9001, False, 0.0),
                                          (9001, 9001, False, 0.1)])
def test_rows_that_take_no_part_may_overflow(N, V, mean, eps, D):
    """Any finite hidden values, also such that a logit overflows fp32, in ignored rows and rows with a bad label, the last row among
    them (ragged tiles repeat it): the bits of the same call with those rows zero."""
    from paper_2601_02609_amd import binding as B
    print(f"[overflow] N={N} D={D} V={V} smoothing={eps}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + D)
    H = torch.randn(N, D, device="cuda", generator=g).bfloat16()
    W = (torch.randn(V, D, device="cuda", generator=g) * (2.5 / D ** 0.5)).bfloat16()
    y = torch.randint(0, V, (N,), device="cuda", generator=g, dtype=torch.int32)
    out = torch.rand(N, device="cuda", generator=g) < 0.2
    out[-1] = True
    y[out] = torch.tensor([IGN, V, -7], device="cuda", dtype=torch.int32)[torch.arange(int(out.sum()), device="cuda") % 3]
    H[out] = 0.0
    lse = torch.logsumexp(H.float() @ W.float().t(), 1)
    dl = torch.full((N,), 1.0 / N, device="cuda")
    ws = B.alloc_workspace(N, D, V)
    signs = torch.randint(0, 2, (int(out.sum()), D), device="cuda", generator=g).float().mul_(2.0).sub_(1.0) * 3e38
    assert not torch.isfinite(signs @ W.float().t()).all()
    got = []
    for rows in (torch.zeros_like(signs), signs):
        H[out] = rows.bfloat16()
        got.append(B.cce_backward_ex(H, W, y, lse, None if mean else dl, IGN, label_smoothing=eps, workspace=ws))
    torch.cuda.synchronize()
    (dH0, dW0), (dH, dW) = got
    assert torch.isfinite(dW).all() and torch.isfinite(dH.float()).all()
    assert torch.equal(dH, dH0) and torch.equal(dW, dW0) and not dH[out].any()
