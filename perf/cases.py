"""The work that the performance of this library is measured on: what a training or evaluation loop
has it do, through the public binding, from the smallest calls to the largest.

A case is a dict of plain values.  "path" says which entry points a pass goes through:

    step      cce_forward + cce_backward: one optimizer step's loss and gradients, every row computed
    compact   cce_forward_compact + cce_backward_compact: the loop knows its number of valid rows
    micro     cce_forward_ex + cce_backward_ex: one micro-batch of gradient accumulation (dW is added
              to), mean reduction, label smoothing and z-loss
    score     cce_forward_ex with the mean: evaluation (perplexity), no gradients
    fp8       quantisation of both operands, cce_fp8_forward + cce_fp8_backward
    shard     one device's share of a vocabulary-parallel step: its statistics, the merge with those of
              the other devices (already received), the backward of the share
    around    the steps in front of and behind the head: RMSNorm with residual add (forward, backward),
              gradient norm, clipping coefficient, AdamW with the bf16 copy

N tokens, D hidden size, V vocabulary; "ignore" is the fraction of rows whose label is the ignore
index (padding), "w_scale" / "zipf" the logit scale and the label distribution, as in inputs.py.
"""
from __future__ import annotations

import math

import torch

from paper_2601_02609_amd import binding as B

IGN = -100
DEV = "cuda"


def listed():
    return [
        # unit-test sized call: launches and latency are all there is
        dict(name="tiny", path="step", N=256, D=64, V=1000, ignore=0.10, w_scale=2.5, zipf=0.0, hidden="iid"),
        # one short fine-tuning sequence against a full vocabulary: few rows, W and dW dominate
        dict(name="short_sequence", path="step", N=509, D=896, V=151936, ignore=0.0, w_scale=2.5, zipf=1.1, hidden="rms"),
        # the headline training step (8 sequences of 1024, 15 % padding), all rows computed
        dict(name="headline", path="step", N=8192, D=896, V=151936, ignore=0.15, w_scale=2.5, zipf=1.1, hidden="rms"),
        # the same step by a loop that knows its padding
        dict(name="headline_compact", path="compact", N=8192, D=896, V=151936, ignore=0.15, w_scale=2.5, zipf=1.1, hidden="rms"),
        # packed sequences (no padding) of a 1B-class model
        dict(name="packed_1b", path="step", N=16384, D=2048, V=151936, ignore=0.0, w_scale=2.5, zipf=1.1, hidden="rms"),
        # 7B-class shape: the largest step
        dict(name="step_7b", path="step", N=32768, D=3584, V=151936, ignore=0.05, w_scale=2.5, zipf=1.1, hidden="rms"),
        # small vocabulary, wide hidden state, a quarter of the rows padding
        dict(name="small_vocab_compact", path="compact", N=16384, D=4096, V=32000, ignore=0.25, w_scale=3.0, zipf=1.3, hidden="rms"),
        # a ragged micro-batch of gradient accumulation with the loss variants
        dict(name="micro_batch", path="micro", N=3001, D=1024, V=50257, ignore=0.10, w_scale=2.5, zipf=1.1, hidden="rms"),
        # evaluation of an odd number of tokens
        dict(name="score", path="score", N=4099, D=2048, V=128256, ignore=0.05, w_scale=2.5, zipf=1.1, hidden="rms"),
        # the headline step with its logit products in FP8
        dict(name="headline_fp8", path="fp8", N=8192, D=896, V=151936, ignore=0.15, w_scale=2.5, zipf=1.1, hidden="rms"),
        # one of eight devices in a vocabulary-parallel headline step
        dict(name="shard_of_8", path="shard", N=8192, D=896, V=18992, parts=8, ignore=0.15, w_scale=2.5, zipf=1.1, hidden="rms"),
        # final norm and optimizer step of the headline head
        dict(name="around_the_head", path="around", N=8192, D=896, V=151936, ignore=0.0, w_scale=2.5, zipf=1.1, hidden="rms"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any path, sizes spread over their range (odd token counts and vocabularies as
    they come, D a multiple of the library's granule), at most about 4 TFLOP per logit product."""
    path = rng.choice(["step", "step", "step", "compact", "compact", "micro", "score", "fp8", "shard", "around"])
    granule = 128 if path == "fp8" else 64
    while True:
        N = _log_int(rng, 200, 32768)
        D = granule * max(1, round(_log_int(rng, 64, 4096) / granule))
        V = _log_int(rng, 1000, 151936)
        if 2.0 * N * D * V <= 4e12:
            break
    case = dict(path=path, N=N, D=D, V=V, ignore=rng.choice([0.0, 0.05, 0.1, 0.15, 0.25, 0.4]),
                w_scale=rng.choice([2.5, 3.0]), zipf=rng.choice([0.0, 1.1, 1.3]), hidden="rms")
    if path == "shard":
        case["parts"] = rng.choice([2, 4, 8])
    return case


# ------------------------------------------------------------------------------------------ inputs

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal_bf16(g, rows, cols, scale):
    """N(0, scale^2) in bf16, drawn in row blocks (bounds the fp32 temporary)."""
    out = torch.empty(rows, cols, dtype=torch.bfloat16, device=DEV)
    step = max(1, (1 << 28) // cols)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        out[r:r + n] = torch.randn(n, cols, device=DEV, generator=g).mul_(scale).bfloat16()
    return out


def _hidden(g, case):
    x = torch.randn(case["N"], case["D"], device=DEV, generator=g)
    if case["hidden"] == "rms":
        x /= x.square().mean(dim=1, keepdim=True).sqrt()
    return x.bfloat16()


def _labels(g, case, V):
    """Zipf (or uniform) labels over [0, V), a fixed number of scattered rows set to the ignore index."""
    N = case["N"]
    if case["zipf"] > 0.0:
        cdf = torch.arange(1, V + 1, dtype=torch.float64, device=DEV).pow_(-case["zipf"]).cumsum(0)
        u = torch.rand(N, dtype=torch.float64, device=DEV, generator=g) * cdf[-1]
        y = torch.searchsorted(cdf, u).clamp_(max=V - 1).int()
    else:
        y = torch.randint(0, V, (N,), device=DEV, generator=g, dtype=torch.int32)
    y[torch.randperm(N, device=DEV, generator=g)[:_n_ignored(case)]] = IGN
    return y


def _n_ignored(case):
    return int(round(case["ignore"] * case["N"]))


def _n_valid(case):
    return case["N"] - _n_ignored(case)


def prepare(case, seed):
    g = _generator(seed)
    N, D, V, path = case["N"], case["D"], case["V"], case["path"]
    s = dict(case=case)
    if path == "around":
        s.update(x=_hidden(g, case), residual=_hidden(g, case), gamma=(1.0 + 0.1 * torch.randn(D, device=DEV, generator=g)).bfloat16(),
                 dy=_normal_bf16(g, N, D, 1e-3))
        master = torch.randn(V * D, device=DEV, generator=g).mul_(case["w_scale"] / math.sqrt(D))
        s.update(master=master, weight=master.bfloat16(),
                 grad=torch.randn(V * D, device=DEV, generator=g).mul_(1e-4),
                 m=torch.randn(V * D, device=DEV, generator=g).mul_(1e-4),
                 v=torch.rand(V * D, device=DEV, generator=g).mul_(1e-8),
                 norm_ws=torch.empty(int(B.lib().cce_rmsnorm_workspace_bytes(N, D)), dtype=torch.uint8, device=DEV),
                 sum_ws=torch.empty(int(B.lib().cce_sumsq_workspace_bytes()), dtype=torch.uint8, device=DEV))
        return s
    v_total = V * case.get("parts", 1)
    s.update(H=_hidden(g, case), W=_normal_bf16(g, V, D, case["w_scale"] / math.sqrt(D)), y=_labels(g, case, v_total))
    if path == "compact":
        s["workspace"] = B.alloc_compact_workspace(N, D, V, _n_valid(case), DEV)
    else:
        s["workspace"] = B.alloc_workspace(N, D, V, DEV)
    if path in ("step", "compact", "fp8"):
        s["dloss"] = torch.full((N,), 1.0 / max(_n_valid(case), 1), device=DEV)       # mean over the valid rows
    if path != "score":
        s["dW"] = torch.zeros(V, D, dtype=torch.float32, device=DEV)                  # the parameter's gradient buffer
    if path == "micro":
        s["dW"] += torch.randn(V, D, device=DEV, generator=g).mul_(1e-5)              # what earlier micro-batches left
    if path == "shard":
        # what the other devices sent: (max, sum of exp(z - max), label logit or 0, unused) per token
        parts = case["parts"]
        stats = torch.zeros(parts, N, 4, device=DEV)
        sigma = case["w_scale"]
        stats[:, :, 0] = sigma * (math.sqrt(2.0 * math.log(max(V, 2))) + 0.3 * torch.randn(parts, N, device=DEV, generator=g))
        stats[:, :, 1] = V * torch.exp(0.5 * sigma * sigma - stats[:, :, 0])
        owner = torch.where(s["y"] >= 0, s["y"] // V, -1)
        z = sigma * torch.randn(N, device=DEV, generator=g)
        for p in range(parts):
            stats[p, :, 2] = torch.where(owner == p, z, torch.zeros_like(z))
        s["stats"] = stats
    return s


# ------------------------------------------------------------------------------------------ passes

def run(s):
    case = s["case"]
    path = case["path"]
    if path == "step":
        loss, lse = B.cce_forward(s["H"], s["W"], s["y"], IGN, workspace=s["workspace"])
        dH, dW = B.cce_backward(s["H"], s["W"], s["y"], lse, s["dloss"], IGN, workspace=s["workspace"], d_weight=s["dW"])
        return dict(loss=loss, lse=lse, dH=dH, dW=dW)
    if path == "compact":
        n = _n_valid(case)
        loss, lse = B.cce_forward_compact(s["H"], s["W"], s["y"], n, IGN, workspace=s["workspace"])
        dH, dW = B.cce_backward_compact(s["H"], s["W"], s["y"], lse, s["dloss"], n, IGN,
                                        workspace=s["workspace"], d_weight=s["dW"])
        return dict(loss=loss, lse=lse, dH=dH, dW=dW)
    if path == "micro":
        loss, lse, mean = B.cce_forward_ex(s["H"], s["W"], s["y"], IGN, label_smoothing=0.1, z_loss=1e-4, want_mean=True,
                                           workspace=s["workspace"])
        dH, dW = B.cce_backward_ex(s["H"], s["W"], s["y"], lse, None, IGN, label_smoothing=0.1, z_loss=1e-4,
                                   workspace=s["workspace"], d_weight=s["dW"], accumulate_dw=True)
        return dict(loss=loss, lse=lse, mean=mean, dH=dH, dW=dW)
    if path == "score":
        loss, lse, mean = B.cce_forward_ex(s["H"], s["W"], s["y"], IGN, want_mean=True, workspace=s["workspace"])
        return dict(loss=loss, lse=lse, mean=mean)
    if path == "fp8":
        hq, hs = B.cce_quantize_e4m3(s["H"])
        wq, ws = B.cce_quantize_e4m3(s["W"])
        loss, lse = B.cce_fp8_forward(hq, hs, wq, ws, s["y"], IGN, workspace=s["workspace"])
        dH, dW = B.cce_fp8_backward(hq, hs, wq, ws, s["H"], s["W"], s["y"], lse, s["dloss"], IGN,
                                    workspace=s["workspace"], d_weight=s["dW"])
        return dict(loss=loss, lse=lse, dH=dH, dW=dW)
    if path == "shard":
        V = case["V"]
        v_total = V * case["parts"]
        B.cce_shard_forward(s["H"], s["W"], s["y"], 0, stats=s["stats"][0], workspace=s["workspace"])
        loss, lse, mean = B.cce_shard_merge(s["stats"], s["y"], v_total, IGN, want_mean=True)
        dH, dW = B.cce_shard_backward(s["H"], s["W"], s["y"], lse, None, 0, v_total, IGN,
                                      workspace=s["workspace"], d_weight=s["dW"])
        return dict(loss=loss, lse=lse, mean=mean, dH=dH, dW=dW)
    y, rstd = B.cce_rmsnorm_residual_forward(s["x"], s["residual"], s["gamma"], 1e-6)
    dx, dgamma = B.cce_rmsnorm_residual_backward(s["residual"], s["gamma"], rstd, s["dy"], workspace=s["norm_ws"])
    sumsq = B.cce_grad_sumsq(s["grad"], workspace=s["sum_ws"])
    coef = B.cce_clip_coef(sumsq, 1.0)
    B.cce_adamw_step(s["master"], s["grad"], s["m"], s["v"], 100, lr=1e-3, weight_decay=0.1, param_bf16=s["weight"],
                     clip_coef=coef)
    return dict(h=s["residual"], y=y, rstd=rstd, dx=dx, dgamma=dgamma, sumsq=sumsq, coef=coef,
                master=s["master"], weight=s["weight"], m=s["m"], v=s["v"])


# ------------------------------------------------------------------------------------------ bounds

def work(case):
    """Each input read once, each output written once; the products of the rows that take part (the
    logits are formed twice because they are not kept: 2 + 2 NVD, and the two contractions 4 NVD)."""
    N, D, V, path = case["N"], case["D"], case["V"], case["path"]
    nvd = float(_n_valid(case)) * V * D
    if path == "around":
        # norm: x, residual read, h, y written; backward: h, dy read, dx written; optimizer: p, g, m, v
        # read, p, m, v and the bf16 copy written (the gradient once more for its norm)
        return dict(bytes=14.0 * N * D + 34.0 * V * D, flops=30.0 * V * D)
    if path == "score":
        return dict(bytes=2.0 * N * D + 2.0 * V * D + 12.0 * N, flops=2.0 * nvd)
    bytes_ = 4.0 * N * D + 6.0 * V * D + 16.0 * N
    if path == "micro":
        bytes_ += 4.0 * V * D
    return dict(bytes=bytes_, flops=8.0 * nvd)


def tolerance(case):
    """Measured against the same path in 64 bits: 1.9e-3 ... 3.4e-3 on the gradients (bf16 gradient
    tiles, bf16 dHidden), up to 9e-8 on loss and lse (fp32 sums).  Around the head: 1e-7 on the fp32
    results, and one unit in the last place (2^-8) of a few bf16 values, where another summation
    order rounds the other way: 1e-5 of the norm between two orders, 1.7e-3 to the unrounded result."""
    return {"step": {"rel": 1e-2}, "compact": {"rel": 1e-2}, "micro": {"rel": 1e-2}, "fp8": {"rel": 1e-2},
            "shard": {"rel": 1e-2}, "score": {"rel": 2e-6}, "around": {"rel": 1e-3}}[case["path"]]


# ------------------------------------------------------------------------------------------ in 64 bits

def _e4m3_values(x):
    """The float64 values that a bf16 matrix keeps after block-wise E4M3: blocks of 128 columns, the
    scale amax / 448 rounded up to a power of two, clamp, round to nearest even."""
    rows, cols = x.shape
    b = x.double().view(rows, cols // 128, 128)
    amax = b.abs().amax(dim=2, keepdim=True)
    e = torch.where(amax > 0, torch.ceil(torch.log2(amax / 448.0)), torch.zeros_like(amax)).clamp_(-127, 127)
    scale = torch.exp2(e)
    q = (b / scale).clamp_(-448.0, 448.0).float().to(torch.float8_e4m3fn)
    return (q.double() * scale).view(rows, cols)


def _row_blocks(W, values):
    """W in blocks of rows, each as float64 `values` of it and as plain float64."""
    for v0 in range(0, W.shape[0], 4096):
        w = W[v0:v0 + 4096]
        yield v0, values(w), w.double()


def exact(case, seed):
    """What run() returns for these inputs, in 64 bits throughout, vocabulary block by block."""
    if case["path"] == "around":
        return _exact_around(prepare(case, seed))
    s = prepare(case, seed)
    N, V, path = case["N"], case["V"], case["path"]
    values = _e4m3_values if path == "fp8" else torch.Tensor.double
    H, W, y = s["H"].double(), s["W"], s["y"].long()
    Hz = values(s["H"])
    V_total = V * case.get("parts", 1)
    eps, lam = (0.1, 1e-4) if path == "micro" else (0.0, 0.0)
    valid = y != IGN
    rows = torch.arange(N, device=DEV)

    m = torch.full((N,), -math.inf, dtype=torch.float64, device=DEV)
    d, zy, zsum = (torch.zeros(N, dtype=torch.float64, device=DEV) for _ in range(3))
    for v0, wz, _ in _row_blocks(W, values):
        z = Hz @ wz.t()
        mn = torch.maximum(m, z.amax(dim=1))
        d = d * torch.exp(m - mn) + torch.exp(z - mn[:, None]).sum(dim=1)
        m = mn
        zsum += z.sum(dim=1)
        here = (y >= v0) & (y < v0 + wz.shape[0])
        zy[here] = z[rows[here], y[here] - v0]
    if path == "shard":
        for other in s["stats"][1:].double():
            mn = torch.maximum(m, other[:, 0])
            d = d * torch.exp(m - mn) + other[:, 1] * torch.exp(other[:, 0] - mn)
            m, zy = mn, zy + other[:, 2]
    zero = torch.zeros_like(m)
    lse = torch.where(valid, m + torch.log(d), zero)
    loss = torch.where(valid, (1 - eps) * (lse - zy) + eps * (lse - zsum / V_total) + lam * lse * lse, zero)
    out = dict(loss=loss, lse=lse)
    n_valid = max(int(valid.sum()), 1)
    if path in ("micro", "score", "shard"):
        out["mean"] = loss.sum() / n_valid
    if path == "score":
        return out

    g_row = torch.where(valid, s["dloss"].double() if "dloss" in s else zero + 1.0 / n_valid, zero)
    dH = torch.zeros_like(H)
    dW = torch.empty(W.shape, dtype=torch.float64, device=DEV)
    for v0, wz, w in _row_blocks(W, values):
        g = torch.exp(Hz @ wz.t() - lse[:, None]) * (1 + 2 * lam * lse)[:, None] - eps / V_total
        here = (y >= v0) & (y < v0 + w.shape[0])
        g[rows[here], y[here] - v0] -= 1 - eps
        g *= g_row[:, None]
        dH += g @ w
        torch.mm(g.t(), H, out=dW[v0:v0 + w.shape[0]])
    if path == "micro":
        dW += s["dW"].double()
    out.update(dH=dH, dW=dW)
    return out


def _exact_around(s):
    eps, lr, wd, b1, b2, adam_eps, t = 1e-6, 1e-3, 0.1, 0.9, 0.999, 1e-8, 100
    h = s["x"].double() + s["residual"].double()
    hb, gamma, dy = h.float().bfloat16().double(), s["gamma"].double(), s["dy"].double()    # the norm acts on the stored bf16 sum
    rstd = (hb.square().mean(dim=1) + eps).rsqrt()
    xhat = hb * rstd[:, None]
    dx = rstd[:, None] * (dy * gamma - xhat * (dy * gamma * xhat).mean(dim=1, keepdim=True))
    g = s["grad"].double()
    sumsq = g.square().sum()
    coef = torch.clamp(1.0 / (sumsq.sqrt() + 1e-6), max=1.0)
    g *= coef
    m = b1 * s["m"].double() + (1 - b1) * g
    v = b2 * s["v"].double() + (1 - b2) * g * g
    p = s["master"].double() * (1 - lr * wd)
    p -= lr * (m / (1 - b1 ** t)) / ((v / (1 - b2 ** t)).sqrt() + adam_eps)
    return dict(h=h, y=xhat * gamma, rstd=rstd, dx=dx, dgamma=(dy * xhat).sum(dim=0), sumsq=sumsq, coef=coef,
                master=p, weight=p, m=m, v=v)
