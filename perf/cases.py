"""What a user of the Skiparse-2D attention library has it do, as cases that can be timed.

A case is one call sequence ("path") on one shape:

  layer      one sparse attention block in inference: q, k, v and the result in the original token order
  dense      one full-attention block of a hybrid stack
  train      forward that keeps the log-sum-exp, then dq, dk, dv
  chain      the first block of a chain of sparse blocks: q, k, v rearranged once, the result in the next block's layout
  fp8        the 8-bit block: q, k, v quantised while they are rearranged, attention on the codes
  rearrange  a hidden state into one pattern's layout, switched to the other's, and back to the original order

Shapes are token grids (T, H, W) of latent video (21 frames) or single images, with `heads` heads of `head_dim` channels, the sparse
ratio `s` and the pattern.  `pad` is the any-resolution mode, `fused` the layer without permuted copies, `qk_norm` the values of a
model that normalises q and k per head.
"""
from __future__ import annotations

import math

import torch

import paper_2605_28691_amd as sk

PATHS = ("layer", "dense", "train", "chain", "fp8", "rearrange")


def _case(name, path, B, heads, head_dim, T, H, W, s=2, pattern="token", pad=False, fused=True, qk_norm=False):
    c = dict(path=path, B=B, heads=heads, head_dim=head_dim, T=T, H=H, W=W, s=s, pattern=pattern, pad=pad, fused=fused, qk_norm=qk_norm)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest layer of the tests: launch and call latency, nothing else
        _case("tiny_layer", "layer", 1, 2, 64, 2, 8, 8),
        # a training step on a short clip of small frames, as in the first minutes of bringing a model up: 400 tokens a subsequence
        _case("small_train", "train", 1, 12, 128, 5, 16, 20, pattern="group"),
        # one image at 480x832 through a 12-head block (image batches of a joint image/video model), rows of 52 tokens
        _case("image_480p_layer", "layer", 1, 12, 128, 1, 30, 52, qk_norm=True),
        # one image at 768x1280 in training, 40 heads
        _case("image_768p_train", "train", 1, 40, 128, 1, 48, 80, pattern="group"),
        # odd sizes: two short clips on a ragged grid, head_dim 64, any-resolution mode, 8-bit
        _case("ragged_fp8", "fp8", 2, 16, 64, 9, 17, 21, pattern="group", pad=True),
        # an 81-frame 480x832 video through a 12-head block
        _case("video_480p_layer", "layer", 1, 12, 128, 21, 30, 52, qk_norm=True),
        # the same in training
        _case("video_480p_train", "train", 1, 12, 128, 21, 30, 52, qk_norm=True),
        # an 81-frame 768x1280 video, hidden state of 5120 channels moved between the layouts
        _case("video_768p_rearrange", "rearrange", 1, 40, 128, 21, 48, 80),
        # the same video through a 12-head chain of sparse blocks
        _case("video_768p_chain", "chain", 1, 12, 128, 21, 48, 80),
        # the same video in 8 bits, 40 heads
        _case("video_768p_fp8", "fp8", 1, 40, 128, 21, 48, 80, pattern="group"),
        # an 81-frame 720x1280 video in training: 45 rows padded to 48, masked
        _case("video_720p_train", "train", 1, 40, 128, 21, 45, 80, pad=True),
        # a full-attention block of the hybrid stack at 768x1280: the largest call
        _case("video_768p_dense", "dense", 1, 40, 128, 21, 48, 80, s=1),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    most = 1.4e14  # operations of the largest listed case
    while True:
        path = rng.choice(("layer", "layer", "train", "train", "chain", "fp8", "rearrange", "dense"))
        s = 1 if path == "dense" else rng.choice((2, 2, 2, 2, 3, 4))
        pattern = rng.choice(("token", "group"))
        pad = path in ("layer", "train", "fp8") and rng.random() < 0.35
        # the other pattern's layout exists on multiples of s*s only
        unit = 1 if pad or path == "dense" else s * s if pattern == "group" or path in ("chain", "rearrange") else s
        T = rng.choice((1, 21, _log_int(rng, 2, 21)))  # an image, an 81-frame video, a clip
        H = max(1, round(_log_int(rng, 8, 48) / unit)) * unit
        W = max(1, round(_log_int(rng, 8, 80) / unit)) * unit
        c = _case(None, path, rng.choice((1, 1, 1, 2, 3)), _log_int(rng, 1, 40), rng.choice((128, 128, 128, 64)), T, H, W, s, pattern, pad,
                  fused=path != "layer" or pad or rng.random() < 0.8, qk_norm=rng.random() < 0.3)
        if work(c)["flops"] <= most and c["B"] * T * H * W * c["heads"] * c["head_dim"] <= 21 * 48 * 80 * 40 * 128:
            return c


def _randn(shape, gen):
    """N(0,1) in bf16, made a batch element at a time so that the float32 original stays small."""
    return torch.stack([torch.randn(shape[1:], generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16) for _ in range(shape[0])])


def _normed(x, gen):
    """Zero mean and unit variance per token and head, times a gain per head in [1/2, 2]: what a per-head norm of q and k leaves."""
    f = x.float()
    f = f - f.mean(dim=-1, keepdim=True)
    f = f / f.std(dim=-1, keepdim=True, unbiased=False)
    gain = torch.pow(2.0, torch.rand((x.shape[2], 1), generator=gen, device="cuda") * 2.0 - 1.0)
    return (f * gain).to(torch.bfloat16)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    shape = (case["B"], case["T"] * case["H"] * case["W"], case["heads"], case["head_dim"])
    state = {"case": case, "q": _randn(shape, gen)}
    if case["path"] == "rearrange":
        return state  # the hidden state
    state["k"], state["v"] = _randn(shape, gen), _randn(shape, gen)
    if case["qk_norm"]:
        state["q"], state["k"] = _normed(state["q"], gen), _normed(state["k"], gen)
    if case["path"] == "train":
        state["dout"] = _randn(shape, gen)
    return state


def run(state):
    c = state["case"]
    grid, path, pad = (c["T"], c["H"], c["W"]), c["path"], c["pad"]
    at = (*grid, c["s"], c["pattern"])
    q = state["q"]
    if path == "rearrange":
        y = sk.skiparse_permute(q, *at)
        z = sk.skiparse_switch_pattern(y, *at)
        return y, z, sk.skiparse_unpermute(z, *grid, c["s"], "group" if c["pattern"] == "token" else "token")
    k, v = state["k"], state["v"]
    if path == "layer":
        return sk.skiparse_attn_fwd(q, k, v, *at, fused=c["fused"], pad=pad)
    if path == "dense":
        return sk.dense_attn_fwd(q, k, v, *grid)
    if path == "train":
        out, lse = sk.skiparse_attn_fwd_lse(q, k, v, *at, pad=pad)
        return (out, *sk.skiparse_attn_bwd(q, k, v, out, state["dout"], lse, *at, pad=pad))
    if path == "chain":
        qs, ks, vs = (sk.skiparse_permute(t, *at) for t in (q, k, v))
        return sk.skiparse_attn_fwd_sparse(qs, ks, vs, *at, out_layout="other")
    (q8, sq), (k8, sk_), (v8, sv) = (sk.skiparse_quantize_fp8(t, *at, pad=pad) for t in (q, k, v))
    return sk.skiparse_attn_fwd_fp8(q8, k8, v8, sq, sk_, sv, *at, pad=pad)


def _real_pairs(case):
    """Sum over the subsequences of one batch element of (real tokens)^2: the query-key pairs of one head."""
    T, H, W, s = case["T"], case["H"], case["W"], case["s"]
    step = s if case["pattern"] == "group" else 1

    def per_class(n):
        return [sum(1 for x in range(n) if (x // step) % s == p) for p in range(s)]

    return sum((T * a * b) ** 2 for a in per_class(H) for b in per_class(W))


def work(case):
    """Bytes and operations of one pass that no implementation can do without: every input read once, every result written once; the
    products of attention over the real tokens (2 forward, 5 backward)."""
    tokens = case["B"] * case["T"] * case["H"] * case["W"]
    tensor = 2 * tokens * case["heads"] * case["head_dim"]
    if case["path"] == "rearrange":
        return {"bytes": 4 * tensor, "flops": 0}
    product = 2.0 * case["B"] * case["heads"] * case["head_dim"] * _real_pairs(case)
    if case["path"] == "train":
        return {"bytes": 8 * tensor, "flops": 7 * product}
    return {"bytes": 4 * tensor, "flops": 2 * product}


def tolerance(case):
    if case["path"] == "rearrange":
        return "exact"  # rows are moved
    # Against the same quantities in 64 bits, measured on the small shapes of every path: 2.3e-3 (bf16 probabilities and results), 2.5e-3
    # for the gradients, 2.6e-2 for the 8-bit path on its own codes (probabilities rounded to three mantissa bits).
    return {"rel": 1e-1} if case["path"] == "fp8" else {"rel": 1e-2}


def _rows_of_classes(T, H, W, s, step):
    """Token numbers of every class (p, q), p slow, in raster order; a class of the token-wise pattern has step 1, of the group-wise s."""
    n = torch.arange(T * H * W, device="cuda").view(T, H, W)
    h, w = torch.arange(H, device="cuda"), torch.arange(W, device="cuda")
    return [n[:, h // step % s == p][:, :, w // step % s == q].reshape(-1) for p in range(s) for q in range(s)]


def exact(case, seed):
    """What run() returns, in 64 bits and plain torch: attention inside every class, its gradients by the textbook formulas.  The 8-bit
    path is held against attention on the tensors before they are quantised."""
    state = prepare(case, seed)
    T, H, W, s, path = case["T"], case["H"], case["W"], case["s"], case["path"]
    step = s if case["pattern"] == "group" else 1
    if path == "rearrange" or work(case)["flops"] > 4e13:
        return None  # rows that are moved; over about 20 seconds
    q, k, v = state["q"], state["k"], state["v"]
    out = torch.zeros(q.shape, dtype=torch.float64, device="cuda")
    grads = [torch.zeros_like(out) for _ in range(3)] if path == "train" else []
    scale = q.shape[3] ** -0.5
    for rows in _rows_of_classes(T, H, W, s, step):
        for b in range(q.shape[0]):
            for a in range(q.shape[2]):
                if not rows.numel():
                    continue
                qd, kd, vd = (t[b, rows, a].double() for t in (q, k, v))
                kt, vt = kd.t().contiguous(), vd.t().contiguous()
                od = torch.empty_like(qd)
                dq, dk, dv = torch.empty_like(qd), torch.zeros_like(kd), torch.zeros_like(vd)
                chunk = max(1, (1 << 27) // rows.numel())
                for i in range(0, rows.numel(), chunk):
                    prob = torch.softmax((qd[i : i + chunk] @ kt) * scale, dim=1)
                    od[i : i + chunk] = prob @ vd
                    if grads:
                        do = state["dout"][b, rows[i : i + chunk], a].double()
                        dv += prob.t().contiguous() @ do
                        ds = prob * (do @ vt - (do * od[i : i + chunk]).sum(dim=1, keepdim=True))
                        dq[i : i + chunk] = (ds @ kd) * scale
                        dk += (ds.t().contiguous() @ qd[i : i + chunk]) * scale
                out[b, rows, a] = od
                for grad, part in zip(grads, (dq, dk, dv)):
                    grad[b, rows, a] = part
    if path == "chain":  # the other pattern's layout: subsequences slow, batch fast
        other = _rows_of_classes(T, H, W, s, 1 if step == s else s)
        return torch.cat([out[:, rows] for rows in other])
    return (out, *grads) if path == "train" else out
