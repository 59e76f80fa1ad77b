"""The workloads that this library's speed is judged by.

MonarchAttention is called in four ways by a program that uses it: the forward
pass on whole sequences (`monarch_attn_fwd`), the same on a padded batch of
sequences of different lengths (`monarch_attn_fwd_varlen`), and a training
step of either, forward and gradient through torch's autograd
(`monarch_attention_autograd`).  The listed cases are the model conversions
that the repository's inputs name (ViT-B/16, DiT-XL/2, RoBERTa-base, BART-base,
a graph transformer) and the points of its long-sequence benchmark, from 16
heads of 256 tokens to 16 heads of 16384.  `draw` spreads over the same
ranges: block counts and block sizes from 4 to 128, sequences that do not fill
their last block, head dimensions 32 to 128, 1 to 3 steps, bf16, fp16 and fp32.

A case: kind (fwd, varlen, train, train_varlen), B, H, N, m, b, d, T, dtype,
inputs (vit, lm or speed: how Q and K are drawn) and, for padded batches, the
shortest length `low`.
"""
import math

import torch

import paper_2505_18698_amd as ma

_DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def _case(name, kind, B, H, N, m, b, d, T, dtype, inputs, low=0):
    return {"name": name, "kind": kind, "B": B, "H": H, "N": N, "m": m, "b": b, "d": d, "T": T, "dtype": dtype,
            "inputs": inputs, "low": low}


def listed():
    return [
        # One short sequence, 16 heads: a single request, where launches and latency count.
        _case("fwd_n256", "fwd", 1, 16, 256, 16, 16, 64, 2, "bf16", "speed"),
        # ViT-B/16 with its class token, 32 images: many small ragged heads (the last block is short).
        _case("fwd_vit_n197", "fwd", 32, 12, 197, 15, 14, 64, 2, "bf16", "vit"),
        # DiT-XL/2 at 256 x 256, 32 images: the denoiser's attention, a head dimension of 72, three steps.
        _case("fwd_dit_n256", "fwd", 32, 16, 256, 16, 16, 72, 3, "bf16", "vit"),
        # RoBERTa-base on 1024 tokens, a batch of 16 full sequences: medium blocks, many heads.
        _case("fwd_roberta_n1024", "fwd", 16, 12, 1024, 32, 32, 64, 2, "bf16", "lm"),
        # RoBERTa-base on question answering: 16 sequences of 64 to 384 tokens padded to 384.
        _case("varlen_roberta_n384", "varlen", 16, 12, 384, 16, 24, 64, 1, "bf16", "lm", 64),
        # BART-base encoder on one document of 2048 tokens in fp16: few heads, rectangular blocks.
        _case("fwd_bart_n2048_f16", "fwd", 1, 12, 2048, 64, 32, 64, 2, "f16", "lm"),
        # The 4K point of the benchmark: 16 heads, one step.
        _case("fwd_n4096", "fwd", 1, 16, 4096, 64, 64, 64, 1, "bf16", "speed"),
        # The 16K point, the headline: 16 heads, two steps, the largest forward call.
        _case("fwd_n16384", "fwd", 1, 16, 16384, 128, 128, 64, 2, "bf16", "speed"),
        # Fine-tuning a converted ViT-B/16: forward and gradient of the same small ragged heads.
        _case("train_vit_n197", "train", 32, 12, 197, 15, 14, 64, 2, "bf16", "vit"),
        # Fine-tuning RoBERTa-base on a padded batch, blocks of 48 rows.
        _case("train_varlen_roberta_n384", "train_varlen", 16, 12, 384, 8, 48, 64, 1, "bf16", "lm", 64),
        # A graph transformer on 7600 nodes trained in fp32: 4 heads of 48, the last block short.
        _case("train_gps_n7600_f32", "train", 1, 4, 7600, 60, 128, 48, 2, "f32", "vit"),
        # Long-context training at 16K: the largest call.
        _case("train_n16384", "train", 1, 16, 16384, 128, 128, 64, 2, "bf16", "speed"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _tile(rows):
    return 16 if rows <= 16 else 32 if rows <= 32 else 64 if rows <= 64 else 128


def draw(rng):
    kind = rng.choice(("fwd", "fwd", "varlen", "train", "train", "train_varlen"))
    dtype = rng.choice(("bf16", "bf16", "bf16", "f16", "f32"))
    while True:
        m, b = _log_int(rng, 4, 128), _log_int(rng, 4, 128)
        d = rng.choice((32, 48, 64, 64, 64, 72, 80, 96, 128))
        width = 64 if d <= 64 else 96 if d <= 96 else 128
        if dtype != "f32" or max(_tile(m), _tile(b)) * width <= 8192:
            break
    N = m * b if rng.random() < 0.4 else rng.randint((m - 1) * b + 1, m * b)
    case = _case("", kind, 1, 1, N, m, b, d, rng.choice((1, 2, 2, 3)), dtype, rng.choice(("vit", "lm", "speed")),
                 max(1, N // 6) if "varlen" in kind else 0)
    del case["name"]
    # As many heads as cost at most half of the largest listed case, and at most 512.
    top, one = work(listed()[-1]), work(case)
    most = min(0.5 * top["bytes"] / one["bytes"], 0.5 * top["flops"] / one["flops"], 512)
    heads = _log_int(rng, 4, max(4, int(most)))
    case["H"] = rng.choice([h for h in (4, 6, 8, 12, 16) if h <= heads])
    case["B"] = max(1, heads // case["H"])
    return case


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32)


def _rotary(x):
    n, d = x.shape[-2:]
    p = torch.arange(n, device=x.device, dtype=torch.float64)[:, None]
    r = torch.arange(d // 2, device=x.device, dtype=torch.float64)[None, :]
    ang = p * 10000.0 ** (-2.0 * r / d)
    c, s = ang.cos().float(), ang.sin().float()
    x0, x1 = x[..., 0::2], x[..., 1::2]
    return torch.stack((x0 * c - x1 * s, x0 * s + x1 * c), dim=-1).flatten(-2)


def _inputs(case, seed):
    """q, k, v, dout and lens: float tensors of the case's type, lens an int32 tensor (None without padding).

    vit:   K = Z, Q = 0.7 Z + 0.7 E: the peaky attention of a trained ViT.
    lm:    the same plus a vector shared by all positions of a head, then a
           rotary phase, so that scores decay with the distance.
    speed: iid, scaled so that the largest softmax weight of a row is about
           0.1 on average.
    """
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, H, N, d = (case[x] for x in "BHNd")
    dt = _DTYPES[case["dtype"]]
    v, dout = _randn(gen, B, H, N, d), _randn(gen, B, H, N, d)
    z, e = _randn(gen, B, H, N, d), _randn(gen, B, H, N, d)
    if case["inputs"] == "speed":
        alpha = 1.23 + 0.073 * math.log2(max(N, 64) / 256)
        q, k = alpha * e, alpha * z
    else:
        q, k = 0.7 * z + 0.7 * e, z
        if case["inputs"] == "lm":
            u = _randn(gen, B, H, 1, d)
            q, k = _rotary(q + u), _rotary(k + u)
    lens = None
    if case["low"]:
        lens = torch.randint(case["low"], N + 1, (B,), generator=gen, device="cuda", dtype=torch.int32)
    return tuple(x.to(dt).contiguous() for x in (q, k, v, dout)) + (lens,)


def prepare(case, seed):
    q, k, v, dout, lens = _inputs(case, seed)
    state = {"kind": case["kind"], "shape": (case["m"], case["b"], case["T"]), "lens": lens}
    if case["kind"].startswith("train"):
        state["qkv"] = tuple(x.requires_grad_() for x in (q, k, v))
        state["dout"] = dout
    else:
        state["qkv"] = (q, k, v)
        state["out"] = torch.empty_like(q)
    return state


def run(state):
    q, k, v = state["qkv"]
    m, b, T = state["shape"]
    kind, lens = state["kind"], state["lens"]
    if kind == "fwd":
        return ma.monarch_attn_fwd(q, k, v, state["out"], m, b, T)
    if kind == "varlen":
        return ma.monarch_attn_fwd_varlen(q, k, v, state["out"], lens, m, b, T)
    out = ma.monarch_attention_autograd(q, k, v, m, b, T, lens)
    dq, dk, dv = torch.autograd.grad(out, (q, k, v), state["dout"])
    return out.detach(), dq, dk, dv


def work(case):
    """Every tensor once; the products of the forward pass (two per update and
    Y) and, for a training step, of its gradient (each update's scores and four
    products of their gradients, and two more with V and Y)."""
    heads, N, d, m, b, T = (case[x] for x in ("H", "N", "d", "m", "b", "T"))
    heads *= case["B"]
    size = 4 if case["dtype"] == "f32" else 2
    train = case["kind"].startswith("train")
    real = (case["low"] + N) / (2 * N) if case["low"] else 1.0  # share of the rows that are real, on average
    tensors = (4 + 4 * real) if train else (1 + 3 * real)
    flops = 2 * N * d * (T * 2 * (m + b) + b)
    if train:
        flops += 2 * N * d * (T * 5 * (m + b) + 2 * b)
    return {"bytes": heads * N * d * size * tensors, "flops": heads * flops}


def tolerance(case):
    # About four times the largest error against 64 bits that the path shows
    # over the listed and some hundred drawn cases.  16-bit types round the
    # states between the half-steps, and every step carries the rounding of the
    # ones before it.
    train = case["kind"].startswith("train")
    if case["dtype"] == "f32":
        return {"rel": 3e-5 if train else 1e-5}
    if case["dtype"] == "f16":
        return {"rel": 4e-3}
    return {"rel": 4e-2 if train else 2.5e-2}


def _exact_heads(q, k, v, n, m, b, T):
    """The T-step forward pass of heads [h, N, d] of which n rows are real, in 64 bits: eqs. R_update, L_update."""
    h, N, d = q.shape
    keep = (torch.arange(m * b, device=q.device) < n)
    pad = torch.zeros(h, m * b - N, d, device=q.device, dtype=q.dtype)
    q, k, v = (torch.where(keep[:, None], torch.cat((x, pad), 1), 0.0) for x in (q, k, v))
    kb, vb = k.view(h, m, b, d), v.view(h, m, b, d)
    qb = q.view(h, m, b, d).transpose(1, 2)  # Qbar[j][l] = Q[l b + j]
    keys = keep.view(m, 1, b)
    live = keys.any(-1)  # [m, 1]: blocks with a real key
    s = 1.0 / math.sqrt(d)
    aR, cR = q.view(h, m, b, d), torch.ones(h, m, b, device=q.device, dtype=q.dtype)
    for t in range(T):
        z = s * torch.matmul(aR, kb.transpose(2, 3)) / cR[..., None]
        z = torch.where(live[..., None], torch.where(keys, z, -math.inf), 0.0)
        logr = torch.log_softmax(z, dim=-1)
        R = torch.where(keys, logr.exp(), 0.0)
        cL = (R * torch.where(keys, logr, 0.0)).sum(-1)
        aL = torch.matmul(R, kb)  # [h, m, b, d]
        z = s * torch.matmul(qb, aL.permute(0, 2, 3, 1)) - cL.permute(0, 2, 1)[:, :, None, :]  # [h, j, l, k]
        L = torch.softmax(torch.where(live[:, 0], z, -1e300), dim=-1)
        L = torch.where(live[:, 0], L, 0.0)
        cR = torch.where(live, L.sum(2).permute(0, 2, 1), 1.0)
        aR = torch.matmul(L.transpose(2, 3), qb).permute(0, 2, 1, 3)
    Y = torch.matmul(R, vb)
    O = torch.matmul(L, Y.transpose(1, 2))  # [h, j, l, d]
    O = O.transpose(1, 2).reshape(h, m * b, d)
    return torch.where(keep[:, None], O, 0.0)[:, :N]


def exact(case, seed):
    q, k, v, dout, lens = _inputs(case, seed)
    train = case["kind"].startswith("train")
    B, H, N, d, m, b, T = (case[x] for x in ("B", "H", "N", "d", "m", "b", "T"))
    outs = [torch.empty(B * H, N, d, device=q.device, dtype=torch.float64) for _ in range(4 if train else 1)]
    lens = [N] * B if lens is None else lens.tolist()
    # a batch element's heads share their length; heads in parts of about 1 GB
    part = max(1, min(B * H, int(2e6 * 40 / (m * b * (m + b) * T))))
    for i in range(B):
        n = lens[i]
        if n == N and case["low"] == 0:
            if i:
                break
            first, last = 0, B * H  # no padding: all heads alike
        else:
            first, last = i * H, (i + 1) * H
        for h in range(first, last, part):
            sl = slice(h, min(last, h + part))
            x = [t.reshape(B * H, N, d)[sl].double().requires_grad_(train) for t in (q, k, v)]
            o = _exact_heads(*x, n, m, b, T)
            outs[0][sl] = o.detach()
            if train:
                for dst, g in zip(outs[1:], torch.autograd.grad(o, x, dout.view(B * H, N, d)[sl].double())):
                    dst[sl] = g
    outs = [o.view(B, H, N, d) for o in outs]
    return tuple(outs) if train else outs[0]
