"""Timed cases of tile-sparse 3D attention: what a program that uses this package calls,
from single small calls to full video lengths, forward and gradients.

A case is a dict of plain values:
  name   (listed cases only)
  op     "fwd"       tile_attn, the torch wrapper: out = attention under one shared mask
         "dense"     dense_attn, the torch wrapper of the full-mask control
         "heads"     tile_attn_fwd_heads: one mask per head, and the row log-sum-exp
         "noalloc"   tile_attn_fwd_heads_noalloc: the same call without device allocation
         "mmdit"     tile_attn_fwd_mmdit: P text tokens before the video, and the log-sum-exp
         "bwd"       tile_attn_bwd: dq, dk, dv from the forward's out and log-sum-exp
         "bwd_mmdit" tile_attn_bwd_mmdit: the same for the MM-DiT form
  B, H, F, T, d, P    batch, heads, latent frames, tokens per frame, head dim, text tokens
  form, g             mask family: "col", "sym" or "dense", with g global frames
  dist                "iid" or "frame_shift" (tokens of a frame share a mean)

The sizes are those of workloads.py (720p: 45 x 80 = 3600 tokens per latent frame, 29 and
93 input frames -> 8 and 24 latent frames; 30 x 40 grids; the CogVideoX-5B shape), one GPU's
share of the heads, and the small odd shapes of the tests.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2502_06155_amd as ta


def _case(op, B, H, F, T, d, form, g, P=0, dist="iid", name=None):
    c = {"op": op, "B": B, "H": H, "F": F, "T": T, "d": d, "P": P, "form": form, "g": g, "dist": dist}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # The smallest problem anyone runs (an 8 x 8 latent grid): one call's latency.
        _case("fwd", 1, 2, 4, 64, 64, "col", 1, name="fwd-tiny"),
        # One 29-frame 720p attention layer, the full-mask control every sparse speed-up
        # is quoted against (a teacher's layer).
        _case("dense", 1, 24, 8, 3600, 96, "dense", 0, name="fwd-29f-dense"),
        # The headline: one 93-frame 720p layer of the sparse student, diagonal + 1 global.
        _case("fwd", 1, 24, 24, 3600, 96, "col", 1, name="fwd-93f-col"),
        # One GPU's share (a quarter of the heads) of that layer with the masks of a
        # layer-wise search, one per head, on frame-correlated tokens, as a training step
        # runs it (with the log-sum-exp).
        _case("heads", 1, 6, 24, 3600, 96, "sym", 2, dist="frame_shift", name="fwd-share-heads"),
        # A long, low-resolution video: many short frames.
        _case("fwd", 1, 24, 48, 1200, 96, "sym", 2, name="fwd-long-sym"),
        # The 93-frame layer with 128-wide heads.
        _case("fwd", 1, 18, 24, 3600, 128, "col", 1, name="fwd-93f-d128"),
        # A CogVideoX-5B layer: 226 text tokens, ragged frames (1350 tokens), 64-wide heads.
        _case("mmdit", 1, 48, 13, 1350, 64, "sym", 1, P=226, name="fwd-cog-sym"),
        # Gradients of a small odd shape (a unit test's or a toy training step's).
        _case("bwd", 2, 4, 5, 257, 96, "col", 1, name="bwd-small"),
        # Gradients of the 29-frame layer under the paper's 1:7 mask.
        _case("bwd", 1, 24, 8, 3600, 96, "sym", 1, name="bwd-29f-sym"),
        # Gradients of the headline layer: the student's training step.
        _case("bwd", 1, 24, 24, 3600, 96, "col", 1, name="bwd-93f-col"),
        # The same with 128-wide heads.
        _case("bwd", 1, 18, 24, 3600, 128, "col", 1, name="bwd-93f-d128"),
        # Gradients of the CogVideoX-5B layer.
        _case("bwd_mmdit", 1, 48, 13, 1350, 64, "sym", 2, P=226, name="bwd-cog-sym"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: every entry point, head dim and mask family,
    frames of 33 to 3700 tokens (odd ones among them), 2 to 48 frames, 1 to 48 heads."""
    while True:
        op = rng.choice(["fwd", "fwd", "dense", "heads", "noalloc", "mmdit", "bwd", "bwd", "bwd_mmdit"])
        d = rng.choice([64, 96, 128])
        F = _log_int(rng, 2, 48)
        T = _log_int(rng, 33, 3700)
        H = _log_int(rng, 1, 48)
        B = rng.choice([1, 1, 1, 2, 3])
        form = "dense" if op == "dense" else rng.choice(["col", "sym"])
        g = 0 if op == "dense" else rng.randint(1, max(1, min(F - 1, 8)))
        P = _log_int(rng, 5, 1000) if op in ("mmdit", "bwd_mmdit") else 0
        dist = rng.choice(["iid", "iid", "frame_shift"])
        case = _case(op, B, H, F, T, d, form, g, P=P, dist=dist)
        # At most half of the largest listed case's operations (the least efficient shapes
        # then still cost no more than it does), and not below a tiny call's.
        if 5e7 <= work(case)["flops"] <= 7e12:
            return case


def _masks(case):
    """F x F, or H x F x F for the per-head entry points: head h keeps g, then 1, then
    2 g global frames, in turn in the case's form and the other one."""
    F, g, form = case["F"], case["g"], case["form"]
    if case["op"] not in ("heads", "noalloc"):
        return ta.tile_attn_make_mask(F, g, form)
    other = {"col": "sym", "sym": "col", "dense": "dense"}[form]
    kinds = [(g, form), (1, form), (min(F, 2 * g), other)]
    return np.stack([ta.tile_attn_make_mask(F, *kinds[h % 3]) for h in range(case["H"])])


def _inputs(case, seed, n):
    """n bf16 [B, H, P + F T, d] tensors of N(0, 1), as normalised queries, keys, values and
    upstream gradients are; frame_shift adds 0.5 N(0, I_d) per tensor, head and frame to
    the first three."""
    gen = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17)
    B, H, F, T, d, P = (case[k] for k in ("B", "H", "F", "T", "d", "P"))
    out = []
    for i in range(n):
        x = torch.randn((B, H, P + F * T, d), generator=gen, device="cuda", dtype=torch.float32)
        if case["dist"] == "frame_shift" and i < 3:
            mu = torch.randn((B, H, F, 1, d), generator=gen, device="cuda", dtype=torch.float32)
            x[:, :, P:].view(B, H, F, T, d).add_(mu, alpha=0.5)
        out.append(x.to(torch.bfloat16))
    return out


def _lse(case):
    return torch.empty((case["B"], case["H"], case["P"] + case["F"] * case["T"]), dtype=torch.float32,
                       device="cuda")


def _forward(case, q, k, v, out, lse, masks):
    dims = [case[x] for x in ("B", "H", "F", "T")]
    scale, stream = case["d"] ** -0.5, torch.cuda.current_stream()
    if case["P"]:
        ta.tile_attn_fwd_mmdit(q, k, v, out, *dims, case["P"], case["d"], masks, scale, lse, stream)
    elif case["op"] == "noalloc":
        ta.tile_attn_fwd_heads_noalloc(q, k, v, out, *dims, case["d"], masks, scale, lse, stream)
    else:
        ta.tile_attn_fwd_heads(q, k, v, out, *dims, case["d"], masks, scale, lse, stream)


def prepare(case, seed):
    masks = _masks(case)
    bwd = case["op"] in ("bwd", "bwd_mmdit")
    q, k, v, *rest = _inputs(case, seed, 4 if bwd else 3)
    st = {"case": case, "masks": masks, "q": q, "k": k, "v": v}
    if case["op"] in ("heads", "noalloc", "mmdit") or bwd:
        st["out"], st["lse"] = torch.empty_like(q), _lse(case)
    if bwd:  # a training step's forward has run: its output and log-sum-exp are in hand
        _forward(case, q, k, v, st["out"], st["lse"], masks)
        st["dout"] = rest[0]
        st["grads"] = [torch.empty_like(q) for _ in range(3)]
    return st


def run(state):
    case, masks = state["case"], state["masks"]
    q, k, v = state["q"], state["k"], state["v"]
    op, T = case["op"], case["T"]
    if op == "fwd":
        return {"out": ta.tile_attn(q, k, v, masks, T)}
    if op == "dense":
        return {"out": ta.dense_attn(q, k, v, T)}
    if op in ("heads", "noalloc", "mmdit"):
        _forward(case, q, k, v, state["out"], state["lse"], masks)
        return {"out": state["out"], "lse": state["lse"]}
    dims = [case[x] for x in ("B", "H", "F", "T")]
    dq, dk, dv = state["grads"]
    scale, stream = case["d"] ** -0.5, torch.cuda.current_stream()
    args = (q, k, v, state["out"], state["dout"], state["lse"], dq, dk, dv, *dims)
    if op == "bwd":
        ta.tile_attn_bwd(*args, case["d"], masks, scale, stream)
    else:
        ta.tile_attn_bwd_mmdit(*args, case["P"], case["d"], masks, scale, stream)
    return {"dq": dq, "dk": dk, "dv": dv}


def _kept_pairs(case):
    """Query-key pairs over all heads: video pairs of the kept tiles and the text's pairs."""
    masks, (H, T, F, P) = _masks(case), (case["H"], case["T"], case["F"], case["P"])
    nnz = int(masks.astype(bool).sum()) * (1 if masks.ndim == 3 else H)
    text = P * (P + F * T) + P * F * T
    return case["B"] * (nnz * T * T + H * text)


def work(case):
    """Two products of 2 d operations per kept pair forward, five in the gradients (the
    scores, dP, and one for each of dq, dk, dv); every tensor once."""
    B, H, d = case["B"], case["H"], case["d"]
    rows = B * H * (case["P"] + case["F"] * case["T"])
    pairs = _kept_pairs(case)
    if case["op"] in ("bwd", "bwd_mmdit"):
        return {"bytes": rows * (8 * 2 * d + 4), "flops": 10.0 * d * pairs}
    lse = 4 if case["op"] in ("heads", "noalloc", "mmdit") else 0
    return {"bytes": rows * (4 * 2 * d + lse), "flops": 4.0 * d * pairs}


def tolerance(case):
    """bf16 in and out, fp32 accumulation, the weights (and dS) rounded to bf16 for the
    matrix cores: measured 2.3e-3 from 64 bits in the outputs and gradients at every size
    (short rows reach 2.6e-3). Two such results differ by at most the sum of the two."""
    return {"rel": 1e-2}


def exact(case, seed):
    """The same call in float64 with torch, one query segment of one head at a time (a
    frame; with text tokens also the text, which keeps and is kept by everything)."""
    bwd = case["op"] in ("bwd", "bwd_mmdit")
    B, H, F, T, d, P = (case[k] for k in ("B", "H", "F", "T", "d", "P"))
    x = _inputs(case, seed, 4 if bwd else 3)
    masks = _masks(case)
    scale = d ** -0.5
    f64 = dict(dtype=torch.float64, device="cuda")
    S = P + F * T
    out, lse = torch.zeros((B, H, S, d), **f64), torch.zeros((B, H, S), **f64)
    grads = [torch.zeros((B, H, S, d), **f64) for _ in range(3)] if bwd else None
    for b in range(B):
        for h in range(H):
            q, k, v, *g = (t[b, h].double() for t in x)
            m = masks[h] if masks.ndim == 3 else masks
            segs = [(P + i * T, P + (i + 1) * T, m[i]) for i in range(F)]
            if P:
                segs.append((0, P, [1] * F))
            for s0, s1, row in segs:
                keys = torch.cat([torch.arange(0, P, device="cuda")] +
                                 [torch.arange(P + j * T, P + (j + 1) * T, device="cuda")
                                  for j in range(F) if row[j]])
                kk, vv = k[keys], v[keys]
                s = (q[s0:s1] @ kk.t()).mul_(scale)
                z = torch.logsumexp(s, 1)
                p = s.sub_(z[:, None]).exp_()
                o = p @ vv
                out[b, h, s0:s1], lse[b, h, s0:s1] = o, z
                if bwd:
                    go = g[0][s0:s1]
                    dp = (go @ vv.t()).sub_((go * o).sum(1, keepdim=True)).mul_(p)
                    grads[0][b, h, s0:s1] = (dp @ kk).mul_(scale)
                    grads[1][b, h].index_add_(0, keys, (dp.t() @ q[s0:s1]).mul_(scale))
                    grads[2][b, h].index_add_(0, keys, p.t() @ go)
    if bwd:
        return dict(zip(("dq", "dk", "dv"), grads))
    return {"out": out, "lse": lse} if case["op"] in ("heads", "noalloc", "mmdit") else {"out": out}
