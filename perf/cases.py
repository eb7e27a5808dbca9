"""Performance cases of the framework: the calls a user's program makes, over the sizes it makes them at.

A case is a dict of plain values.  `prepare` makes what the program holds before the call (inputs on
the GPU from a seed, packed weights, workspaces, output buffers), `run` is one pass through the public
entry points, `work` what a pass cannot do without, `tolerance` how far the results of two correct
implementations of the same precision may lie apart.

Kinds of cases
  stack      EncoderStack.step: the forward of an encoder stack with token pruning on a schedule
  attention  rs_attention_fwd on the views of one packed [B, N, 3, H, 64] buffer
  topk       rs_shift_topk: score, selection and compaction of tokens
  grid       rs_grid_token_prune / rs_grid_line_prune: pruning of 2-D feature maps
"""
from __future__ import annotations

import torch

import paper_2508_00367_amd as rs

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_DISTS = {"l2": rs.RS_DIST_L2, "l1": rs.RS_DIST_L1, "cos": rs.RS_DIST_COS}


def _stack(name, dtype, B, N, D, blocks, prune, amount, after, prefix=1, op="mlp", streams=1):
    """Heads are 64 wide and the MLP is four times as wide as the tokens in every model here.
    prune: "pct" (amount = percent of the tokens outside the prefix) or "count" (amount = tokens), dropped
    after each of the blocks that `after` lists (counted from 1)."""
    return dict(name=name, kind="stack", dtype=dtype, B=B, N=N, D=D, blocks=blocks, prune=prune, amount=amount,
                after=after, prefix=prefix, op=op, streams=streams)


_ONE_TO_11 = "1,2,3,4,5,6,7,8,9,10,11"


def listed():
    return [
        # One image at a time through a small model: online classification, where latency counts.
        _stack("vit_s16_one_image", "bf16", 1, 197, 384, 12, "count", 16, _ONE_TO_11),
        # The single-precision block of the parity configuration: four images, one launch chain of 8 kernels.
        _stack("vit_block_fp32", "f32", 4, 197, 192, 1, "pct", 30, "1"),
        # A whole small model in single precision, as a user runs it who compares against bf16.
        _stack("deit_t_fp32", "f32", 64, 197, 192, 12, "pct", 20, "1,4,7"),
        # Small model, small batch, tokens dropped after every block: 197 -> 21 tokens, grids from 100 row tiles to 11.
        _stack("vit_s16", "bf16", 64, 197, 384, 12, "count", 16, _ONE_TO_11),
        # The headline workload: base model, batch 256 as two parts on two streams, 10 % dropped after blocks 4-11.
        _stack("vit_b16", "bf16", 256, 197, 768, 12, "pct", 10, "4,5,6,7,8,9,10,11", streams=2),
        # Narrow model at a large batch: little arithmetic per byte of activations.
        _stack("deit_t", "bf16", 512, 197, 192, 12, "pct", 20, "1,4,7"),
        # Eight clips of 8 x 196 + 1 tokens, half dropped three times: long and short sequences, few of them.
        _stack("video_vit_b16", "bf16", 8, 1569, 768, 12, "pct", 50, "2,5,8"),
        # The largest: four clips of 16 x 256 + 1 tokens, 24 blocks, attention-heavy.
        _stack("video_vit_l14", "bf16", 4, 4097, 1024, 24, "pct", 30, "4,8,12,16"),
        # Fused attention alone, for a program with linear layers of its own: joint space-time attention.
        dict(name="attention_video", kind="attention", dtype="bf16", B=8, N=1569, H=12),
        # Score, selection and compaction alone on image tokens, far beyond the caches.
        dict(name="topk_images", kind="topk", dtype="bf16", B=4096, N=197, D=768, prefix=1, keep=177, dist="l2", separate=False),
        # The same on the tokens of a few long clips, cosine distance, rows gathered from a third tensor.
        dict(name="topk_clips", kind="topk", dtype="f32", B=8, N=1569, D=768, prefix=1, keep=784, dist="cos", separate=True),
        # Feature maps of a convolution stage (56 x 56 x 64 -> 48 x 48), removed position by position.
        dict(name="grid_tokens", kind="grid", dtype="bf16", variant="token", B=64, H=56, W=56, C=64, rows=48, cols=48, dist="l2"),
    ]


# ---------------------------------------------------------------------------- drawn cases
def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _draw_schedule(rng, blocks, N, prefix):
    """A schedule of the three manners the workloads have: every block, every third block, late blocks."""
    manner = rng.choice(("every", "third", "late", "first"))
    after = {"every": range(1, blocks), "third": range(1, blocks, 3), "late": range(max(1, blocks // 3), blocks),
             "first": range(1, min(4, blocks))}[manner]
    after = list(after) or [1]
    if rng.random() < 0.3:
        return "count", rng.randint(1, max(1, (N - prefix) // (len(after) + 1))), after
    return "pct", rng.randint(5, 50 if len(after) <= 4 else 12), after


def draw(rng):
    kind = rng.choices(("image", "video", "f32", "attention", "topk", "grid"), (35, 15, 12, 12, 15, 11))[0]
    if kind in ("image", "video", "f32"):
        prefix = rng.choice((0, 1, 1, 1, 2))
        blocks = rng.randint(1, 4) if kind == "f32" else rng.randint(4, 12)
        if kind == "image":
            D, N, B = rng.choice((192, 384, 384, 768, 768, 1024)), _log(rng, 50, 260), _log(rng, 1, 512)
        elif kind == "video":
            D, N, B = rng.choice((384, 768, 768, 1024)), _log(rng, 393, 4097), _log(rng, 1, 20)
        else:
            D, N, B = rng.choice((192, 192, 384, 768)), _log(rng, 50, 400), _log(rng, 1, 64)
        # no costlier than the largest listed stack of the same precision
        limit = 1.5e11 if kind == "f32" else 3e12
        while B > 1 and B * sum(rs.block_flops(N, D, 4 * D)) * blocks > limit:
            B = (B + 1) // 2
        while sum(rs.block_flops(N, D, 4 * D)) * B * blocks > limit:
            N = N * 2 // 3
        prune, amount, after = _draw_schedule(rng, blocks, N, prefix)
        streams = 2 if kind != "f32" and B >= 16 and rng.random() < 0.4 else 1
        c = _stack("", "f32" if kind == "f32" else "bf16", B, N, D, blocks, prune, amount, ",".join(map(str, after)),
                   prefix=prefix, op=rng.choice(("mlp", "mlp", "mlp", "attn")), streams=streams)
    elif kind == "attention":
        dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
        N, H = _log(rng, 17, 4097), rng.choice((3, 6, 12, 16))
        B = _log(rng, 1, 256)
        while B > 1 and 256.0 * B * H * N * N > (3e10 if dtype == "f32" else 3e11):
            B = (B + 1) // 2
        c = dict(kind="attention", dtype=dtype, B=B, N=N, H=H)
        if dtype == "f32" and 256.0 * H * N * N > 3e10:
            c["N"] = 1000
    elif kind == "topk":
        N, D = _log(rng, 50, 4097), rng.choice((192, 384, 768, 1024))
        prefix = rng.choice((0, 1, 1, 2))
        dtype = rng.choice(("bf16", "bf16", "f32"))
        B = max(1, min(_log(rng, 1, 4096), int(4096 * 197 * 768 * (1 if dtype == "bf16" else 0.5) / (N * D))))
        c = dict(kind="topk", dtype=dtype, B=B, N=N, D=D, prefix=prefix, keep=rng.randint(1, N - prefix - 1),
                 dist=rng.choice(("l2", "l2", "l1", "cos")), separate=rng.random() < 0.4)
    else:
        H, C = rng.choice(((56, 64), (56, 256), (28, 128), (28, 512), (14, 256), (14, 1024), (7, 512)))
        W = H + rng.randint(-3, 3)
        B = max(1, min(_log(rng, 1, 256), int(256 * 56 * 56 * 64 / (H * W * C))))
        c = dict(kind="grid", dtype=rng.choice(("bf16", "bf16", "f32")), variant=rng.choice(("token", "line")), B=B, H=H, W=W,
                 C=C, rows=rng.randint((H + 1) // 2, H - 1), cols=rng.randint((W + 1) // 2, W - 1), dist=rng.choice(("l2", "l2", "l1", "cos")))
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------- one case
def _workload(c):
    return dict(dtype=c["dtype"], B=c["B"], N=c["N"], D=c["D"], H=c["D"] // 64, Dm=4 * c["D"], blocks=c["blocks"],
                n_prefix=c["prefix"], op=c["op"],
                prune={"kind": "drop_pct", "pct": c["amount"], "after": [int(a) for a in c["after"].split(",")]} if c["prune"] == "pct"
                else {"kind": "drop_count", "r": c["amount"], "after": [int(a) for a in c["after"].split(",")]})


def _tiered_tokens(g, wl, dtype):
    """Tokens [B, N, D] of random direction whose lengths come in tiers, one per pruning step of the
    schedule (a factor of 1.25 apart, tier by tier in random places of the sequence): salient tokens
    stand out from the background the way they do in trained models, and the tokens a step drops do
    not hang on the last bit of a score, so that the outputs of two implementations have the same
    tokens in the same rows."""
    B, N, D, P = wl["B"], wl["N"], wl["D"], wl["n_prefix"]
    drops = []
    for n_in, n_keep in rs.keep_counts(N, P, wl["blocks"], wl["prune"]):
        if n_in - P > n_keep:
            drops.append(n_in - P - n_keep)
    drops.append(N - P - sum(drops))
    tier = torch.repeat_interleave(torch.arange(len(drops), device="cuda"), torch.tensor(drops, device="cuda"))
    place = torch.rand((B, N - P), device="cuda", generator=g).argsort(dim=1)
    length = torch.cat([torch.full((B, P), len(drops) - 1, device="cuda"), tier[place]], dim=1)
    x = torch.randn((B, N, D), device="cuda", generator=g)
    x *= (2.0 * 1.25 ** length.to(torch.float32) * D ** 0.5 / x.norm(dim=2)).unsqueeze(2)
    return x.to(dtype)


def _block_weights(g, D, Dm, dtype):
    def normal(*shape):
        return (torch.randn(shape, device="cuda", generator=g) * 0.02).to(dtype)
    one, zero = torch.ones(D, device="cuda", dtype=dtype), torch.zeros(D, device="cuda", dtype=dtype)
    return {"ln1_g": one, "ln1_b": zero, "w_qkv": normal(D, 3 * D), "b_qkv": normal(3 * D), "w_proj": normal(D, D),
            "b_proj": normal(D), "ln2_g": one, "ln2_b": zero, "w_fc1": normal(D, Dm), "b_fc1": normal(Dm),
            "w_fc2": normal(Dm, D), "b_fc2": normal(D)}


def _maps(g, shape, dtype):
    """f_in ~ N(0, 1) with a magnitude per position, f_out = f_in + a change whose size varies by position."""
    pos = shape[:-1] + (1,)
    f_in = torch.randn(shape, device="cuda", generator=g) * torch.exp(0.5 * torch.randn(pos, device="cuda", generator=g))
    f_in = f_in.to(dtype)
    change = torch.randn(shape, device="cuda", generator=g) * (0.3 * torch.exp(0.7 * torch.randn(pos, device="cuda", generator=g)))
    return change.add_(f_in).to(dtype), f_in


def prepare(case, seed):
    c, dt = case, _DTYPES[case["dtype"]]
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    if c["kind"] == "stack":
        wl = _workload(c)
        x0 = _tiered_tokens(g, wl, dt)
        weights = [_block_weights(g, wl["D"], wl["Dm"], dt) for _ in range(wl["blocks"])]
        stack = rs.EncoderStack(wl, x0, weights, streams=c["streams"])
        torch.cuda.synchronize()          # the parts' streams do not wait for the stream the inputs were made on
        return dict(case=c, stack=stack)
    if c["kind"] == "attention":
        qkv = torch.randn((c["B"], c["N"], 3, c["H"], 64), device="cuda", generator=g).to(dt)
        return dict(case=c, qkv=qkv, o=torch.empty((c["B"], c["N"], c["H"], 64), device="cuda", dtype=dt))
    if c["kind"] == "topk":
        B, N, D, K = c["B"], c["N"], c["D"], c["prefix"] + c["keep"]
        f_out, f_in = _maps(g, (B, N, D), dt)
        return dict(case=c, f_out=f_out, f_in=f_in, src=torch.randn((B, N, D), device="cuda", generator=g).to(dt) if c["separate"] else None,
                    scores=torch.empty((B, N), device="cuda"), kept=torch.empty((B, K), device="cuda", dtype=torch.int32),
                    gathered=torch.empty((B, K, D), device="cuda", dtype=dt))
    B, H, W, C, R, Q = (c[k] for k in ("B", "H", "W", "C", "rows", "cols"))
    f_out, f_in = _maps(g, (B, H, W, C), dt)
    s = dict(case=c, f_out=f_out, f_in=f_in, scores=torch.empty((B, H, W), device="cuda"),
             gathered=torch.empty((B, R, Q, C), device="cuda", dtype=dt))
    if c["variant"] == "token":
        s.update(kept_cols=torch.empty((B, H, Q), device="cuda", dtype=torch.int32), col_scores=torch.empty((B, Q, H), device="cuda"),
                 kept_rows=torch.empty((B, Q, R), device="cuda", dtype=torch.int32))
    else:
        s.update(row_scores=torch.empty((B, H), device="cuda"), col_scores=torch.empty((B, W), device="cuda"),
                 kept_rows=torch.empty((B, R), device="cuda", dtype=torch.int32), kept_cols=torch.empty((B, Q), device="cuda", dtype=torch.int32))
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "stack":
        return s["stack"].step()
    if c["kind"] == "attention":
        rs.rs_attention_fwd(s["qkv"][:, :, 0], s["qkv"][:, :, 1], s["qkv"][:, :, 2], s["o"], 0.125)
        return s["o"]
    if c["kind"] == "topk":
        rs.rs_shift_topk(s["f_out"], s["f_in"], s["src"], c["prefix"], c["keep"], s["scores"], s["kept"], s["gathered"], dist=_DISTS[c["dist"]])
        return {k: s[k] for k in ("scores", "kept", "gathered")}
    if c["variant"] == "token":
        rs.rs_grid_token_prune(s["f_out"], s["f_in"], None, c["rows"], c["cols"], s["scores"], s["kept_cols"], s["col_scores"],
                               s["kept_rows"], s["gathered"], dist=_DISTS[c["dist"]])
        return {k: s[k] for k in ("scores", "kept_cols", "col_scores", "kept_rows", "gathered")}
    rs.rs_grid_line_prune(s["f_out"], s["f_in"], None, c["rows"], c["cols"], s["scores"], s["row_scores"], s["col_scores"],
                          s["kept_rows"], s["kept_cols"], s["gathered"], dist=_DISTS[c["dist"]])
    return {k: s[k] for k in ("scores", "row_scores", "col_scores", "kept_rows", "kept_cols", "gathered")}


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "stack":
        wl = _workload(c)
        B, N, D, P = wl["B"], wl["N"], wl["D"], wl["n_prefix"]
        lin, att = rs.forward_flops(N, P, D, wl["Dm"], wl["blocks"], wl["prune"])
        last = P + rs.keep_counts(N, P, wl["blocks"], wl["prune"])[-1][1]
        return {"bytes": (B * (N + last) * D + wl["blocks"] * 12 * D * D) * e, "flops": B * (lin + att)}
    if c["kind"] == "attention":
        return {"bytes": 4 * c["B"] * c["N"] * c["H"] * 64 * e, "flops": 4 * c["B"] * c["H"] * c["N"] ** 2 * 64}
    if c["kind"] == "topk":
        B, N, D, K = c["B"], c["N"], c["D"], c["prefix"] + c["keep"]
        return {"bytes": B * (2 * N * D * e + K * D * e * (2 if c["separate"] else 1) + 4 * N + 4 * K), "flops": 3 * B * N * D}
    B, H, W, C, R, Q = (c[k] for k in ("B", "H", "W", "C", "rows", "cols"))
    small = 4 * (H * Q + Q * H + Q * R) if c["variant"] == "token" else 4 * (H + W + R + Q)
    return {"bytes": B * (2 * H * W * C * e + R * Q * C * e + 4 * H * W + small), "flops": 3 * B * H * W * C}


def tolerance(case):
    """About four times the distance of the path from the same computation in 64 bits: 5e-3 .. 1.2e-2
    (worst element 7.5e-2) for bf16 stacks of 4 to 24 blocks, 2.4e-7 (2e-6) for fp32 ones, 2.2e-3
    (1e-2) for bf16 attention, 4e-7 (1.7e-6) for the fp32 scores of any input type."""
    if case["kind"] == "stack":
        return {"rel": 2.5e-2, "max": 0.25} if case["dtype"] == "bf16" else {"rel": 1e-6, "max": 1e-5}
    if case["kind"] == "attention":
        return {"rel": 9e-3, "max": 5e-2} if case["dtype"] == "bf16" else {"rel": 2e-6, "max": 1e-5}
    # two scores within rounding of each other at the threshold may change places, rarely, and then a
    # few indices and rows behind them move
    return {"rel": 2e-6, "max": 1e-5, "differ": 1e-3}
