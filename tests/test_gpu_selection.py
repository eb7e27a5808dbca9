"""The selection of long sequences where it can go wrong: every length at which it changes its manner
(counting / keys in LDS / keys in global memory, 256 / 1024 threads), scores that are all equal, heavily
tied, within one binade, or spread over the whole exponent range.  Integer work: kept indices must
equal the checker's bit for bit.  A row holds its score in one element (f_out = [v, 0, ...], f_in = 0), so
that the score is v exactly."""
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2508_00367_amd as rs
import synth_inputs as si
from rs_testlib import host_round, norm_err, to_dev

pytestmark = pytest.mark.gpu


def _scores(kind, B, N, rng):
    if kind == "equal":
        return np.full((B, N), 3.0, np.float32)
    if kind == "tied":
        return rng.integers(0, 7, size=(B, N)).astype(np.float32)
    if kind == "binade":
        return (1.0 + rng.integers(0, 1 << 12, size=(B, N)) * 2.0 ** -12).astype(np.float32)
    return np.exp2(rng.integers(-60, 60, size=(B, N))).astype(np.float32) * rng.integers(1, 9, size=(B, N)).astype(np.float32)


@pytest.mark.parametrize("kind", ["equal", "tied", "binade", "wide"])
@pytest.mark.parametrize("N,P,K", [(256, 1, 100), (257, 1, 256), (300, 2, 1), (1024, 0, 512), (1025, 1, 7), (1569, 1, 784),
                                   (4097, 1, 2868), (12288, 3, 6000), (12289, 1, 12287)])
def test_selection_of_long_sequences(N, P, K, kind):
    print("selection", kind, N, P, K, flush=True)
    sys.stdout.flush()
    B = 3
    v = _scores(kind, B, N, np.random.default_rng(N + K))
    f_out = torch.zeros((B, N, 8), device="cuda")
    f_out[:, :, 0] = torch.from_numpy(v)
    f_in = torch.zeros_like(f_out)
    scores = torch.empty((B, N), device="cuda")
    kept = torch.full((B, P + K), -1, device="cuda", dtype=torch.int32)
    src = torch.arange(B * N, device="cuda", dtype=torch.float32).view(B, N, 1).expand(B, N, 8).contiguous()
    out = torch.full((B, P + K, 8), -1.0, device="cuda")
    rs.rs_shift_topk(f_out, f_in, src, P, K, scores, kept, out, dist=rs.RS_DIST_L1)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(scores.cpu().numpy(), v)
    want = oracle.topk(v.astype(np.float64), P, K)
    np.testing.assert_array_equal(kept.cpu().numpy(), want)
    np.testing.assert_array_equal(out[:, :, 0].cpu().numpy(), want + np.arange(B)[:, None] * N)


# image batches on both sides of the rule that picks the one-pass kernel (rounds of 256 images at least
# three quarters full, more than 104 tokens), and its longest and shortest sequences; against it, scores, then
# selection and gather in one launch (up to 256 images) or two
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,N,D,P,K", [(191, 197, 64, 1, 150), (192, 197, 64, 1, 150), (256, 105, 72, 0, 1), (256, 104, 72, 0, 1),
                                       (300, 208, 8, 2, 206), (513, 130, 256, 1, 60), (600, 207, 384, 1, 100)])
def test_one_pass_and_three_launches_agree(B, N, D, P, K, dtype):
    print("one pass", B, N, D, P, K, dtype, flush=True)
    g = torch.Generator().manual_seed(B + N)
    f_in = torch.randn((B, N, D), generator=g).to(dtype).cuda()
    f_out = torch.randn((B, N, D), generator=g).to(dtype).cuda()
    res = []
    for src in (None, f_in.clone()):          # rows from a tensor of their own: never the one-pass kernel
        scores = torch.full((B, N), float("nan"), device="cuda")
        kept = torch.full((B, P + K), -1, device="cuda", dtype=torch.int32)
        out = torch.full((B, P + K, D), float("nan"), device="cuda", dtype=dtype)
        rs.rs_shift_topk(f_out, f_in, src, P, K, scores, kept, out)
        torch.cuda.synchronize()
        res.append((kept, out))
        # fp32 sums of D terms in some order: relative error at most D 2^-24 on either side
        want = (f_out.double() - f_in.double()).norm(dim=2)
        assert float(((scores - want).abs() / want).max()) < D * 2.0 ** -24 + 2.0 ** -23
        np.testing.assert_array_equal(kept.cpu().numpy(), oracle.topk(scores.cpu().numpy().astype(np.float64), P, K))
        rows = torch.take_along_dim(f_in, kept.long()[:, :, None], dim=1)
        assert torch.equal(out, rows)


# the block's prune step in one launch (at most 256 tokens, rows of at most 4 KB) and just past it: sequence
# lengths around the 64-token registers of the selecting wave, one survivor, all but one, no prefix, many
# images, rows of one to four vectors per lane
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,N,D,P,K", [(1, 256, 64, 0, 1), (3, 255, 128, 2, 252), (600, 20, 64, 1, 7), (2, 64, 576, 1, 62),
                                       (2, 65, 1024, 1, 30), (2, 129, 1088, 0, 128), (1, 257, 64, 1, 100)])
def test_block_prune_step(B, N, D, P, K, dtype):
    """A pruning block against the same block that keeps every token (its y is the unpruned output): the same
    scores, the kept set exact on them, the kept rows and their LayerNorm statistics copied bit for bit."""
    print("block prune step", B, N, D, P, K, dtype, flush=True)
    g = torch.Generator(device="cuda").manual_seed(N * D + K)
    rnd = lambda *s, std=0.05: (torch.randn(s, device="cuda", generator=g) * std).to(dtype)
    w = dict(w_qkv=rnd(D, 3 * D), w_proj=rnd(D, D), w_fc1=rnd(D, 64), w_fc2=rnd(64, D))
    x = rnd(B, N, D, std=1.0)
    res = []
    for n_keep in (K, N - P):
        cfg = rs.make_cfg(B, N, D, D // 64, 64, P, n_keep, dtype)
        ws = torch.empty(rs.rs_block_workspace_size(cfg), dtype=torch.uint8, device="cuda")
        y = torch.full((B, P + n_keep, D), float("nan"), device="cuda", dtype=dtype)
        stats = torch.full((B, P + n_keep, 2), float("nan"), device="cuda")
        kept = torch.full((B, P + n_keep), -1, device="cuda", dtype=torch.int32)
        scores = torch.full((B, N), float("nan"), device="cuda")
        rs.rs_block_fwd_chained(cfg, rs.make_weights(w), x, None, y, stats, kept, scores, ws)
        torch.cuda.synchronize()
        res.append((y, stats, kept, scores))
    (y, stats, kept, scores), (y_all, stats_all, _, scores_all) = res
    assert torch.equal(scores, scores_all)
    np.testing.assert_array_equal(kept.cpu().numpy(), oracle.topk(scores.cpu().numpy().astype(np.float64), P, K))
    idx = kept.long()[:, :, None]
    assert torch.equal(y, torch.take_along_dim(y_all, idx, dim=1))
    assert torch.equal(stats, torch.take_along_dim(stats_all, idx, dim=1))


# images whose rows fit the one-pass kernel's registers: up to 16, 32 and 64 16-byte vectors and beyond, odd ones among them
@pytest.mark.parametrize("dist", [rs.RS_DIST_L2, rs.RS_DIST_L1, rs.RS_DIST_COS])
@pytest.mark.parametrize("N,D,dtype", [(105, 8, "bf16"), (130, 64, "bf16"), (197, 72, "bf16"), (208, 136, "bf16"), (197, 192, "bf16"),
                                       (197, 384, "bf16"), (119, 520, "bf16"), (197, 768, "bf16"), (105, 8, "f32"), (197, 40, "f32"),
                                       (208, 64, "f32"), (197, 192, "f32"), (130, 264, "f32"), (197, 384, "f32")])
def test_an_image_does_not_depend_on_the_batch(N, D, dtype, dist):
    """The one-pass kernel (256 images) and the separate launches (3, 1): the same scores, survivors and rows, bit for bit."""
    print("batch", N, D, dtype, dist, flush=True)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(N + D)
    f_in = torch.randn((256, N, D), device="cuda", generator=g).to(t)
    f_out = (f_in.float() * 1.1 + 0.3 * torch.randn((256, N, D), device="cuda", generator=g)).to(t)
    outs = []
    for B in (256, 3, 1):
        scores = torch.full((B, N), float("nan"), device="cuda")
        kept = torch.full((B, N // 2), -1, device="cuda", dtype=torch.int32)
        rows = torch.zeros((B, N // 2, D), device="cuda", dtype=t)
        rs.rs_shift_topk(f_out[:B], f_in[:B], None, 1, N // 2 - 1, scores, kept, rows, dist=dist)
        torch.cuda.synchronize()
        outs.append((scores, kept, rows))
    for B, out in zip((3, 1), outs[1:]):
        for a, b in zip(outs[0], out):
            assert torch.equal(a[:B], b)
    assert not torch.isnan(outs[0][0]).any()


# pruning blocks whose selection and gather are launches of their own: many sequences beyond 256 tokens, rows beyond 4 KB
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,N,D,P,K", [(66, 300, 64, 1, 100), (65, 257, 1088, 0, 128), (2, 65, 2112, 1, 30), (1, 6145, 64, 1, 700)])
def test_block_prune_step_in_two_launches(B, N, D, P, K, dtype):
    test_block_prune_step(B, N, D, P, K, dtype)


# the one-pass kernel (192 images and more, more than 104 tokens): rows of one to three 512-byte chunks, whole and in part, every
# token kept, the prefix alone, one token, a second round of images
@pytest.mark.parametrize("dist", [rs.RS_DIST_L2, rs.RS_DIST_L1, rs.RS_DIST_COS])
@pytest.mark.parametrize("B,N,D,P,K,dtype", [
    (192, 197, 768, 1, 177, "bf16"), (200, 105, 64, 1, 7, "bf16"), (256, 208, 384, 0, 100, "bf16"), (450, 119, 520, 2, 0, "bf16"),
    (192, 197, 192, 1, 196, "bf16"), (255, 130, 256, 0, 130, "bf16"), (192, 207, 760, 1, 1, "bf16"), (192, 197, 384, 1, 177, "f32"),
    (449, 105, 8, 0, 1, "f32"), (192, 160, 264, 2, 158, "f32")])
def test_one_pass_kernel(B, N, D, P, K, dtype, dist):
    """Against the oracle: a sample of the scores (fp32 sums of D terms; 1 - cos carries a few ulps of 1), every image's
    survivors exact on the call's own scores, every kept row."""
    print("one pass kernel", B, N, D, P, K, dtype, dist, flush=True)
    f_in = host_round(si.tokens(5, B, N, D, spread=0.5), dtype)
    f_out = host_round(f_in + si.generic(5, 8, (B, N, D), std=0.3) * np.exp(si.generic(5, 9, (B, N, 1), std=0.7)), dtype)
    scores = torch.full((B, N), float("nan"), device="cuda")
    kept = torch.full((B * (P + K) + 1,), -7, device="cuda", dtype=torch.int32)
    rows = torch.full((B * (P + K) + 1, D), float("nan"), device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    k2, r2 = kept[:-1].view(B, P + K), rows[:-1].view(B, P + K, D)
    rs.rs_shift_topk(to_dev(f_out, dtype), to_dev(f_in, dtype), None, P, K, scores, k2, r2, dist=dist)
    torch.cuda.synchronize()
    assert kept[-1] == -7 and torch.isnan(rows[-1].float()).all()
    sc, sample = scores.cpu().numpy(), [0, B // 2, B - 1]
    want, _, _ = oracle.shift_topk(f_out[sample], f_in[sample], None, P, K, dist)
    assert (np.abs(sc[sample] - want).max() < 2e-6) if dist == rs.RS_DIST_COS else (norm_err(sc[sample], want) < 1e-5)
    keep = k2.cpu().numpy()
    np.testing.assert_array_equal(keep, oracle.topk(sc.astype(np.float64), P, K))
    np.testing.assert_array_equal(r2.float().cpu().numpy(), np.take_along_axis(f_in, keep[:, :, None].astype(np.int64), axis=1))


def _order(v, P, K):
    """The selection written out: NaN above +inf, equal scores by the lower index, survivors in ascending order."""
    key = np.where(np.isnan(v), np.inf, v.astype(np.float64))
    out = []
    for row, nan in zip(key, np.isnan(v)):
        rank = sorted(range(P, len(row)), key=lambda i: (not nan[i], -row[i], i))
        out.append(list(range(P)) + sorted(rank[:K]))
    return np.array(out, np.int32).reshape(len(v), P + K)


# one wave's registers, keys in LDS (256 and 1024 threads), keys in global memory; with the gather in the same launch and alone
@pytest.mark.parametrize("gather", ["same tensor", "own tensor", "none"])
@pytest.mark.parametrize("B,N,P,K", [(3, 60, 1, 20), (3, 200, 0, 40), (200, 197, 1, 90), (3, 256, 1, 4), (3, 300, 1, 150), (70, 300, 0, 33),
                                     (3, 1500, 2, 700), (2, 7000, 1, 60), (2, 12300, 1, 6000)])
def test_selection_of_special_scores(B, N, P, K, gather):
    """Scores of NaN, +inf, the largest finite value, subnormals and zeros of either sign among ordinary ones."""
    print("special scores", B, N, P, K, gather, flush=True)
    rng = np.random.default_rng(N + K)
    special = np.array([np.nan, np.inf, 3.4028235e38, 1e-42, 1.4e-45, 0.0, -0.0, 1.0, 1.0000001, 2.0], np.float32)
    v = rng.choice(special, size=(B, N), p=[.08, .08, .08, .08, .08, .15, .1, .15, .1, .1])
    f_out = torch.zeros((B, N, 8), device="cuda")
    f_out[:, :, 0] = torch.from_numpy(v)
    f_in = torch.zeros_like(f_out)
    src = torch.arange(B * N, device="cuda", dtype=torch.float32).view(B, N, 1).expand(B, N, 8).contiguous()
    scores = torch.full((B, N), -1.0, device="cuda")
    kept = torch.full((B, P + K), -1, device="cuda", dtype=torch.int32)
    out = None if gather == "none" else torch.full((B, P + K, 8), -1.0, device="cuda")
    rs.rs_shift_topk(f_out, f_in, src if gather == "own tensor" else None, P, K, scores, kept, out, dist=rs.RS_DIST_L1)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(scores.cpu().numpy(), np.abs(v))
    want = _order(v, P, K)
    np.testing.assert_array_equal(kept.cpu().numpy(), want)
    if gather == "own tensor":
        np.testing.assert_array_equal(out[:, :, 3].cpu().numpy(), want + np.arange(B)[:, None] * N)
    elif gather == "same tensor":
        assert (out == 0).all()
