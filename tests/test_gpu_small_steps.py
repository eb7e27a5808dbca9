"""Branches of the dispatch by size, at their edges: query rows of short attention on two workgroups, the fp32
linear layers' 64-row tiles shared by the waves, the fp32 LayerNorm of narrow rows (with kept_idx written on its
way)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_00367_amd as rs
import synth_inputs as si
from rs_testlib import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [128, 129, 160, 161, 192, 193, 224, 255, 256])
def test_short_attention_on_two_workgroups_same_bits(N):
    """An image's rows do not depend on how many images there are (up to 128 heads: two workgroups per head)."""
    print("short attention", N, flush=True)
    g = torch.Generator(device="cuda").manual_seed(N)
    qkv = torch.randn((44, N, 3, 3, 64), device="cuda", generator=g).bfloat16()
    outs = []
    for B in (44, 42, 1):
        o = torch.full((B, N, 3, 64), float("nan"), device="cuda", dtype=torch.bfloat16)
        d = qkv[:B]
        rs.rs_attention_fwd(d[:, :, 0], d[:, :, 1], d[:, :, 2], o, 0.125)
        torch.cuda.synchronize()
        outs.append(o)
    assert not torch.isnan(outs[0].float()).any()
    for o in outs[1:]:
        assert torch.equal(o.view(torch.int16), outs[0][:o.shape[0]].view(torch.int16))


# 516 tiles of 64 rows (K <= 384) and more than 1024; 1, 2, 4, 6, 7 slices; one and 63 rows in the last tile
@pytest.mark.parametrize("M,K,N", [(10945, 256, 192), (10943, 384, 192), (32961, 64, 64), (65473, 448, 64), (21889, 128, 192)])
def test_fp32_linear_shared_tiles(M, K, N):
    """Bound: a product is exact to 2^-24 relative and each of the K / 4 + 2 additions behind an element
    rounds once.  The rows of the first tile once more as a problem of their own (K split over the waves): the same bits."""
    print("fp32 linear", M, K, N, flush=True)
    a, w = si.generic(43, 1, (M, K)), si.generic(43, 2, (K, N), std=0.05)
    b, res = si.generic(43, 3, (N,)), si.generic(43, 4, (M, N))
    da, dw, db, dr = (to_dev(t, "f32") for t in (a, w, b, res))
    out = torch.full((M + 1, N), float("nan"), device="cuda")
    rs.rs_linear_fwd(da, dw, db, dr, out[:M], rs.RS_EPI_BIAS_RES)
    small = torch.empty((100, N), device="cuda")
    rs.rs_linear_fwd(da[:100], dw, db, dr[:100], small, rs.RS_EPI_BIAS_RES)
    torch.cuda.synchronize()
    assert torch.isnan(out[M]).all() and torch.equal(out[:100], small)
    got = to_host(out[:M])
    assert np.isfinite(got).all()
    rows = np.unique(np.r_[0:70, M - 70:M])
    ref = oracle.linear(a[rows], w, b) + res[rows]
    bound = (K / 4 + 3) * 2.0 ** -24 * (np.abs(a[rows]).astype(np.float64) @ np.abs(w) + np.abs(b) + np.abs(res[rows])).max()
    assert np.abs(got[rows] - ref).max() <= bound


@pytest.mark.parametrize("B,N,D", [(1, 1, 64), (3, 5, 128), (2, 17, 192), (1, 33, 256), (2, 9, 320)])
def test_fp32_block_keeps_all_tokens(B, N, D):
    """A fp32 block that drops nothing: kept_idx counts up, output and scores as the fp64 checker's."""
    print("fp32 block", B, N, D, flush=True)
    x, w = si.tokens(44, B, N, D), si.block_weights(44, 0, D, 2 * D)
    dw = {k: to_dev(v, "f32") for k, v in w.items()}
    cfg = rs.make_cfg(B, N, D, D // 64, 2 * D, 0, N, torch.float32)
    ws = torch.empty(rs.rs_block_workspace_size(cfg), dtype=torch.uint8, device="cuda")
    y, scores = torch.empty((B, N, D), device="cuda"), torch.empty((B, N), device="cuda")
    kept = torch.full((B * N + 1,), -7, device="cuda", dtype=torch.int32)
    rs.rs_block_fwd(cfg, rs.make_weights(dw), to_dev(x, "f32"), y, kept[:-1].view(B, N), scores, ws)
    torch.cuda.synchronize()
    ref = oracle.block(x, w, D // 64)
    assert kept[-1] == -7 and np.array_equal(kept[:-1].cpu().numpy().reshape(B, N), np.tile(np.arange(N), (B, 1)))
    assert np.abs(to_host(y) - ref["xhat"]).max() <= 1e-5 * np.abs(ref["xhat"]).max()
    assert np.abs(to_host(scores) - ref["scores"]).max() <= 1e-5 * np.abs(ref["scores"]).max()
