"""The tile the bf16 linear layers pick by shape, on both sides of every step of the rule (64 x 64, 128 x 64,
128 x 128, 256 x 128, 256 x 256 tiles of at most one workgroup per CU; several rounds; rows behind whole
rounds) and at the edges of the tiles and of the ring's trip (1 to 13 slices of K).  All kernels add the
products in one order, so the result must equal the 128 x 128 ring kernel's bit for bit; float64
confirms sampled rows: an output is a fp32 sum rounded to bf16 once, so its error is at most 2^-8 of its
size plus (K + 3) 2^-24 sum |a w|."""
import numpy as np
import pytest
import torch

import paper_2508_00367_amd as rs
from rs_testlib import to_host

pytestmark = pytest.mark.gpu

SHAPES = [  # M, K, N
    (1, 64, 64), (63, 128, 192), (64, 192, 64), (65, 256, 128), (197, 320, 448),          # 64 x 64, 1 .. 5 slices
    (1344, 384, 768), (1345, 384, 768),                                                    # 252 / 264 tiles of 64 x 64
    (2688, 448, 768), (2689, 448, 768),                                                    # 252 / 264 of 128 x 64
    (5376, 576, 768), (5377, 704, 768),                                                    # 252 / 258 of 128 x 128
    (10752, 320, 768), (10753, 832, 768),                                                  # 252 / 258 of 256 x 128
    (21760, 64, 768), (21761, 448, 768), (21761, 192, 768), (33000, 512, 768),             # whole round, 1.01, 1.5 rounds
    (24000, 2048, 768)]                                                                    # whole rounds + 64 x 64 .. rest


@pytest.mark.parametrize("epi", [rs.RS_EPI_BIAS_RES, rs.RS_EPI_BIAS_GELU])
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_tile_choice(M, K, N, epi):
    print("tile choice", M, K, N, epi, flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    a = torch.randn((M, K), device="cuda", generator=g).bfloat16()
    w = (torch.randn((N, K), device="cuda", generator=g) * 0.05).bfloat16()
    b = torch.randn((N,), device="cuda", generator=g).bfloat16()
    res = torch.randn((M, N), device="cuda", generator=g).bfloat16() if epi == rs.RS_EPI_BIAS_RES else None
    outs = []
    try:
        for variant in (0, 3):
            rs.rs_tune_gemm_variant(variant)
            out = torch.full((M + 1, N), float("nan"), device="cuda", dtype=torch.bfloat16)
            rs.rs_linear_fwd(a, w, b, res, out[:M], epi)
            torch.cuda.synchronize()
            assert torch.isnan(out[M].float()).all()          # nothing written behind the last row
            outs.append(out[:M])
    finally:
        rs.rs_tune_gemm_variant(0)
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    if epi == rs.RS_EPI_BIAS_RES:
        rows = np.unique(np.r_[0:min(M, 20), M // 2:min(M, M // 2 + 20), max(0, M - 20):M])
        ah, wh = to_host(a[rows]), to_host(w)
        ref = ah @ wh.T + to_host(b) + to_host(res[rows])
        mag = np.abs(ah) @ np.abs(wh).T + np.abs(to_host(b)) + np.abs(to_host(res[rows]))
        err = np.abs(to_host(outs[0][rows]) - ref)
        assert (err <= 2.0 ** -8 * np.abs(ref) + (K + 3) * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("M,K,N", [(64, 2048, 65600), (257, 2048, 65600)])
def test_one_row_panel_wider_than_a_round(M, K, N):
    """More column tiles in one row panel than the chip has CUs, one panel and one row behind it: the same bits as the
    128 x 128 tiles', and sampled columns within a fp32 sum's error plus one rounding to bf16."""
    print("wide panel", M, K, N, flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    a = torch.randn((M, K), device="cuda", generator=g).bfloat16()
    w = (torch.randn((N, K), device="cuda", generator=g) * 0.05).bfloat16()
    b = torch.randn((N,), device="cuda", generator=g).bfloat16()
    outs = []
    try:
        for variant in (0, 3):
            rs.rs_tune_gemm_variant(variant)
            out = torch.full((M + 1, N), float("nan"), device="cuda", dtype=torch.bfloat16)
            rs.rs_linear_fwd(a, w, b, None, out[:M], rs.RS_EPI_BIAS)
            torch.cuda.synchronize()
            assert torch.isnan(out[M].float()).all()
            outs.append(out[:M].view(torch.int16))
    finally:
        rs.rs_tune_gemm_variant(0)
    assert torch.equal(*outs)
    cols = np.r_[0:40, 65500:N]
    ah, wh, bh = to_host(a), to_host(w[cols]), to_host(b[cols])
    ref, mag = ah @ wh.T + bh, np.abs(ah) @ np.abs(wh).T + np.abs(bh)
    err = np.abs(to_host(outs[0].view(torch.bfloat16)[:, cols]) - ref)
    assert (err <= 2.0 ** -8 * np.abs(ref) + (K + 3) * 2.0 ** -24 * mag).all()
