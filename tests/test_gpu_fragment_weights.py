"""The block's linear layers on weights in fragment order, each kernel at the edges of its tiles: rows around the 128-row
tile of the direct kernel (variant 4), widths that end inside its 256-feature tile and leave some of its waves
without features, 1 to 13 slices of K (none, one and several trips of its four-stage ring, with 0 to 3 slices left).  All
kernels add in one order, so every variant gives the bits of the 128 x 128 ring kernel (3); the parity tests hold that
order against the oracle."""
import pytest
import torch

import paper_2508_00367_amd as rs

pytestmark = pytest.mark.gpu

CASES = [  # B, N, D, Dm
    (1, 1, 64, 64), (1, 127, 64, 128), (1, 128, 128, 192), (3, 43, 192, 320), (1, 257, 256, 64), (2, 192, 320, 448), (5, 77, 448, 832),
    (2, 197, 576, 256), (40, 197, 384, 1536),                                  # by shape: direct for every layer but the projection
    (17, 197, 768, 3072),                                                      # by shape: slim, direct and 128 x 128
    (66, 197, 768, 3072),                                                      # by shape: direct, and persistent for fc2
    (60, 197, 832, 576), (120, 197, 576, 832),                                 # by shape: slim 256 x 128, up to one round and two
    (113, 197, 768, 3072),                                                     # by shape: fc2 persistent, its last 501 rows apart
    (335, 197, 64, 576), (335, 197, 128, 256)]                                 # by shape: ring; fc2 of the first slim 256 x 128, of the second ring


@pytest.mark.parametrize("dist", [rs.RS_DIST_L2, rs.RS_DIST_COS])
@pytest.mark.parametrize("B,N,D,Dm", CASES)
def test_kernels_on_fragments_same_bits(B, N, D, Dm, dist):
    print("fragments", B, N, D, Dm, dist, flush=True)
    g = torch.Generator(device="cuda").manual_seed(B + N + D + Dm)
    nrm = lambda *s, std=0.05: (torch.randn(s, device="cuda", generator=g) * std).bfloat16()
    w = {"ln1_g": nrm(D) + 1, "ln1_b": nrm(D), "w_qkv": nrm(D, 3 * D), "b_qkv": nrm(3 * D), "w_proj": nrm(D, D), "b_proj": nrm(D),
         "ln2_g": nrm(D) + 1, "ln2_b": nrm(D), "w_fc1": nrm(D, Dm), "b_fc1": nrm(Dm), "w_fc2": nrm(Dm, D), "b_fc2": nrm(D)}
    x = nrm(B, N, D, std=2.0)
    cfg = rs.make_cfg(B, N, D, D // 64, Dm, 1, N - 1, torch.bfloat16, dist=dist)
    packed = torch.empty(rs.rs_packed_weights_size(cfg), dtype=torch.uint8, device="cuda")
    rs.rs_pack_weights(cfg, rs.make_weights(w), packed)
    ws = torch.empty(rs.rs_block_workspace_size(cfg), dtype=torch.uint8, device="cuda")
    outs = []
    try:
        for variant in (3, 0, 1, 2, 4):
            rs.rs_tune_gemm_variant(variant)
            y = torch.full((B * N + 1, D), float("nan"), device="cuda", dtype=torch.bfloat16)
            kept, scores = torch.zeros((B, N), device="cuda", dtype=torch.int32), torch.zeros((B, N), device="cuda")
            rs.rs_block_fwd(cfg, rs.make_weights(w, packed), x, y[:B * N].view(B, N, D), kept, scores, ws)
            torch.cuda.synchronize()
            assert torch.isnan(y[-1].float()).all()          # nothing written behind the last row
            outs.append((y[:-1].view(torch.int16), scores))
    finally:
        rs.rs_tune_gemm_variant(0)
    assert not torch.isnan(outs[0][0].view(torch.bfloat16).float()).any()
    for o in outs[1:]:
        assert torch.equal(o[0], outs[0][0]) and torch.equal(o[1], outs[0][1])
