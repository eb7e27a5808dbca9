"""The block's linear layers on weights in fragment order, each kernel at the edges of its tiles: rows around the 128-row
tile of the direct kernel (variant 4), widths that end inside its 256-feature tile and leave some of its waves
without features, 1 to 13 slices of K (none, one and several trips of its four-stage ring, with 0 to 3 slices left).  All
kernels add in one order, so every variant gives the bits of the 128 x 128 ring kernel (3); the parity tests hold that
order against the oracle."""
import pytest
import torch

import paper_2508_00367_amd as rs

pytestmark = pytest.mark.gpu

SMALL = [  # B, N, D, Dm
    (1, 1, 64, 64), (1, 127, 64, 128), (1, 128, 128, 192), (3, 43, 192, 320), (1, 257, 256, 64), (2, 192, 320, 448), (5, 77, 448, 832),
    (2, 197, 576, 256)]
# and with the kernels that the choice by shape takes on 256 CUs, for the layers qkv, proj, fc1, fc2 (the CPU tests hold it to that)
BY_SHAPE = [
    ((30, 197, 384, 1536), ["slim 256x128", "slim 128x128", "direct", "slim 128x128"]),
    ((40, 197, 384, 1536), ["direct", "slim 128x128", "direct", "slim 128x128"]),
    ((17, 197, 768, 3072), ["direct", "slim 128x128", "direct", "slim 128x128"]),
    ((66, 197, 768, 3072), ["direct", "direct", "direct", "persistent"]),
    ((223, 197, 384, 1536), ["direct", "direct", "direct", "direct"]),                         # fc2 with a last round a third full
    ((46, 197, 832, 576), ["direct", "slim 256x128", "direct", "slim 256x128"]),               # up to one round
    ((120, 197, 576, 832), ["direct", "slim 256x128", "direct", "slim 256x128"]),              # up to two
    ((113, 197, 768, 3072), ["direct", "direct", "direct", "persistent + slim 64x64"]),        # 501 rows beyond whole rounds
    ((335, 197, 64, 576), ["direct", "ring", "direct", "slim 256x128"]), ((335, 197, 128, 256), ["direct", "ring", "direct", "ring"])]
CASES = SMALL + [c for c, _ in BY_SHAPE]


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


@pytest.mark.parametrize("variant", [0, 1, 2, 4])
@pytest.mark.parametrize("B,N", [(1, 127), (1, 129), (3, 43), (40, 197)])
def test_row_statistics_at_eight_byte_alignment(B, N, variant):
    """x_stats need be 8-byte aligned only; the direct kernel copies them 16 bytes at a time, two rows, also the last one of an odd count."""
    print("statistics alignment", B, N, variant, flush=True)
    D, Dm = 384, 256
    g = torch.Generator(device="cuda").manual_seed(B + N)
    nrm = lambda *s, std=0.05: (torch.randn(s, device="cuda", generator=g) * std).bfloat16()
    w = {"ln1_g": nrm(D) + 1, "ln1_b": nrm(D), "w_qkv": nrm(D, 3 * D), "b_qkv": nrm(3 * D), "w_proj": nrm(D, D), "b_proj": nrm(D),
         "ln2_g": nrm(D) + 1, "ln2_b": nrm(D), "w_fc1": nrm(D, Dm), "b_fc1": nrm(Dm), "w_fc2": nrm(Dm, D), "b_fc2": nrm(D)}
    x = nrm(B, N, D, std=2.0)
    cfg = rs.make_cfg(B, N, D, D // 64, Dm, 1, N - 1, torch.bfloat16)
    ws = torch.empty(rs.rs_block_workspace_size(cfg), dtype=torch.uint8, device="cuda")
    stats = torch.empty((B * N, 2), device="cuda")
    xf = x.view(B * N, D).float()
    stats[:, 0], stats[:, 1] = xf.mean(1), torch.rsqrt(xf.var(1, unbiased=False) + 1e-6)
    outs = []
    try:
        for v, shift in ((3, 0), (variant, 0), (variant, 2)):
            rs.rs_tune_gemm_variant(v)
            buf = torch.full((B * N * 2 + 4,), float("nan"), device="cuda")
            at = buf[shift:shift + B * N * 2].view(B * N, 2)
            at.copy_(stats)
            assert at.data_ptr() % 16 == 4 * shift
            y, kept = torch.full((B, N, D), float("nan"), device="cuda", dtype=torch.bfloat16), torch.zeros((B, N), device="cuda", dtype=torch.int32)
            rs.rs_block_fwd_chained(cfg, rs.make_weights(w), x, at, y, None, kept, None, ws)
            torch.cuda.synchronize()
            outs.append(y.view(torch.int16))
    finally:
        rs.rs_tune_gemm_variant(0)
    assert torch.isfinite(outs[0].view(torch.bfloat16).float()).all()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
