"""The MLP half of a block in one kernel (bf16, D = 192, 16384 rows and more): rows on both sides of the rule
and off the 128-row tiles, the smallest and largest hidden width, every distance and every pair of operands of
the shift, blocks that prune and blocks that keep all tokens (statistics of the output and kept_idx written by
the kernel).  It adds in the order of the separate launches, which a forced tile variant runs: the same bits."""
import pytest
import torch

import paper_2508_00367_amd as rs

pytestmark = pytest.mark.gpu

CASES = [  # B, N, Dm, dropped tokens, op, dist
    (127, 129, 768, 0, rs.RS_SHIFT_MLP, rs.RS_DIST_L2),             # 16383 rows: separate launches either way
    (128, 128, 768, 0, rs.RS_SHIFT_MLP, rs.RS_DIST_L2),             # 16384
    (113, 145, 192, 30, rs.RS_SHIFT_MLP, rs.RS_DIST_L1),            # 16385, one row in the last tile
    (96, 197, 960, 40, rs.RS_SHIFT_MLP, rs.RS_DIST_COS),
    (91, 181, 576, 0, rs.RS_SHIFT_BLOCK, rs.RS_DIST_COS),
    (91, 181, 384, 17, rs.RS_SHIFT_MLP_NORMED, rs.RS_DIST_L2),
    (180, 197, 768, 39, rs.RS_SHIFT_MLP_STREAM, rs.RS_DIST_L2),     # two workgroups on some CUs
    (180, 197, 768, 39, rs.RS_SHIFT_ATTN, rs.RS_DIST_L2)]


@pytest.mark.parametrize("B,N,Dm,drop,op,dist", CASES)
def test_mlp_fused_same_bits(B, N, Dm, drop, op, dist):
    print("fused MLP", B, N, Dm, drop, op, dist, flush=True)
    D, P = 192, 1
    g = torch.Generator(device="cuda").manual_seed(B + N + Dm)

    def normal(*shape, scale=0.05):
        return (torch.randn(shape, device="cuda", generator=g) * scale).bfloat16()
    w = {"ln1_g": normal(D) + 1, "ln1_b": normal(D), "w_qkv": normal(D, 3 * D), "b_qkv": normal(3 * D), "w_proj": normal(D, D),
         "b_proj": normal(D), "ln2_g": normal(D) + 1, "ln2_b": normal(D), "w_fc1": normal(D, Dm), "b_fc1": normal(Dm),
         "w_fc2": normal(Dm, D), "b_fc2": normal(D)}
    x = normal(B, N, D, scale=2.0)
    cfg = rs.make_cfg(B, N, D, 3, Dm, P, N - P - drop, torch.bfloat16, op=op, dist=dist)
    packed = torch.empty(rs.rs_packed_weights_size(cfg), dtype=torch.uint8, device="cuda")
    rs.rs_pack_weights(cfg, rs.make_weights(w), packed)
    ws = torch.empty(rs.rs_block_workspace_size(cfg), dtype=torch.uint8, device="cuda")
    K = N - drop
    outs = []
    try:
        for variant in (0, 3):
            rs.rs_tune_gemm_variant(variant)
            y = torch.full((B * K + 1, D), float("nan"), device="cuda", dtype=torch.bfloat16)
            kept = torch.full((B * K + 1,), -7, device="cuda", dtype=torch.int32)
            scores = torch.zeros((B, N), device="cuda")
            stats = torch.full((B * K + 1, 2), float("nan"), device="cuda")
            rs.rs_block_fwd_chained(cfg, rs.make_weights(w, packed), x, None, y[:B * K].view(B, K, D), stats[:B * K],
                                    kept[:B * K].view(B, K), scores, ws)
            torch.cuda.synchronize()
            assert torch.isnan(y[-1].float()).all() and torch.isnan(stats[-1]).all() and kept[-1] == -7
            outs.append((y[:-1].view(torch.int16), kept, scores, stats[:-1]))
    finally:
        rs.rs_tune_gemm_variant(0)
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    assert not torch.isnan(outs[0][3]).any()


@pytest.mark.parametrize("B,N", [(127, 129), (128, 128), (113, 145)])
def test_statistics_given_or_formed(B, N):
    """The first LayerNorm's statistics handed over or formed inside the QKV kernel: the same block output, and the
    separate statistics launch's bits (which a block that keeps every token leaves for its output)."""
    print("statistics", B, N, flush=True)
    D, Dm, M = 192, 384, B * N
    g = torch.Generator(device="cuda").manual_seed(M)

    def normal(*shape, scale=0.05):
        return (torch.randn(shape, device="cuda", generator=g) * scale).bfloat16()
    w = {"ln1_g": normal(D) + 1, "ln1_b": normal(D), "w_qkv": normal(D, 3 * D), "b_qkv": normal(3 * D), "w_proj": normal(D, D),
         "b_proj": normal(D), "ln2_g": normal(D) + 1, "ln2_b": normal(D), "w_fc1": normal(D, Dm), "b_fc1": normal(Dm),
         "w_fc2": normal(Dm, D), "b_fc2": normal(D)}
    cfg = rs.make_cfg(B, N, D, 3, Dm, 1, N - 1, torch.bfloat16)
    ws = torch.empty(rs.rs_block_workspace_size(cfg), dtype=torch.uint8, device="cuda")
    kept = torch.empty((B, N), device="cuda", dtype=torch.int32)
    x, mid = normal(B, N, D, scale=2.0), torch.empty((B, N, D), device="cuda", dtype=torch.bfloat16)
    stats = torch.empty((M, 2), device="cuda")
    rs.rs_block_fwd_chained(cfg, rs.make_weights(w), x, None, mid, stats, kept, None, ws)
    outs = []
    for given in (stats, None):
        y = torch.empty_like(mid)
        rs.rs_block_fwd_chained(cfg, rs.make_weights(w), mid, given, y, None, kept, None, ws)
        torch.cuda.synchronize()
        outs.append(y.view(torch.int16))
    assert torch.equal(*outs)
