"""A block's scratch: a workspace of exactly rs_block_workspace_size bytes is enough and nothing behind it is written, for
every pair of operands of the shift, with the caller's packed weights (hidden activations at a padded pitch) and
without (plain pitch): the same bits.  And the longest blocks that fit the static buffer, against the workspace."""
import ctypes

import pytest
import torch

import paper_2508_00367_amd as rs

pytestmark = pytest.mark.gpu

OPS = [rs.RS_SHIFT_MLP, rs.RS_SHIFT_ATTN, rs.RS_SHIFT_BLOCK, rs.RS_SHIFT_MLP_STREAM, rs.RS_SHIFT_MLP_NORMED]


def _block(B, N, D, Dm):
    g = torch.Generator(device="cuda").manual_seed(B * N + D + Dm)
    nrm = lambda *s, std=0.05: (torch.randn(s, device="cuda", generator=g) * std).bfloat16()
    w = {"ln1_g": nrm(D) + 1, "ln1_b": nrm(D), "w_qkv": nrm(D, 3 * D), "b_qkv": nrm(3 * D), "w_proj": nrm(D, D), "b_proj": nrm(D),
         "ln2_g": nrm(D) + 1, "ln2_b": nrm(D), "w_fc1": nrm(D, Dm), "b_fc1": nrm(Dm), "w_fc2": nrm(Dm, D), "b_fc2": nrm(D)}
    return w, nrm(B, N, D, std=2.0)


def _pack(cfg, w):
    size = rs.rs_packed_weights_size(cfg)
    buf = torch.full((size + 256,), 0x5A, device="cuda", dtype=torch.uint8)
    rs.rs_pack_weights(cfg, rs.make_weights(w), buf)
    torch.cuda.synchronize()
    assert (buf[size:] == 0x5A).all()
    return buf


@pytest.mark.parametrize("op", OPS)
@pytest.mark.parametrize("B,N,D,Dm", [(1, 1, 64, 512), (2, 33, 64, 768), (3, 70, 128, 512), (5, 197, 384, 1536), (128, 129, 192, 768)])
def test_exact_workspace(B, N, D, Dm, op):
    print("workspace", B, N, D, Dm, op, flush=True)
    w, x = _block(B, N, D, Dm)
    keep = max(N - 1 - N // 4, 0)
    cfg = rs.make_cfg(B, N, D, D // 64, Dm, 1, keep, torch.bfloat16, op=op)
    need, packed = rs.rs_block_workspace_size(cfg), _pack(cfg, w)
    outs = []
    for weights in (rs.make_weights(w, packed), rs.make_weights(w)):
        ws = torch.full((need + 4096,), 0x5A, device="cuda", dtype=torch.uint8)
        y = torch.zeros((B, 1 + keep, D), device="cuda", dtype=torch.bfloat16)
        kept = torch.zeros((B, 1 + keep), device="cuda", dtype=torch.int32)
        scores, stats = torch.zeros((B, N), device="cuda"), torch.zeros((B, 1 + keep, 2), device="cuda")
        rs.rs_block_fwd_chained(cfg, weights, x, None, y, stats, kept, scores, ws[:need])
        torch.cuda.synchronize()
        assert (ws[need:] == 0x5A).all()
        outs.append((y.view(torch.int16), kept, scores, stats))
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    assert not torch.isnan(outs[0][2]).any()


@pytest.mark.parametrize("B,N,D", [(130, 131, 192), (41, 197, 384), (17, 200, 768), (15, 135, 1024)])
def test_static_buffer_filled_to_the_end(B, N, D):
    print("static", B, N, D, flush=True)
    w, x = _block(B, N, D, 4 * D)
    cfg = rs.make_cfg(B, N, D, D // 64, 4 * D, 1, N - 20, torch.bfloat16)
    assert rs.rs_block_workspace_size(cfg) <= rs.rs_block_static_scratch_size()
    packed = _pack(cfg, w)
    weights = rs.make_weights(w, packed)          # holds addresses only
    ws = torch.empty(rs.rs_block_workspace_size(cfg), device="cuda", dtype=torch.uint8)
    outs = []
    for static in (False, True):
        y = torch.zeros((B, N - 19, D), device="cuda", dtype=torch.bfloat16)
        kept = torch.zeros((B, N - 19), device="cuda", dtype=torch.int32)
        scores = torch.zeros((B, N), device="cuda")
        if static:
            st = rs.lib().rs_block_fwd_static(ctypes.byref(cfg), ctypes.byref(weights), x.data_ptr(), y.data_ptr(), kept.data_ptr(),
                                              scores.data_ptr(), torch.cuda.current_stream().cuda_stream)
            assert st == rs.RS_OK, rs.rs_last_error()
        else:
            rs.rs_block_fwd(cfg, weights, x, y, kept, scores, ws)
        torch.cuda.synchronize()
        outs.append((y.view(torch.int16), kept, scores))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("D,Dm", [(64, 64), (64, 512), (192, 768), (128, 576)])
def test_packed_buffer_is_whole(D, Dm):
    """Every byte is written, so that two buffers packed from the same weights are the same."""
    print("packed buffer", D, Dm, flush=True)
    w, _ = _block(1, 1, D, Dm)
    cfg = rs.make_cfg(1, 1, D, D // 64, Dm, 0, 1, torch.bfloat16)
    bufs = [torch.full((rs.rs_packed_weights_size(cfg),), fill, device="cuda", dtype=torch.uint8) for fill in (0x5A, 0xA5)]
    for b in bufs:
        rs.rs_pack_weights(cfg, rs.make_weights(w), b)
    torch.cuda.synchronize()
    assert torch.equal(*bufs)
