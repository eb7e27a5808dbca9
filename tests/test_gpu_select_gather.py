"""Selection and gather in one launch (rs_shift_topk of at most 64 sequences of 257 .. 6144 tokens or 256 images
of at most 256), on both sides of every limit, for rows of one to four vectors per lane and longer ones,
with many equal scores (whole-number differences): the checker's selection and the rows it names, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_00367_amd as rs

pytestmark = pytest.mark.gpu

CASES = [  # B, N, D, prefix, keep, dtype
    (256, 64, 64, 1, 20, "bf16"), (257, 64, 64, 1, 20, "bf16"),
    (3, 256, 384, 0, 1, "bf16"), (3, 257, 384, 0, 1, "bf16"), (64, 300, 192, 2, 297, "bf16"), (65, 300, 192, 2, 297, "bf16"),
    (2, 1023, 520, 1, 511, "bf16"), (2, 1040, 1032, 1, 17, "bf16"), (1, 777, 1024, 0, 700, "f32"), (1, 777, 1032, 0, 700, "f32"),
    (1, 6144, 8, 1, 6142, "f32"), (1, 6145, 8, 1, 6142, "f32"), (5, 1, 64, 0, 0, "f32"), (2, 300, 64, 5, 0, "bf16"),
    (2, 300, 64, 5, 295, "bf16")]


@pytest.mark.parametrize("B,N,D,P,K,dt", CASES)
def test_select_gather(B, N, D, P, K, dt):
    print("select + gather", B, N, D, P, K, dt, flush=True)
    t = torch.bfloat16 if dt == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(N + D)
    f_in = torch.randint(-8, 9, (B, N, D), device="cuda", generator=g).to(t)
    f_out = f_in.clone()
    f_out[:, :, :4] += torch.randint(0, 4, (B, N, 4), device="cuda", generator=g).to(t)   # few distinct scores
    src = torch.randn((B, N, D), device="cuda", generator=g).to(t)
    scores = torch.empty((B, N), device="cuda")
    kept = torch.full((B * (P + K) + 1,), -7, device="cuda", dtype=torch.int32)
    out = torch.full((B * (P + K) + 1, D), float("nan"), device="cuda").to(t)
    k2, o2 = kept[:-1].view(B, P + K), out[:-1].view(B, P + K, D)
    rs.rs_shift_topk(f_out, f_in, src, P, K, scores, k2, o2, dist=rs.RS_DIST_L1)
    torch.cuda.synchronize()
    assert torch.equal(scores, (f_out.float() - f_in.float()).abs().sum(dim=2))
    want = oracle.topk(scores.cpu().numpy().astype(np.float64), P, K)
    assert np.array_equal(k2.cpu().numpy(), want)
    rows = torch.gather(src, 1, k2.long().unsqueeze(2).expand(-1, -1, D))
    assert torch.equal(o2, rows) and kept[-1] == -7 and torch.isnan(out[-1].float()).all()
