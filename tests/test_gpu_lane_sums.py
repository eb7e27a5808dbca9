"""Sums over the lanes of a wave and of its groups of 8, 16 and 32, at the row lengths where the group changes or its last
lanes hold nothing.  The L1 score of whole-number rows is exact in any order, so a lane that is added twice
or left out shows as a wrong whole number; each lane's share is of a size of its own."""
import sys

import numpy as np
import pytest
import torch

import paper_2508_00367_amd as rs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,N", [(2, 30), (3, 300), (300, 110)])  # short, long, and enough images for the one-pass kernel
@pytest.mark.parametrize("D", [8, 64, 72, 128, 136, 248, 256, 264, 504, 512, 520, 768, 1024, 1032, 2048])
def test_scores_of_whole_numbers_are_exact(B, N, D, dtype):
    print("lane sums", B, N, D, dtype, flush=True)
    sys.stdout.flush()
    g = np.random.default_rng(D + N)
    # |x| <= 256 is exact in bf16; sums stay below 2^20
    x = g.integers(-256, 257, size=(N, D)).astype(np.float32)
    x *= (g.random((N, D)) < 0.5)
    f_out = torch.from_numpy(x).to("cuda", dtype).expand(B, N, D).contiguous()
    f_in = torch.zeros_like(f_out)
    scores = torch.empty((B, N), device="cuda")
    K = N // 2
    kept = torch.empty((B, 1 + K), device="cuda", dtype=torch.int32)
    out = torch.empty((B, 1 + K, D), device="cuda", dtype=dtype)
    rs.rs_shift_topk(f_out, f_in, f_in, 1, K, scores, kept, out, dist=rs.RS_DIST_L1)
    torch.cuda.synchronize()
    want = np.abs(x.astype(np.float64)).sum(1)
    np.testing.assert_array_equal(scores.cpu().numpy(), np.broadcast_to(want, (B, N)))
