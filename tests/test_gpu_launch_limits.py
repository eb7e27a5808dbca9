"""Calls of so many small items that a launch reaches 2^32 threads: the largest the fused kernels take, the first that goes
through the separate launches, and the largest those take.  A position's score is the same everywhere, so the
whole of every output is known."""
import pytest
import torch

import paper_2508_00367_amd as rs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [(1 << 23) - 1, 1 << 23, (1 << 24) - 1])
def test_grid_lines_of_many_maps(B):
    print("grid lines", B, flush=True)
    f_in = torch.zeros((B, 1, 2, 8), device="cuda", dtype=torch.bfloat16)
    f_out = torch.ones_like(f_in)
    scores, row_scores, col_scores = (torch.full((B, n), -1.0, device="cuda") for n in (2, 1, 2))
    kept_rows, kept_cols = (torch.full((B, 1), -1, device="cuda", dtype=torch.int32) for _ in range(2))
    gathered = torch.zeros((B, 1, 1, 8), device="cuda", dtype=torch.bfloat16)
    rs.rs_grid_line_prune(f_out, f_in, None, 1, 1, scores.view(B, 1, 2), row_scores, col_scores, kept_rows, kept_cols, gathered,
                          dist=rs.RS_DIST_L1)
    torch.cuda.synchronize()
    for t in (scores, row_scores, col_scores):
        assert (t == 8.0).all()
    assert (kept_rows == 0).all() and (kept_cols == 0).all() and (gathered == 1).all()


@pytest.mark.parametrize("B,H", [((1 << 24) - 8, 1), ((1 << 24) - 7, 1), ((1 << 23) - 1, 2), ((1 << 24) - 1, 1)])
def test_grid_tokens_of_many_rows(B, H):
    print("grid tokens", B, H, flush=True)
    f_in = torch.zeros((B, H, 2, 8), device="cuda", dtype=torch.bfloat16)
    f_out = torch.ones_like(f_in)
    scores, col_scores = torch.full((B, H, 2), -1.0, device="cuda"), torch.full((B, 1, H), -1.0, device="cuda")
    kept_cols, kept_rows = (torch.full(s, -1, device="cuda", dtype=torch.int32) for s in ((B, H, 1), (B, 1, 1)))
    gathered = torch.zeros((B, 1, 1, 8), device="cuda", dtype=torch.bfloat16)
    rs.rs_grid_token_prune(f_out, f_in, None, 1, 1, scores, kept_cols, col_scores, kept_rows, gathered, dist=rs.RS_DIST_L1)
    torch.cuda.synchronize()
    assert (scores == 8.0).all() and (col_scores == 8.0).all()
    assert (kept_rows == 0).all() and (kept_cols == 0).all() and (gathered == 1).all()


@pytest.mark.parametrize("B,N,D", [((1 << 20) - 1, 64, 264), (1 << 20, 64, 264), ((1 << 20) + 1, 64, 264), (1 << 26, 1, 264)])
def test_topk_of_many_images(B, N, D):
    """Short images of long rows, 35 GB and more per tensor."""
    print("topk", B, N, D, flush=True)
    f_in = torch.zeros((B, N, D), device="cuda", dtype=torch.bfloat16)
    f_out = torch.zeros_like(f_in)
    f_out[:, :, 0] = 1.0
    f_out[:, N // 2, 0] = 2.0
    scores = torch.full((B, N), -1.0, device="cuda")
    kept = torch.full((B, 1), -1, device="cuda", dtype=torch.int32)
    gathered = torch.full((B, 1, D), 3.0, device="cuda", dtype=torch.bfloat16)
    rs.rs_shift_topk(f_out, f_in, None, 0, 1, scores, kept, gathered, dist=rs.RS_DIST_L1)
    torch.cuda.synchronize()
    assert (scores[:, N // 2] == 2.0).all() and (scores == 1.0).sum() == B * (N - 1)
    assert (kept == N // 2).all() and (gathered == 0.0).all()
    del f_in, f_out, scores, kept, gathered
    torch.cuda.empty_cache()
