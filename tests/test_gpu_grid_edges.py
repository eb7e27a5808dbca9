"""Grid pruning at the edges of its kernels: channel counts around the lane groups (8, 16, 32, 64 lanes and
rows of several steps), lines of 256 and 257 positions (selected inside the kernel / by launches of
their own), one position, one survivor.  Selections must be exact on the GPU's own scores."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_00367_amd as rs

pytestmark = pytest.mark.gpu

CASES = [(2, 5, 9, 8, 3, 4), (2, 14, 13, 256, 9, 7), (1, 7, 6, 264, 5, 5), (1, 6, 7, 512, 1, 1), (1, 3, 5, 1032, 2, 4),
         (2, 6, 256, 16, 4, 129), (1, 256, 5, 64, 200, 3), (1, 257, 4, 8, 30, 2), (1, 4, 257, 72, 2, 256), (3, 1, 1, 136, 1, 1)]


def _maps(B, H, W, C, dtype):
    g = torch.Generator().manual_seed(H * W + C)
    f_in = torch.randn((B, H, W, C), generator=g).to(dtype).cuda()
    f_out = torch.randn((B, H, W, C), generator=g).to(dtype).cuda()
    d = f_out.double() - f_in.double()
    return f_out, f_in, d.norm(dim=3)


def _close(scores, want, C):      # fp32 sums of C terms: relative error at most C 2^-24, and the square root's rounding
    assert float(((scores - want).abs() / want).max()) < C * 2.0 ** -24 + 2.0 ** -23


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,H,W,C,R,Q", CASES)
def test_grid_token_edges(B, H, W, C, R, Q, dtype):
    print("grid token", B, H, W, C, R, Q, dtype, flush=True)
    f_out, f_in, want = _maps(B, H, W, C, dtype)
    scores = torch.full((B, H, W), float("nan"), device="cuda")
    kc = torch.full((B, H, Q), -1, device="cuda", dtype=torch.int32)
    cs = torch.full((B, Q, H), float("nan"), device="cuda")
    kr = torch.full((B, Q, R), -1, device="cuda", dtype=torch.int32)
    out = torch.full((B, R, Q, C), float("nan"), device="cuda", dtype=dtype)
    rs.rs_grid_token_prune(f_out, f_in, None, R, Q, scores, kc, cs, kr, out)
    torch.cuda.synchronize()
    _close(scores, want, C)
    s = scores.cpu().numpy().astype(np.float64)
    kc_want = oracle.topk(s.reshape(B * H, W), 0, Q).reshape(B, H, Q)
    np.testing.assert_array_equal(kc.cpu().numpy(), kc_want)
    cs_want = np.take_along_axis(s, kc_want.astype(np.int64), axis=2).transpose(0, 2, 1)
    np.testing.assert_array_equal(cs.cpu().numpy(), cs_want)
    kr_want = oracle.topk(np.ascontiguousarray(cs_want).reshape(B * Q, H), 0, R).reshape(B, Q, R)
    np.testing.assert_array_equal(kr.cpu().numpy(), kr_want)
    got, src = out.float().cpu().numpy(), f_out.float().cpu().numpy()
    for b in range(B):
        for j in range(Q):
            rows = kr_want[b, j]
            np.testing.assert_array_equal(got[b, :, j], src[b, rows, kc_want[b, rows, j]])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,H,W,C,R,Q", CASES)
def test_grid_line_edges(B, H, W, C, R, Q, dtype):
    print("grid line", B, H, W, C, R, Q, dtype, flush=True)
    f_out, f_in, want = _maps(B, H, W, C, dtype)
    scores = torch.full((B, H, W), float("nan"), device="cuda")
    rsc, csc = torch.full((B, H), float("nan"), device="cuda"), torch.full((B, W), float("nan"), device="cuda")
    kr = torch.full((B, R), -1, device="cuda", dtype=torch.int32)
    kc = torch.full((B, Q), -1, device="cuda", dtype=torch.int32)
    out = torch.full((B, R, Q, C), float("nan"), device="cuda", dtype=dtype)
    rs.rs_grid_line_prune(f_out, f_in, None, R, Q, scores, rsc, csc, kr, kc, out)
    torch.cuda.synchronize()
    _close(scores, want, C)
    for got, dim, n in ((rsc, 2, W), (csc, 1, H)):      # means of n positive scores: n additions and a division
        ref = scores.double().mean(dim=dim)
        assert float(((got - ref).abs() / ref).max()) < (n + 1) * 2.0 ** -24
    kr_want = oracle.topk(rsc.cpu().numpy().astype(np.float64), 0, R)
    kc_want = oracle.topk(csc.cpu().numpy().astype(np.float64), 0, Q)
    np.testing.assert_array_equal(kr.cpu().numpy(), kr_want)
    np.testing.assert_array_equal(kc.cpu().numpy(), kc_want)
    np.testing.assert_array_equal(out.float().cpu().numpy(), oracle.grid_gather(f_out.float().cpu().numpy(), kr_want, kc_want))
