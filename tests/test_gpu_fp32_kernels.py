"""The fp32 matrix-core kernels at the edges of their tiles, against the fp64 checker.

Bound of the linear layers: a product is exact to 2^-24 relative and every one of the K / 4 + 2
additions behind an element rounds once, so |error| <= (K / 4 + 3) 2^-24 sum_k |a w| in the worst
case; asserted with the largest such sum of the sampled rows."""
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2508_00367_amd as rs
import synth_inputs as si
from rs_testlib import TOL, norm_err, to_dev, to_host

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# rows around the 32- and 64-row tiles; 1, 2, 3, 4 and 7 slices of 64; one column tile and several; the
# last two make more than 1024 64 x 64 tiles, which is where the taller tile takes over
@pytest.mark.parametrize("M,K,N", [(1, 64, 64), (31, 128, 64), (32, 192, 128), (33, 256, 64), (63, 448, 192), (65, 64, 320),
                                   (65473, 64, 64), (21900, 192, 192)])
def test_fp32_linear_tile_edges(M, K, N):
    _say("fp32 linear", M, K, N)
    a, w = si.generic(41, 1, (M, K)), si.generic(41, 2, (K, N), std=0.05)
    b, res = si.generic(41, 3, (N,)), si.generic(41, 4, (M, N))
    out = torch.full((M, N), float("nan"), device="cuda")
    rs.rs_linear_fwd(to_dev(a, "f32"), to_dev(w, "f32"), to_dev(b, "f32"), to_dev(res, "f32"), out, rs.RS_EPI_BIAS_RES)
    torch.cuda.synchronize()
    got = to_host(out)
    assert np.isfinite(got).all()
    rows = np.unique(np.r_[0:min(M, 70), max(0, M - 70):M])
    ref = oracle.linear(a[rows], w, b) + res[rows]
    bound = (K / 4 + 3) * 2.0 ** -24 * (np.abs(a[rows]).astype(np.float64) @ np.abs(w) + np.abs(b) + np.abs(res[rows])).max()
    err = np.abs(got[rows] - ref).max()
    _say("  err %.2e bound %.2e" % (err, bound))
    assert err <= bound


# sequence lengths around the 32-key tiles and the four waves that share them (128 keys per turn)
@pytest.mark.parametrize("N", [1, 31, 32, 33, 64, 96, 97, 127, 128, 129, 161])
def test_fp32_attention_key_split_edges(N):
    B, H = 2, 3
    _say("fp32 attention", N)
    qkv = si.generic(42, 1, (B, N, 3, H, 64))
    buf = torch.full((B, N + 40, 3, H, 64), float("nan"), device="cuda")   # NaN behind the last key of every image
    buf[:, :N] = to_dev(qkv, "f32")
    d = buf[:, :N]
    o = torch.full((B, N, H, 64), float("nan"), device="cuda")
    rs.rs_attention_fwd(d[:, :, 0], d[:, :, 1], d[:, :, 2], o, 0.125)
    torch.cuda.synchronize()
    err = norm_err(to_host(o), oracle.attention(qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2], 0.125))
    _say("  err %.2e" % err)
    assert err < TOL["f32"]


# the keys whose scores are -inf: the first tile of each wave that shares the keys (0-31, 32-63, 64-95, 96-127), all of
# one wave's tiles, all but one key, and the keys of a whole image (a row without any score is NaN, as its softmax is)
MASKED = {"first": range(0, 32), "second": range(32, 64), "third": range(64, 96), "fourth": range(96, 128),
          "padding": range(96, 161), "two_waves": [*range(32, 96), *range(160, 161)], "wave": [*range(0, 32), *range(128, 160)],
          "all_but_one": [i for i in range(161) if i != 70], "all": range(161)}


@pytest.mark.parametrize("how", ["infinite", "overflow", "large scale"])
@pytest.mark.parametrize("N", [128, 129, 161])
@pytest.mark.parametrize("masked", list(MASKED))
def test_fp32_attention_masked_keys(masked, N, how):
    """Keys masked through a reserved channel: -inf in k, or a product that overflows, against the fp64 softmax."""
    B, H = 2, 2
    scale = 2.0 if how == "large scale" else 0.125
    _say("fp32 attention masked", masked, N, how)
    keys = [i for i in MASKED[masked] if i < N]
    qkv = si.generic(45, 1, (B, N, 3, H, 64))
    qkv[:, :, 0, :, 63], qkv[:, :, 1, :, 63] = (2.0 if how == "overflow" else 1.0), 0.0
    seen = np.setdiff1d(np.arange(N), keys)
    ref = np.full((B, N, H, 64), np.nan)
    if len(seen):
        q, k, v = (qkv[:, :, i].astype(np.float64).transpose(0, 2, 1, 3) for i in range(3))
        s = q @ k[:, :, seen].transpose(0, 1, 3, 2) * scale
        p = np.exp(s - s.max(axis=-1, keepdims=True))
        ref = (p @ v[:, :, seen] / p.sum(axis=-1, keepdims=True)).transpose(0, 2, 1, 3)
    qkv[:, keys, 1, :, 63] = -3e38 if how == "overflow" else -np.inf
    d = to_dev(qkv, "f32")
    o = torch.full((B, N, H, 64), 7.0, device="cuda")
    rs.rs_attention_fwd(d[:, :, 0], d[:, :, 1], d[:, :, 2], o, scale)
    torch.cuda.synchronize()
    if not len(seen):
        assert torch.isnan(o).all()
        return
    err = norm_err(to_host(o), ref)
    _say("  err %.2e" % err)
    assert err < TOL["f32"]


@pytest.mark.parametrize("stride", [(1 << 27) - 8, 1 << 27, (1 << 27) + 8])
@pytest.mark.parametrize("N", [1, 3, 37])
def test_fp32_attention_far_rows(N, stride):
    """Token strides around 2^27 elements (four rows beyond 32-bit byte offsets): the bits of the same rows side by side."""
    _say("fp32 attention far rows", N, stride)
    rows = to_dev(si.generic(46, 1, (1, N, 3, 1, 64)), "f32")
    buf = torch.empty(((N - 1) * stride + 192,), device="cuda")
    far = buf.as_strided((1, N, 3, 1, 64), (0, stride, 64, 64, 1))
    far.copy_(rows)
    outs = []
    for d in (rows, far):
        o = torch.full((1, N + 1, 1, 64), float("nan"), device="cuda")
        rs.rs_attention_fwd(d[:, :, 0], d[:, :, 1], d[:, :, 2], o[:, :N], 0.125)
        torch.cuda.synchronize()
        assert torch.isnan(o[:, N]).all() and torch.isfinite(o[:, :N]).all()
        outs.append(o[:, :N])
    assert torch.equal(*outs)


@pytest.mark.parametrize("where", ["q", "k", "v"])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_fp32_attention_special_values(where, value):
    """One NaN or infinity: the rows it reaches are those of the softmax written out, all others are as without it."""
    B, N, H, n, c = 1, 140, 2, 77, 9
    _say("fp32 attention special", where, value)
    qkv = si.generic(47, 1, (B, N, 3, H, 64))
    qkv[0, n, "qkv".index(where), 1, c] = value
    with np.errstate(invalid="ignore", over="ignore"):
        q, k, v = (qkv[:, :, i].astype(np.float64).transpose(0, 2, 1, 3) for i in range(3))
        s = q @ k.transpose(0, 1, 3, 2) * 0.125
        p = np.exp(s - np.max(s, axis=-1, keepdims=True))
        ref = (p @ v / p.sum(axis=-1, keepdims=True)).transpose(0, 2, 1, 3)
    d = to_dev(qkv, "f32")
    o = torch.full((B, N, H, 64), 7.0, device="cuda")
    rs.rs_attention_fwd(d[:, :, 0], d[:, :, 1], d[:, :, 2], o, 0.125)
    torch.cuda.synchronize()
    got, fin = to_host(o), np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), fin) and np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    assert norm_err(got[fin], ref[fin]) < TOL["f32"]


@pytest.mark.parametrize("value", [-1e4, -1e9, -1e10, -1e11, -1e30, float(np.finfo(np.float32).min)])
@pytest.mark.parametrize("N,masked", [(31, range(0, 22)), (128, range(0, 127)), (128, range(96, 128)), (161, range(32, 64)),
                                      (161, range(0, 96)), (200, [*range(0, 40), *range(64, 200)])])
def test_fp32_attention_low_values_as_a_mask(N, masked, value):
    """Low finite values through a reserved channel swallow the rest of a score: such keys weigh nothing beside others."""
    B, H = 2, 2
    _say("fp32 attention low value", N, masked, value)
    qkv = si.generic(48, 1, (B, N, 3, H, 64))
    qkv[:, :, 0, :, 63], qkv[:, :, 1, :, 63] = 1.0, 0.0
    seen = np.setdiff1d(np.arange(N), list(masked))
    q, k, v = (qkv[:, :, i].astype(np.float64).transpose(0, 2, 1, 3) for i in range(3))
    s = q @ k[:, :, seen].transpose(0, 1, 3, 2) * 0.125
    p = np.exp(s - s.max(axis=-1, keepdims=True))
    ref = (p @ v[:, :, seen] / p.sum(axis=-1, keepdims=True)).transpose(0, 2, 1, 3)
    qkv[:, list(masked), 1, :, 63] = value
    d = to_dev(qkv, "f32")
    o = torch.full((B, N, H, 64), 7.0, device="cuda")
    rs.rs_attention_fwd(d[:, :, 0], d[:, :, 1], d[:, :, 2], o, 0.125)
    torch.cuda.synchronize()
    err = norm_err(to_host(o), ref)
    assert err < TOL["f32"]


# M, K, N that go to the 64-row tiles the waves share on 256 CUs, and the workgroups per CU (the CPU tests hold the choice to that): 1.5
# rounds at short K, a last round at least 0.9 full at long K, four to five and more rounds; 2, 6, 14, 24, 26 and 34 slices; one row in the last tile
SHARED_TILES = [(6208, 64, 256, 4), (24576, 64, 64, 4), (29505, 448, 64, 4), (10088, 768, 192, 4), (9857, 832, 192, 4), (21845, 192, 192, 3), (8193, 192, 768, 4),
                (25601, 768, 192, 3), (4545, 1088, 1024, 3)]


@pytest.mark.parametrize("M,K,N", [c[:3] for c in SHARED_TILES])
def test_fp32_shared_tiles_same_bits(M, K, N):
    """The bits of the same rows in calls too small for the shared tiles."""
    _say("fp32 shared tiles", M, K, N)
    g = torch.Generator(device="cuda").manual_seed(M + K)
    a, w = torch.randn((M, K), device="cuda", generator=g), torch.randn((K, N), device="cuda", generator=g)
    b, res = torch.randn((N,), device="cuda", generator=g), torch.randn((M, N), device="cuda", generator=g)
    whole, parts = (torch.full((M + 1, N), float("nan"), device="cuda") for _ in range(2))
    rs.rs_linear_fwd(a, w, b, res, whole[:M], rs.RS_EPI_BIAS_RES)
    step = 1024 if N > 64 else 2048
    for r in range(0, M, step):
        rs.rs_linear_fwd(a[r:r + step], w, b, res[r:r + step], parts[r:min(r + step, M)], rs.RS_EPI_BIAS_RES)
    torch.cuda.synchronize()
    assert torch.isnan(whole[M]).all() and torch.equal(whole[:M], parts[:M]) and torch.isfinite(whole[:M]).all()
