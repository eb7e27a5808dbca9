"""Long-sequence attention with 128 and with 256 query rows per workgroup: one head alone goes to the smaller tile, the same head
among enough others that the larger one fills the chip as well goes to that, and a row's arithmetic is the same in
both.  Lengths around the tiles of rows and of keys, and rows that end in every wave of the smaller tile."""
import pytest
import torch

import oracle
import paper_2508_00367_amd as rs
from rs_testlib import TOL, norm_err, to_host

pytestmark = pytest.mark.gpu


# 256 rows per workgroup on 256 CUs with so many heads, 128 with one; the CPU tests hold the rule to that
ROW_TILES = [(257, 128), (288, 128), (320, 128), (384, 128), (385, 128), (416, 128), (448, 128), (449, 128), (511, 128), (512, 128), (640, 160),
             (1025, 40)]


@pytest.mark.parametrize("N,heads", ROW_TILES)
def test_row_tiles_same_bits(N, heads):
    print("attention row tiles", N, heads, flush=True)
    g = torch.Generator(device="cuda").manual_seed(N)
    qkv = torch.randn((1, N, 3, heads, 64), device="cuda", generator=g).bfloat16()
    one = torch.full((1, N + 1, 1, 64), float("nan"), device="cuda", dtype=torch.bfloat16)
    many = torch.full((1, N + 1, heads, 64), float("nan"), device="cuda", dtype=torch.bfloat16)
    h = heads - 1
    rs.rs_attention_fwd(qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2], many[:, :N], 0.125)
    rs.rs_attention_fwd(qkv[:, :, 0, h:], qkv[:, :, 1, h:], qkv[:, :, 2, h:], one[:, :N], 0.125)
    torch.cuda.synchronize()
    assert torch.isnan(one[:, N]).all() and torch.isnan(many[:, N]).all()      # nothing written behind the last row
    ref = oracle.attention(*(to_host(qkv[:, :, i, h:]) for i in range(3)), 0.125)
    assert norm_err(to_host(one[:, :N]), ref) < TOL["bf16"] and norm_err(to_host(many[:, :N, h:]), ref) < TOL["bf16"]
    assert torch.equal(one[0, :N, 0].view(torch.int16), many[0, :N, h].view(torch.int16))


@pytest.mark.parametrize("heads", [1, 128])
@pytest.mark.parametrize("pad", [0, 8, (1 << 24) - 8, 1 << 24])
@pytest.mark.parametrize("N", [1, 31, 33, 48, 49, 65, 129, 257])
def test_output_rows_at_any_stride(N, pad, heads):
    """Output rows side by side, ragged and around 2^24 elements apart (32 rows beyond 32-bit byte offsets): the same bits,
    and nothing between the rows or behind the last one.  257 rows: the long kernel, of 4 waves with one head and of 8 with 128."""
    print("attention output stride", N, pad, heads, flush=True)
    if N > 129 and pad > 8:
        N = 131 if pad & 8 else 257           # one of the far strides for the long kernel, 8.6 GB
    width = heads * 64
    stride = pad if pad > width else width + pad
    g = torch.Generator(device="cuda").manual_seed(N)
    qkv = torch.randn((1, N, 3, heads, 64), device="cuda", generator=g).bfloat16()
    near = torch.empty((1, N, heads, 64), device="cuda", dtype=torch.bfloat16)
    buf = torch.full((N * stride + 64,), 7.0, device="cuda", dtype=torch.bfloat16)
    far = buf.as_strided((1, N, heads, 64), (0, stride, 64, 1))
    for o in (near, far):
        rs.rs_attention_fwd(qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2], o, 0.125)
    torch.cuda.synchronize()
    assert torch.equal(near, far)
    some = slice(0, heads, max(1, heads - 1))  # the first and the last head
    assert norm_err(to_host(near[:, :, some]), oracle.attention(*(to_host(qkv[:, :, i, some]) for i in range(3)), 0.125)) < TOL["bf16"]
    if stride > width:
        assert (buf[:N * stride].view(N, stride)[:, width:width + min(64, stride - width)] == 7.0).all()
    assert (buf[N * stride:] == 7.0).all()
