"""Long-sequence attention with 128 and with 256 query rows per workgroup: one head alone goes to the smaller tile, the same head
among enough others that the larger one fills the chip as well goes to that, and a row's arithmetic is the same in
both.  Lengths around the tiles of rows and of keys, and rows that end in every wave of the smaller tile."""
import pytest
import torch

import oracle
import paper_2508_00367_amd as rs
from rs_testlib import TOL, norm_err, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,heads", [(257, 160), (288, 160), (320, 160), (384, 160), (385, 128), (416, 128), (448, 128), (449, 128), (511, 128),
                                     (512, 128), (640, 160), (1025, 256)])
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
    if 0 < N % 256 <= 64:
        return                                # the rows behind whole tiles may be the tail kernel's, which splits the keys
    assert torch.equal(one[0, :N, 0].view(torch.int16), many[0, :N, h].view(torch.int16))


@pytest.mark.parametrize("stride", [64, 72, (1 << 24) - 8, 1 << 24])
@pytest.mark.parametrize("N", [1, 31, 33, 48, 49, 65, 129, 257])
def test_output_rows_at_any_stride(N, stride):
    """Output rows side by side, ragged and around 2^24 elements apart (32 rows beyond 32-bit byte offsets): the same bits,
    and nothing between the rows or behind the last one."""
    print("attention output stride", N, stride, flush=True)
    if N > 129 and stride > 72:
        N = 131 if stride & 8 else 257        # one of the far strides for the long kernel, 8.6 GB
    g = torch.Generator(device="cuda").manual_seed(N)
    qkv = torch.randn((1, N, 3, 1, 64), device="cuda", generator=g).bfloat16()
    near = torch.empty((1, N, 1, 64), device="cuda", dtype=torch.bfloat16)
    buf = torch.full((N * stride + 64,), 7.0, device="cuda", dtype=torch.bfloat16)
    far = buf.as_strided((1, N, 1, 64), (0, stride, 64, 1))
    for o in (near, far):
        rs.rs_attention_fwd(qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2], o, 0.125)
    torch.cuda.synchronize()
    assert torch.equal(near, far)
    assert norm_err(to_host(near), oracle.attention(*(to_host(qkv[:, :, i]) for i in range(3)), 0.125)) < TOL["bf16"]
    if stride > 64:
        assert (buf[:N * stride].view(N, stride)[:, 64:128] == 7.0).all()
    assert (buf[N * stride:] == 7.0).all()
