"""The e4m3 codes and scales of B's columns, bit for bit against those of the
rows of its transpose, in each form of the encode: LDS tiles, blocks of 512 k x
32 columns, blocks of 128 x 128; operands that start on and off a 16-byte
boundary, rows that all start at the same offset from one and rows that do not,
codes at any alignment, edges in both directions, zero columns, NaN and
infinities."""
import pytest
import torch

import paper_2305_03448_amd as desc
from gpu_util import case, dev, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

CASES = [(300, 27000), (511, 17000), (511, 66000), (127, 70000),     # 128 x 128
         (512, 33000), (4096, 4100), (4095, 8200), (8000, 2003),     # 512 x 32
         (2100, 4101), (300, 27003), (6144, 5001), (6145, 5001)]     # odd rows, up to K = 6144


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("K,N", CASES)
def test_column_codes(K, N, offset):
    case(f"quant e4m3 cols {K}x{N} offset {offset}")
    g = torch.Generator(device=dev()).manual_seed(97)
    B = torch.empty(K * N + offset, device=dev())[offset:].view(K, N)
    B.copy_(torch.randn(K, N, device=dev(), generator=g))
    B[:, 5] = 0
    B[:, N - 2] = 1e-43                   # 448 / amax is infinite
    B[K - 1, N - 1] = float("nan")
    B[K // 2, 7] = float("inf")
    q = torch.full((N * K + offset + 16,), 0x55, dtype=torch.uint8, device=dev())
    s = torch.full((N + 1,), -7.0, device=dev())
    desc.desc_quant_e4m3_cols(B, q[offset:offset + N * K].view(N, K), s[:N])
    want_q = torch.empty(N, K, dtype=torch.uint8, device=dev())
    want_s = torch.empty(N, device=dev())
    desc.desc_quant_e4m3_rows(B.t().contiguous(), want_q, want_s)
    assert torch.equal(q[offset:offset + N * K].view(N, K), want_q)
    assert torch.equal(s[:N].view(torch.int32), want_s.view(torch.int32))
    assert bool((q[:offset] == 0x55).all()) and bool((q[offset + N * K:] == 0x55).all())
    assert float(s[N]) == -7.0
