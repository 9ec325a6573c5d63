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


@pytest.mark.parametrize("M,N,K", [(16, 40000, 32), (16, 40001, 32), (2501, 40016, 32),
                                   (16, 81920, 33), (15, 81921, 33), (15, 81921, 128), (16, 81924, 129),
                                   (1300, 83200, 100), (1301, 83200, 100)])
def test_pre_pass_of_wide_operands(M, N, K):
    """Both sides of the lines between the pre-pass of one launch and of two: the
    codes that the product leaves in its workspace."""
    case(f"gemm fp8 {M}x{N}x{K}")
    g = torch.Generator(device=dev()).manual_seed(99)
    A, B = torch.randn(M, K, device=dev(), generator=g), torch.randn(K, N, device=dev(), generator=g)
    C = torch.empty(M, N, device=dev())
    ws = torch.full((desc.desc_gemm_workspace("fp8", M, N, K),), 0x5A, dtype=torch.uint8,
                    device=dev())
    desc.desc_gemm(A, B, C, mode="fp8", ws=ws)
    up = lambda x, m: -(-x // m) * m
    rows, kp = (up(M, 256), up(N, 256)), up(K, 128)
    scales = up(rows[0] * kp, 256) + up(rows[1] * kp, 256)
    for at, r, X, scale in ((0, rows[0], A, scales),
                            (up(rows[0] * kp, 256), rows[1], B.t(), scales + up(4 * rows[0], 256))):
        q = torch.empty(X.shape, dtype=torch.uint8, device=dev())
        want = torch.empty(X.shape[0], device=dev())
        desc.desc_quant_e4m3_rows(X.contiguous(), q, want)
        got = ws[at:at + r * kp].view(r, kp)
        assert torch.equal(got[:X.shape[0], :K], q)
        assert not bool(got[X.shape[0]:].any()) and not bool(got[:, K:].any())
        assert torch.equal(ws[scale:scale + 4 * X.shape[0]].view(torch.float32), want)
