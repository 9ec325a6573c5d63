"""The FP8 GEMM's one-launch pre-pass (K up to 2048): the codes and scales it
leaves in the workspace against those of desc_quant_e4m3_rows of A and of B
transposed, bit for bit, and the padding of its planes against zero.  K at both
sides of each kernel's limit and of a thread's 4, 8 and 16 rows, N at both
sides of a strip of 16 columns, an operand that starts one element past a
16-byte boundary, zero rows and columns, tiny ones (whose scale factor
overflows), infinities and NaN."""
import pytest
import torch

import paper_2305_03448_amd as desc
from gpu_util import case, dev, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

CASES = [(1, 1, 1), (5, 15, 3), (9, 16, 127), (8, 17, 128), (7, 257, 129), (300, 33, 511),
         (31, 300, 512), (257, 15, 513), (3, 47, 1023), (64, 64, 1025), (33, 272, 2047),
         (255, 31, 2048)]


def _up(x, m):
    return -(-x // m) * m


def _prepass(A, B):
    """(codes, scales) of A [Mp][Kp] and B^T [Np][Kp] as the call left them."""
    M, K = A.shape
    N = B.shape[1]
    C = torch.empty(M, N, device=dev())
    ws = torch.full((desc.desc_gemm_workspace("fp8", M, N, K),), 0x5A, dtype=torch.uint8,
                    device=dev())
    desc.desc_gemm(A, B, C, mode="fp8", ws=ws)
    out, at = [], 0
    rows, kp = (_up(M, 256), _up(N, 256)), _up(K, 128)
    for r in rows:
        out.append(ws[at:at + r * kp].view(r, kp))
        at += _up(r * kp, 256)
    for r in rows:
        out.append(ws[at:at + 4 * r].view(torch.float32))
        at += _up(4 * r, 256)
    return out


def _rows(X):
    q = torch.empty(X.shape, dtype=torch.uint8, device=dev())
    s = torch.empty(X.shape[0], device=dev())
    desc.desc_quant_e4m3_rows(X, q, s)
    return q, s


@pytest.fixture
def staged():
    names = [desc.desc_config_name("gemm_fp8", c) for c in range(desc.desc_config_count("gemm_fp8"))]
    for cls in range(4):
        desc.desc_config_set("gemm_fp8", cls, names.index("m128n128k128"))
    yield
    for cls in range(4):
        desc.desc_config_set("gemm_fp8", cls, -1)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("shape", CASES)
def test_codes_and_scales(shape, offset, staged):
    M, N, K = shape
    case(f"fp8 one-launch pre-pass {shape} offset {offset}")
    g = torch.Generator().manual_seed(71)
    A = torch.randn(M, K, generator=g) * 3
    B = torch.randn(K, N, generator=g) * 0.1
    if M > 4 and N > 4:
        A[1] = 0
        B[:, 2] = 0
        A[2] = 1e-43                     # 448 / amax is infinite
        B[:, 3] = 1e-43
        A[3, K // 2] = float("inf")
        B[K - 1, 4] = float("nan")
    bufA = torch.empty(M * K + offset, device=dev())
    bufB = torch.empty(K * N + offset, device=dev())
    dA, dB = bufA[offset:].view(M, K), bufB[offset:].view(K, N)
    dA.copy_(A)
    dB.copy_(B)
    qa, qb, sa, sb = _prepass(dA, dB)
    for got, scale, X in ((qa, sa, A), (qb, sb, B.t())):
        q, want = _rows(X.contiguous().to(dev()))
        r = X.shape[0]
        assert torch.equal(got[:r, :K], q)
        assert not bool(got[r:].any()) and not bool(got[:, K:].any())
        assert torch.equal(torch.nan_to_num(scale[:r]), torch.nan_to_num(want))
        assert torch.equal(torch.isnan(scale[:r]), torch.isnan(want))
        assert not bool(scale[r:].any())
