"""Products on both sides of the lines that choose a form by M, N and K,
against exact integer products: operands that are and are not in 16-byte
groups, NaN beside every row, and guard words around C."""
import numpy as np
import pytest
import torch

import paper_2305_03448_amd as desc
import workloads
from gpu_util import case, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]


def _check(M, N, K, pad, mode="f32"):
    case(f"gemm {mode} {M}x{N}x{K} pad {pad}")
    g = workloads.rng(91)
    A = g.integers(-4, 5, size=(M, K)).astype(np.float32)
    B = g.integers(-4, 5, size=(K, N)).astype(np.float32)

    def padded(x):
        t = torch.full((x.shape[0], x.shape[1] + pad), float("nan"), device="cuda")
        t[:, :x.shape[1]] = torch.from_numpy(x).cuda()
        return t[:, :x.shape[1]]
    buf = torch.full((M + 1, N + pad), -7.0, device="cuda")
    desc.desc_gemm(padded(A), padded(B), buf[:M, :N], mode=mode)
    want = (A.astype(np.float64) @ B.astype(np.float64)).astype(np.float32)
    got = buf.cpu().numpy()
    assert np.array_equal(got[:M, :N], want)
    assert (got[M:] == -7).all() and (got[:, N:] == -7).all(), "wrote outside C"


@pytest.mark.parametrize("pad", [0, 1, 4])
@pytest.mark.parametrize("M,N,K", [
    (16384, 64, 32), (16385, 64, 32),            # 256 tiles of 64 x 64, 257
    (3201, 500, 64), (3200, 512, 65),            # K limit of operands in groups
    (20000, 30, 16), (20000, 30, 17),            # and of the others
    (30000, 47, 32), (30000, 47, 33), (30000, 23, 16), (30000, 24, 16),
    (24576, 100, 16), (49153, 64, 16)])          # one residency, and past it
def test_short_k(M, N, K, pad):
    _check(M, N, K, pad)


@pytest.mark.parametrize("M,N,K", [
    (3071, 4097, 128), (3073, 3969, 128),         # 792 and 800 tiles of 128 x 128
    (4000, 4000, 127), (4000, 4000, 131),         # 1024, both sides of its least K
    (4097, 3969, 128)])                           # 1056
def test_one_residency_of_clamped_tiles(M, N, K):
    _check(M, N, K, 1)
    _check(M, N, K, 0)


@pytest.mark.parametrize("pad", [0, 1, 4])
@pytest.mark.parametrize("M,N,K", [(3200, 512, 15), (3200, 512, 16), (3200, 512, 28), (3201, 509, 28),
                                   (3200, 512, 31), (3200, 512, 32), (50000, 31, 20)])
def test_split_below_one_stage(M, N, K, pad):
    # small integers are bfloat16 values: exact products
    _check(M, N, K, pad, "bf16x3")


@pytest.mark.parametrize("M,N,K", [
    (512, 512, 64), (545, 512, 64),               # 256 tiles of 32 x 32, 288
    (1024, 512, 512), (512, 1025, 512),           # 512, 528
    (32, 16384, 256), (32, 16384, 257), (33, 8192, 257), (16000, 17, 1024), (16000, 17, 1025),
    (1024, 1024, 64), (1025, 1024, 64)])          # 256 tiles of 64 x 64, 272
def test_fp8_forms_of_few_tiles(M, N, K):
    # e4m3 values 448 / 2^i with 448 in every row and column: unit scales, and
    # products and sums that are exact in the instruction and in FP32
    case(f"gemm fp8 {M}x{N}x{K}")
    g = workloads.rng(95)
    A, B = (np.float32(448) * (g.integers(-1, 2, size=s) / 2.0 ** g.integers(0, 3, size=s))
            .astype(np.float32) for s in ((M, K), (K, N)))
    A[:, K // 2] = 448
    B[K // 2, :] = 448
    buf = torch.full((M + 1, N), -7.0, device="cuda")
    desc.desc_gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), buf[:M], mode="fp8")
    want = (torch.from_numpy(A).cuda().double() @ torch.from_numpy(B).cuda().double()).float()
    assert torch.equal(buf[:M], want)
    assert bool((buf[M] == -7).all()), "wrote outside C"
