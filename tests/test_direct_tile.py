"""The direct GEMM tile (FP32 and split BF16) and the clamped LDS-staged one: their index maps on
the host, every form on the GPU at the edges of its tiles, and the mixed tiles
of the grouped GEMM, against exact integer products."""
import os
import subprocess

import numpy as np
import pytest
import torch

import paper_2305_03448_amd as desc
import workloads
from gpu_util import bf16x3_bound, case, needs_gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2305_03448_amd", "csrc")


def test_direct_tile_maps(tmp_path):
    exe = str(tmp_path / "direct_tile_checks")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC,
                    os.path.join(ROOT, "tests", "direct_tile_checks.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.count("OK ") == 7, r.stdout


FORMS = [(128, 128), (64, 128), (128, 64), (96, 96), (64, 96), (96, 64), (64, 64), (48, 64),
         (64, 48), (48, 48), (32, 64), (64, 32), (32, 32), (16, 64), (64, 16), (16, 32), (32, 16),
         (16, 16)]


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("bm,bn,name", [(m, n, f"d{m}x{n}") for m, n in FORMS]
                         + [(128, 128, "m128n128k16_c")])
def test_direct_form_edges(bm, bn, name):
    # integers: every sum is exact in FP32 in any order, so equality is asked.
    # The padding beside A's rows and B's columns holds NaN, which must stay out.
    op = "gemm_f32"
    names = [desc.desc_config_name(op, c) for c in range(desc.desc_config_count(op))]
    try:
        for cls in range(4):
            desc.desc_config_set(op, cls, names.index(name))
        for M, N, K, pad in [(bm, bn, 256, 0), (bm + 1, bn + 1, 17, 3), (bm - 1, bn - 1, 15, 1),
                             (1, 4, 1, 0), (2 * bm + 5, 3 * bn + 2, 1041, 0), (3, 2, 33, 1),
                             (bm, 2 * bn - 3, 0, 0), (5, bn + 2, 64, 2)]:
            case(f"gemm f32 {name} {M}x{N}x{K} pad {pad}")
            g = workloads.rng(50)
            A = g.integers(-4, 5, size=(M, K)).astype(np.float32)
            B = g.integers(-4, 5, size=(K, N)).astype(np.float32)

            def padded(x):
                t = torch.full((x.shape[0], x.shape[1] + pad), float("nan"), device="cuda")
                t[:, :x.shape[1]] = torch.from_numpy(x).cuda()
                return t[:, :x.shape[1]]
            buf = torch.full((M + 1, N + pad), -7.0, device="cuda")
            desc.desc_gemm(padded(A), padded(B), buf[:M, :N])
            want = (A.astype(np.int64) @ B.astype(np.int64)).astype(np.float32)
            got = buf.cpu().numpy()
            assert np.array_equal(got[:M, :N], want)
            assert (got[M:] == -7).all() and (got[:, N:] == -7).all(), "wrote outside C"
    finally:
        for cls in range(4):
            desc.desc_config_set(op, cls, -1)


SPLIT_FORMS = [(128, 128), (64, 128), (128, 64), (64, 64), (48, 48), (32, 64), (32, 32), (16, 64),
               (16, 32), (32, 16), (16, 16)]


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("bm,bn", SPLIT_FORMS)
def test_direct_split_form_edges(bm, bn):
    # small integers are bfloat16 values (lo = 0) and their sums exact in FP32:
    # equality; then N(0, 1) within the mode's a-priori bound
    op = "gemm_bf16x3"
    names = [desc.desc_config_name(op, c) for c in range(desc.desc_config_count(op))]
    try:
        for cls in range(4):
            desc.desc_config_set(op, cls, names.index(f"d{bm}x{bn}"))
        for M, N, K, pad in [(bm, bn, 256, 0), (bm + 1, bn + 1, 33, 3), (bm - 1, bn - 1, 31, 1),
                             (1, 4, 1, 0), (2 * bm + 5, 3 * bn + 2, 1041, 0), (3, 2, 65, 1)]:
            case(f"gemm bf16x3 d{bm}x{bn} {M}x{N}x{K} pad {pad}")
            g = workloads.rng(52)

            def padded(x):
                t = torch.full((x.shape[0], x.shape[1] + pad), float("nan"), device="cuda")
                t[:, :x.shape[1]] = torch.from_numpy(x).cuda()
                return t[:, :x.shape[1]]
            for normal in (False, True):
                draw = ((lambda s: g.standard_normal(s).astype(np.float32)) if normal
                        else (lambda s: g.integers(-4, 5, size=s).astype(np.float32)))
                A, B = draw((M, K)), draw((K, N))
                buf = torch.full((M + 1, N + pad), -7.0, device="cuda")
                desc.desc_gemm(padded(A), padded(B), buf[:M, :N], mode="bf16x3")
                got = buf.cpu().numpy()
                assert (got[M:] == -7).all() and (got[:, N:] == -7).all(), "wrote outside C"
                A, B = A.astype(np.float64), B.astype(np.float64)
                err = np.abs(got[:M, :N] - A @ B)
                assert (err <= (bf16x3_bound(K) * (np.abs(A) @ np.abs(B)) if normal else 0)).all()
    finally:
        for cls in range(4):
            desc.desc_config_set(op, cls, -1)


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("count", [1, 45, 1100])   # small tiles; both sizes; prefixes outside LDS
def test_grouped_mixed_tiles(count):
    # odd shapes and strides, NaN beside every row, K = 0, N below a group of
    # four, whole tiles, a row stride beyond the tiles' 2^31-byte spans
    case(f"grouped f32 mixed tiles, {count} problems")
    g = workloads.rng(51)
    edge = [(128, 128, 16), (129, 255, 33), (300, 3, 70), (5, 700, 0), (384, 256, 160), (1, 1, 1)]
    top = 400 if count < 1000 else 40
    shapes = (edge + [tuple(int(v) for v in g.integers(1, top, size=3)) for _ in range(count)])
    # enough whole 128 x 128 tiles for the large form
    shapes = shapes[:count] if count == 1 else shapes[:count] + [(1024, 1536, 50), (1000, 1800, 48)]
    problems, want, bufs = [], [], []
    for i, (M, N, K) in enumerate(shapes):
        A = g.integers(-4, 5, size=(M, K)).astype(np.float32)
        B = g.integers(-4, 5, size=(K, N)).astype(np.float32)
        pad = i % 3

        def padded(x, ld=0):
            t = torch.full((x.shape[0], max(x.shape[1] + pad, ld)), float("nan"), device="cuda")
            t[:, :x.shape[1]] = torch.from_numpy(x).cuda()
            return t[:, :x.shape[1]]
        buf = torch.full((M + 1, N + pad), -7.0, device="cuda")
        # rows of A 2^24 floats apart: 64 of them span 2^32 bytes
        ld = 1 << 24 if count == 45 and (M, N, K) == (129, 255, 33) else 0
        problems.append((padded(A, ld), padded(B), buf[:M, :N]))
        bufs.append(buf)
        want.append((A.astype(np.int64) @ B.astype(np.int64)).astype(np.float32))
    d = desc.grouped_descriptors(problems, torch.device("cuda"))
    desc.desc_gemm_grouped(d, mode="f32")
    torch.cuda.synchronize()
    for (M, N, K), buf, w in zip(shapes, bufs, want):
        got = buf.cpu().numpy()
        assert np.array_equal(got[:M, :N], w), (M, N, K)
        assert (got[M:] == -7).all() and (got[:, N:] == -7).all(), "wrote outside C"


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("name,t", [("fused32x32", 32), ("d32x32", 32), ("d64x64", 64),
                                    ("by_shape", 32)])
def test_fp8_small_forms(name, t):
    # e4m3 values 448 / 2^i with 448 in every row and column: unit scales, and
    # products and sums that are exact in the instruction and in FP32
    op = "gemm_fp8"
    names = [desc.desc_config_name(op, c) for c in range(desc.desc_config_count(op))]

    def padded(x, pad):
        b = torch.full((x.shape[0], x.shape[1] + pad), float("nan"), device="cuda")
        b[:, :x.shape[1]] = torch.from_numpy(x).cuda()
        return b[:, :x.shape[1]]
    try:
        for cls in range(4):
            desc.desc_config_set(op, cls, names.index(name))
        for M, N, K, pad in [(t, t, 64, 0), (t + 1, t - 1, 65, 3), (1, 1, 1, 0), (3 * t + 5, 2, 63, 1),
                             (2 * t, 5 * t + 3, 1024, 0), (t - 1, 2 * t + 7, 1025, 2),
                             (40, 70, 2500, 1), (7, 5, 0, 0), (600, 900, 130, 0)]:
            case(f"gemm fp8 {name} {M}x{N}x{K} pad {pad}")
            g = workloads.rng(53)
            A, B = (np.float32(448) * (g.integers(-1, 2, size=s) / 2.0 ** g.integers(0, 3, size=s))
                    .astype(np.float32) for s in ((M, K), (K, N)))
            if K:
                A[:, K // 2] = 448
                B[K // 2, :] = 448
            buf = torch.full((M + 1, N + pad), -7.0, device="cuda")
            desc.desc_gemm(padded(A, pad), padded(B, pad), buf[:M, :N], mode="fp8")
            got = buf.cpu().numpy()
            assert np.array_equal(got[:M, :N], (A.astype(np.float64) @ B.astype(np.float64))
                                  .astype(np.float32))
            assert (got[M:] == -7).all() and (got[:, N:] == -7).all(), "wrote outside C"
        # magnitudes whose scale overflows, zero rows, infinities and NaN: the
        # same bits as the plane form (K = 40 is one instruction a tile)
        A, B = (g.standard_normal(s).astype(np.float32) for s in ((70, 40), (40, 50)))
        A[3] *= np.float32(1e-38); A[5] = 0; A[7, 2] = np.inf; A[9, 1] = np.nan; B[:, 4] = 0
        B[:, 6] *= np.float32(1e-39); B[5, 8] = -np.inf
        out = []
        for cfg in (name, "m128n128k128"):
            for cls in range(4):
                desc.desc_config_set(op, cls, names.index(cfg))
            C = torch.empty((70, 50), device="cuda")
            desc.desc_gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), C, mode="fp8")
            out.append(C.cpu().numpy())
        assert np.array_equal(out[0], out[1], equal_nan=True)
    finally:
        for cls in range(4):
            desc.desc_config_set(op, cls, -1)
