"""The 256 x 256 tiles staged to LDS directly, against the register-staged
tiles of the same size, bit for bit: both add the same products of the same
planes to each accumulator in ascending K order, so every element of C is the
same.  Shapes: one tile and several, whole and ragged edges, one to four
stages of K (odd counts run a stage of zeros), C with a padded row stride
whose padding stays untouched, and a result that takes the non-temporal
stores."""
import pytest
import torch

import paper_2305_03448_amd as desc
from gpu_util import case, dev, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

FORMS = {"fp8": ("gemm_fp8", "m256n256k128_w8d1", "m256n256k128_dma"),
         "bf16x3": ("gemm_bf16x3", "m256n256k32_w8d1", "m256n256k32_dma")}
SHAPES = [(256, 256, 128), (1, 1, 1), (255, 257, 129), (300, 513, 384), (513, 40, 512),
          (257, 256, 1000)]


def _config(op, name):
    for c in range(desc.desc_config_count(op)):
        if desc.desc_config_name(op, c) == name:
            return c
    raise AssertionError(f"{op} has no configuration {name}")


def _run(mode, form, A, B, C, N):
    op = FORMS[mode][0]
    M, K = A.shape
    ws = torch.zeros(desc.desc_gemm_workspace(mode, M, N, K), dtype=torch.uint8, device=dev())
    for cls in range(4):
        desc.desc_config_set(op, cls, _config(op, form))
    try:
        desc.desc_gemm(A, B, C[:, :N], mode=mode, ws=ws)
    finally:
        for cls in range(4):
            desc.desc_config_set(op, cls, -1)
    return C


@pytest.mark.parametrize("mode", sorted(FORMS))
@pytest.mark.parametrize("shape", SHAPES)
def test_same_bits_as_register_staged(mode, shape):
    M, N, K = shape
    case(f"direct-to-LDS {mode} {shape}")
    g = torch.Generator().manual_seed(61)
    A = torch.randn(M, K, generator=g).to(dev())
    B = torch.randn(K, N, generator=g).to(dev())
    out = [_run(mode, form, A, B, torch.full((M, N + 3), -7.0, device=dev()), N)
           for form in FORMS[mode][1:]]
    assert torch.equal(out[0], out[1])
    assert bool((out[1][:, N:] == -7.0).all())


@pytest.mark.parametrize("mode", sorted(FORMS))
def test_result_past_the_cache(mode):
    M, N, K = 8193, 8192, 64
    case(f"direct-to-LDS {mode} {M} x {N} x {K}, non-temporal")
    g = torch.Generator(device=dev()).manual_seed(67)
    A = torch.randn(M, K, generator=g, device=dev())
    B = torch.randn(K, N, generator=g, device=dev())
    out = [_run(mode, form, A, B, torch.empty(M, N, device=dev()), N) for form in FORMS[mode][1:]]
    assert torch.equal(out[0], out[1])
