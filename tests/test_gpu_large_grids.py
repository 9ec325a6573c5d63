"""Calls whose block counts pass what one grid dimension takes in the form that
is fastest for ordinary sizes.  A launch of 2^32 threads or more along x is not
refused: it runs the count modulo 2^32, so a form may only be chosen where its
grid fits."""
import pytest
import torch

import paper_2305_03448_amd as desc
from gpu_util import case, dev, needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]


WIDE = 65535 * 32 + 33               # columns: more than 65535 blocks of 32


@pytest.fixture(autouse=True)
def _release():
    yield
    torch.cuda.empty_cache()


@pytest.mark.parametrize("elem,rows,cols", [(8, 2, (1 << 29) + 1), (4, 4, (1 << 30) + 1),
                                            (2, 8, (1 << 30) + 1), (1, 16, (1 << 30) + 1),
                                            (4, 1, (1 << 30) + 1)])
def test_transpose_of_many_columns(elem, rows, cols):
    case(f"transpose {elem}-byte {rows}x{cols}")
    dtype = {1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}[elem]
    # rows of random values whose period shares no factor with a tile
    g = torch.Generator(device=dev()).manual_seed(81)
    part = torch.randint(0, (1 << (8 * elem - 1)) - 1, (65521,), device=dev(), generator=g).to(dtype)
    x = torch.empty(rows, cols, dtype=dtype, device=dev())
    for r in range(rows):
        x[r] = part.roll(r).repeat(-(-cols // part.numel()))[:cols]
    y = torch.zeros(cols + 1, rows, dtype=dtype, device=dev())
    y[cols] = 77                         # beside the result
    desc.desc_transpose_batched(x, y[:cols])
    for r in range(rows):
        assert torch.equal(y[:cols, r], x[r])
    assert bool((y[cols] == 77).all())


@pytest.mark.parametrize("M", [1 << 30, (1 << 30) + (1 << 20) + 3])
def test_f32_product_of_many_rows(M):
    case(f"gemm f32 {M}x1x1")
    A = (torch.arange(M, dtype=torch.int32, device=dev()) % 1021).float().view(M, 1)
    C = torch.full((M + 1, 1), -7.0, device=dev())
    desc.desc_gemm(A, torch.full((1, 1), 3.0, device=dev()), C[:M], mode="f32")
    assert torch.equal(C[:M], A * 3)     # integers: exact
    assert float(C[M]) == -7.0


def test_fp8_product_whose_pre_pass_is_not_launched():
    """2^26 rows of K up to 2048: more blocks of 512 threads than a grid counts,
    eight rows to a block.  The call says so, or its result is right: never a
    product of codes that were not written."""
    M, N, K = 1 << 26, 1, 1
    case(f"gemm fp8 {M}x{N}x{K}")
    A = torch.full((M, K), 3.0, device=dev())
    B = torch.full((K, N), 2.0, device=dev())
    C = torch.full((M, N), -7.0, device=dev())
    ws = torch.zeros(desc.desc_gemm_workspace("fp8", M, N, K), dtype=torch.uint8, device=dev())
    try:
        desc.desc_gemm(A, B, C, mode="fp8", ws=ws)
    except desc.DescError:
        return
    # 448 * 448 scaled by 3 / 448 and 2 / 448: three roundings of 2^-24 each
    assert bool(((C - 6.0).abs() <= 6.0 * 2.0 ** -21).all())


def _e4m3(shape, seed):
    """448 / 2^i (i = 0..2), of either sign, or 0, with 448 in row K // 2 (or
    column K // 2): unit scales, and products and short sums exact in FP32."""
    g = torch.Generator(device=dev()).manual_seed(seed)
    s = torch.randint(-1, 2, shape, device=dev(), generator=g, dtype=torch.int8).float()
    return 448 * s / 2.0 ** torch.randint(0, 3, shape, device=dev(), generator=g, dtype=torch.int8)


def test_fp8_product_of_many_columns():
    M, N, K = 1, WIDE, 2049
    case(f"gemm fp8 {M}x{N}x{K}")
    A, part = _e4m3((M, K), 81), _e4m3((K, 1023), 82)
    A[:, K // 2] = 448
    part[K // 2] = 448
    B = part.repeat(1, -(-N // 1023))[:, :N].contiguous()
    want = (A.double() @ part.double()).float().repeat(1, -(-N // 1023))[:, :N]
    C = torch.full((M, N), -7.0, device=dev())
    desc.desc_gemm(A, B, C, mode="fp8")
    assert torch.equal(C, want)


@pytest.mark.parametrize("K", [511, 512])
def test_fp8_column_codes_of_many_columns(K):
    N = WIDE
    case(f"quant e4m3 cols {K}x{N}")
    g = torch.Generator(device=dev()).manual_seed(83)
    part = torch.randn(K, 1023, device=dev(), generator=g)
    B = part.repeat(1, -(-N // 1023))[:, :N].contiguous()
    q = torch.full((N, K), 0x55, dtype=torch.uint8, device=dev())
    s = torch.full((N,), -7.0, device=dev())
    desc.desc_quant_e4m3_cols(B, q, s)
    want_q = torch.empty(1023, K, dtype=torch.uint8, device=dev())
    want_s = torch.empty(1023, device=dev())
    desc.desc_quant_e4m3_rows(part.t().contiguous(), want_q, want_s)
    for at in range(0, N, 1023):
        n = min(1023, N - at)
        assert torch.equal(q[at:at + n], want_q[:n]) and torch.equal(s[at:at + n], want_s[:n]), at


def test_row_codes_of_many_rows():
    M, K = (1 << 24) + 5, 4
    case(f"quant e4m3 rows {M}x{K}")
    g = torch.Generator(device=dev()).manual_seed(85)
    part = torch.randn(4099, K, device=dev(), generator=g)
    A = part.repeat(-(-M // 4099), 1)[:M].contiguous()
    q = torch.full((M + 1, K), 0x55, dtype=torch.uint8, device=dev())
    s = torch.full((M + 1,), -7.0, device=dev())
    desc.desc_quant_e4m3_rows(A, q[:M], s[:M])
    want_q = torch.empty(4099, K, dtype=torch.uint8, device=dev())
    want_s = torch.empty(4099, device=dev())
    desc.desc_quant_e4m3_rows(part, want_q, want_s)
    assert torch.equal(q[:M], want_q.repeat(-(-M // 4099), 1)[:M])
    assert torch.equal(s[:M], want_s.repeat(-(-M // 4099))[:M])
    assert bool((q[M] == 0x55).all()) and float(s[M]) == -7.0


@pytest.mark.parametrize("B", [(1 << 24) + 3, (1 << 26) + 3])
def test_many_rows_reduced_and_scanned(B):
    """More segments than one grid counts, a block each or four to a block."""
    L = 2
    case(f"batched {B}x{L}")
    x = (torch.arange(B * L, dtype=torch.int32, device=dev()) % 1021).view(B, L)
    r = torch.full((B + 1,), 5, dtype=torch.int64, device=dev())
    desc.desc_reduce_batched_i32(x, r[:B])
    both = x[:, 0] + x[:, 1]
    assert torch.equal(r[:B], both.long()) and int(r[B]) == 5
    del r
    y = torch.full((B + 1, L), -5, dtype=torch.int32, device=dev())
    desc.desc_scan_batched_i32(x, y[:B])
    assert torch.equal(y[:B, 0], x[:, 0]) and torch.equal(y[:B, 1], both)
    assert bool((y[B] == -5).all())


def test_chunk_sums_of_many_chunks():
    chunks, E = (1 << 24) + 3, 1024
    case(f"chunk sums {chunks}x{E}")
    x = torch.empty(chunks, E, dtype=torch.int32, device=dev())
    ids = torch.arange(chunks, dtype=torch.int32, device=dev()) % 1021
    x[:] = ids.view(-1, 1)
    out = torch.full((chunks + 1,), -5, dtype=torch.int64, device=dev())
    desc.desc_reduce_blocks_i32(x.view(-1)[:-1], E, out[:chunks])
    want = ids.long() * E
    want[-1] -= ids[-1]
    assert torch.equal(out[:chunks], want) and int(out[chunks]) == -5
