"""Every configuration of the word transpose keeps its tile on matrices that are
not whole tiles of aligned groups, at the edges of that tile, and the choice by
shape is a configuration of its own that the shipped table names."""
import pytest
import torch

import paper_2305_03448_amd as desc
from gpu_util import case, needs_gpu

OP = "transpose_32"


def test_the_shipped_table_chooses_by_shape():
    with open(desc.TUNE_FILE) as f:
        rows = [line.split() for line in f if line.startswith(OP + " ")]
    assert [(r[1], r[2]) for r in rows] == [(str(c), "by_shape") for c in range(4)]


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("name,t", [("t32", 32), ("t32_nt", 32), ("t64", 64), ("t64_nt", 64),
                                    ("t128", 128), ("t128_nt", 128), ("t128_b512", 128),
                                    ("t128_nt_b512", 128), ("by_shape", 128)])
def test_edges_of_a_configured_tile(name, t):
    names = [desc.desc_config_name(OP, c) for c in range(desc.desc_config_count(OP))]
    try:
        for cls in range(4):
            desc.desc_config_set(OP, cls, names.index(name))
        for batch, rows, cols, off in [(1, t, t, 0), (1, t, t, 1), (2, t - 1, t + 1, 0),
                                       (1, t + 3, t - 3, 3), (3, 2 * t + 5, 3 * t - 2, 0),
                                       (1, 4, 4, 1), (1, 3, 2 * t, 0), (1, 2 * t + 4, 4, 0),
                                       (1, 4 * t + 4, 5 * t, 0)]:
            case(f"transpose {name} {batch}x{rows}x{cols} offset {off}")
            n = batch * rows * cols
            raw = torch.randint(-(1 << 31), 1 << 31, (n + off,), device="cuda").to(torch.int32)
            x = raw[off:].view(batch, rows, cols)
            buf = torch.zeros(n + off + 8, dtype=torch.int32, device="cuda")
            y = buf[off:off + n].view(batch, cols, rows)
            desc.desc_transpose_batched(x, y)
            assert torch.equal(y, x.transpose(1, 2))
            assert int(buf[:off].abs().sum()) == 0 and int(buf[off + n:].abs().sum()) == 0
    finally:
        for cls in range(4):
            desc.desc_config_set(OP, cls, -1)


# Both sides of the sizes at which the tile changes: 2^16 words, 4 x 2^20 bytes
# and 16-bit elements, 6 x 2^20 words.
@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("elem,batch,rows,cols", [
    (4, 1, 255, 257), (4, 1, 257, 256), (4, 5, 1121, 1121), (4, 6, 1025, 1025), (1, 1, 2047, 2049),
    (1, 1, 2049, 2048), (2, 3, 1182, 1182), (2, 3, 1183, 1183), (1, 7, 77, 7777), (2, 7, 7777, 78)])
def test_sizes_where_the_tile_changes(elem, batch, rows, cols):
    case(f"transpose {elem}-byte {batch}x{rows}x{cols}")
    dtype = {1: torch.uint8, 2: torch.int16, 4: torch.int32}[elem]
    n = batch * rows * cols
    x = torch.randint(0, 256, (n * elem,), dtype=torch.uint8,
                      device="cuda").view(dtype).view(batch, rows, cols)
    buf = torch.zeros(n + 16, dtype=dtype, device="cuda")
    y = buf[8:8 + n].view(batch, cols, rows)
    desc.desc_transpose_batched(x, y)
    assert torch.equal(y, x.transpose(1, 2))
    assert int(buf[:8].abs().sum()) == 0 and int(buf[8 + n:].abs().sum()) == 0


# Streaming accesses, from 402 MB of both arrays in whole 128-byte output
# lines: whole lines of rows, a column count that is no multiple of a group.
@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("elem,rows,cols", [(1, 16384, 12291), (2, 8192, 12291), (4, 8192, 6147),
                                            (8, 4096, 6147)])
def test_streaming_form(elem, rows, cols):
    assert 2 * elem * rows * cols >= 3 << 27 and rows * elem % 128 == 0
    case(f"transpose {elem}-byte {rows}x{cols}")
    dtype = {1: torch.uint8, 2: torch.int16, 4: torch.int32, 8: torch.int64}[elem]
    x = torch.randint(0, 256, (rows * cols * elem,), dtype=torch.uint8,
                      device="cuda").view(dtype).view(rows, cols)
    buf = torch.zeros(rows * cols + 128, dtype=dtype, device="cuda")
    y = buf[:rows * cols].view(cols, rows)
    assert y.data_ptr() % 128 == 0
    desc.desc_transpose_batched(x, y)
    assert torch.equal(y, x.t())
    assert int(buf[rows * cols:].abs().sum()) == 0
    # one element further the output is not in whole lines: the other form
    y = buf[1:rows * cols + 1].view(cols, rows)
    buf.zero_()
    desc.desc_transpose_batched(x, y)
    assert torch.equal(y, x.t())
    assert int(buf[0]) == 0 and int(buf[rows * cols + 1:].abs().sum()) == 0
