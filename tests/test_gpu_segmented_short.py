"""The segmented forms' unit edges with many segments (a block of units, one
per wave) and with few, bit for bit against the CPU oracle: segments of 0 to 5
elements, at 256 elements (one round of a wave's loads), at 1024 (the longest
segment one wave takes alone) and at every unit size, segments of several
units between short ones (their sums meet in atomics, their scans in
look-backs that cross blocks and stay inside one), with 2047 segments (the
other form), 2048 and 8193, and inputs that start one element past a 16-byte
boundary.  Integer results: no tolerance."""
import numpy as np
import pytest
import torch

import oracle
import paper_2305_03448_amd as desc
import workloads
from gpu_util import case, dev, needs_gpu, to_dev

pytestmark = [pytest.mark.gpu, needs_gpu]

EDGES = [0, 1, 2, 3, 4, 5, 255, 256, 257, 1020, 1023, 1024, 1025, 1027, 8191, 8192, 8193]


def _lengths(kind, S):
    g = workloads.rng(41)
    if kind == "short":                  # every unit a whole short segment
        out = g.integers(0, 1025, S)
    elif kind == "edges":                # short ones and units of every remainder, in turns
        out = np.resize(np.array(EDGES + [1] * 11 + [70]), S)
        out = np.where((np.arange(S) % 64) < len(EDGES), out, out % 7)
    else:                                # "long": several units between short ones
        out = g.integers(0, 6, S)
        out[[1, 2, 5, S // 2, S - 1]] = [3 * 8192 + 1, 16385, 40_000, 9 * 8192, 32769]
    return np.asarray(out, np.int64)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("S", [2047, 2048, 8193])
@pytest.mark.parametrize("kind", ["short", "edges", "long"])
def test_unit_edges_with_many_segments(kind, S, offset):
    off = workloads.offsets_from_lengths(_lengths(kind, S))
    n = int(off[-1])
    x = workloads.int_uniform(n, seed=43)
    xt, ot = to_dev(x, offset), to_dev(off)
    wr = torch.zeros(desc.desc_reduce_segmented_i32_workspace(n, S), dtype=torch.uint8, device=dev())
    wy = torch.zeros(desc.desc_scan_segmented_i32_workspace(n, S), dtype=torch.uint8, device=dev())
    want_r, want_y = oracle.reduce_segmented_i32(x, off), oracle.scan_segmented_i32(x, off)
    for rep in range(2):                 # the second call finds the first one's state
        case(f"many segments {kind} S={S} n={n} offset={offset} rep={rep}")
        r = torch.full((S,), 5, dtype=torch.int64, device=dev())
        y = torch.full((n,), -5, dtype=torch.int32, device=dev())
        desc.desc_reduce_segmented_i32(xt, ot, r, ws=wr)
        desc.desc_scan_segmented_i32(xt, ot, y, ws=wy)
        assert np.array_equal(r.cpu().numpy(), want_r)
        assert np.array_equal(y.cpu().numpy(), want_y)
    assert desc.workspace_status(wr) == 0 and desc.workspace_status(wy) == 0


@pytest.mark.parametrize("mean", [12_288, 12_289, 32_769, 49_153])
def test_unit_by_mean_length(mean):
    """Few segments on both sides of each mean length where the unit changes."""
    S = 9
    lengths = np.full(S, mean, np.int64)
    lengths[1] -= 5000
    lengths[7] += 5000
    off = workloads.offsets_from_lengths(lengths)
    x = workloads.int_uniform(int(off[-1]), seed=47)
    case(f"unit by mean length {mean}")
    xt, ot = to_dev(x, 1), to_dev(off)
    r = torch.full((S,), 5, dtype=torch.int64, device=dev())
    y = torch.full((x.size,), -5, dtype=torch.int32, device=dev())
    desc.desc_reduce_segmented_i32(xt, ot, r)
    desc.desc_scan_segmented_i32(xt, ot, y)
    assert np.array_equal(r.cpu().numpy(), oracle.reduce_segmented_i32(x, off))
    assert np.array_equal(y.cpu().numpy(), oracle.scan_segmented_i32(x, off))


def test_replays_with_many_segments():
    off = workloads.offsets_from_lengths(_lengths("long", 2048))
    n, S = int(off[-1]), 2048
    x = workloads.int_uniform(n, seed=53)
    xt, ot = to_dev(x), to_dev(off)
    wr = torch.zeros(desc.desc_reduce_segmented_i32_workspace(n, S), dtype=torch.uint8, device=dev())
    wy = torch.zeros(desc.desc_scan_segmented_i32_workspace(n, S), dtype=torch.uint8, device=dev())
    r = torch.empty(S, dtype=torch.int64, device=dev())
    y = torch.empty(n, dtype=torch.int32, device=dev())
    want_r, want_y = oracle.reduce_segmented_i32(x, off), oracle.scan_segmented_i32(x, off)
    case("many segments: capture")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        desc.desc_reduce_segmented_i32(xt, ot, r, ws=wr)
        desc.desc_scan_segmented_i32(xt, ot, y, ws=wy)
    for rep in range(3):
        case(f"many segments: replay {rep}")
        r.fill_(7)
        y.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(r.cpu().numpy(), want_r)
        assert np.array_equal(y.cpu().numpy(), want_y)
