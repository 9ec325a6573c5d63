"""The segmented forms that give a block one unit per wave: which units the
blocks take, on the host, and offsets that run backwards, on the GPU.

Such offsets give unspecified results, but the workspace is sized for the
units of non-decreasing ones: a unit past them has no status word, and what
it wrote would land in the unit prefix that other blocks read."""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_2305_03448_amd as desc
import workloads
from gpu_util import case, dev, needs_gpu, to_dev

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2305_03448_amd", "csrc")

CHECK = r'''
#include <cstdio>
#include <vector>
#include "layouts.hpp"
using namespace desc;
// Blocks of kW units cover the units of a call once, whatever the launched
// bound, and none past it even when more are planned.
template <int kW>
static bool covers() {
  for (idx_t bound = 0; bound <= 6 * kW; ++bound)
    for (idx_t total = 0; total <= 12 * kW; ++total) {
      std::vector<int> taken(bound, 0);
      for (idx_t b = 0; b < (bound + kW - 1) / kW; ++b) {
        const layout::BlockRange r = layout::block_units<kW>(b, total, bound);
        for (int w = 0; w < r.count; ++w) {
          if (r.first + w >= bound) return false;
          ++taken[r.first + w];
        }
      }
      for (idx_t u = 0; u < bound; ++u)
        if (taken[u] != (u < total ? 1 : 0)) return false;
    }
  return true;
}
int main() {
  const bool ok = covers<4>() && covers<8>() && covers<16>();
  std::puts(ok ? "OK" : "FAIL");
  return !ok;
}
'''


def test_blocks_take_no_unit_past_the_bound(tmp_path):
    src, exe = str(tmp_path / "c.cpp"), str(tmp_path / "c")
    with open(src, "w") as f:
        f.write(CHECK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, src, "-o", exe], check=True)
    assert subprocess.run([exe], capture_output=True, text=True, timeout=60).stdout == "OK\n"


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("S", [2049, 4098, 8195])
def test_offsets_that_run_backwards(S):
    """Every second segment is the whole array: S / 2 times the planned units.
    The call ends, writes nothing beside its output, and the workspace serves
    the next one."""
    n = 300 * S
    case(f"backward offsets S={S} n={n}")
    x = workloads.int_uniform(n, seed=61)
    xt = to_dev(x)
    bad = torch.zeros(S + 1, dtype=torch.int64)
    bad[1::2] = n
    lengths = np.full(S, 300, np.int64)
    off = workloads.offsets_from_lengths(lengths)
    ws = torch.zeros(desc.desc_scan_segmented_i32_workspace(n, S), dtype=torch.uint8, device=dev())
    buf = torch.full((n + 16,), -7, dtype=torch.int32, device=dev())
    sums = torch.full((S + 16,), -7, dtype=torch.int64, device=dev())
    wr = torch.zeros(desc.desc_reduce_segmented_i32_workspace(n, S), dtype=torch.uint8, device=dev())
    for o in (bad, torch.from_numpy(off)):
        ot = o.to(dev())
        desc.desc_scan_segmented_i32(xt, ot, buf[8:8 + n], ws=ws)
        desc.desc_reduce_segmented_i32(xt, ot, sums[8:8 + S], ws=wr)
        torch.cuda.synchronize()
    for b in (buf, sums):
        assert (b[:8] == -7).all() and (b[-8:] == -7).all()
    assert np.array_equal(buf[8:8 + n].cpu().numpy(), oracle.scan_segmented_i32(x, off))
    assert np.array_equal(sums[8:8 + S].cpu().numpy(), oracle.reduce_segmented_i32(x, off))


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("S", [2048, 4099])
@pytest.mark.parametrize("runs", [1, 3, 50])
def test_long_segments_among_short_ones(S, runs):
    """A few long segments between segments of 0 to 6 elements: several units of
    one segment in a block, segments that straddle blocks, and the wait limit
    not reached."""
    g = workloads.rng(67)
    lengths = g.integers(0, 7, S)
    at = (np.arange(runs) * (S // runs) + 1) % S
    lengths[at] = 2_000_000 // runs + np.arange(runs)
    off = workloads.offsets_from_lengths(np.asarray(lengths, np.int64))
    n = int(off[-1])
    x = workloads.int_uniform(n, seed=71)
    case(f"{runs} long segments among S={S} n={n}")
    xt, ot = to_dev(x, 1), to_dev(off)
    ws = torch.zeros(desc.desc_scan_segmented_i32_workspace(n, S), dtype=torch.uint8, device=dev())
    want = oracle.scan_segmented_i32(x, off)
    for rep in range(3):
        y = torch.full((n,), -5, dtype=torch.int32, device=dev())
        desc.desc_scan_segmented_i32(xt, ot, y, ws=ws)
        assert np.array_equal(y.cpu().numpy(), want)
    assert desc.workspace_status(ws) == 0


@pytest.mark.gpu
@needs_gpu
def test_one_long_segment_does_not_chain_the_blocks():
    """The units of a long segment are published side by side whatever form the
    number of segments selects: at 2047 a block per unit, from 2048 several units
    a block.  In turn they take over 30 times as long, side by side about the
    same; 5 is asked."""
    n, times = 1 << 22, []
    for S in (2047, 4096):
        off = torch.zeros(S + 1, dtype=torch.int64)
        off[1:] = n - 3 * torch.arange(S - 1, -1, -1)
        x = torch.ones(n, dtype=torch.int32, device=dev())
        y, ot = torch.empty_like(x), off.to(dev())
        ws = torch.zeros(desc.desc_scan_segmented_i32_workspace(n, S), dtype=torch.uint8, device=dev())
        case(f"one long segment among S={S}")
        took = []
        for _ in range(9):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            desc.desc_scan_segmented_i32(x, ot, y, ws=ws)
            b.record()
            b.synchronize()
            took.append(a.elapsed_time(b))
        times.append(sorted(took)[len(took) // 2])
        assert int(y[n - 3 * (S - 1) - 1]) == n - 3 * (S - 1)
    assert times[1] < 5 * times[0], times


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("n", [384 * 8192, 384 * 8192 + 1])
def test_few_long_segments(n):
    """Both sides of the total at which a few long segments change their unit."""
    S = 3
    lengths = np.array([n // 3 - 7, n // 3 + 9, n - 2 * (n // 3) - 2], np.int64)
    off = workloads.offsets_from_lengths(lengths)
    x = workloads.int_uniform(n, seed=73)
    case(f"few long segments n={n}")
    xt, ot = to_dev(x, 1), to_dev(off)
    y = torch.full((n,), -5, dtype=torch.int32, device=dev())
    r = torch.full((S,), 5, dtype=torch.int64, device=dev())
    desc.desc_scan_segmented_i32(xt, ot, y)
    desc.desc_reduce_segmented_i32(xt, ot, r)
    assert np.array_equal(y.cpu().numpy(), oracle.scan_segmented_i32(x, off))
    assert np.array_equal(r.cpu().numpy(), oracle.reduce_segmented_i32(x, off))


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("S", [63, 64, 65, 129])
def test_both_searches_of_a_units_segment(S):
    """Both sides of the segment count at which the search changes, with empty
    segments at the ends and between, and segments of several units."""
    g = workloads.rng(79)
    lengths = g.integers(0, 40_000, S)
    lengths[[0, 1, S // 2, S // 2 + 1, S - 1]] = 0
    off = workloads.offsets_from_lengths(np.asarray(lengths, np.int64))
    x = workloads.int_uniform(int(off[-1]), seed=83)
    case(f"segment searches S={S}")
    xt, ot = to_dev(x), to_dev(off)
    y = torch.full((x.size,), -5, dtype=torch.int32, device=dev())
    desc.desc_scan_segmented_i32(xt, ot, y)
    assert np.array_equal(y.cpu().numpy(), oracle.scan_segmented_i32(x, off))
    rows = workloads.int_uniform(S * 9001, seed=89).reshape(S, 9001)
    r = torch.full((S,), 5, dtype=torch.int64, device=dev())
    desc.desc_reduce_batched_i32(to_dev(rows), r)
    assert np.array_equal(r.cpu().numpy(), rows.astype(np.int64).sum(1))


@pytest.mark.gpu
@needs_gpu
@pytest.mark.parametrize("S,mean", [(2048, 1024), (2048, 1025), (5999, 1025), (6000, 1025),
                                    (6000, 1536), (6000, 1537)])
def test_mean_lengths_where_the_scan_changes_form(S, mean):
    g = workloads.rng(97)
    lengths = np.minimum(g.integers(0, 2 * mean, S), g.integers(0, 9000, S))
    lengths[3] += mean * S - int(lengths.sum())          # one takes up the rest
    off = workloads.offsets_from_lengths(np.asarray(lengths, np.int64))
    x = workloads.int_uniform(int(off[-1]), seed=101)
    case(f"scan of S={S} segments of {mean} on average")
    y = torch.full((x.size,), -5, dtype=torch.int32, device=dev())
    desc.desc_scan_segmented_i32(to_dev(x, 1), to_dev(off), y)
    assert np.array_equal(y.cpu().numpy(), oracle.scan_segmented_i32(x, off))
