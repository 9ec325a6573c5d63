"""The work that a program has this library do, as a list of timed cases.

Every case is one pass through the public entry points of the binding, on
operands that are on the GPU before the call and with the workspace that such
a program keeps between calls.  `listed()` names the cases, `draw(rng)` gives
further ones of the same ranges, `prepare`/`run` make the inputs and the call,
`work` says what a pass cannot do without, and `exact` computes the result in
64 bits with plain torch.

Families (the "op" of a case):
  reduce     a full reduction: exact int32 sum, min/max or fixed-order float sum
  scan       a prefix sum: int32 inclusive or exclusive, or fixed-order float
  transpose  out-of-place transposes of 1-, 2-, 4- or 8-byte elements
  gemm       one matrix product in FP32, three-product BF16 or row/column FP8
  segmented  the sums and the prefix sums of many segments of one array
  grouped    many matrix products of different shapes in one call
"""
from __future__ import annotations

import math

import torch

import paper_2305_03448_amd as desc

LARGEST_N = 1 << 28                  # elements of a reduction or a scan
LARGEST_TRANSPOSE = 1 << 29          # bytes read and written by a transpose
LARGEST_MNK = 4096 ** 3              # multiply-adds of a matrix product
LARGEST_SEGMENTED = 310_000_000      # elements of all segments together
LARGEST_GROUPED_MNK = 78_000_000_000  # multiply-adds of a group of products


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # A total over a small array, as a program asks for between larger
        # steps: the launch and the host path are all of its time.
        {"name": "reduce_1000", "op": "reduce", "kind": "sum_i32", "n": 1000, "offset": 0},
        # The 2^22-element sum of the benchmark: still a latency-bound call.
        {"name": "reduce_2_22", "op": "reduce", "kind": "sum_i32", "n": 1 << 22, "offset": 0},
        # An ordinary prefix sum of odd length (offsets of a compaction).
        {"name": "scan_1000003", "op": "scan", "kind": "inclusive", "n": 1_000_003, "offset": 0},
        # The benchmark's scan: streaming, the largest array.
        {"name": "scan_2_28", "op": "scan", "kind": "inclusive", "n": 1 << 28, "offset": 0},
        # The benchmark's transpose.
        {"name": "transpose_8192", "op": "transpose", "elem": 4, "batch": 1, "rows": 8192,
         "cols": 8192},
        # A batch of odd-sized 16-bit matrices (a layout change of activations).
        {"name": "transpose_u16_batch", "op": "transpose", "elem": 2, "batch": 12, "rows": 1000,
         "cols": 777},
        # An ordinary FP32 product whose sizes fit no tile.
        {"name": "gemm_f32_ragged", "op": "gemm", "mode": "f32", "M": 1000, "N": 1500, "K": 777,
         "pad": 0},
        # Few rows against a square matrix (one decoding step of a small batch).
        {"name": "gemm_f32_few_rows", "op": "gemm", "mode": "f32", "M": 32, "N": 4096, "K": 4096,
         "pad": 0},
        # The benchmark's products in the two precision modes.
        {"name": "gemm_bf16x3_4096", "op": "gemm", "mode": "bf16x3", "M": 4096, "N": 4096,
         "K": 4096, "pad": 0},
        {"name": "gemm_fp8_4096", "op": "gemm", "mode": "fp8", "M": 4096, "N": 4096, "K": 4096,
         "pad": 0},
        # The benchmark's segmented workload: sums, then prefix sums, of 4096
        # segments of log-uniform lengths up to 2^20.
        {"name": "segmented_4096", "op": "segmented", "segments": 4096, "max_len": 1 << 20},
        # The benchmark's group: 512 products, each size a multiple of 64 up to 1024.
        {"name": "grouped_f32_512", "op": "grouped", "mode": "f32", "G": 512, "step": 64,
         "largest": 1024},
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    """An integer spread over the logarithm of [lo, hi], odd ones as often as even."""
    v = int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))
    return max(lo, min(hi, v))


def draw(rng):
    op = rng.choice(["reduce", "scan", "transpose", "gemm", "gemm", "segmented", "grouped"])
    if op in ("reduce", "scan"):
        kinds = (["sum_i32", "minmax_i32", "sum_f32"] if op == "reduce"
                 else ["inclusive", "exclusive", "float"])
        return {"op": op, "kind": rng.choice(kinds), "n": _log_int(rng, 256, LARGEST_N - 3),
                "offset": rng.choice([0, 0, 1, 3])}
    if op == "transpose":
        while True:
            c = {"op": op, "elem": rng.choice([1, 2, 4, 8]), "batch": _log_int(rng, 1, 64),
                 "rows": _log_int(rng, 16, 16384), "cols": _log_int(rng, 16, 16384)}
            if 2 * c["elem"] * c["batch"] * c["rows"] * c["cols"] <= LARGEST_TRANSPOSE:
                return c
    if op == "gemm":
        mode = rng.choice(["f32", "bf16x3", "fp8"])
        while True:
            m, n, k = (_log_int(rng, 16, 8192) for _ in range(3))
            if rng.random() < 0.5:              # sizes in whole tiles as often as odd ones
                m, n, k = (64 * max(1, round(v / 64)) for v in (m, n, k))
            if m * n * k <= LARGEST_MNK:
                return {"op": op, "mode": mode, "M": m, "N": n, "K": k,
                        "pad": rng.choice([0, 0, 1, 64])}
    if op == "segmented":
        while True:
            c = {"op": op, "segments": _log_int(rng, 1, 16384),
                 "max_len": _log_int(rng, 16, 1 << 20)}
            if int(_segment_offsets(c)[-1]) <= LARGEST_SEGMENTED:
                return c
    while True:
        c = {"op": "grouped", "mode": rng.choice(["f32", "bf16x3"]), "G": _log_int(rng, 1, 512),
             "step": rng.choice([1, 8, 64]), "largest": _log_int(rng, 128, 2048)}
        if sum(m * n * k for m, n, k in _group_shapes(c)) <= LARGEST_GROUPED_MNK:
            return c


# ------------------------------------------------------------------ inputs
def _generator(seed: int):
    return torch.Generator(device="cuda").manual_seed(seed)


def _ints(n: int, gen, offset: int = 0, lo: int = -1024, hi: int = 1024):
    """n int32 values uniform over [lo, hi], at an address `offset` elements off."""
    return torch.randint(lo, hi + 1, (n + offset,), dtype=torch.int32, device="cuda",
                         generator=gen)[offset:]


def _floats(shape, gen):
    return torch.randn(shape, dtype=torch.float32, device="cuda", generator=gen)


def _zeros(nbytes: int):
    return torch.zeros(max(nbytes, 256), dtype=torch.uint8, device="cuda")


def _segment_offsets(case):
    """Log-uniform lengths over [1, max_len] and their running total (they
    belong to the case, not to the seed: its work depends on them)."""
    g = torch.Generator().manual_seed(10)
    u = torch.rand(case["segments"], dtype=torch.float64, generator=g)
    lengths = torch.floor(2.0 ** (u * math.log2(case["max_len"] + 1))).to(torch.int64)
    lengths = lengths.clamp(1, case["max_len"])
    return torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(lengths, 0)])


def _group_shapes(case):
    """The shapes belong to the case, not to the seed: its work depends on them."""
    g = torch.Generator().manual_seed(12)
    step = case["step"]
    top = max(1, case["largest"] // step)
    return (step * torch.randint(1, top + 1, (case["G"], 3), generator=g)).tolist()


def _matrices(case, seed):
    """A and B, rows `pad` elements further apart than they are long."""
    g = _generator(seed)
    M, N, K, pad = case["M"], case["N"], case["K"], case["pad"]
    return _floats((M, K + pad), g)[:, :K], _floats((K, N + pad), g)[:, :N]


_DTYPE = {1: torch.uint8, 2: torch.int16, 4: torch.float32, 8: torch.float64}


def _inputs(case, seed):
    op = case["op"]
    g = _generator(seed)
    if op in ("reduce", "scan"):
        if case["kind"] in ("sum_f32", "float"):
            return _floats((case["n"] + case["offset"],), g)[case["offset"]:]
        if case["kind"] == "minmax_i32":
            return _ints(case["n"], g, case["offset"], -(1 << 31), (1 << 31) - 1)
        return _ints(case["n"], g, case["offset"])
    if op == "transpose":
        shape = (case["batch"], case["rows"], case["cols"])
        nbytes = case["elem"] * math.prod(shape)
        if case["elem"] >= 4:
            return torch.randn(shape, dtype=_DTYPE[case["elem"]], device="cuda", generator=g)
        raw = torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device="cuda", generator=g)
        return raw.view(_DTYPE[case["elem"]]).view(shape)
    if op == "gemm":
        return _matrices(case, seed)
    if op == "segmented":
        off = _segment_offsets(case)
        return _ints(int(off[-1]), g), off.cuda()
    return [(_floats((m, k), g), _floats((k, n), g)) for m, n, k in _group_shapes(case)]


def prepare(case, seed):
    op = case["op"]
    x = _inputs(case, seed)
    st = {"op": op, "case": case, "x": x}
    if op == "reduce":
        n, kind = case["n"], case["kind"]
        dtype, count = {"sum_i32": (torch.int64, 1), "minmax_i32": (torch.int32, 2),
                        "sum_f32": (torch.float64, 1)}[kind]
        st["out"] = torch.empty(count, dtype=dtype, device="cuda")
        st["ws"] = _zeros(desc.desc_reduce_i32_workspace(n) if kind == "sum_i32"
                          else desc.desc_reduce_op_workspace(n))
    elif op == "scan":
        st["out"] = torch.empty_like(x)
        st["ws"] = _zeros(desc.desc_scan_f32_workspace(case["n"]) if case["kind"] == "float"
                          else desc.desc_scan_i32_workspace(case["n"]))
    elif op == "transpose":
        st["out"] = torch.empty((case["batch"], case["cols"], case["rows"]), dtype=x.dtype,
                                device="cuda")
    elif op == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        st["out"] = torch.empty((M, N), dtype=torch.float32, device="cuda")
        need = desc.desc_gemm_workspace(case["mode"], M, N, K)
        st["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    elif op == "segmented":
        values, off = x
        n, S = values.numel(), case["segments"]
        st["sums"] = torch.empty(S, dtype=torch.int64, device="cuda")
        st["out"] = torch.empty_like(values)
        st["ws_sums"] = _zeros(desc.desc_reduce_segmented_i32_workspace(n, S))
        st["ws"] = _zeros(desc.desc_scan_segmented_i32_workspace(n, S))
    else:
        # the products lie one after another in one array
        sizes = [(a.shape[0], b.shape[1]) for a, b in x]
        st["out"] = torch.empty(sum(m * n for m, n in sizes), dtype=torch.float32, device="cuda")
        parts = st["out"].split([m * n for m, n in sizes])
        st["problems"] = desc.grouped_descriptors(
            [(a, b, c.view(mn)) for (a, b), c, mn in zip(x, parts, sizes)], torch.device("cuda"))
        need = (desc.desc_gemm_grouped_workspace(case["G"]) if case["mode"] == "f32" else
                desc.desc_gemm_grouped_workspace_for(case["mode"], st["problems"].cpu()))
        st["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    return st


# ------------------------------------------------------------------ one pass
_REDUCE = {"sum_i32": desc.desc_reduce_i32, "minmax_i32": desc.desc_reduce_minmax_i32,
           "sum_f32": desc.desc_reduce_sum_f32}
_SCAN = {"inclusive": desc.desc_scan_i32, "exclusive": desc.desc_scan_exclusive_i32,
         "float": desc.desc_scan_f32}


def run(state):
    op, case, x = state["op"], state["case"], state["x"]
    if op == "reduce":
        return _REDUCE[case["kind"]](x, state["out"], ws=state["ws"])
    if op == "scan":
        return _SCAN[case["kind"]](x, state["out"], ws=state["ws"])
    if op == "transpose":
        return desc.desc_transpose_batched(x, state["out"])
    if op == "gemm":
        return desc.desc_gemm(x[0], x[1], state["out"], mode=case["mode"], ws=state["ws"])
    if op == "segmented":
        sums = desc.desc_reduce_segmented_i32(x[0], x[1], state["sums"], ws=state["ws_sums"])
        return sums, desc.desc_scan_segmented_i32(x[0], x[1], state["out"], ws=state["ws"])
    desc.desc_gemm_grouped(state["problems"], mode=case["mode"], ws=state["ws"])
    return state["out"]


# ------------------------------------------------------------------ what a pass needs
def _product(mode, m, n, k):
    # the three-product mode is defined as three products per multiply-add
    return {"bytes": 4 * (m * k + k * n + m * n),
            "flops": (6 if mode == "bf16x3" else 2) * m * n * k}


def work(case):
    op = case["op"]
    if op == "reduce":
        return {"bytes": 4 * case["n"] + 8, "flops": 0}
    if op == "scan":
        return {"bytes": 8 * case["n"], "flops": 0}
    if op == "transpose":
        return {"bytes": 2 * case["elem"] * case["batch"] * case["rows"] * case["cols"],
                "flops": 0}
    if op == "gemm":
        return _product(case["mode"], case["M"], case["N"], case["K"])
    if op == "segmented":
        # sums: values, offsets and results; prefix sums: values, offsets, results
        n, S = int(_segment_offsets(case)[-1]), case["segments"]
        return {"bytes": (4 * n + 8 * (S + 1) + 8 * S) + (8 * n + 8 * (S + 1)), "flops": 0}
    parts = [_product(case["mode"], m, n, k) for m, n, k in _group_shapes(case)]
    return {"bytes": sum(p["bytes"] for p in parts), "flops": sum(p["flops"] for p in parts)}


# ------------------------------------------------------------------ the result in 64 bits
def _wrap32(x):
    """int64 values as the int32 that equals them modulo 2^32."""
    return ((x + (1 << 31)) % (1 << 32) - (1 << 31)).to(torch.int32)


def _e4m3(x, dim):
    """x as its e4m3 codes under one scale per row (dim 1) or column (dim 0),
    and that scale, with the float32 steps that define the codes."""
    top = x.abs().amax(dim, keepdim=True)
    inv = torch.where(top > 0, 448.0 / top, torch.ones_like(top))
    codes = (x * inv).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return codes.to(torch.float64), top.to(torch.float64) / 448.0


def _split(x):
    hi = x.to(torch.bfloat16).to(torch.float32)
    lo = (x - hi).to(torch.bfloat16)
    return hi.to(torch.float64), lo.to(torch.float64)


def _exact_product(mode, a, b):
    if mode == "fp8":
        (qa, sa), (qb, sb) = _e4m3(a, 1), _e4m3(b, 0)
        return (qa @ qb) * sa * sb
    if mode == "bf16x3":
        (ah, al), (bh, bl) = _split(a), _split(b)
        return ah @ bh + ah @ bl + al @ bh
    return a.to(torch.float64) @ b.to(torch.float64)


def exact(case, seed):
    op = case["op"]
    x = _inputs(case, seed)
    if op == "reduce":
        if case["kind"] == "sum_i32":
            return x.to(torch.int64).sum().reshape(1)
        if case["kind"] == "minmax_i32":
            return torch.stack([x.min(), x.max()])
        return x.to(torch.float64).sum().reshape(1)
    if op == "scan":
        if case["kind"] == "float":
            return torch.cumsum(x.to(torch.float64), 0)
        total = torch.cumsum(x, 0, dtype=torch.int64)
        return _wrap32(total if case["kind"] == "inclusive" else total - x)
    if op == "transpose":
        return x.transpose(1, 2).contiguous()
    if op == "gemm":
        return _exact_product(case["mode"], *x)
    if op == "segmented":
        values, off = x
        total = torch.cumsum(values, 0, dtype=torch.int64)
        before = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), total])
        starts = before[off[:-1]]
        owner = torch.repeat_interleave(starts, off[1:] - off[:-1])
        return before[off[1:]] - starts, _wrap32(total - owner)
    return torch.cat([_exact_product(case["mode"], a, b).reshape(-1) for a, b in x])
