"""Cases of GEMM + All-Scatter and of the heap tile copy, through the package's
public entry points (``Heap``, ``GatheredOutput.run``, ``symtile_tile_copy``).

A GEMM case is one rank's call of a column-parallel layer: A [M, K] times the
rank's shard [K, N], the product stored into the rank's column block of the
gathered [M, world*N] output in every slot, with the arrival counters.  The
large, the wide, the small and the tiny shape are this repository's own
workloads; the others are generic: few rows (a decode step), odd row counts,
shapes that are no multiple of a tile.  Every schedule is there, since which
one a program takes depends on what it overlaps the call with.  A copy case
moves every rank's block to its ring neighbour, tile by tile.
"""
from __future__ import annotations

import math

import torch

import paper_2511_12500_amd as sym

VARIANTS = {"fused": sym.FUSED_SEQ, "bulk": sym.BULK_SYNC, "wg_spec": sym.WG_SPEC,
            "unfused_pc": sym.UNFUSED_PC, "wave_spec": sym.WAVE_SPEC}
DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
COPY_DTYPES = {"f16": sym.F16, "bf16": sym.BF16, "f32": sym.F32}


def gemm(M, K, N, world, rank, dtype, dist, variant, tile_m, tile_n, split=0, policy=2,
         gemm_wgs=0, copy_wgs=0, name=None):
    """``policy``: output stores (0 default, 1 non-temporal, 2 write-through)."""
    c = {"kind": "gemm", "M": M, "K": K, "N": N, "world": world, "rank": rank, "dtype": dtype,
         "dist": dist, "variant": variant, "tile_m": tile_m, "tile_n": tile_n, "split": split,
         "policy": policy, "gemm_wgs": gemm_wgs, "copy_wgs": copy_wgs}
    return c if name is None else dict(c, name=name)


def copy(rows, cols, world, dtype, tile_r, tile_c, mode, shift=1, name=None):
    c = {"kind": "copy", "rows": rows, "cols": cols, "world": world, "dtype": dtype,
         "tile_r": tile_r, "tile_c": tile_c, "mode": mode, "shift": shift}
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # two ranks exchange a tiny tile grid: nothing but latency
        gemm(128, 256, 64, 2, 0, "f16", "uniform", "fused", 64, 64, policy=0,
             name="tiny_f16_fused"),
        # a decode step of the large layer: few rows, the weights are the traffic
        gemm(64, 8192, 3584, 8, 3, "bf16", "normal_sqrtk", "fused", 64, 64, split=4,
             name="decode_bf16_fused_split4"),
        # a small layer: 64 tiles, so K is split to fill the chip
        gemm(1024, 4096, 1024, 8, 0, "bf16", "normal_sqrtk", "fused", 128, 128, split=4,
             name="small_bf16_fused_split4"),
        # a prefill whose row count, K and N are no multiple of a tile; library defaults
        gemm(1000, 2056, 1480, 4, 1, "bf16", "normal_sqrtk", "bulk", 128, 128, policy=0,
             name="ragged_bf16_bulk"),
        # a middle-sized layer, GEMM and copy as two kernels on two streams
        gemm(2048, 4096, 2048, 4, 2, "f16", "uniform_sqrtk", "unfused_pc", 256, 128,
             name="middle_f16_unfused_pc"),
        # the wide layer: 128 tiles, two K slices each
        gemm(8192, 8192, 1024, 8, 0, "f16", "uniform_sqrtk", "fused", 256, 256, split=2,
             name="wide_f16_fused_split2"),
        # the same with its CUs shared between producers and consumers
        gemm(8192, 8192, 1024, 8, 5, "f16", "uniform_sqrtk", "wg_spec", 256, 128,
             gemm_wgs=128, copy_wgs=128, name="wide_f16_wg_spec"),
        # the large layer (the benchmark's call), fused
        gemm(4096, 8192, 3584, 8, 0, "bf16", "normal_sqrtk", "fused", 256, 256,
             name="large_bf16_fused"),
        # GEMM kernel, then scatter kernel
        gemm(4096, 8192, 3584, 8, 0, "bf16", "normal_sqrtk", "bulk", 256, 256,
             name="large_bf16_bulk"),
        # a copy wave in every workgroup
        gemm(4096, 8192, 3584, 8, 7, "bf16", "normal_sqrtk", "wave_spec", 256, 128,
             name="large_bf16_wave_spec"),
        # the heap copy benchmark: a 256 MiB heap, every block to the next rank
        copy(2048, 2048, 8, "f32", 128, 128, "put", name="copy_f32_put_t128"),
        # a 16-bit activation fetched from the previous rank, tiles at ragged edges
        copy(1500, 1160, 4, "bf16", 64, 64, "get", name="copy_bf16_get_t64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tile_and_split(rng, M, K, N, variant):
    """The largest tile that gives about one work unit per CU, in K slices where
    the schedule has them; programs do not always pick that one, so some draws
    take a neighbour."""
    if variant == "wave_spec":
        return 256, 128, 0
    shapes = [(256, 256), (256, 128), (128, 128), (64, 64)]
    grid = [-(-M // a) * -(-N // b) for a, b in shapes]
    splits = variant in ("fused", "bulk")
    pick = len(shapes) - 1
    for i, g in enumerate(grid):
        if g >= 190 or (splits and g >= 48 and K >= 2048):
            pick = i
            break
    if rng.random() < 0.25:
        pick = max(0, min(len(shapes) - 1, pick + rng.choice((-1, 1))))
    split = 0
    if splits and grid[pick] < 190:
        s = min(224 // grid[pick], K // 512, 8)
        split = s if s > 1 else 0
    return shapes[pick][0], shapes[pick][1], split


def draw(rng):
    if rng.random() < 0.2:
        dtype = rng.choice(("f32", "f32", "bf16", "f16"))
        quantum = 4 if dtype == "f32" else 8
        rows = _log_int(rng, 128, 2048)
        cols = _log_int(rng, 128, 2048) // quantum * quantum
        tile = rng.choice((64, 128, 256))
        return copy(rows, cols, rng.choice((2, 4, 8)), dtype, tile, tile,
                    rng.choice(("put", "put", "get")), rng.choice((1, 1, 1, -1)))
    variant = rng.choice(("fused", "fused", "fused", "bulk", "wg_spec", "unfused_pc", "wave_spec"))
    M = _log_int(rng, 64, 8192)
    K = _log_int(rng, 256, 8192) // 8 * 8
    N = _log_int(rng, 64, 4096) // 8 * 8
    if rng.random() < 0.5:      # layer widths are mostly multiples of 128
        K, N = K // 128 * 128, max(64, N // 128 * 128)
    while M * K * N > 4096 * 8192 * 3584:
        M //= 2
    if variant not in ("fused", "bulk") and M * N < 64 * 256 * 128:
        variant = "fused"       # nothing to overlap: no CUs or waves are set aside to copy
    world = rng.choice((2, 4, 8, 8))
    tile_m, tile_n, split = _tile_and_split(rng, M, K, N, variant)
    dtype, dist = rng.choice((("bf16", "normal_sqrtk"), ("bf16", "normal_sqrtk"),
                              ("f16", "uniform_sqrtk")))
    return gemm(M, K, N, world, rng.randrange(world), dtype, dist, variant, tile_m, tile_n, split,
                rng.choice((2, 2, 2, 0, 1)))


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _values(shape, dist, K, gen):
    if dist == "normal_sqrtk":
        return torch.randn(shape, generator=gen, device="cuda") / math.sqrt(K)
    x = torch.rand(shape, generator=gen, device="cuda") * 2.0 - 1.0
    return x if dist == "uniform" else x / math.sqrt(K)


def _gemm_inputs(case, seed):
    gen = _generator(seed)
    dt = DTYPES[case["dtype"]]
    A = _values((case["M"], case["K"]), case["dist"], case["K"], gen).to(dt)
    return A, _values((case["K"], case["N"]), case["dist"], case["K"], gen).to(dt)


def _copy_input(case, seed):
    return torch.rand((case["world"], case["rows"], case["cols"]), generator=_generator(seed),
                      device="cuda").to(DTYPES[case["dtype"]])


def _tiles(n, t):
    return -(-n // t)


def prepare(case, seed):
    w = case["world"]
    if case["kind"] == "copy":
        dt = DTYPES[case["dtype"]]
        shape = (case["rows"], case["cols"])
        nbytes = shape[0] * shape[1] * dt.itemsize
        tiles = (_tiles(shape[0], case["tile_r"]), _tiles(shape[1], case["tile_c"]))
        heap = sym.Heap(w, 2 * nbytes + tiles[0] * tiles[1] * 4 + 4096)
        src, dst = heap.alloc(nbytes), heap.alloc(nbytes)
        flags = heap.alloc(tiles[0] * tiles[1] * 4)
        heap.slots_view(src, shape, dt).copy_(_copy_input(case, seed))
        return {"case": case, "heap": heap, "src": src, "dst": dst, "flags": flags,
                "received": heap.slots_view(dst, shape, dt),
                "counters": heap.slots_view(flags, tiles, torch.int32)}
    M, N = case["M"], case["N"]
    tiles = _tiles(M, case["tile_m"]) * _tiles(N, case["tile_n"])
    heap = sym.Heap(w, M * w * N * 2 + w * tiles * 4 + 4096)
    out = sym.GatheredOutput(heap, M, N, DTYPES[case["dtype"]], case["tile_m"], case["tile_n"])
    A, B = _gemm_inputs(case, seed)
    r = case["rank"]
    return {"case": case, "heap": heap, "out": out, "A": A, "B": B,
            "block": out.C_all()[:, :, r * N:(r + 1) * N], "arrived": out.arrived_all()[:, r]}


def run(state):
    c = state["case"]
    if c["kind"] == "copy":
        sym.symtile_tile_copy(
            state["heap"].handle, state["src"], state["dst"], c["rows"], c["cols"], c["cols"],
            COPY_DTYPES[c["dtype"]], c["tile_r"], c["tile_c"], c["shift"], -1, state["flags"],
            stream=sym.current_stream(), mode=sym.GET if c["mode"] == "get" else sym.PUT)
        return {"received": state["received"], "counters": state["counters"]}
    state["out"].run(state["A"], state["B"], c["rank"], VARIANTS[c["variant"]],
                     gemm_wgs=c["gemm_wgs"], copy_wgs=c["copy_wgs"], nontemporal=c["policy"],
                     split_k=c["split"])
    return {"block": state["block"], "arrived": state["arrived"]}


def exact(case, seed):
    if case["kind"] == "copy":
        return {"received": _copy_input(case, seed).double().roll(case["shift"], 0),
                "counters": None}
    A, B = _gemm_inputs(case, seed)
    return {"block": (A.double() @ B.double()).expand(case["world"], -1, -1), "arrived": None}


def work(case):
    w = case["world"]
    if case["kind"] == "copy":
        tiles = _tiles(case["rows"], case["tile_r"]) * _tiles(case["cols"], case["tile_c"])
        block = case["rows"] * case["cols"] * DTYPES[case["dtype"]].itemsize
        return {"bytes": w * (2 * block + 4 * tiles), "flops": 0}
    M, K, N = case["M"], case["K"], case["N"]
    tiles = _tiles(M, case["tile_m"]) * _tiles(N, case["tile_n"])
    return {"bytes": 2 * (M * K + K * N + w * M * N) + 4 * w * tiles, "flops": 2 * M * K * N}


def tolerance(case):
    """The output is an fp32 sum rounded once to 16 bits.  Against the sum in 64
    bits that rounding is 1.7e-3 of the result in bf16 and 2.1e-4 in fp16, and at
    most half an ulp (2^-8, 2^-11 of the value) anywhere; four times that."""
    if case["kind"] == "copy":
        return "exact"
    return {"rel": 6.6e-3, "max": 1.6e-2} if case["dtype"] == "bf16" else {"rel": 8.4e-4,
                                                                           "max": 2e-3}
