"""Workloads that time libxred through its Python entry points.

A case is a dict of plain values: ``kind`` names the entry point, the other
fields give types, sizes and options (``*_bytes`` are bytes of one source).
``listed()`` are the standing cases, ``draw(rng)`` gives one more of the same
ranges, ``prepare`` builds what a program holds before the call, ``run`` makes
one pass, ``work`` counts the bytes and operations a pass cannot do without,
and ``exact`` computes the same outputs in 64 bits with plain torch.

Ranges: sources of 8 KiB (small inference messages) to 128 MiB (one gradient
bucket over 8 ranks), 2 to 64 sources, batches of 8 to 4096 messages of 8 KiB
to 1 MiB, rings and step sequences of 2 to 32 chunks, 2 to 16 simulated ranks;
lengths that are and are not whole vectors, buffers that are views at an
element offset, every op and the dtypes gradients and counters come in.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2510_20171_amd as xr

KIB, MIB = 1 << 10, 1 << 20

TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16,
         "e4m3": torch.float8_e4m3fn, "i32": torch.int32, "i64": torch.int64}
SIZE = {"f32": 4, "bf16": 2, "f16": 2, "e4m3": 1, "i32": 4, "i64": 8}
ACC = {"f32": torch.float32, "bf16": torch.float32, "f16": torch.float32, "e4m3": torch.float32,
       "i32": torch.int32, "i64": torch.int64}
ARENA = 256   # bytes: every message of a batch starts on such a boundary
MOST_BYTES = 1200 * MIB   # read and written by a drawn case


def listed():
    return [
        # the smallest message of an inference AllReduce over 8 ranks: all launch and call cost
        {"name": "allreduce_8k", "kind": "allreduce", "dtype": "bf16", "op": "sum", "nsrc": 8,
         "count": 4096, "views": "aligned"},
        # a mid-sized fp32 message over 4 ranks
        {"name": "allreduce_f32_4m", "kind": "allreduce", "dtype": "f32", "op": "sum", "nsrc": 4,
         "count": 1 << 20, "views": "aligned"},
        # a rank's part of a large AllReduce (256 MiB over 8 ranks), ragged
        {"name": "allreduce_32m", "kind": "allreduce", "dtype": "bf16", "op": "sum", "nsrc": 8,
         "count": (1 << 24) + 3, "views": "aligned"},
        # a whole gradient bucket over 8 ranks: the headline workload
        {"name": "allreduce_bucket", "kind": "allreduce", "dtype": "bf16", "op": "sum",
         "nsrc": 8, "count": 1 << 26, "views": "aligned"},
        # many ranks, fp32 extrema (gradient-norm clipping, overflow checks)
        {"name": "allreduce_max_p32", "kind": "allreduce", "dtype": "f32", "op": "max",
         "nsrc": 32, "count": 1 << 23, "views": "aligned"},
        # gradients that sit at another element offset in every rank's flat buffer, averaged
        {"name": "allreduce_views", "kind": "allreduce", "dtype": "f16", "op": "avg", "nsrc": 8,
         "count": 10_000_019, "views": "mixed"},
        # ReduceScatter whose shards have an odd length
        {"name": "scatter_odd", "kind": "scatter", "dtype": "bf16", "op": "sum", "nsrc": 8,
         "count": (1 << 23) + 1, "rank": 3},
        # a ring's 16 chunks in one launch
        {"name": "ring_16x2m", "kind": "ring", "dtype": "bf16", "op": "sum", "nsrc": 16,
         "count": 1 << 20, "flags": False},
        # the same ring a step at a time as chunks arrive, 8 MB chunks of odd length cut from
        # one buffer, the accumulator kept in fp32
        {"name": "steps_16x8m", "kind": "steps", "dtype": "bf16", "op": "sum", "nsrc": 16,
         "count": 4_000_037, "final": True},
        # a layer's small messages handed over as tensors, one launch
        {"name": "batched_host_256", "kind": "batched", "dtype": "bf16", "op": "sum", "nsrc": 8,
         "items": 256, "min_bytes": 8 * KIB, "max_bytes": MIB, "sizes": 4999, "how": "host"},
        # thousands of messages described in device memory
        {"name": "batched_device_4096", "kind": "batched", "dtype": "bf16", "op": "sum",
         "nsrc": 8, "items": 4096, "min_bytes": 8 * KIB, "max_bytes": MIB, "sizes": 4999,
         "how": "device"},
        # a whole simulated AllReduce over 8 ranks, every step in one launch
        {"name": "sim_ring_8x32m", "kind": "sim", "dtype": "bf16", "op": "sum", "nsrc": 8,
         "count": 1 << 24, "schedule": "ring1"},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _count(rng, lo_bytes, hi_bytes, es):
    """Elements, log-uniform in bytes; half of the draws are whole 128-byte lines."""
    n = max(1, int(_log_uniform(rng, lo_bytes, hi_bytes) / es))
    return max(64, n // 128 * 128) if rng.random() < 0.5 else n | 1


def draw(rng):
    kind = rng.choices(["allreduce", "scatter", "ring", "steps", "batched", "sim"],
                       [5, 2, 1, 2, 3, 2])[0]
    dtype = rng.choices(["bf16", "f32", "f16", "e4m3", "i32", "i64"], [4, 2, 1, 1, 1, 0.5])[0]
    whole_fold = kind in ("allreduce", "scatter", "batched")
    ops = ["sum", "max", "min"] + (["avg"] if whole_fold and dtype[0] != "i" else [])
    op = rng.choices(ops, [5, 1, 0.5, 1][:len(ops)])[0]
    es = SIZE[dtype]
    case = {"kind": kind, "dtype": dtype, "op": op}
    if kind in ("allreduce", "scatter"):
        p = rng.choice([2, 3, 4, 6, 8, 8, 8, 12, 16, 24, 32, 64])
        # a scatter's send buffers hold p shards, which bounds them by memory as well
        hi = min(128 * MIB, MOST_BYTES // (p + 1), (4 << 30) // (p * p if kind == "scatter" else p))
        case.update(nsrc=p, count=_count(rng, 8 * KIB, hi, es))
        if kind == "scatter":
            case.update(rank=rng.randrange(p))
        else:
            case.update(views=rng.choices(["aligned", "shared", "mixed"], [6, 2, 2])[0])
    elif kind == "ring":
        # the ring's accumulators stay on chip: at most 4 MiB a chunk here, for every dtype
        case.update(nsrc=rng.randint(2, 32), count=_count(rng, 16 * KIB, 4 * MIB, es),
                    flags=rng.random() < 0.5)
    elif kind == "steps":
        case.update(nsrc=rng.randint(2, 16), count=_count(rng, 64 * KIB, 16 * MIB, es),
                    final=rng.random() < 0.5)
    elif kind == "batched":
        how = rng.choice(["host", "device", "graph", "noalloc"])
        case.update(nsrc=rng.choice([2, 4, 8, 8, 8, 16]),
                    items=int(_log_uniform(rng, 8, 1024 if how == "host" else 4096)),
                    min_bytes=8 * KIB,
                    max_bytes=rng.choice([16 * KIB, 128 * KIB, MIB]), sizes=rng.randrange(10_000),
                    how=how)
    else:
        schedule = rng.choice(["ring", "rhd", "ring1", "rhd1"])
        g = rng.choice([2, 4, 8, 16] if schedule[:3] == "rhd" else [2, 3, 4, 6, 8, 16])
        case.update(nsrc=g, count=_count(rng, 64 * KIB, 512 * MIB // g // 2, es),
                    schedule=schedule)
    return case


# ------------------------------------------------------------------ inputs --
def _values(n, dtype, gen):
    """n values as gradients have them (small and normal), or whole 32/64-bit integers."""
    if dtype in ("i32", "i64"):
        info = torch.iinfo(TORCH[dtype])
        return torch.empty(n, dtype=TORCH[dtype], device="cuda").random_(
            info.min, info.max, generator=gen)
    if dtype == "e4m3":   # scaled into the format's range, as fp8 gradients are
        out = torch.empty(n, dtype=TORCH[dtype], device="cuda")
        for lo in range(0, n, 1 << 24):
            part = out[lo:lo + (1 << 24)]
            part.copy_(torch.empty(part.numel(), device="cuda").normal_(generator=gen))
        return out
    scale = 1e-3 if dtype != "f16" else 1e-2   # fp16 gradients are loss-scaled
    return torch.empty(n, dtype=TORCH[dtype], device="cuda").normal_(0.0, scale, generator=gen)


def _sizes(case):
    """Elements of every message of a batch: bytes log-uniform between the bounds."""
    g = np.random.default_rng(case["sizes"])
    u = g.uniform(math.log(case["min_bytes"]), math.log(case["max_bytes"]), case["items"])
    return np.maximum(1, np.rint(np.exp(u) / SIZE[case["dtype"]])).astype(np.int64)


def _offsets(case):
    """Element offset of every source and output in their arenas, and the arenas' lengths."""
    step = ARENA // SIZE[case["dtype"]]
    padded = (_sizes(case) + step - 1) // step * step
    out = np.concatenate([[0], np.cumsum(padded)])
    src = np.concatenate([[0], np.cumsum(np.repeat(padded, case["nsrc"]))])
    return src[:-1].reshape(-1, case["nsrc"]), int(src[-1]), out[:-1], int(out[-1])


def _view_offset(case, p):
    """Elements by which source p of an AllReduce starts past an aligned address."""
    return {"aligned": 0, "shared": 3, "mixed": (3 * p + 1) % 8}[case["views"]]


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype, n, p = case["dtype"], case.get("count"), case["nsrc"]
    empty = lambda k, t=TORCH[dtype]: torch.empty(k, dtype=t, device="cuda")  # noqa: E731
    state = {"case": case}
    if case["kind"] == "allreduce":
        flat = [_values(n + 8, dtype, gen) for _ in range(p)]
        state["srcs"] = [f[_view_offset(case, q):][:n] for q, f in enumerate(flat)]
        out = empty(n + 8)
        state["out"] = out[3:][:n] if case["views"] == "shared" else out[:n]
    elif case["kind"] == "scatter":
        state["srcs"] = [_values(n * p, dtype, gen) for _ in range(p)]
        state["out"] = empty(n)
    elif case["kind"] == "ring":
        state["chunks"] = [_values(n, dtype, gen) for _ in range(p)]
        state["out"] = empty(n)
        state["ready"] = torch.ones(p, dtype=torch.int32, pin_memory=True) if case["flags"] else None
    elif case["kind"] == "steps":
        state["chunks"] = list(_values(n * p, dtype, gen).split(n))
        state["acc"], state["out"] = empty(n, ACC[dtype]), empty(n)
    elif case["kind"] == "sim":
        state["sends"] = [_values(n, dtype, gen) for _ in range(p)]
        state["recvs"] = [empty(n) for _ in range(p)]
    else:
        sizes = _sizes(case)
        src_at, src_len, out_at, out_len = _offsets(case)
        arena = state["arena"] = _values(src_len, dtype, gen)
        out = state["out"] = empty(out_len).zero_()   # the padding between outputs stays zero
        if case["how"] == "host":
            state["items"] = [([arena[a:a + s] for a in row.tolist()], out[o:o + s])
                              for row, o, s in zip(src_at, out_at.tolist(), sizes.tolist())]
        else:
            state["items"], state["ptrs"] = _device_items(case, arena, out, src_at, out_at, sizes)
        if case["how"] == "graph":
            _batched(state)   # the kernel is loaded before the capture
            graph = state["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                _batched(state)
    return state


def _device_items(case, arena, out, src_at, out_at, sizes):
    """The batch's descriptors and source pointers in device memory."""
    es = SIZE[case["dtype"]]
    ptrs = torch.from_numpy(arena.data_ptr() + es * src_at).to("cuda")
    rows = np.zeros(case["items"], xr._lib.ITEM_DTYPE)
    rows["srcs"] = ptrs.data_ptr() + 8 * case["nsrc"] * np.arange(case["items"])
    rows["dst"] = out.data_ptr() + es * out_at
    rows["count"] = sizes
    rows["nsrc"] = case["nsrc"]
    return torch.from_numpy(rows.view(np.uint8).copy()).to("cuda"), ptrs


# -------------------------------------------------------------------- runs --
def _batched(state):
    case = state["case"]
    call = xr.batched_reduce_noalloc if case["how"] == "noalloc" else xr.batched_reduce
    call(state["items"], case["op"], dtype=case["dtype"])


def run(state):
    case = state["case"]
    kind, op = case["kind"], case["op"]
    if kind == "allreduce":
        xr.allreduce_local(state["srcs"], state["out"], op)
        return state["out"]
    if kind == "scatter":
        xr.reduce_scatter_local(state["srcs"], case["rank"], state["out"], op)
        return state["out"]
    if kind == "ring":
        xr.ring_reduce(state["chunks"], state["out"], op, ready=state["ready"])
        return state["out"]
    if kind == "steps":
        chunks, acc, out = state["chunks"], state["acc"], state["out"]
        xr.reduce_copy_step(chunks[0], acc, None, op, init=True)
        for c in chunks[1:-1]:
            xr.reduce_copy_step(c, acc, None, op)
        if case["final"]:
            xr.reduce_copy_step(chunks[-1], acc, out, op, final=True)
        else:
            xr.reduce_copy_step(chunks[-1], acc, None, op)
            xr.acc_cast(acc, out)
        return [acc, out]
    if kind == "sim":
        xr.allreduce_sim(state["sends"], state["recvs"], op, schedule=case["schedule"])
        return state["recvs"]
    if case["how"] == "graph":
        state["graph"].replay()
    else:
        _batched(state)
    return state["out"]


def work(case):
    """Every source read once, every output written once, one operation per folded element
    (a step sequence cannot keep its accumulator out of memory between its calls: it is
    written by every call but a final one and read by every call but the first; a simulated
    AllReduce reads every rank's buffer and writes every rank's result)."""
    es, p = SIZE[case["dtype"]], case["nsrc"]
    n = int(_sizes(case).sum()) if case["kind"] == "batched" else case["count"]
    moved = (p + 1) * n * es
    if case["kind"] == "steps":
        acc = torch.empty((), dtype=ACC[case["dtype"]]).element_size()
        moved += n * acc * (2 * p - 2 if case["final"] else 2 * p)
    elif case["kind"] == "sim":
        moved = 2 * p * n * es
    return {"bytes": moved, "flops": (p - 1) * n}


def tolerance(case):
    """Every result is a fixed-order fold with one rounding per operation, the same bits on
    every run and for every launch shape: that is what the entry points promise."""
    return "exact"


# ------------------------------------------------------------------- exact --
def _fold(tensors, op):
    """The fold in 64 bits: float64, or int64 (which wraps as the narrower types do)."""
    wide = torch.float64 if tensors[0].is_floating_point() else torch.int64
    acc = tensors[0].to(wide)
    for t in tensors[1:]:
        if op in ("sum", "avg"):
            acc += t.to(wide)
        elif op == "max":
            acc = torch.maximum(acc, t.to(wide))
        else:
            acc = torch.minimum(acc, t.to(wide))
    if op == "avg":
        acc /= len(tensors)
    return acc


def exact(case, seed):
    state = prepare(dict(case, how="device") if case["kind"] == "batched" else case, seed)
    kind, op, n, p = case["kind"], case["op"], case.get("count"), case["nsrc"]
    # whole numbers come back in the outputs' own type
    back = (lambda t: t.to(TORCH[case["dtype"]])) if case["dtype"][0] == "i" else (lambda t: t)
    if kind == "allreduce":
        return back(_fold(state["srcs"], op))
    if kind == "scatter":
        at = n * case["rank"]
        return back(_fold([s[at:at + n] for s in state["srcs"]], op))
    if kind == "ring":
        return back(_fold(state["chunks"], op))
    if kind == "steps":
        done = p - 1 if case["final"] else p
        return [back(_fold(state["chunks"][:done], op)), back(_fold(state["chunks"], op))]
    if kind == "sim":
        return [back(_fold(state["sends"], op))] * p
    src_at, _, out_at, out_len = _offsets(case)
    arena = state["arena"]
    result = torch.zeros(out_len, dtype=torch.float64 if arena.is_floating_point() else torch.int64,
                         device="cuda")
    for row, o, s in zip(src_at.tolist(), out_at.tolist(), _sizes(case).tolist()):
        result[o:o + s] = _fold([arena[a:a + s] for a in row], op)
    return back(result)
