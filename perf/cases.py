"""The work this library is used for, as cases that can be timed and checked one by one.

A case is a plain dict.  ``prepare`` makes what a program holds before the call (inputs, outputs, workspace), ``run`` is
one pass through the public entry points of ``paper_2411_17887_amd.tcuscan``, ``exact`` the same result from plain torch
in 64 bits.  Four kinds of work, by ``op``:

  scan       row-wise prefix sums of a dense rows x cols matrix (tcuscan_scan), every input type, inclusive / exclusive,
             forward / reverse
  segmented  prefix sums of rows of different lengths stored back to back (tcuscan_segmented)
  compact    stream compaction of 32-bit values by a 0/1 mask (tcuscan_compact_u32)
  sort       radix sort of 32-bit keys, alone or with 32-bit payloads (tcuscan_split_radix_sort_u32)
"""
from __future__ import annotations

import math

import torch

from paper_2411_17887_amd import tcuscan

IN_BYTES = {"i32": 4, "f16": 2, "i8": 1, "f32": 4, "bf16": 2}
FLOATS = ("f16", "f32", "bf16")


def listed():
    return [
        # The smallest call: one workgroup, nothing but launch latency (offsets of a small batch, a digit table).
        scan("scan_i32_4096", "i32", 1, 4096),
        # A medium single row: a cumulative distribution over a sampling weight vector.
        scan("scan_f16_16m", "f16", 1, 1 << 24),
        # The destination indices of a 2^28-element filter: exclusive scan of a 0/1 mask.
        scan("mask_scan_i8_268m", "i8", 1, 1 << 28, exclusive=True),
        # A long signal of odd length in fp32.
        scan("scan_f32_100m", "f32", 1, 100_000_007),
        # A batch of long rows in bf16 (cumulative sums along the sequence dimension).
        scan("rows_bf16_4096x65536", "bf16", 4096, 65536),
        # The same with rows that do not start at 16-byte boundaries, from the end (returns-to-go: suffix sums).
        scan("suffix_bf16_4095x65537", "bf16", 4095, 65537, reverse=True),
        # Many short rows of odd length (histograms of a tree learner: one row per feature and node).
        scan("hist_f32_127000x2101", "f32", 127_000, 2101),
        # Ragged rows, short: per-user or per-document sequences, mean length 200.
        segmented("ragged_f32_mean200", "f32", 1 << 26, 335_544),
        # Ragged rows, long: a batch of 64 sequences packed back to back.
        segmented("ragged_bf16_64rows", "bf16", 1 << 27, 64),
        # A filter: 32-bit values kept by a mask, the positions not asked for.
        compact("compact_268m", 1 << 28),
        # A full sort of 32-bit keys.
        sort("sort_keys_67m", 1 << 26),
        # A medium sort of (key, payload) pairs of odd length (an argsort).
        sort("sort_pairs_4m", (1 << 22) + 9, pairs=True),
    ]


def scan(name, kind, rows, cols, exclusive=False, reverse=False):
    return dict(name=name, op="scan", kind=kind, rows=rows, cols=cols, exclusive=exclusive, reverse=reverse)


def segmented(name, kind, total, rows, exclusive=False, reverse=False):
    return dict(name=name, op="segmented", kind=kind, rows=rows, total=total, exclusive=exclusive, reverse=reverse)


def compact(name, n, density=0.5, positions=False):
    return dict(name=name, op="compact", n=n, density=density, positions=positions)


def sort(name, n, bits=32, pairs=False):
    return dict(name=name, op="sort", n=n, bits=bits, pairs=pairs)


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], its logarithm uniform."""
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    op = rng.choice(["scan", "scan", "segmented", "segmented", "compact", "sort"])
    kind = rng.choice(["i32", "f16", "i8", "f32", "bf16"])
    most = (1 << 28) * 6 // (IN_BYTES[kind] + 4)                  # elements: no more bytes than the largest row-wise case
    options = dict(exclusive=rng.random() < 0.4, reverse=rng.random() < 0.3)
    if op == "scan":
        if rng.random() < 0.4:                                    # one row
            rows, cols = 1, _log_int(rng, 4096, most)
        else:                                                     # a batch: row length first, then as many rows as fit
            cols = _log_int(rng, 64, 1 << 22)
            rows = _log_int(rng, 1, most // cols)
            if rows * cols < 4096:
                rows = -(-4096 // cols)
        if rng.random() < 0.3:                                    # as often as in use, a multiple of 64
            cols = max(64, cols // 64 * 64)
        case = scan("", kind, rows, cols, **options)
    elif op == "segmented":
        total = _log_int(rng, 1 << 14, most // 2)
        mean = _log_int(rng, 16, total // 4)
        case = segmented("", kind, total, max(1, total // mean), **options)
    elif op == "compact":
        positions = rng.random() < 0.3
        n = _log_int(rng, 1 << 12, 1 << 28) if not positions else _log_int(rng, 1 << 12, 170_000_000)
        case = compact("", n, density=round(rng.uniform(0.02, 0.98), 3), positions=positions)
    else:
        pairs = rng.random() < 0.5
        bits = rng.choice([32, 32, 32, 24, 16, rng.randint(1, 31)])
        case = sort("", _log_int(rng, 1 << 10, 1 << (25 if pairs else 26)), bits=bits, pairs=pairs)
    case.pop("name")
    return case


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _values(kind, n, exclusive, g):
    """Inputs of the distributions the benchmark's configurations use."""
    if kind == "i32":
        return torch.randint(-128, 128, (n,), generator=g, device="cuda", dtype=torch.int32)
    if kind == "i8":                       # a mask for exclusive scans (destination indices), whole-range counts otherwise
        lo, hi = (0, 2) if exclusive else (-128, 128)
        return torch.randint(lo, hi, (n,), generator=g, device="cuda", dtype=torch.int8)
    if kind == "f32":
        return torch.randn(n, generator=g, device="cuda", dtype=torch.float32)
    u = torch.rand(n, generator=g, device="cuda", dtype=torch.float32)
    if kind == "f16":
        return u.mul_(0.9995).to(torch.float16)                   # [0, 1), also after rounding
    return u.mul_(2.0).sub_(1.0).to(torch.bfloat16)


def _keys(n, g):
    return torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)


def _offsets(rows, total, g):
    """rows + 1 offsets of rows with exponentially distributed lengths that fill `total` elements (some of them empty)."""
    w = -torch.log1p(-torch.rand(rows, generator=g, device="cuda", dtype=torch.float64))
    ends = torch.cumsum(w, 0)
    off = torch.zeros(rows + 1, dtype=torch.int64, device="cuda")
    off[1:] = (ends / ends[-1] * total).floor().to(torch.int64).clamp_(0, total)
    off[-1] = total
    return off


def _out_dtype(kind):
    return torch.float32 if kind in FLOATS else torch.int32


def _flags(case):
    return (tcuscan.EXCLUSIVE if case["exclusive"] else 0) | (tcuscan.REVERSE if case["reverse"] else 0)


def prepare(case, seed):
    g, s = _generator(seed), {"case": case}
    if case["op"] == "scan":
        n = case["rows"] * case["cols"]
        s["x"] = _values(case["kind"], n, case["exclusive"], g)
        s["out"] = torch.empty(n, dtype=_out_dtype(case["kind"]), device="cuda")
        s["ws"] = tcuscan.new_workspace(case["rows"], case["cols"], case["kind"])
    elif case["op"] == "segmented":
        n, rows = case["total"], case["rows"]
        s["x"] = _values(case["kind"], n, case["exclusive"], g)
        s["offsets"] = _offsets(rows, n, g)
        s["out"] = torch.empty(n, dtype=_out_dtype(case["kind"]), device="cuda")
        s["ws"] = tcuscan.new_segmented_workspace(rows, n, case["kind"])
    elif case["op"] == "compact":
        n = case["n"]
        s["values"] = _keys(n, g)
        s["mask"] = (torch.rand(n, generator=g, device="cuda") < case["density"]).to(torch.int8)
        s["out"] = torch.zeros(n, dtype=torch.int32, device="cuda")
        s["positions"] = torch.empty(n, dtype=torch.int32, device="cuda") if case["positions"] else None
        s["count"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        s["ws"] = tcuscan.new_workspace(1, n, "i8")
    else:
        n = case["n"]
        s["keys_in"] = _keys(n, g)
        s["keys"], s["keys_tmp"] = torch.empty_like(s["keys_in"]), torch.empty_like(s["keys_in"])
        s["vals_in"] = torch.arange(n, dtype=torch.int32, device="cuda") if case["pairs"] else None
        s["vals"] = torch.empty_like(s["keys_in"]) if case["pairs"] else None
        s["vals_tmp"] = torch.empty_like(s["keys_in"]) if case["pairs"] else None
        s["flags"] = torch.empty(n, dtype=torch.int8, device="cuda")
        s["positions"] = torch.empty(n, dtype=torch.int32, device="cuda")
        s["ws"] = tcuscan.new_workspace(1, n, "i8")
    return s


def run(s):
    case = s["case"]
    if case["op"] == "scan":
        tcuscan.scan(s["x"], s["out"], case["rows"], case["cols"], case["kind"], flags=_flags(case), ws=s["ws"])
        return s["out"]
    if case["op"] == "segmented":
        tcuscan.segmented(s["x"], s["out"], s["offsets"], case["rows"], case["total"], case["kind"], flags=_flags(case), ws=s["ws"])
        return s["out"]
    if case["op"] == "compact":
        tcuscan.compact_u32(s["values"], s["mask"], s["out"], s["positions"], count=s["count"], ws=s["ws"])
        return {"kept": s["out"], "count": s["count"], "positions": s["positions"]}
    s["keys"].copy_(s["keys_in"])                                 # the sort is in place: new keys arrive for every pass
    if s["vals"] is not None:
        s["vals"].copy_(s["vals_in"])
    tcuscan.split_radix_sort_u32(s["keys"], s["keys_tmp"], s["flags"], s["positions"], vals=s["vals"], vals_tmp=s["vals_tmp"],
                                 bits=case["bits"], ws=s["ws"])
    return {"keys": s["keys"], "vals": s["vals"]}


def work(case):
    """Every input read once, every output written once; one addition per element of a scan."""
    if case["op"] == "scan":
        n = case["rows"] * case["cols"]
        return {"bytes": n * (IN_BYTES[case["kind"]] + 4), "flops": n}
    if case["op"] == "segmented":
        n = case["total"]
        return {"bytes": n * (IN_BYTES[case["kind"]] + 4) + 8 * (case["rows"] + 1), "flops": n}
    if case["op"] == "compact":
        n = case["n"]
        return {"bytes": 5 * n + 4 * case["density"] * n + (4 * n if case["positions"] else 0), "flops": n}
    return {"bytes": 8 * case["n"] * (2 if case["pairs"] else 1), "flops": 0}


def tolerance(case):
    """Integers, kept values and sorted keys are unique.  Floating-point prefix sums are fp32 sums in an unspecified order:
    against 64 bits the path is off by 7e-8 to 5e-7 (2-norm), and by 1e-6 at the worst element from call to call."""
    if case["op"] in ("scan", "segmented") and case["kind"] in FLOATS:
        return {"rel": 2e-6, "max": 1e-5}
    return "exact"


def exact(case, seed):
    s = prepare(case, seed)
    if case["op"] == "scan":
        x = s["x"].view(case["rows"], case["cols"]).to(torch.float64 if case["kind"] in FLOATS else torch.int64)
        del s
        y = _row_sums(x, case)
        return (y if case["kind"] in FLOATS else y.to(torch.int32)).reshape(-1)
    if case["op"] == "segmented":
        x = s["x"].to(torch.float64 if case["kind"] in FLOATS else torch.int64)
        off = s["offsets"]
        lens = off[1:] - off[:-1]
        row = torch.repeat_interleave(torch.arange(case["rows"], device="cuda"), lens)
        if case["reverse"]:                                       # flip everything: rows and elements in reverse order
            x, row, lens = x.flip(0), (case["rows"] - 1) - row.flip(0), lens.flip(0)
        start = torch.cumsum(lens, 0) - lens
        inc = torch.cumsum(x, 0)
        before = torch.cat([inc.new_zeros(1), inc])[start]        # everything in front of the row
        y = inc - before[row]
        if case["exclusive"]:
            y = y - x
        if case["reverse"]:
            y = y.flip(0)
        return y if case["kind"] in FLOATS else y.to(torch.int32)
    if case["op"] == "compact":
        keep = s["mask"] != 0
        kept = s["values"][keep]
        out = torch.zeros_like(s["values"])
        out[: kept.numel()] = kept
        pos = (torch.cumsum(s["mask"], 0, dtype=torch.int64) - s["mask"]).to(torch.int32) if case["positions"] else None
        return {"kept": out, "count": torch.tensor([kept.numel()], dtype=torch.int32), "positions": pos}
    low = (s["keys_in"].to(torch.int64) & 0xFFFFFFFF) & ((1 << case["bits"]) - 1)
    order = torch.sort(low, stable=True).indices
    return {"keys": s["keys_in"][order], "vals": s["vals_in"][order] if case["pairs"] else None}


def _row_sums(x, case):
    if case["reverse"]:
        x = x.flip(1)
    y = torch.cumsum(x, 1)
    if case["exclusive"]:
        y = y - x
    return y.flip(1) if case["reverse"] else y
