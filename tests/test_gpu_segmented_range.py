"""GPU parity of segmented scans that go over the rows' range as a whole, where the search for a tile's row starts can go
wrong: numbers of rows at the edges of its windows and rounds, stretches of empty rows longer than a window, calls at the edge
between the small and the large kernel, tiles with more rows than expected; bad offsets in every kernel."""
import numpy as np
import pytest

from paper_2411_17887_amd import inputs, tcuscan
from gpu_util import out_dtype, to_device
from test_gpu_segmented import GUARD, INT_GEN, RND_GEN, check, offsets_from, run_segmented

pytestmark = pytest.mark.gpu

LARGE = 3 << 22                     # elements from which on the large kernel runs


def spread(rng, rows, total):
    """`rows` lengths, exponentially distributed, that fill `total` elements."""
    ends = np.cumsum(rng.exponential(size=rows))
    off = np.floor(ends / ends[-1] * total).astype(np.int64)
    off[-1] = total
    return np.diff(np.concatenate([[0], off]))


def with_empty(lens, at, count):
    return np.concatenate([lens[:at], np.zeros(count, np.int64), lens[at:]])


def layout(name, rng):
    """Row lengths.  Windows hold 1024 offsets (small kernel), 256 (a run of the large one) and 2048 (its tiles of long rows)."""
    kind, _, arg = name.partition(":")
    n = int(arg) if arg else 0
    if kind == "small":             # n rows in a call of one launch
        return spread(rng, n, 300_000 + n)
    if kind == "long":              # n long rows in a large call
        return spread(rng, n, LARGE + 12345)
    if kind == "short":             # n elements per row on average in a large call
        return spread(rng, LARGE // n, LARGE + 77)
    if kind == "empty_small":       # n empty rows in the middle, and at the end
        return with_empty(with_empty(spread(rng, 5000, 200_003), 2500, n), 5000 + n, n)
    if kind == "empty_short":
        return with_empty(with_empty(spread(rng, 100_000, LARGE + 9), 40_000, n), 100_000 + n, n)
    if kind == "empty_long":
        return with_empty(spread(rng, 900, 2 * LARGE + 5), 450, n)
    if kind == "dense":             # rows of one element for a stretch, one row for the rest: many more rows in a tile than expected
        return np.concatenate([np.ones(40_000, np.int64), [n - 40_000]])
    raise AssertionError(name)


@pytest.mark.parametrize("flags", [0, 3])
@pytest.mark.parametrize("name,kinds", [
    ("small:1022", "i32 bf16"), ("small:1023", "i8 i32"), ("small:1024", "i32 f16"), ("small:3000", "i8"), ("small:1100000", "i32 i8"),
    ("long:254", "i8 f32"), ("long:255", "i32 bf16"), ("long:256", "i8 i32"), ("long:2046", "i8"), ("long:2047", "bf16 i8"), ("long:2500", "i8"),
    ("short:16", "i32 i8"), ("short:200", "i8 f32"), ("short:1900", "i32 f16"), ("short:4200", "i8"),
    ("empty_small:5000", "i32 i8"), ("empty_small:1100000", "i8"), ("empty_short:300000", "i32 i8"), ("empty_long:5000", "i8 bf16"),
    ("dense:300000", "i32 i8"), ("dense:13000000", "i8 i32"),
])
def test_row_starts_are_found(name, kinds, flags):
    rng = np.random.default_rng(len(name) + flags)
    lens = layout(name, rng)
    off = offsets_from(lens, start=flags)                        # (also a range that does not start at a boundary)
    for kind in kinds.split():
        x = (INT_GEN if kind in INT_GEN else RND_GEN)[kind](int(off[-1]) + 5, 77)
        got, fault = run_segmented(x, kind, off, flags=flags)
        assert fault == 0
        check(x, kind, off, got, bool(flags & 1), bool(flags & 2))


@pytest.mark.parametrize("total", [LARGE - 1, LARGE, LARGE + 8191, 4 * LARGE - 3, 4 * LARGE])
@pytest.mark.parametrize("rows", [3, 700, 3000])
def test_edges_of_the_rules_and_one_workspace(total, rows):
    """One workspace through both forms and a call of one row in between: status words, first rows and row maps do not get mixed up."""
    rng = np.random.default_rng(total + rows)
    off = offsets_from(spread(rng, rows, total))
    x = inputs.int32_full(total, 5)
    ws = tcuscan.new_segmented_workspace(rows, total, "i32")
    want = None
    for flat in (True, False, True):
        tcuscan.set_segmented_form(flat)
        try:
            got, fault = run_segmented(x, "i32", off, ws=ws)
        finally:
            tcuscan.set_segmented_form(True)
        assert fault == 0
        if want is None:
            check(x, "i32", off, got, False, False)
            want = got
        assert np.array_equal(got, want)
        got, fault = run_segmented(x[:50_000], "i32", np.array([0, 50_000], np.int64), ws=ws)
        assert fault == 0 and np.array_equal(got, np.cumsum(x[:50_000], dtype=np.int64).astype(np.int32))


@pytest.mark.parametrize("name", ["small:3000", "small:60000", "long:250", "long:2500", "short:200"])
@pytest.mark.parametrize("break_at", ["swap", "beyond", "negative"])
def test_bad_offsets_raise_the_fault_word_in_every_kernel(name, break_at):
    import torch
    lens = layout(name, np.random.default_rng(3))
    off = offsets_from(lens)
    total, k = int(off[-1]), lens.size * 2 // 3
    if break_at == "swap":
        off[k] = off[k + 2] + 1 if off[k + 2] < total else off[k - 2] - 1
    else:
        off[k] = total + 1000 if break_at == "beyond" else -1000
    d_in = torch.ones(total + 4096, dtype=torch.int32, device="cuda")
    d_out = torch.full((total + 8192,), -77, dtype=torch.int32, device="cuda")
    ws = tcuscan.new_segmented_workspace(lens.size, total, "i32")
    tcuscan.segmented(d_in, d_out[4096:], torch.from_numpy(off).cuda(), lens.size, total, "i32", ws=ws)
    assert tcuscan.workspace_fault(ws) == 2
    assert bool((d_out[:4096] == -77).all()) and bool((d_out[4096 + total:] == -77).all())          # nothing outside the arrays is written


@pytest.mark.parametrize("kind", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("flags", [0, 3])
@pytest.mark.parametrize("mean", [1451, 30_000])
def test_large_calls_round_as_rarely_as_results_held_back(mean, flags, kind):
    """What lies before a run is added to its sums once.  An addition is off by up to half a unit in the last place, 2.5e-8 of the
    sum in the root mean square; eight of them at the size of the result (granule, lanes, tile, run, wavefronts, workgroups) make 7.1e-8."""
    import torch
    total, dtype = LARGE + 8191, {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[kind]
    off = torch.from_numpy(offsets_from(spread(np.random.default_rng(mean), total // mean, total))).cuda()
    x = torch.rand(total, generator=torch.Generator(device="cuda").manual_seed(mean), device="cuda").mul_(0.9995).to(dtype)
    out, rows = torch.empty(total, device="cuda"), off.numel() - 1
    tcuscan.segmented(x, out, off, rows, total, kind, flags=flags, ws=tcuscan.new_segmented_workspace(rows, total, kind))
    inc = torch.cumsum(x.double(), 0)
    ex = torch.cat([inc.new_zeros(1), inc])
    row = torch.repeat_interleave(torch.arange(rows, device="cuda"), off[1:] - off[:-1])
    ref = ex[off[row + 1]] - inc if flags == 3 else inc - ex[off[row]]             # 3: exclusive and reverse
    err = float((out.double() - ref).norm() / ref.norm())
    assert err < 7.1e-8


def run_shifted(x, kind, off, flags, ws, shift_in, shift_out, inplace=False):
    """run_segmented with arrays that start some elements into their allocations."""
    import torch
    big = to_device(np.concatenate([np.zeros(shift_in, x.dtype), x]), kind)
    d_in = big[shift_in:]
    big_out = torch.full((x.size + shift_out,), GUARD, dtype=out_dtype(kind), device="cuda")
    d_out = d_in if inplace else big_out[shift_out:]
    tcuscan.segmented(d_in, d_out, torch.from_numpy(off).cuda(), off.size - 1, x.size, kind, flags=flags, ws=ws)
    torch.cuda.synchronize()
    assert bool((big_out[:shift_out] == GUARD).all()) and bool((big[:shift_in] == 0).all())
    return d_out.cpu().numpy().copy(), tcuscan.workspace_fault(ws)


@pytest.mark.parametrize("kind", ["i32", "f16", "i8", "f32", "bf16"])
@pytest.mark.parametrize("rows,total", [(1, 1 << 19), (1, 600_001), (1, 1 << 22), (3, 1_700_003), (8, 1 << 22), (7, 4_000_001)])
def test_few_long_rows_of_a_small_call(rows, total, kind):
    """Status words of small tiles in a layout for large ones, up to eight to a slot: all directions, tickets, misaligned and
    in place, and the same workspace under calls that have a word to a slot."""
    import torch
    off = offsets_from(spread(np.random.default_rng(rows + total), rows, total))
    x = (INT_GEN if kind in INT_GEN else RND_GEN)[kind](total, 9)
    ws = tcuscan.new_segmented_workspace(rows, total, kind)
    for flags in range(4):
        for policy in ((0, 1) if flags == 2 else (0,)):
            tcuscan.set_chain_policy(policy)
            try:
                got, fault = run_shifted(x, kind, off, flags, ws, 3 * (flags == 1), 5 * (flags == 1))
            finally:
                tcuscan.set_chain_policy(0)
            assert fault == 0
            check(x, kind, off, got, bool(flags & 1), bool(flags & 2))
            n = total // 16                                            # a status word to a slot, on the same workspace
            if tcuscan.segmented_workspace_bytes(1, n, kind) <= ws.numel() * 8:
                got, fault = run_segmented(x[:n], kind, offsets_from([n]), flags=flags, ws=ws)
                assert fault == 0
                check(x[:n], kind, offsets_from([n]), got, bool(flags & 1), bool(flags & 2))


def test_few_long_rows_recorded_into_a_graph():
    """Recorded with status words that share slots; eager calls on the same workspace between the replays."""
    import torch
    rows, total = 2, 1_300_007
    off = offsets_from(spread(np.random.default_rng(4), rows, total))
    d_off, ws = torch.from_numpy(off).cuda(), tcuscan.new_segmented_workspace(rows, total, "i8")
    d_in, d_out = torch.empty(total, dtype=torch.int8, device="cuda"), torch.empty(total, dtype=torch.int32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tcuscan.segmented(d_in, d_out, d_off, rows, total, "i8", ws=ws)
    for seed in (1, 2, 3):
        x = INT_GEN["i8"](total, seed)
        d_in.copy_(torch.from_numpy(x))
        d_out.fill_(-77)
        graph.replay()
        torch.cuda.synchronize()
        check(x, "i8", off, d_out.cpu().numpy(), False, False)
        d_out.fill_(-77)
        tcuscan.segmented(d_in, d_out, d_off, rows, total, "i8", flags=3, ws=ws)
        torch.cuda.synchronize()
        check(x, "i8", off, d_out.cpu().numpy(), True, True)
    assert tcuscan.workspace_fault(ws) == 0


@pytest.mark.parametrize("flags", range(4))
@pytest.mark.parametrize("kind", ["i32", "f16", "i8", "f32", "bf16"])
def test_ends_of_the_range(kind, flags):
    """Ranges that begin and end at every element of a granule, in arrays that begin at every element of one (then the first run
    begins in front of the array), down to arrays smaller than a granule; the small kernels."""
    per = {"i8": 16, "f16": 8, "bf16": 8}.get(kind, 4)
    x = (INT_GEN if kind in INT_GEN else RND_GEN)[kind](40_000, 3)
    for n in (1, 2, per - 1, per, per + 1, 2 * per + 1, 64 * per - 1, 64 * per + 3, 2048 + per // 2, 8192, 8193, 8192 + 2048 + 1, 39_000 + per - 1):
        for shift in {0, 1, per // 2, per - 1}:
            for skip in {0, 1, per - 1, per, per + 1}:
                off = offsets_from([n // 3, 0, n - n // 3 - n // 5, n // 5], start=skip)
                y = x[:n + skip + (n + shift) % 3]
                ws = tcuscan.new_segmented_workspace(off.size - 1, y.size, kind)
                got, fault = run_shifted(y, kind, off, flags, ws, shift, (shift * 5 + skip) % 7)
                assert fault == 0
                check(y, kind, off, got, bool(flags & 1), bool(flags & 2))


@pytest.mark.parametrize("flags", range(4))
@pytest.mark.parametrize("kind", ["i32", "f16", "i8", "f32", "bf16"])
def test_ends_of_a_large_range_of_long_rows(kind, flags):
    per = {"i8": 16, "f16": 8, "bf16": 8}.get(kind, 4)
    x = (INT_GEN if kind in INT_GEN else RND_GEN)[kind](LARGE + 70_000, 4)
    for case, (n, shift_in, shift_out, skip) in enumerate([(LARGE, 0, 0, 0), (LARGE + 1, 1, 1, 0), (LARGE + 65_536 - 1, per - 1, per - 1, 1), (LARGE + per + 1, 1, 0, per + 2),
                                                           (LARGE + 32_768 + 2, 8, 8, 3), (LARGE + 3, 0, 4, 0), (LARGE + 5, 4, 20, 31), (LARGE + 7, 24, 24, 2)]):
        rows = (1, 3, 300, 2500)[case % 4]
        off = offsets_from(spread(np.random.default_rng(case), rows, n), start=skip)
        y = x[:n + skip + case % 3]
        ws = tcuscan.new_segmented_workspace(rows, y.size, kind)
        got, fault = run_shifted(y, kind, off, flags, ws, shift_in, shift_out)
        assert fault == 0
        check(y, kind, off, got, bool(flags & 1), bool(flags & 2))


@pytest.mark.parametrize("flags", range(4))
@pytest.mark.parametrize("kind", ["i32", "f16", "i8", "f32", "bf16"])
def test_large_ranges_of_short_rows(kind, flags):
    """The form with first rows found in front: arrays that start at and off 16-byte boundaries and lines, ranges that start late."""
    per = {"i8": 16, "f16": 8, "bf16": 8}.get(kind, 4)
    x = (INT_GEN if kind in INT_GEN else RND_GEN)[kind](LARGE + 70_000, 6)
    for case, (n, mean, shift_in, shift_out, skip) in enumerate([(LARGE, 200, 1, 1, 0), (LARGE + 8191, 17, per - 1, 3, per + 2), (LARGE + 65_531, 1900, 24, 24, 2),
                                                                 (LARGE + 5, 700, 0, 2, 0), (LARGE + 16_384, 60, 8, 40, 31)]):
        off = offsets_from(spread(np.random.default_rng(case), n // mean, n), start=skip)
        y = x[:n + skip + case % 3]
        ws = tcuscan.new_segmented_workspace(off.size - 1, y.size, kind)
        got, fault = run_shifted(y, kind, off, flags, ws, shift_in, shift_out)
        assert fault == 0
        check(y, kind, off, got, bool(flags & 1), bool(flags & 2))


@pytest.mark.parametrize("flags", range(4))
@pytest.mark.parametrize("kind", ["i32", "f32", "bf16"])
@pytest.mark.parametrize("name", ["long:250", "long:2500", "short:200"])
def test_large_ranges_in_place_and_by_ticket(name, kind, flags):
    off = offsets_from(layout(name, np.random.default_rng(flags)), start=3)
    x = (INT_GEN if kind in INT_GEN else RND_GEN)[kind](int(off[-1]), 7)
    ws = tcuscan.new_segmented_workspace(off.size - 1, x.size, kind)
    for shift, policy in ((0, 1), (5, 0)):
        tcuscan.set_chain_policy(policy)
        try:
            got, fault = run_shifted(x, kind, off, flags, ws, shift, shift, inplace=kind != "bf16")
        finally:
            tcuscan.set_chain_policy(0)
        assert fault == 0
        if kind != "bf16":                                             # what lies outside the rows is still the input
            assert np.array_equal(got[:3], x[:3].view(got.dtype))
            got[:3] = GUARD
        check(x, kind, off, got, bool(flags & 1), bool(flags & 2))


@pytest.mark.parametrize("kind", ["i32", "i8", "bf16"])
@pytest.mark.parametrize("name", ["long:250", "long:2500", "short:200"])
def test_large_ranges_recorded_into_a_graph(name, kind):
    """Replays with other inputs, and eager calls from the end on the same workspace between them."""
    import torch
    off = offsets_from(layout(name, np.random.default_rng(11)))
    rows, total = off.size - 1, int(off[-1])
    d_off, ws = torch.from_numpy(off).cuda(), tcuscan.new_segmented_workspace(rows, total, kind)
    gen = (INT_GEN if kind in INT_GEN else RND_GEN)[kind]
    d_in, d_out = to_device(gen(total, 0), kind), torch.empty(total, dtype=out_dtype(kind), device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tcuscan.segmented(d_in, d_out, d_off, rows, total, kind, ws=ws)
    for seed in (1, 2, 3):
        x = gen(total, seed)
        d_in.copy_(to_device(x, kind))
        for flags in (0, 3):
            d_out.fill_(GUARD)
            torch.cuda.synchronize()
            if flags == 0:
                graph.replay()
            else:
                tcuscan.segmented(d_in, d_out, d_off, rows, total, kind, flags=flags, ws=ws)
            torch.cuda.synchronize()
            check(x, kind, off, d_out.cpu().numpy(), bool(flags & 1), bool(flags & 2))
    assert tcuscan.workspace_fault(ws) == 0


@pytest.mark.parametrize("kind", ["i32", "i8", "f32"])
def test_first_rows_are_not_taken_for_status_words(kind):
    """Short rows of a large call leave first rows in the workspace; plain scans, calls of one launch and few long rows with status
    words that share slots follow on it, in an order in which each comes right behind the first rows."""
    import torch
    total = LARGE + 4099
    x = (INT_GEN if kind in INT_GEN else RND_GEN)[kind](total, 8)
    off = {name: offsets_from(layout(name, np.random.default_rng(5))) for name in ("short:200", "long:2500", "long:250", "small:3000")}
    off["one"] = offsets_from([1_000_003])
    ws = torch.zeros(max(tcuscan.segmented_workspace_bytes(o.size - 1, int(o[-1]), kind) for o in off.values()) // 8 + 1, dtype=torch.int64, device="cuda")
    x = np.concatenate([x, x[:20_000]])
    plain = torch.empty(total, dtype=out_dtype(kind), device="cuda")
    for name in ("long:2500", "plain", "one", "small:3000", "long:250"):
        for then in ("short:200", name, name):
            if then == "plain":
                tcuscan.scan(to_device(x[:total], kind), plain, 1, total, kind, ws=ws)
                torch.cuda.synchronize()
                whole = offsets_from([total])
                check(x[:total], kind, whole, plain.cpu().numpy(), False, False)
                continue
            o = off[then]
            y = x[:int(o[-1])]
            got, fault = run_segmented(y, kind, o, ws=ws)
            assert fault == 0, (name, then)
            check(y, kind, o, got, False, False)
