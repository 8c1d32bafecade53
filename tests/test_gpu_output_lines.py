"""Rows whose outputs start inside 128-byte lines: tiled from the line below (or from the 16-byte boundary of the input)."""
import pytest

from paper_2411_17887_amd import tcuscan

pytestmark = pytest.mark.gpu

KINDS = ["i32", "f16", "i8", "f32", "bf16"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("flags", [0, 3])
def test_rows_that_start_inside_output_lines(kind, flags):
    """Rows tiled from the 128-byte line of the output: row lengths on either side of a line, of a tile and of the tile
    counts the short-row kernel is built for; arrays whose input and output fit no common line; an output that starts
    inside a line.  Exact integers, floats with small integer values (exact in every order)."""
    import torch
    tile = {"i8": 1024, "f16": 512, "bf16": 512}.get(kind, 256)
    lengths = [tile - 1, tile + 1, 2 * tile - 33, 2 * tile - 31, 2 * tile + 1, 3 * tile - 5, 5 * tile // 2 + 1, 8192 - 31, 8192 - 1, 8192 + 33, 40000 + 1]
    lengths += [k * tile - 16 for k in range(3, 12) if k * tile - 16 <= 2816]
    for cols in lengths + [20 * tile + 7]:
        rows = (8 << 20) // cols + 3                       # the form is taken from 2^23 outputs on
        n = rows * cols
        for shift_in, shift_out in ((0, 0), (0, 4), (16 // {"i8": 1, "f16": 2, "bf16": 2}.get(kind, 4), 8), (1, 1), (0, 1)):
            g = torch.Generator(device="cuda")
            g.manual_seed(cols + shift_in)
            x = torch.randint(-3, 4, (n + shift_in,), generator=g, device="cuda").to(
                {"i32": torch.int32, "i8": torch.int8, "f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[kind])[shift_in:]
            buf = torch.full((n + shift_out + 40,), -99, dtype=torch.int32 if kind in ("i32", "i8") else torch.float32, device="cuda")
            out = buf[shift_out:shift_out + n]
            ws = tcuscan.new_workspace(rows, cols, kind)
            tcuscan.scan(x, out, rows, cols, kind, flags=flags, ws=ws)
            ref = x.view(rows, cols).to(torch.int64)
            if flags & tcuscan.REVERSE:
                ref = ref.flip(1)
            ref = torch.cumsum(ref, 1) - (ref if flags & tcuscan.EXCLUSIVE else 0)
            if flags & tcuscan.REVERSE:
                ref = ref.flip(1)
            assert bool((out.view(rows, cols).to(torch.int64) == ref).all()), (kind, rows, cols, shift_in, shift_out)
            assert bool((buf[:shift_out] == -99).all()) and bool((buf[shift_out + n:] == -99).all())
            assert ws is None or tcuscan.workspace_fault(ws) == 0


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("policy", [tcuscan.TILE_SMALL, tcuscan.TILE_LARGE, tcuscan.TILE_HUGE], ids=["small", "large", "huge"])
def test_tile_policy_is_obeyed_by_rows_that_cross_lines(kind, policy):
    """The status words that a call leaves in a fresh workspace say how many tiles it ran: rows at 16-byte boundaries on the
    tile asked for, odd rows on it too, with the large one in place of the huge (their path has none)."""
    import torch
    rows = 9                                                                     # 9 x 1,000,001 > 2^23 outputs
    for cols in (1_000_016, 1_000_001):
        sizes = [tcuscan.tile_elems(kind), tcuscan.large_tile_elems(kind), tcuscan.huge_tile_elems(kind)]
        tile = sizes[policy - 1] if cols % 16 == 0 else sizes[min(policy, 2) - 1]
        x = torch.randint(-2, 3, (rows, cols), device="cuda").to(
            {"i32": torch.int32, "i8": torch.int8, "f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[kind])
        out = torch.empty(rows, cols, dtype=torch.int32 if kind in ("i32", "i8") else torch.float32, device="cuda")
        ws = tcuscan.new_workspace(rows, cols, kind)
        tcuscan.set_tile_policy(policy)
        try:
            tcuscan.scan(x, out, rows, cols, kind, flags=0, ws=ws)
            torch.cuda.synchronize()
        finally:
            tcuscan.set_tile_policy(tcuscan.TILE_AUTO)
        assert -(-cols // tile) == -(-(cols + 31) // tile)                       # the elements in front cost no tile here
        assert int((ws.view(torch.int64)[32::8] != 0).sum().item()) == rows * -(-cols // tile), (cols, tile)
        assert bool((out.to(torch.int64) == torch.cumsum(x.to(torch.int64), 1)).all())


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("flags", [0, 1, 2, 3])
def test_short_rows_on_either_side_of_the_form_rules(kind, flags):
    """Rows of one wavefront each whose form changes with their length, at 16-byte boundaries and odd, on both sides of each
    switch: 17/16 and 3/2 of two tiles, two to five tiles; in calls with and without the order by dies (16384 rows), and for
    three tiles with and without lines (2^25 outputs).  Exact."""
    import torch
    esz = {"i8": 1, "f16": 2, "bf16": 2}.get(kind, 4)
    tile = 1024 // esz
    lengths = [17 * tile // 16, 3 * tile // 2, 2 * tile - 32, 2 * tile + 16] + ([3 * tile - 48, 4 * tile + 16] if esz > 1 else [5 * tile // 2])
    for base in lengths:
        for cols in (base - 16, base, base + 1):
            for rows in {16384 - 64, 16384 + 64} | ({(1 << 25) // cols + 5} if esz == 4 and 2 * tile < cols <= 4 * tile else set()):
                if rows * cols < 1 << 23:
                    rows = (1 << 23) // cols + 1
                g = torch.Generator(device="cuda")
                g.manual_seed(cols)
                x = torch.randint(-3, 4, (rows, cols), generator=g, device="cuda").to(
                    {"i32": torch.int32, "i8": torch.int8, "f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[kind])
                buf = torch.full((rows * cols + 40,), -99, dtype=torch.int32 if kind in ("i32", "i8") else torch.float32, device="cuda")
                out = buf[:rows * cols].view(rows, cols)
                tcuscan.scan(x, out, rows, cols, kind, flags=flags, ws=tcuscan.new_workspace(rows, cols, kind))
                ref = x.to(torch.int32)
                if flags & tcuscan.REVERSE:
                    ref = ref.flip(1)
                ref = torch.cumsum(ref, 1, dtype=torch.int32) - (ref if flags & tcuscan.EXCLUSIVE else 0)
                if flags & tcuscan.REVERSE:
                    ref = ref.flip(1)
                assert bool((out.to(torch.int32) == ref).all()), (rows, cols)
                assert bool((buf[rows * cols:] == -99).all())


@pytest.mark.parametrize("kind,cols,total,tile", [
    ("i8", 200_001, 1 << 24, "small"), ("i8", 400_001, 60_000_000, "small"), ("i8", 400_001, 100_000_000, "large"), ("i8", 600_001, 60_000_000, "large"),
    ("bf16", 400_001, 1 << 24, "small"), ("f16", 500_001, 1 << 24, "small"), ("bf16", 400_001, 1 << 26, "large"), ("f16", 600_001, 1 << 25, "large"),
    ("f32", 400_001, 1 << 26, "small"), ("i32", 600_001, 1 << 26, "large")])
def test_tile_of_odd_rows(kind, cols, total, tile):
    """Which tile odd rows take, told by the status words that a call leaves in a fresh workspace, and the sums."""
    import torch
    rows = total // cols + 1
    elems = tcuscan.tile_elems(kind) if tile == "small" else tcuscan.large_tile_elems(kind)
    x = torch.randint(-2, 3, (rows, cols), device="cuda").to(
        {"i32": torch.int32, "i8": torch.int8, "f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[kind])
    out = torch.empty(rows, cols, dtype=torch.int32 if kind in ("i32", "i8") else torch.float32, device="cuda")
    ws = tcuscan.new_workspace(rows, cols, kind)
    tcuscan.scan(x, out, rows, cols, kind, flags=0, ws=ws)
    assert int((ws.view(torch.int64)[32::8] != 0).sum().item()) == rows * -(-(cols + 31) // elems)
    assert bool((out.to(torch.int32) == torch.cumsum(x.to(torch.int32), 1, dtype=torch.int32)).all())


@pytest.mark.parametrize("kind", KINDS)
def test_long_rows_on_either_side_of_the_form_rules(kind):
    """Rows of workgroup tiles whose form changes with their length, at 16-byte boundaries and odd: rows that leave their one
    tile half empty, lengths at which the elements in front would cost a tile, in a small and a big call.  A workspace larger
    than advised changes nothing: the status words left behind are those of the tiles of the rows themselves."""
    import torch
    esz = {"i8": 1, "f16": 2, "bf16": 2}.get(kind, 4)
    tile = tcuscan.tile_elems(kind)
    lengths = [13 * tile // 32, tile // 2, 9 * tile // 16, tile - 16, tile - 32, 2 * tile - 16, 2 * tile - 32, 3 * tile - 16, 8 * tile - 16]
    for base in lengths:
        for cols in (base, base - 15, base + 1):
            for total in (1 << 23, (1 << 25) + 1):
                rows = total // cols + 1
                x = torch.randint(-3, 4, (rows, cols), device="cuda").to(
                    {"i32": torch.int32, "i8": torch.int8, "f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[kind])
                buf = torch.full((rows * cols + 40,), -99, dtype=torch.int32 if kind in ("i32", "i8") else torch.float32, device="cuda")
                out = buf[:rows * cols].view(rows, cols)
                ref = torch.cumsum(x.to(torch.int32), 1, dtype=torch.int32)
                advised = tcuscan.workspace_bytes(rows, cols, kind)
                for extra in (0, 64 * rows):
                    ws = torch.zeros((advised + extra + 7) // 8 + 1, dtype=torch.int64, device="cuda")
                    buf.fill_(-99)
                    tcuscan.scan(x, out, rows, cols, kind, flags=0, ws=ws)
                    assert bool((out.to(torch.int32) == ref).all()) and bool((buf[rows * cols:] == -99).all()), (rows, cols)
                    tpr = -(-(cols + (16 // esz - 1 if cols * esz % 16 else 0)) // tile)      # all on the small tile here
                    assert int((ws[32::8] != 0).sum().item()) == (rows * tpr if tpr > 1 else 0), (rows, cols, extra)


DTYPES = {"i32": "int32", "i8": "int8", "f16": "float16", "bf16": "bfloat16", "f32": "float32"}


def values_with_loud_neighbours(kind, row_of, n, seed):
    """Integers over their whole range; floats of -3 .. 3, with every third row infinite, NaN or the largest finite value: an
    element of a neighbouring row that is not masked shows in the sums of a quiet row.  -> values, "this element is quiet"."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dtype = getattr(torch, DTYPES[kind])
    if kind == "i8":
        return torch.randint(-128, 128, (n,), generator=g, device="cuda").to(dtype), torch.ones(n, dtype=torch.bool, device="cuda")
    if kind == "i32":
        return torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device="cuda").to(dtype), torch.ones(n, dtype=torch.bool, device="cuda")
    x = torch.randint(-3, 4, (n,), generator=g, device="cuda").to(dtype)
    loud = torch.tensor([float("inf"), float("nan"), -float("inf"), torch.finfo(dtype).max], device="cuda").to(dtype)
    quiet = row_of % 3 != 1
    return torch.where(quiet, x, loud[row_of // 3 % 4]), quiet


def row_sums(x, quiet, starts, row_of, flags):
    """Sums of the rows that begin at `starts`, in 64 bits; loud rows count as zero."""
    import torch
    v = torch.where(quiet, x, torch.zeros_like(x)).to(torch.int64)
    inc = torch.cumsum(v, 0)
    before = torch.cat([inc.new_zeros(1), inc])
    ends = torch.cat([starts[1:], starts.new_tensor([v.numel()])])
    if flags & tcuscan.REVERSE:
        return before[ends][row_of] - (inc if flags & tcuscan.EXCLUSIVE else inc - v)
    return inc - before[starts][row_of] - (v if flags & tcuscan.EXCLUSIVE else 0)


def agree(got, ref, quiet):
    import torch
    if got.dtype == torch.int32:
        return bool((got == ref.to(torch.int32)).all())                          # modulo 2^32
    return bool((got[quiet].to(torch.int64) == ref[quiet]).all())


@pytest.mark.parametrize("how,kind", [(how, kind) for how in ("workspace", "tickets", "static") for kind in KINDS]
                         + [("in place", "i32"), ("in place", "f32")])
def test_rows_from_lines_are_masked_and_chained(kind, how):
    """All four kinds of scan, rows of one wavefront and of workgroup tiles, odd and at 16-byte boundaries, with loud
    neighbours; through a workspace, with tickets, through the fixed scratch, in place (32-bit)."""
    import torch
    for rows, cols in ((6000, 1501), (8300, 2024), (260, 33001), (130, 65552), (1000, 9001)):
        n = rows * cols
        row_of = torch.arange(n, device="cuda") // cols
        x, quiet = values_with_loud_neighbours(kind, row_of, n, cols)
        starts = torch.arange(rows, device="cuda") * cols
        ws = tcuscan.new_workspace(rows, cols, kind)
        for flags in (0, 1, 2, 3):
            src = x.clone()
            out = src if how == "in place" else torch.full((n,), -99, dtype=torch.int32 if kind in ("i32", "i8") else torch.float32, device="cuda")
            tcuscan.set_chain_policy(1 if how == "tickets" else 0)
            try:
                if how == "static":
                    tcuscan.scan_static(src, out, rows, cols, kind, flags=flags)
                else:
                    tcuscan.scan(src, out, rows, cols, kind, flags=flags, ws=ws)
            finally:
                tcuscan.set_chain_policy(0)
            assert agree(out, row_sums(x, quiet, starts, row_of, flags), quiet), (rows, cols, flags)
        assert ws is None or tcuscan.workspace_fault(ws) == 0


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("rows", [300, 5000])
def test_segmented_rows_from_lines(kind, rows):
    """Long rows of different lengths, prepared in one launch (few rows) and in three, outputs that start inside a line,
    inputs that fit them and one that does not, elements in front of the first row and behind the last, loud neighbours."""
    segmented_rows_from_lines(kind, rows, 45_000_000)


@pytest.mark.parametrize("kind,rows", [("i32", 300), ("f32", 300), ("f32", 4000), ("i32", 4500)])
def test_segmented_rows_from_lines_in_tiles_of_their_own(kind, rows):
    """The same from where 32-bit rows have tiles of their own: rows of 2^14 elements and more, or fewer than 4096 of them."""
    segmented_rows_from_lines(kind, rows, 80_000_000)


def segmented_rows_from_lines(kind, rows, about):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(rows)
    lengths = torch.randint(0, 2 * (about // rows), (rows,), generator=g, device="cuda")
    lengths[::17] = 0
    off = torch.cat([lengths.new_tensor([37]), 37 + torch.cumsum(lengths, 0)])
    n, total = int(lengths.sum().item()), int(off[-1].item()) + 91
    assert n > 1 << 23
    row_of = torch.repeat_interleave(torch.arange(rows, device="cuda"), lengths)
    x, quiet = values_with_loud_neighbours(kind, row_of, n, 7)
    starts = off[:-1] - 37
    for shift_in, shift_out in ((0, 0), (1, 1), (16, 16), (0, 4), (0, 1)):
        src = torch.full((total + shift_in,), 99, device="cuda").to(x.dtype)[shift_in:]
        src[37:37 + n] = x
        for flags in (0, 1, 2, 3) if shift_out == 4 else (shift_out & 3,):
            buf = torch.full((total + shift_out + 40,), -99, dtype=torch.int32 if kind in ("i32", "i8") else torch.float32, device="cuda")
            out = buf[shift_out:shift_out + total]
            ws = tcuscan.new_segmented_workspace(rows, total, kind)
            tcuscan.segmented(src, out, off, rows, total, kind, flags=flags, ws=ws)
            assert tcuscan.workspace_fault(ws) == 0
            assert agree(out[37:37 + n], row_sums(x, quiet, starts, row_of, flags), quiet), (shift_in, shift_out, flags)
            assert bool((buf[:shift_out + 37] == -99).all()) and bool((buf[shift_out + 37 + n:] == -99).all())
