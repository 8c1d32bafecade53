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
