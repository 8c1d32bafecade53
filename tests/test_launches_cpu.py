"""The host side of a call: which kernels it enqueues, for which arguments (no GPU: see launch_recorder.py)."""
import pytest

import launch_recorder
from paper_2411_17887_amd import tcuscan

KEYS, TMP, VALS, VALS_TMP, FLAGS, POS, WS = (0x10000 + (i << 36) for i in range(7))
WS_BYTES = 1 << 40


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    shim = launch_recorder.build(tmp_path_factory.mktemp("shim"))
    return lambda calls: launch_recorder.launches(shim, calls)


def sort(n, bits, vals=0, vals_tmp=0, ws=WS):
    return ("tcuscan_split_radix_sort_u32", [KEYS, vals, n, bits, TMP, vals_tmp, FLAGS, POS, ws, WS_BYTES if ws else 0, 0])


@pytest.mark.parametrize("form", [0, 1, 2])
def test_keys_alone_take_the_same_kernels_with_a_scratch_for_payloads(run, form):
    """d_vals_tmp without d_vals is accepted and not used: no kernel that moves payloads is launched."""
    sizes = [(n, bits) for n in (200, 5000, 9000, 16384, 16385, 100_003, 1_000_000, 1 << 22, 6_050_000, 7_000_000, 1 << 30) for bits in (7, 8, 16, 24, 25, 32)]
    got = run([("tcuscan_set_sort_fusion", [form])] + [sort(n, bits, vals_tmp=tmp) for n, bits in sizes for tmp in (0, VALS_TMP)])[1:]
    for at, (n, bits) in enumerate(sizes):
        alone, with_tmp = got[2 * at: 2 * at + 2]
        assert alone[0] == 0 and alone[1], (n, bits)
        assert with_tmp == alone, (n, bits)


@pytest.mark.parametrize("pairs", [False, True])
def test_launches_of_small_sorts(run, pairs):
    """Up to 8192 keys one launch; up to 16384 two, for more than eight bits, also with tickets and without a workspace."""
    v = dict(vals=VALS, vals_tmp=VALS_TMP) if pairs else {}
    arg = "true" if pairs else "false"
    sizes = [(n, bits) for n in (2, 8192, 8193, 12_289, 16_384) for bits in (8, 9, 32)]
    others = [("tcuscan_set_chain_policy", [1]), sort(9000, 32, **v)] + ([] if pairs else [sort(9000, 32, ws=0)])      # (pairs need one)
    got = run([sort(n, bits, **v) for n, bits in sizes] + others)
    for (n, bits), (rc, launched) in zip(sizes, got):
        one = n <= 8192 or bits == 8
        assert rc == 0 and [(k.kernel, k.grid) for k in launched] == ([] if one else [(f"spread_kernel<{arg}>", -(-n // 4096))]) + [(f"block_sort_kernel<{arg}>", 1 if one else 256)]
    for rc, launched in got[len(sizes) + 1:]:
        assert rc == 0 and [k.kernel for k in launched] == [f"spread_kernel<{arg}>", f"block_sort_kernel<{arg}>"]


@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("policy", [0, 1])                # 1: tiles by ticket
def test_launches_of_sorts_with_buckets(run, pairs, policy):
    """The second pass and the buckets in one launch of 256 workgroups, as long as its tiles are no more than that."""
    v = dict(vals=VALS, vals_tmp=VALS_TMP) if pairs else {}
    sizes = [(n, bits) for n in (16_385, 1 << 19, (1 << 19) + 1, 1 << 21, (1 << 21) + 1, (1 << 22) - 1, 1 << 22, 6_055_225) for bits in (17, 24, 32)]
    got = run([("tcuscan_set_chain_policy", [policy])] + [sort(n, bits, **v) for n, bits in sizes])[1:]
    for (n, bits), (rc, launched) in zip(sizes, got):
        rows = 4 if n <= 1 << 19 else 8 if n < 5 << 20 else 16
        later = rows if n < 1 << 22 else 16
        later_tiles = -(-n // (1024 * later))
        launched = [k for k in launched if "fill_zero" not in k.kernel]
        passes = 1 + -(-(bits - 8) // 8)
        second = [("pass_or_buckets_kernel", 256)] if n <= 1 << 21 else [("block_sort_kernel", 256), ("digit_pass_kernel", later_tiles)]
        want = [("digit_pass_kernel", -(-n // (1024 * rows)))] + second + [("digit_pass_kernel", later_tiles)] * (passes - 2)
        assert rc == 0 and launched[0].kernel.startswith("digit_histograms_kernel"), (n, bits)
        assert [(k.kernel.split("<")[0], k.grid) for k in launched[1:]] == want, (n, bits)
        assert n > 1 << 21 or later_tiles <= 256, (n, bits)


def test_compactions_whose_masks_are_counted_ahead(run):
    """Tiles may then be stored before tiles in front of them are read: not where the output or the count lies in the values or the mask."""
    n, count = 1 << 25, POS
    values, mask, out = KEYS + (1 << 32), FLAGS, TMP

    def call(values=values, mask=mask, out=out, n=n, positions=0, count=count):
        return ("tcuscan_compact_u32", [values, mask, out, n, positions, count, WS, WS_BYTES, 0])
    cases = [(call(), True), (call(n=n - 1), False), (call(positions=VALS), False), (call(count=0), True),
             (call(mask=mask + 16), True), (call(mask=mask + 1), False), (call(values=values + 4, out=out + 4), True),
             (call(out=values), False), (call(out=values + 4 * n), True), (call(out=values + 4 * n - 4), False),
             (call(out=values - 4 * n), True), (call(out=values - 4 * n + 4), False), (call(out=mask), False), (call(out=mask - 4 * n), True),
             (call(out=mask + n - 4), False), (call(out=mask + n), True), (call(out=mask - 4 * n + 4), False),
             (call(count=values), False), (call(count=values + 4 * n - 4), False), (call(count=values + 4 * n), True), (call(count=values - 4), True),
             (call(count=mask + 8), False), (call(count=mask + n), True), (call(count=out), True)]
    for at, ((_, ahead), (rc, launched)) in enumerate(zip(cases, run([c for c, _ in cases]))):
        name = launched[-1].kernel
        assert rc == 0 and name.startswith("compact_kernel<"), (at, launched)
        assert (name.split(", ")[-1] == "true>") == ahead, (at, name)


IN, OUT, OFFSETS = KEYS, TMP, VALS
KINDS = ("i32", "f16", "i8", "f32", "bf16")


def segmented(kind, total, rows, flags=0, ws=WS, d_in=IN, d_out=OUT):
    return ("tcuscan_segmented", [d_in, d_out, OFFSETS, rows, total, tcuscan.DTYPES[kind], flags, ws, WS_BYTES, 0])


@pytest.mark.parametrize("kind", KINDS)
def test_few_long_rows_of_a_small_call_have_small_tiles(run, kind):
    """Up to 2^22 elements, also where the layout counts large tiles: status words then share slots, and stay inside them."""
    shapes = [(1 << 19, 1), (600_000, 1), (1_048_575, 1), (1_048_577, 2), (2_400_000, 4), (4_000_000, 7), (1 << 22, 1), (1 << 22, 8), (300_000, 3)]
    strides = set()
    for (total, rows), (rc, launched) in zip(shapes, run([segmented(kind, total, rows) for total, rows in shapes])):
        assert rc == 0 and len(launched) == 1 and launched[0].kernel.startswith("seg_flat"), (total, rows, launched)
        tiles = total // 8192 + 2
        own_tile = 8192 if total // rows < 1 << 19 else tcuscan.large_tile_elems(kind)
        slots = total // own_tile + 2 * rows + 1
        assert launched[0].grid == tiles and (8 * tiles << launched[0].stride) <= 64 * slots, (total, rows, launched)
        assert launched[0].stride == 3 or (16 * tiles << launched[0].stride) > 64 * slots
        strides.add(launched[0].stride)
    assert len(strides) >= 2


def test_which_rows_of_large_calls_keep_tiles_of_their_own(run):
    """32-bit rows, 256 to 4095 of them or long ones, from 9 x 2^22 elements on (f32 rows of 2^16 and more: 3 x 2^24)."""
    M = 1 << 20
    shapes = [("i32", 36 * M, 36 * M // 12_000, True), ("i32", 36 * M - 1, 36 * M // 12_000, False), ("f32", 36 * M, 36 * M // 12_000, True), ("i32", 64 * M, 4096, True),
              ("i32", 64 * M - 4096, 4096, False), ("i32", 60 * M, 4096, False), ("f32", 60 * M, 4095, True), ("f32", 128 * M, 8192, True), ("f32", 40 * M, 255, False),
              ("i32", 40 * M, 256, True), ("f32", 40 * M, 256, False), ("f32", 40 * M, 641, True), ("f32", 48 * M, 256, True), ("bf16", 128 * M, 2000, False), ("i8", 128 * M, 2000, False)]
    for (kind, total, rows, own), (rc, launched) in zip(shapes, run([segmented(kind, total, rows) for kind, total, rows, _ in shapes])):
        last = launched[-1].kernel
        assert rc == 0 and last.startswith("scan_kernel<" if own else "seg_stream_kernel<"), (kind, total, rows, launched)


@pytest.mark.parametrize("kind", KINDS)
def test_a_workspace_with_first_rows_in_it_is_cleared(run, kind):
    """A large call of short rows leaves first rows where others expect status words: the next call of another kind on that workspace
    clears its own, and the call after that need not."""
    n = 14_000_000
    two = segmented(kind, n, n // 200)
    plain = ("tcuscan_scan", [IN, OUT, 1, n, tcuscan.DTYPES[kind], 0, WS, WS_BYTES, 0])
    one = segmented(kind, n, n // 20_000)
    other = segmented(kind, n, n // 20_000, ws=WS + (1 << 30))
    for after in (plain, one):
        got = [[k.kernel.split("<")[0] for k in launched] for rc, launched in run([after, two, after, after, two, other, after])]
        alone = got[0]
        assert len(alone) == 1
        assert got[1] == ["seg_first_rows_kernel", "seg_stream_kernel"] == got[4]
        assert got[2] == ["fill_zero_kernel"] + alone and got[3] == alone
        assert got[6] == ["fill_zero_kernel"] + alone
