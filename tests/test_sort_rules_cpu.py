"""Rules by which a sort takes one form or another, from the sources themselves and from what a call enqueues (no GPU)."""
import numpy as np
import pytest

import large_sort_model as model
from test_launches_cpu import VALS, VALS_TMP, run, sort    # noqa: F401  (run: a fixture)


@pytest.mark.parametrize("bits", [1, 10, 11, 12, 14, 16, 20, 31, 32])
def test_more_keys_than_values_are_not_sorted_by_bins(bits):
    """Bins of more than one key on average lose to the two passes that so few bits take."""
    for n in (1, 2, 2049, 2500, 4096, 4097, 7812, 13_671, 16_384, 20_480):
        assert model.shim().shim_bins_suffice(n, bits) == (n <= 1 << bits), (n, bits)


@pytest.mark.parametrize("n,large", [(256 * 18_000 + 255, False), (256 * 18_001, True), (256 * 20_480 + 255, True), (256 * 20_481, False)])
def test_which_pairs_have_the_kernel_with_20_rows(run, n, large):    # noqa: F811
    """Buckets of 18,433 to 20,480 pairs, on more bits than two passes sort."""
    widths = (17, 24, 25, 32)
    v = dict(vals=VALS, vals_tmp=VALS_TMP)
    got = run([sort(n, bits, **v) for bits in widths] + [sort(n, bits) for bits in widths])
    names = [[k.kernel.split("<")[0] for k in launched if k.kernel.startswith("block_sort")] for rc, launched in got]
    assert names[:4] == [["block_sort_pairs20_kernel" if large and bits > 24 else "block_sort_kernel"] for bits in widths]
    assert names[4:] == [["block_sort_kernel"]] * 4


FEW, MOST = 3 << 23, 4700 << 14


def test_which_sorts_have_two_passes_and_small_buckets():
    for n in (FEW - 1, FEW, (4701 << 13) - 1, 4701 << 13, MOST, MOST + 1):
        for bits in range(1, 33):
            log = 13 if n >> 13 <= 4700 else 14
            assert model.shim().shim_large_wanted(n, bits) == (FEW <= n <= MOST and bits >= 25 and bits >= log + 12), (n, bits)


@pytest.mark.parametrize("pairs", [False, True])
def test_scratch_of_large_sorts_fits_the_words_it_is_given(pairs):
    """Its parts follow each other on 16-byte boundaries, hold what the kernels put there, and end inside n words, three of which a scratch off such a boundary loses."""
    for n in [FEW, FEW + 1, (4701 << 13) - 1, 4701 << 13, MOST - 1, MOST] + [int(x) for x in np.linspace(FEW, MOST, 97)]:
        p = model.plan(n, pairs)
        buckets, tiles, ranges = 1 << p.log, -(-n // 16384), 1 << (p.log - p.low)
        assert p.found >= 8 * 4 * 256 + 4 and all(at % 4 == 0 for at in (p.found, p.counts, p.ranges, p.huge, p.status))
        assert p.counts - p.found >= 8 + 256 + 2 * 16384 and p.ranges - p.counts >= 8 * buckets and p.huge - p.ranges >= 4 * p.most_tiles
        assert p.status - p.huge >= p.huge_tiles and p.end - p.status >= 4 * 256 * max(tiles, p.most_tiles) and p.end + 3 <= n
        # the second pass has a tile more per range at most; every tile of a huge bucket reads more than 10,240 keys
        assert p.most_tiles >= tiles + ranges and p.huge_tiles * 10_240 >= 1.1 * 1024 * p.huge_work
        assert p.low <= 8 and p.log - p.low <= 8 and (32 - p.log + 1) // 2 <= 10
        # evenly spread keys: what the fullest bucket, the fullest 256th and the count of buckets with keys are expected to be, with room
        even = 8192 / buckets
        assert p.some_most >= even + 8 and p.wide_most >= 32 + 5 * 32 ** 0.5 and p.few_most <= 0.95 * buckets * (1 - np.exp(-2048 / buckets))


@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("share", [0.0, 0.0002, 0.001, 0.003])
def test_a_value_many_times_over_does_not_cost_the_buckets(pairs, share):
    """One value in up to three of a thousand places: its bucket alone is sorted otherwise."""
    n = FEW + 4567
    rng = np.random.default_rng(int(share * 1e4))
    k = rng.integers(0, 1 << 32, n, dtype=np.uint32)
    k[rng.random(n) < share] = 123456789
    got = model.found(k, 32, pairs)
    assert got["tried"] == 1 and got["split"] == 1 and (got["huge"] > 0) == (share > 0.0003)


def test_keys_that_crowd_take_four_passes():
    n = FEW + 99
    rng = np.random.default_rng(1)
    r = rng.integers(0, 1 << 32, n, dtype=np.uint32)
    for k in (rng.standard_normal(n).astype(np.float32).view(np.uint32), np.full(n, 7, np.uint32), r & np.uint32(0xFFFF), r & np.uint32(0xFF800000), r >> np.uint32(3),
              np.where(rng.random(n) < 0.05, np.uint32(5), r)):
        assert model.found(k, 32, False)["tried"] == 0
