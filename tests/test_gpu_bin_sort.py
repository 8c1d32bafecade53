"""Sorts whose workgroups put their keys in order by one partition into bins: sizes around the first and last rows per lane that have it,
bins as full as they may be and one key fuller, keys that differ in few bits, and keys that crowd, against numpy's stable sort."""
import numpy as np
import pytest

from paper_2411_17887_amd import inputs
from test_gpu_digit_sort import check
from test_gpu_sort_forms import check_large

pytestmark = pytest.mark.gpu


def spread(n, seed):
    """n keys that differ in all 32 bits, evenly spread and shuffled: no two share a bin."""
    k = (np.arange(n, dtype=np.uint64) * np.uint64((1 << 32) // n)).astype(np.uint32)
    k[-1] |= np.uint32(0x80000000)
    np.random.default_rng(seed).shuffle(k)
    return k


@pytest.mark.parametrize("pairs", [False, True], ids=["keys", "pairs"])
@pytest.mark.parametrize("n", [2047, 2048, 2049, 2050, 3071, 3073, 4097, 5000, 8191, 8192])
def test_one_workgroup(n, pairs):
    check(inputs.int32_full(n, n).view(np.uint32), pairs, 32)
    check(spread(n, n), pairs, 32)


@pytest.mark.parametrize("bits", [11, 12, 13, 14, 20, 31])
@pytest.mark.parametrize("n", [2049, 8192])
def test_few_bits_and_equal_keys_stay_in_order(n, bits):
    check(inputs.int32_full(n, bits).view(np.uint32), True, bits)


@pytest.mark.parametrize("full", [2, 4, 5, 15, 16, 17, 300])
@pytest.mark.parametrize("n", [3000, 8192])
def test_bins_up_to_their_limit_and_beyond(n, full):
    """Some bins hold `full` keys, that differ below the bin's bits or are equal: 16 are sorted there, 17 go by passes."""
    k = spread(n, full)
    rng = np.random.default_rng(n + full)
    for group in range(3):
        at = rng.permutation(n)[:full]
        k[at] = (np.uint32(0x12345678 + (group << 29)) & np.uint32(0xFFFFF000)) | (rng.integers(0, 4, full).astype(np.uint32) * np.uint32(group))
    check(k, True, 32)


@pytest.mark.parametrize("mask", [0xFFFF0000, 0x00FFFF00, 0xF0F0F0F0, 0x80000001, 0xFF000000, 0x00000000, 0x0000FFFF])
@pytest.mark.parametrize("n", [2500, 8000, 200_000])
def test_bits_that_never_differ(n, mask):
    """Bins by the highest bit that differs; passes that leave out digits in which no key differs from another."""
    k = inputs.int32_full(n, n).view(np.uint32)
    check(k & np.uint32(mask), True, 32)
    check(k & np.uint32(mask) | np.uint32(0x05A0A050 & ~mask), True, 32)


@pytest.mark.parametrize("n", [2049, 5000, 16_000, 400_000])
def test_crowded_and_ordered_keys(n):
    rng = np.random.default_rng(n)
    normal = rng.standard_normal(n).astype(np.float32).view(np.uint32)
    ramp = np.arange(n, dtype=np.uint32)
    few = rng.integers(0, 2, n).astype(np.uint32) * np.uint32(0x40000001)
    one_other = np.full(n, 9, np.uint32)
    one_other[n // 2] = 0xFFFFFFFF
    for k in (normal, ramp, ramp[::-1].copy(), np.sort(inputs.int32_full(n, 3).view(np.uint32)), few, one_other):
        check(k, True, 32)


@pytest.mark.parametrize("bits", [32, 24, 18])
def test_buckets_of_every_size_that_has_bins(bits):
    """Buckets of the top digit from 2000 to 20,500 keys: all row counts with bins, fillers in the last rows, and the first without."""
    rng = np.random.default_rng(bits)
    sizes = 2000 + np.arange(256) * 73 % 18_600
    top = np.repeat(np.arange(256, dtype=np.uint32), sizes)
    rng.shuffle(top)
    low = rng.integers(0, 1 << (bits - 8), top.size, dtype=np.uint32)
    check(top << np.uint32(bits - 8) | low, True, bits)
    check(top << np.uint32(bits - 8) | low, False, bits)


LARGE = 3 << 23                                          # the first size with two passes and small buckets; up to 4700 << 14 keys


@pytest.mark.parametrize("pairs", [False, True], ids=["keys", "pairs"])
@pytest.mark.parametrize("n", [LARGE - 1, LARGE, (4701 << 13) - 1, 4701 << 13])         # 2^13, 2^14 buckets
def test_two_passes_and_small_buckets(n, pairs):
    check(inputs.int32_full(n, n).view(np.uint32), pairs, 32)


@pytest.mark.parametrize("bits", [24, 25, 26, 28, 31])
def test_widths_of_large_sorts(bits):
    check(inputs.int32_full(LARGE, bits).view(np.uint32), bits % 2 == 0, bits)


def large_keys(name, n):
    r, i = inputs.int32_full(n, 17).view(np.uint32), np.arange(n, dtype=np.uint32)
    share = lambda parts: i % np.uint32(parts) == 0
    return {
        "two_thirds_of_the_range": (r.astype(np.uint64) * 2 // 3).astype(np.uint32),
        "five_eighths_empty": r % np.uint32(3 << 29),                                   # buckets of 5800 to 9600 keys: the sample says no
        "lower_half_of_the_range": r >> np.uint32(1),                                   # buckets of 5800 to 6500 keys, for eight wavefronts
        "equal_in_buckets": r & np.uint32(0xFFFF0000),                                  # many equal keys in every bucket
        "few_bits_in_buckets": r & np.uint32(0xFFE000FF),                               # 2048 buckets of some 12,300 keys: the sample says no
        "few_bits_in_every_bucket": r & np.uint32(0xFFF800FF),
        "crowded": np.random.default_rng(3).standard_normal(n).astype(np.float32).view(np.uint32),
        "equal": np.full(n, 7, np.uint32),
        "in_order": np.sort(r),
        "one_bucket_of_10240": np.where(i < 10240, r & np.uint32(0x7FFFF), r | np.uint32(1 << 19)),       # what the larger workgroups hold
        "one_bucket_of_10241": np.where(i < 10241, r & np.uint32(0x7FFFF), r | np.uint32(1 << 19)),       # and more, which no sample sees
        "one_bucket_of_20000": np.where(i < 20000, r & np.uint32(0x7FFFF), r | np.uint32(1 << 19)),
        "every_thousandth_equal": np.where(share(1000), np.uint32(5), r),
        "every_tenth_equal": np.where(share(10), np.uint32(5), r),
    }[name].astype(np.uint32)


HALF = 1 << 12                                           # of the buckets


@pytest.mark.parametrize("name,split,large,huge", [
    ("two_thirds_of_the_range", 1, 0, 0), ("five_eighths_empty", 0, 0, 0), ("lower_half_of_the_range", 1, HALF, 0), ("equal_in_buckets", 1, 0, 0),
    ("few_bits_in_buckets", 0, 0, 0), ("few_bits_in_every_bucket", 1, 0, 0), ("crowded", 0, 0, 0), ("equal", 0, 0, 0), ("in_order", 1, 0, 0),
    ("one_bucket_of_10240", 1, HALF + 1, 0), ("one_bucket_of_10241", 1, HALF, 2), ("one_bucket_of_20000", 1, HALF, 3), ("every_thousandth_equal", 1, 0, 4),
    ("every_tenth_equal", 0, 0, 0)])
def test_large_sorts_of_keys_that_split_unevenly(name, split, large, huge):
    """The order, and the way it was come by: buckets or four passes, buckets for eight wavefronts, tiles of larger ones."""
    got = check_large(large_keys(name, LARGE + 77_777), True, 32)
    assert (got["split"], got["large"], got["huge"]) == (split, large, huge)


def test_large_sorts_by_ticket_and_in_a_graph():
    import torch
    from paper_2411_17887_amd import tcuscan
    n = LARGE + 99_999
    tcuscan.set_chain_policy(1)
    try:
        check(inputs.int32_full(n, 1).view(np.uint32), True, 32)
        check(large_keys("crowded", n), True, 32)
    finally:
        tcuscan.set_chain_policy(0)
    k = torch.from_numpy(inputs.int32_full(n, 7)).cuda()
    keys, tmp, pos = torch.empty_like(k), torch.empty_like(k), torch.empty_like(k)
    flags, ws = torch.empty(n, dtype=torch.int8, device="cuda"), tcuscan.new_workspace(1, n, "i8")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        keys.copy_(k)
        tcuscan.split_radix_sort_u32(keys, tmp, flags, pos, ws=ws)
    for new in (inputs.int32_full(n, 8), np.full(n, 5, np.int32), large_keys("one_bucket_of_20000", n).view(np.int32), inputs.int32_full(n, 9)):
        k.copy_(torch.from_numpy(new))
        torch.cuda.synchronize()
        pos.fill_(-1)                                                     # eager work on the scratch between the replays
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(keys.cpu().numpy().view(np.uint32), np.sort(new.view(np.uint32)))


@pytest.mark.parametrize("name", ["random", "crowded"])
def test_a_tile_of_a_large_sort_that_does_not_know_its_places_is_not_stored(name):
    """Tile 3 of every pass keeps silent: all kernels end, nothing is written outside the arrays, the fault word reads 1, and the same call sorts again."""
    import torch
    from paper_2411_17887_amd import tcuscan
    n = LARGE + 99_999
    k = inputs.int32_full(n, 2).view(np.uint32) if name == "random" else large_keys(name, n)
    room = (n + 3) // 4 * 4 + 128
    buf = torch.full((5, room), -7, dtype=torch.int32, device="cuda")
    d_k, d_kt, d_v, d_vt, d_p = (buf[i, 64:64 + n] for i in range(5))
    d_f, ws = torch.empty(n, dtype=torch.int8, device="cuda"), tcuscan.new_workspace(1, n, "i8")
    order = np.argsort(k, kind="stable")
    for silent in (True, False):
        d_k.copy_(torch.from_numpy(k.view(np.int32)))
        d_v.copy_(torch.arange(n, dtype=torch.int32))
        if silent:
            tcuscan.test_chain_fault(4096, 3)
        try:
            tcuscan.split_radix_sort_u32(d_k, d_kt, d_f, d_p, vals=d_v, vals_tmp=d_vt, ws=ws)
            torch.cuda.synchronize()
        finally:
            tcuscan.test_chain_fault(0, -1)
        assert tcuscan.workspace_fault(ws) == (1 if silent else 0)
        for b in buf:
            assert bool((b[:64] == -7).all()) and bool((b[64 + n:] == -7).all())
        tcuscan.workspace_init(ws)
    assert np.array_equal(d_k.cpu().numpy().view(np.uint32), k[order]) and np.array_equal(d_v.cpu().numpy(), order.astype(np.int32))
