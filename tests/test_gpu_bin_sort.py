"""Sorts whose workgroups put their keys in order by one partition into bins: sizes around the first and last rows per lane that have it,
bins as full as they may be and one key fuller, keys that differ in few bits, and keys that crowd, against numpy's stable sort."""
import numpy as np
import pytest

from paper_2411_17887_amd import inputs
from test_gpu_digit_sort import check

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
