"""Sorts at the edges between the forms that a bucket or a whole sort may take, against numpy's stable sort."""
import numpy as np
import pytest

from paper_2411_17887_amd import inputs
from test_gpu_digit_sort import check

pytestmark = pytest.mark.gpu


def keys_of_buckets(sizes, bits, seed, low=None):
    """Shuffled keys of `bits` bits, sizes[b] of them in the bucket b that their top log2(len(sizes)) bits name; low(bucket, count, rng): their other bits."""
    rng = np.random.default_rng(seed)
    below = bits - (len(sizes) - 1).bit_length()
    top = np.repeat(np.arange(len(sizes), dtype=np.uint32), sizes)
    if low is None:
        rest = rng.integers(0, 1 << below, top.size, dtype=np.uint32)
    else:
        rest = np.concatenate([low(b, int(s), rng) for b, s in enumerate(sizes)]).astype(np.uint32)
    k = top << np.uint32(below) | rest
    rng.shuffle(k)
    return k


@pytest.mark.parametrize("mean", [18_000, 18_001, 18_500, 20_480, 20_481])
def test_pairs_in_buckets_of_19_and_20_rows(mean):
    """Means at which these buckets get a kernel of their own, and one key fewer and more; buckets of 17,000 to 20,480 keys, crowded ones among them."""
    n = 256 * mean + (255 if mean in (18_000, 20_480) else 0)
    sizes = np.full(256, mean)
    sizes[:128] += np.arange(128) * 7 % 1000
    sizes[128:] -= np.arange(128) * 7 % 1000
    sizes[-1] += n - sizes.sum()
    def low(b, count, rng):
        return rng.integers(0, 1 << 24, count) if b % 3 else np.abs(rng.standard_normal(count)).astype(np.float32).view(np.uint32) >> 8
    check(keys_of_buckets(sizes, 32, mean, low), True, 32)
