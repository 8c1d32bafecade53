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


LARGE = 3 << 23                                          # the first size with two passes and small buckets


def check_large(k, pairs, bits, off=0):
    """Sorts k, looks the result up in numpy's stable sort, and what the kernels have found out (the first words of the scratch) in the model; returns the latter.
    `off`: bytes that the scratch begins after a 16-byte boundary."""
    import torch
    from paper_2411_17887_amd import tcuscan
    import large_sort_model as model
    n = k.size
    d_k = torch.from_numpy(k.view(np.int32)).cuda()
    d_v = torch.arange(n, dtype=torch.int32, device="cuda") if pairs else None
    buf = torch.full((4, (n + 3) // 4 * 4 + 128), -7, dtype=torch.int32, device="cuda")
    d_kt, d_vt, d_p = buf[0, 64:64 + n], buf[1, 64:64 + n], buf[2, 64 + off // 4:64 + off // 4 + n]
    d_f, ws = torch.empty(n, dtype=torch.int8, device="cuda"), tcuscan.new_workspace(1, n, "i8")
    tcuscan.split_radix_sort_u32(d_k, d_kt, d_f, d_p, vals=d_v, vals_tmp=d_vt if pairs else None, bits=bits, ws=ws)
    torch.cuda.synchronize()
    assert tcuscan.workspace_fault(ws) == 0
    for b, at in ((buf[0], 64), (buf[1], 64), (buf[2], 64 + off // 4)):
        assert bool((b[:at] == -7).all()) and bool((b[at + n:] == -7).all())
    order = np.argsort(k & np.uint32((1 << bits) - 1), kind="stable")
    assert np.array_equal(d_k.cpu().numpy().view(np.uint32), k[order])
    assert not pairs or np.array_equal(d_v.cpu().numpy(), order.astype(np.int32))
    begin = model.plan(n, pairs).found + (-(off // 4)) % 4                          # (the scratch is used from a 16-byte boundary on)
    got = dict(zip(("split", "tried", "large", "huge", "work"), d_p[begin:begin + 5].tolist()))
    want = model.found(k, bits, pairs)
    assert got == want
    return got


def bucket_sizes(n, mean_of, sizes):
    """2^13 sizes that add up to n: `sizes` for some buckets of every 256th, the same for the others."""
    s = np.zeros(1 << 13, np.int64)
    at = np.arange(1 << 13).reshape(256, 32)[:, :mean_of].reshape(-1)[:len(sizes)]
    s[at] = sizes
    rest = np.setdiff1d(np.arange(1 << 13), at)
    left = n - s.sum()
    s[rest] = left // rest.size
    s[rest[:left - s.sum() + s[at].sum()]] += 1
    assert s.sum() == n and s.min() >= 0
    return s


@pytest.mark.parametrize("kind", ["random", "few_low_bits", "crowded", "equal"])
@pytest.mark.parametrize("pairs", [False, True], ids=["keys", "pairs"])
def test_buckets_for_every_row_count_of_both_kernels(pairs, kind):
    """2000 to 5120 keys for four wavefronts, 5121 to 10,240 for eight, by bins and by passes, all in one sort and in the sample's favour."""
    n = LARGE + 4321
    small = np.repeat([2000, 2048, 2049, 2560, 2561, 3072, 3073, 3584, 3585, 4096, 4097, 4608, 4609, 5119, 5120], 16)
    large = np.repeat([5121, 6144, 6145, 7168, 7169, 8192, 8193, 9216, 9217, 10239, 10240], 12)
    sizes = np.concatenate([small, large])
    np.random.default_rng(5).shuffle(sizes)
    s = bucket_sizes(n, 2, sizes)
    def low(b, count, rng):
        if kind == "random" or b % 32 >= 2:
            return rng.integers(0, 1 << 19, count)
        if kind == "few_low_bits":
            return rng.integers(0, 1 << 6, count) << 9 | 5
        if kind == "crowded":
            return (np.abs(rng.standard_normal(count)).astype(np.float32).view(np.uint32) >> 13) & 0x7FFFF
        return np.full(count, b & 0x7FFFF)
    got = check_large(keys_of_buckets(s, 32, 7, low), pairs, 32)
    assert got["split"] == 1 and got["large"] == len(large) and got["huge"] == 0


@pytest.mark.parametrize("pairs", [False, True], ids=["keys", "pairs"])
@pytest.mark.parametrize("bits", [25, 32])
def test_buckets_of_more_keys_than_a_workgroup_sorts(pairs, bits):
    """10,241 keys to 2^18, tiles full and with one key, random and of one value."""
    n = LARGE + 7
    sizes = np.array([10_241, 16_383, 16_384, 16_385, 24_576, 24_577, 40_000, 65_536, 100_001, 10_240, 150_000])
    s = bucket_sizes(n, 1, sizes)
    low = lambda b, count, rng: rng.integers(0, 1 << (bits - 13), count) if b % 64 else np.where(rng.random(count) < 0.7, 77, rng.integers(0, 1 << (bits - 13), count))
    got = check_large(keys_of_buckets(s, bits, 9, low), pairs, bits)
    assert got["split"] == 1 and got["huge"] == sum(-(-x // 8192) for x in sizes if x > 10_240)


@pytest.mark.parametrize("share", [0.0002, 0.0005, 0.001, 0.004, 0.02])
@pytest.mark.parametrize("pairs", [False, True], ids=["keys", "pairs"])
def test_one_value_many_times_over(pairs, share):
    n = LARGE + 12_345
    rng = np.random.default_rng(int(1e4 * share))
    k = inputs.int32_full(n, 31).view(np.uint32).copy()
    k[rng.random(n) < share] = 0
    got = check_large(k, pairs, 32)
    assert got["split"] == (1 if share < 0.01 else 0)


@pytest.mark.parametrize("name", ["one_bucket_over_the_limit", "few_values", "too_much_work"])
def test_counts_against_the_sample(name):
    """A bucket of more than 2^18 keys, and more work in huge buckets than they are worth, that the sample may not see: four passes on digits counted after all."""
    n = LARGE + 5
    if name == "one_bucket_over_the_limit":                # (all of its keys where the sample does not look: 2048 groups of four)
        k = inputs.int32_full(n, 3).view(np.uint32).copy()
        k[:270_000] = np.where(np.arange(270_000) < 262_145 + 4000, np.uint32(9), k[:270_000])
        part = n // 4 // 2048
        g = np.arange(2048, dtype=np.uint64)
        at = (4 * (g * part + ((g * 0x9E3779B1 & 0xFFFFFFFF) >> 8) % part)[:, None] + np.arange(4, dtype=np.uint64)).reshape(-1)
        at = at[at < 270_000]
        k[at] = inputs.int32_full(at.size, 4).view(np.uint32)
        tried = 1
    elif name == "few_values":                             # 700 values: 36,000 keys and five tiles each
        k = (inputs.int32_full(n, 3).view(np.uint32) % np.uint32(700)) * np.uint32(6_135_667)
        tried = 0
    else:                                                  # 1300 values and a few others: 18,000 keys and three tiles each, and the sample sees more buckets than that
        r = inputs.int32_full(n, 3).view(np.uint32)
        k = np.where(r % np.uint32(10) < np.uint32(9), r % np.uint32(700) * np.uint32(6_135_667), r).astype(np.uint32)
        tried = None
    got = check_large(k, True, 32)
    assert got["split"] == 0 and (tried is None or got["tried"] == tried)


def test_scratch_off_a_16_byte_boundary():
    k = inputs.int32_full(LARGE + 3, 21).view(np.uint32)
    for off in (4, 8, 12):
        assert check_large(k, off == 8, 32, off)["split"] == 1


@pytest.mark.parametrize("pairs", [False, True], ids=["keys", "pairs"])
@pytest.mark.parametrize("n", [4700 << 14, (4700 << 14) + 1])
def test_most_keys_that_have_small_buckets(n, pairs):
    """The last size with them, and the first without."""
    if n == 4700 << 14:
        assert check_large(inputs.int32_full(n, 5).view(np.uint32), pairs, 32)["split"] == 1
    else:
        check(inputs.int32_full(n, 5).view(np.uint32), pairs, 32)


@pytest.mark.parametrize("name", ["half", "two_thirds", "quarter_of_the_buckets"])
def test_uneven_keys_alone(name):
    r = inputs.int32_full(LARGE + 77, 8).view(np.uint32)
    k = {"half": r >> np.uint32(1), "two_thirds": (r.astype(np.uint64) * 2 // 3).astype(np.uint32), "quarter_of_the_buckets": r & np.uint32(0xFFE7FFFF) | np.uint32(1 << 20)}[name]
    got = check_large(k, False, 32)
    assert name == "quarter_of_the_buckets" or (got["split"] == 1 and got["huge"] == 0)


@pytest.mark.parametrize("pairs", [False, True], ids=["keys", "pairs"])
def test_a_silent_tile_in_front_of_huge_buckets(pairs):
    """Tile 3 of the first two passes keeps silent, so the array has gaps: the passes over huge buckets end and write inside the arrays, and the same call sorts again."""
    import torch
    from paper_2411_17887_amd import tcuscan
    n = LARGE + 99_999
    k = inputs.int32_full(n, 2).view(np.uint32).copy()
    k[::1000] = 5
    buf = torch.full((5, (n + 3) // 4 * 4 + 128), -7, dtype=torch.int32, device="cuda")
    d_k, d_kt, d_v, d_vt, d_p = (buf[i, 64:64 + n] for i in range(5))
    d_f, ws = torch.empty(n, dtype=torch.int8, device="cuda"), tcuscan.new_workspace(1, n, "i8")
    for silent in (True, False):
        d_k.copy_(torch.from_numpy(k.view(np.int32)))
        d_v.copy_(torch.arange(n, dtype=torch.int32))
        if silent:
            tcuscan.test_chain_fault(4096, 3)
        try:
            tcuscan.split_radix_sort_u32(d_k, d_kt, d_f, d_p, vals=d_v if pairs else None, vals_tmp=d_vt if pairs else None, ws=ws)
            torch.cuda.synchronize()
        finally:
            tcuscan.test_chain_fault(0, -1)
        assert tcuscan.workspace_fault(ws) == (1 if silent else 0)
        for b in buf:
            assert bool((b[:64] == -7).all()) and bool((b[64 + n:] == -7).all())
        tcuscan.workspace_init(ws)
    order = np.argsort(k, kind="stable")
    assert np.array_equal(d_k.cpu().numpy().view(np.uint32), k[order])
    assert not pairs or np.array_equal(d_v.cpu().numpy(), order.astype(np.int32))
