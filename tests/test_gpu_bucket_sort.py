"""Sorts that split on the top digit first: sizes around the limits of the form and of a workgroup's rows per lane, keys that
split and keys that do not, with and without the workspace that small sorts need not have, against numpy's stable sort."""
import numpy as np
import pytest

from paper_2411_17887_amd import inputs, tcuscan
from test_gpu_digit_sort import check, sort_on_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs", [False, True], ids=["keys", "pairs"])
@pytest.mark.parametrize("n", [7168, 7169, 8193, 16384, 16385, 32768, 32769, (1 << 17), (1 << 17) + 1, (1 << 18) + 5, (3 << 20) - 1, 3 << 20, 4194313, 6_000_000, 6_250_000])
def test_random_keys(n, pairs):
    check(inputs.int32_full(n, n).view(np.uint32), pairs, 32)


@pytest.mark.parametrize("bits", [9, 16, 17, 20, 24, 25, 31])
@pytest.mark.parametrize("n", [9001, 16000, 40001, 300_007])
def test_widths(n, bits):
    check(inputs.int32_full(n, n + bits).view(np.uint32), True, bits)


def keys_of(name, n):
    i, r = np.arange(n, dtype=np.uint32), inputs.int32_full(n, 4).view(np.uint32)
    return {
        "equal": np.full(n, 0xFFFFFFFF, np.uint32),                       # looks like the filler behind a workgroup's last key
        "small": r & np.uint32(0xFFFF),                                   # everything in one bucket
        "half": np.where(i % 2 == 0, r, r & np.uint32(0xFFFFFF)),         # just over half the keys in one bucket
        "lanes": (i % 64) * np.uint32(0x01010101),                        # every lane of a row a digit of its own
        "pairs_of_lanes": (i % 2) * np.uint32(0x5A5A5A5A) + (r & np.uint32(1)),
        "one_bucket_over": np.where(i < 24577, r & np.uint32(0xFFFFFF), r | np.uint32(0x01000000)),      # a key more than a workgroup sorts
        "one_bucket_full": np.where(i < 24576, r & np.uint32(0xFFFFFF), r | np.uint32(0x01000000)),
    }[name]


@pytest.mark.parametrize("n", [9000, 16384, 16385, 24577, 60_000, 1_000_003])
@pytest.mark.parametrize("name", ["equal", "small", "half", "lanes", "pairs_of_lanes", "one_bucket_over", "one_bucket_full"])
def test_keys_that_split_unevenly(name, n):
    check(keys_of(name, n).astype(np.uint32), True, 32)


@pytest.mark.parametrize("n", [16_385, 20_000, 131_073, 600_000, 1_500_000, 6_055_225, 6_055_226])
@pytest.mark.parametrize("over", [0, 1])
def test_a_bucket_at_the_limit(n, over):
    """The largest bucket that a workgroup sorts, and a key more, which takes the passes; both sides of the largest sort with buckets."""
    limit = min(24_576, 6144 + n // 80)
    r = inputs.int32_full(n, n + over).view(np.uint32)
    keys = r % np.uint32(255 << 24) + np.uint32(1 << 24)
    keys[np.random.default_rng(n).permutation(n)[:limit + over]] &= np.uint32(0xFFFFFF)
    assert np.count_nonzero(keys < 1 << 24) == limit + over
    check(keys, True, 32)


@pytest.mark.parametrize("policy", [0, 1])                # 1: tiles by ticket
@pytest.mark.parametrize("name", ["small", "lanes", "random"])
@pytest.mark.parametrize("n", [16_385, 1 << 19, (1 << 19) + 1, 1 << 21, (1 << 21) + 1, (1 << 22) - 1, 1 << 22])
def test_the_second_pass_with_and_beside_the_buckets(n, name, policy):
    """Up to 2^21 keys one launch does the buckets or the second pass; tile shapes of the later passes change at 2^19 and 2^22."""
    keys = inputs.int32_full(n, n).view(np.uint32) if name == "random" else keys_of(name, n).astype(np.uint32)
    tcuscan.set_chain_policy(policy)
    try:
        check(keys, True, 32)
        check(keys, False, 24)
    finally:
        tcuscan.set_chain_policy(0)


@pytest.mark.parametrize("bits", [32, 20])
def test_buckets_of_every_size_a_workgroup_has_code_for(bits):
    """Bucket b of the top digit holds 0, 1, 63, 64, 65 or about b * 96 keys: all row counts, each with part of a row."""
    rng = np.random.default_rng(bits)
    sizes = np.arange(256) * 96 + rng.integers(0, 64, 256)
    sizes[[3, 50, 51, 52, 53]] = [0, 1, 63, 64, 65]
    top = np.repeat(np.arange(256, dtype=np.uint32), sizes)
    rng.shuffle(top)
    low = rng.integers(0, 1 << (bits - 8), top.size, dtype=np.uint32)
    check(top << np.uint32(bits - 8) | low, True, bits)


def test_without_a_workspace_where_none_is_needed():
    """9000 to 16384 keys need no workspace; without one there is no word for a wait that gives up, and one workgroup sorts."""
    import torch
    n = 16384
    k = inputs.int32_full(n, 2).view(np.uint32)
    d_k = torch.from_numpy(k.view(np.int32).copy()).cuda()
    tcuscan.split_radix_sort_u32(d_k, torch.empty_like(d_k), torch.empty(n, dtype=torch.int8, device="cuda"),
                                 torch.empty(n, dtype=torch.int32, device="cuda"), ws=None)
    assert np.array_equal(d_k.cpu().numpy().view(np.uint32), np.sort(k))


@pytest.mark.parametrize("n", [9000, 16385, 200_000])
def test_tickets_keep_to_the_scratch(n):
    tcuscan.set_chain_policy(1)
    try:
        k = inputs.int32_full(n, 6).view(np.uint32)
        got, _ = sort_on_gpu(k, False, 32)
    finally:
        tcuscan.set_chain_policy(0)
    assert np.array_equal(got, np.sort(k))


@pytest.mark.parametrize("n", [9000, 100_003])
def test_recorded_into_a_graph(n):
    import torch
    k = torch.from_numpy(inputs.int32_full(n, 7)).cuda()
    keys, tmp, pos = torch.empty_like(k), torch.empty_like(k), torch.empty_like(k)
    flags, ws = torch.empty(n, dtype=torch.int8, device="cuda"), tcuscan.new_workspace(1, n, "i8")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        keys.copy_(k)
        tcuscan.split_radix_sort_u32(keys, tmp, flags, pos, ws=ws)
    for seed in (8, 9, 10):
        new = inputs.int32_full(n, seed) if seed != 9 else np.full(n, 5, np.int32)
        k.copy_(torch.from_numpy(new))
        torch.cuda.synchronize()
        pos.fill_(-1)                                                     # eager work on the scratch between the replays
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(keys.cpu().numpy().view(np.uint32), np.sort(new.view(np.uint32)))


@pytest.mark.parametrize("bits", [24, 32])
@pytest.mark.parametrize("n", [9000, 100_003])
@pytest.mark.parametrize("form", [0, 1, 2])
def test_keys_alone_with_a_scratch_for_payloads(form, n, bits):
    """The scratch is not used, and not written."""
    import torch
    k = inputs.int32_full(n, n + bits).view(np.uint32)
    d_k = torch.from_numpy(k.view(np.int32).copy()).cuda()
    tmp = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    tcuscan.set_sort_fusion(form)
    try:
        tcuscan.split_radix_sort_u32(d_k, torch.empty_like(d_k), torch.empty(n, dtype=torch.int8, device="cuda"), torch.empty_like(d_k),
                                     vals_tmp=tmp, bits=bits, ws=tcuscan.new_workspace(1, n, "i8"))
        torch.cuda.synchronize()
    finally:
        tcuscan.set_sort_fusion(1)
    assert np.array_equal(d_k.cpu().numpy().view(np.uint32), k[np.argsort(k & np.uint32((1 << bits) - 1), kind="stable")])
    assert bool((tmp == -7).all())
