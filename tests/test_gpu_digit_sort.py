"""The sort's passes on eight bits and its one-workgroup form, at the sizes where their tiles, shapes and pass counts
change, against numpy's stable sort (bit for bit)."""
import numpy as np
import pytest

from paper_2411_17887_amd import inputs, tcuscan

pytestmark = pytest.mark.gpu


def sort_on_gpu(k, pairs, bits):
    import torch
    n = k.size
    d_k = torch.from_numpy(k.view(np.int32).copy()).cuda()
    d_v = torch.arange(n, dtype=torch.int32, device="cuda") if pairs else None
    guard = torch.full((n + 64,), -7, dtype=torch.int32, device="cuda")     # the scratch the sort may write: n words, no more
    d_f = torch.empty(max(n, 16), dtype=torch.int8, device="cuda")
    ws = tcuscan.new_workspace(1, n, "i8")
    tcuscan.split_radix_sort_u32(d_k, torch.empty_like(d_k), d_f, guard, vals=d_v,
                                 vals_tmp=None if d_v is None else torch.empty_like(d_v), bits=bits, ws=ws)
    torch.cuda.synchronize()
    assert ws is None or tcuscan.workspace_fault(ws) == 0
    assert bool((guard[n:] == -7).all())
    return d_k.cpu().numpy().view(np.uint32), None if d_v is None else d_v.cpu().numpy()


def check(k, pairs, bits):
    gk, gv = sort_on_gpu(k, pairs, bits)
    order = np.argsort(k & np.uint32((1 << bits) - 1), kind="stable")
    assert np.array_equal(gk, k[order])
    assert gv is None or np.array_equal(gv, order.astype(np.int32))


# one workgroup: 1024, 2048, 4096, 8192, 12288, 16384 keys; tiles of 4096 up to 2^19 keys, of 8192 below 5 * 2^20, of 16384 from there
@pytest.mark.parametrize("pairs", [False, True], ids=["keys", "pairs"])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 1023, 1024, 1025, 2048, 2049, 4095, 4096, 4097, 8192, 8193, 12288, 12289, 16383, 16384, 16385, 5 * 4096, 5 * 4096 + 1,
                               (1 << 19) - 1, 1 << 19, (1 << 19) + 1, 70 * 8192 - 1, (5 << 20) - 1, 5 << 20, 321 * 16384 + 1])
def test_sizes_around_tiles_and_shapes(n, pairs):
    check(inputs.int32_full(n, 3 * n + 1).view(np.uint32), pairs, 32)


@pytest.mark.parametrize("bits", [1, 3, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32])
@pytest.mark.parametrize("n", [1000, 16000, 40001, (1 << 20) + 3])
def test_digit_widths_and_pass_counts(n, bits):
    check(inputs.int32_full(n, n + bits).view(np.uint32), True, bits)


@pytest.mark.parametrize("n", [5000, 100003, (5 << 20) + 77])
def test_few_distinct_keys(n):
    i = np.arange(n, dtype=np.uint32)
    for k in (np.full(n, 0xFFFFFFFF, np.uint32), np.zeros(n, np.uint32), i % 3, i[::-1].copy(), (i % 2) * np.uint32(0xFFFFFFFF),
              np.where(i % 1000 == 0, inputs.int32_full(n, 8).view(np.uint32), np.uint32(0x80808080))):
        check(k.astype(np.uint32), True, 32)


def test_tickets():
    tcuscan.set_chain_policy(1)
    try:
        for n in (16385, 300007, (5 << 20) + 5):
            check(inputs.int32_full(n, n).view(np.uint32), True, 32)
    finally:
        tcuscan.set_chain_policy(0)


def test_a_look_back_that_gives_up_ends_and_raises_the_fault_word():
    """A poll limit of one: a tile whose predecessor has not published when it asks gives up.  Every kernel ends, nothing
    is written outside the arrays, and either the fault word says so or the result is right."""
    import torch
    n = 300 * 4096 + 11
    k = inputs.int32_full(n, 6).view(np.uint32)
    buf = torch.full((2, (n + 3) // 4 * 4 + 128), -7, dtype=torch.int32, device="cuda")      # rows start at 16-byte boundaries
    d_k, d_kt = buf[0, 64:64 + n], buf[1, 64:64 + n]
    d_k.copy_(torch.from_numpy(k.view(np.int32)))
    d_f, d_p = torch.empty(n, dtype=torch.int8, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
    ws = tcuscan.new_workspace(1, n, "i8")
    tcuscan.test_chain_fault(1, -1)
    try:
        tcuscan.split_radix_sort_u32(d_k, d_kt, d_f, d_p, bits=32, ws=ws)
        torch.cuda.synchronize()
    finally:
        tcuscan.test_chain_fault(0, -1)
    for b in (buf[0], buf[1]):
        assert bool((b[:64] == -7).all()) and bool((b[64 + n:] == -7).all())
    if tcuscan.workspace_fault(ws) == 0:
        assert np.array_equal(d_k.cpu().numpy().view(np.uint32), np.sort(k))


def test_more_than_2_to_30_keys():
    """Status words and byte offsets of 64 bits from 2^30 keys on."""
    import torch
    n = (1 << 30) + 12345
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    d_k = torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    sums = int(d_k.to(torch.int64).sum().item()), int((d_k.to(torch.int64) ** 2 % 1000003).sum().item())
    d_f, d_p = torch.empty(n, dtype=torch.int8, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
    ws = tcuscan.new_workspace(1, n, "i8")
    tcuscan.split_radix_sort_u32(d_k, torch.empty_like(d_k), d_f, d_p, bits=32, ws=ws)
    torch.cuda.synchronize()
    assert tcuscan.workspace_fault(ws) == 0
    u = d_k.to(torch.int64) & 0xFFFFFFFF
    assert bool((u[1:] >= u[:-1]).all())
    del u
    assert (int(d_k.to(torch.int64).sum().item()), int((d_k.to(torch.int64) ** 2 % 1000003).sum().item())) == sums


@pytest.mark.parametrize("tickets", [0, 1])
def test_payloads_from_2_to_30_keys_on(tickets):
    """The 64-bit form with payloads: every payload is the index of its key, so keys and payloads together say that the
    sort is a permutation, in order and stable."""
    import torch
    n = (1 << 30) + 12345
    g = torch.Generator(device="cuda")
    g.manual_seed(7 + tickets)
    k = torch.randint(-(1 << 31), 1 << 31, (n,), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    d_k, d_v = k.clone(), torch.arange(n, dtype=torch.int32, device="cuda")
    d_f, d_p = torch.empty(n, dtype=torch.int8, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
    ws = tcuscan.new_workspace(1, n, "i8")
    tcuscan.set_chain_policy(tickets)
    try:
        tcuscan.split_radix_sort_u32(d_k, torch.empty_like(d_k), d_f, d_p, vals=d_v, vals_tmp=torch.empty_like(d_v), bits=32, ws=ws)
        torch.cuda.synchronize()
    finally:
        tcuscan.set_chain_policy(0)
    assert tcuscan.workspace_fault(ws) == 0
    del d_f, d_p, ws
    both = ((d_k.to(torch.int64) & 0xFFFFFFFF) << 31) | d_v.to(torch.int64)      # 63 bits: by key, then by index
    assert bool((both[1:] > both[:-1]).all())                                    # so all payloads differ
    del both
    assert int(d_v.min().item()) == 0 and int(d_v.max().item()) == n - 1
    assert bool((k[d_v.to(torch.int64)] == d_k).all())


@pytest.mark.parametrize("pairs", [False, True], ids=["keys", "pairs"])
def test_a_tile_that_does_not_know_its_places_is_not_stored(pairs):
    """Tile 3 keeps silent, so the wait of tile 4 gives up, and every later tile does.  One pass: keys of tiles 0 .. 3 are
    where they belong, no other place of the array is touched.  Four passes: all kernels end and nothing is written outside
    the arrays.  The fault word reads 1 either way, and once it is cleared the same call sorts again."""
    import torch
    tile = 4096
    n = 40 * tile + 11
    k = inputs.int32_full(n, 21).view(np.uint32)
    room = (n + 3) // 4 * 4 + 128                                                # rows start at 16-byte boundaries
    for bits in (8, 32):
        buf = torch.full((4, room), -7, dtype=torch.int32, device="cuda")
        d_k, d_kt, d_v, d_vt = (buf[i, 64:64 + n] for i in range(4))
        d_f, d_p = torch.empty(n, dtype=torch.int8, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
        ws = tcuscan.new_workspace(1, n, "i8")

        def sort():
            d_k.copy_(torch.from_numpy(k.view(np.int32)))
            d_v.copy_(torch.arange(n, dtype=torch.int32))
            tcuscan.split_radix_sort_u32(d_k, d_kt, d_f, d_p, vals=d_v if pairs else None, vals_tmp=d_vt if pairs else None, bits=bits, ws=ws)
            torch.cuda.synchronize()

        tcuscan.test_chain_fault(4096, 3)
        try:
            sort()
        finally:
            tcuscan.test_chain_fault(0, -1)
        assert tcuscan.workspace_fault(ws) == 1
        for b in buf:
            assert bool((b[:64] == -7).all()) and bool((b[64 + n:] == -7).all())
        order = np.argsort(k & np.uint32((1 << bits) - 1), kind="stable")
        if bits == 8:
            at = np.empty(n, np.int64)
            at[order] = np.arange(n)
            want_k, want_v = k.copy(), np.arange(n, dtype=np.int32)
            want_k[at[:4 * tile]], want_v[at[:4 * tile]] = k[:4 * tile], np.arange(4 * tile)
            assert np.array_equal(d_k.cpu().numpy().view(np.uint32), want_k)
            assert not pairs or np.array_equal(d_v.cpu().numpy(), want_v)
        tcuscan.workspace_init(ws)
        sort()
        assert tcuscan.workspace_fault(ws) == 0
        assert np.array_equal(d_k.cpu().numpy().view(np.uint32), k[order])
        assert not pairs or np.array_equal(d_v.cpu().numpy(), order.astype(np.int32))
