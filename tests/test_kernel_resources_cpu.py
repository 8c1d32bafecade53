"""What the built kernels take of a compute unit, from the metadata of the library's code objects (no GPU)."""
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2411_17887_amd import tcuscan

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + name]:
                yield blob[at + offset:at + offset + size]
            p += 24 + name
        at = blob.find(MAGIC, at + 1)


def kernels_of(elf):
    """The `amdhsa.kernels` records of one code object: a note of type 32, MessagePack inside."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * entry + 4)
        if kind != 7:                                            # SHT_NOTE
            continue
        offset, size = struct.unpack_from("<QQ", elf, shoff + i * entry + 0x18)
        p = offset
        while p < offset + size:
            name, desc, note = struct.unpack_from("<III", elf, p)
            body = p + 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
            p = body + (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    with open(tcuscan.LIB_PATH, "rb") as f:
        found = [k for elf in code_objects(f.read()) for k in kernels_of(elf)]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True, check=True).stdout.split("\n")
    plain = [re.sub(r"^void |\(anonymous namespace\)::", "", n) for n in names]
    assert len(found) > 50
    return {n[:n.rindex("(")]: k for n, k in zip(plain, found)}


@pytest.mark.parametrize("kernel", ["block_sort_kernel<true>", "block_sort_kernel<false>", "pass_or_buckets_kernel<4, true>", "pass_or_buckets_kernel<8, true>",
                                    "pass_or_buckets_kernel<4, false>", "pass_or_buckets_kernel<8, false>", "spread_kernel<true>", "spread_kernel<false>",
                                    "fine_sort_kernel<true>", "fine_sort_kernel<false>"])
def test_sorts_of_few_keys_and_usual_buckets_have_no_scratch(kernels, kernel):
    """A kernel with scratch starts later, whatever its workgroups do with it."""
    assert kernels[kernel][".private_segment_fixed_size"] == 0 and kernels[kernel][".vgpr_spill_count"] == 0


def test_passes_keep_two_workgroups_on_a_compute_unit(kernels):
    passes = {n: k for n, k in kernels.items() if n.startswith("digit_pass_kernel<16, 16,") and "unsigned int" in n}
    assert len(passes) >= 8
    for n, k in passes.items():
        assert k[".vgpr_count"] <= 64 and k[".private_segment_fixed_size"] == 0 and k[".group_segment_fixed_size"] <= 80 * 1024, n
