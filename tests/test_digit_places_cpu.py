"""Destinations of a sort pass on digits (paper_2411_17887_amd/csrc/digit_places.h), compiled for the CPU.

What has to hold for both widths of a place: whatever number of keys a look-back returned as lying in front of a tile's
digit -- also one that is smaller than the digit's place inside the tile, which a wait that gave up can return -- every
range the guard lets through is stored to bytes 4 * before .. 4 * (before + count) - 1 and nowhere else."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
TILE = 16384


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("digit_places") / "libshim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wall", "-Wextra", "-Werror", "-o", so,
                    os.path.join(HERE, "digit_places_shim.cpp")], check=True)
    L = ctypes.CDLL(so)
    for f in (L.shim_place32, L.shim_place64, L.shim_fits32, L.shim_fits64):
        f.argtypes = [ctypes.c_ulonglong, ctypes.c_uint, ctypes.c_uint]
    L.shim_bucket_limit.argtypes, L.shim_bucket_limit.restype = [ctypes.c_ulonglong, ctypes.c_uint], ctypes.c_uint
    L.shim_place32.restype = L.shim_place64.restype = ctypes.c_ulonglong
    return L


@pytest.mark.parametrize("width,n", [(32, 16385), (32, (1 << 30) - 2), (64, (1 << 30) - 1), (64, (1 << 30) + 12345), (64, (1 << 32) - 1)])
def test_every_range_the_guard_lets_through_goes_to_its_own_bytes(shim, width, n):
    place, range_fits = (shim.shim_place32, shim.shim_fits32) if width == 32 else (shim.shim_place64, shim.shim_fits64)
    unknown = (1 << (width - 2)) - 1                 # what a wait that gave up answers; counts may have been added to it
    stored = 0
    for start in (0, 1, 5000, TILE - 1):
        for count in {c for c in (0, 1, 1000, TILE - start) if start + c <= TILE}:
            for before in {b for b in (0, 1, start - 1, start, start + 1, n - count - 1, n - count, n - count + 1, n, n + 1, 0xFFFFFFFF,
                                        unknown, unknown + 1, unknown + n) if 0 <= b < 1 << width}:
                fits = before + count <= n
                assert not (fits and before >= unknown)
                assert bool(range_fits(before, count, n)) == fits
                if fits and count:
                    for i in (start, start + count // 2, start + count - 1):
                        assert place(before, start, i) == 4 * (before + i - start) <= 4 * (n - 1), (before, start, i)
                        stored += 1
    assert stored > 30


def test_buckets_that_a_workgroup_sorts_while_passes_would_sort_all_keys(shim):
    """The limit on a bucket's keys: never more than fit, never so many that the passes were faster where both were measured, and
    enough for the buckets of random keys (mean and six standard deviations) up to 6,055,225 keys."""
    fit = 24576
    for n, slower in [(20_000, 9000), (33_000, 9000), (70_000, 9000), (131_072, 12_000), (262_144, 14_000), (400_000, 16_384), (600_000, 16_384), (1_000_000, 24_000)]:
        assert shim.shim_bucket_limit(n, fit) < slower
    last = 0
    for n in sorted([*range(16_385, 7_000_000, 4099), 6_055_225, 6_055_226]):
        limit = shim.shim_bucket_limit(n, fit)
        assert last <= limit <= fit
        assert (n / 256 + 6 * (n / 256) ** 0.5 <= limit) == (n <= 6_055_225), n
        last = limit
