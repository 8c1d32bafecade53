"""What a sort by two passes and small buckets finds out about its keys, in numpy: the sample's verdict and the buckets' (large_sort_plan.h, sort.hip)."""
from __future__ import annotations

import collections
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
FIELDS = ("log low most_tiles huge_tiles huge_work some_most huge_most wide_most work_most few_most found counts ranges huge status end").split()
Plan = collections.namedtuple("Plan", FIELDS)
SAMPLE_QUADS, SMALL, LARGE, HUGE, HUGE_TILE = 2048, 5120, 10240, 1 << 18, 8192


@functools.lru_cache(None)
def shim():
    so = os.path.join(tempfile.mkdtemp(prefix="sort_rules"), "libshim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wall", "-Wextra", "-Werror", "-o", so, os.path.join(HERE, "sort_rules_shim.cpp")], check=True)
    L = ctypes.CDLL(so)
    L.shim_large_wanted.argtypes = [ctypes.c_ulonglong, ctypes.c_int]
    L.shim_large_plan.argtypes = [ctypes.c_ulonglong, ctypes.c_int, ctypes.POINTER(ctypes.c_ulonglong)]
    return L


def plan(n: int, pairs: bool) -> Plan:
    out = (ctypes.c_ulonglong * len(FIELDS))()
    shim().shim_large_plan(n, int(pairs), out)
    return Plan(*map(int, out))


def sample_says(k: np.ndarray, bits: int, pairs: bool) -> bool:
    p, n = plan(k.size, pairs), k.size
    part = n // 4 // SAMPLE_QUADS
    g = np.arange(SAMPLE_QUADS, dtype=np.uint64)
    at = g * part + ((g * 0x9E3779B1 & 0xFFFFFFFF) >> 8) % part
    keys = k[(4 * at[:, None] + np.arange(4, dtype=np.uint64)).reshape(-1)]
    bucket = (keys >> np.uint32(bits - p.log)) & np.uint32((1 << p.log) - 1)
    c, used = np.bincount(bucket, minlength=1 << p.log).astype(np.int64), np.unique(bucket[::4]).size
    wide = c.reshape(256, -1).sum(1)
    some = c[c > p.some_most]
    work = int((some * (1 + some * n // (4 * SAMPLE_QUADS * HUGE_TILE))).sum())
    return bool(c.max() <= p.huge_most and wide.max() <= p.wide_most and work <= p.work_most and used >= p.few_most)


def found(k: np.ndarray, bits: int, pairs: bool) -> dict:
    """split, tried, large, huge, work as the kernels leave them; `huge` and `large` count only where the sample has said that it is worth it."""
    p = plan(k.size, pairs)
    if not sample_says(k, bits, pairs):
        return dict(split=0, tried=0, large=0, huge=0, work=0)
    size = np.bincount((k >> np.uint32(bits - p.log)) & np.uint32((1 << p.log) - 1), minlength=1 << p.log).astype(np.int64)
    huge = size[(size > LARGE) & (size <= HUGE)]
    tiles = (huge + HUGE_TILE - 1) // HUGE_TILE
    work = int(((huge >> 10) * tiles).sum())
    over = work > p.huge_work or int(tiles.sum()) > p.huge_tiles or size.max() > HUGE
    return dict(split=0 if over else 1, tried=1, large=int(((size > SMALL) & (size <= LARGE)).sum()), huge=int(tiles.sum()), work=work)
