"""Which kernels a call enqueues, seen without a GPU: `launches` runs calls of the C entry points in a process in which
launch_recorder_shim.cpp takes the place of the HIP runtime.  The addresses passed are never followed."""
from __future__ import annotations

import collections
import json
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2411_17887_amd", "libtcuscan.so")

# stride: log2 of the 64-bit words between the status words of the small segmented kernels (else 0)
Launch = collections.namedtuple("Launch", "kernel grid block stride")

_CHILD = """
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
shim.shim_launches.restype = ctypes.c_char_p
out = []
for name, args in json.load(sys.stdin):
    shim.shim_clear()
    fn = getattr(lib, name)
    fn.restype = ctypes.c_size_t if name.endswith("_bytes") else ctypes.c_int
    rc = fn(*[ctypes.c_size_t(a & (2 ** 64 - 1)) for a in args])
    out.append([rc, shim.shim_launches().decode()])
print(json.dumps(out))
"""


def build(folder) -> str:
    so = os.path.join(str(folder), "launch_recorder_shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-o", so, os.path.join(HERE, "launch_recorder_shim.cpp")], check=True)
    return so


def launches(shim: str, calls):
    """calls: [(entry point, [integers])], made in order in one process.  Returns for each (status, [Launch])."""
    done = subprocess.run([sys.executable, "-c", _CHILD, shim, LIB], input=json.dumps(calls), capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stderr
    result = []
    for rc, text in json.loads(done.stdout):
        rows = [line.split(" ", 3) for line in text.splitlines()]
        result.append((rc, [Launch(_plain(name), int(grid), int(block), int(stride)) for grid, block, stride, name in rows]))
    return result


def _plain(name: str) -> str:
    """`void (anonymous namespace)::kernel<1, true>(...)` -> `kernel<1, true>`."""
    name = name.replace("(anonymous namespace)::", "")
    name = re.sub(r"^void ", "", name)
    return name[:name.rindex("(")] if name.endswith(")") else name
