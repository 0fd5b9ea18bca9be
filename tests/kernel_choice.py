"""The kernels that a call's sizes lead to: the sort's automatic choice (csrc/sort_choice.h), the
ingestion's (csrc/ingest_choice.h) and the join's rules (csrc/join_choice.h), the headers themselves,
compiled for the host."""
from __future__ import annotations

import ctypes
import functools
import subprocess
import tempfile
from pathlib import Path

CSRC = Path(__file__).resolve().parent.parent / "paper_2609_22441_amd" / "csrc"
MERGE, RADIX, RANK, PART, SPLIT = 1, 2, 3, 4, 5

SHIM = """#include "ingest_choice.h"
#include "join_choice.h"
#include "sort_choice.h"
extern "C" int choice(int64_t total, int64_t n_viewers, int64_t max_keys) {
    return ccj::sort_choice(total, n_viewers, max_keys);
}
extern "C" int apart(int64_t n_records, int64_t row_bytes) {
    return ccj::commit_apart(n_records, row_bytes);
}
extern "C" int64_t ranges(int64_t n, int64_t viewers, int64_t most) {
    return ccj::ranges_of_viewers(n, viewers, most);
}
extern "C" int plain(int64_t rows, int64_t stride, int64_t width) {
    return ccj::plain_copy(rows, stride, width);
}
extern "C" int fences(int64_t total_keys, int64_t viewers, int long_lists) {
    return ccj::least_fences(total_keys, viewers, long_lists);
}
"""


@functools.lru_cache(maxsize=None)
def _shim():
    with tempfile.TemporaryDirectory() as d:
        src, out = Path(d) / "choice.cpp", Path(d) / "choice.so"
        src.write_text(SHIM)
        subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", f"-I{CSRC}",
                        str(src), "-o", str(out)], check=True)
        lib = ctypes.CDLL(str(out))
    lib.choice.argtypes = [ctypes.c_int64] * 3
    lib.apart.argtypes = [ctypes.c_int64] * 2
    lib.ranges.argtypes, lib.ranges.restype = [ctypes.c_int64] * 3, ctypes.c_int64
    lib.plain.argtypes = [ctypes.c_int64] * 3
    lib.fences.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    return lib


def choice(sizes, max_keys=0) -> int:
    """The method of a call with viewers of these sizes."""
    return _shim().choice(int(sum(sizes)), len(sizes), max_keys)


def commit_apart(n_records, row_bytes) -> bool:
    return bool(_shim().apart(n_records, row_bytes))


def least_fences(viewers, keys) -> int:
    """Of viewers with `keys` keys each (lists of more than 32,768 on average count as long)."""
    return _shim().fences(viewers * keys, viewers, keys > 32_768)


def ranges_of_viewers(n, viewers, most) -> int:
    return _shim().ranges(n, viewers, most)


def plain_copy(rows, stride, width) -> bool:
    return bool(_shim().plain(rows, stride, width))
