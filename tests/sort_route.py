"""The sort's automatic choice (csrc/sort_choice.h) for a call's sizes: the header itself, compiled
for the host."""
from __future__ import annotations

import ctypes
import functools
import subprocess
import tempfile
from pathlib import Path

CSRC = Path(__file__).resolve().parent.parent / "paper_2609_22441_amd" / "csrc"
MERGE, RADIX, RANK, PART, SPLIT = 1, 2, 3, 4, 5

SHIM = """#include "sort_choice.h"
extern "C" int choice(int64_t total, int64_t n_viewers, int64_t max_keys) {
    return ccj::sort_choice(total, n_viewers, max_keys);
}
"""


@functools.lru_cache(maxsize=None)
def _shim():
    with tempfile.TemporaryDirectory() as d:
        src, out = Path(d) / "choice.cpp", Path(d) / "choice.so"
        src.write_text(SHIM)
        subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", f"-I{CSRC}",
                        str(src), "-o", str(out)], check=True)
        f = ctypes.CDLL(str(out)).choice
    f.argtypes = [ctypes.c_int64] * 3
    return f


def choice(sizes, max_keys=0) -> int:
    """The method of a call with viewers of these sizes."""
    return _shim()(int(sum(sizes)), len(sizes), max_keys)
