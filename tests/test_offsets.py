"""The kernels' check of the table boundaries (embc_offsets.h), compiled for the host: offsets
whose tables are valid one by one but share positions are bad, and the tables of accepted
boundaries are disjoint ranges of the lookups."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2010_11305_amd", "csrc")

SOURCE = """
#include "embc_offsets.h"
extern "C" int bad(const int32_t* off, int T, int32_t B, int64_t L, int first, int stride) {
  return embc::bad_boundaries(off, T, B, L, first, stride);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("offsets")
    src, so = d / "offsets.cpp", d / "offsets.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def bad(lib, off, T, B, L, threads=1):
    off = np.ascontiguousarray(off, dtype=np.int32)
    assert off.size == T * B + 1
    p = off.ctypes.data_as(ctypes.c_void_p)
    return any(lib.bad(p, T, B, ctypes.c_int64(L), i, threads) for i in range(threads))


@pytest.mark.parametrize("threads", [1, 3, 1024])
def test_tables_that_share_positions_are_bad(lib, threads):
    L, B = 20_000, 2
    off = [0, 10_000, 20_000, 20_000, 0, 10_000, 20_000]   # tables 0 and 2 are valid by themselves
    for t in (0, 2):
        assert not bad(lib, off[t * B:(t + 1) * B + 1], 1, B, L)
    assert bad(lib, off, 3, B, L, threads)


@pytest.mark.parametrize("threads", [1, 3, 1024])
def test_against_the_definition(lib, threads):
    rng = np.random.default_rng(3)
    seen = set()
    for _ in range(300):
        T, B, L = int(rng.integers(1, 7)), int(rng.integers(1, 4)), int(rng.integers(0, 30))
        off = np.sort(rng.integers(0, L + 1, T * B + 1))
        for _ in range(int(rng.integers(0, 3))):
            off[rng.integers(off.size)] = rng.integers(-2, L + 3)
        edge = off[::B]
        want = bool(np.any(edge < 0) or np.any(edge > L) or np.any(np.diff(edge) < 0))
        assert bad(lib, off, T, B, L, threads) == want, (off, T, B, L)
        seen.add(want)
    assert seen == {True, False}
