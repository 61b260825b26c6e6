"""The route a backward call takes: the library's own rule (embc_route.h), compiled for the host."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2010_11305_amd", "csrc")

SOURCE = """
#include "embc_route.h"
extern "C" int route(int64_t L, int32_t B, int T, int dim) {
  return embc::small_call(L, B, T) ? 0 : embc::mid_call(L, B, T, dim) ? 1 : 2;
}
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "route.cpp"), os.path.join(d, "route.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", src, "-o", so], check=True)
        return ctypes.CDLL(so)


def route(cfg, lookups, batch=None):
    """"small", "mid" or "general" for a call of `lookups` on the tables of cfg."""
    B = cfg["batch"] if batch is None else batch
    r = _lib().route(ctypes.c_int64(int(lookups)), int(B), len(cfg["rows"]), int(cfg["dim"]))
    return ("small", "mid", "general")[r]
