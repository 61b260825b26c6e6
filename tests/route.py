"""The route a backward or forward call takes: the library's own rule (embc_route.h), compiled for the host."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2010_11305_amd", "csrc")

SOURCE = """
#include "embc_route.h"
extern "C" int route(int64_t L, int32_t B, int T, int dim, int64_t set_rows) {
  return embc::small_call(L, B, T, set_rows) ? 0 : embc::mid_call(L, B, T, dim) ? 1 : 2;
}
extern "C" int64_t set_rows(int64_t n_sets, int64_t rows) { return embc::small_set_rows(n_sets, rows); }
extern "C" int fused(int64_t L, int64_t nbags, int dim, int assoc) { return embc::fused_call(L, nbags, dim, assoc); }
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "route.cpp"), os.path.join(d, "route.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", src, "-o", so], check=True)
        lib = ctypes.CDLL(so)
        lib.set_rows.restype = ctypes.c_int64
        return lib


def set_rows(cfg):
    """The most rows of a table that share one of few sets (0 without a cache)."""
    frac, assoc = cfg.get("cache_fraction", 0.0), cfg.get("assoc", 1)
    if frac <= 0:
        return 0
    sets = [(max(1, int(np.floor(frac * n)) // assoc), n) for n in cfg["rows"]]
    return max(_lib().set_rows(ctypes.c_int64(s), ctypes.c_int64(-(-n // s))) for s, n in sets)


def route(cfg, lookups, batch=None):
    """"small", "mid" or "general" for a call of `lookups` on the tables of cfg."""
    B = cfg["batch"] if batch is None else batch
    r = _lib().route(ctypes.c_int64(int(lookups)), int(B), len(cfg["rows"]), int(cfg["dim"]),
                     ctypes.c_int64(set_rows(cfg)))
    return ("small", "mid", "general")[r]


def one_kernel_forward(cfg, lookups):
    return bool(_lib().fused(ctypes.c_int64(int(lookups)), ctypes.c_int64(cfg["batch"] * len(cfg["rows"])),
                             int(cfg["dim"]), int(cfg["assoc"])))
