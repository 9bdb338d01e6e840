"""The integer arithmetic of the road search on the layer runs (csrc/run_search.h),
compiled for the CPU: which hits pass the road's bound."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1309_6275_amd", "csrc")
SHIM = r"""
#include "run_search.h"
extern "C" uint32_t road_words(uint32_t b) { return ht::road_words(b); }
extern "C" uint32_t visit_num() { return ht::kVisitNum; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("run_search")
    (d / "shim.cpp").write_text(SHIM)
    so = d / "shim.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-fPIC", "-shared", "-I", CSRC, "-o",
                    str(so), str(d / "shim.cpp")], check=True)
    L = ctypes.CDLL(str(so))
    for f in ("road_words", "visit_num"):
        getattr(L, f).restype = ctypes.c_uint32
    return L


def bits(x):
    return int(np.float32(x).view(np.uint32))


def test_road_words_keep_every_hit_on_the_road(lib):
    """A hit with |f| <= thr has a word below the bound whatever its number; hits that
    are no members (infinite or not a number) never have."""
    num = lib.visit_num()
    rng = np.random.default_rng(5)
    thr = np.concatenate([10.0 ** rng.uniform(-6, 6, 400), [0.0, 0.25007220, 1.0, 2.0, 3.0e38]])
    for t in np.float32(thr):
        end = lib.road_words(bits(t))
        for step in (0, 1, 2, 100, 511, 512, 513, 5000):
            f = max(bits(t) - step, 0)
            for n in (0, 1, num):
                assert ((f & ~num) | n) < end, (t, step, n)
        # not loose: beyond the next step of the words nothing passes
        assert end <= bits(t) + num + 1
    for t in (1.0, np.inf, np.finfo(np.float32).max):
        end = lib.road_words(bits(t))
        for b in (bits(np.inf), bits(np.nan), 0x7fffffff):
            assert ((b & ~num) | 0) >= end
