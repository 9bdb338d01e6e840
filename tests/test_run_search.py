"""The integer arithmetic of the road search on the layer runs (csrc/run_search.h),
compiled for the CPU: which hits pass the road's bound, which hits of a run the
lanes visit, and where the seeds are read."""
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
extern "C" void seed_lane(int lane, const int* n, const int* st, int* out) {
  const ht::SeedLane v = ht::seed_lane(lane, n[0], n[1], n[2], st[0], st[1], st[2]);
  out[0] = v.s; out[1] = v.st; out[2] = v.n; out[3] = v.e;
}
extern "C" int seed_record(int s, const int* run, uint32_t hp) {
  return ht::seed_record(s, run[0], run[1], run[2], hp);
}
extern "C" uint32_t visit_num() { return ht::kVisitNum; }
// The places of a run of len hits that each of n lanes visits for its arcs [arc[0],
// arc[1]) and [arc[2], arc[3]), as the kernel's loops take them: seen[lane * len +
// place] counts the visits.  Returns 0, or the line of the check that failed.
extern "C" int visits(int n, int len, const int* arcs, int* seen) {
  using namespace ht;
  for (int g0 = 0; g0 < len; g0 += kStage) {
    const int ge = len < g0 + kStage ? len : g0 + kStage;
    int num = 0, num1 = 0;
    for (int arc = 0; arc < 2; ++arc) {
      for (bool more = true; more;) {
        more = false;
        for (int l = 0; l < n; ++l) {
          const int* a = arcs + 4 * l;
          const Arcs v = order_arcs(a[0], a[1], a[2], a[3]);
          const int e = stage_first(arc ? v.b0 : v.a0, g0) + num - (arc ? num1 : 0);
          if (e >= stage_end(arc ? v.b1 : v.a1, g0)) continue;
          more = true;
          for (int u = 0; u < kVisit; ++u) {
            if (e < g0 || e + u >= ge + 4) return __LINE__;   // outside the staged hits and the pad
            if (num + u > (int)kVisitNum) return __LINE__;
            if (arc == 1 && visit_place(v, g0, num + u, num1) != e + u) return __LINE__;
            if (e + u < ge) seen[l * len + e + u]++;          // behind: no members
          }
        }
        if (more) num += kVisit;
      }
      if (arc == 0) num1 = num;
    }
  }
  return 0;
}
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


def test_every_place_of_both_arcs_is_visited_once(lib):
    """Runs below and above a stage, arcs with and without a gap, adjacent ones across
    the stages' ends among them."""
    rng = np.random.default_rng(6)
    for trial in range(4000):
        n = int(rng.integers(1, 5))
        len_ = int(rng.choice([rng.integers(1, 257), rng.integers(257, 1400)]))
        arcs = np.zeros((n, 4), np.int32)
        for l in range(n):
            p = np.sort(rng.integers(0, len_ + 1, 4))
            if rng.random() < 0.5:  # the second arc a few hits behind the first
                p[2] = min(p[1] + rng.integers(0, 4), len_)
                p[3] = max(p[2], p[3])
            if rng.random() < 0.5:
                p = p[[2, 3, 0, 1]]
            if rng.random() < 0.1:
                p[rng.integers(0, 2) * 2 + np.arange(2)] = 0
            arcs[l] = p
        seen = np.zeros((n, len_), np.int32)
        rc = lib.visits(n, len_, arcs.ctypes.data_as(ctypes.c_void_p),
                        seen.ctypes.data_as(ctypes.c_void_p))
        assert rc == 0, (rc, len_, arcs)
        for l in range(n):
            want = np.zeros(len_, bool)
            want[arcs[l, 0]:arcs[l, 1]] = True
            want[arcs[l, 2]:arcs[l, 3]] = True
            assert np.all(seen[l][want] == 1), (len_, arcs[l])
            assert seen[l].max() <= 1


def test_seed_records_lie_in_their_runs(lib):
    """A list of members (each a place in its layer's run) and its three seed layers,
    whose runs lie anywhere in the stored records: every lane, with a seed member or
    without one, reads a record of a seed layer's run."""
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    rng = np.random.default_rng(8)
    for _ in range(200):
        layers = int(rng.integers(3, 17))
        lens = rng.integers(1, 40, layers)          # run lengths
        lens[rng.random(layers) < 0.4] = 1
        n = np.minimum(rng.integers(1, 15, layers), lens)  # members
        place = [np.sort(rng.choice(lens[l], n[l], replace=False)) for l in range(layers)]
        first = np.cumsum(n) - n
        hp = np.concatenate(place)
        seeds = np.sort(rng.choice(layers, 3, replace=False))
        if rng.random() < 0.2:
            seeds[1] = seeds[0]
        run = np.int32(rng.integers(0, 1000, layers))
        ns, st, rs = (np.int32(a[seeds]) for a in (n, first, run))
        if ns.sum() > 64:
            continue
        seen = []
        for lane in range(64):
            out = np.zeros(4, np.int32)
            lib.seed_lane(lane, p(ns), p(st), p(out))
            s, l_st, l_n, e = (int(v) for v in out)
            word = int(rng.integers(0, 65536)) << 16 | int(hp[e])
            rec = lib.seed_record(s, p(rs), ctypes.c_uint32(word))
            L = seeds[s if s >= 0 else 2]
            assert run[L] <= rec < run[L] + lens[L], (lane, s)
            if s >= 0:
                assert rec == run[L] + place[L][e - first[L]] and (l_st, l_n) == (first[L], n[L])
                seen.append((s, e))
            else:
                assert l_n == 0 and 0 <= l_st <= hp.size
        assert len(set(seen)) == len(seen) == ns.sum()
