"""The rules of the launch planning (csrc/plan.hpp, plain C++): compiled here
with g++ and asked directly, no GPU."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_09465_amd", "csrc")

SHIM = r"""
#include <cstdint>
#include "plan.hpp"
using namespace iugkp;
extern "C" {
int64_t split_total(const double *t, int n, int64_t lds_words, int has_null, int K, int n_cu,
                    int64_t lds_max)
{
  std::vector<double> v(t, t + n);
  const double chunk = split_chunk(v, lds_words, has_null != 0, K, n_cu, lds_max);
  int64_t total = 0;
  for (double p : v) total += split_parts(p, chunk);
  return total;
}
// one search: the forms of `iters` iterations, form f taking t[f] (ran), and the
// form kept after each (kept)
void search(const int *cand, int n, int def, int rounds, const float *t, int iters, int *ran,
            int *kept)
{
  FormSearch s;
  s.rounds = rounds;
  s.cand.assign(cand, cand + n);
  s.def = def;
  for (int i = 0; i < iters; ++i) {
    ran[i] = s.pick();
    s.record(t[kForms * (i % 2) + ran[i]]);    // (even iterations, odd ones)
    kept[i] = s.kept();
  }
}
// bit 0: blocks are timed, bit 1: they run first
int quiet(const double *lam, int K, double flights, int T)
{
  const std::vector<double> b(lam, lam + K);
  return (quiet_blocks(b, flights, T) ? 1 : 0) | (quiet_blocks_first(b, flights) ? 2 : 0);
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    so = d / "libplan.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC,
                    str(d / "shim.cpp"), "-o", str(so)], check=True)
    lib = C.CDLL(str(so))
    lib.split_total.restype = C.c_int64
    lib.split_total.argtypes = [C.c_void_p, C.c_int, C.c_int64, C.c_int, C.c_int, C.c_int, C.c_int64]
    lib.search.restype = None
    lib.search.argtypes = [C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_void_p, C.c_int, C.c_void_p,
                           C.c_void_p]
    lib.quiet.restype = C.c_int
    lib.quiet.argtypes = [C.c_void_p, C.c_int, C.c_double, C.c_int]
    return lib


CUS, LDS = 256, 163840


# (tiles of particles, LDS words of a window, null collisions, launches together)
@pytest.mark.parametrize("n,particles,words,null,K", [
    (165, 3072, 12700, 0, 1),       # 164 x 161 cells: a CU's LDS per workgroup
    (174, 3120, 2158, 0, 1),        # a long film
    (84, 6912, 12700, 0, 1), (15, 16000, 102, 0, 1), (90, 40000, 6000, 0, 3), (3, 1, 10, 0, 1),
])
def test_split_tiles_stay_resident_together(plan, n, particles, words, null, K):
    """Tiles that fit the device at once are not split beyond it, except with null
    collisions, whose chains a second round evens out."""
    t = np.full(n, float(particles))
    total = plan.split_total(t.ctypes.data, n, words, null, K, CUS, LDS)
    room = max(1, CUS * min(8, max(1, LDS // (8 * words))) // K)
    assert n <= total <= room
    assert plan.split_total(t.ctypes.data, n, words, 1, K, CUS, LDS) >= total


def test_split_tiles_fill_the_device(plan):
    """A film of few tiles takes hundreds of workgroups, many tiles stay whole."""
    t = np.full(15, 6.7e4)
    assert 300 <= plan.split_total(t.ctypes.data, 15, 102, 0, 1, CUS, LDS) <= 1024
    t = np.full(4000, 300.0)
    assert plan.split_total(t.ctypes.data, 4000, 5000, 0, 1, CUS, LDS) == 4000


@pytest.mark.parametrize("cand,default,rounds,times,best", [
    ([0, 1, 2, 3], 2, 1, [4, 3, 1, 2, 9] * 2, 2), ([1, 2, 4], 4, 1, [1, 5, 6, 1, 7] * 2, 1),
    ([0, 4], 0, 1, [5, 1, 1, 1, 2] * 2, 4), ([], 4, 1, [1, 1, 1, 1, 2] * 2, 4),
    ([4], 0, 1, [1, 1, 1, 1, 2] * 2, 4),
    # (uneven iterations: the sum over three rounds decides)
    ([0, 1, 4], 0, 3, [9, 3, 0, 0, 3] + [1, 5, 0, 0, 3], 4),
])
def test_form_search(plan, cand, default, rounds, times, best):
    """The planner's choice first, every candidate in turn, then the fastest of them."""
    c, t = np.array(cand + [0], np.int32), np.array(times, np.float32)
    ran, kept = np.zeros(12, np.int32), np.zeros(12, np.int32)
    plan.search(c.ctypes.data, len(cand), default, rounds, t.ctypes.data, 12, ran.ctypes.data,
                kept.ctypes.data)
    head = ([default] + cand * rounds) if cand else []
    assert ran.tolist() == head + [best] * (12 - len(head))
    n = len(cand) * rounds
    assert kept.tolist() == [-1] * n + [best] * (12 - n)


@pytest.mark.parametrize("lam,flights,blocks,want", [
    # (free paths in cells, flights per band, blocks per band)
    ([172.0, 19.0], 4e3, 9, 0),                             # few flights for a block
    ([2560.0, 284.0], 4e6, 9, 0), ([40.0], 1e7, 9, 0),      # long paths
    ([512.0, 57.0, 20.0], 4e6, 9, 0), ([256.0, 20.0, 10.0], 4e6, 9, 1),
    ([12.8], 1e7, 9, 3), ([5.0], 1.1e6, 9, 1),              # gray
    ([5120.0 / (2 * k + 1) ** 2 for k in range(40)], 1.25e6, 36, 3),
])
def test_blocks_without_face_tallies(plan, lam, flights, blocks, want):
    a = np.array(lam)
    assert plan.quiet(a.ctypes.data, len(lam), flights, blocks * len(lam)) == want
