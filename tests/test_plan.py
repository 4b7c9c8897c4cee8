"""The rules of the launch planning (csrc/plan.hpp, plain C++): compiled here
with g++ and asked directly, no GPU."""
import ctypes as C
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_09465_amd", "csrc")

SHIM = r"""
#include <cstdint>
#include <map>
#include <random>
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

unsigned propose(unsigned xcc, int ta, int tx, int G, int may_xcd, int fewer, uint64_t waited,
                 unsigned arrivals)
{
  return elect_proposal(xcc, ta, tx, G, may_xcd != 0, fewer != 0, waited, arrivals);
}
int rank(unsigned choice, unsigned xcc, int ta, int tx, int G) { return elect_rank(choice, xcc, ta, tx, G); }
int size(unsigned choice, int G) { return elect_size(choice, G); }

// record bytes of a step, and whether they fit this much free memory
int64_t records(int nx, int ny, int K, uint32_t N, int64_t free_bytes, int *fit)
{
  const BlockPlan p = plan_block_step(nx, ny, K, N, true, true, false, 256, 163840);
  *fit = records_fit(p, static_cast<size_t>(free_bytes));
  return static_cast<int64_t>(p.record_bytes());
}

int bands(int stripes, double flights, int T, int rounds)
{
  return bands_form(stripes != 0, flights, T, rounds) + 10 * bands_timed(stripes != 0, flights, T);
}

int band_level(const int *windows, int n, int blocks) { return mg_band_level(windows, n, blocks); }

// out: blocks of all bands, rounds, LDS bytes, round 0's units
void blocks(int nx, int ny, int K, uint32_t N, int null, int faces, int rays, int64_t *out)
{
  const BlockPlan p = plan_block_step(nx, ny, K, N, null != 0, faces != 0, rays != 0, 256, 163840);
  out[0] = p.T;
  out[1] = p.rounds;
  out[2] = static_cast<int64_t>(p.lds);
  out[3] = static_cast<int64_t>(p.units.size());
}

// The rounds of a planned step with the kernels' bookkeeping, a share `stay` of
// each unit's flights ending in it and the rest leaving in uneven shares over
// the four sides: 0, or the first bound that does not hold.
int rounds(int nx, int ny, int K, uint32_t N, int null, int faces, int rays, double stay, int seed,
           int64_t *most)
{
  const BlockPlan p = plan_block_step(nx, ny, K, N, null != 0, faces != 0, rays != 0, 256, 163840);
  if (p.T == 0) return 1;
  std::mt19937 gen(seed);
  std::uniform_real_distribution<double> uni(0.0, 1.0);
  // every cell and wall face in one block, every chunk of a block in one unit
  int64_t emitters = 0, chunks0 = 0;
  std::map<int, int64_t> next;
  for (int t = 0; t < p.T; ++t) {
    const BlockDesc &d = p.blk[t];
    emitters += d.n_e;
    if (d.ex < 1 || d.ey < 1 || d.base != chunks0) return 2;
    chunks0 += (static_cast<int64_t>(d.n_e) * N + kChunk - 1) / kChunk;
    if (8 * static_cast<size_t>(block_words(d.ex, d.ey, null, faces, null && !rays)) > p.lds) return 3;
  }
  if (p.blk[p.T].base != chunks0) return 4;
  if (emitters != static_cast<int64_t>(K) * (static_cast<int64_t>(nx) * ny + 2 * (nx + ny))) return 5;
  if (p.lds + kBlockStaticLds > 163840) return 6;
  // a unit: its block and its chunks (records each)
  struct U { int t; std::vector<int> ch; uint32_t slab, cap; };
  std::vector<U> units;
  for (const BlockUnit &u : p.units) {
    const BlockDesc &d = p.blk[u.t];
    const int64_t P = static_cast<int64_t>(d.n_e) * N;
    U v{u.t, {}, u.slab, u.cap};
    if (u.first != next[u.t]) return 7;
    next[u.t] += u.count;
    for (uint32_t i = 0; i < u.count; ++i)
      v.ch.push_back(static_cast<int>(std::min<int64_t>(kChunk, P - static_cast<int64_t>(u.first + i) * kChunk)));
    units.push_back(v);
  }
  most[0] = most[1] = most[2] = 0;
  for (int r = 0; r < p.rounds && !units.empty(); ++r) {
    std::map<int, std::vector<int>> in;                   // a block's chunks of the next round
    if (units.size() > p.n_units) return 10;
    most[0] = std::max<int64_t>(most[0], units.size());
    for (const U &u : units) {
      if (u.ch.size() > kUnitChunksMax || u.ch.empty()) return 11;
      most[2] = std::max<int64_t>(most[2], u.ch.size());
      if (static_cast<size_t>(u.slab) + u.cap > p.n_chunks) return 12;
      most[1] = std::max<int64_t>(most[1], u.slab + u.cap);
      int64_t n = 0;
      for (int c : u.ch) n += c;
      n = static_cast<int64_t>(n * (1.0 - stay));
      double w[4], sum = 0.0;
      for (double &x : w) sum += x = std::pow(uni(gen), 6.0);
      int64_t opened = 0, left = n;
      for (int d = 0; d < 4; ++d) {
        const int64_t m = d < 3 ? std::min<int64_t>(left, static_cast<int64_t>(n * w[d] / sum)) : left;
        left -= m;
        const int64_t nc = (m + kChunk - 1) / kChunk;
        if (nc > u.cap || nc > kUnitChunksMax) return 13;
        opened += nc;
        const int to = p.blk[u.t].nb[d];
        for (int64_t i = 0; i < nc; ++i)
          in[to].push_back(static_cast<int>(std::min<int64_t>(kChunk, m - i * kChunk)));
      }
      if (opened > u.cap) return 14;
    }
    int64_t total = 0;
    for (auto &b : in) total += b.second.size();
    const uint32_t share = unit_chunks(static_cast<uint32_t>(total), p.target, 256);
    units.clear();
    uint32_t before = 0;
    for (auto &b : in) {
      for (size_t c = 0; c < b.second.size(); c += share) {
        U v{b.first, {}, 0, 0};
        v.ch.assign(b.second.begin() + c, b.second.begin() + std::min<size_t>(b.second.size(), c + share));
        v.slab = before + static_cast<uint32_t>(c + units.size() * kOpenChunks);
        v.cap = static_cast<uint32_t>(v.ch.size()) + kOpenChunks;
        units.push_back(v);
      }
      before += static_cast<uint32_t>(b.second.size());
    }
  }
  return 0;
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
    lib.propose.restype = C.c_uint
    lib.propose.argtypes = [C.c_uint, C.c_int, C.c_int, C.c_int, C.c_int, C.c_int, C.c_uint64, C.c_uint]
    lib.rank.argtypes = [C.c_uint, C.c_uint, C.c_int, C.c_int, C.c_int]
    lib.size.argtypes = [C.c_uint, C.c_int]
    lib.records.restype = C.c_int64
    lib.records.argtypes = [C.c_int, C.c_int, C.c_int, C.c_uint32, C.c_int64, C.POINTER(C.c_int)]
    lib.bands.restype = C.c_int
    lib.bands.argtypes = [C.c_int, C.c_double, C.c_int, C.c_int]
    lib.blocks.restype = None
    lib.blocks.argtypes = [C.c_int, C.c_int, C.c_int, C.c_uint32, C.c_int, C.c_int, C.c_int, C.c_void_p]
    lib.rounds.argtypes = [C.c_int, C.c_int, C.c_int, C.c_uint32, C.c_int, C.c_int, C.c_int, C.c_double,
                           C.c_int, C.c_void_p]
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


@pytest.mark.parametrize("stripes,flights,blocks,rounds,form", [
    (1, 7.5e5, 16, 5, 12), (1, 2e6, 16, 5, 14), (1, 3.1e6, 16, 5, 4), (1, 6e4, 2, 1, 14), (1, 7e4, 4, 2, 10),
    (0, 2.3e5, 16, 2, 10), (0, 4.2e7, 1960, 13, 4), (0, 8.6e5, 56, 10, 14), (0, 4e5, 8, 1, 14),
    (0, 1.1e6, 8, 1, 4), (1, 8e6, 98, 13, 12),
])
def test_form_of_bands_with_face_tallies(plan, stripes, flights, blocks, rounds, form):
    """(form + 10 where the forms are timed)"""
    assert plan.bands(stripes, flights, blocks, rounds) == form


@pytest.mark.parametrize("shape", [
    # nx, ny, bands, flights per emitter, null collisions, face tallies, rays
    (61, 61, 1, 80, 1, 1, 0), (1, 400, 1, 50, 1, 1, 0), (301, 71, 1, 19, 1, 0, 0),
    (90, 77, 1, 31, 0, 0, 1), (150, 141, 1, 10, 1, 1, 1), (120, 120, 3, 9, 1, 1, 0),
    (48, 48, 40, 1, 1, 1, 0), (512, 512, 1, 60, 1, 1, 0), (256, 256, 1, 600, 1, 1, 0),
])
def test_block_rounds_stay_in_bounds(plan, shape):
    """Units, chunks, lists and LDS of every round, wherever the flights go."""
    for stay, seed in ((0.0, 1), (0.0, 2), (0.3, 3), (0.9, 4)):
        most = np.zeros(3, np.int64)
        assert plan.rounds(*shape, stay, seed, most.ctypes.data) == 0
    if shape[3] == 600:
        assert most[2] == 256            # (units of the largest size)


def test_blocks_beyond_their_tables(plan):
    """No blocks where they would be more than a launch holds, or their chunks more
    than a list entry can number."""
    out = np.zeros(4, np.int64)
    for args in ((800, 800, 40, 1, 1, 1, 0), (560, 560, 80, 1, 1, 1, 0), (512, 512, 1, 8100, 1, 1, 0)):
        plan.blocks(*args, out.ctypes.data)
        assert out[0] == 0
    plan.blocks(700, 700, 40, 1, 1, 1, 0, out.ctypes.data)
    assert 0 < out[0] <= 4096


def test_block_records_leave_room(plan):
    """About 128 bytes a flight; a step whose records would take more than an
    eighth of the free memory has no blocks (1e9 flights on an empty 288 GB)."""
    fit = C.c_int(0)
    ne = 512 * 512 + 4 * 512
    for N, free, want in ((190, 288 << 30, 1), (3800, 288 << 30, 0), (190, 40 << 30, 0)):
        b = plan.records(512, 512, 1, N, free, C.byref(fit))
        assert 1.0 <= b / (128.0 * ne * N) < 1.1
        assert fit.value == want == (b <= free // 8)


def _run_groups(plan, groups, fewer, seed, slots=256, xcds=8, ticks=1000, steps=4000):
    """Groups (launched, wanted) of workgroups of a CU each on one device, their
    dispatches interleaved at random, `ticks` of the clock a step: the sizes that
    ran, or None for a group that never did."""
    rng = random.Random(seed)
    queue = [g for g, (launch, _) in enumerate(groups) for _ in range(launch)]
    rng.shuffle(queue)
    free = [slots // xcds] * xcds
    ran = [None] * len(groups)
    choice, arrived, on_xcd = [0] * len(groups), [0] * len(groups), [[0] * xcds for _ in groups]
    waiting, members = [], [[] for _ in groups]
    for step in range(steps):
        for x in range(xcds):
            while free[x] and queue:
                g = queue.pop()
                free[x] -= 1
                waiting.append((g, x, arrived[g], on_xcd[g][x], step))
                arrived[g] += 1
                on_xcd[g][x] += 1
        still = []
        for g, x, ta, tx, t0 in waiting:
            launch, want = groups[g]
            if not choice[g]:
                choice[g] = plan.propose(x, ta, tx, want, int(launch > want), fewer, ticks * (step - t0),
                                         arrived[g])
            if not choice[g]:
                still.append((g, x, ta, tx, t0))
            elif plan.rank(choice[g], x, ta, tx, want) >= 0:
                members[g].append((x, plan.rank(choice[g], x, ta, tx, want)))
            else:
                free[x] += 1
        waiting = still
        for g, (launch, want) in enumerate(groups):
            n = plan.size(choice[g], want) if choice[g] else 0
            if n and len(members[g]) == n:                       # (every barrier is met)
                assert sorted(r for _, r in members[g]) == list(range(n))
                if choice[g] < 0x100:
                    assert len({x for x, _ in members[g]}) == 1
                for x, _ in members[g]:
                    free[x] += 1
                members[g], ran[g] = [], n
        if all(ran):
            break
    return ran


@pytest.mark.parametrize("groups", [
    [(64, 64)] * 4, [(64, 64)] * 9, [(256, 32)] * 9, [(64, 64)] * 5 + [(256, 32)] * 6 + [(128, 16)] * 4,
    [(200, 200)] * 3,
])
def test_elected_groups_never_keep_each_other_waiting(plan, groups):
    """However the workgroups of several solves are dispatched, each solve runs:
    whole where they fit together, on fewer workgroups where they do not."""
    for seed in range(6):
        ran = _run_groups(plan, groups, 1, seed)
        assert all(ran), (seed, ran)
        assert all(1 <= n <= want for n, (_, want) in zip(ran, groups))
        if sum(launch for launch, _ in groups) <= 256:
            assert ran == [want for _, want in groups]
    if groups == [(200, 200)] * 3:          # (only whole groups: they never run)
        assert not all(_run_groups(plan, groups, 0, 0))


# windows of the finest prolongation with 0, 1 and 2 levels fewer in LDS (0: no row
# fits), tree blocks of the mesh, and the choice that measured fastest or, of two
# within 5%, either
@pytest.mark.parametrize("windows, blocks, want", [
    ((1, 1, 1), 256, 0),      # 256 x 256
    ((7, 1, 1), 175, 1),      # 447 x 100
    ((7, 1, 1), 250, 1),      # 400 x 160
    ((13, 2, 2), 827, 1),     # 460 x 460
    ((3, 2, 2), 1211, 0),     # 467 x 664: the LDS level is as good as the window
    ((0, 8, 2), 40, 2),       # the first that fits is not the best
    ((0, 0, 0), 57, -1),      # 720 x 20: rows too long for two levels more
    ((0, 0, 4), 124, -1),     # 720 x 44
    ((0, 4, 4), 360, -1),     # 720 x 128
    ((0, 6, 3), 648, 2),      # 648 x 256
    ((0, 4, 3), 63, -1),      # 800 x 20 of a batch
])
def test_banded_multigrid_level(plan, windows, blocks, want):
    w = np.array(windows, dtype=np.int32)
    assert plan.band_level(w.ctypes.data_as(C.POINTER(C.c_int)), len(w), blocks) == want
