// plan.hpp -- rules of the host's launch planning, plain C++ (no device code).
#pragma once

#include <algorithm>
#include <cstddef>
#include <vector>

namespace iugkp {

// A tile's particles are split over several workgroups where the tiles alone
// leave compute units idle (a 100-cell film has 15): up to kSplitTarget
// workgroups per launch (two per compute unit), kSplitTargetNull with null
// collisions, whose chains differ in length, of at least kSplitMin particles
// (one per lane) and of one particle per kSplitWords words of LDS window, which
// every workgroup clears and flushes; and where the tiles fit the device at
// once, so do their shares (a second round of workgroups waits for the first:
// 164 x 161 cells, 286 workgroups of a CU's LDS each, 47 us against 35 unsplit;
// with null collisions a second round evens the chains out: 115 x 190, path 1.3
// cells, ratio 180, 3.8 ms against 5.5 with the limit; 199 x 74, path 350, ratio
// 23, with face tallies 0.50 against 0.80).
// Measured: film of 100 cells, 1e5 particles, particle step 658 -> 30 us (512 /
// 2048 particles at least: 27 / 38 us, but the two-time film's solve 1.85 ms
// against 2.2 / 3.0); 61 x 45 cells, 3e5 particles 104 -> 46 us; 128 x 100 with
// null collisions, 1e6 particles 1188 -> 729 us (one particle per 4 or 2 words:
// 806 / 1182).  Cavities of 24 .. 400 cells a side without null collisions,
// time against unsplit tiles, geometric mean and worst: without face tallies
// 0.88 and 1.24 (target 1024 and no limit: 0.92 and 1.41), with them 0.93 and
// 1.11 (0.94 and 1.13).
constexpr int kSplitTarget = 512, kSplitTargetNull = 1024;
constexpr int kSplitMin = 256;
constexpr int kSplitWords = 8;

inline int split_parts(double particles, double chunk)
{
  return std::max(1, static_cast<int>(particles / chunk + 0.5));
}

// Particles per workgroup for tiles of tiles[i] particles whose window takes
// lds_words of a compute unit's lds_max bytes, one of K such launches together.
inline double split_chunk(const std::vector<double> &tiles, size_t lds_words, bool has_null, int K,
                          int n_cu, size_t lds_max)
{
  double all = 0.0;
  for (double p : tiles) all += p;
  const int target = std::max(1, (has_null ? kSplitTargetNull : kSplitTarget) / K);
  double chunk = std::max({all / target, static_cast<double>(kSplitMin),
                           static_cast<double>(lds_words) / kSplitWords});
  const size_t per_cu = std::min<size_t>(8, std::max<size_t>(1, lds_max / std::max<size_t>(1, 8 * lds_words)));
  const size_t room = std::max<size_t>(1, n_cu * per_cu / K);
  auto total = [&] {
    size_t n = 0;
    for (double p : tiles) n += split_parts(p, chunk);
    return n;
  };
  if (!has_null && tiles.size() <= room)
    while (total() > room) chunk *= 1.05;
  return chunk;
}

// The forms of a handle's particle step.
enum : int {
  kFormTiles256 = 0,        // emitter tiles, 256 threads a workgroup (or the handle's block size)
  kFormTiles512 = 1,        // emitter tiles, 512 threads
  kFormStripes = 2,         // row stripes
  kFormPieces = 3,          // row stripes with the y faces in pieces (without null collisions)
  kFormBlocks = 4,          // domain blocks
  kForms = 5
};

// Which form the iterations of one kind (with or without face tallies) take.
// Measured, not guessed, where there are candidates: the first iteration runs
// the planner's choice (not timed: first launches), the next ones a candidate
// each, timed by the step's events, the others the fastest.  Every form gives
// the same tallies bit for bit, so the search changes only the time.
struct FormSearch {
  std::vector<int> cand;    // forms to time (none: the planner's choice stays)
  int def = kFormTiles256;  // the planner's choice
  int form = -1;            // the fastest, once known
  float ms[kForms] = {-1.f, -1.f, -1.f, -1.f, -1.f};
  int rounds = 1;           // iterations timed per candidate, in turn
  size_t next = 0;          // iterations timed
  bool warm = false;        // the first iteration has run
  bool timing = false;      // the iteration in flight is a candidate's

  // the form of the next iteration (ready: it is like those to come)
  int pick(bool ready = true)
  {
    timing = false;
    if (form >= 0) return form;
    if (cand.empty()) return def;
    if (!warm || !ready) {
      warm = true;
      return def;
    }
    timing = true;
    return cand[next % cand.size()];
  }
  // after it, with its time; whether that settled the choice
  bool record(float t)
  {
    if (!timing) return false;
    timing = false;
    float &sum = ms[cand[next % cand.size()]];
    sum = (next < cand.size() ? 0.f : sum) + t / static_cast<float>(rounds);
    if (++next < cand.size() * rounds) return false;
    form = cand[0];
    for (int f : cand)
      if (ms[f] < ms[form]) form = f;
    return true;
  }
  // the form kept, or -1 while it is searched
  int kept() const { return form >= 0 ? form : cand.empty() ? def : -1; }
};

// Iterations without face tallies: the tile march resolves long segments in
// closed form and sends few tallies out of its windows, so blocks can only win
// on short ones, and where the line lies depends on how evenly the tiles share
// the work (two materials side by side, free path 10 cells, ratio 20, 60 flights
// per emitter: 192 x 192 cells 1.14 ms by blocks against 0.88, 256 x 256 1.72
// against 3.50, 262 x 262 1.80 against 1.84).  So both are timed where blocks may
// win: half of the flights on paths below kQuietCells, and enough of them for a
// block (of 1700 drawn problems blocks were more than 7% faster in none that
// this leaves out).  The first iterations run by blocks where they mostly win:
// half of the flights on paths below kQuietFirst, kQuietFlights in all.
constexpr double kQuietCells = 24.0, kQuietPerBlock = 5e3;
constexpr double kQuietFirst = 16.0, kQuietFlights = 3e6;

// the share of the bands on paths (in cells) below `cells`
inline double short_paths(const std::vector<double> &lam, double cells)
{
  double n = 0.0;
  for (double l : lam) n += l < cells ? 1.0 : 0.0;
  return n / static_cast<double>(lam.size());
}
// lam: each band's free path in cells (a gray problem: its only one); flights:
// of each band; T: blocks of all bands
inline bool quiet_blocks(const std::vector<double> &lam, double flights, int T)
{
  return short_paths(lam, kQuietCells) >= 0.5 &&
         flights * static_cast<double>(lam.size()) >= kQuietPerBlock * T;
}
inline bool quiet_blocks_first(const std::vector<double> &lam, double flights)
{
  return short_paths(lam, kQuietFirst) >= 0.5 &&
         flights * static_cast<double>(lam.size()) >= kQuietFlights;
}

}  // namespace iugkp
