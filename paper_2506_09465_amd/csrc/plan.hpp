// plan.hpp -- rules of the host's launch planning, plain C++ (no device code).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace iugkp {

// A tile's particles are split over several workgroups where the tiles alone
// leave compute units idle (a 100-cell film has 15): up to kSplitTarget
// workgroups per launch (two per compute unit), kSplitTargetMore where their
// shares are heavy (of half a particle per word of LDS window, which every
// workgroup clears and flushes: 192 x 192 cells, 60 particles per emitter 111 us
// against 121, with 15 61 against 81) and with null collisions, whose chains
// differ in length; of at least kSplitMin particles (one per lane) and of one per
// kSplitWords words.  Where the tiles fit the device at once, so do their shares:
// a second round of workgroups waits for the first (164 x 161 cells, 286
// workgroups of a CU's LDS each, 47 us against 35 unsplit; with null collisions a
// second round evens the chains out: 115 x 190, path 1.3 cells, ratio 180, 3.8
// ms against 5.5 with the limit; 199 x 74, path 350, ratio 23, with face tallies
// 0.50 against 0.80).
// Measured: film of 100 cells, 1e5 particles, particle step 658 -> 30 us (512 /
// 2048 particles at least: 27 / 38 us, but the two-time film's solve 1.85 ms
// against 2.2 / 3.0); 61 x 45 cells, 3e5 particles 104 -> 46 us; 128 x 100 with
// null collisions, 1e6 particles 1188 -> 729 us (one particle per 4 or 2 words:
// 806 / 1182).  Cavities of 24 .. 400 cells a side without null collisions,
// time against unsplit tiles, geometric mean and worst: without face tallies
// 0.89 and 1.25 (target 1024 and no limit: 0.92 and 1.42), with them 0.93 and
// 1.08 (0.94 and 1.24).
constexpr int kSplitTarget = 512, kSplitTargetMore = 1024;
constexpr double kSplitHeavy = 0.5;
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
  const bool more = has_null || all * K >= kSplitTargetMore * kSplitHeavy * static_cast<double>(lds_words);
  const int target = std::max(1, (more ? kSplitTargetMore : kSplitTarget) / K);
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
  // whether a later iteration may run in form f
  bool may_run(int f) const
  {
    return kept() >= 0 ? kept() == f : def == f || std::find(cand.begin(), cand.end(), f) != cand.end();
  }
};

// An iteration of fewer flights takes a few ms in any form, and its longest chain
// of null collisions sets its time (125 x 66 cells, ratio 187, by tiles 0.36 to
// 0.86 ms from one to the next): its forms are timed three times over.
constexpr double kFewFlights = 3e6;
inline int timed_rounds(double flights) { return flights < kFewFlights ? 3 : 1; }

// Iterations without face tallies: the tile march resolves long segments in
// closed form and sends few tallies out of its windows, so blocks can only win
// on short ones, and where the line lies depends on how evenly the tiles share
// the work (two materials side by side, free path 10 cells, ratio 20, 60 flights
// per emitter: 192 x 192 cells 1.14 ms by blocks against 0.88, 256 x 256 1.72
// against 3.50, 262 x 262 1.80 against 1.84).  So both are timed where blocks may
// win: half of the flights on paths below kQuietCells, and enough of them for a
// block (of 1700 drawn problems blocks were more than 7% faster in none that
// this leaves out).  The first iterations run by blocks where they mostly win:
// half of the flights on paths below kQuietFirst, kFewFlights in all.
constexpr double kQuietCells = 24.0, kQuietPerBlock = 5e3;
constexpr double kQuietFirst = 16.0;

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
         flights * static_cast<double>(lam.size()) >= kFewFlights;
}

// Frequency bands, iterations with face tallies: blocks, row stripes for the bands
// with long paths and tiles for the others, or tiles.  Stripes where every band
// has long paths (stripes) and blocks would be many rounds of few flights (two
// bands of 376 x 97 cells, 10 per emitter: 0.39 ms against 0.78 by blocks; in
// fewer rounds blocks, 72 x 58: 0.10 against 0.20).  Tiles where a few rounds of
// blocks are nearly empty (8 bands of 43 x 215, 1.5e4 flights a block: 0.83 ms
// against 1.45 by blocks and 0.89 with stripes; 376 x 376 in ten rounds 1.67
// against 1.23).  Over 127 drawn problems 1.6% from the fastest of the three in
// the geometric mean, always blocks 8%, never blocks 54%.  With few flights a
// block the lines are not sharp (40 bands of 78 x 179, 1.9e4 a block, ratio 3:
// 0.41 ms by blocks, 0.59 by tiles): there the forms are timed, at little cost;
// with kFewFlights or more, blocks were the fastest in every problem whose bands
// do not all have long paths (where they do, also with more flights a block: two
// bands of 290 x 34, 1.5e5 a block, 0.31 ms with stripes, 0.41 by blocks).
constexpr int kBandRounds = 4;
constexpr double kBandPerBlock = 2e4, kBandPerBlockTimed = 1e5;

// flights: of all bands; T: blocks of all bands
inline bool bands_timed(bool stripes, double flights, int T)
{
  const bool few = flights < kBandPerBlockTimed * T;
  return stripes ? few || flights < kFewFlights : few && flights < kFewFlights;
}
inline int bands_form(bool stripes, double flights, int T, int rounds)
{
  if (stripes && rounds >= kBandRounds && flights < kBandPerBlockTimed * T) return kFormStripes;
  return rounds >= kBandRounds || flights >= kBandPerBlock * T ? kFormBlocks : kFormTiles256;
}

// ---------------------------------------------------------------------------
// The banded multigrid's first level in LDS.  With more levels there its group
// passes fewer barriers, but the levels' rows leave less LDS for the windows of a
// band phase; a window more in the longest phase (the finest prolongation) costs a
// solve about as much as a level fewer in LDS (460 x 460 cells, the first level
// that may be / the next: 13 windows and 2, 3.46 / 1.99 ms; 467 x 664: 3 and 2,
// 2.83 / 2.96).  So the level is taken with the fewest of both together, of at most
// kMgBandLevels, and where even that is more than kMgBandCost, or kMgBandCostFew on
// a group that is small, the phases run without bands (banded / not: 720 x 20 cells
// with 3 levels and 3 windows more 1.71 / 1.11 ms, 720 x 128 with 1 and 3 2.14 /
// 1.85, 600 x 100 with 2 and 1 1.48 / 1.42; 648 x 256 with 2 and 2 2.02 / 2.35).
// ---------------------------------------------------------------------------
constexpr int kMgBandLevels = 3, kMgBandCost = 5, kMgBandCostFew = 3, kMgBandFewBlocks = 400;

// windows[k]: of the finest prolongation, with k levels fewer in LDS than could be
// there, 0 where no row fits; blocks: of the mesh.  The k to take, -1 for no bands.
inline int mg_band_level(const int *windows, int n, int blocks)
{
  int k = -1, cost = 1 + (blocks <= kMgBandFewBlocks ? kMgBandCostFew : kMgBandCost);
  for (int i = 0; i < n; ++i)
    if (windows[i] > 0 && windows[i] - 1 + i < cost) {
      k = i;
      cost = windows[i] - 1 + i;
    }
  return k;
}

// ---------------------------------------------------------------------------
// The workgroups of a CG solve's group, elected on the device (elect_group in
// kernels.hpp): what a workgroup proposes, and who belongs to the group.  The
// first proposal holds.
// ---------------------------------------------------------------------------
constexpr unsigned kElectSpread = 0x100u, kElectFailed = 0x200u, kElectFewer = 0x10000u;
constexpr unsigned long long kElectTicks = 2000;         // 20 us of the 100 MHz clock
constexpr unsigned long long kElectPatience = 1000000;   // 10 ms

// A workgroup's proposal after `waited` ticks, 0 for none: the ta-th to arrive
// anywhere and the tx-th on its XCD xcc, `arrivals` of a group of G being there.
// may_xcd: enough workgroups are launched for a whole group on one XCD; fewer:
// any number of workgroups can run the solve.
constexpr unsigned elect_proposal(unsigned xcc, int ta, int tx, int G, bool may_xcd, bool fewer,
                                  unsigned long long waited, unsigned arrivals)
{
  if (tx == G - 1) return 1u + xcc;
  if (!may_xcd && ta == G - 1) return kElectSpread;
  if (waited > kElectTicks && arrivals >= static_cast<unsigned>(G)) return kElectSpread;
  if (fewer && waited > kElectPatience) return kElectFewer + arrivals;
  return 0u;
}
// its rank in the group chosen, -1: it leaves
constexpr int elect_rank(unsigned choice, unsigned xcc, int ta, int tx, int G)
{
  if (choice >= kElectFewer) return ta < static_cast<int>(choice - kElectFewer) ? ta : -1;
  if (choice == kElectSpread) return ta < G ? ta : -1;
  return choice == 1u + xcc && tx < G ? tx : -1;
}
constexpr int elect_size(unsigned choice, int G)
{
  return choice >= kElectFewer ? static_cast<int>(choice - kElectFewer) : G;
}

// ---------------------------------------------------------------------------
// Domain blocks (blocks.hpp): how a mesh is cut, and what the rounds can need.
// ---------------------------------------------------------------------------
constexpr int kChunk = 64;                 // records per chunk
constexpr int kRecBytes = 64;
constexpr int kOpenChunks = 4;             // partly filled chunks a unit can leave
constexpr int kUnitChunksMax = 256;        // chunks of one unit of work
constexpr int kUnitChunksMin = 32;         // two per wavefront, fewer where that leaves CUs idle
constexpr int kUnitChunksLow = 8;          // (256 x 256, 3e6 flights 2.25 -> 2.01 ms)
constexpr int kBlocksMax = 4096;           // blocks of a launch, all bands
constexpr uint32_t kChunksMax = 1u << 25;  // (a list entry holds 25 bits of a chunk's number)
constexpr size_t kBlockStaticLds = 6144;   // static LDS of the march, rounded up
// units of work per round: more balance better, fewer pay for fewer LDS images
// (512 / 1024 / 2048 units: two-material square 30.5 / 31.5 / 33.0 ms,
// expected-value cavity 8.6 / 8.1 / 9.3 ms)
constexpr int kBlockTarget = 512, kBlockTargetEv = 1024;

struct BlockDesc {
  int inst, x0, y0, ex, ey;
  int n_e;                                 // emitters: the block's cells, then its wall faces
  uint32_t base;                           // first chunk of the flights sampled here
  int nb[4];                               // blocks entered at -x, +x, -y, +y
};

struct BlockUnit {
  int t;                                   // block
  uint32_t first, count;                   // chunks of its input
  uint32_t slab, cap;                      // output chunks [slab, slab + cap)
};

// chunks of a unit where `total` chunks are to be cut
constexpr uint32_t unit_chunks(uint32_t total, uint32_t target, uint32_t cus)
{
  const uint32_t want = (total + target - 1u) / target, each = (total + cus - 1u) / cus;
  uint32_t lo = each < static_cast<uint32_t>(kUnitChunksMin) ? each : static_cast<uint32_t>(kUnitChunksMin);
  if (lo < static_cast<uint32_t>(kUnitChunksLow)) lo = static_cast<uint32_t>(kUnitChunksLow);
  const uint32_t n = want > lo ? want : lo;
  return n < static_cast<uint32_t>(kUnitChunksMax) ? n : static_cast<uint32_t>(kUnitChunksMax);
}

// LDS words of a block's tallies, and of its acceptance ratios rounded to 32
// bits (analog flights with null collisions)
constexpr int block_words(int ex, int ey, int has_w, int faces, int ratios)
{
  return ex * ey * (has_w ? 2 : 1) + (faces ? ex * (ey + 1) : 0) + 2 * (ex + ey) +
         (ratios ? (ex * ey + 1) / 2 : 0);
}

struct BlockPlan {
  int T = 0;                               // blocks of all bands (0: no blocks)
  int rounds = 0, target = 0;
  bool faces = false;                      // the LDS has room for y-face tallies
  size_t lds = 0;                          // bytes of a workgroup's dynamic LDS
  std::vector<BlockDesc> blk;              // [T + 1] (the last: the number of sampled chunks)
  std::vector<BlockUnit> units;            // round 0's
  size_t n_units = 0, n_chunks = 0;        // most units of a round, most output chunks
  // device memory of the records, which is nearly all of it
  size_t record_bytes() const { return (rounds > 1 ? 2 : 1) * n_chunks * (kChunk * kRecBytes); }
};

// The records (128 bytes a flight) may take an eighth of the device's free
// memory: they stay for the handle's life beside its other arrays, other
// handles and the caller's own.
inline bool records_fit(const BlockPlan &p, size_t free_bytes)
{
  return p.record_bytes() <= free_bytes / 8;
}

// The mesh of each of K bands cut into blocks whose tallies fit a workgroup's
// LDS (the fewest rounds, then the fewest blocks), round 0's units of work for N
// flights per emitter, and the most that a later round can need.  No blocks
// beyond kBlocksMax of them or kChunksMax chunks.
inline BlockPlan plan_block_step(int nx, int ny, int K, uint32_t N, bool has_null, bool faces,
                                 bool rays, int n_cu, size_t lds_max)
{
  auto cdiv = [](int a, int b) { return (a + b - 1) / b; };
  const int ratios = has_null && !rays;
  const int words = static_cast<int>((lds_max - kBlockStaticLds) / 8);
  int nbx = 0, nby = 0;
  for (int sum = 2; nbx == 0 && sum <= nx + ny; ++sum)
    for (int x = 1; x < sum; ++x) {
      const int y = sum - x;
      if (x > nx || y > ny) continue;
      if (block_words(cdiv(nx, x), cdiv(ny, y), has_null, faces, ratios) > words) continue;
      if (nbx == 0 || x * y < nbx * nby) {
        nbx = x;
        nby = y;
      }
    }
  const int T1 = nbx * nby;
  BlockPlan p;
  if (nbx == 0 || T1 > kBlocksMax / K) return p;
  const int T = K * T1;
  p.target = rays ? kBlockTargetEv : kBlockTarget;
  const double flights = (static_cast<double>(nx) * ny + 2.0 * (nx + ny)) * N * K;
  // chunks of a unit of round 0
  const double share = static_cast<double>(
      unit_chunks(static_cast<uint32_t>(std::min(flights / kChunk + T, 4e9)),
                  static_cast<uint32_t>(p.target), static_cast<uint32_t>(n_cu)));
  p.blk.resize(static_cast<size_t>(T) + 1);
  unsigned long long slab = 0, base = 0;
  int ex_max = 1, ey_max = 1;
  for (int k = 0; k < K; ++k)
    for (int by = 0; by < nby; ++by)
      for (int bx = 0; bx < nbx; ++bx) {
        const int t = k * T1 + by * nbx + bx;
        BlockDesc &d = p.blk[t];
        d.inst = k;
        d.x0 = static_cast<int>(static_cast<long long>(nx) * bx / nbx);
        d.y0 = static_cast<int>(static_cast<long long>(ny) * by / nby);
        d.ex = static_cast<int>(static_cast<long long>(nx) * (bx + 1) / nbx) - d.x0;
        d.ey = static_cast<int>(static_cast<long long>(ny) * (by + 1) / nby) - d.y0;
        ex_max = std::max(ex_max, d.ex);
        ey_max = std::max(ey_max, d.ey);
        d.n_e = d.ex * d.ey + (bx == 0 ? d.ey : 0) + (bx == nbx - 1 ? d.ey : 0) +
                (by == 0 ? d.ex : 0) + (by == nby - 1 ? d.ex : 0);
        d.nb[0] = bx > 0 ? t - 1 : t;               // (the mesh's edge: never entered)
        d.nb[1] = bx < nbx - 1 ? t + 1 : t;
        d.nb[2] = by > 0 ? t - nbx : t;
        d.nb[3] = by < nby - 1 ? t + nbx : t;
        const unsigned long long P = static_cast<unsigned long long>(d.n_e) * N;
        const unsigned long long nc = (P + kChunk - 1) / kChunk;
        d.base = static_cast<uint32_t>(base);
        base += nc;
        if (base >= kChunksMax) return BlockPlan{};
        const unsigned long long parts =
            static_cast<unsigned long long>(std::ceil(static_cast<double>(nc) / share));
        for (unsigned long long i = 0; i < parts; ++i) {
          BlockUnit u;
          u.t = t;
          u.first = static_cast<uint32_t>(nc * i / parts);
          u.count = static_cast<uint32_t>(nc * (i + 1) / parts) - u.first;
          u.cap = u.count + kOpenChunks;
          u.slab = static_cast<uint32_t>(slab);
          slab += u.cap;
          p.units.push_back(u);
        }
      }
  p.blk.back().base = static_cast<uint32_t>(base);
  // most units of a round, and most chunks: at most one chunk per 64 flights
  // and kOpenChunks partly filled ones per unit of the round that wrote them,
  // again kOpenChunks per unit of the round that reads them
  const double full = static_cast<double>(base) + 1.0;
  const double u_max =
      std::max({static_cast<double>(p.units.size()), static_cast<double>(p.target + T),
                (full / kUnitChunksMax + T + 1.0) /
                    (1.0 - static_cast<double>(kOpenChunks) / kUnitChunksMax)});
  const double chunks = std::max(static_cast<double>(slab), full + 2.0 * kOpenChunks * (u_max + 1.0));
  if (chunks >= static_cast<double>(kChunksMax)) return BlockPlan{};
  p.n_units = static_cast<size_t>(u_max) + 1;
  p.n_chunks = static_cast<size_t>(chunks) + 1;
  p.rounds = nbx + nby - 1;
  p.faces = faces;
  p.lds = static_cast<size_t>(block_words(ex_max, ey_max, has_null, faces, ratios)) * 8;
  p.T = T;
  return p;
}

}  // namespace iugkp
