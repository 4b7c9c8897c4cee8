// blocks.hpp -- the particle step by domain blocks: flights hop between
// workgroups instead of tallying outside their own LDS.
//
// The mesh (of every frequency band) is cut into blocks whose tallies (D, W,
// y faces, wall faces) fit the LDS of one workgroup.  A flight is a 64-byte
// record: block_sample_kernel samples every flight into its start block's
// records, and round r follows the records of each block until the flight ends
// there or enters the next block, whose records of round r + 1 it joins.  A
// flight keeps its direction through null collisions, so it is a straight ray
// and visits at most nbx + nby - 1 blocks: that many rounds end every flight.
// All tallies are integer sums, so the result is the emitter tiles' bit for
// bit.
//
// Why: an emitter tile's window holds the cells around the emitters, and
// flights that go further (expected-value rays, chains of null collisions)
// tally through global atomics, which bound the step (2.1e10 of them a second,
// of the 2.4e10 that random words of a small array take).
// Here every tally is an LDS atomic, and a hop costs 128 bytes of traffic.
//
// Records are kept in chunks of 64 (a wavefront's load), field by field
// (16-byte planes, so that stores and loads are contiguous).  A unit of work is
// (block, range of its chunks); it owns a slab of output chunks sized for its
// input and fills one chunk per neighbour at a time (its wavefronts together:
// with a chunk per wavefront the late rounds' chunks held a few records each).
// Its chunks are listed per neighbour, and between rounds one workgroup sorts
// the lists by block and cuts them into the next round's units
// (block_plan_kernel).  Workgroups claim units until none is left; no workgroup
// waits for another.
#pragma once

#include "plan.hpp"

namespace iugkp {

constexpr int kBlockThreads = 1024;
constexpr int kBlockWaves = kBlockThreads / 64;

struct BlockRun {
  const BlockDesc *blk;                    // [T + 1] (the last: the number of sampled chunks)
  int T;
  uint32_t target, cus;                    // units per round aimed at, compute units
  const BlockUnit *units0;                 // round 0's units
  uint32_t n_units0;
  BlockUnit *units[2];                     // a later round's, by parity
  uint32_t *n_units;                       // [2]
  uint32_t *next;                          // [rounds] units claimed
  uint4 *rec[2];                           // record chunks
  uint32_t *list[2];                       // chunk << 7 | records, per unit and neighbour
  uint32_t *out_n;                         // [unit][4] chunks listed
  uint32_t *seg_off, *seg_pos, *seg_pre;   // a block's input: its list pieces, their first
                                           // chunk in the block's sequence
};

// Walking lanes below which a wavefront serves its others (candidate collision
// and next free path, or the next flight), and faces per lane between two
// looks.  Serving costs about three analog steps (two-material square, 5e7
// flights, 16 / 24 / 32 / 48 lanes: 32.1 / 31.8 / 32.4 / 33.0 ms) and a third of
// an expected-value step (24 / 32 / 40 / 48 lanes: 13.7 / 13.1 / 12.7 / 12.5 ms).
constexpr int kBlockWalkers = 24, kBlockWalkersEv = 48;
constexpr int kBlockSteps = 4;

// One record at position pos of a chunk.
__device__ __forceinline__ void put_record(uint4 *rec, uint32_t chunk, uint32_t pos, double a,
                                           double b, double c, double d, double e, double f, uint4 g)
{
  uint4 *const p = rec + static_cast<size_t>(chunk) * (kChunk * kRecBytes / 16) + pos;
  auto pair = [](double v, double w) {
    return make_uint4(static_cast<uint32_t>(__double2loint(v)), static_cast<uint32_t>(__double2hiint(v)),
                      static_cast<uint32_t>(__double2loint(w)), static_cast<uint32_t>(__double2hiint(w)));
  };
  p[0] = pair(a, b);
  p[kChunk] = pair(c, d);
  p[2 * kChunk] = pair(e, f);
  p[3 * kChunk] = g;
}

// Every flight's start, direction and first free path (analog), a wavefront
// per chunk: sampled beside the walk, a few lanes at a time, it took a third of
// round 0.  Flight p of a block: emitter p mod n_e of its list, index p / n_e.
// Records go to rec[1]; a flight without weight is kept as one of weight 0.
constexpr int kSampleThreads = 256;
template <bool EV>
__global__ __launch_bounds__(kSampleThreads) void block_sample_kernel(const Inst *__restrict__ insts,
                                                                      BlockRun run)
{
  __shared__ unsigned long long s_fl;
  if (threadIdx.x == 0) s_fl = 0;
  __syncthreads();
  const int lane = static_cast<int>(threadIdx.x & 63);
  const unsigned long long total = run.blk[run.T].base;
  const uint32_t g0 = static_cast<uint32_t>(total * blockIdx.x / gridDim.x);
  const uint32_t g1 = static_cast<uint32_t>(total * (blockIdx.x + 1ull) / gridDim.x);
  int t = 0;
  {
    int hi = run.T;                              // last block that starts at or before g0
    while (hi - t > 1) {
      const int mid = (t + hi) >> 1;
      if (run.blk[mid].base <= g0) t = mid;
      else hi = mid;
    }
  }
  uint32_t n_fl = 0;
  for (uint32_t g = g0 + (threadIdx.x >> 6); g < g1; g += kSampleThreads / 64) {
    while (run.blk[t + 1].base <= g) ++t;
    const BlockDesc bd = run.blk[t];
    const Inst &in = insts[bd.inst];
    const Mesh m = in.m;
    const uint32_t slot = in.crn ? in.epoch : in.sc->iter;
    const FlyIn fa = {m, in.lam_min, slot, in.key0, in.key1, 0, in.has_null, in.ratio, in.e_off};
    const uint32_t p = (g - bd.base) * kChunk + static_cast<uint32_t>(lane);
    const uint32_t n_e = static_cast<uint32_t>(bd.n_e), k = p / n_e;
    if (k >= in.N) continue;
    uint32_t i = p - k * n_e, e;
    const uint32_t ex = static_cast<uint32_t>(bd.ex), ey = static_cast<uint32_t>(bd.ey);
    if (i < ex * ey) {
      const uint32_t r = i / ex;
      e = static_cast<uint32_t>((bd.y0 + static_cast<int>(r)) * m.nx + bd.x0) + (i - r * ex);
    } else {
      // its wall faces: left, right, bottom, top
      i -= ex * ey;
      const uint32_t wl = bd.x0 == 0 ? ey : 0u, wr = bd.x0 + bd.ex == m.nx ? ey : 0u;
      const uint32_t wb = bd.y0 == 0 ? ex : 0u;
      int f;
      if (i < wl) f = bd.y0 + static_cast<int>(i);
      else if (i < wl + wr) f = m.ny + bd.y0 + static_cast<int>(i - wl);
      else if (i < wl + wr + wb) f = 2 * m.ny + bd.x0 + static_cast<int>(i - wl - wr);
      else f = 2 * m.ny + m.nx + bd.x0 + static_cast<int>(i - wl - wr - wb);
      e = static_cast<uint32_t>(m.n_cells + f);
    }
    const long long q = in.base[e] + ((k < in.rem[e]) ? 1 : 0);
    if (q != 0) ++n_fl;
    int ix, iy;
    double x0, y0, sx, sy;
    sample_particle(fa, e, k, ix, iy, x0, y0, sx, sy);
    const uint32_t cell = static_cast<uint32_t>(ix) | (static_cast<uint32_t>(iy) << 16);
    if constexpr (EV) {
      put_record(run.rec[1], g, lane, x0, y0, sx, sy, 0.0, 0.0,
                 make_uint4(static_cast<uint32_t>(q),
                            static_cast<uint32_t>(static_cast<unsigned long long>(q) >> 32), cell, 0u));
    } else {
      const double2 us = draw2(2u, k, e + fa.e_off, slot, fa.key0, fa.key1);
      const double ell = -(fa.lam_min * log_own(1.0 - us.x));
      put_record(run.rec[1], g, lane, x0, y0, sx, sy, ell, __longlong_as_double(q),
                 make_uint4(e, k, 0u, cell));
    }
  }
  if (n_fl) atomicAdd(&s_fl, static_cast<unsigned long long>(n_fl));
  __syncthreads();
  // (a ray, or an analog flight's first free path, is one segment)
  if (threadIdx.x == 0 && s_fl) {
    atomicAdd(&insts[0].sc->flights, s_fl);
    atomicAdd(&insts[0].sc->segments, s_fl);
  }
}

template <bool EV>
__global__ __launch_bounds__(kBlockThreads) void block_march_kernel(const Inst *__restrict__ insts,
                                                                    BlockRun run, int round,
                                                                    int faces_mode)
{
  extern __shared__ long long lds_words[];
  __shared__ unsigned long long s_cnt[2];
  __shared__ uint32_t s_unit, s_next, s_alloc;
  __shared__ uint32_t s_ent[kUnitChunksMax];        // the unit's chunks
  __shared__ uint32_t s_out[4];                     // records written per neighbour, and
  __shared__ uint32_t s_map[4][kUnitChunksMax + 1]; // the chunks that hold them (1 + chunk; 0: none yet)
  enum : int { kIdle = 0, kWalk = 1, kEnd = 2, kExit = 3, kLeave = 4, kDraw = 5 };
  const int par = round & 1;
  const uint32_t n_units = round == 0 ? run.n_units0 : run.n_units[par];
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63;
  const unsigned long long below = (1ull << lane) - 1ull;
  auto uni = [](uint32_t v) { return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v))); };
  for (;;) {
    if (tid == 0) s_unit = atomicAdd(&run.next[round], 1u);
    __syncthreads();
    const uint32_t unit = uni(s_unit);
    if (unit >= n_units) return;
    const BlockUnit un = round == 0 ? run.units0[unit] : run.units[par][unit];
    const BlockDesc bd = run.blk[un.t];
    const Inst &in = insts[bd.inst];
    const Mesh m = in.m;
    const int has_null = in.has_null, faces = faces_mode;
    const int bx0 = bd.x0, by0 = bd.y0, ex = bd.ex, ey = bd.ey;
    long long *const lD = lds_words;
    long long *const lW = lD + ex * ey;
    long long *const lY = lW + (has_null ? ex * ey : 0);
    long long *const lB = lY + (faces ? ex * (ey + 1) : 0);
    const int words = block_words(ex, ey, has_null, faces, 0);
    float *const lR = reinterpret_cast<float *>(lds_words + words);
    for (int i = tid; i < words; i += kBlockThreads) lds_words[i] = 0;
    if (!EV && has_null)
      for (int i = tid; i < ex * ey; i += kBlockThreads) {
        const int r = i / ex;
        lR[i] = static_cast<float>(in.ratio[(by0 + r) * m.nx + bx0 + (i - r * ex)]);
      }
    for (int i = tid; i < 4 * (kUnitChunksMax + 1); i += kBlockThreads) (&s_map[0][0])[i] = 0;
    if (tid < 2) s_cnt[tid] = 0;
    if (tid < 4) s_out[tid] = 0;
    if (tid == 0) {
      s_next = 0;
      s_alloc = 0;
    }
    if (round == 0) {
      const uint32_t last = run.blk[un.t + 1].base - bd.base - 1u;
      const uint32_t rest = static_cast<uint32_t>(static_cast<unsigned long long>(bd.n_e) * in.N -
                                                  static_cast<unsigned long long>(last) * kChunk);
      for (uint32_t i = tid; i < un.count; i += kBlockThreads) {
        const uint32_t p = un.first + i;
        s_ent[i] = ((bd.base + p) << 7) | (p == last ? rest : static_cast<uint32_t>(kChunk));
      }
    } else {
      // the unit's chunks: position p of the block's input sequence
      const uint32_t g0 = run.seg_off[un.t], g1 = run.seg_off[un.t + 1];
      for (uint32_t i = tid; i < un.count; i += kBlockThreads) {
        const uint32_t p = un.first + i;
        uint32_t lo = g0, hi = g1;                  // last piece that starts at or before p
        while (hi - lo > 1) {
          const uint32_t mid = (lo + hi) >> 1;
          if (run.seg_pre[mid] <= p) lo = mid;
          else hi = mid;
        }
        s_ent[i] = run.list[par ^ 1][run.seg_pos[lo] + (p - run.seg_pre[lo])];
      }
    }
    __syncthreads();
    const double lam_min = in.lam_min, dx = m.dx, dy = m.dy;
    const uint32_t slot = in.crn ? in.epoch : in.sc->iter;
    const uint32_t e_off = in.e_off, key0 = in.key0, key1 = in.key1;
    const double *const ratio = in.ratio;
    const double inv_lam = 1.0 / lam_min;           // = ratio / lambda_min where ratio is 1
    auto add = [&](long long *p, long long v) {
      atomicAdd(reinterpret_cast<unsigned long long *>(p), static_cast<unsigned long long>(v));
    };

    // the lane's flight: next faces ahead (as doubles) and their times, faces to
    // cross until it leaves the block, its cell in the block's arrays
    int st = kIdle, dir = 0;
    uint32_t e = 0, k = 0, j = 0;
    long long q = 0;
    double x0 = 0.0, y0 = 0.0, sx = 0.0, sy = 0.0, inv_sx = 0.0, inv_sy = 0.0;
    double kx = 0.0, ky = 0.0, tx = 0.0, ty = 0.0;
    int rx = 0, ry = 0, c = 0;
    double ell = 0.0, uacc = 0.0;                   // analog: free path, acceptance draw
    double T = 0.0, tprev = 0.0, surv = 1.0;        // expected: optical depth, last face, e^-T
    long long S = 0;
    bool fresh = false;                             // needs a new free path
    unsigned long long n_seg = 0;
    uint32_t n_cross = 0;
    int bad = 0;
    // the wavefront's input chunk
    bool dry = false;
    uint32_t c_id = 0, c_pos = 0, c_cnt = 0;
    auto cell_x = [&]() { return static_cast<int>(kx) - (sx > 0.0 ? 1 : 0); };
    auto cell_y = [&]() { return static_cast<int>(ky) - (sy > 0.0 ? 1 : 0); };
    auto store_rec = [&](uint32_t chunk, uint32_t pos) {
      const uint32_t cell = static_cast<uint32_t>(cell_x()) | (static_cast<uint32_t>(cell_y()) << 16);
      if constexpr (EV)
        put_record(run.rec[par], chunk, pos, x0, y0, sx, sy, T, tprev,
                   make_uint4(static_cast<uint32_t>(q),
                              static_cast<uint32_t>(static_cast<unsigned long long>(q) >> 32), cell, 0u));
      else
        put_record(run.rec[par], chunk, pos, x0, y0, sx, sy, ell, __longlong_as_double(q),
                   make_uint4(e, k, j, cell));
    };
    uint4 ra = {}, rb = {}, rc = {}, rd = {};       // a record on its way in
    auto load_rec = [&](uint32_t chunk, uint32_t pos) {
      const uint4 *const p = run.rec[par ^ 1] + static_cast<size_t>(chunk) * (kChunk * kRecBytes / 16) + pos;
      ra = p[0];
      rb = p[kChunk];
      rc = p[2 * kChunk];
      rd = p[3 * kChunk];
    };
    auto take_rec = [&](int &ix, int &iy) {
      auto dbl = [](uint32_t lo, uint32_t hi) { return __hiloint2double(static_cast<int>(hi), static_cast<int>(lo)); };
      x0 = dbl(ra.x, ra.y);
      y0 = dbl(ra.z, ra.w);
      sx = dbl(rb.x, rb.y);
      sy = dbl(rb.z, rb.w);
      uint32_t cell;
      if constexpr (EV) {
        T = dbl(rc.x, rc.y);
        tprev = dbl(rc.z, rc.w);
        q = static_cast<long long>((static_cast<unsigned long long>(rd.y) << 32) | rd.x);
        cell = rd.z;
      } else {
        ell = dbl(rc.x, rc.y);
        q = __double_as_longlong(dbl(rc.z, rc.w));
        e = rd.x;
        k = rd.y;
        j = rd.z;
        cell = rd.w;
      }
      ix = static_cast<int>(cell & 0xffffu);
      iy = static_cast<int>(cell >> 16);
    };
    // from a flight in cell (ix, iy): reciprocals, faces ahead, way to the edge
    auto enter = [&](int ix, int iy) {
      inv_sx = (sx != 0.0) ? 1.0 / sx : 0.0;
      inv_sy = (sy != 0.0) ? 1.0 / sy : 0.0;
      const int lx = ix - bx0, ly = iy - by0;
      kx = static_cast<double>(sx > 0.0 ? ix + 1 : ix);
      ky = static_cast<double>(sy > 0.0 ? iy + 1 : iy);
      rx = sx > 0.0 ? ex - lx : sx < 0.0 ? lx + 1 : 0x7fffffff;
      ry = sy > 0.0 ? ey - ly : sy < 0.0 ? ly + 1 : 0x7fffffff;
      c = ly * ex + lx;
    };

    for (;;) {
      if (__popcll(__ballot(st == kWalk)) < (EV ? kBlockWalkersEv : kBlockWalkers)) {
        // ---- flights at the block's edge: absorbed by a wall face, or leaving
        if (__ballot(st == kExit)) {
          if (st == kExit) {
            if (rx == 0) {
              const bool up = sx > 0.0;
              if (up ? bx0 + ex == m.nx : bx0 == 0) {
                add(&lB[(up ? ey : 0) + cell_y() - by0], EV ? S : q);
                st = kIdle;
              } else {
                dir = up ? 1 : 0;
                st = kLeave;
              }
            } else {
              const bool up = sy > 0.0;
              if (up ? by0 + ey == m.ny : by0 == 0) {
                add(&lB[2 * ey + (up ? ex : 0) + cell_x() - bx0], EV ? S : q);
                st = kIdle;
              } else {
                dir = up ? 3 : 2;
                st = kLeave;
              }
            }
          }
        }
        // ---- candidate collisions
        if constexpr (!EV) {
          if (st == kEnd) {
            const int ix = cell_x(), iy = cell_y();
            bool real = true;
            if (has_null) {
              add(&lW[c], q);
              // accept with probability sigma / sigma_max = tau_min / tau_c: both
              // rounded to 32 bits decide it unless those are equal (rounding keeps
              // the order)
              const float uf = static_cast<float>(uacc), rf = lR[c];
              real = uf < rf;
              if (uf == rf) real = uacc < ratio[ix + m.nx * iy];
              real = real || j == kMaxSegments - 1;
            }
            if (real) {
              add(&lD[c], q);
              st = kIdle;
            } else {
              // null collision: keep the direction, restart from the stopping point
              x0 = clamp_to(x0 + ell * sx, static_cast<double>(ix) * dx, static_cast<double>(ix + 1) * dx);
              y0 = clamp_to(y0 + ell * sy, static_cast<double>(iy) * dy, static_cast<double>(iy + 1) * dy);
              ++j;
              fresh = true;
              st = kDraw;
            }
          }
        }
        // ---- idle and leaving lanes load the unit's next flights; the leaving
        // ones store theirs behind those loads (memory operations complete in
        // order: a load behind the stores would wait for them)
        bool got = false;
        for (;;) {
          const bool wants = (st == kIdle || st == kLeave) && !got;
          const unsigned long long want = __ballot(wants);
          if (!want || dry) break;
          const uint32_t rank = static_cast<uint32_t>(__popcll(want & below));
          const uint32_t n = static_cast<uint32_t>(__popcll(want));
          if (c_pos == c_cnt) {
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&s_next, 1u);
            at = uni(at);
            if (at >= un.count) {
              dry = true;
              break;
            }
            const uint32_t ent = uni(s_ent[at]);
            c_id = ent >> 7;
            c_cnt = ent & 127u;
            c_pos = 0;
          }
          if (wants && rank < c_cnt - c_pos) {
            load_rec(c_id, c_pos + rank);
            got = true;
          }
          c_pos = min(c_cnt, c_pos + n);
        }
        const bool mine = st == kLeave;
        if (__ballot(mine)) {
          // places [v, v + n) of each neighbour's sequence, claimed by lanes 0 to
          // 3; whoever takes a chunk's first place opens the chunk, the others
          // wait for that (the opener waits for nobody in between)
          unsigned long long mask = 0;
          uint32_t n = 0;
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            const unsigned long long md = __ballot(mine && dir == d);
            mask = dir == d ? md : mask;
            n = lane == d ? static_cast<uint32_t>(__popcll(md)) : n;
          }
          uint32_t v = 0;
          if (lane < 4 && n) {
            v = atomicAdd(&s_out[lane], n);
            const uint32_t last = (v + n - 1u) / kChunk;
            const uint32_t opens = (v + kChunk - 1u) / kChunk;
            if (opens <= last)
              __hip_atomic_store(&s_map[lane][last], 1u + un.slab + atomicAdd(&s_alloc, 1u),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
          const uint32_t at = static_cast<uint32_t>(__shfl(static_cast<int>(v), dir, 64)) +
                              static_cast<uint32_t>(__popcll(mask & below));
          uint32_t id = 1u;
          do {
            if (mine)
              id = __hip_atomic_load(&s_map[dir][at / kChunk], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_WORKGROUP);
          } while (__any(id == 0u));
          if (mine) {
            store_rec(id - 1u, at % kChunk);
            st = kIdle;
          }
        }
        if (got) {
          int ix, iy;
          take_rec(ix, iy);
          enter(ix, iy);
          fresh = false;
          st = q != 0 ? kDraw : kIdle;
          if constexpr (EV) {
            surv = expm_own(T);
            S = static_cast<long long>(rint(static_cast<double>(q) * surv));
          }
        }
        // ---- free paths: a new one, or the acceptance draw of the one under way
        if (st == kDraw) {
          if constexpr (!EV) {
            const double2 us = draw2(2u + j, k, e + e_off, slot, key0, key1);
            if (fresh) {
              ell = -(lam_min * log_own(1.0 - us.x));
              ++n_seg;
            }
            uacc = us.y;
          }
          tx = (sx != 0.0) ? (kx * dx - x0) * inv_sx : INFINITY;
          ty = (sy != 0.0) ? (ky * dy - y0) * inv_sy : INFINITY;
          st = kWalk;
        }
        if (!__ballot(st == kWalk)) {
          if (dry) break;
          continue;                                 // (every flight loaded had no weight)
        }
      }
      // ---- the walk, a few faces per lane.  Straight-line: both face times are
      // formed anew (the one not crossed comes out the same), and walls and the
      // block's edge are one countdown.
      const double one_x = (sx > 0.0) ? 1.0 : -1.0, one_y = (sy > 0.0) ? 1.0 : -1.0;
      const int step_x = (sx > 0.0) ? 1 : -1, step_y = (sy > 0.0) ? ex : -ex;
      long long *const y_at = lY + (sy > 0.0 ? ex : 0);
      const long long qy = (sy > 0.0) ? q : -q;
#pragma unroll 1
      for (int s = 0; s < kBlockSteps; ++s) {
        if (st == kWalk) {
          const bool along_x = tx <= ty;
          const double tt = along_x ? tx : ty;
          bool go;
          if constexpr (EV) {
            const double qd = static_cast<double>(q);
            auto cand = [&](double w, double r) {
              const double x = w / r;
              if (!(fabs(x) <= 4611686018427387904.0)) {
                bad = 1;
                return;
              }
              const long long wi = static_cast<long long>(rint(x));
              if (wi) add(&lW[c], wi);
            };
            go = tt < INFINITY;
            if (!go) {                              // (no direction in the plane)
              if (S) add(&lD[c], S);
              if (has_null) cand(qd * surv, ratio[cell_x() + m.nx * cell_y()]);
              st = kIdle;
            } else {
              const double r = has_null ? ratio[cell_x() + m.nx * cell_y()] : 1.0;
              const double Tn = T + (tt - tprev) * (has_null ? r / lam_min : inv_lam);
              const double sn = expm_own(Tn);
              const long long Sn = static_cast<long long>(rint(qd * sn));
              if (S != Sn) add(&lD[c], S - Sn);
              if (has_null) cand(qd * (surv - sn), r);
              T = Tn;
              surv = sn;
              S = Sn;
              tprev = tt;
              go = Sn != 0;
              if (!go) st = kIdle;
            }
          } else {
            go = tt < ell;
            if (!go) st = kEnd;
          }
          if (go) {
            ++n_cross;
            if (faces && !along_x) add(&y_at[c], EV ? (sy > 0.0 ? S : -S) : qy);
            kx = kx + (along_x ? one_x : 0.0);
            ky = ky + (along_x ? 0.0 : one_y);
            tx = (sx != 0.0) ? (kx * dx - x0) * inv_sx : INFINITY;
            ty = (sy != 0.0) ? (ky * dy - y0) * inv_sy : INFINITY;
            c += along_x ? step_x : step_y;
            rx -= along_x ? 1 : 0;
            ry -= along_x ? 0 : 1;
            if (rx == 0 || ry == 0) st = kExit;
          }
        }
      }
    }
    if (bad) atomicOr(&in.sc->flags, 2);
    if (n_seg || n_cross) {
      atomicAdd(&s_cnt[0], n_seg);
      atomicAdd(&s_cnt[1], static_cast<unsigned long long>(n_cross));
    }
    __syncthreads();
    // the tallies, row by row (neighbouring lanes update one cache line)
    auto flush = [&](const long long *src, long long *dst, int rows) {
      for (int i = tid; i < rows * ex; i += kBlockThreads) {
        const long long v = src[i];
        if (v == 0) continue;
        const int r = i / ex;
        atom_add(&dst[(by0 + r) * m.nx + bx0 + (i - r * ex)], v);
      }
    };
    flush(lD, in.D, ey);
    if (has_null) flush(lW, in.W, ey);
    if (faces) flush(lY, in.Phiy, ey + 1);
    for (int i = tid; i < 2 * (ex + ey); i += kBlockThreads) {
      const long long v = lB[i];
      if (v == 0) continue;
      const int b = i < ey ? by0 + i
                    : i < 2 * ey ? m.ny + by0 + (i - ey)
                    : i < 2 * ey + ex ? 2 * m.ny + bx0 + (i - 2 * ey)
                                      : 2 * m.ny + m.nx + bx0 + (i - 2 * ey - ex);
      atom_add(&in.B[b], v);
    }
    if (tid < 2 && s_cnt[tid]) atomicAdd(tid == 0 ? &in.sc->segments : &in.sc->crossings, s_cnt[tid]);
    // the chunks written, per neighbour
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const uint32_t n = s_out[d], nc = (n + kChunk - 1u) / kChunk;
      for (uint32_t i = tid; i < nc; i += kBlockThreads)
        run.list[par][4 * static_cast<size_t>(un.slab) + static_cast<size_t>(d) * un.cap + i] =
            ((s_map[d][i] - 1u) << 7) | min(static_cast<uint32_t>(kChunk), n - i * kChunk);
      if (tid == 0) run.out_n[4 * static_cast<size_t>(unit) + d] = nc;
    }
    __syncthreads();
  }
}

// Between rounds, by one workgroup: the listed chunks of the round `round`
// sorted by the block they enter (pieces of one unit's list), and the next
// round's units of at most kUnitChunksMax chunks with their output slabs.
// (dynamic LDS: per block a packed counter, pieces << 32 | chunks, and its
// first piece, unit and slab)
__global__ __launch_bounds__(1024) void block_plan_kernel(BlockRun run, int round)
{
  extern __shared__ unsigned long long plan_lds[];
  __shared__ uint32_t s_sum[3][1024];
  const int par = round & 1, tid = static_cast<int>(threadIdx.x), T = run.T;
  unsigned long long *const cnt = plan_lds;
  const uint32_t n_in = round == 0 ? run.n_units0 : run.n_units[par];
  const BlockUnit *const in = round == 0 ? run.units0 : run.units[par];
  BlockUnit *const out = run.units[par ^ 1];
  for (int t = tid; t < T; t += 1024) cnt[t] = 0;
  __syncthreads();
  for (uint32_t i = tid; i < 4 * n_in; i += 1024) {
    const uint32_t n = run.out_n[i];
    if (n) atomicAdd(&cnt[run.blk[in[i >> 2].t].nb[i & 3]], (1ull << 32) | n);
  }
  __syncthreads();
  // the chunks of all blocks, and a unit's share of them
  const int per = (T + 1023) / 1024, t0 = min(T, tid * per), t1 = min(T, t0 + per);
  uint32_t segs = 0, chunks = 0;
  for (int t = t0; t < t1; ++t) {
    segs += static_cast<uint32_t>(cnt[t] >> 32);
    chunks += static_cast<uint32_t>(cnt[t]);
  }
  // inclusive sums over the threads
  auto scan = [&](uint32_t *s, uint32_t v) -> uint32_t {
    s[tid] = v;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
      const uint32_t o = tid >= d ? s[tid - d] : 0u;
      __syncthreads();
      s[tid] += o;
      __syncthreads();
    }
    return s[tid];
  };
  const uint32_t seg1 = scan(s_sum[0], segs), chunk1 = scan(s_sum[1], chunks);
  const uint32_t total = s_sum[1][1023];
  const uint32_t share = unit_chunks(total, run.target, run.cus);
  uint32_t units = 0;
  for (int t = t0; t < t1; ++t) units += (static_cast<uint32_t>(cnt[t]) + share - 1u) / share;
  const uint32_t unit1 = scan(s_sum[2], units);
  if (tid == 1023) {
    run.n_units[par ^ 1] = unit1;
    run.seg_off[T] = seg1;
  }
  // each block's units; its counter becomes its cursor
  uint32_t sg = seg1 - segs, un = unit1 - units, ch = chunk1 - chunks;
  for (int t = t0; t < t1; ++t) {
    const uint32_t ns = static_cast<uint32_t>(cnt[t] >> 32), nc = static_cast<uint32_t>(cnt[t]);
    run.seg_off[t] = sg;
    cnt[t] = static_cast<unsigned long long>(sg) << 32;
    for (uint32_t c = 0; c < nc; c += share) {
      BlockUnit u;
      u.t = t;
      u.first = c;
      u.count = min(share, nc - c);
      u.slab = ch + c + un * kOpenChunks;
      u.cap = u.count + kOpenChunks;
      out[un] = u;
      ++un;
    }
    sg += ns;
    ch += nc;
  }
  __syncthreads();
  for (uint32_t i = tid; i < 4 * n_in; i += 1024) {
    const uint32_t n = run.out_n[i];
    if (!n) continue;
    const BlockUnit u = in[i >> 2];
    const unsigned long long at = atomicAdd(&cnt[run.blk[u.t].nb[i & 3]], (1ull << 32) | n);
    const uint32_t pos = static_cast<uint32_t>(at >> 32);
    run.seg_pre[pos] = static_cast<uint32_t>(at);
    run.seg_pos[pos] = 4u * u.slab + (i & 3u) * u.cap;
  }
}

}  // namespace iugkp
