// mgcg.hpp -- the Newton system A x = b (Sec. 3.3) solved by conjugate
// gradients preconditioned with one multigrid V-cycle, as one persistent
// cooperative launch.
//
// The hierarchy: level k+1 aggregates 2x2 cells of level k (NX = ceil(nx/2),
// NY = ceil(ny/2)) down to one cell; the coarse operator is the Galerkin
// product P^T A P for the piecewise-constant prolongation P, again a 3/5-point
// operator whose faces sum the fine faces they cover.  The V-cycle: two damped
// Jacobi sweeps (omega 0.8) from zero, the residual summed over each
// aggregate, the coarser V-cycle, the correction scaled by 1.8, two sweeps
// again; the one-cell level is solved exactly.  The CG is the single-reduction
// form of Chronopoulos and Gear with u = M r:
//   x = 0, r = b, u = M r, w = A u, gamma = (r, u), delta = (w, u)
//   repeat: p = u + beta p, s = w + beta s, x += alpha p, r -= alpha s,
//           u = M r, w = A u, gamma' = (r, u), delta = (w, u), rho = (r, r);
//           stop if rho <= tol^2 (b, b); beta = gamma' / gamma,
//           alpha = gamma' / (delta - beta gamma' / alpha)
// Every operation is written in the order the host-side definition fixes, so
// the result does not depend on the launch shape.
//
// Work split.  Levels with more than kMgLocalMax cells ("grid levels") are
// spread over all G workgroups: wave v of the group takes the 256-cell blocks
// v, v + G waves, ... of the level, lane l the cells l + 64 q of a block.  A
// phase reads what other workgroups wrote in the phase before it, behind a
// group barrier, with coherent loads and stores.  Per grid level the descent
// takes two phases (second pre-sweep; residual and restriction, which also
// does the first sweep of the next level) and the ascent two (correction with
// the first post-sweep; second post-sweep, which for a level whose finer
// level has at most one cell per thread is recomputed where that level reads
// it instead).  The remaining small levels run
// redundantly in every workgroup's LDS, so the coarse solve needs no barrier
// of its own and its result is at hand wherever the next grid level needs it.
#pragma once

#include <type_traits>

namespace iugkp {

constexpr double kMgOmega = 0.8;        // damped Jacobi weight
constexpr double kMgScale = 1.8;        // coarse-correction scale
constexpr int kMgLevelsMax = 40;
// Levels up to this size live in LDS: of single solves, whose groups save the
// barriers of a level more (256 x 256 cells 778 us per solve, with 256 856), and
// of a batch's, whose workgroups use the LDS for longer band windows (256 uneven
// cavities: 256 / 512 / 1024 343 / 343 / 374 ms, eight of 128 x 128 68 / 64 / 61).
constexpr int kMgLocalMax = 1024, kMgLocalMaxBatch = 512;

struct MGLevel {
  int nx, ny, n, has_y;
  const double *gx, *gy, *diag;         // operator of the level
  // banded grid levels: its faces with those at the mesh's edge zeroed, and
  // the diagonal's reciprocals (mg_recip); padded for reads past a row's end
  const double *gxz, *gyz, *rd;
  double *b, *xa, *xb, *xd, *e;         // grid levels (level 0: b = r, e = u)
  int lb, lx, lt;                       // LDS levels: offsets (doubles) of the vectors,
  int dg, rdl, lgx, lgy;                // and of the rows (MgLds)
  float rnx;                            // 1 / nx
  int rec;                              // small levels: offset of the records (MgSlot)
  // the banded form, filled by each workgroup of the group: its coarse rows and
  // its rows (level 0: its 256-cell blocks), and the windows each takes
  int c0, c1, r0, r1, wdown, wup;
};

// An LDS level.  Its arrays have rows of S = nx + 1 values, the last one a pad:
// vectors a row of pads before and after too (2D; in 1D one pad before), so
// that cell (ix, iy), at j = ix + iy S + (2D: S, 1D: 1), has its neighbours at
// j +- 1 and j +- S, an absent one a pad.  Pads of x and t hold zeros, and the
// faces at the mesh's edge are stored as zeros: an absent neighbour's term is
// v - 0 * 0, which is v for every v, so no pass tests for the edges.  Rows: the
// diagonal, its reciprocal, the left and the lower face of cell (ix, iy) at ix +
// iy S (its right and upper ones are its neighbours'; the lower faces have a
// row more).
struct MgLds {
  int nx, ny, n, S, lb, lx, lt, dg, rd, gx, gy;
  float rnx;
};
// The levels below the first LDS level, where each has at most a cell per
// thread and there are at most kMgSlots (a solve's iteration runs mostly in
// their passes' latency, so indices stay in registers and every access is at a
// constant from one of them): a record per cell, rows padded as above (a row
// more at the end), pads all zeros: an absent child's residual is 0 as well.
constexpr int kMgSlots = 6;
constexpr int kMgRec = 7;               // dg, rd, left face, lower face, b, x, t
enum : int { kMgDg = 0, kMgRd = 1, kMgGl = 2, kMgGd = 3, kMgB = 4, kMgX = 5, kMgT = 6 };
__host__ __device__ inline int mg_rec_words(int nx, int ny)
{
  return kMgRec * ((ny + 3) * (nx + 1) + 2);
}
struct MgSlot {
  int n, row, crow;                     // cells; words of a row, and of the next level's
  int own;                              // this thread's cell
  int child;                            // the first child of this thread's cell
  int par, parl, pard;                  // its parent, the left one's and the lower one's
};
__host__ __device__ inline int mg_vec_words(int nx, int ny, bool y)
{
  return y ? (ny + 2) * (nx + 1) + 2 : nx + 4;
}
__host__ __device__ inline int mg_row_words(int nx, int ny, bool y)   // per array
{
  return y ? (ny + 1) * (nx + 1) + 2 : nx + 3;
}

struct MGArgs {
  const MGLevel *lv;                    // [L] level table
  int L, Lg;                            // levels; levels 0..Lg-1 are grid levels
  const double *b;                      // right-hand side
  double *x, *p, *s, *w;                // solution and the own-cell CG state
  double *part;                         // [nb][3] block sums of (r, u), (w, u), (r, r)
  double tol2;
  int max_iters;
  unsigned int *barrier;                // zero at the start of the solve, as are
  unsigned int *flags;                  // the group's barrier words
  DevScalars *sc;
  // the banded form (mgband.hpp): second buffers of r and s, and the dynamic
  // LDS layout, [stage0) the coarse result kept across a band phase, then
  // stage_n doubles holding the LDS levels or a band window's staging
  double *r2, *s2;
  int band, stage0, stage_n;
  int zero0, zero_n;                    // the x and t vectors of the LDS levels
  int slots;                            // levels with records, 0: none
};

// Row c of A_k: the diagonal, the four face conductances and the neighbour
// indices, an absent neighbour's index clamped to c itself.  Every load is
// unconditional, so a cell's loads issue together instead of one latency per
// neighbour.
struct MGRow {
  double dg, gl, gr, gd, gu;
  int jl, jr, jd, ju;
  int ix, iy;
  unsigned m;                           // left, right, down, up neighbour present
};

__device__ __forceinline__ void mg_row_index(MGRow &r, int nx, int ny, int ix, int iy)
{
  const int c = iy * nx + ix;
  r.ix = ix;
  r.iy = iy;
  r.m = (ix > 0 ? 1u : 0u) | (ix < nx - 1 ? 2u : 0u) | (iy > 0 ? 4u : 0u) |
        (iy < ny - 1 ? 8u : 0u);
  r.jl = (r.m & 1u) ? c - 1 : c;
  r.jr = (r.m & 2u) ? c + 1 : c;
  r.jd = (r.m & 4u) ? c - nx : c;
  r.ju = (r.m & 8u) ? c + nx : c;
}

__device__ __forceinline__ MGRow mg_row_at(const MGLevel &l, int ix, int iy)
{
  const int nx = l.nx, c = iy * nx + ix;
  MGRow r;
  mg_row_index(r, nx, l.ny, ix, iy);
  const int fx = iy * (nx + 1) + ix;
  r.dg = l.diag[c];
  r.gl = l.gx[fx];
  r.gr = l.gx[fx + 1];
  r.gd = l.gy[l.has_y ? iy * nx + ix : 0];       // (1D: a valid dummy, never used)
  r.gu = l.gy[l.has_y ? (iy + 1) * nx + ix : 0];
  return r;
}

__device__ __forceinline__ MGRow mg_row(const MGLevel &l, int c)
{
  const int iy = c / l.nx;
  return mg_row_at(l, c - iy * l.nx, iy);
}

// The reciprocal with which mg_div divides by d: not a number where d or a
// quotient may leave the range in which its steps are exact.
__host__ __device__ inline double mg_recip(double d)
{
  return (d >= 0x1p-300 && d <= 0x1p300) ? 1.0 / d : __builtin_nan("");
}

// a / d, correctly rounded, from y = mg_recip(d): two Newton corrections of a
// y; the last, from a quotient within one unit of the exact one with the
// remainder exact and y correctly rounded, rounds correctly (Markstein 1990).
// Quotients that are zero, out of range or not finite are divided.  5
// dependent operations instead of a division's 11.
__device__ __forceinline__ double mg_div(double a, double d, double y)
{
  double q = a * y;
  q = __builtin_fma(__builtin_fma(-q, d, a), y, q);
  q = __builtin_fma(__builtin_fma(-q, d, a), y, q);
  const unsigned e = (static_cast<unsigned>(__double2hiint(q)) >> 20) & 0x7ffu;
  if (__builtin_expect(e - 723u > 600u, 0)) q = a / d;
  return q;
}

// A row of the operator with zero faces at the mesh's edge, and the damped
// Jacobi sweep of its cell: v = {v_c, v_l, v_r, v_dn, v_up}, an absent
// neighbour's value 0.
struct MGRowZ {
  double dg, rd, gl, gr, gd, gu;
};
__device__ __forceinline__ double mg_apply_z(const MGRowZ &r, double vc, double vl, double vr,
                                             double vd, double vu)
{
  double acc = r.dg * vc;
  acc = acc - r.gl * vl;
  acc = acc - r.gr * vr;
  acc = acc - r.gd * vd;
  return acc - r.gu * vu;
}
__device__ __forceinline__ double mg_sweep_z(const MGRowZ &r, double b, double vc, double vl,
                                             double vr, double vd, double vu)
{
  const double t = b - mg_apply_z(r, vc, vl, vr, vd, vu);
  return vc + mg_div(kMgOmega * t, r.dg, r.rd);
}
// the sweep from zero
__device__ __forceinline__ double mg_sweep_first_z(double bv, double dg, double rd)
{
  return 0.0 + mg_div(kMgOmega * bv, dg, rd);
}

// i / nx for i < 2^20 (rnx = 1 / nx: the quotient's error stays below half
// the distance of (i + 0.5) / nx from a whole number)
__device__ __forceinline__ int mg_row_of(int i, float rnx)
{
  return static_cast<int>((static_cast<float>(i) + 0.5f) * rnx);
}

// aggregates (on a level of nxc columns) of the cell of row r and of its
// four neighbours (an absent one: the cell's own)
__device__ __forceinline__ void mg_parents(const MGRow &r, int nxc, int (&pc)[5])
{
  const int px = r.ix >> 1, py = r.iy >> 1;
  pc[0] = py * nxc + px;
  pc[1] = (r.m & 1u) ? py * nxc + ((r.ix - 1) >> 1) : pc[0];
  pc[2] = (r.m & 2u) ? py * nxc + ((r.ix + 1) >> 1) : pc[0];
  pc[3] = (r.m & 4u) ? ((r.iy - 1) >> 1) * nxc + px : pc[0];
  pc[4] = (r.m & 8u) ? ((r.iy + 1) >> 1) * nxc + px : pc[0];
}

// (A_k v)_c: diag v_c - g_l v_{c-1} - g_r v_{c+1} - g_dn v_{c-nx} - g_up v_{c+nx},
// absent neighbours skipped (their term computed on a clamped value and
// discarded)
template <class Get>
__device__ __forceinline__ double mg_apply_row(const MGRow &r, int c, Get v)
{
  const double vc = v(c), vl = v(r.jl), vr = v(r.jr), vd = v(r.jd), vu = v(r.ju);
  double acc = r.dg * vc;
  const double a1 = acc - r.gl * vl;
  acc = (r.m & 1u) ? a1 : acc;
  const double a2 = acc - r.gr * vr;
  acc = (r.m & 2u) ? a2 : acc;
  const double a3 = acc - r.gd * vd;
  acc = (r.m & 4u) ? a3 : acc;
  const double a4 = acc - r.gu * vu;
  acc = (r.m & 8u) ? a4 : acc;
  return acc;
}

// the same on values already loaded: v = {v_c, v_l, v_r, v_dn, v_up}
__device__ __forceinline__ double mg_apply_vals(const MGRow &r, const double (&v)[5])
{
  double acc = r.dg * v[0];
  const double a1 = acc - r.gl * v[1];
  acc = (r.m & 1u) ? a1 : acc;
  const double a2 = acc - r.gr * v[2];
  acc = (r.m & 2u) ? a2 : acc;
  const double a3 = acc - r.gd * v[3];
  acc = (r.m & 4u) ? a3 : acc;
  const double a4 = acc - r.gu * v[4];
  acc = (r.m & 8u) ? a4 : acc;
  return acc;
}

template <class Get>
__device__ __forceinline__ double mg_apply(const MGLevel &l, int c, Get v)
{
  return mg_apply_row(mg_row(l, c), c, v);
}

// Loads and stores of values that other workgroups (kSpanOne: only other waves
// of this one) write between barriers.
template <int SPAN>
__device__ __forceinline__ double mld(const double *p)
{
  return __hip_atomic_load(const_cast<double *>(p), __ATOMIC_RELAXED,
                           SPAN == kSpanOne ? __HIP_MEMORY_SCOPE_WORKGROUP
                                            : __HIP_MEMORY_SCOPE_AGENT);
}
template <int SPAN>
__device__ __forceinline__ void mst(double *p, double v)
{
  xst<SPAN>(p, v);
}

// Sums of the nb published NV-tuples (layout [nb][NV]) in the fixed order of
// the host-side definition: the 256-element tree over each chunk, then over
// the chunk sums (nb <= 65536).  Every thread gets every result.
template <int NV, int SPAN>
__device__ __forceinline__ void group_tree_n(const double *part, int nb, double *red,
                                             double (&out)[NV])
{
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int nch = (nb + kTree - 1) / kTree;
  auto chunk = [&](int k, double (&r)[NV]) {
    // (every load issued before the first tree)
    double v[NV][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = k * kTree + lane + 64 * q;
#pragma unroll
      for (int j = 0; j < NV; ++j) v[j][q] = i < nb ? mld<SPAN>(&part[NV * i + j]) : 0.0;
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) r[j] = wave_tree256(v[j][0], v[j][1], v[j][2], v[j][3]);
  };
  if (nch == 1) {
    double r[NV];
    chunk(0, r);
#pragma unroll
    for (int j = 0; j < NV; ++j) out[j] = lane0(r[j]);
    return;
  }
  for (int k = wave; k < nch; k += nw) {
    double r[NV];
    chunk(k, r);
    if (lane == 0)
#pragma unroll
      for (int j = 0; j < NV; ++j) red[j * kTree + k] = r[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = lane + 64 * q;
      v[q] = k < nch ? red[j * kTree + k] : 0.0;
    }
    out[j] = lane0(wave_tree256(v[0], v[1], v[2], v[3]));
  }
  __syncthreads();
}

// the first damped Jacobi sweep, from zero: 0 + (omega b) / diag
__device__ __forceinline__ double mg_sweep_first(double bv, double dg)
{
  return 0.0 + (kMgOmega * bv) / dg;
}
struct MgV2 {
  double a, b;
};

// The level table copied into LDS (read from global memory at every pass, a
// descriptor cost a memory round trip before the pass could load its data).
// Ends with a workgroup barrier; the one before it waits for a previous solve
// of this workgroup to be done with the table.
__device__ __forceinline__ void mg_stage_levels(const MGLevel *src, int L, MGLevel *dst)
{
  constexpr int kW = static_cast<int>(sizeof(MGLevel) / sizeof(int));
  static_assert(sizeof(MGLevel) % sizeof(int) == 0, "level descriptors are whole words");
  __syncthreads();
  const int *from = reinterpret_cast<const int *>(src);
  int *to = reinterpret_cast<int *>(dst);
  for (int i = threadIdx.x; i < L * kW; i += blockDim.x) to[i] = from[i];
  __syncthreads();
}

// The cells i = tid, tid + nt, ... of [0, N), Q per thread at a time: the Q
// loads first (an index past the end replaced by the first), then the Q
// finishes, so that a thread's loads are in flight together.
template <int Q, class Ld, class Fin>
__device__ __forceinline__ void mg_cells(int N, Ld load, Fin finish)
{
  const int nt = static_cast<int>(blockDim.x);
  for (int i0 = static_cast<int>(threadIdx.x); i0 < N; i0 += Q * nt) {
    using V = decltype(load(0));
    V v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = i0 + q * nt;
      v[q] = load(i < N ? i : i0);
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i = i0 + q * nt;
      if (i < N) finish(i, v[q]);
    }
  }
}

// A pointer to global memory, read as a scalar: a pointer loaded from memory is
// otherwise taken for one to any memory, with slower accesses that also wait
// for the LDS.
template <class T>
__device__ __forceinline__ T *mg_global(T *p)
{
  typedef __attribute__((address_space(1))) T GT;
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(v));
  const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(v >> 32));
  return (T *)(GT *)((static_cast<unsigned long long>(hi) << 32) | lo);
}
__device__ __forceinline__ int mg_scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }

// a grid level's descriptor as scalars
__device__ __forceinline__ MGLevel mg_level(const MGLevel &l)
{
  MGLevel f = l;
  f.nx = mg_scalar(l.nx);
  f.ny = mg_scalar(l.ny);
  f.n = mg_scalar(l.n);
  f.has_y = mg_scalar(l.has_y);
  f.gx = mg_global(l.gx);
  f.gy = mg_global(l.gy);
  f.diag = mg_global(l.diag);
  f.gxz = mg_global(l.gxz);
  f.gyz = mg_global(l.gyz);
  f.rd = mg_global(l.rd);
  f.b = mg_global(l.b);
  f.xa = mg_global(l.xa);
  f.xb = mg_global(l.xb);
  f.xd = mg_global(l.xd);
  f.e = mg_global(l.e);
  f.rnx = __int_as_float(mg_scalar(__float_as_int(l.rnx)));
  f.rec = mg_scalar(l.rec);
  f.c0 = mg_scalar(l.c0);
  f.c1 = mg_scalar(l.c1);
  f.r0 = mg_scalar(l.r0);
  f.r1 = mg_scalar(l.r1);
  f.wdown = mg_scalar(l.wdown);
  f.wup = mg_scalar(l.wup);
  return f;
}

// an LDS level's descriptor as scalars
__device__ __forceinline__ MgLds mg_lds_level(const MGLevel &l)
{
  MgLds f;
  f.nx = mg_scalar(l.nx);
  f.ny = mg_scalar(l.ny);
  f.n = mg_scalar(l.n);
  f.S = f.nx + 1;
  f.lb = mg_scalar(l.lb);
  f.lx = mg_scalar(l.lx);
  f.lt = mg_scalar(l.lt);
  f.dg = mg_scalar(l.dg);
  f.rd = mg_scalar(l.rdl);
  f.gx = mg_scalar(l.lgx);
  f.gy = mg_scalar(l.lgy);
  f.rnx = __int_as_float(mg_scalar(__float_as_int(l.rnx)));
  return f;
}

// a solve's arguments, those of a batch being read from memory
__device__ __forceinline__ MGArgs mg_args(const MGArgs &in)
{
  MGArgs a = in;
  a.lv = mg_global(in.lv);
  a.b = mg_global(in.b);
  a.x = mg_global(in.x);
  a.p = mg_global(in.p);
  a.s = mg_global(in.s);
  a.w = mg_global(in.w);
  a.part = mg_global(in.part);
  a.barrier = mg_global(in.barrier);
  a.flags = mg_global(in.flags);
  a.sc = mg_global(in.sc);
  a.r2 = mg_global(in.r2);
  a.s2 = mg_global(in.s2);
  return a;
}

// the rows of the LDS levels, and zeros in the pads of their vectors (no barrier)
__device__ __forceinline__ void mg_lds_rows(const MGLevel *lv, int Lg, int L, double *lds,
                                            int zero0, int zero_n, int slots)
{
  const bool Y = lv[Lg].ny > 1;
  for (int k = Lg + 1; slots && k < L; ++k) {
    const MGLevel F = mg_level(lv[k]);
    const int S = F.nx + 1;
    for (int i = threadIdx.x; i < mg_rec_words(F.nx, F.ny) / kMgRec; i += blockDim.x) {
      const int r = i / S - 1, col = i - (r + 1) * S;
      const bool cell = r >= 0 && r < F.ny && col < F.nx;
      const int c = cell ? r * F.nx + col : 0;
      double *const R = lds + F.rec + kMgRec * i;
      const double dg = F.diag[c], gl = F.gx[cell ? r * S + col : 0], gd = Y ? F.gy[c] : 0.0;
      R[kMgDg] = cell ? dg : 0.0;
      R[kMgRd] = cell ? mg_recip(dg) : 0.0;
      R[kMgGl] = cell && col > 0 ? gl : 0.0;
      R[kMgGd] = cell && r > 0 ? gd : 0.0;
      R[kMgB] = 0.0;
      R[kMgX] = 0.0;
      R[kMgT] = 0.0;
    }
  }
  for (int k = Lg; k < (slots ? Lg + 1 : L); ++k) {
    const MGLevel F = mg_level(lv[k]);
    const int S = F.nx + 1;
    mg_cells<1>(
        Y ? (F.ny + 1) * S : S,
        [&](int i) {
          const int r = i / S, col = i - r * S;
          const bool cell = col < F.nx && r < F.ny;
          const int c = cell ? r * F.nx + col : 0;
          MGRowZ v;
          v.dg = F.diag[c];
          v.gl = F.gx[cell ? r * S + col : 0];
          v.gd = Y ? F.gy[cell ? r * F.nx + col : 0] : 0.0;
          if (!cell || col == 0) v.gl = 0.0;
          if (!cell || r == 0) v.gd = 0.0;
          return v;
        },
        [&](int i, const MGRowZ &v) {
          lds[F.dg + i] = v.dg;
          lds[F.rdl + i] = mg_recip(v.dg);
          lds[F.lgx + i] = v.gl;
          if (Y) lds[F.lgy + i] = v.gd;
        });
  }
  for (int i = threadIdx.x; i < zero_n; i += blockDim.x) lds[zero0 + i] = 0.0;
}

// this thread's places in the records of levels Lg + 1 .. Lg + slots
__device__ __forceinline__ void mg_slots(const MGLevel *lv, int Lg, int slots,
                                         MgSlot (&sl)[kMgSlots])
{
  const int tid = static_cast<int>(threadIdx.x);
#pragma unroll
  for (int s = 0; s < kMgSlots; ++s) {
    MgSlot v{0, 0, 0, 0, 0, 0, 0, 0};
    if (s < slots) {
      const MGLevel &F = lv[Lg + 1 + s], &U = lv[Lg + s], &C = lv[Lg + 1 + (s + 1 < slots ? s + 1 : s)];
      const int S = F.nx + 1, Sc = C.nx + 1, Su = U.nx + 1;
      const int i = tid < F.n ? tid : 0, r = i / F.nx, col = i - r * F.nx;
      v.n = mg_scalar(F.n);
      v.row = mg_scalar(kMgRec * S);
      v.crow = mg_scalar(kMgRec * Sc);
      v.own = F.rec + kMgRec * ((r + 1) * S + col);
      v.child = U.rec + kMgRec * ((2 * r + 1) * Su + 2 * col);
      v.par = C.rec + kMgRec * (((r >> 1) + 1) * Sc + (col >> 1));
      v.parl = v.par - ((col & 1) ? 0 : kMgRec);
      v.pard = v.par - ((r & 1) ? 0 : kMgRec * Sc);
    }
    sl[s] = v;
  }
}

// The part of the V-cycle on the records: from level Lg + 1's b and x to its t.
// Levels of at most 64 cells are run by wavefront 0 alone: its LDS operations
// execute in order, so their passes need no workgroup barrier.
__device__ __forceinline__ void mg_slot_cycle(double *lds, const MgSlot (&sl)[kMgSlots], int slots)
{
  const int tid = static_cast<int>(threadIdx.x);
  auto meet = [](bool alone) {
    if (alone) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  };
  auto row = [](const double *V, int S) {
    return MGRowZ{V[kMgDg], V[kMgRd], V[kMgGl], V[kMgGl + kMgRec], V[kMgGd], V[kMgGd + S]};
  };
  // from field `in` to the other of x and t
  auto sweep = [&](const MgSlot &f, int in, int out) {
    if (tid < f.n) {
      double *const V = lds + f.own;
      const double *const X = V + in;
      V[out] = mg_sweep_z(row(V, f.row), V[kMgB], X[0], X[-kMgRec], X[kMgRec], X[-f.row], X[f.row]);
    }
    meet(f.n <= 64);
  };
#pragma unroll
  for (int s = 0; s + 1 < kMgSlots; ++s) {
    if (s + 1 >= slots) break;
    if (sl[s].n <= 64 && tid >= 64) break;
    sweep(sl[s], kMgX, kMgT);
    const MgSlot &c = sl[s + 1];
    if (tid < c.n) {
      const int S = sl[s].row;
      const double *const F = lds + c.child, *const F2 = F + S, *const F3 = F2 + S;
      const double *const T = F + kMgT, *const T2 = F2 + kMgT;
      constexpr int R = kMgRec;
      const double v00 = T[0], v01 = T[R], v10 = T2[0], v11 = T2[R];
      const double m0 = F2[kMgGd], m1 = F2[kMgGd + R];
      const MGRowZ r0{F[kMgDg], 0.0, F[kMgGl], F[kMgGl + R], F[kMgGd], m0};
      const MGRowZ r1{F[kMgDg + R], 0.0, r0.gr, F[kMgGl + 2 * R], F[kMgGd + R], m1};
      const MGRowZ r2{F2[kMgDg], 0.0, F2[kMgGl], F2[kMgGl + R], m0, F3[kMgGd]};
      const MGRowZ r3{F2[kMgDg + R], 0.0, r2.gr, F2[kMgGl + 2 * R], m1, F3[kMgGd + R]};
      const double q0 = F[kMgB] - mg_apply_z(r0, v00, T[-R], v01, T[-S], v10);
      const double q1 = F[kMgB + R] - mg_apply_z(r1, v01, v00, T[2 * R], T[R - S], v11);
      const double q2 = F2[kMgB] - mg_apply_z(r2, v10, T2[-R], v11, v00, T2[S]);
      const double q3 = F2[kMgB + R] - mg_apply_z(r3, v11, v10, T2[2 * R], v01, T2[R + S]);
      const double v = (q0 + q1) + (q2 + q3);
      const bool last = s + 2 == slots;
      double *const C = lds + c.own;
      const double q = mg_div(last ? v : kMgOmega * v, C[kMgDg], C[kMgRd]);
      C[kMgB] = v;
      C[last ? kMgT : kMgX] = last ? q : 0.0 + q;
    }
    meet(c.n <= 64);
  }
#pragma unroll
  for (int s = kMgSlots - 2; s >= 0; --s) {
    if (s + 1 >= slots) continue;
    const MgSlot &f = sl[s];
    if (f.n <= 64 && tid >= 64) continue;
    if (f.n > 64 && sl[s + 1].n <= 64) __syncthreads();
    if (tid < f.n) {
      double *const V = lds + f.own;
      const double *const T = V + kMgT, *const P = lds + kMgT;
      const double vc = T[0] + kMgScale * P[f.par];
      const double vl = T[-kMgRec] + kMgScale * P[f.parl];
      const double vr = T[kMgRec] + kMgScale * P[f.parl + kMgRec];
      const double vd = T[-f.row] + kMgScale * P[f.pard];
      const double vu = T[f.row] + kMgScale * P[f.pard + f.crow];
      V[kMgX] = mg_sweep_z(row(V, f.row), V[kMgB], vc, vl, vr, vd, vu);
    }
    meet(f.n <= 64);
    sweep(f, kMgX, kMgT);
  }
}

// The V-cycle of the LDS levels Lg..L-1, run by every workgroup on its own
// copy: b of level Lg from global memory (b_global; the pads' zeros written
// here, the LDS being used for other things between two cycles) or already in
// LDS; its result ends in E (cell by cell), or in level Lg's t vector (E null).
// Descent: b loaded with the first sweep; per level the second sweep, then the
// restriction with the next level's first sweep (the one-cell level: its exact
// solve).  Ascent: the correction fused into the first post-sweep (the
// neighbours' corrected values recomputed), the second post-sweep.
template <int SPAN, bool Y>
__device__ __forceinline__ void mg_lds_cycle_y(const MGLevel *lv, int Lg, int L, double *lds,
                                               double *E, bool b_global, int zero0, int zero_n,
                                               const MgSlot (&sl)[kMgSlots], int slots)
{
  // A pass over an LDS level, then a workgroup barrier; a level of at most one
  // cell per lane is run by wavefront 0 alone (the others wait at the end of
  // the small levels): its LDS operations execute in order, so a pass needs no
  // workgroup barrier.  Each pass is in the code once, for both: the
  // instruction cache holds an iteration.
  bool alone = false;
  auto run = [&](int nl, auto cell) {
    const int bd = alone ? 64 : static_cast<int>(blockDim.x);
#pragma unroll 1
    for (int i = threadIdx.x; i < nl; i += bd) cell(i);
    if (alone) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  };
  // two cells per thread at a time where the level has more cells than threads
  auto run2 = [&](int nl, auto compute, auto store) {
    const int bd = static_cast<int>(blockDim.x);
#pragma unroll 1
    for (int i = threadIdx.x; i < nl; i += 2 * bd) {
      const int i1 = i + bd < nl ? i + bd : i;
      const auto v0 = compute(i), v1 = compute(i1);
      store(i, v0);
      store(i1, v1);
    }
    __syncthreads();
  };
  auto front = [](const MgLds &F) { return Y ? F.S : 1; };
  auto row = [&](const MgLds &F, int jc) {
    const double *C = lds + jc;
    MGRowZ r;
    r.dg = C[F.dg];
    r.rd = C[F.rd];
    r.gl = C[F.gx];
    r.gr = C[F.gx + 1];
    r.gd = Y ? C[F.gy] : 0.0;
    r.gu = Y ? C[F.gy + F.S] : 0.0;
    return r;
  };
  auto sweep = [&](const MgLds &F, const double *X, int i) {
    const int jc = i + mg_row_of(i, F.rnx), j = jc + front(F);
    const double *V = X + j;
    return mg_sweep_z(row(F, jc), lds[F.lb + j], V[0], V[-1], V[1], Y ? V[-F.S] : 0.0,
                      Y ? V[F.S] : 0.0);
  };
  auto at = [&](const MgLds &F, int i) { return i + mg_row_of(i, F.rnx) + front(F); };
  {
    const MgLds T = mg_lds_level(lv[Lg]);
    const bool one = L - 1 == Lg;
    if (b_global) {
      for (int i = threadIdx.x; i < zero_n; i += blockDim.x) lds[zero0 + i] = 0.0;
      const double *src = mg_global(lv[Lg].b);
      mg_cells<2>(
          T.n, [&](int i) { return mld<SPAN>(&src[i]); },
          [&](int i, double v) { lds[T.lb + at(T, i)] = v; });
      __syncthreads();
    }
    run(T.n, [&](int i) {
      const int jc = i + mg_row_of(i, T.rnx), j = jc + front(T);
      const double bv = lds[T.lb + j], dg = lds[T.dg + jc], rd = lds[T.rd + jc];
      const double q = mg_div(one ? bv : kMgOmega * bv, dg, rd);
      if (!one) lds[T.lx + j] = 0.0 + q;
      else if (E) E[i] = q;
      else lds[T.lt + j] = q;
    });
    if (one) return;
  }
  // descent step at level k (second sweep, restriction with the next
  // level's first sweep) and ascent step (corrected first post-sweep,
  // second post-sweep)
  // (Rec: the coarser level has records)
  auto down = [&](auto Rec, int k) {
    const MgLds F = mg_lds_level(lv[k]), Cl = mg_lds_level(lv[k + 1]);
    const double *X = lds + F.lx;
    double *Tm = lds + F.lt;
    if constexpr (decltype(Rec)::value)
      run2(F.n, [&](int i) { return sweep(F, X, i); }, [&](int i, double v) { Tm[at(F, i)] = v; });
    else
      run(F.n, [&](int i) { Tm[at(F, i)] = sweep(F, X, i); });
    const bool last = (k + 1 == L - 1);
    run(
        Cl.n,
        [&](int C) {
          // the four children's residuals: their twelve values and rows loaded
          // once each; an absent child's row is read at its neighbour, and its
          // residual not used
          const int J = mg_row_of(C, Cl.rnx), I = C - J * Cl.nx;
          const int S = F.S, jc = 2 * J * S + 2 * I;
          const bool right = 2 * I + 1 < F.nx, up = Y && 2 * J + 1 < F.ny;
          const int sy = up ? S : 0;
          const double *V = Tm + jc + front(F), *Bv = lds + F.lb + jc + front(F), *R = lds + jc;
          const double v00 = V[0], v01 = V[1], vl0 = V[-1], vr0 = V[2];
          const double v10 = Y ? V[S] : 0.0, v11 = Y ? V[S + 1] : 0.0;
          const double gx0 = R[F.gx], gx1 = R[F.gx + 1], gx2 = R[F.gx + 2];
          const double gm0 = Y ? R[F.gy + S] : 0.0, gm1 = Y ? R[F.gy + S + 1] : 0.0;
          MGRowZ r0{R[F.dg], 0.0, gx0, gx1, Y ? R[F.gy] : 0.0, gm0};
          MGRowZ r1{R[F.dg + 1], 0.0, gx1, gx2, Y ? R[F.gy + 1] : 0.0, gm1};
          const double q0 = Bv[0] - mg_apply_z(r0, v00, vl0, v01, Y ? V[-S] : 0.0, v10);
          const double q1 = Bv[1] - mg_apply_z(r1, v01, v00, vr0, Y ? V[1 - S] : 0.0, v11);
          double q2 = 0.0, q3 = 0.0;
          if (Y) {
            const double *V2 = V + sy, *R2 = R + sy;
            const double hx0 = R2[F.gx], hx1 = R2[F.gx + 1], hx2 = R2[F.gx + 2];
            MGRowZ r2{R2[F.dg], 0.0, hx0, hx1, gm0, R2[F.gy + S]};
            MGRowZ r3{R2[F.dg + 1], 0.0, hx1, hx2, gm1, R2[F.gy + S + 1]};
            q2 = Bv[sy] - mg_apply_z(r2, v10, V2[-1], v11, v00, V2[S]);
            q3 = Bv[sy + 1] - mg_apply_z(r3, v11, v10, V2[2], v01, V2[S + 1]);
          }
          const double v = (q0 + (right ? q1 : 0.0)) + ((up ? q2 : 0.0) + (right && up ? q3 : 0.0));
          if constexpr (decltype(Rec)::value) {
            double *const R = lds + mg_scalar(lv[k + 1].rec) + kMgRec * (C + J + Cl.S);
            const double q = mg_div(last ? v : kMgOmega * v, R[kMgDg], R[kMgRd]);
            R[kMgB] = v;
            R[last ? kMgT : kMgX] = last ? q : 0.0 + q;
          } else {
            const int jC = C + J;
            const double q = mg_div(last ? v : kMgOmega * v, lds[Cl.dg + jC], lds[Cl.rd + jC]);
            lds[Cl.lb + jC + front(Cl)] = v;
            lds[(last ? Cl.lt : Cl.lx) + jC + front(Cl)] = last ? q : 0.0 + q;
          }
        });
  };
  auto up = [&](auto Rec, int k) {
    const MgLds F = mg_lds_level(lv[k]), Cl = mg_lds_level(lv[k + 1]);
    constexpr int W = decltype(Rec)::value ? kMgRec : 1;
    const double *Ec = decltype(Rec)::value ? lds + mg_scalar(lv[k + 1].rec) + kMgT + kMgRec * Cl.S
                                            : lds + Cl.lt + front(Cl);
    double *X = lds + F.lx, *Tm = lds + F.lt;
    auto first = [&](int i) {
      const int iy = mg_row_of(i, F.rnx), ix = i - iy * F.nx;
      const int S = F.S, jc = i + iy, Sc = Cl.S;
      const double *V = Tm + jc + front(F);
      const double *P = Ec + W * ((iy >> 1) * Sc + (ix >> 1));
      // (a left or lower absent neighbour's parent is a pad as well)
      const int pl = (ix & 1) - 1, pr = ix & 1;
      const double e0 = P[0], el = P[W * pl], er = P[W * pr];
      const double vc = V[0] + kMgScale * e0, vl = V[-1] + kMgScale * el;
      double vr = V[1] + kMgScale * er, vd = 0.0, vu = 0.0;
      vr = ix < F.nx - 1 ? vr : 0.0;
      if (Y) {
        vd = V[-S] + kMgScale * P[(iy & 1) ? 0 : -W * Sc];
        vu = V[S] + kMgScale * P[(iy & 1) ? W * Sc : 0];
        vu = iy < F.ny - 1 ? vu : 0.0;
      }
      return mg_sweep_z(row(F, jc), lds[F.lb + jc + front(F)], vc, vl, vr, vd, vu);
    };
    auto second = [&](int i, double v) {
      if (k == Lg && E) E[i] = v;
      else Tm[at(F, i)] = v;
    };
    if constexpr (decltype(Rec)::value) {
      run2(F.n, first, [&](int i, double v) { X[at(F, i)] = v; });
      run2(F.n, [&](int i) { return sweep(F, X, i); }, second);
    } else {
      run(F.n, [&](int i) { X[at(F, i)] = first(i); });
      run(F.n, [&](int i) { second(i, sweep(F, X, i)); });
    }
  };
  if constexpr (Y) {
    if (slots) {
      down(std::true_type{}, Lg);
      mg_slot_cycle(lds, sl, slots);
      if (sl[0].n <= 64) __syncthreads();
      up(std::true_type{}, Lg);
      return;
    }
  }
  // the levels of at most 64 cells (from ks on) by wavefront 0 alone
  int ks = Lg;
  while (ks < L - 1 && mg_scalar(lv[ks].n) > 64) ++ks;
  const bool first_wave = threadIdx.x < 64;
#pragma unroll 1
  for (int k = Lg; k < L - 1; ++k) {
    alone = k >= ks;
    if (alone && !first_wave) break;
    down(std::false_type{}, k);
  }
#pragma unroll 1
  for (int k = L - 2; k >= Lg; --k) {
    alone = k >= ks;
    if (!alone || first_wave) up(std::false_type{}, k);
    if (k == ks) __syncthreads();
  }
}

template <int SPAN>
__device__ __forceinline__ void mg_lds_cycle(const MGLevel *lv, int Lg, int L, double *lds,
                                             double *E, bool b_global, int zero0, int zero_n,
                                               const MgSlot (&sl)[kMgSlots], int slots)
{
  if (__builtin_amdgcn_readfirstlane(lv[Lg].ny) > 1)
    mg_lds_cycle_y<SPAN, true>(lv, Lg, L, lds, E, b_global, zero0, zero_n, sl, slots);
  else
    mg_lds_cycle_y<SPAN, false>(lv, Lg, L, lds, E, b_global, zero0, zero_n, sl, slots);
}

// The preconditioned CG of one system, run by the G workgroups of a group of
// which this one is number bid (G = 1: one workgroup alone, with workgroup
// barriers in place of the group's).
template <int SPAN>
__device__ __forceinline__ void mgcg_solve(const MGArgs &in, int G, int bid, double *lds,
                                           double *red, MGLevel *s_lv)
{
  const MGArgs a = mg_args(in);
  const int nw = blockDim.x >> 6, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int gwv = bid * nw + wave, gstride = G * nw;
  if (bid == 0 && threadIdx.x == 0) a.sc->cg_t0 = static_cast<unsigned long long>(wall_clock64());
  const int L = a.L, Lg = a.Lg;
  mg_stage_levels(a.lv, L, s_lv);
  const MGLevel *lv = s_lv;
  const MGLevel L0 = mg_level(lv[0]);
  const int n = L0.n, nb = (n + kTree - 1) / kTree;
  unsigned int epoch = 0;

  auto bar = [&]() -> bool {
    if (G == 1) {
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      return true;
    }
    return flag_barrier<SPAN>(a.barrier, a.flags, bid, G, epoch);
  };
  // The cells of a grid level this thread owns, Q of a block at a time: the Q
  // are computed first (an index past the end replaced by the block's first
  // cell), then the valid ones stored, so a batch's loads issue before its
  // first store.  Q trades loads in flight against registers.
  auto for_cells = [&](auto Qc, int nl, auto compute, auto store) {
    constexpr int Q = decltype(Qc)::value;
    const int nbl = (nl + kTree - 1) / kTree;
    for (int blk = gwv; blk < nbl; blk += gstride)
#pragma unroll 1
      for (int q0 = 0; q0 < 4; q0 += Q) {
        using R = decltype(compute(0));
        R v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int c = blk * kTree + lane + 64 * (q0 + q);
          v[q] = compute(c < nl ? c : blk * kTree);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int c = blk * kTree + lane + 64 * (q0 + q);
          if (c < nl) store(c, v[q]);
        }
      }
  };
  using Q1 = std::integral_constant<int, 1>;
  using Q2 = std::integral_constant<int, 2>;
  using Q4 = std::integral_constant<int, 4>;
  // A phase that touches no own-cell state: the cells of the level spread
  // over every thread of the group (consecutive threads, consecutive cells),
  // two at a time when the level has more cells than the group has threads.
  const int nthr = G * static_cast<int>(blockDim.x);
  const int tid = bid * static_cast<int>(blockDim.x) + static_cast<int>(threadIdx.x);
  auto for_flat = [&](auto Qmax, int nl, auto compute, auto store) {
    auto run = [&](auto Qc) {
      constexpr int Q = decltype(Qc)::value;
      for (int c0 = tid; c0 < nl; c0 += Q * nthr) {
        using R = decltype(compute(0));
        R v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int c = c0 + q * nthr;
          v[q] = compute(c < nl ? c : c0);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int c = c0 + q * nthr;
          if (c < nl) store(c, v[q]);
        }
      }
    };
    if (decltype(Qmax)::value > 1 && nl > nthr) run(std::integral_constant<int, 2>{});
    else run(std::integral_constant<int, 1>{});
  };
  auto sweep_first = [&](double bv, double dg) { return mg_sweep_first(bv, dg); };
  using V2 = MgV2;

  // rows of the LDS levels, once per solve
  mg_lds_rows(lv, Lg, L, lds, a.zero0, a.zero_n, a.slots);
  MgSlot sl[kMgSlots];
  mg_slots(lv, Lg, a.slots, sl);
  __syncthreads();

  // the V-cycle on r (published as lv[0].b, and lv[0].xa = the first sweep
  // when level 0 is a grid level); u ends in lv[0].e, or in LDS when Lg = 0
  auto vcycle = [&]() -> bool {
    for (int k = 0; k < Lg; ++k) {
      const MGLevel F = mg_level(lv[k]);
      for_flat(
          Q2{}, F.n,
          [&](int c) {
            auto xa = [&](int j) { return mld<SPAN>(&F.xa[j]); };
            const MGRow r = mg_row(F, c);
            const double t = mld<SPAN>(&F.b[c]) - mg_apply_row(r, c, xa);
            return xa(c) + (kMgOmega * t) / r.dg;
          },
          [&](int c, double v) { mst<SPAN>(&F.xb[c], v); });
      if (!bar()) return false;
      const MGLevel Cl = mg_level(lv[k + 1]);
      const bool grid_next = (k + 1 < Lg);
      for_flat(
          Q1{}, Cl.n,
          [&](int C) {
            // the four children (absent ones clamped to the first and
            // discarded): every row and value loaded before any arithmetic
            const int J = C / Cl.nx, I = C - J * Cl.nx;
            MGRow rw[4];
            double bv[4], xv[4][5];
            bool in[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int ix = 2 * I + (k & 1), iy = 2 * J + (k >> 1);
              in[k] = (ix < F.nx && iy < F.ny);
              const int cx = in[k] ? ix : 2 * I, cy = in[k] ? iy : 2 * J;
              const int f = cy * F.nx + cx;
              rw[k] = mg_row_at(F, cx, cy);
              bv[k] = mld<SPAN>(&F.b[f]);
              xv[k][0] = mld<SPAN>(&F.xb[f]);
              xv[k][1] = mld<SPAN>(&F.xb[rw[k].jl]);
              xv[k][2] = mld<SPAN>(&F.xb[rw[k].jr]);
              xv[k][3] = mld<SPAN>(&F.xb[rw[k].jd]);
              xv[k][4] = mld<SPAN>(&F.xb[rw[k].ju]);
            }
            double q[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const double res = bv[k] - mg_apply_vals(rw[k], xv[k]);
              q[k] = in[k] ? res : 0.0;
            }
            const double B = (q[0] + q[1]) + (q[2] + q[3]);
            return V2{B, sweep_first(B, Cl.diag[C])};
          },
          [&](int C, V2 v) {
            mst<SPAN>(&Cl.b[C], v.a);
            if (grid_next) mst<SPAN>(&Cl.xa[C], v.b);
          });
      if (!bar()) return false;
    }
    // the LDS levels, in every workgroup
    mg_lds_cycle<SPAN>(lv, Lg, L, lds, Lg > 0 ? lds : nullptr, true, a.zero0, a.zero_n,
                       sl, a.slots);
    // Ascent.  The last sweep of a grid level whose finer level has at most
    // one cell per thread is not stored: that finer level's first post-sweep
    // recomputes it at the (at most three) aggregates its cell and neighbours
    // use, with the same operations, so it needs no phase and no barrier of
    // its own.
    auto fused = [&](int k) { return k >= 1 && lv[k - 1].n <= nthr; };
    for (int k = Lg - 1; k >= 0; --k) {
      const MGLevel F = mg_level(lv[k]), Cl = mg_level(lv[k + 1]);
      const bool recompute = (k + 1 < Lg) && fused(k + 1);
      // the coarse level's final value at aggregate P: from LDS, or the
      // second post-sweep of a grid level evaluated here
      auto e_grid = [&](int P) {
        const MGRow rc = mg_row(Cl, P);
        const double b = mld<SPAN>(&Cl.b[P]);
        double v5[5];
        v5[0] = mld<SPAN>(&Cl.xd[P]);
        v5[1] = mld<SPAN>(&Cl.xd[rc.jl]);
        v5[2] = mld<SPAN>(&Cl.xd[rc.jr]);
        v5[3] = mld<SPAN>(&Cl.xd[rc.jd]);
        v5[4] = mld<SPAN>(&Cl.xd[rc.ju]);
        const double t = b - mg_apply_vals(rc, v5);
        return v5[0] + (kMgOmega * t) / rc.dg;
      };
      auto post1 = [&](auto FromLds) {
        // (one cell at a time when the coarse values are recomputed: three
        // rows and stencils of loads per cell)
        using QP = std::conditional_t<decltype(FromLds)::value == 2, Q1, Q2>;
        for_flat(
            QP{}, F.n,
            [&](int c) {
              // x after the coarse correction, x_b + s e(parent), on the cell
              // and its neighbours: loads first, then the arithmetic
              const MGRow r = mg_row(F, c);
              const int js[5] = {c, r.jl, r.jr, r.jd, r.ju};
              int pc[5];
              mg_parents(r, Cl.nx, pc);
              double xb5[5], e5[5];
#pragma unroll
              for (int q = 0; q < 5; ++q) xb5[q] = mld<SPAN>(&F.xb[js[q]]);
              if constexpr (decltype(FromLds)::value == 1) {
#pragma unroll
                for (int q = 0; q < 5; ++q) e5[q] = lds[pc[q]];
              } else if constexpr (decltype(FromLds)::value == 0) {
#pragma unroll
                for (int q = 0; q < 5; ++q) e5[q] = mld<SPAN>(&Cl.e[pc[q]]);
              } else {
                // distinct aggregates: the cell's own, the one across an x
                // face (left or right) and the one across a y face
                const int px = (pc[1] != pc[0]) ? pc[1] : pc[2];
                const int py = (pc[3] != pc[0]) ? pc[3] : pc[4];
                const double e0 = e_grid(pc[0]), ex = e_grid(px), ey = e_grid(py);
                e5[0] = e0;
                e5[1] = (pc[1] == pc[0]) ? e0 : ex;
                e5[2] = (pc[2] == pc[0]) ? e0 : ex;
                e5[3] = (pc[3] == pc[0]) ? e0 : ey;
                e5[4] = (pc[4] == pc[0]) ? e0 : ey;
              }
              const double bc = mld<SPAN>(&F.b[c]);
              double xc5[5];
#pragma unroll
              for (int q = 0; q < 5; ++q) xc5[q] = xb5[q] + kMgScale * e5[q];
              const double t = bc - mg_apply_vals(r, xc5);
              return xc5[0] + (kMgOmega * t) / r.dg;
            },
            [&](int c, double v) { mst<SPAN>(&F.xd[c], v); });
      };
      // e of the coarse level: 1 from LDS, 0 stored by its last sweep, 2 recomputed
      if (k + 1 == Lg) post1(std::integral_constant<int, 1>{});
      else if (recompute) post1(std::integral_constant<int, 2>{});
      else post1(std::integral_constant<int, 0>{});
      if (!bar()) return false;
      if (fused(k)) continue;               // (recomputed by the next level)
      for_flat(
          Q2{}, F.n,
          [&](int c) {
            auto xd = [&](int j) { return mld<SPAN>(&F.xd[j]); };
            const MGRow r = mg_row(F, c);
            const double t = mld<SPAN>(&F.b[c]) - mg_apply_row(r, c, xd);
            return xd(c) + (kMgOmega * t) / r.dg;
          },
          [&](int c, double v) { mst<SPAN>(&F.e[c], v); });
      if (!bar()) return false;
    }
    return true;
  };
  auto uget = [&](int j) {
    if (Lg > 0) return mld<SPAN>(&L0.e[j]);
    return lds[L0.lt + j + mg_row_of(j, L0.rnx) + (L0.ny > 1 ? L0.nx + 1 : 1)];
  };
  // w = A u on the own cells and the block sums of (r, u), (w, u), (r, r)
  auto matvec = [&]() -> bool {
    for (int blk = gwv; blk < nb; blk += gstride) {
      double g[4], d[4], rr[4], wq[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c0 = blk * kTree + lane + 64 * q;
        const int c = c0 < n ? c0 : blk * kTree;
        const double uc = uget(c);
        const double wv = mg_apply(L0, c, uget);
        const double rv = mld<SPAN>(&L0.b[c]);
        const bool in = c0 < n;
        wq[q] = wv;
        g[q] = in ? rv * uc : 0.0;
        d[q] = in ? wv * uc : 0.0;
        rr[q] = in ? rv * rv : 0.0;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = blk * kTree + lane + 64 * q;
        if (c < n) a.w[c] = wq[q];
      }
      const double sg = wave_tree256(g[0], g[1], g[2], g[3]);
      const double sd = wave_tree256(d[0], d[1], d[2], d[3]);
      const double sr = wave_tree256(rr[0], rr[1], rr[2], rr[3]);
      if (lane == 0) {
        mst<SPAN>(&a.part[3 * blk], sg);
        mst<SPAN>(&a.part[3 * blk + 1], sd);
        mst<SPAN>(&a.part[3 * blk + 2], sr);
      }
    }
    return bar();
  };

  int status = -7, it = 0;
  double alpha = 0.0, beta = 0.0, gamma = 0.0, delta = 0.0, thr = 0.0;
  // start: x = 0, r = b
  for_cells(
      Q4{}, n, [&](int c) { return V2{a.b[c], sweep_first(a.b[c], L0.diag[c])}; },
      [&](int c, V2 v) {
        a.x[c] = 0.0;
        mst<SPAN>(&L0.b[c], v.a);
        if (Lg > 0) mst<SPAN>(&L0.xa[c], v.b);
      });
  if (!bar() || !vcycle() || !matvec()) {
    status = -3;
  } else {
    double s3[3];
    group_tree_n<3, SPAN>(a.part, nb, red, s3);
    gamma = s3[0];
    delta = s3[1];
    thr = a.tol2 * s3[2];
    if (s3[2] == 0.0) status = 0;
    else if (!(delta > 0.0)) status = -6;
    else alpha = gamma / delta;
  }
  while (status == -7 && it < a.max_iters) {
    const bool first = (it == 0);
    struct U5 {
      double p, s, x, r, xa;
    };
    for_cells(
        Q4{}, n,
        [&](int c) {
          const double uc = uget(c);
          const double wv = a.w[c];
          const double pv = first ? uc : uc + beta * a.p[c];
          const double sv = first ? wv : wv + beta * a.s[c];
          const double xv = a.x[c] + alpha * pv;
          const double rv = mld<SPAN>(&L0.b[c]) - alpha * sv;
          return U5{pv, sv, xv, rv, sweep_first(rv, L0.diag[c])};
        },
        [&](int c, U5 v) {
          a.p[c] = v.p;
          a.s[c] = v.s;
          a.x[c] = v.x;
          mst<SPAN>(&L0.b[c], v.r);
          if (Lg > 0) mst<SPAN>(&L0.xa[c], v.xa);
        });
    if (!bar() || !vcycle() || !matvec()) {
      status = -3;
      break;
    }
    ++it;
    double s3[3];
    group_tree_n<3, SPAN>(a.part, nb, red, s3);
    const double gamma_new = s3[0];
    delta = s3[1];
    if (s3[2] <= thr) {
      status = 0;
      break;
    }
    beta = gamma_new / gamma;
    double tq = beta * gamma_new;
    tq = tq / alpha;
    const double den = delta - tq;
    if (!(den > 0.0)) {
      status = -6;
      break;
    }
    alpha = gamma_new / den;
    gamma = gamma_new;
  }
  if (bid == 0 && threadIdx.x == 0) {
    a.sc->cg_iters = it;
    a.sc->cg_status = status;
    a.sc->cg_t1 = static_cast<unsigned long long>(wall_clock64());
  }
}

}  // namespace iugkp

#include "mgband.hpp"

namespace iugkp {

// The single solve's group of G workgroups, elected (elect_group), of more where
// the group may find room on one XCD; of fewer than G where they do not come.
__global__ __launch_bounds__(kCgThreadsMax) void mgcg_kernel(MGArgs a, int G)
{
  extern __shared__ double lds[];
  __shared__ double red[3 * kTree];
  __shared__ MGLevel s_lv[kMgLevelsMax];
  int rank = blockIdx.x;
  bool one_xcd = false;
  if (G > 1 && !elect_group<true>(a.barrier, G, rank, one_xcd, a.sc)) return;
  if (one_xcd) mgcg_solve<kSpanXcd>(a, G, rank, lds, red, s_lv);
  else mgcg_solve<kSpanDevice>(a, G, rank, lds, red, s_lv);
}

// the banded form (mgband.hpp), for the meshes whose rows leave it few windows;
// workgroups of at most kMgBandThreads threads, whose lanes then have the
// registers its batched loads take
constexpr int kMgBandThreads = 512;
// A chain of short dependent phases bounds it: the latency of a few loads per
// thread, of LDS passes and of 2 Lg barriers per iteration, and the fetch of the
// code, which an iteration runs through once.  So each phase is in the code
// once, unrolled little (two cells in the phases that load most; four and eight
// made 76000 instructions of it, and 70 us per iteration), levels' addresses are
// scalars to global memory, the rows each workgroup takes are worked out once
// per solve, and the small levels run from registers' addresses on records.
// us per iteration, before and after: 512 x 512 cells 123 and 100, 256 x 256 68
// and 44, 128 x 128 50 and 24, 64 x 64 38 and 17, 30 x 20 20 and 13; the 256 x
// 256 cavity to steady state 24.4 to 17.8 ms.
__global__ __launch_bounds__(kMgBandThreads) void mgcg_band_kernel(MGArgs a, int G)
{
  extern __shared__ double lds[];
  __shared__ double red[3 * kTree];
  __shared__ MGLevel s_lv[kMgLevelsMax];
  int rank = blockIdx.x;
  bool one_xcd = false;
  if (G > 1 && !elect_group<true>(a.barrier, G, rank, one_xcd, a.sc)) return;
  if (one_xcd) mgcg_band_solve<kSpanXcd, 2, 1>(a, G, rank, lds, red, s_lv);
  else mgcg_band_solve<kSpanDevice, 2, 1>(a, G, rank, lds, red, s_lv);
}

// ---------------------------------------------------------------------------
// Batched CG over a pool of resident workgroups.  The host hands every active
// Newton instance a group of workgroups and writes, per workgroup, the list of
// (instance, rank) jobs it takes part in; all lists follow one global job
// order, so the earliest unfinished job always has every member at hand and
// the pool cannot deadlock.  The solve of an instance does not depend on how
// many workgroups serve it or where.  Instances with the plain CG and those
// with the multigrid-preconditioned one have pools of their own, launched one
// after the other (one body with both would need more registers than a lane
// has).
// ---------------------------------------------------------------------------
struct CgJob {
  int inst, rank, G, tb;     // tb: blocks per workgroup, bit 30 = register form
};
constexpr int kCgJobReg = 1 << 30;

__global__ __launch_bounds__(kCgThreadsMax) void cg_batch_kernel(const Inst *__restrict__ insts,
                                                                 const int *__restrict__ off,
                                                                 const CgJob *__restrict__ jobs)
{
  const int e0 = off[blockIdx.x], e1 = off[blockIdx.x + 1];
  for (int e = e0; e < e1; ++e) {
    const CgJob jb = jobs[e];
    const Inst &in = insts[jb.inst];
    CGArgs a;
    a.m = in.m;
    a.gx = in.gx;
    a.gy = in.gy;
    a.diag = in.diag;
    a.b = in.rhs;
    a.x = in.cg_x;
    a.gr = in.cg_r;
    a.gw = in.cg_w;
    a.gp = in.cg_p;
    a.gs = in.cg_s;
    a.pub = in.cg_pub;
    a.part = in.cg_mpart;
    a.TB = jb.tb & (kCgJobReg - 1);
    a.tol2 = in.tol2;
    a.max_iters = in.cg_max;
    a.barrier = in.cg_barrier;
    a.sc = in.sc;
    if (!(jb.tb & kCgJobReg)) cg_global_run(a, jb.rank, jb.G);
    else if (jb.G == 1) cg_reg_run<kSpanOne, false>(a, 0, 1);
    else cg_reg_run<kSpanDevice, false>(a, jb.rank, jb.G);
    __syncthreads();
  }
}

// (A batch's groups are small, their workgroups with many cells per thread: four
// and two cells of them in flight.)
// the multigrid instances' pool: job (instance, rank) runs member `rank` of
// the instance's group of G workgroups (mg: the instances' arguments); 8-wave
// workgroups, whose lanes have the registers the solve takes when its
// arguments come from memory
constexpr int kMgPoolWaves = 8;
__global__ __launch_bounds__(64 * kMgPoolWaves) void mgcg_batch_kernel(const int *__restrict__ off,
                                                                   const CgJob *__restrict__ jobs,
                                                                   const MGArgs *__restrict__ mg)
{
  extern __shared__ double lds[];
  __shared__ double red[3 * kTree];
  __shared__ MGLevel s_lv[kMgLevelsMax];
  const int e0 = off[blockIdx.x], e1 = off[blockIdx.x + 1];
  for (int e = e0; e < e1; ++e) {
    const CgJob jb = jobs[e];
    const MGArgs &a = mg[jb.inst];
    if (a.band) mgcg_band_solve<kSpanDevice, 4, 2>(a, jb.G, jb.rank, lds, red, s_lv);
    else mgcg_solve<kSpanDevice>(a, jb.G, jb.rank, lds, red, s_lv);
    __syncthreads();
  }
}

// Level k+1's faces from level k's: a coarse x face sums the fine x faces of
// its two rows at the fine face under it, a coarse y face the fine y faces of
// its two columns (an absent row or column adds 0).
__global__ void mg_coarsen_faces_kernel(MGLevel f, MGLevel c, int has_y, double *gx, double *gy)
{
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int nfx = c.ny * (c.nx + 1);
  if (i < nfx) {
    const int J = i / (c.nx + 1), K = i - J * (c.nx + 1);
    const int k = (2 * K < f.nx) ? 2 * K : f.nx;
    const double a = f.gx[(2 * J) * (f.nx + 1) + k];
    const double b = (2 * J + 1 < f.ny) ? f.gx[(2 * J + 1) * (f.nx + 1) + k] : 0.0;
    gx[i] = a + b;
  }
  if (has_y && i < (c.ny + 1) * c.nx) {
    const int K = i / c.nx, I = i - K * c.nx;
    const int k = (2 * K < f.ny) ? 2 * K : f.ny;
    const double a = f.gy[k * f.nx + 2 * I];
    const double b = (2 * I + 1 < f.nx) ? f.gy[k * f.nx + 2 * I + 1] : 0.0;
    gy[i] = a + b;
  }
}

// diagonal = the sum of the cell's faces: (left + right) + down + up
__global__ void mg_coarsen_diag_kernel(MGLevel c, int has_y, double *diag)
{
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= c.n) return;
  const int J = i / c.nx, I = i - J * c.nx;
  double d = c.gx[J * (c.nx + 1) + I] + c.gx[J * (c.nx + 1) + I + 1];
  if (has_y) {
    d = d + c.gy[J * c.nx + I];
    d = d + c.gy[(J + 1) * c.nx + I];
  }
  diag[i] = d;
}

// the banded form's copies of a level's operator (MGLevel)
__global__ void mg_rows_kernel(MGLevel l, double *gxz, double *gyz, double *rd)
{
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int S = l.nx + 1;
  if (i < l.ny * S) {
    const int ix = i % S;
    gxz[i] = (ix > 0 && ix < l.nx) ? l.gx[i] : 0.0;
  }
  if (i < (l.ny + 1) * l.nx) gyz[i] = (i >= l.nx && i < l.ny * l.nx) ? l.gy[i] : 0.0;
  if (i < l.n) rd[i] = mg_recip(l.diag[i]);
}

}  // namespace iugkp
