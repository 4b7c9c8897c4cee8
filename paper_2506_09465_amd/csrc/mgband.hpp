// mgband.hpp -- the multigrid-preconditioned CG of mgcg.hpp in row bands:
// the same hierarchy, V-cycle and CG recurrences (Sec. 3.3's Newton system),
// every value computed by the same operations in the same order, with about
// half the group barriers.
//
// A grid level's work is split by rows: member g of the group takes a band of
// rows and computes, in LDS, everything its band's outputs need, the few rows
// around the band included (recomputed there by both neighbours, with the same
// operations, so the values agree bit for bit).  One phase per level on the
// way down and one on the way up:
//   descent of level k: (level 0: the CG update of r, s, p, x), the two
//     pre-sweeps and the residual on the band's rows and two rows around
//     them, the restriction to the band's coarse rows;
//   coarse phase: the LDS levels' V-cycle in every workgroup, then the ascent
//     of the finest grid level above it;
//   ascent of level k: the coarse correction and the two post-sweeps (level
//     0: also w = A u and the block sums of (r, u), (w, u), (r, r), its band
//     then whole 256-cell blocks).
// A band phase reads only what earlier phases wrote (behind a group barrier);
// r and s, read around the band by the neighbours while the owner writes the
// next iterate, alternate between two buffers.  Per iteration: 2 Lg group
// barriers for Lg grid levels (1 when every level is an LDS level).  A band
// too long for the LDS is run in windows of rows, one after the other.
#pragma once

namespace iugkp {

// the part [lo, hi) of [0, N) that member g of G takes
__device__ __forceinline__ void band_split(int N, int g, int G, int &lo, int &hi)
{
  lo = static_cast<int>(static_cast<long long>(N) * g / G);
  hi = static_cast<int>(static_cast<long long>(N) * (g + 1) / G);
}

// CG update modes of the residual: the start (r = b, x = p = s = 0) and the
// iterations (the first with beta = 0)
constexpr int kMgStart = 0, kMgNext = 1;

// Window sizes, in the rows of the level, that a stage of `words` doubles
// holds (also used by the host to check that one row fits).  A staged buffer
// has rows of nx + 1 values, the last a zero pad, behind two zeros (kMgFront):
// an absent left or right neighbour reads the pad, a lower or upper one the
// zeros in front; kMgSlack words past the end may be read.
constexpr int kMgFront = 2, kMgSlack = 4;
constexpr int kMgWindow = 3 * (kMgFront + kMgSlack);
__host__ __device__ inline int band_down_rows(int words, int nx)   // coarse rows
{
  return ((words - kMgWindow) / (nx + 1) - 10) / 6;
}
__host__ __device__ inline int band_up_rows(int words, int nx)
{
  return ((words - kMgWindow) / (nx + 1) - 8) / 3;
}
__host__ __device__ inline int band_up0_blocks(int words, int nx, int block)
{
  const int rmax = ((words - kMgWindow) / (nx + 1) - 14) / 3;     // rows the blocks may span
  return ((rmax - 2) * nx + 1) / block;
}

// (Q0, Q1: cells of a thread in flight in the passes that load vectors, and in the sweeps)
template <int SPAN, int Q0, int Q1>
__device__ __forceinline__ void mgcg_band_solve(const MGArgs &in, int G, int bid, double *lds,
                                                double *red, MGLevel *s_lv)
{
  const MGArgs a = mg_args(in);
  const int nt = static_cast<int>(blockDim.x), tid = static_cast<int>(threadIdx.x);
  const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
  if (bid == 0 && tid == 0) a.sc->cg_t0 = static_cast<unsigned long long>(wall_clock64());
  const int L = a.L, Lg = a.Lg;
  mg_stage_levels(a.lv, L, s_lv);
  const MGLevel *lv = s_lv;
  const MGLevel L0 = mg_level(lv[0]);
  const int n = L0.n, nb = (n + kTree - 1) / kTree;
  // LDS: level Lg's result (kept through a band phase), the LDS levels' rows
  // (for the whole solve), then their vectors or a band window's staging
  double *const E = lds;
  double *const S = lds + a.stage0;
  const int SN = a.stage_n;
  unsigned int epoch = 0;
  mg_lds_rows(lv, Lg, L, lds, a.zero0, a.zero_n, a.slots);
  MgSlot sl[kMgSlots];
  mg_slots(lv, Lg, a.slots, sl);
  // (a division at every use would cost the phase more than a pass)
  if (tid < Lg) {
    MGLevel &F = s_lv[tid];
    band_split(lv[tid + 1].ny, bid, G, F.c0, F.c1);
    band_split(tid == 0 ? nb : F.ny, bid, G, F.r0, F.r1);
    const int dn = max(1, band_down_rows(SN, F.nx));
    const int up = max(1, tid == 0 ? band_up0_blocks(SN, F.nx, kTree) : band_up_rows(SN, F.nx));
    F.wdown = (F.c1 - F.c0 + dn - 1) / dn;
    F.wup = (F.r1 - F.r0 + up - 1) / up;
  }
  __syncthreads();

  auto bar = [&]() -> bool {
    if (G == 1) {
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      return true;
    }
    return flag_barrier<SPAN>(a.barrier, a.flags, bid, G, epoch);
  };

  // part w of nwin of the rows [lo, hi)
  auto window = [](int lo, int hi, int w, int nwin, int &a0, int &a1) {
    const unsigned m = static_cast<unsigned>(hi - lo);
    a0 = lo + static_cast<int>(m * w / nwin);
    a1 = lo + static_cast<int>(m * (w + 1) / nwin);
  };
  // a staged buffer of `rows` rows of nx values: its pads, and its words
  auto pads = [&](double *V, int rows, int nx) {
    for (int r = tid; r <= rows; r += nt) V[r * (nx + 1) + 1] = 0.0;
    if (tid == 0) V[0] = 0.0;
  };
  auto words = [](int rows, int nx) { return rows * (nx + 1) + kMgFront + kMgSlack; };
  // row of A at cell c (mesh row iy)
  auto row_at = [&](const MGLevel &F, int c, int iy) {
    MGRowZ r;
    r.dg = F.diag[c];
    r.rd = F.rd[c];
    r.gl = F.gxz[c + iy];
    r.gr = F.gxz[c + iy + 1];
    r.gd = F.gyz[c];
    r.gu = F.gyz[c + F.nx];
    return r;
  };
  // the five values of V around index j (mesh row iy of ny)
  struct V5 {
    double c, l, r, d, u;
  };
  auto around = [](const double *V, int j, int S, int iy, int ny) {
    return V5{V[j], V[j - 1], V[j + 1], V[iy > 0 ? j - S : 0], V[iy < ny - 1 ? j + S : 0]};
  };

  // Descent of grid level k for the coarse rows of this member: b and the
  // first sweep on the fine rows and two around them, the second sweep on
  // those and one around them (stored for the own rows), the residual and its
  // restriction on the own coarse rows.  Level 0's b is the updated residual:
  //   start: r = b, x = p = s = 0
  //   then:  s = w + beta s, r = r - alpha s, p = u + beta p, x = x + alpha p
  // computed on every staged cell and stored, with s, p and x, for the own ones.
  // (The loads of a cell have no branch between them, which would wait for
  // those before it: a cell of the halo loads u, p and x of the first own one.)
  struct Upd {
    double w, s, r, u, p, x, d, rd;
  };
  struct Bd {
    double b, d, rd;
  };
  auto descend = [&](int k, int mode, double alpha, double beta, const double *r_old,
                     double *r_new, const double *s_old, double *s_new) {
    const MGLevel F = mg_level(lv[k]), Cl = mg_level(lv[k + 1]);
    const int nx = F.nx, ny = F.ny, S1 = nx + 1;
    const int nwin = F.wdown;
#pragma unroll 1
    for (int w = 0; w < nwin; ++w) {
      int wY0 = F.c0, wY1 = F.c1;
      if (nwin > 1) window(F.c0, F.c1, w, nwin, wY0, wY1);
      const int fy0 = 2 * wY0, fy1 = min(2 * wY1, ny);
      const int by0 = max(0, fy0 - 2), by1 = min(ny, fy1 + 2);
      const int xy0 = max(0, fy0 - 1), xy1 = min(ny, fy1 + 1);
      const int nB = (by1 - by0) * nx, nX = (xy1 - xy0) * nx;
      const int wB = words(by1 - by0, nx);
      double *const B = S, *const X1 = S + wB, *const X2 = S + 2 * wB;
      pads(X1, by1 - by0, nx);
      pads(X2, xy1 - xy0, nx);
      const int ob0 = (fy0 - by0) * nx, ob1 = (fy1 - by0) * nx;   // own cells of the window
      auto at = [&](int i) { return i + mg_row_of(i, F.rnx) + kMgFront; };
      if (k == 0 && mode == kMgStart) {
        mg_cells<1>(
            nB, [&](int i) { const int c = by0 * nx + i; return Bd{a.b[c], F.diag[c], F.rd[c]}; },
            [&](int i, const Bd &v) {
              const int c = by0 * nx + i, j = at(i);
              if (i >= ob0 && i < ob1) {
                a.x[c] = 0.0;
                a.p[c] = 0.0;
                mst<SPAN>(&a.s[c], 0.0);
                mst<SPAN>(&r_new[c], v.b);
              }
              B[j] = v.b;
              X1[j] = mg_sweep_first_z(v.b, v.d, v.rd);
            });
      } else if (k == 0) {
        mg_cells<Q0>(
            nB,
            [&](int i) {
              const int c = by0 * nx + i, o = by0 * nx + (i >= ob0 && i < ob1 ? i : ob0);
              return Upd{mld<SPAN>(&a.w[c]),  mld<SPAN>(&s_old[c]), mld<SPAN>(&r_old[c]),
                         mld<SPAN>(&L0.e[o]), a.p[o],               a.x[o],
                         F.diag[c],           F.rd[c]};
            },
            [&](int i, const Upd &v) {
              const int c = by0 * nx + i, j = at(i);
              const double sv = v.w + beta * v.s;
              const double bv = v.r - alpha * sv;
              if (i >= ob0 && i < ob1) {
                const double pv = v.u + beta * v.p;
                a.p[c] = pv;
                a.x[c] = v.x + alpha * pv;
                mst<SPAN>(&s_new[c], sv);
                mst<SPAN>(&r_new[c], bv);
              }
              B[j] = bv;
              X1[j] = mg_sweep_first_z(bv, v.d, v.rd);
            });
      } else {
        mg_cells<Q1>(
            nB,
            [&](int i) {
              const int c = by0 * nx + i;
              return Bd{mld<SPAN>(&F.b[c]), F.diag[c], F.rd[c]};
            },
            [&](int i, const Bd &v) {
              const int j = at(i);
              B[j] = v.b;
              X1[j] = mg_sweep_first_z(v.b, v.d, v.rd);
            });
      }
      __syncthreads();
      const int dj = (xy0 - by0) * S1;               // X2's index to B's
      const int ox0 = (fy0 - xy0) * nx, ox1 = (fy1 - xy0) * nx;
      mg_cells<Q1>(
          nX, [&](int i) { return row_at(F, xy0 * nx + i, xy0 + mg_row_of(i, F.rnx)); },
          [&](int i, const MGRowZ &rw) {
            const int r = mg_row_of(i, F.rnx), j = i + r + kMgFront;
            const V5 x = around(X1, j + dj, S1, xy0 + r, ny);
            const double v = mg_sweep_z(rw, B[j + dj], x.c, x.l, x.r, x.d, x.u);
            X2[j] = v;
            if (i >= ox0 && i < ox1) mst<SPAN>(&F.xb[xy0 * nx + i], v);
          });
      __syncthreads();
      // (four children: their twelve values and rows loaded once each; an
      // absent child's are read at its neighbour, and its residual not used)
      struct Four {
        double dg[4], gx0[3], gx1[3], gd[2], gm[2], gu[2];
      };
      mg_cells<1>(
          (wY1 - wY0) * Cl.nx,
          [&](int i) {
            const int R = mg_row_of(i, Cl.rnx), I = i - R * Cl.nx, iy = 2 * (wY0 + R);
            const bool up = iy + 1 < ny;
            const int c = iy * nx + 2 * I, c1 = up ? c + nx : c;
            const int f = c + iy, f1 = up ? f + S1 : f;
            const int e = 2 * I + 1 < nx ? 1 : 0;
            return Four{{F.diag[c], F.diag[c + e], F.diag[c1], F.diag[c1 + e]},
                        {F.gxz[f], F.gxz[f + 1], F.gxz[f + 2]},
                        {F.gxz[f1], F.gxz[f1 + 1], F.gxz[f1 + 2]},
                        {F.gyz[c], F.gyz[c + e]},
                        {F.gyz[c + nx], F.gyz[c + nx + e]},
                        {F.gyz[c1 + nx], F.gyz[c1 + nx + e]}};
          },
          [&](int i, const Four &f) {
            const int R = mg_row_of(i, Cl.rnx), I = i - R * Cl.nx, iy = 2 * (wY0 + R);
            const bool right = 2 * I + 1 < nx, up = iy + 1 < ny;
            const int j = (iy - xy0) * S1 + 2 * I + kMgFront;
            // (the zeros in front for a row outside the mesh)
            const int jd = iy > 0 ? j - S1 : 0, j1 = up ? j + S1 : 0;
            const int j2 = iy + 2 < ny ? j + 2 * S1 : 0;
            const double *V = X2, *Bv = B + dj;
            const double v00 = V[j], v01 = V[j + 1], v10 = V[j1], v11 = V[j1 + 1];
            const double vl = V[j - 1], vr = V[j + 2], wl = V[up ? j1 - 1 : 0], wr = V[j1 + 2];
            const MGRowZ r0{f.dg[0], 0.0, f.gx0[0], f.gx0[1], f.gd[0], f.gm[0]};
            const MGRowZ r1{f.dg[1], 0.0, f.gx0[1], f.gx0[2], f.gd[1], f.gm[1]};
            const MGRowZ r2{f.dg[2], 0.0, f.gx1[0], f.gx1[1], f.gm[0], f.gu[0]};
            const MGRowZ r3{f.dg[3], 0.0, f.gx1[1], f.gx1[2], f.gm[1], f.gu[1]};
            const double q0 = Bv[j] - mg_apply_z(r0, v00, vl, v01, V[jd], v10);
            const double q1 = Bv[j + 1] - mg_apply_z(r1, v01, v00, vr, V[jd + 1], v11);
            const double q2 = Bv[j1] - mg_apply_z(r2, v10, wl, v11, v00, V[j2]);
            const double q3 = Bv[j1 + 1] - mg_apply_z(r3, v11, v10, wr, v01, V[j2 + 1]);
            mst<SPAN>(&Cl.b[wY0 * Cl.nx + i],
                      (q0 + (right ? q1 : 0.0)) + ((up ? q2 : 0.0) + (right && up ? q3 : 0.0)));
          });
      __syncthreads();
    }
  };

  // The corrected x of the mesh rows [cy0, cy1) into XC, and b of the rows
  // [py0, py1) into B, for an ascent of level F.
  struct Xcb {
    double xb, e, b;
  };
  auto correct = [&](const MGLevel &F, const MGLevel &Cl, const double *bsrc, bool e_lds, int cy0,
                     int cy1, int py0, int py1, double *XC, double *B) {
    const int nx = F.nx, S1 = nx + 1;
    const int ob0 = (py0 - cy0) * nx, ob1 = (py1 - cy0) * nx, dj = (py0 - cy0) * S1;
    pads(XC, cy1 - cy0, nx);
    auto cells = [&](auto e_of) {
      mg_cells<Q0>(
          (cy1 - cy0) * nx,
          [&](int i) {
            const int r = mg_row_of(i, F.rnx), iy = cy0 + r, ix = i - r * nx;
            const int c = cy0 * nx + i, o = cy0 * nx + (i >= ob0 && i < ob1 ? i : ob0);
            return Xcb{mld<SPAN>(&F.xb[c]), e_of((iy >> 1) * Cl.nx + (ix >> 1)), mld<SPAN>(&bsrc[o])};
          },
          [&](int i, const Xcb &v) {
            const int j = i + mg_row_of(i, F.rnx) + kMgFront;
            XC[j] = v.xb + kMgScale * v.e;
            if (i >= ob0 && i < ob1) B[j - dj] = v.b;
          });
    };
    if (e_lds) cells([&](int P) { return E[P]; });
    else cells([&](int P) { return mld<SPAN>(&Cl.e[P]); });
  };
  // A sweep on V (first mesh row vy0) of the mesh rows [y0, y1) of level F, b in
  // B (first mesh row by0); out(i, j, v): cell i of the rows, j = its index in
  // a buffer that starts with them
  auto sweep = [&](const MGLevel &F, const double *V, int vy0, const double *B, int by0, int y0,
                   int y1, auto out) {
    const int nx = F.nx, S1 = nx + 1, dv = (y0 - vy0) * S1, db = (y0 - by0) * S1;
    mg_cells<Q1>(
        (y1 - y0) * nx, [&](int i) { return row_at(F, y0 * nx + i, y0 + mg_row_of(i, F.rnx)); },
        [&](int i, const MGRowZ &rw) {
          const int r = mg_row_of(i, F.rnx), j = i + r + kMgFront;
          const V5 x = around(V, j + dv, S1, y0 + r, F.ny);
          out(i, j, mg_sweep_z(rw, B[j + db], x.c, x.l, x.r, x.d, x.u));
        });
  };

  // the products of one 256-cell block and its published sums; u and w
  // stored (rows: the block's four rows of A per lane, loaded together)
  auto block_sums = [&](int blk, auto row, auto vals) {
    MGRowZ rw[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c0 = blk * kTree + lane + 64 * q;
      rw[q] = row(c0 < n ? c0 : blk * kTree);
    }
    double g[4], d[4], rr[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c0 = blk * kTree + lane + 64 * q;
      const bool in = c0 < n;
      const int c = in ? c0 : blk * kTree;
      double uc, wv, rv;
      vals(c, rw[q], uc, wv, rv);
      g[q] = in ? rv * uc : 0.0;
      d[q] = in ? wv * uc : 0.0;
      rr[q] = in ? rv * rv : 0.0;
      if (in) {
        mst<SPAN>(&L0.e[c], uc);
        mst<SPAN>(&a.w[c], wv);
      }
    }
    const double sg = wave_tree256(g[0], g[1], g[2], g[3]);
    const double sd = wave_tree256(d[0], d[1], d[2], d[3]);
    const double sr = wave_tree256(rr[0], rr[1], rr[2], rr[3]);
    if (lane == 0) {
      mst<SPAN>(&a.part[3 * blk], sg);
      mst<SPAN>(&a.part[3 * blk + 1], sd);
      mst<SPAN>(&a.part[3 * blk + 2], sr);
    }
  };

  // Ascent of grid level k, from the coarse result in LDS (e_lds) or from level
  // k+1's e.  k >= 1, for this member's rows: x after the coarse correction on
  // the rows and two around them, the first post-sweep on the rows and one
  // around them, the second on the rows (stored as e of level k).  Level 0, with
  // w = A u and the block sums, for this member's 256-cell blocks, a window of
  // whole blocks at a time: corrected x on the blocks' rows and three around
  // them, the first post-sweep on two around, u on one around, w on the blocks.
  // r: level 0's current residual.
  auto ascend = [&](int k, bool e_lds, const double *r) {
    const MGLevel F = mg_level(lv[k]), Cl = mg_level(lv[k + 1]);
    const int nx = F.nx, ny = F.ny, S1 = nx + 1;
    const bool top = k == 0;
    const int nwin = F.wup;
#pragma unroll 1
    for (int w = 0; w < nwin; ++w) {
      int w0 = F.r0, w1 = F.r1;                      // rows, or blocks of level 0
      if (nwin > 1) window(F.r0, F.r1, w, nwin, w0, w1);
      int ya = w0, yb = w1;                          // rows of the second post-sweep
      if (top) {
        ya = max(0, w0 * kTree / nx - 1);
        yb = min(ny, (min(w1 * kTree, n) - 1) / nx + 2);
      }
      const int cy0 = max(0, ya - 2), cy1 = min(ny, yb + 2);
      const int py0 = max(0, ya - 1), py1 = min(ny, yb + 1);
      // (u overwrites the corrected x, read only by the first post-sweep)
      double *const XC = S, *const B = XC + words(cy1 - cy0, nx), *const P1 = B + words(py1 - py0, nx);
      double *const U = S;
      correct(F, Cl, top ? r : F.b, e_lds, cy0, cy1, py0, py1, XC, B);
      pads(P1, py1 - py0, nx);
      __syncthreads();
      sweep(F, XC, cy0, B, py0, py0, py1, [&](int, int j, double v) { P1[j] = v; });
      __syncthreads();
      if (top) pads(U, yb - ya, nx);
      sweep(F, P1, py0, B, py0, ya, yb, [&](int i, int j, double v) {
        if (top) U[j] = v;
        else mst<SPAN>(&F.e[ya * nx + i], v);
      });
      __syncthreads();
      if (top) {
        const int db = (ya - py0) * S1;
        for (int blk = w0 + wave; blk < w1; blk += nw)
          block_sums(
              blk, [&](int c) { return row_at(F, c, ya + mg_row_of(c - ya * nx, F.rnx)); },
              [&](int c, const MGRowZ &rw, double &uc, double &wv, double &rv) {
                const int i = c - ya * nx, q = mg_row_of(i, F.rnx), j = i + q + kMgFront;
                const V5 u = around(U, j, S1, ya + q, ny);
                uc = u.c;
                wv = mg_apply_z(rw, u.c, u.l, u.r, u.d, u.u);
                rv = B[j + db];
              });
        __syncthreads();
      }
    }
  };

  // The coarse phase: the LDS levels' V-cycle in every workgroup; with no grid
  // level, the CG update
  // of every cell first (its own cells stored) and w = A u with the block
  // sums of the own blocks after.
  auto coarse = [&](int mode, double alpha, double beta, const double *r_old, double *r_new,
                    const double *s_old, double *s_new) {
    const MGLevel T = lv[Lg];
    const bool Y = T.ny > 1;
    auto at0 = [&](int c) { return c + mg_row_of(c, T.rnx) + (Y ? T.nx + 1 : 1); };
    int o0 = 0, o1 = 0;
    if (Lg == 0) {
      band_split(nb, bid, G, o0, o1);
      const int c0 = o0 * kTree, c1 = min(o1 * kTree, n);
      if (mode == kMgStart)
        mg_cells<1>(
            n, [&](int c) { return a.b[c]; },
            [&](int c, double v) {
              if (c >= c0 && c < c1) {
                a.x[c] = 0.0;
                a.p[c] = 0.0;
                mst<SPAN>(&a.s[c], 0.0);
                mst<SPAN>(&r_new[c], v);
              }
              lds[T.lb + at0(c)] = v;
            });
      else
        mg_cells<1>(
            n,
            [&](int c) {
              const int o = c >= c0 && c < c1 ? c : c0;
              return Upd{mld<SPAN>(&a.w[c]), mld<SPAN>(&s_old[c]), mld<SPAN>(&r_old[c]),
                         mld<SPAN>(&L0.e[o]), a.p[o], a.x[o], 0.0, 0.0};
            },
            [&](int c, const Upd &v) {
              const double sv = v.w + beta * v.s;
              const double bv = v.r - alpha * sv;
              if (c >= c0 && c < c1) {
                const double pv = v.u + beta * v.p;
                a.p[c] = pv;
                a.x[c] = v.x + alpha * pv;
                mst<SPAN>(&s_new[c], sv);
                mst<SPAN>(&r_new[c], bv);
              }
              lds[T.lb + at0(c)] = bv;
            });
    }
    __syncthreads();
    mg_lds_cycle<SPAN>(lv, Lg, L, lds, Lg > 0 ? E : nullptr, Lg > 0, a.zero0, a.zero_n,
                       sl, a.slots);
    if (Lg == 0) {
      for (int blk = o0 + wave; blk < o1; blk += nw)
        block_sums(
            blk,
            [&](int c) {
              const double *C = lds + c + mg_row_of(c, T.rnx);
              return MGRowZ{C[T.dg], 0.0, C[T.lgx], C[T.lgx + 1], Y ? C[T.lgy] : 0.0,
                            Y ? C[T.lgy + T.nx + 1] : 0.0};
            },
            [&](int c, const MGRowZ &rw, double &uc, double &wv, double &rv) {
              const int j = at0(c);
              const double *V = lds + T.lt + j;
              uc = V[0];
              wv = mg_apply_z(rw, V[0], V[-1], V[1], Y ? V[-(T.nx + 1)] : 0.0,
                              Y ? V[T.nx + 1] : 0.0);
              rv = lds[T.lb + j];
            });
    }
  };

  // one application of the preconditioner and the operator to the updated
  // residual, with its block sums
  auto iterate = [&](int mode, double alpha, double beta, int cur) -> bool {
    const double *r_old = cur ? a.r2 : L0.b;
    double *r_new = (mode == kMgStart) ? L0.b : (cur ? L0.b : a.r2);
    const double *s_old = cur ? a.s2 : a.s;
    double *s_new = cur ? a.s : a.s2;
#pragma unroll 1
    for (int k = 0; k < Lg; ++k) {
      descend(k, mode, alpha, beta, r_old, r_new, s_old, s_new);
      if (!bar()) return false;
    }
    coarse(mode, alpha, beta, r_old, r_new, s_old, s_new);
    if (Lg == 0) return bar();
#pragma unroll 1
    for (int k = Lg - 1; k >= 0; --k) {
      ascend(k, k == Lg - 1, r_new);
      if (!bar()) return false;
    }
    return true;
  };

  int status = -7, it = 0, cur = 0;
  double alpha = 0.0, beta = 0.0, gamma = 0.0, delta = 0.0, thr = 0.0;
  int mode = kMgStart;
#pragma unroll 1
  do {
    if (!iterate(mode, alpha, beta, cur)) {
      status = -3;
      break;
    }
    double s3[3];
    group_tree_n<3, SPAN>(a.part, nb, red, s3);
    const double gamma_new = s3[0];
    delta = s3[1];
    if (mode == kMgStart) {
      thr = a.tol2 * s3[2];
      if (s3[2] == 0.0) status = 0;
      else if (!(delta > 0.0)) status = -6;
      else alpha = gamma_new / delta;
      mode = kMgNext;
    } else {
      cur ^= 1;
      ++it;
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
    }
    gamma = gamma_new;
  } while (status == -7 && it < a.max_iters);
  if (bid == 0 && tid == 0) {
    a.sc->cg_iters = it;
    a.sc->cg_status = status;
    a.sc->cg_t1 = static_cast<unsigned long long>(wall_clock64());
  }
}

}  // namespace iugkp
