// af_cells.h -- the cell update's tile for the FP64 stage (gfx950).  The
// FP32-bulk stage's tile (cells_tile in af_tiles.h) keeps its own: its results
// depend on how its FP32 sums are ordered and fused.
#pragma once
#include "af_points.h"
#include "af_tiles.h"

namespace afm {
namespace fp64 {

// One launch computes the cell averages of the stage for a tile of
// (CBX-3) x (CBY-3) cells; the block's CBX x CBY threads cover the cells whose
// flux-limiter box is needed plus one trailing row/column whose left and bottom
// interfaces close the region.  Per thread (cell (i,j)):
//   1  sensor primitives of the cells and a two-cell ring, then shock-sensor
//      indicators of the cells and one ring (LDS)
//   2  the x-interface at the cell's left and the y-interface below it --
//      Simpson flux, LLF flux, theta^s; the LLF flux goes to the cell on the
//      low side, in x by lane exchange (a tile row is 16 or 32 lanes of a
//      wavefront), in y through LDS
//   3  the LLF update G; sources, flux-limiter step (1), the density box and
//      the sufficient test of step (2); the cells that fail it are listed
//   4  step (2) of the listed cells, a lane per vertex
//   5  interface coefficients, limited update in flux form (see cells_tile for
//      the formulas)
// The neighbour's wave speeds are evaluated again from the average that is
// loaded anyway: exchanging them costs the same instructions (the tile's first
// lanes evaluate theirs in any case), LDS and a barrier.  Two groups of threads
// per tile, as the point tile has, do not pay here: each interface and round of
// indicators is shorter, but phases 3 and 5 run on half the waves (272 us against
// 231 us with one, blast 1024^2).
template <int CBX, int CBY>
struct CellsLDS64 {
  static constexpr int N = CBX * CBY;
  // theta^s (F_simpson - F^LLF) at the x-interface left of each cell, the
  // y-interface below; before: the primitives
  double df[2][NV][CBY][CBX];
  double fly[NV][CBY][CBX];    // F^LLF at the y-interface
  double a1[NV][N];            // A^{Lim,1} of the listed cells, then their Lambda
  double ts[2][CBY][CBX];      // theta^s
  union {
    double phi[4][CBY + 1][CBX + 1];  // indicators
    struct {
      double lam[2][CBY][CBX];        // Lambda_D, Lambda_U
      double eps[2][N];               // eps_rho, eps_p of the listed cells
      unsigned short q[N];            // listed cells: ty * CBX + tx
    } l;
  };
  int n;                              // cells listed
};

// a / b for b normal and r its reciprocal to the last place or so: the
// quotient's residual corrects it, which rounds as an IEEE division does.
__device__ __forceinline__ double div_by(double a, double b, double r) {
#pragma clang fp contract(off)
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// sensor_prims (p_t, v1, v2, B1, B2) with one reciprocal for its divisions.
__device__ __forceinline__ void cell_prims(const double U[NV], double gm1, double q[5]) {
#pragma clang fp contract(off)
  const double m2 = U[1] * U[1] + U[2] * U[2] + U[3] * U[3];
  const double b2 = U[4] * U[4] + U[5] * U[5] + U[6] * U[6];
  const double r = rcp_r(U[0]);
  q[0] = gm1 * (U[7] - div_by(0.5 * m2, U[0], r) - b2 / 2.0) + b2 / 2.0;
  q[1] = div_by(U[1], U[0], r);
  q[2] = div_by(U[2], U[0], r);
  q[3] = U[4];
  q[4] = U[5];
}

// sensor_from_prims at the place p of the primitives' fields (rows of PW,
// fields of PN), the divisions by 2 dx and 2 dy by their reciprocals.
template <int PW, int PN>
__device__ __forceinline__ void cell_indicators(const double* p, const Geo& g, double phi[4]) {
#pragma clang fp contract(off)
  const double c = p[0], l = p[-1], r = p[1], d = p[-PW], u = p[PW];
  phi[0] = fabs(r - 2.0 * c + l) / fabs(r + 2.0 * c + l);
  phi[1] = fabs(u - 2.0 * c + d) / fabs(u + 2.0 * c + d);
  const double x2 = 2.0 * g.dx, y2 = 2.0 * g.dy, rx = 0.5 * g.rdx, ry = 0.5 * g.rdy;
  const double *v1 = p + PN, *v2 = p + 2 * PN, *b1 = p + 3 * PN, *b2 = p + 4 * PN;
  const double dv = div_by(v1[1] - v1[-1], x2, rx) + div_by(v2[PW] - v2[-PW], y2, ry);
  const double cv = div_by(v2[1] - v2[-1], x2, rx) - div_by(v1[PW] - v1[-PW], y2, ry);
  phi[2] = fmax(-dv / sqrt(dv * dv + cv * cv + 1e-40), 0.0);
  phi[3] = fabs(b1[1] - b1[-1] + b2[PW] - b2[-PW]) / (fabs(b1[0] + b2[0]) + 1e-40);
}

// A thread's place in the cell tile, derived anew in each phase (see PtPlace).
struct CellPlace {
  int tx, ty, i, j;
};
template <int CBX, int CBY>
__device__ __forceinline__ CellPlace cell_place(const Geo& g, int bx, int by, int tid) {
  asm volatile("" : "+v"(tid));
  CellPlace t;
  t.tx = tid % CBX;
  t.ty = tid / CBX;
  t.i = clamp_cell(bx * (CBX - 3) - 1 + t.tx, g.nx);
  t.j = clamp_cell(by * (CBY - 3) - 1 + t.ty, g.ny);
  return t;
}

// The interface of direction DIR on the low side of the thread's cell, between
// the averages of the low side and A, w0 = V(i,j) its first edge point: F^LLF
// into Fl, theta^s (F_simpson - F^LLF) into LDS.
template <int DIR, int CBX, int CBY>
__device__ __forceinline__ void cell_interface(CellsLDS64<CBX, CBY>& L, const Geo& g, CState u, const CellPlace& t,
                                               const double A[NV], const double w0[NV], double Fl[NV]) {
  double AN[NV], w1[NV], w2[NV];
  if (DIR == 0) {
    ldX(g, u.x, t.i, t.j, w1);
    ldV(g, u.v, t.i, t.j + 1, w2);
    ldA(g, u.a, t.i - 1, t.j, AN);
  } else {
    ldY(g, u.y, t.i, t.j, w1);
    ldV(g, u.v, t.i + 1, t.j, w2);
    ldA(g, u.a, t.i, t.j - 1, AN);
  }
  // what needs no load first
  double pa[4], pb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    pa[q] = DIR == 0 ? L.phi[q][t.ty + 1][t.tx] : L.phi[q][t.ty][t.tx + 1];
    pb[q] = L.phi[q][t.ty + 1][t.tx + 1];
  }
  const double ts = sensor_theta(g.kappa, pa, pb, DIR);
  L.ts[DIR][t.ty][t.tx] = ts;
  DirEval eA, eN;
  eval_dir(A, g, DIR, eA);
  double Fh[NV], F[NV];
  flux_dir(w0, g.gm1, DIR, Fh);
  flux_dir(w1, g.gm1, DIR, F);
#pragma unroll
  for (int c = 0; c < NV; ++c) Fh[c] += 4.0 * F[c];
  flux_dir(w2, g.gm1, DIR, F);
#pragma unroll
  for (int c = 0; c < NV; ++c) Fh[c] = (Fh[c] + F[c]) * (1.0 / 6.0);
  eval_dir(AN, g, DIR, eN);
  const double al = alpha_llf(eN, eA, AN, A);
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    Fl[c] = 0.5 * (eN.F[c] + eA.F[c] - al * (A[c] - AN[c]));
    L.df[DIR][c][t.ty][t.tx] = ts * Fh[c] + (1.0 - ts) * Fl[c] - Fl[c];
  }
}

// Whether the thread's cell is one the tile updates.
template <int CBX, int CBY>
__device__ __forceinline__ bool cell_output(const Geo& g, int i0, int j0, int tx, int ty) {
  return tx >= 1 && tx < CBX - 2 && ty >= 1 && ty < CBY - 2 && i0 + tx < g.nx && j0 + ty < g.ny;
}

// Component c of the anti-diffusive update H_I (I = L, R, D, U) of cell (tx, ty).
template <int CBX, int CBY>
__device__ __forceinline__ double cell_H(const CellsLDS64<CBX, CBY>& L, int tx, int ty, double lx, double ly, int I,
                                         int c) {
  const int txr = tx + 1 < CBX ? tx + 1 : tx, tyu = ty + 1 < CBY ? ty + 1 : ty;
  switch (I) {
    case 0: return lx * L.df[0][c][ty][tx];
    case 1: return -lx * L.df[0][c][ty][txr];
    case 2: return ly * L.df[1][c][ty][tx];
    default: return -ly * L.df[1][c][tyu][tx];
  }
}

// Step (2) of the flux limiter for the listed cells, sixteen lanes a cell
// (limiter_box_lanes).
template <int CBX, int CBY>
__device__ __forceinline__ void box_listed(CellsLDS64<CBX, CBY>& L, const Geo& g, int i0, int j0, double lx,
                                           double ly, Counters* cn, int tid) {
  const int n = L.n;
  for (int m = tid / 16; m < n; m += CBX * CBY / 16) {
    const int tx = L.l.q[m] % CBX, ty = L.l.q[m] / CBX;
    double A1[NV], lam[4];
#pragma unroll
    for (int c = 0; c < NV; ++c) A1[c] = L.a1[c][m];
    auto H = [&](int I, int c) -> double { return cell_H(L, tx, ty, lx, ly, I, c); };
    limiter_box_lanes(A1, H, g.gm1, L.l.eps[0][m], L.l.eps[1][m], lam, cn, cell_output<CBX, CBY>(g, i0, j0, tx, ty),
                      tid);
    if ((tid & 15) == 0) {
#pragma unroll
      for (int I = 0; I < 4; ++I) L.a1[I][m] = lam[I];
      L.l.lam[0][ty][tx] = lam[2];
      L.l.lam[1][ty][tx] = lam[3];
    }
  }
}

// One tile of the cell update.  tid: the thread in the tile's CBX CBY.
// src: the point kernel's nine-point sources, or null (every cell computes
// its own from the stage input, as the ghost cells do).  wslot: as in
// points_tile.
template <int CBX, int CBY>
__device__ __forceinline__ void cells_tile(const Geo& g, CState u, const double* __restrict__ src, const double* un,
                                           double* out, double dt, double ca, double cb, Counters* cn, int bx, int by,
                                           CellsLDS64<CBX, CBY>& L, double* __restrict__ wslot, int tid) {
  constexpr int CNT = CBX * CBY;
  const int i0 = bx * (CBX - 3) - 1, j0 = by * (CBY - 3) - 1;
  const double lx = dt * g.rdx, ly = dt * g.rdy;

  // 1a: sensor primitives on [i0-2, i0+CBX+1) x [j0-2, j0+CBY+1): one or two
  //     per thread, the loads of both issued first
  constexpr int PW = CBX + 3, PH = CBY + 3;
  static_assert(CNT < PW * PH && PW * PH <= 2 * CNT && 5 * PW * PH <= 2 * NV * CNT, "primitives in df's place");
  double* const prim = &L.df[0][0][0][0];
  {
    const int it2 = tid + CNT;
    const bool two = it2 < PW * PH;
    double U[NV], U2[NV], q[5];
    ldA(g, u.a, clamp_prim(i0 - 2 + tid % PW, g.nx), clamp_prim(j0 - 2 + tid / PW, g.ny), U);
    if (two) ldA(g, u.a, clamp_prim(i0 - 2 + it2 % PW, g.nx), clamp_prim(j0 - 2 + it2 / PW, g.ny), U2);
    cell_prims(U, g.gm1, q);
#pragma unroll
    for (int m = 0; m < 5; ++m) prim[m * PW * PH + tid] = q[m];
    if (two) {
      cell_prims(U2, g.gm1, q);
#pragma unroll
      for (int m = 0; m < 5; ++m) prim[m * PW * PH + it2] = q[m];
    }
  }
  __syncthreads();
  // the div B of the LLF source (the primitives hold B exactly); the cell's
  // average, source and first edge point: in flight while the indicators are
  // formed (more of the interfaces' loads here costs more in registers than it
  // hides)
  double A[NV], S[NV], w0[NV], divb;
  {
    const CellPlace t = cell_place<CBX, CBY>(g, bx, by, tid);
    const int pc = (t.ty + 2) * PW + (t.tx + 2);
    divb = (prim[3 * PW * PH + pc + 1] - prim[3 * PW * PH + pc - 1]) * (0.5 * g.rdx);
    divb += (prim[4 * PW * PH + pc + PW] - prim[4 * PW * PH + pc - PW]) * (0.5 * g.rdy);
    ldA(g, u.a, t.i, t.j, A);
    if (src) ldA(g, src, t.i, t.j, S);
    ldV(g, u.v, t.i, t.j, w0);
    if (tid == 0) L.n = 0;
  }
  // 1b: indicators on [i0-1, i0+CBX) x [j0-1, j0+CBY)
  for (int it = tid; it < (CBX + 1) * (CBY + 1); it += CNT) {
    const int a = it % (CBX + 1), b = it / (CBX + 1);
    double ph[4];
    cell_indicators<PW, PW * PH>(prim + (b + 1) * PW + (a + 1), g, ph);
#pragma unroll
    for (int q = 0; q < 4; ++q) L.phi[q][b][a] = ph[q];
  }
  __syncthreads();

  // 2
  double G[NV];
  {
    const CellPlace t = cell_place<CBX, CBY>(g, bx, by, tid);
    // the nine-point source: the point kernel's for the grid's cells; a ghost
    // cell across an outflow boundary (its mirrored stencil differs from its
    // image's) computes its own
    if (!src || (g.bcx && (t.i < 0 || t.i >= g.nx)) || (g.bcy && (t.j < 0 || t.j >= g.ny)))
      source_of_cell(g, u, t.i, t.j, S);
    double Fl[NV];
    cell_interface<0, CBX, CBY>(L, g, u, t, A, w0, Fl);
    // the right neighbour's flux: lane tx + 1 (the last column, whose update
    // is never used, takes its own)
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      const double fr = __shfl_down(Fl[c], 1);
      G[c] = A[c] + lx * (Fl[c] - (t.tx + 1 < CBX ? fr : Fl[c]));
    }
    pin8(G);
    cell_interface<1, CBX, CBY>(L, g, u, t, A, w0, Fl);
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      L.fly[c][t.ty][t.tx] = Fl[c];
      G[c] += ly * Fl[c];
    }
  }
  __syncthreads();

  // 3
  double Lam[4];
  int listed = -1;
  {
    const CellPlace t = cell_place<CBX, CBY>(g, bx, by, tid);
    const int tx = t.tx, ty = t.ty, txr = tx + 1 < CBX ? tx + 1 : tx, tyu = ty + 1 < CBY ? ty + 1 : ty;
    const double tsmin =
        fmin(fmin(L.ts[0][ty][tx], L.ts[0][ty][txr]), fmin(L.ts[1][ty][tx], L.ts[1][tyu][tx]));
#pragma unroll
    for (int c = 0; c < NV; ++c) G[c] -= ly * L.fly[c][tyu][tx];
    const bool output = cell_output<CBX, CBY>(g, i0, j0, tx, ty);
    double A1[NV], er, ep;
    {
      double Sl[NV], P[NV];
      psi(A, P);
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        Sl[c] = divb * P[c];
        S[c] = tsmin * S[c] + (1.0 - tsmin) * Sl[c];
      }
      const double th = source_step(G, S, Sl, dt, g.gm1, A1, er, ep, cn, output);
      // from here on G - dt S^Lim
#pragma unroll
      for (int c = 0; c < NV; ++c) G[c] -= dt * (th * S[c] + (1.0 - th) * Sl[c]);
    }
    auto H = [&](int I, int c) -> double { return cell_H(L, tx, ty, lx, ly, I, c); };
    if (!box_clear(A1, H, g.gm1, er, ep, Lam)) {
      listed = atomicAdd(&L.n, 1);
#pragma unroll
      for (int c = 0; c < NV; ++c) L.a1[c][listed] = A1[c];
      L.l.eps[0][listed] = er;
      L.l.eps[1][listed] = ep;
      L.l.q[listed] = (unsigned short)(ty * CBX + tx);
    } else {
      L.l.lam[0][ty][tx] = Lam[2];
      L.l.lam[1][ty][tx] = Lam[3];
    }
  }
  __syncthreads();
  // 4
  if (L.n > 0) {
    box_listed<CBX, CBY>(L, g, i0, j0, lx, ly, cn, tid);
    __syncthreads();
  }
  // 5: unique interface coefficients and the limited update: Lambda_R of the
  //    left neighbour and Lambda_L of the right one by lane shuffles,
  //    Lambda_U of the cell below and Lambda_D of the cell above through LDS
  double wm = 0.0;
  {
    const CellPlace t = cell_place<CBX, CBY>(g, bx, by, tid);
    const int tx = t.tx, ty = t.ty, i = t.i, j = t.j;
    if (listed >= 0) {
#pragma unroll
      for (int I = 0; I < 4; ++I) Lam[I] = L.a1[I][listed];
    }
    const double lamR_left = __shfl_up(Lam[1], 1), lamL_right = __shfl_down(Lam[0], 1);
    if (cell_output<CBX, CBY>(g, i0, j0, tx, ty)) {
      const long off = (long)j * g.nx + i;
      double Un[NV];
      if (ca != 0.0) load8(un, g.sc, off, Un);
      const double thL = fmin(lamR_left, Lam[0]);
      const double thR = fmin(Lam[1], lamL_right);
      const double thD = fmin(L.l.lam[1][ty - 1][tx], Lam[2]);
      const double thU = fmin(Lam[3], L.l.lam[0][ty + 1][tx]);
      if (thL < 1.0) { count(&cn->n_theta_active); count_min_theta(cn, thL); }
      if (thD < 1.0) { count(&cn->n_theta_active); count_min_theta(cn, thD); }
      if (g.bcx && i == g.nx - 1 && thR < 1.0) { count(&cn->n_theta_active); count_min_theta(cn, thR); }
      if (g.bcy && j == g.ny - 1 && thU < 1.0) { count(&cn->n_theta_active); count_min_theta(cn, thU); }
      const double hl = thL * lx, hr = thR * lx, hd = thD * ly, hu = thU * ly;
#pragma unroll
      for (int c = 0; c < NV; ++c)
        G[c] += (hl * L.df[0][c][ty][tx] - hr * L.df[0][c][ty][tx + 1]) +
                (hd * L.df[1][c][ty][tx] - hu * L.df[1][c][ty + 1][tx]);
      if (!in_G_fast(G)) count(&cn->n_not_admissible);
      if (ca != 0.0) {
#pragma unroll
        for (int c = 0; c < NV; ++c) G[c] = ca * Un[c] + cb * G[c];
      }
#pragma unroll
      for (int c = 0; c < NV; ++c) out[c * g.sc + off] = G[c];
      if (wslot) wm = dt_speed(G, g);
    }
  }
  if (wslot) {
    __syncthreads();  // ts is read no more: the scratch
    block_max_store(wm, tid, CNT, &L.ts[0][0][0], wslot);
  }
}

}  // namespace fp64

// LDS of a cell tile's workgroup, and the tile in either precision by all its
// threads (a flat block of CBX CBY).
template <class R, int CBX, int CBY> struct CellsTile { using LDS = fp64::CellsLDS64<CBX, CBY>; };
template <int CBX, int CBY> struct CellsTile<float, CBX, CBY> { using LDS = CellsLDS<float, CBX, CBY>; };
template <class R, int CBX, int CBY> using CellsTileLDS = typename CellsTile<R, CBX, CBY>::LDS;

template <class R, int CBX, int CBY>
__device__ __forceinline__ void cells_tile_any(const Geo& g, CState u, const double* __restrict__ src,
                                               const double* un, double* out, double dt, double ca, double cb,
                                               Counters* cn, int bx, int by, CellsTileLDS<R, CBX, CBY>& L,
                                               double* __restrict__ wslot) {
  if constexpr (IsF32<R>::value)
    cells_tile<R, CBX, CBY>(g, u, src, un, out, dt, ca, cb, cn, bx, by, L, wslot);
  else
    fp64::cells_tile<CBX, CBY>(g, u, src, un, out, dt, ca, cb, cn, bx, by, L, wslot, (int)threadIdx.x);
}

}  // namespace afm
