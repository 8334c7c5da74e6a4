// af_points.h -- the point update's tile for the FP64 stage (gfx950).  The
// FP32-bulk stage's tile is in af_tiles.h: its results depend on how its FP32
// sums are ordered and fused, so that it keeps the order below its own, and on
// one thread per point it is the faster one too (1303 us a step of the blast
// 1024^2 against 1457 us on this layout).
#pragma once
#include "af_tiles.h"

namespace afm {
namespace fp64 {

constexpr int PNT = 2 * PB * PB;

// Point accumulators: high-order RHS h = -R_x - R_y with the div part, and
// the bound that decides whether the point's first-order LLF state has to be
// formed (see llf_bound).
struct PointAcc {
  double h[NV];
  double divh, bnd;
};

__device__ __forceinline__ void acc_zero(PointAcc& P) {
#pragma unroll
  for (int c = 0; c < NV; ++c) P.h[c] = 0.0;
  P.divh = P.bnd = 0.0;
}

// ------------------------------------------- when the LLF state is needed
// The scaling limiter returns the high-order state unchanged whenever that
// state and the first-order LLF state both satisfy rho, p >= 1e-13.  The
// Lemma of Section 3.1 gives the LLF state's lower bounds without forming it:
// with c = 1 - dt (sum of the four alpha / Delta + |div B| / sqrt(rho)) > 0 and
// admissible neighbours,
//   rho(U^LLF) >= c rho(U)   and   p(U^LLF) >= c p(U).
// The viscosity of a pair is at most max |v_n| + max c_f + |jump B| /
// (2 sqrt(min rho)), and each direction's share of |div B| / sqrt(rho) is
// bounded by the same last term, so that a direction adds at most
//   2 dt/Delta (max |v_n| + max c_f + sqrt(max |jump B|^2 max 1/rho)).
// A point whose two directions add up to at most LLF_BOUND has c >= 0.1;
// when also p(U) >= 2e-12, rho(U) >= 2e-12 and E of the stencil <= 5e11 p(U)
// (0.1 p(U) is then far above the 1e-16 E that rounding leaves in p(U^LLF)),
// the LLF state is known to pass its test, and neither it nor its fluxes are
// formed.  Every other point is listed: a point whose high-order state is not
// admissible for its limiter, any other for the count of LLF states outside G,
// the only thing that its LLF state decides (both of the limiter's bounds are at
// most 1e-13).  The bound costs a line about 30 instructions where its two LLF
// fluxes cost 130 (a tile of the blast 1024^2 issues 11.0 thousand wave
// instructions, where it took 14.0 with every LLF flux formed); at CFL 0.2 smooth
// flow stays near 0.4, above CFL 0.45 most points of a grid can fail it.
constexpr double LLF_BOUND = 0.9, LLF_MIN = 2e-12, LLF_EMAX = 5e11;

// One direction's term for a point: vc, llf_speeds of the three states; jump,
// the larger |jump B|^2 of the point's two pairs; em, the three states' largest
// E; p0, the point's pressure, pn, the neighbours' smallest; rj, the largest
// 1/rho.  A term that rules the shortcut out is 4 or more.
__device__ __forceinline__ double llf_bound(double vc, double jump, double em, double p0, double pn, double rj,
                                            double lam) {
  const double j = __builtin_amdgcn_sqrt(jump * rj);
  const bool ok = (pn > 0.0) & (p0 >= LLF_MIN) & (em <= LLF_EMAX * p0);
  return ok ? 2.0 * lam * (vc + j) : 4.0;
}
// max |v_n| + max c_f of a point (1/rho r0) and its neighbours (ra, rb); out
// of any bound where a density is not positive or the point's is too small.
__device__ __forceinline__ double llf_speeds(double v0, double va, double vb, double c0, double ca, double cb,
                                             double r0, double ra, double rb) {
  const bool ok = (fmin(r0, fmin(ra, rb)) > 0.0) & (r0 <= 1.0 / LLF_MIN);
  const double vc = fmax(v0, fmax(va, vb)) + fmax(c0, fmax(ca, cb));
  return ok ? vc : 1e30;
}
__device__ __forceinline__ double jump2(const double a[NV], const double b[NV]) {
  const double d1 = a[4] - b[4], d2 = a[5] - b[5], d3 = a[6] - b[6];
  return d1 * d1 + d2 * d2 + d3 * d3;
}

// LDS layout (fields of PB x PB values): the states of the tile's V, X, Y (the
// centre values take V's place once the vertices are finished), then what
// lines need of each point: 1/rho, total pressure, pressure and c_f in the
// direction of the lines in flight (both directions for V and the centre).
// point_exchange: where the vertical lines' part of the vertex accumulators
// goes to the other group, on fields that are read no more by then; after that
// LIST_, the tile's list of points, and QXY_, QYX_ (look_listed) on three of them.
constexpr int SV_ = 0, SX_ = 8, SY_ = 16, SC_ = SV_;
constexpr int QV_ = 24, QX_ = 29, QY_ = 33, QC_ = QV_;  // (1/rho, p_t, p, c_f[, c_f in y])
constexpr int POINT_FIELDS = 40;
__device__ __forceinline__ constexpr int point_exchange(int c) {  // ten fields
  return c < 5 ? QV_ + c : c == 5 ? QX_ + 3 : c == 6 ? QY_ + 3 : 30 + c;
}

// The listed points: kind << 8 | ty << 4 | tx (kind 0 V, 1 X, 2 Y), at most three
// for each of the (PB-2)^2 cells.  From the front those whose limiter acts, from
// the back those whose LLF state is only looked at.
constexpr int LOOK_END = 3 * (PB - 2) * (PB - 2);
struct PointList {
  int limit, look;
  unsigned short q[LOOK_END];
};
constexpr int LIST_ = 37, QXY_ = 38, QYX_ = 39;  // QXY_, QYX_: c_f of X in y, of Y in x (look_listed)
static_assert(sizeof(PointList) <= PB * PB * sizeof(double), "list in a spare field");
__device__ __forceinline__ PointList& point_list(double (*s)[PB][PB]) {
  return *reinterpret_cast<PointList*>(&s[LIST_][0][0]);
}
struct PointEnd {  // what a finished point still needs
  bool limit, look;
};
// Called by whole wavefronts: one LDS atomic each and list.
__device__ __forceinline__ void list_point(double (*s)[PB][PB], PointEnd end, int kind, int ty, int tx) {
  if (__builtin_expect(!__ballot(end.limit | end.look), 1)) return;
  PointList& L = point_list(s);
  const unsigned long long lim = __ballot(end.limit), look = __ballot(end.look);
  const int lane = __lane_id();
  int a = 0, b = 0;
  if (lane == 0) {
    if (lim) a = atomicAdd(&L.limit, __popcll(lim));
    if (look) b = atomicAdd(&L.look, __popcll(look));
  }
  a = __builtin_amdgcn_readfirstlane(a);
  b = __builtin_amdgcn_readfirstlane(b);
  const unsigned long long below = (1ull << lane) - 1;
  const int at = end.limit ? a + __popcll(lim & below) : LOOK_END - 1 - b - __popcll(look & below);
  if (end.limit | end.look) L.q[at] = (unsigned short)(kind << 8 | ty << 4 | tx);
}

// --------------------------------------------------- point tile
// 512 threads: two groups of PB x PB (wave-uniform), each on the whole tile.
//   load    group 0: V and its record, the cell average; group 1: X, Y, records
//   lines   0: b (V, and X's central part);  1: a (V, and Y's central part)
//   middle  0: centre value (kept in registers), nine-point source;
//           1: V finished with group 0's part of it
//   records 0: centre;                       1: X in x, Y in y
//   lines   0: c, X finished;                1: d, Y finished
//   end     listed points: limiter, four lanes a point; LLF states to be counted,
//           a lane each where they are many
// What bounds it is latency: dependent FP64 chains (reciprocals, square
// roots), LDS reads and barriers, so waves in flight decide.  Two groups that
// share one tile's LDS give four waves per SIMD at 80 KB per workgroup (two
// workgroups per CU) where one thread per cell gives two, and each thread
// keeps two line families' accumulators instead of four.  At 128 registers
// nothing may spill: spilled values go through HBM (60 of them a thread made
// the kernel 454 us instead of 207).  The direction-free part of a record is
// formed once per point and serves both directions.  A point's flux and
// spectral radius are rebuilt from its state and record (23 instructions; a
// stored flux would cost five more LDS reads).
__device__ __forceinline__ void pin_acc(PointAcc& P) {
#pragma unroll
  for (int c = 0; c < NV; ++c) asm volatile("" : "+v"(P.h[c]));
  asm volatile("" : "+v"(P.divh), "+v"(P.bnd));
}

// c_f in direction dir (eq. (cf)) of a state with pressure p and 1/rho ri,
// |B|^2 b2, with the operations of eval_dir.
__device__ __forceinline__ double fast_speed(const double U[NV], double gamma, double ri, double b2, double p,
                                             int dir) {
  const double Bn = dir ? U[5] : U[4];
  const double c2 = gamma * p * ri;
  const double s = c2 + b2 * ri;
  double disc = s * s - 4.0 * c2 * Bn * Bn * ri;
  disc = disc > 0.0 ? disc : 0.0;
  return sqrt_r(0.5 * (s + sqrt_r(disc)));
}

// A tile point's record into the fields from q on: 1/rho, total pressure,
// pressure, c_f in direction dir -- for V and the centre (both = true) in x
// and in y.
__device__ __forceinline__ void put_record(double (*s)[PB][PB], const Geo& g, int q, int ty, int tx, const double U[NV],
                                           bool both, int dir) {
  double ri, v1, v2, v3, b2, p;
  prim_r<double>(U, g.gm1, ri, v1, v2, v3, b2, p);
  s[q][ty][tx] = ri;
  s[q + 1][ty][tx] = p + 0.5 * b2;
  s[q + 2][ty][tx] = p;
  s[q + 3][ty][tx] = fast_speed(U, g.gamma, ri, b2, p, both ? 0 : dir);
  if (both) s[q + 4][ty][tx] = fast_speed(U, g.gamma, ri, b2, p, 1);
}

// State (field base sb) and flux (record base qb) of the tile point (ty, tx).
__device__ __forceinline__ void lean_pt(double (*s)[PB][PB], int sb, int qb, int ty, int tx, int dir, double F[NV],
                                        double U[NV]) {
  lds8(s, sb, ty, tx, U);
  const double ri = s[qb][ty][tx];
  flux_of<double, double>(U, dir, U[1] * ri, U[2] * ri, U[3] * ri, s[qb + 1][ty][tx], F);
}

// FVS line in direction dir through the tile point (ty, tx) of the type with
// state base so, record qo and c_f field co; the line's other type (sb, qb,
// cb) sits at -h/2 (point (ym, xm)) and +h/2 (the point itself), the own
// type's neighbours at -h (ym, xm) and +h (yp, xp).  alpha (the maximum
// spectral radius over the five) comes first, so that the FVS sums fold
// into one vector,
//   Q = F(-h) - 4F(-h/2) + 4F(+h/2) - F(+h)
//       + alpha (U(-h) - 4U(-h/2) + 6U - 4U(+h/2) + U(+h)),   h-part -= Q/(2h),
// in which the point's own flux does not occur.  Returns Q, the field sum dB
// and the direction's term of the LLF bound.  CENTRAL: the line's +h/2 point
// (the tile point of the other type) also takes its central difference
// across this line, between this point and the +h neighbour, into P2
// (families b and a), from the same fluxes.
template <bool CENTRAL>
__device__ __forceinline__ void lean_fvs(double (*s)[PB][PB], int dir, int so, int qo, int fo, int sb, int qb, int fb,
                                         int ty, int tx, int ym, int xm, int yp, int xp, double rh, double lam,
                                         double Q[NV], double& dB, double& bnd, PointAcc& P2) {
  const int bn = 4 + dir, mn = 1 + dir;
  const double ro = s[qo][ty][tx], rm = s[qo][ym][xm], rp = s[qo][yp][xp], rb = s[qb][ty][tx];
  const double co = s[fo][ty][tx], cm = s[fo][ym][xm], cp = s[fo][yp][xp], cb = s[fb][ty][tx];
  const double vo = fabs(s[so + mn][ty][tx] * ro), vm = fabs(s[so + mn][ym][xm] * rm),
          vp = fabs(s[so + mn][yp][xp] * rp), vb = fabs(s[sb + mn][ty][tx] * rb);
  double alpha = vo + co;
  alpha = fmax(alpha, vm + cm);
  alpha = fmax(alpha, fabs(s[sb + mn][ym][xm] * s[qb][ym][xm]) + s[fb][ym][xm]);
  alpha = fmax(alpha, vb + cb);
  alpha = fmax(alpha, vp + cp);
  double vc = llf_speeds(vo, vm, vp, co, cm, cp, ro, rm, rp), rj = fmax(ro, fmax(rm, rp)), vcb, rjb;
  asm volatile("" : "+v"(alpha), "+v"(vc), "+v"(rj));
  if constexpr (CENTRAL) {
    vcb = llf_speeds(vb, vo, vp, cb, co, cp, rb, ro, rp);
    rjb = fmax(rb, fmax(ro, rp));
    asm volatile("" : "+v"(vcb), "+v"(rjb));
  }
  double F[NV], Uo[NV], U[NV];
  if constexpr (CENTRAL) {
    lean_pt(s, so, qo, ty, tx, dir, F, Uo);
#pragma unroll
    for (int c = 0; c < NV; ++c) P2.h[c] += F[c] * rh;
    P2.divh -= Uo[bn] * rh;
  } else {
    lds8(s, so, ty, tx, Uo);
  }
#pragma unroll
  for (int c = 0; c < NV; ++c) Q[c] = 6.0 * alpha * Uo[c];
  // -h
  lean_pt(s, so, qo, ym, xm, dir, F, U);
#pragma unroll
  for (int c = 0; c < NV; ++c) Q[c] += F[c] + alpha * U[c];
  dB = U[bn];
  double jump = jump2(Uo, U), em = fmax(Uo[7], U[7]);
  pin8(Q);
  // +h
  lean_pt(s, so, qo, yp, xp, dir, F, U);
#pragma unroll
  for (int c = 0; c < NV; ++c) Q[c] += alpha * U[c] - F[c];
  dB -= U[bn];
  if constexpr (CENTRAL) {
#pragma unroll
    for (int c = 0; c < NV; ++c) P2.h[c] -= F[c] * rh;
    P2.divh += U[bn] * rh;
  }
  const double po = s[qo + 2][ty][tx], pp = s[qo + 2][yp][xp];
  bnd = llf_bound(vc, fmax(jump, jump2(Uo, U)), fmax(em, U[7]), po, fmin(s[qo + 2][ym][xm], pp), rj, lam);
  pin8(Q);
  {
    double Ui[NV];
    if constexpr (CENTRAL) {
      lds8(s, sb, ty, tx, Ui);
      P2.bnd += llf_bound(vcb, fmax(jump2(Ui, Uo), jump2(Ui, U)), fmax(Ui[7], fmax(Uo[7], U[7])), s[qb + 2][ty][tx],
                          fmin(po, pp), rjb, lam);
    }
    // -h/2, +h/2
    lean_pt(s, sb, qb, ym, xm, dir, F, Ui);
#pragma unroll
    for (int c = 0; c < NV; ++c) Q[c] -= 4.0 * (F[c] + alpha * Ui[c]);
    dB -= 4.0 * Ui[bn];
    lean_pt(s, sb, qb, ty, tx, dir, F, Ui);
#pragma unroll
    for (int c = 0; c < NV; ++c) Q[c] += 4.0 * (F[c] - alpha * Ui[c]);
    dB += 4.0 * Ui[bn];
  }
}

// A line's sums into the point's accumulators.
__device__ __forceinline__ void add_line(PointAcc& P, const double Q[NV], double dB, double bnd, double sh) {
#pragma unroll
  for (int c = 0; c < NV; ++c) P.h[c] -= Q[c] * sh;
  P.divh += dB * sh;
  P.bnd += bnd;
}

// The high-order state of a finished point from its accumulators, and, where
// the limiter returns it unchanged, SSP combination and store: where the bound
// shows it (see llf_bound), and where the state satisfies rho, p >= 1e-13 whatever
// the LLF state is (to be looked at: that one is still to be counted).  Elsewhere
// it goes to the same place of `stash` (to be limited).  un: the point's set of
// U^n (read only when ca != 0).
__device__ __forceinline__ PointEnd finish(const Geo& g, double dt, const double U0[NV], const PointAcc& P, double ca,
                                           double cb, const double* un, double* out, double* stash, long plane,
                                           long off, bool speeds, double& wm) {
  double UH[NV], Un[NV], Ps[NV];
  if (ca != 0.0) load8(un, plane, off, Un);  // in flight over the tests
  psi(U0, Ps);
#pragma unroll
  for (int c = 0; c < NV; ++c) UH[c] = U0[c] + dt * (P.h[c] - P.divh * Ps[c]);
  auto put = [&](double W[NV]) {
#pragma unroll
    for (int c = 0; c < NV; ++c) out[c * plane + off] = W[c];
    // a step's last stage: the next step's wave-speed maximum over its outputs
    if (speeds) wm = fmax(wm, dt_speed(W, g));
  };
  auto store = [&]() {  // with the SSP combination
    if (ca != 0.0) {
#pragma unroll
      for (int c = 0; c < NV; ++c) Un[c] = ca * Un[c] + cb * UH[c];
      put(Un);
      asm volatile("");  // the stores stay in the branch: joined, they cost 16 moves
    } else {
      put(UH);
    }
  };
  if (__builtin_expect(!((P.bnd <= LLF_BOUND) & (UH[0] >= EPS_FLOOR) & p_at_least(UH, EPS_FLOOR, g.gm1)), 0)) {
    // the limiter would look at the state again: by more than what its form of
    // the pressure can round (behind the empty asm, or it is formed for all)
    double E = UH[7];
    asm volatile("" : "+v"(E));
    if ((UH[0] >= EPS_FLOOR) & p_at_least(UH, fma(1e-14 * g.gm1, E, EPS_FLOOR), g.gm1)) {
      store();
      return PointEnd{false, true};
    }
#pragma unroll
    for (int c = 0; c < NV; ++c) stash[c * plane + off] = UH[c];
    return PointEnd{true, false};
  }
  store();
  return PointEnd{false, false};
}

// The value of a kind (0 V, 1 X, 2 Y) out of three uniform ones.  The empty
// asm keeps the choice on values: the compiler otherwise chooses an address
// within the struct that holds them, which then lies in scratch memory.
template <class T>
__device__ __forceinline__ T of_kind(int kind, T v, T x, T y) {
  asm("" : "+s"(v));
  asm("" : "+s"(x));
  asm("" : "+s"(y));
  return kind == 0 ? v : kind == 1 ? x : y;
}

// The state of point (i,j) of a kind of the stage input.
__device__ __forceinline__ void load_point(const Geo& g, CState u, int kind, int i, int j, double U[NV]) {
  const int ii = kind == 2 ? map_cell(i, g.nx, g.bcx) : map_node(i, g.nx, g.bcx);
  const int jj = kind == 1 ? map_cell(j, g.ny, g.bcy) : map_node(j, g.ny, g.bcy);
  load8(of_kind(kind, u.v, u.x, u.y), of_kind(kind, g.sv, g.sx, g.sy),
        (long)jj * of_kind(kind, g.nxp, g.nxp, g.nx) + ii, U);
}

// The tile's nl points to be limited, their high-order states in `stash`: the
// first-order LLF state (Section 3.3), the scaling limiter, SSP combination,
// store; and the LLF states of the first n - nl points to be looked at.  V and the FVS direction of X and Y take the own type's neighbours at
// +-h, the central direction of X and Y the two vertices; the point's own flux
// cancels between the two pairs of a direction,
//   U^LLF = U - sum (dt/Delta) [(F+ - F-) - al+ (U+ - U) + al- (U - U-)] / 2 - dt div B Psi.
// Four lanes share a point, a neighbour each, and every wave of the tile
// takes its part of the list: a shock's points lie in few tiles, whose time
// this is.  One lane per point, where the point was found, took 20 us of a
// 37 us launch (200 x 137 grid with 300 such points).
__device__ __forceinline__ void limit_listed(double (*s)[PB][PB], const Geo& g, CState u, CState un, MState out,
                                             MState stash, double dt, double ca, double cb, Counters* cn, int bx,
                                             int by, int tid, int nl, int n, bool speeds, double& wm) {
  const PointList& L = point_list(s);
  for (int k = tid / 4; k < n; k += PNT / 4) {
    const bool act = k < nl;
    const int e = L.q[act ? k : LOOK_END - 1 - (k - nl)], kind = e >> 8, m = tid & 3, dir = m >> 1;
    const int i = bx * (PB - 2) - 1 + (e & 15), j = by * (PB - 2) - 1 + (e >> 4 & 15);
    const bool hi = m & 1, own = kind == 0 || dir == kind - 1, lead = m == 0;
    const int d = hi ? 1 : (own ? -1 : 0);
    const long plane = of_kind(kind, g.sv, g.sx, g.sy), off = (long)j * of_kind(kind, g.nxp, g.nxp, g.nx) + i;
    double U0[NV], UH[NV], l[NV], divl;
    load_point(g, u, kind, i, j, U0);
    if (act) load8(of_kind(kind, stash.v, stash.x, stash.y), plane, off, UH);
    {
      double W[NV];
      DirEval e0, e1;
      load_point(g, u, own ? kind : 0, dir ? i : i + d, dir ? j + d : j, W);
      eval_dir<double>(U0, g, dir, e0);
      eval_dir<double>(W, g, dir, e1);
      const double al = alpha_llf(e0, e1, U0, W);
      const double lam = 0.5 * dt * (dir ? g.rdy : g.rdx), sg = hi ? lam : -lam;
#pragma unroll
      for (int c = 0; c < NV; ++c) l[c] = lam * (al * (W[c] - U0[c])) - sg * e1.F[c];
      divl = (hi ? 0.5 : -0.5) * (dir ? g.rdy * W[5] : g.rdx * W[4]);
    }
#pragma unroll
    for (int x = 1; x < 4; x <<= 1) {
#pragma unroll
      for (int c = 0; c < NV; ++c) l[c] += __shfl_xor(l[c], x);
      divl += __shfl_xor(divl, x);
    }
    double W[NV];
    psi(U0, W);
#pragma unroll
    for (int c = 0; c < NV; ++c) l[c] = U0[c] + (l[c] - dt * divl * W[c]);
    if (lead && !in_G_fast(l)) count(&cn->n_llf_not_admissible);
    if (!act) continue;
    limit_point(UH, l, g.gm1, W, cn, lead);
    if (!lead) continue;
    if (!in_G_fast(W)) count(&cn->n_not_admissible);
    if (ca != 0.0) {
      load8(of_kind(kind, un.v, un.x, un.y), plane, off, U0);
#pragma unroll
      for (int c = 0; c < NV; ++c) W[c] = ca * U0[c] + cb * W[c];
    }
    double* const o = of_kind(kind, out.v, out.x, out.y);
#pragma unroll
    for (int c = 0; c < NV; ++c) o[c * plane + off] = W[c];
    if (speeds) wm = fmax(wm, dt_speed(W, g));
  }
}

// More points to be looked at than what limit_listed does in one round, and they
// take look_listed.
constexpr int LOOK_MIN = PNT / 4;
// Their LLF states, a lane each, from the tile's states and records in LDS (the
// vertices and the records in the other direction are put back first).  Four
// lanes each with their states from memory take too long where most points of a
// tile fail the bound: Orszag-Tang vortex 512^2 at CFL 0.5, 457 us a step with
// limit_listed alone, 323 with this (without any bound, every LLF flux formed
// beside its line: 329).  What bounds it is VALU issue, 380 instructions a point.
__device__ __forceinline__ void look_listed(double (*s)[PB][PB], const Geo& g, double dt, Counters* cn, int tid,
                                            int n) {
  const PointList& L = point_list(s);
  for (int k = tid; k < n; k += PNT) {
    const int e = L.q[LOOK_END - 1 - k], kind = e >> 8, ty = e >> 4 & 15, tx = e & 15;
    const int so = 8 * kind, qo = kind == 0 ? QV_ : kind == 1 ? QX_ : QY_;
    double U0[NV], l[NV], div = 0.0, w0 = 1.0;  // l: without the point's own part w0 U0
    lds8(s, so, ty, tx, U0);
    const double r0 = s[qo][ty][tx], sq0 = s[qo + 2][ty][tx];
#pragma unroll
    for (int c = 0; c < NV; ++c) l[c] = 0.0;
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
      // c_f fields of the point and of its neighbours, which are vertices in
      // the central direction
      const bool own = kind == 0 || dir == kind - 1;
      const int f0 = kind == 0 ? QV_ + 3 + dir : kind == 1 ? (dir ? QXY_ : QX_ + 3) : (dir ? QY_ + 3 : QYX_);
      const int sn = own ? so : SV_, qn = own ? qo : QV_, fn = own ? f0 : QV_ + 3 + dir;
      const double c0 = s[f0][ty][tx], v0 = U0[1 + dir] * r0, lam = 0.5 * dt * (dir ? g.rdy : g.rdx);
#pragma unroll 1
      for (int hi = 0; hi < 2; ++hi) {
        const int d = hi ? 1 : (own ? -1 : 0), yy = dir ? ty + d : ty, xx = dir ? tx : tx + d;
        double F[NV], W[NV];
        lean_pt(s, sn, qn, yy, xx, dir, F, W);
        const double cw = s[fn][yy][xx], vw = W[1 + dir] * s[qn][yy][xx], t = sq0 + s[qn + 2][yy][xx];
        // alpha_llf: |Roe average| lies between |v0| and |vw|; the jump by one
        // reciprocal root of (t |jump B|)^2
        const double j2 = jump2(U0, W), x = fmax(j2 * t * t, 1e-290);
        double r = __builtin_amdgcn_rsq(x);
        r = r * fma(-0.5 * x * r, r, 1.5);
        double al = fmax(fabs(v0), fabs(vw)) + fmax(c0, cw) + j2 * r;
        al *= lam;
        const double sg = hi ? -lam : lam;
#pragma unroll
        for (int c = 0; c < NV; ++c) l[c] = fma(al, W[c], fma(sg, F[c], l[c]));
        w0 -= al;
        div -= sg * W[4 + dir];
      }
    }
    double Ps[NV];
    psi(U0, Ps);
#pragma unroll
    for (int c = 0; c < NV; ++c) l[c] = fma(w0, U0[c], fma(-div, Ps[c], l[c]));
    if (!in_G_fast(l)) count(&cn->n_llf_not_admissible);
  }
}

// A thread's place in the point tile.  Derived anew in each phase from the
// thread index behind an empty asm: carried across the phases these ten
// integers cost registers that the accumulators need (at 128 registers what
// spills goes through HBM: 100 spilled values a thread doubled the kernel's
// time).
struct PtPlace {
  int grp, tx, ty, i, j, txl, txr, tyd, tyu;
  bool outV, outX, outY, owner;
};
__device__ __forceinline__ PtPlace pt_place(const Geo& g, int bx, int by, int tid) {
  asm volatile("" : "+v"(tid));
  PtPlace t;
  t.grp = __builtin_amdgcn_readfirstlane(tid / (PB * PB));  // a wavefront lies in one group
  t.tx = tid % PB;
  t.ty = tid / PB % PB;
  const int i = bx * (PB - 2) - 1 + t.tx, j = by * (PB - 2) - 1 + t.ty;
  t.i = clamp_pt(i, g.nxp);
  t.j = clamp_pt(j, g.nyp);
  const bool inner = t.tx >= 1 && t.tx < PB - 1 && t.ty >= 1 && t.ty < PB - 1;
  t.outV = inner && i < g.nxp && j < g.nyp;
  t.outX = inner && i < g.nxp && j < g.ny;
  t.outY = inner && i < g.nx && j < g.nyp;
  t.owner = inner && i < g.nx && j < g.ny;
  t.txl = t.tx > 0 ? t.tx - 1 : t.tx;
  t.txr = t.tx < PB - 1 ? t.tx + 1 : t.tx;
  t.tyd = t.ty > 0 ? t.ty - 1 : t.ty;
  t.tyu = t.ty < PB - 1 ? t.ty + 1 : t.ty;
  return t;
}

// ------------------------------------------------- centre value and source
// The centre value and the nine-point source are formed by the point tile and,
// where the cell tile does not wait for it, by the cell tile; their fused
// multiply-adds are written out, so that both get the same bits.

// One component of the unlimited centre value (Section 2.1): f, minus four times
// the sum of the four face values; v, the sum of the four vertex values.
__device__ __forceinline__ double centre_raw(double a, double f, double v) {
#pragma clang fp contract(off)
  return (fma(36.0, a, f) - v) * 0.0625;
}

// Psi of a state.
__device__ __forceinline__ void psi_fma(const double U[NV], double P[NV]) {
#pragma clang fp contract(off)
  const double ri = rcp_r(U[0]);
  P[0] = 0.0;
  P[1] = U[4];
  P[2] = U[5];
  P[3] = U[6];
  P[4] = U[1] * ri;
  P[5] = U[2] * ri;
  P[6] = U[3] * ri;
  P[7] = fma(P[4], U[4], fma(P[5], U[5], P[6] * U[6]));
}

// source_nine of FP64.
template <class BF, class PF>
__device__ __forceinline__ void source_nine_fma(BF Bat, PF Psiat, double rdx, double rdy, double S[NV]) {
#pragma clang fp contract(off)
  double B1[3][3], B2[3][3];
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int a = 0; a < 3; ++a) Bat(a, b, B1[a][b], B2[a][b]);
  auto d3 = [](int at, double u0, double u1, double u2) {
#pragma clang fp contract(off)
    return at == 0 ? fma(4.0, u1, fma(-3.0, u0, -u2)) : at == 1 ? u2 - u0 : fma(-4.0, u1, fma(3.0, u2, u0));
  };
  const double wq[3] = {1.0 / 6.0, 2.0 / 3.0, 1.0 / 6.0};
  double f[9];
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int a = 0; a < 3; ++a)
      f[3 * b + a] = (wq[a] * wq[b]) *
                     fma(d3(a, B1[0][b], B1[1][b], B1[2][b]), rdx, d3(b, B2[a][0], B2[a][1], B2[a][2]) * rdy);
#pragma unroll
  for (int c = 0; c < NV; ++c) S[c] = 0.0;
  // Three samples per trip: their loads are in flight together, while the
  // states of all nine are never live together.
#pragma unroll 3
  for (int q = 0; q < 9; ++q) {
    const int a = q % 3, b = q / 3;
    double fq = f[0];
#pragma unroll
    for (int r = 1; r < 9; ++r) fq = q == r ? f[r] : fq;
    double P[NV];
    Psiat(a, b, P);
#pragma unroll
    for (int c = 1; c < NV; ++c) S[c] = fma(fq, P[c], S[c]);
  }
}

// The nine-point source of cell (i,j) from the stage input.
__device__ void source_of_cell(const Geo& g, CState u, int i, int j, double S[NV]) {
  double C[NV];
  {
    double A[NV], Uc[NV], f[NV], w[NV], q[NV];
    ldA(g, u.a, i, j, A);
    ldX(g, u.x, i, j, f);
    ldX(g, u.x, i + 1, j, w);
    ldY(g, u.y, i, j, Uc);
    ldY(g, u.y, i, j + 1, q);
#pragma unroll
    for (int c = 0; c < NV; ++c) f[c] = -4.0 * ((f[c] + w[c]) + (Uc[c] + q[c]));
    ldV(g, u.v, i, j, Uc);
    ldV(g, u.v, i + 1, j, w);
#pragma unroll
    for (int c = 0; c < NV; ++c) Uc[c] += w[c];
    ldV(g, u.v, i, j + 1, q);
    ldV(g, u.v, i + 1, j + 1, w);
#pragma unroll
    for (int c = 0; c < NV; ++c) Uc[c] = centre_raw(A[c], f[c], Uc[c] + (q[c] + w[c]));
    limit_centre(Uc, A, g.gm1, C, nullptr, false);
  }
  auto at = [&](int a, int b, const double*& base, long& plane, long& off) {
    const int aa = a >> 1, bb = b >> 1;
    if (b == 1) {
      base = u.x;
      plane = g.sx;
      off = (long)map_cell(j, g.ny, g.bcy) * g.nxp + map_node(i + aa, g.nx, g.bcx);
    } else if (a == 1) {
      base = u.y;
      plane = g.sy;
      off = (long)map_node(j + bb, g.ny, g.bcy) * g.nx + map_cell(i, g.nx, g.bcx);
    } else {
      base = u.v;
      plane = g.sv;
      off = (long)map_node(j + bb, g.ny, g.bcy) * g.nxp + map_node(i + aa, g.nx, g.bcx);
    }
  };
  auto Bat = [&](int a, int b, double& b1, double& b2) {
    if (a == 1 && b == 1) {
      b1 = C[4];
      b2 = C[5];
      return;
    }
    const double* base;
    long plane, off;
    at(a, b, base, plane, off);
    b1 = base[4 * plane + off];
    b2 = base[5 * plane + off];
  };
  auto Psiat = [&](int a, int b, double P[NV]) {
    if (a == 1 && b == 1) {
      psi_fma(C, P);
      return;
    }
    const double* base;
    long plane, off;
    at(a, b, base, plane, off);
    double w[NV];
    load8(base, plane, off, w);
    psi_fma(w, P);
  };
  source_nine_fma(Bat, Psiat, g.rdx, g.rdy, S);
}

// The unlimited centre value of the thread's cell from the tile's states and
// its average A.  The pins keep the eight samples from being loaded all at
// once.
__device__ __forceinline__ void tile_centre(double (*s)[PB][PB], const PtPlace& t, const double A[NV],
                                            double Uc[NV]) {
  double f[NV], w[NV], q[NV];
  lds8(s, SX_, t.ty, t.tx, f);
  lds8(s, SX_, t.ty, t.txr, w);
#pragma unroll
  for (int c = 0; c < NV; ++c) f[c] += w[c];
  pin8(f);
  lds8(s, SY_, t.ty, t.tx, Uc);
  lds8(s, SY_, t.tyu, t.tx, q);
#pragma unroll
  for (int c = 0; c < NV; ++c) f[c] = -4.0 * (f[c] + (Uc[c] + q[c]));
  pin8(f);
  lds8(s, SV_, t.ty, t.tx, Uc);
  lds8(s, SV_, t.ty, t.txr, w);
#pragma unroll
  for (int c = 0; c < NV; ++c) Uc[c] += w[c];
  pin8(Uc);
  lds8(s, SV_, t.tyu, t.tx, q);
  lds8(s, SV_, t.tyu, t.txr, w);
#pragma unroll
  for (int c = 0; c < NV; ++c) Uc[c] = centre_raw(A[c], f[c], Uc[c] + (q[c] + w[c]));
}

// The nine-point source of the thread's cell from the tile's point values and
// the limited centre value C, to src (component planes of g.sc).
__device__ __forceinline__ void tile_source(double (*s)[PB][PB], const Geo& g, const PtPlace& t, const double C[NV],
                                            double* __restrict__ src) {
  auto Bat = [&](int a, int b, double& b1, double& b2) {
    if (a == 1 && b == 1) {
      b1 = C[4];
      b2 = C[5];
      return;
    }
    const int base = b == 1 ? SX_ : (a == 1 ? SY_ : SV_);
    const int yy = b == 2 ? t.tyu : t.ty, xx = a == 2 ? t.txr : t.tx;
    b1 = s[base + 4][yy][xx];
    b2 = s[base + 5][yy][xx];
  };
  auto Psiat = [&](int a, int b, double P[NV]) {
    if (a == 1 && b == 1) {
      psi_fma(C, P);
      return;
    }
    const int base = b == 1 ? SX_ : (a == 1 ? SY_ : SV_);
    double w[NV];
    lds8(s, base, b == 2 ? t.tyu : t.ty, a == 2 ? t.txr : t.tx, w);
    psi_fma(w, P);
  };
  double S[NV];
  source_nine_fma(Bat, Psiat, g.rdx, g.rdy, S);
#pragma unroll
  for (int c = 0; c < NV; ++c) src[c * g.sc] = S[c];
}

// One tile of the point update.  tid: the thread in the 512 of the tile.
// stash: a state in which points may hold an intermediate value at their own
// place until they are written: out, or another where out is un.  src: where
// the nine-point sources go, or null.  wslot: null, or where the workgroup's
// maximum of rho_1/dx + rho_2/dy over the values it stores goes (a step's
// last stage).
__device__ __forceinline__ void points_tile(const Geo& g, CState u, CState un, MState out, MState stash,
                                            double* __restrict__ src, double dt, double ca, double cb, Counters* cn,
                                            int bx, int by, double (*s)[PB][PB], double* __restrict__ wslot, int tid) {
  double wm = 0.0;
  const bool speeds = wslot != nullptr;
  const double rdx = g.rdx, rdy = g.rdy;
  // dt / Delta of the bound, which holds for no step backward in time
  const double lxr = dt >= 0.0 ? dt * g.rdx : 1e300, lyr = dt >= 0.0 ? dt * g.rdy : 1e300;
  PointEnd end{false, false};  // the thread's vertex

  // the tile's point values into LDS, with the records of lines b and a
  {
    const PtPlace t = pt_place(g, bx, by, tid);
    double w[NV];
    if (t.grp == 0) {
      ldV(g, u.v, t.i, t.j, w);
      sts8(s, SV_, t.ty, t.tx, w);
      put_record(s, g, QV_, t.ty, t.tx, w, true, 0);
    } else {
      double w2[NV];
      ldX(g, u.x, t.i, t.j, w);
      ldY(g, u.y, t.i, t.j, w2);
      sts8(s, SX_, t.ty, t.tx, w);
      put_record(s, g, QX_, t.ty, t.tx, w, false, 1);
      sts8(s, SY_, t.ty, t.tx, w2);
      put_record(s, g, QY_, t.ty, t.tx, w2, false, 0);
    }
  }
  __syncthreads();

  // b: vertical lines through V and X.  V: FVS in y over V(l-1), X(l-1), V,
  // X(l), V(l+1).  X: central in y between V(k,j) and V(k,j+1).
  // a: horizontal lines through V and Y.  V: FVS in x over V(k-1), Y(k-1),
  // V, Y(k), V(k+1).  Y: central in x between V(i,l) and V(i+1,l).
  PointAcc P2;  // X's (group 0) or Y's (group 1)
  double Q[NV], dB, bnd;
  acc_zero(P2);
  {
    const PtPlace t = pt_place(g, bx, by, tid);
    if (t.grp == 0)
      lean_fvs<true>(s, 1, SV_, QV_, QV_ + 4, SX_, QX_, QX_ + 3, t.ty, t.tx, t.tyd, t.tx, t.tyu, t.tx, rdy, lyr, Q,
                        dB, bnd, P2);
    else
      lean_fvs<true>(s, 0, SV_, QV_, QV_ + 3, SY_, QY_, QY_ + 3, t.ty, t.tx, t.ty, t.txl, t.ty, t.txr, rdx, lxr, Q,
                        dB, bnd, P2);
  }
  pin8(Q);
  pin_acc(P2);
  __syncthreads();
  // group 0 hands its part of V over
  {
    const PtPlace t = pt_place(g, bx, by, tid);
    if (t.grp == 0) {
      PointAcc PV;
      acc_zero(PV);
      add_line(PV, Q, dB, bnd, 0.5 * rdy);
#pragma unroll
      for (int c = 0; c < NV; ++c) s[point_exchange(c)][t.ty][t.tx] = PV.h[c];
      s[point_exchange(8)][t.ty][t.tx] = PV.divh;
      s[point_exchange(9)][t.ty][t.tx] = PV.bnd;
    }
  }
  __syncthreads();
  double C[NV];
  {
    const PtPlace t = pt_place(g, bx, by, tid);
    if (t.grp == 0) {
      // centre values in FP64 (the last column/row's are never used); the
      // owner of a cell also writes the cell's nine-point source for the
      // cell kernel
      double A[NV];
      ldA(g, u.a, t.i, t.j, A);
      tile_centre(s, t, A, C);
      limit_centre(C, A, g.gm1, C, cn, t.owner);
      if (t.owner && src) tile_source(s, g, t, C, src + (long)t.j * g.nx + t.i);
    } else if (t.outV) {
      PointAcc PV;
#pragma unroll
      for (int c = 0; c < NV; ++c) PV.h[c] = s[point_exchange(c)][t.ty][t.tx];
      PV.divh = s[point_exchange(8)][t.ty][t.tx];
      PV.bnd = s[point_exchange(9)][t.ty][t.tx];
      add_line(PV, Q, dB, bnd, 0.5 * rdx);
      double w[NV];
      lds8(s, SV_, t.ty, t.tx, w);
      end = finish(g, dt, w, PV, ca, cb, un.v, out.v, stash.v, g.sv, (long)t.j * g.nxp + t.i, speeds, wm);
    }
  }
  pin_acc(P2);
  __syncthreads();
  // the centre values take the vertices' place; records of lines c and d
  if (tid == 0) point_list(s).limit = point_list(s).look = 0;
  {
    const PtPlace t = pt_place(g, bx, by, tid);
    if (t.grp == 0) {
      sts8(s, SC_, t.ty, t.tx, C);
      put_record(s, g, QC_, t.ty, t.tx, C, true, 0);
    } else {
      double w[NV];
      double b2;
      lds8(s, SX_, t.ty, t.tx, w);
      b2 = (w[4] * w[4] + w[5] * w[5] + w[6] * w[6]);
      double ri = s[QX_][t.ty][t.tx];
      s[QX_ + 3][t.ty][t.tx] = fast_speed(w, g.gamma, ri, b2, s[QX_ + 2][t.ty][t.tx], 0);
      lds8(s, SY_, t.ty, t.tx, w);
      b2 = (w[4] * w[4] + w[5] * w[5] + w[6] * w[6]);
      ri = s[QY_][t.ty][t.tx];
      s[QY_ + 3][t.ty][t.tx] = fast_speed(w, g.gamma, ri, b2, s[QY_ + 2][t.ty][t.tx], 1);
    }
  }
  __syncthreads();

  // c: horizontal lines through X and C.  X: FVS in x over X(k-1), C(k-1),
  // X, C(k), X(k+1).
  // d: vertical lines through Y and C.  Y: FVS in y over Y(l-1), C(l-1), Y,
  // C(l), Y(l+1).
  {
    const PtPlace t = pt_place(g, bx, by, tid);
    if (t.grp == 0)
      lean_fvs<false>(s, 0, SX_, QX_, QX_ + 3, SC_, QC_, QC_ + 3, t.ty, t.tx, t.ty, t.txl, t.ty, t.txr, rdx, lxr, Q,
                         dB, bnd, P2);
    else
      lean_fvs<false>(s, 1, SY_, QY_, QY_ + 3, SC_, QC_, QC_ + 4, t.ty, t.tx, t.tyd, t.tx, t.tyu, t.tx, rdy, lyr, Q,
                         dB, bnd, P2);
  }
  pin8(Q);
  pin_acc(P2);
  {
    const PtPlace t = pt_place(g, bx, by, tid);
    double w[NV];
    if (t.grp == 1) list_point(s, end, 0, t.ty, t.tx);
    end = PointEnd{false, false};
    if (t.grp == 0) {
      if (t.outX) {
        add_line(P2, Q, dB, bnd, 0.5 * rdx);
        lds8(s, SX_, t.ty, t.tx, w);
        end = finish(g, dt, w, P2, ca, cb, un.x, out.x, stash.x, g.sx, (long)t.j * g.nxp + t.i, speeds, wm);
      }
    } else if (t.outY) {
      add_line(P2, Q, dB, bnd, 0.5 * rdy);
      lds8(s, SY_, t.ty, t.tx, w);
      end = finish(g, dt, w, P2, ca, cb, un.y, out.y, stash.y, g.sy, (long)t.j * g.nx + t.i, speeds, wm);
    }
    list_point(s, end, 1 + t.grp, t.ty, t.tx);
  }
  __syncthreads();
  const int nl = point_list(s).limit, nk = point_list(s).look;
  if (__builtin_expect(nl | nk, 0))
    limit_listed(s, g, u, un, out, stash, dt, ca, cb, cn, bx, by, tid, nl, nk > LOOK_MIN ? nl : nl + nk, speeds, wm);
  if (__builtin_expect(nk > LOOK_MIN, 0)) {
    const PtPlace t = pt_place(g, bx, by, tid);
    double w[NV];
    if (t.grp == 0) {
      ldV(g, u.v, t.i, t.j, w);
      sts8(s, SV_, t.ty, t.tx, w);
      put_record(s, g, QV_, t.ty, t.tx, w, true, 0);
      s[QV_ + 2][t.ty][t.tx] = sqrt_r(w[0]);
    } else {
      lds8(s, SX_, t.ty, t.tx, w);
      double b2 = w[4] * w[4] + w[5] * w[5] + w[6] * w[6];
      s[QXY_][t.ty][t.tx] = fast_speed(w, g.gamma, s[QX_][t.ty][t.tx], b2, s[QX_ + 2][t.ty][t.tx], 1);
      s[QX_ + 2][t.ty][t.tx] = sqrt_r(w[0]);
      lds8(s, SY_, t.ty, t.tx, w);
      b2 = w[4] * w[4] + w[5] * w[5] + w[6] * w[6];
      s[QYX_][t.ty][t.tx] = fast_speed(w, g.gamma, s[QY_][t.ty][t.tx], b2, s[QY_ + 2][t.ty][t.tx], 0);
      s[QY_ + 2][t.ty][t.tx] = sqrt_r(w[0]);
    }
    __syncthreads();
    look_listed(s, g, dt, cn, tid, nk);
  }
  if (wslot) {
    __syncthreads();  // the LDS is reused as the reduction's scratch
    block_max_store(wm, tid, PNT, reinterpret_cast<double*>(&s[0][0][0]), wslot);
  }
}

}  // namespace fp64

// Threads of a point tile's workgroup and the waves per SIMD its registers
// are limited to.
template <class R> constexpr int point_threads() { return IsF32<R>::value ? PB * PB : fp64::PNT; }
template <class R> constexpr int point_waves() { return IsF32<R>::value ? 2 : 4; }

// One tile of the point update in either precision, by all threads of the
// workgroup (a flat block of point_threads<R>()).
template <class R>
__device__ __forceinline__ void points_tile(const Geo& g, CState u, CState un, MState out, MState stash,
                                            double* __restrict__ src, double dt, double ca, double cb, Counters* cn,
                                            int bx, int by, R (*s)[PB][PB], double* __restrict__ wslot) {
  const int tid = (int)threadIdx.x;
  if constexpr (IsF32<R>::value)
    points_tile_f32<R>(g, u, un, out, src, dt, ca, cb, cn, bx, by, s, wslot, tid % PB, tid / PB, true);
  else
    fp64::points_tile(g, u, un, out, stash, src, dt, ca, cb, cn, bx, by, s, wslot, tid);
}

}  // namespace afm
