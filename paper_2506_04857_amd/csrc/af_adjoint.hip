// af_adjoint.hip -- kernels and C ABI of the recorded stage and of its
// discrete adjoint (the transposed Jacobian of one SSP-RK3 stage with the
// limiter and sensor decisions frozen as the forward took them).
//
// One thread per entity (centre, point, sensor cell, interface, limiter
// cell, update cell); launches run in dependency order on the context's
// stream.  The reverse sweep scatters with hardware FP64 atomics into the
// adjoint states and into the intermediate adjoint buffers of the
// workspace (the centre's adjoint and, on larger grids, the points' lines are
// gathered instead), so its sums are order-dependent at the rounding level (not
// bitwise reproducible run to run).
// No contraction of a*b+c into fused multiply-adds in this translation unit
// (it must precede the includes to cover the entity functions): the
// recording forward and the reverse sweep then round like the FP64 oracle,
// so exact cancellations on symmetric data stay exact and the branches taken
// at them (|0|, max ties) are the oracle's.
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>

#include <new>
#include <string>

#include "af_adjoint_stage.h"
#include "af_mhd.h"

using namespace afadj;

namespace {

constexpr int ABLK = 256;

struct DevAdd {
  __device__ static void add(double* p, double v) { unsafeAtomicAdd(p, v); }
};

__device__ __forceinline__ long gtid() { return (long)blockIdx.x * ABLK + threadIdx.x; }
inline int nblk(long n) { return (int)((n + ABLK - 1) / ABLK); }

// ---------------------------------------------------------------- record
__global__ __launch_bounds__(ABLK) void kr_centre(AGeo g, StateC u, Tape t) {
  const long q = gtid();
  if (q >= (long)g.nx * g.ny) return;
  rec_centre(g, u, t, (int)(q % g.nx), (int)(q / g.nx));
}
__global__ __launch_bounds__(ABLK) void kr_sensor(AGeo g, StateC u, Tape t) {
  const Ext e = ext_of(g);
  const long q = gtid();
  if (q >= (long)e.sw * e.sh) return;
  rec_sensor(g, u, t, (int)(q % e.sw) - 2, (int)(q / e.sw) - 2);
}
__global__ __launch_bounds__(ABLK) void kr_iface(AGeo g, StateC u, Tape t) {
  const Ext e = ext_of(g);
  const long nx = (long)e.xw * e.xh, q = gtid();
  if (q < nx)
    rec_iface(g, u, t, 0, (int)(q % e.xw) - 1, (int)(q / e.xw) - 1);
  else if (q < nx + (long)e.yw * e.yh)
    rec_iface(g, u, t, 1, (int)((q - nx) % e.yw) - 1, (int)((q - nx) / e.yw) - 1);
}
__global__ __launch_bounds__(ABLK) void kr_limiter(AGeo g, StateC u, Tape t, const double* dt) {
  const Ext e = ext_of(g);
  const long q = gtid();
  if (q >= (long)e.ew * e.eh) return;
  rec_limiter(g, u, t, (int)(q % e.ew) - 1, (int)(q / e.ew) - 1, *dt);
}
__global__ __launch_bounds__(ABLK) void kr_update(AGeo g, StateC un, StateC u, Tape t, double* out, const double* dt,
                                                  double a, double b) {
  const long q = gtid();
  if (q >= (long)g.nx * g.ny) return;
  rec_update(g, un, u, t, out, (int)(q % g.nx), (int)(q / g.nx), *dt, a, b);
}
// Points of the three sets in one launch: X, then Y, then V.
__device__ __forceinline__ bool point_of(const AGeo& g, long q, int& kind, int& k, int& l) {
  const long nX = (long)g.nxp * g.ny, nY = (long)g.nx * g.nyp, nV = (long)g.nxp * g.nyp;
  if (q < nX) {
    kind = 0;
    k = (int)(q % g.nxp);
    l = (int)(q / g.nxp);
  } else if (q < nX + nY) {
    q -= nX;
    kind = 1;
    k = (int)(q % g.nx);
    l = (int)(q / g.nx);
  } else if (q < nX + nY + nV) {
    q -= nX + nY;
    kind = 2;
    k = (int)(q % g.nxp);
    l = (int)(q / g.nxp);
  } else {
    return false;
  }
  return true;
}
__global__ __launch_bounds__(ABLK) void kr_points(AGeo g, StateC un, StateC u, Tape t, StateM out, const double* dt,
                                                  double a, double b) {
  int kind, k, l;
  if (!point_of(g, gtid(), kind, k, l)) return;
  double* o = kind == 0 ? out.x : kind == 1 ? out.y : out.v;
  rec_point(g, un, u, t, o, kind, k, l, *dt, a, b);
}

// --------------------------------------------------------------- reverse
__global__ __launch_bounds__(ABLK) void ka_zero(double* p, long n) {
  for (long q = gtid(); q < n; q += (long)gridDim.x * ABLK) p[q] = 0.0;
}
__global__ __launch_bounds__(ABLK) void ka_update(AGeo g, Tape t, AdjBuf ab, StateC lo, StateM ln, StateM lk,
                                                  const double* dt, double a, double b) {
  const long q = gtid();
  if (q >= (long)g.nx * g.ny) return;
  adj_update<DevAdd>(g, t, ab, lo, ln, lk, (int)(q % g.nx), (int)(q / g.nx), *dt, a, b);
}
__global__ __launch_bounds__(ABLK) void ka_limiter(AGeo g, StateC u, Tape t, AdjBuf ab, StateM lk, const double* dt) {
  const Ext e = ext_of(g);
  const long q = gtid();
  if (q >= (long)e.ew * e.eh) return;
  adj_limiter<DevAdd>(g, u, t, ab, lk, (int)(q % e.ew) - 1, (int)(q / e.ew) - 1, *dt);
}
__global__ __launch_bounds__(ABLK) void ka_iface(AGeo g, StateC u, Tape t, AdjBuf ab, StateM lk) {
  const Ext e = ext_of(g);
  const long nx = (long)e.xw * e.xh, q = gtid();
  if (q < nx)
    adj_iface<DevAdd>(g, u, t, ab, lk, 0, (int)(q % e.xw) - 1, (int)(q / e.xw) - 1);
  else if (q < nx + (long)e.yw * e.yh)
    adj_iface<DevAdd>(g, u, t, ab, lk, 1, (int)((q - nx) % e.yw) - 1, (int)((q - nx) / e.yw) - 1);
}
__global__ __launch_bounds__(ABLK) void ka_sensor(AGeo g, StateC u, Tape t, AdjBuf ab, StateM lk) {
  const Ext e = ext_of(g);
  const long q = gtid();
  if (q >= (long)e.sw * e.sh) return;
  adj_sensor<DevAdd>(g, u, t, ab, lk, (int)(q % e.sw) - 2, (int)(q / e.sw) - 2);
}
__global__ __launch_bounds__(ABLK) void ka_points(AGeo g, StateC u, Tape t, AdjBuf ab, StateC lo, StateM ln, StateM lk,
                                                  const double* dt, double a, double b) {
  int kind, k, l;
  if (!point_of(g, gtid(), kind, k, l)) return;
  adj_point<DevAdd>(g, u, t, ab, lo, ln, lk, kind, k, l, *dt, a, b);
}
// At most LIMITED_GRID workgroups, a wave per SIMD, which is what its registers
// admit: mostly it only reads the decisions (a workgroup per 256 points queues
// for registers beside the cells' kernels: 60 us where this takes 8).
constexpr int LIMITED_GRID = 256;
__global__ __launch_bounds__(ABLK) void ka_limited(AGeo g, StateC u, Tape t, AdjBuf ab, StateC lo, StateM lk,
                                                   const double* dt, double b) {
  int kind, k, l;
  for (long q = gtid(); point_of(g, q, kind, k, l); q += (long)gridDim.x * ABLK)
    adj_point_limited<DevAdd>(g, u, t, ab, lo, lk, kind, k, l, *dt, b);
}
__global__ __launch_bounds__(ABLK) void ka_lines(AGeo g, StateC u, Tape t, AdjBuf ab, StateC lo, StateM ln, StateM lk,
                                                 const double* dt, double a, double b) {
  int kind, k, l;
  if (!point_of(g, gtid(), kind, k, l)) return;
  adj_point_lines<DevAdd>(g, u, t, ab, lo, ln, lk, kind, k, l, *dt, a, b);
}
__global__ __launch_bounds__(ABLK) void ka_lines_gather(AGeo g, StateC u, Tape t, AdjBuf ab, StateM lk,
                                                        const double* dt) {
  int kind, k, l;
  const long cells = (long)g.nx * g.ny, q = gtid();
  if (q < cells) {
    kind = 3;
    k = (int)(q % g.nx);
    l = (int)(q / g.nx);
  } else if (!point_of(g, q - cells, kind, k, l)) {
    return;
  }
  adj_lines_gather<DevAdd>(g, u, t, ab, lk, kind, k, l, *dt);
}
__global__ __launch_bounds__(ABLK) void ka_centre(AGeo g, StateC u, Tape t, AdjBuf ab, StateM lk) {
  const long q = gtid();
  if (q >= (long)g.nx * g.ny) return;
  adj_centre<DevAdd>(g, u, t, ab, lk, (int)(q % g.nx), (int)(q / g.nx));
}
__global__ __launch_bounds__(ABLK) void ka_centre_gather(AGeo g, AdjBuf ab, StateM lk) {
  int kind, k, l;
  if (!point_of(g, gtid(), kind, k, l)) return;
  adj_centre_gather(g, ab, lk, kind, k, l);
}

thread_local std::string adj_init_err;

bool valid_params(const af_mhd_params* p) {
  if (!p) return false;
  if (p->nx < 4 || p->ny < 4 || p->nx > (1 << 16) || p->ny > (1 << 16)) return false;
  if (!(p->x1 > p->x0) || !(p->y1 > p->y0) || !(p->gamma > 1.0)) return false;
  if (!(p->cfl > 0.0 && p->cfl <= 1.0) || !(p->kappa >= 0.0)) return false;
  if ((p->bc_x != AF_BC_PERIODIC && p->bc_x != AF_BC_OUTFLOW) || (p->bc_y != AF_BC_PERIODIC && p->bc_y != AF_BC_OUTFLOW))
    return false;
  return p->flags == 0;  // FP64 only
}
AGeo make_ageo(const af_mhd_params* p) {
  AGeo g;
  g.nx = p->nx;
  g.ny = p->ny;
  g.bcx = p->bc_x;
  g.bcy = p->bc_y;
  g.nxp = p->nx + (p->bc_x == AF_BC_OUTFLOW ? 1 : 0);
  g.nyp = p->ny + (p->bc_y == AF_BC_OUTFLOW ? 1 : 0);
  g.dx = (p->x1 - p->x0) / p->nx;
  g.dy = (p->y1 - p->y0) / p->ny;
  g.gamma = p->gamma;
  g.kappa = p->kappa;
  return g;
}
bool aligned8(const void* p) { return p && ((uintptr_t)p & 7) == 0; }
bool valid_state(const af_mhd_state* s) {
  return s && aligned8(s->cell) && aligned8(s->xface) && aligned8(s->yface) && aligned8(s->vert);
}
StateC sc(const af_mhd_state* s) { return StateC{s->cell, s->xface, s->yface, s->vert}; }
StateM sm(const af_mhd_state* s) { return StateM{s->cell, s->xface, s->yface, s->vert}; }
bool same_state(const af_mhd_state* a, const af_mhd_state* b) {
  return a->cell == b->cell || a->xface == b->xface || a->yface == b->yface || a->vert == b->vert;
}

// Points (X, Y and V together) up to which their reverse is one launch that
// scatters, beyond it three that gather.  On a small grid a launch lasts as long
// as one point's chain, so that one is shorter than three; on a large one the
// atomic additions bound the scatter.  Gradients of three steps on one stream,
// scatter / gather: Alfven wave 64^2 1432 / 1514 us, 128^2 1521 / 1520, 160^2
// (77 thousand) 1907 / 1753, 256^2 3560 / 3171, 512^2 11631 / 9955; shock 128^2
// 1816 / 2085, 160^2 2263 / 2323, 200^2 2752 / 2692, 512^2 12123 / 11096.
constexpr long SCATTER_POINTS = 64000;
// Points up to which a stage's kernels all run on the context's stream.  Beyond
// it the points' run on an auxiliary stream beside the cells': that costs two or
// three waits from stream to stream a stage, some 10 us each, and gains where the
// kernels outlast them.  One stream / two: Alfven wave 64^2 1432 / 2092 us, 200^2
// (120 thousand points) 2182 / 2693, 256^2 3171 / 3211, 512^2 9955 / 9311; shock
// 200^2 2692 / 2916, 256^2 4043 / 3621, 512^2 11096 / 9958.
constexpr long ONE_STREAM_POINTS = 160000;
long points_of(const AGeo& g) { return (long)g.nxp * g.ny + (long)g.nx * g.nyp + (long)g.nxp * g.nyp; }
bool gathers(const AGeo& g) { return points_of(g) > SCATTER_POINTS; }

const double RK_A[3] = {0.0, 0.75, 1.0 / 3.0};
const double RK_B[3] = {1.0, 0.25, 2.0 / 3.0};

}  // namespace

struct af_mhd_adj {
  AGeo g;
  AdjBuf ab;
  double* ab_base;
  size_t ab_doubles;
  size_t tape_bytes;
  hipStream_t stream;
  // On large grids (ONE_STREAM_POINTS) the point update and its reverse run on
  // an auxiliary stream beside the cell update and its reverse: the two reverse
  // sides only add into the shared adjoint buffers (atomics), and the centre
  // kernels that read them wait for both.  Null elsewhere: all on `stream`.
  hipStream_t aux = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  // The points' stream.
  hipStream_t side() const { return aux ? aux : stream; }
  // What is enqueued on the points' stream from here on waits for the
  // context's, and the other way round.
  hipError_t fork_now() {
    if (!aux) return hipSuccess;
    const hipError_t e = hipEventRecord(fork, stream);
    return e == hipSuccess ? hipStreamWaitEvent(aux, fork, 0) : e;
  }
  hipError_t join_record() { return aux ? hipEventRecord(join, aux) : hipSuccess; }
  hipError_t join_wait() { return aux ? hipStreamWaitEvent(stream, join, 0) : hipSuccess; }
  std::string err;
  ~af_mhd_adj() {
    if (fork) (void)hipEventDestroy(fork);
    if (join) (void)hipEventDestroy(join);
    if (aux) (void)hipStreamDestroy(aux);
  }
};

namespace {
int fail(af_mhd_adj* c, int code, const std::string& msg) {
  c->err = msg;
  return code;
}
int check_hip(af_mhd_adj* c, const char* where) {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return AF_OK;
  return fail(c, AF_EHIP, std::string(where) + ": " + hipGetErrorString(e));
}
}  // namespace

extern "C" {

size_t af_mhd_adj_tape_bytes(const af_mhd_params* p) {
  if (!valid_params(p)) return 0;
  return tape_layout(make_ageo(p), nullptr, nullptr);
}

size_t af_mhd_adj_workspace_bytes(const af_mhd_params* p) {
  if (!valid_params(p)) return 0;
  const AGeo g = make_ageo(p);
  return adjbuf_layout(g, nullptr, nullptr, nullptr, gathers(g));
}

int af_mhd_adj_init(const af_mhd_params* p, void* workspace_dev, size_t workspace_bytes, void* hip_stream,
                    af_mhd_adj** out) {
  adj_init_err.clear();
  if (!out) return adj_init_err = "af_mhd_adj_init: null output", AF_EINVAL;
  if (!valid_params(p)) return adj_init_err = "af_mhd_adj_init: invalid parameters (FP64 only)", AF_EINVAL;
  if (!workspace_dev || ((uintptr_t)workspace_dev & 255))
    return adj_init_err = "af_mhd_adj_init: workspace null or not 256-byte aligned", AF_EINVAL;
  const AGeo g = make_ageo(p);
  const size_t need = adjbuf_layout(g, nullptr, nullptr, nullptr, gathers(g));
  if (workspace_bytes < need) return adj_init_err = "af_mhd_adj_init: workspace too small", AF_EWORKSPACE;
  af_mhd_adj* c = new (std::nothrow) af_mhd_adj();
  if (!c) return adj_init_err = "af_mhd_adj_init: out of host memory", AF_EINVAL;
  c->g = g;
  size_t zeroed = 0;
  adjbuf_layout(g, static_cast<char*>(workspace_dev), &c->ab, &zeroed, gathers(g));
  c->ab_base = static_cast<double*>(workspace_dev);
  c->ab_doubles = zeroed / sizeof(double);
  c->tape_bytes = tape_layout(g, nullptr, nullptr);
  c->stream = static_cast<hipStream_t>(hip_stream);
  const bool two = points_of(g) > ONE_STREAM_POINTS;
  hipError_t e = two ? hipStreamCreateWithFlags(&c->aux, hipStreamNonBlocking) : hipSuccess;
  if (two && e == hipSuccess) e = hipEventCreateWithFlags(&c->fork, hipEventDisableTiming);
  if (two && e == hipSuccess) e = hipEventCreateWithFlags(&c->join, hipEventDisableTiming);
  if (e != hipSuccess) {
    adj_init_err = std::string("af_mhd_adj_init: ") + hipGetErrorString(e);
    delete c;
    return AF_EHIP;
  }
  *out = c;
  return AF_OK;
}

int af_mhd_adj_record(af_mhd_adj* c, int k, const af_mhd_state* un, const af_mhd_state* uk, af_mhd_state* out,
                      const double* dt_dev, void* tape_dev, size_t tape_bytes) {
  if (!c) return AF_EINVAL;
  if (k < 0 || k > 2 || !valid_state(uk) || !valid_state(out) || (k > 0 && !valid_state(un)) || !aligned8(dt_dev) ||
      !tape_dev || ((uintptr_t)tape_dev & 255))
    return fail(c, AF_EINVAL, "af_mhd_adj_record: bad argument");
  if (tape_bytes < c->tape_bytes) return fail(c, AF_EWORKSPACE, "af_mhd_adj_record: tape too small");
  if (same_state(out, uk)) return fail(c, AF_EINVAL, "af_mhd_adj_record: out aliases uk");
  const AGeo& g = c->g;
  const Ext e = ext_of(g);
  Tape t;
  tape_layout(g, static_cast<char*>(tape_dev), &t);
  const StateC u = sc(uk), n = sc(k == 0 ? uk : un);
  const StateM o = sm(out);
  const double a = RK_A[k], b = RK_B[k];
  hipStream_t s = c->stream;
  (void)hipGetLastError();
  kr_centre<<<nblk((long)g.nx * g.ny), ABLK, 0, s>>>(g, u, t);
  // the points need only the centre values and go beside the cell chain
  // (disjoint outputs and tape fields)
  hipError_t he = c->fork_now();
  if (he != hipSuccess) return fail(c, AF_EHIP, std::string("af_mhd_adj_record: ") + hipGetErrorString(he));
  kr_points<<<nblk(points_of(g)), ABLK, 0, c->side()>>>(g, n, u, t, o, dt_dev, a, b);
  he = c->join_record();
  kr_sensor<<<nblk((long)e.sw * e.sh), ABLK, 0, s>>>(g, u, t);
  kr_iface<<<nblk((long)e.xw * e.xh + (long)e.yw * e.yh), ABLK, 0, s>>>(g, u, t);
  kr_limiter<<<nblk((long)e.ew * e.eh), ABLK, 0, s>>>(g, u, t, dt_dev);
  kr_update<<<nblk((long)g.nx * g.ny), ABLK, 0, s>>>(g, n, u, t, o.a, dt_dev, a, b);
  // the stage's output and tape are complete on s
  if (he == hipSuccess) he = c->join_wait();
  if (he != hipSuccess) return fail(c, AF_EHIP, std::string("af_mhd_adj_record: ") + hipGetErrorString(he));
  return check_hip(c, "af_mhd_adj_record");
}

int af_mhd_adj_stage(af_mhd_adj* c, int k, const af_mhd_state* uk, const void* tape_dev, size_t tape_bytes,
                     const double* dt_dev, const af_mhd_state* lam_out, af_mhd_state* lam_n, af_mhd_state* lam_k) {
  if (!c) return AF_EINVAL;
  if (k < 0 || k > 2 || !valid_state(uk) || !valid_state(lam_out) || !valid_state(lam_k) ||
      (k > 0 && !valid_state(lam_n)) || !aligned8(dt_dev) || !tape_dev || ((uintptr_t)tape_dev & 255))
    return fail(c, AF_EINVAL, "af_mhd_adj_stage: bad argument");
  if (tape_bytes < c->tape_bytes) return fail(c, AF_EWORKSPACE, "af_mhd_adj_stage: tape too small");
  if (same_state(lam_out, lam_k) || (k > 0 && same_state(lam_out, lam_n)))
    return fail(c, AF_EINVAL, "af_mhd_adj_stage: lam_out aliases an accumulator");
  const AGeo& g = c->g;
  const Ext e = ext_of(g);
  Tape t;
  tape_layout(g, static_cast<char*>(const_cast<void*>(tape_dev)), &t);
  const StateC u = sc(uk), lo = sc(lam_out);
  const StateM lk = sm(lam_k), ln = sm(k == 0 ? lam_k : lam_n);  // a_0 = 0: lam_n untouched
  const double a = RK_A[k], b = RK_B[k];
  hipStream_t s = c->stream;
  (void)hipGetLastError();
  // the points' reverse beside the cells'
  const long points = points_of(g);
  const bool gather = gathers(g);
  const hipStream_t side = c->side();
  hipError_t he = hipSuccess;
  if (gather) {  // only the last of the three needs the zeroed buffers
    he = c->fork_now();
    if (he != hipSuccess) return fail(c, AF_EHIP, std::string("af_mhd_adj_stage: ") + hipGetErrorString(he));
    ka_limited<<<nblk(points) < LIMITED_GRID ? nblk(points) : LIMITED_GRID, ABLK, 0, side>>>(g, u, t, c->ab, lo, lk,
                                                                                           dt_dev, b);
  }
  ka_zero<<<nblk((long)c->ab_doubles) < 4096 ? nblk((long)c->ab_doubles) : 4096, ABLK, 0, s>>>(c->ab_base,
                                                                                                (long)c->ab_doubles);
  if (gather) ka_lines<<<nblk(points), ABLK, 0, side>>>(g, u, t, c->ab, lo, ln, lk, dt_dev, a, b);
  he = c->fork_now();
  if (he != hipSuccess) return fail(c, AF_EHIP, std::string("af_mhd_adj_stage: ") + hipGetErrorString(he));
  if (gather)
    ka_lines_gather<<<nblk(points + (long)g.nx * g.ny), ABLK, 0, side>>>(g, u, t, c->ab, lk, dt_dev);
  else
    ka_points<<<nblk(points), ABLK, 0, side>>>(g, u, t, c->ab, lo, ln, lk, dt_dev, a, b);
  he = c->join_record();
  ka_update<<<nblk((long)g.nx * g.ny), ABLK, 0, s>>>(g, t, c->ab, lo, ln, lk, dt_dev, a, b);
  ka_limiter<<<nblk((long)e.ew * e.eh), ABLK, 0, s>>>(g, u, t, c->ab, lk, dt_dev);
  ka_iface<<<nblk((long)e.xw * e.xh + (long)e.yw * e.yh), ABLK, 0, s>>>(g, u, t, c->ab, lk);
  ka_sensor<<<nblk((long)e.sw * e.sh), ABLK, 0, s>>>(g, u, t, c->ab, lk);
  // the centre kernels read what both sides added
  if (he == hipSuccess) he = c->join_wait();
  if (he != hipSuccess) return fail(c, AF_EHIP, std::string("af_mhd_adj_stage: ") + hipGetErrorString(he));
  ka_centre<<<nblk((long)g.nx * g.ny), ABLK, 0, s>>>(g, u, t, c->ab, lk);
  ka_centre_gather<<<nblk(points), ABLK, 0, s>>>(g, c->ab, lk);
  return check_hip(c, "af_mhd_adj_stage");
}

void af_mhd_adj_destroy(af_mhd_adj* c) { delete c; }

const char* af_mhd_adj_last_error(const af_mhd_adj* c) { return c ? c->err.c_str() : adj_init_err.c_str(); }

}  // extern "C"
