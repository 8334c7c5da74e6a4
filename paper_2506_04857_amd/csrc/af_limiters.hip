// af_limiters.hip -- the stage's positivity limiters applied to given inputs
// (af_mhd_limiters_apply), by the very device functions the stage kernels call
// -- the point scaling limiter (Section 3.3), the centre-value limiter (remark
// rmk:cell_center), steps (1) and (2) of the parametrized flux limiter (Section
// 3.2), each with the round-off fallback of the closing remark of Section 4.
// One thread per item; step (2) sixteen, as in the FP64 stage (box_clear,
// limiter_box_lanes), whose first one also runs the FP32-bulk stage's form
// (limiter_box).  A verification aid: on identical inputs they can be compared
// bit for bit with a reference.
#include <hip/hip_runtime.h>

#include "af_device.h"
#include "af_mhd.h"

using namespace afm;

static_assert(sizeof(af_mhd_counters_t) == sizeof(Counters), "counter layouts agree");

namespace {

constexpr int LBLK = 64;

__global__ __launch_bounds__(LBLK) void k_limiters(int kind, long n, double gm1, const double* __restrict__ in,
                                                   double* __restrict__ out, Counters* cn) {
  const long t = (long)blockIdx.x * LBLK + threadIdx.x;
  if (t >= n) return;
  if (kind == AF_LIM_POINT || kind == AF_LIM_CENTRE) {
    const double* q = in + 16 * t;
    double a[NV], b[NV], w[NV];
    for (int c = 0; c < NV; ++c) {
      a[c] = q[c];
      b[c] = q[NV + c];
    }
    if (kind == AF_LIM_POINT)
      limit_point(a, b, gm1, w, cn, true);
    else
      limit_centre(a, b, gm1, w, cn, true);
    for (int c = 0; c < NV; ++c) out[8 * t + c] = w[c];
  } else {
    const double* q = in + 25 * t;
    double G[NV], S[NV], Sl[NV], A1[NV], er, ep;
    for (int c = 0; c < NV; ++c) {
      G[c] = q[c];
      S[c] = q[NV + c];
      Sl[c] = q[2 * NV + c];
    }
    const double th = source_step(G, S, Sl, q[3 * NV], gm1, A1, er, ep, cn, true);
    for (int c = 0; c < NV; ++c) out[9 * t + c] = A1[c];
    out[9 * t + NV] = th;
  }
}

// Step (2): sixteen threads an item.  Where the two stages' forms differ in a
// bit the item's output is NaN.
constexpr int BOX_LANES = 16;
template <bool SHORTCUT>
__global__ __launch_bounds__(LBLK) void k_limiter_box(long n, double gm1, const double* __restrict__ in,
                                                      double* __restrict__ out, Counters* cn) {
  const long t = ((long)blockIdx.x * LBLK + threadIdx.x) / BOX_LANES;
  if (t >= n) return;
  const double* q = in + 42 * t;
  double A1[NV], Lam[4];
  for (int c = 0; c < NV; ++c) A1[c] = q[c];
  const double* Hq = q + NV;
  const double er = q[5 * NV], ep = q[5 * NV + 1];
  auto H = [&](int I, int c) -> double { return Hq[NV * I + c]; };
  if (!SHORTCUT || !box_clear(A1, H, gm1, er, ep, Lam))
    limiter_box_lanes(A1, H, gm1, er, ep, Lam, cn, true, (int)threadIdx.x);
  if (threadIdx.x % BOX_LANES) return;
  double one[4];
  limiter_box<decltype(H), SHORTCUT>(A1, H, gm1, er, ep, one, cn, false);
  bool same = true;
  for (int I = 0; I < 4; ++I) same = same && __double_as_longlong(Lam[I]) == __double_as_longlong(one[I]);
  for (int I = 0; I < 4; ++I) out[4 * t + I] = same ? Lam[I] : __longlong_as_double(0x7ff8000000000000ll);
}

}  // namespace

extern "C" int af_mhd_limiters_apply(int kind, int64_t n, double gamma, const double* in_dev, double* out_dev,
                                     uint32_t flags, af_mhd_counters_t* counts_dev, void* hip_stream) {
  if (kind < AF_LIM_POINT || kind > AF_LIM_BOX || n < 0 || !(gamma > 1.0) || (flags & ~AF_LIM_NO_SHORTCUT))
    return AF_EINVAL;
  if (n == 0) return AF_OK;
  if (!in_dev || !out_dev || !counts_dev || ((uintptr_t)in_dev & 7) || ((uintptr_t)out_dev & 7) ||
      ((uintptr_t)counts_dev & 7))
    return AF_EINVAL;
  const int per = kind == AF_LIM_BOX ? LBLK / BOX_LANES : LBLK;
  const long blocks = (long)((n + per - 1) / per);
  if (blocks > 0x7fffffffL) return AF_EINVAL;
  (void)hipGetLastError();
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  Counters* cn = reinterpret_cast<Counters*>(counts_dev);
  if (kind != AF_LIM_BOX)
    k_limiters<<<(unsigned)blocks, LBLK, 0, s>>>(kind, (long)n, gamma - 1.0, in_dev, out_dev, cn);
  else if (flags & AF_LIM_NO_SHORTCUT)
    k_limiter_box<false><<<(unsigned)blocks, LBLK, 0, s>>>((long)n, gamma - 1.0, in_dev, out_dev, cn);
  else
    k_limiter_box<true><<<(unsigned)blocks, LBLK, 0, s>>>((long)n, gamma - 1.0, in_dev, out_dev, cn);
  return hipGetLastError() == hipSuccess ? AF_OK : AF_EHIP;
}
