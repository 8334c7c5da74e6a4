// Host build of step (2) of the flux limiter as the FP64 cell tile runs it
// without its sufficient test (limiter_box_lanes).  Test infrastructure.
#include <thread>

#include "af_device.h"

// in [n][42] = (A^{Lim,1}, H_L, H_R, H_D, H_U, eps_rho, eps_p), out [n][4];
// counts: Counters.
extern "C" void hc_box_lanes(long n, double gamma, const double* in, double* out, unsigned long long* counts) {
  using namespace afm;
  auto* cn = reinterpret_cast<Counters*>(counts);
  auto lane = [&](int k) {
    lane_id = k;
    for (long t = 0; t < n; ++t) {
      const double* q = in + 42 * t;
      double Lam[4];
      auto H = [&](int I, int c) -> double { return q[NV + NV * I + c]; };
      limiter_box_lanes(q, H, gamma - 1.0, q[5 * NV], q[5 * NV + 1], Lam, cn, true, k);
      if (k == 0)
        for (int I = 0; I < 4; ++I) out[4 * t + I] = Lam[I];
    }
  };
  std::thread th[LANES];
  for (int k = 0; k < LANES; ++k) th[k] = std::thread(lane, k);
  for (auto& t : th) t.join();
}
