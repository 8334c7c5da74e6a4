// Host build of a stage's reverse with the points' entities before the cells'
// (adjoint_hostcheck.cpp takes the cells first).  Test infrastructure.
#include "adjoint_hostcheck.cpp"

extern "C" void hc_adjoint_points_first(const hc_params* p, int k, const double* const* uk, const void* tape, double dt,
                                        const double* const* lam_out, double* const* lam_n, double* const* lam_k,
                                        void* adjbuf) {
  const AGeo g = geo(p);
  Tape t;
  tape_layout(g, (char*)tape, &t);
  AdjBuf ab;
  std::memset(adjbuf, 0, adjbuf_layout(g, (char*)adjbuf, &ab));
  const StateC u{uk[0], uk[1], uk[2], uk[3]};
  const StateC lo{lam_out[0], lam_out[1], lam_out[2], lam_out[3]};
  const StateM lk{lam_k[0], lam_k[1], lam_k[2], lam_k[3]};
  const StateM ln = k == 0 ? lk : StateM{lam_n[0], lam_n[1], lam_n[2], lam_n[3]};
  const double a = RK_A[k], b = RK_B[k];
  const int w[3] = {g.nxp, g.nx, g.nxp}, h[3] = {g.ny, g.nyp, g.nyp};
  for (int kind = 0; kind < 3; ++kind)
    for (int l = 0; l < h[kind]; ++l)
      for (int i = 0; i < w[kind]; ++i) adj_point<HostAdd>(g, u, t, ab, lo, ln, lk, kind, i, l, dt, a, b);
  for (int j = 0; j < g.ny; ++j)
    for (int i = 0; i < g.nx; ++i) adj_update<HostAdd>(g, t, ab, lo, ln, lk, i, j, dt, a, b);
  for (int j = -1; j < g.ny + 1; ++j)
    for (int i = -1; i < g.nx + 1; ++i) adj_limiter<HostAdd>(g, u, t, ab, lk, i, j, dt);
  for (int j = -1; j < g.ny + 1; ++j)
    for (int i = -1; i < g.nx + 2; ++i) adj_iface<HostAdd>(g, u, t, ab, lk, 0, i, j);
  for (int j = -1; j < g.ny + 2; ++j)
    for (int i = -1; i < g.nx + 1; ++i) adj_iface<HostAdd>(g, u, t, ab, lk, 1, i, j);
  for (int j = -2; j < g.ny + 2; ++j)
    for (int i = -2; i < g.nx + 2; ++i) adj_sensor<HostAdd>(g, u, t, ab, lk, i, j);
  for (int j = 0; j < g.ny; ++j)
    for (int i = 0; i < g.nx; ++i) adj_centre<HostAdd>(g, u, t, ab, lk, i, j);
  for (int kind = 0; kind < 3; ++kind)
    for (int l = 0; l < h[kind]; ++l)
      for (int i = 0; i < w[kind]; ++i) adj_centre_gather(g, ab, lk, kind, i, l);
}
