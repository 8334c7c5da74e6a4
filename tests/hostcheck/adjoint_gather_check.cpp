// Host build of the points' reverse in both forms: adj_point's scatters, and
// the gather that the kernels run.  Test infrastructure.
#include "adjoint_hostcheck.cpp"

extern "C" void hc_points(const hc_params* p, int k, const double* const* uk, const void* tape, double dt,
                          const double* const* lam_out, double* const* lam_n, double* const* lam_k, double* lC,
                          void* adjbuf, int gather) {
  const AGeo g = geo(p);
  Tape t;
  tape_layout(g, (char*)tape, &t);
  AdjBuf ab;
  size_t zeroed;
  const size_t nb = adjbuf_layout(g, (char*)adjbuf, &ab, &zeroed);
  std::memset(adjbuf, 0xff, nb);  // NaNs where the gather would read what was not written
  std::memset(adjbuf, 0, zeroed);
  const StateC u{uk[0], uk[1], uk[2], uk[3]};
  const StateC lo{lam_out[0], lam_out[1], lam_out[2], lam_out[3]};
  const StateM lk{lam_k[0], lam_k[1], lam_k[2], lam_k[3]};
  const StateM ln{lam_n[0], lam_n[1], lam_n[2], lam_n[3]};
  const double a = RK_A[k], b = RK_B[k];
  for (int pass = 0; pass < (gather ? 3 : 1); ++pass)
    for (int kind = 0; kind < (pass == 2 ? 4 : 3); ++kind)
      for (int l = 0; l < (kind == 0 || kind == 3 ? g.ny : g.nyp); ++l)
        for (int i = 0; i < (kind == 1 || kind == 3 ? g.nx : g.nxp); ++i) {
          if (!gather) adj_point<HostAdd>(g, u, t, ab, lo, ln, lk, kind, i, l, dt, a, b);
          else if (pass == 0) adj_point_limited<HostAdd>(g, u, t, ab, lo, lk, kind, i, l, dt, b);
          else if (pass == 1) adj_point_lines<HostAdd>(g, u, t, ab, lo, ln, lk, kind, i, l, dt, a, b);
          else adj_lines_gather<HostAdd>(g, u, t, ab, lk, kind, i, l, dt);
        }
  std::memcpy(lC, ab.lC, 8 * (size_t)g.nx * g.ny * sizeof(double));
}
