// White-box check of the cube-graph hierarchy of a box lattice with odd dimensions (host code
// only): the last level is small enough for the dense inverse and has one, V A is symmetric on
// every level, every row without an open boundary sums to zero, the node volumes add up to the
// same total on every level, and restriction weights sum to one.
// Usage: lattice_check NX NY NZ OPEN (OPEN = 1: every side open, 0: only the +x side).
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "bcm_internal.hpp"

int main(int argc, char** argv) {
  if (argc != 5) return 2;
  const int D[3] = {std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3])}, open = std::atoi(argv[4]);
  const int nc = D[0] * D[1] * D[2];
  std::vector<double> origin(3 * size_t(nc));
  std::vector<int8_t> level(nc, 0), fbc(6 * size_t(nc), BCM_BC_NONE);
  std::vector<int32_t> nbr(24 * size_t(nc), -1);
  for (int c = 0; c < nc; ++c) {
    const int q[3] = {c % D[0], (c / D[0]) % D[1], c / (D[0] * D[1])};
    const int st[3] = {1, D[0], D[0] * D[1]};
    for (int d = 0; d < 3; ++d) origin[3 * size_t(c) + d] = 0.5 * q[d];
    for (int f = 0; f < 6; ++f) {
      const int d = f >> 1, o = q[d] + ((f & 1) ? 1 : -1);
      if (o >= 0 && o < D[d]) nbr[(size_t(c) * 6 + f) * 4] = c + (o - q[d]) * st[d];
      else fbc[size_t(c) * 6 + f] = open || f == 1 ? BCM_BC_OUTFLOW : BCM_BC_SLIP;
    }
  }
  bcm_mesh_desc d{nc, 4, origin.data(), level.data(), 0.5, nbr.data(), fbc.data()};
  bcm_mesh* m = nullptr;
  if (bcm_mesh_create(&d, &m) != BCM_OK) {
    std::printf("mesh rejected: %s\n", bcm_last_error());
    return 1;
  }
  int bad = 0;
  auto check = [&](bool ok, const char* what, size_t g, int i) {
    if (!ok) ++bad, std::printf("level %zu node %d: %s\n", g, i, what);
  };
  const auto& H = m->m.coarse;
  check(H.ok && H.levels.back().n <= bcm::kBottomDirectMax, "last level too large", H.levels.size(), 0);
  check(int(H.bottom_inv.size()) == H.levels.back().n * H.levels.back().n, "no bottom inverse", 0, 0);
  double span = 1.0;  // level-0 volumes per unit of this level's relative volume
  for (size_t g = 0; g < H.levels.size(); ++g) {
    const bcm::CoarseLevel& L = H.levels[g];
    double total = 0.0;
    int closed = 0;
    for (int i = 0; i < L.n; ++i) {
      double sum = L.e_diag[i], mag = std::fabs(L.e_diag[i]);
      total += L.e_vol[i] * span;
      for (int w = 0; w < L.W; ++w) {
        const int j = L.e_col[size_t(w) * L.n + i];
        const double v = L.e_val[size_t(w) * L.n + i];
        sum += v;
        if (j == i) continue;
        double back = 0.0;
        for (int u = 0; u < L.W; ++u)
          if (L.e_col[size_t(u) * L.n + j] == i) back += L.e_val[size_t(u) * L.n + j];
        check(std::fabs(L.e_vol[i] * v - L.e_vol[j] * back) <= 1e-12 * L.e_vol[i] * v, "V A not symmetric", g, i);
      }
      check(sum <= 1e-12 * mag, "row sum positive", g, i);
      closed += std::fabs(sum) <= 1e-12 * mag;
      if (g > 0) {
        double ws = 0.0;
        for (int w = 0; w < L.CW; ++w) ws += L.e_child_w[size_t(w) * L.n + i];
        check(std::fabs(ws - 1.0) <= 1e-12, "restriction weights", g, i);
      }
    }
    check(std::fabs(total - nc) <= 1e-9 * nc, "volumes do not add up", g, 0);
    check(open || closed > 0 || L.n <= 4, "no closed row", g, 0);
    std::printf("level %zu: %d nodes, %d colours\n", g, L.n, int(L.color_off.size()) - 1);
    check(L.color_off.size() <= 3, "lattice not two-coloured", g, 0);
    span *= 8.0;
  }
  bcm_mesh_destroy(m);
  std::printf(bad ? "FAILED (%d)\n" : "ok\n", bad);
  return bad ? 1 : 0;
}
