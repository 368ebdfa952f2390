// Reads one case from a file in the layout of host_setup_driver.cpp (state
// length zero), runs the host set-up, and prints
//   affine <0|1> spread <s> closure <c>
// s: the largest difference of two nodes' metrics in one element; c: the
// largest residual of the discrete metric identity with the face normals,
// sum_i (D-hat Ja^i)_d + sum_f l-hat (n shat)_d = 0 (what a uniform flow's time
// derivative is made of); both relative to the largest metric.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <string>
#include <vector>

#include "dgsem.h"
#include "solver_impl.h"

template <typename T>
static bool take(FILE *f, T *dst, size_t count) {
  return count == 0 || std::fread(dst, sizeof(T), count, f) == count;
}

int main(int argc, char **argv) {
  FILE *f = argc == 2 ? std::fopen(argv[1], "rb") : nullptr;
  int32_t flag = 0, ngeo = 0;
  dg_params p;
  int64_t E = 0;
  if (!f || !take(f, &flag, 1) || !take(f, &p, 1) || !take(f, &E, 1) || !take(f, &ngeo, 1)) return 3;
  const size_t ng = (size_t)ngeo + 1;
  std::vector<double> x((size_t)E * 3 * ng * ng * ng);
  std::vector<int64_t> ne((size_t)E * 6);
  std::vector<int8_t> nf((size_t)E * 6), no((size_t)E * 6);
  if (!take(f, x.data(), x.size()) || !take(f, ne.data(), ne.size()) || !take(f, nf.data(), nf.size()) ||
      !take(f, no.data(), no.size()))
    return 3;
  std::fclose(f);
  dg_mesh m{};
  m.n_elems = E;
  m.n_geo = ngeo;
  m.x_geo = x.data();
  m.nbr_elem = ne.data();
  m.nbr_face = nf.data();
  m.nbr_orient = no.data();
  dg::HostSetup hs;
  std::string err;
  if (dg::setup_host(p, m, hs, err)) {
    std::printf("error %s\n", err.c_str());
    return 4;
  }
  const dg::Basis b = dg::make_basis(p.N, p.nodes);
  const int n = b.n, n2 = n * n, n3 = n2 * n;
  double big = 0.0, spread = 0.0, closure = 0.0;
  for (double v : hs.Ja) big = std::max(big, std::fabs(v));
  for (size_t r = 0; r < (size_t)9 * E; ++r) {
    const auto mm = std::minmax_element(hs.Ja.begin() + r * n3, hs.Ja.begin() + (r + 1) * n3);
    spread = std::max(spread, *mm.second - *mm.first);
  }
  for (int64_t e = 0; e < E; ++e)
    for (int d = 0; d < 3; ++d)
      for (int a = 0; a < n3; ++a) {
        const int l[3] = {a % n, (a / n) % n, a / n2}, st[3] = {1, n, n2};
        const int pq[3] = {l[1] + n * l[2], l[0] + n * l[2], l[0] + n * l[1]};
        double s = 0.0;
        for (int i = 0; i < 3; ++i) {
          const double *Ja = hs.Ja.data() + ((size_t)(3 * i + d) * E + e) * n3;
          for (int q = 0; q < n; ++q) s += b.Dhat[l[i] * n + q] * Ja[a + (q - l[i]) * st[i]];
          for (int side = 0; side < 2; ++side)
            s += (side ? b.lhp : b.lhm)[l[i]] * hs.NS[((size_t)d * E * 6 + e * 6 + 2 * i + side) * n2 + pq[i]];
        }
        closure = std::max(closure, std::fabs(s));
      }
  std::printf("affine %d spread %.3e closure %.3e\n", hs.affine ? 1 : 0, spread / big, closure / big);
  return 0;
}
