// Prints the launches of the one-column nested-dissection sweeps of an n x n mesh
// (nd_units in csrc/coarse_nd.cpp): per sweep, r for a wave per output, u and the number
// of depths for units.  Built and run by tests/test_nd_plan.py.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_1808_04713_amd/csrc/internal.hpp"

namespace hdp {
[[noreturn]] void fail(hdp_status s, const std::string& msg) { throw Error{s, msg}; }
void check_hip(hipError_t, const char*) {}
}  // namespace hdp

int main(int, char** v) {
  const int n = std::atoi(v[1]), l = std::atoi(v[2]);
  std::vector<int> leaf, deg(size_t(n) * n, 4);
  std::vector<double> eps(size_t(n) * n, 1.0);
  for (int y = 0; y < n; ++y)
    for (int x = 0; x < n; ++x) leaf.insert(leaf.end(), {0, x, y});
  hdp_mesh mesh{0, 1, 0, 1, n, n, n * n, leaf.data(), deg.data()};
  hdp_problem prob{};
  prob.k = 1.1 * n;
  prob.eps_r = eps.data();
  prob.l = l;
  hdp::Handle h;
  if (std::atoi(v[3])) h.coarse_mode = 2;   // a requested factor
  hdp::build_host(h, &mesh, &prob);
  if (h.coarse_mode != 2) return 3;
  std::vector<int64_t> kidx;
  std::vector<double2> kval;
  hdp::coarse_coo(h, kidx, kval);
  hdp::NDHost f;
  hdp::nd_factor(h, kidx, kval, f);
  for (int bwd = 0; bwd < 2; ++bwd) {
    hdp::ND1Plan p;
    hdp::nd_units(h, f, bwd != 0, p);
    for (auto& L : p.launches) {
      if (L.rows) std::printf("r ");
      else std::printf("u%d ", L.stages);
    }
    std::printf("\n");
  }
  return 0;
}
