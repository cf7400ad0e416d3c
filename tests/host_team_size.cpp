// How many threads the set-up's team (csrc/team.hpp) has after regions of 1, 3, 2 and 100
// parts, each part run once.  Built and run by tests/test_host_team.py.
#include <cstdio>

#include "../paper_1808_04713_amd/csrc/team.hpp"

int main() {
  hdp::Team t;
  for (int n : {1, 3, 2, 100, 3, 1000}) {
    std::vector<std::atomic<int>> done(n);
    for (int again = 0; again < 50; ++again) t.run(n, [&](int q) { ++done[q]; });
    for (auto& d : done)
      if (d != 50) return 1;
    std::printf("%d ", t.size());
  }
  return 0;
}
