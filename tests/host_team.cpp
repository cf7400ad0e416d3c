// The set-up's thread team (csrc/team.hpp) where memory runs out: the k-th allocation
// fails, for every k that its construction and a parallel region come to.  Built and run
// by tests/test_host_team.py.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "../paper_1808_04713_amd/csrc/team.hpp"

static std::atomic<long> left{-1};   // allocations until one fails; < 0: none does

void* operator new(std::size_t n) {
  if (left >= 0 && left-- == 0) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main() {
  int whole = 0, refused = 0;
  for (long k = 0; k < 200; ++k) {
    std::atomic<int> sum{0};
    left = k;
    try {
      hdp::Team t;
      t.run(100, [&](int q) { sum += q; });
      left = -1;
      if (sum != 4950) return 1;
      ++whole;
    } catch (const std::bad_alloc&) {
      left = -1;
      ++refused;
    }
  }
  std::printf("%d %d\n", whole, refused);
  return 0;
}
