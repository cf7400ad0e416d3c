// Prints how the separable element solves would be cut (csrc/sep_cut.hpp).  Built and
// run by tests/test_element_cut.py.
//
// Input, a line each: n nr elements R want padded, for a bucket of one class; output:
// rc eg nchunk threads dynamic_bytes fits mixes: fits for want columns of one element,
// mixes for a bucket of several kernels' classes.
#include <cstdio>

#include "../paper_1808_04713_amd/csrc/sep_cut.hpp"

int main() {
  int n, nr, ne, R, want, padded;
  while (std::scanf("%d %d %d %d %d %d", &n, &nr, &ne, &R, &want, &padded) == 6) {
    hdp::SepBucket b;
    b.n = n;
    b.nr = nr;
    for (int eg = 1; eg <= hdp::SEP_EG_MAX; ++eg) b.count[eg - 1] = (ne + eg - 1) / eg;
    const hdp::SepCut c = hdp::sep_cut(b, R, want, padded != 0);
    std::printf("%d %d %d %d %zu %d %d\n", c.rc, c.eg, c.nchunk, c.threads, c.lds,
                int(hdp::sep_fits(b, want, padded != 0)), int(hdp::sep_mixes(b, c)));
  }
  return 0;
}
