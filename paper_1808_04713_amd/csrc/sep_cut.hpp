// How the separable element solves (separable.hip) are cut into workgroups: host
// arithmetic alone.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace hdp {

// Per element, in class order, its first coefficient, coarse mode and dual slot.
// Classes are bucketed by kernel (sep_len); a bucket's items are runs of
// at most eg elements of one class in class order, for each eg up to SEP_EG_MAX.
constexpr int SEP_EG_MAX = 8;
struct SepElem {
  int64_t base;
  int cmo, s0;
};
struct SepBucket {
  int N = 0, n = 0, nr = 0;   // kernel (sep_len; 0: each class's own), largest n and nr
  int first[SEP_EG_MAX] = {0}, count[SEP_EG_MAX] = {0};   // items for 1, 2, .. elements per workgroup
};

// A compute unit's shared memory, less the records of a workgroup's elements that the
// kernel keeps there itself.
constexpr size_t SEP_LDS_MAX = 160 * 1024 - SEP_EG_MAX * sizeof(SepElem);

// Cut of a bucket's columns: rc columns of one element per workgroup, or all R
// columns of eg elements of a class where R alone leaves lanes idle.
struct SepCut {
  int rc, eg, nchunk, threads;
  size_t lds;
};

// dynamic shared memory: the stage and the coarse values
inline size_t sep_lds(int n, int nr, int ncol, bool padded) {
  return (size_t(n) * n * (padded ? ncol | 1 : ncol) + size_t(nr) * ncol) * 2 * sizeof(double);
}

// whether the waves of a workgroup with one column share its rows too: the kernels of
// two tiles of rows and none beyond (sep_splits in separable.hip)
inline bool sep_split_rows(int n) { return n > 20 && n <= 32; }

// whether rc columns of one element of any class of the bucket fit a workgroup
inline bool sep_fits(const SepBucket& b, int rc, bool padded) { return sep_lds(b.n, b.nr, rc, padded) <= SEP_LDS_MAX; }

// workgroups of four waves that a compute unit's registers hold of the solves' kernels
inline int sep_resident(int n) { return n <= 16 ? 4 : n <= 18 ? 3 : n <= 20 ? 2 : n <= 24 ? 3 : n <= 32 ? 2 : 1; }

// The widest classes of a bucket decide (n, nr its largest).
//
// Many workgroups: of the widths whose
// stage stays within 40 KiB (four workgroups per compute unit, so that the loads
// of some cover the products of others), the one with the least chunks x (tiles of
// 16 lines + 3) is taken: a workgroup's load, store and barriers cost about three
// tiles, and narrow chunks read pieces of cache lines (at 16 modes, where one column
// fills a tile exactly, single columns took twice the time of eight).  But
//  - at 25 to 32 modes the stage of a solve may take 80 KiB: its 150 registers leave
//    room for two workgroups anyway (29 modes, 8 columns of 256 elements: 64 us in
//    chunks of 3, 45 in chunks of 4);
//  - two workgroups per compute unit have to remain;
//  - columns in whole cache lines (8) are not cut between one and two lines, where
//    every chunk shares lines with its neighbours on other XCDs (1,024 elements of 14
//    modes, 64 columns: 180 us in chunks of 11, 156 in chunks of 8).
//
// Few workgroups, all at work at once: what counts is one's own chain, and four tiles, a
// wave each, are no longer a chain than one.  So
//  - all columns together where they make four tiles, one contiguous run to read (256
//    elements, 2 columns: 14.2 us by single columns, 11.1 together at 17 modes, 24.2
//    and 18.6 at 29);
//  - else single columns up to one per compute unit; at 21 to 32 modes, where the four
//    waves share a column's rows as well, up to two (100 elements of 29 modes, 5 columns:
//    22.9 us, in twos 26.0), and two columns up to one (16 elements: 13.6 us apart, 16.7
//    together);
//  - else the fewest chunks of at most four tiles (100 elements, 8 columns: 11.4 us in
//    single columns, 9.9 in fours at 14 modes; 27.2 and 21.2 in twos at 22).
// want > 0 fixes the width (options, autotuner) where it fits a workgroup.
inline SepCut sep_cut(const SepBucket& b, int R, int want, bool padded) {
  const int n = b.n, nr = b.nr;
  auto tiles = [&](int ncol) { return (n * ncol + 15) / 16; };
  SepCut c{1, 1, R, 0, 0};
  const int64_t singles = int64_t(b.count[0]) * R;
  const int one = std::max(1, 64 / n), chunks = (R + one - 1) / one;   // columns in four tiles
  const size_t stage = n > 24 && n <= 32 && !padded ? 80 * 1024 - SEP_EG_MAX * sizeof(SepElem) : 40 * 1024;
  const bool fixed = want > 0 && sep_fits(b, std::min(want, R), padded);
  if (fixed) {
    c.rc = std::min(want, R);
  } else if (R > one ? singles <= (sep_split_rows(n) ? 512 : 256) : singles <= 256 && sep_split_rows(n)) {
    c.rc = 1;
  } else if (int64_t(b.count[0]) * chunks < 256 * sep_resident(n)) {
    c.rc = (R + chunks - 1) / chunks;
  } else {
    int64_t best = INT64_MAX;
    for (int rc = 1; rc <= std::min(R, 64); ++rc) {
      const int nchunk = (R + rc - 1) / rc;
      if (rc > 1 && sep_lds(n, nr, rc, padded) > stage) break;
      if (rc > 1 && int64_t(b.count[0]) * nchunk < 512) continue;
      if (R % 8 == 0 && rc > 8 && rc < 16 && rc < R) continue;
      const int64_t cost = int64_t(nchunk) * (tiles(rc) + 3);
      if (cost < best) { best = cost; c.rc = rc; }
    }
  }
  if (c.rc == R && !fixed) {
    // several elements of a class share a workgroup, as long as some 512
    // workgroups (two per compute unit) remain
    double per = tiles(R);
    for (int eg = 2; eg <= SEP_EG_MAX; ++eg) {
      if (sep_lds(n, nr, R * eg, true) > 40 * 1024 || b.count[eg - 1] < 512) break;
      const double p = double(tiles(R * eg)) / eg;
      if (p < per) { per = p; c.eg = eg; }
    }
  }
  c.nchunk = (R + c.rc - 1) / c.rc;
  const int nt = tiles(c.rc * c.eg), rounds = (nt + 3) / 4;
  c.threads = 64 * ((nt + rounds - 1) / rounds);   // at most four waves, no more than the tiles keep busy
  // one column of 21 to 32 modes is two tiles of lines by two of rows, a wave each: 10.4
  // us on 256 elements of 21 modes and 12.9 at 29, where two waves of all rows took 13.2
  // and 16.7.  Past two workgroups per compute unit the two are the faster (1,024
  // elements of 29 modes: 24.0 us, with four 27.3)
  if (c.rc * c.eg == 1 && sep_split_rows(n) && int64_t(b.count[0]) * c.nchunk <= 512) c.threads = 256;
  c.lds = sep_lds(n, nr, c.rc * c.eg, padded || c.eg > 1);
  return c;
}

// Whether the classes of several kernels of up to SEP_MIX_N modes (bucket m, cut c) run in
// one launch.  A launch of few workgroups takes one workgroup's chain, 5 to 15 us, so a
// kernel after the other adds up their chains; together they cost the longest, at the
// registers of the widest kernel.  The solves of a disk's elements, separate and
// together: 64 of degree 8 to 20, one column 42.5 and 13.4 us (one padded kernel of all
// degrees 12.2), 372 of them at 16 columns 94 and 47; 1,644 of degree 4 to 16 at 7
// columns (1,644 workgroups) 59 and 37, at 12 (3,288) 73 and 71, at 16 80 and 97; 712 of
// degree 6 to 12 at 24 columns (2,136) 47.5 and 47.1, at 33 (3,560) 60 and 62.
constexpr int SEP_MIX_N = 32, SEP_MIX_BLOCKS = 2048;
inline bool sep_mixes(const SepBucket& m, const SepCut& c) {
  return int64_t(m.count[0]) * c.nchunk <= SEP_MIX_BLOCKS;
}

}  // namespace hdp
