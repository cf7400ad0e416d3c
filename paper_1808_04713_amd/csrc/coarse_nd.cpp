// Nested-dissection multifrontal factor of the coarse matrix K (host side).
//
// The coarse matrix K is factored once per mesh; the paper names that factor
// the method's main cost at high frequency (the dielectric-cylinder example of
// Sec. 3.3.1 and the conclusions).  K couples only coarse unknowns that share
// an element, so with the unknowns in nested-
// dissection order (setup.cpp) block elimination creates fill only inside each
// tree node's front: node t owns the unknowns I (a separator, or a leaf set)
// and, after its subtree is eliminated, couples to the ancestor unknowns B.
// The front F = [F_II F_IB; F_BI F_BB] holds the original entries of the rows
// the node owns plus the children's Schur complements (extend-add); then
//   Dinv = F_II^-1,  L = F_BI Dinv,  S = F_BB - L F_IB  (passed to the parent).
// That is K = L D L^T with D = blockdiag(F_II), so K x = g is solved by
//   forward  (leaves first):  Y_I = front_I,  U = front_B - L Y_I
//   backward (root first):    X_I = Dinv Y_I - L^T X_B.
// Pivoting is partial inside each F_II (Gauss-Jordan); the blocks are taken in
// tree order.
#include <algorithm>
#include <cmath>
#include <mutex>
#if !defined(__HIP_DEVICE_COMPILE__) && defined(__x86_64__)
#include <immintrin.h>
#endif

#include "internal.hpp"
#include "team.hpp"

namespace hdp {

namespace {

struct Z {
  double re, im;
};

// Rows of complex numbers, two to a vector: each product's real part is re re - im im
// and its imaginary part re im + im re, rounded as the scalar form rounds them (no
// fused operations), so both forms give the same factor.
#if !defined(__HIP_DEVICE_COMPILE__) && defined(__x86_64__)
#define HDP_HOST_AVX 1
__attribute__((target("avx"))) inline __m256d cmul_avx(__m256d re, __m256d im, __m256d b) {
  return _mm256_addsub_pd(_mm256_mul_pd(re, b), _mm256_mul_pd(im, _mm256_permute_pd(b, 5)));
}

// y -= f x over n entries
__attribute__((target("avx"))) void row_minus_avx(int n, Z f, const Z* x, Z* y) {
  const __m256d re = _mm256_set1_pd(f.re), im = _mm256_set1_pd(f.im);
  int j = 0;
  for (; j + 2 <= n; j += 2) {
    double* yp = &y[j].re;
    _mm256_storeu_pd(yp, _mm256_sub_pd(_mm256_loadu_pd(yp), cmul_avx(re, im, _mm256_loadu_pd(&x[j].re))));
  }
  for (; j < n; ++j) {
    y[j].re -= f.re * x[j].re - f.im * x[j].im;
    y[j].im -= f.re * x[j].im + f.im * x[j].re;
  }
}

// C (4 x 4, ldc) += alpha A (4 x k, lda) P, P a packed k x 4 panel: the sums of a tile
// stay in registers
__attribute__((target("avx"))) void tile_avx(int k, double alpha, const Z* A, int64_t lda, const Z* P, Z* C,
                                             int64_t ldc) {
  __m256d c[4][2];
  for (int r = 0; r < 4; ++r)
    for (int h = 0; h < 2; ++h) c[r][h] = _mm256_loadu_pd(&C[r * ldc + 2 * h].re);
  for (int q = 0; q < k; ++q) {
    const __m256d b0 = _mm256_loadu_pd(&P[4 * q].re), b1 = _mm256_loadu_pd(&P[4 * q + 2].re);
    for (int r = 0; r < 4; ++r) {
      const Z a = A[r * lda + q];
      const __m256d re = _mm256_set1_pd(alpha * a.re), im = _mm256_set1_pd(alpha * a.im);
      c[r][0] = _mm256_add_pd(c[r][0], cmul_avx(re, im, b0));
      c[r][1] = _mm256_add_pd(c[r][1], cmul_avx(re, im, b1));
    }
  }
  for (int r = 0; r < 4; ++r)
    for (int h = 0; h < 2; ++h) _mm256_storeu_pd(&C[r * ldc + 2 * h].re, c[r][h]);
}
#endif

bool host_avx() {
#ifdef HDP_HOST_AVX
  static const bool yes = __builtin_cpu_supports("avx");
  return yes;
#else
  return false;
#endif
}

void row_minus(int n, Z f, const Z* x, Z* y) {
#ifdef HDP_HOST_AVX
  if (host_avx()) return row_minus_avx(n, f, x, y);
#endif
  for (int j = 0; j < n; ++j) {
    y[j].re -= f.re * x[j].re - f.im * x[j].im;
    y[j].im -= f.re * x[j].im + f.im * x[j].re;
  }
}

// C (m x n) += alpha A (m x k) B (k x n), row-major, alpha real: panels of four columns
// of B, packed, against four rows of A at a time; the sums run over k in order.
void zgemm_acc(int m, int n, int k, double alpha, const Z* A, int64_t lda, const Z* B, int64_t ldb, Z* C,
               int64_t ldc) {
  std::vector<Z> P(size_t(k) * 4);
  for (int j = 0; j < n; j += 4) {
    const int nj = std::min(4, n - j);
    if (nj == 4)
      for (int q = 0; q < k; ++q)
        for (int c = 0; c < 4; ++c) P[4 * size_t(q) + c] = B[q * ldb + j + c];
    int i = 0;
#ifdef HDP_HOST_AVX
    if (nj == 4 && host_avx())
      for (; i + 4 <= m; i += 4) tile_avx(k, alpha, A + i * lda, lda, P.data(), C + i * ldc + j, ldc);
#endif
    for (; i < m; ++i)
      for (int c = 0; c < nj; ++c) {
        Z s = C[i * ldc + j + c];
        for (int q = 0; q < k; ++q) {
          const double ar = alpha * A[i * lda + q].re, ai = alpha * A[i * lda + q].im;
          const Z b = B[q * ldb + j + c];
          s.re += ar * b.re - ai * b.im;
          s.im += ar * b.im + ai * b.re;
        }
        C[i * ldc + j + c] = s;
      }
  }
}

// In-place inverse of the n x n row-major A by Gauss-Jordan elimination with
// partial (row) pivoting; false when a pivot column is exactly zero.
bool zinverse(int n, Z* A) {
  std::vector<int> piv(n);
  for (int k = 0; k < n; ++k) {
    int p = k;
    double best = -1;
    for (int i = k; i < n; ++i) {
      const Z v = A[int64_t(i) * n + k];
      const double m = v.re * v.re + v.im * v.im;
      if (m > best) { best = m; p = i; }
    }
    if (!(best > 0)) return false;
    piv[k] = p;
    if (p != k)
      for (int j = 0; j < n; ++j) std::swap(A[int64_t(k) * n + j], A[int64_t(p) * n + j]);
    Z* rk = A + int64_t(k) * n;
    const Z d = rk[k];
    const double den = d.re * d.re + d.im * d.im;
    const Z inv{d.re / den, -d.im / den};
    rk[k] = Z{1, 0};
    for (int j = 0; j < n; ++j) {
      const Z v = rk[j];
      rk[j] = Z{v.re * inv.re - v.im * inv.im, v.re * inv.im + v.im * inv.re};
    }
    for (int i = 0; i < n; ++i) {
      if (i == k) continue;
      Z* ri = A + int64_t(i) * n;
      const Z f = ri[k];
      if (f.re == 0 && f.im == 0) continue;
      ri[k] = Z{0, 0};
      row_minus(n, f, rk, ri);
    }
  }
  for (int k = n - 1; k >= 0; --k)
    if (piv[k] != k)
      for (int i = 0; i < n; ++i) std::swap(A[int64_t(i) * n + k], A[int64_t(i) * n + piv[k]]);
  return true;
}

}  // namespace

void nd_factor(const Handle& h, const std::vector<int64_t>& kidx, const std::vector<double2>& kval, NDHost& f,
               Team* shared) {
  TeamOr threads(shared);
  Team& team = threads.team;
  const int nn = int(h.nd_off.size()) - 1;
  const int64_t nK = h.nK;
  int maxd = 0;
  for (int t = 0; t < nn; ++t) maxd = std::max(maxd, h.nd_depth[t]);
  std::vector<int> node_of(nK);
  for (int t = 0; t < nn; ++t)
    for (int i = h.nd_off[t]; i < h.nd_off[t + 1]; ++i) node_of[i] = t;
  // original entries, each in the front of the node that owns its earlier index
  std::vector<std::vector<int64_t>> bucket(nn);
  int64_t j = 0;   // keys row + nK column, sorted
  for (size_t q = 0; q < kidx.size(); ++q) {
    while (kidx[q] >= (j + 1) * nK) ++j;
    const int64_t i = kidx[q] - j * nK;
    bucket[node_of[std::min(i, j)]].push_back(int64_t(q));
  }
  auto nI_of = [&](int t) { return h.nd_off[t + 1] - h.nd_off[t]; };
  auto nB_of = [&](int t) { return int(h.nd_boff[t + 1] - h.nd_boff[t]); };
  // factor layout and update-vector rows
  f.uoff.assign(nn, 0); f.mD.assign(nn, 0); f.mL.assign(nn, 0); f.mLt.assign(nn, 0);
  int64_t tot = 0, urows = 0;
  f.flops_per_col = 0;
  for (int t = 0; t < nn; ++t) {
    const int64_t nI = nI_of(t), nB = nB_of(t);
    f.mD[t] = tot; tot += nI * nI;
    f.mL[t] = tot; tot += nB * nI;
    f.mLt[t] = tot; tot += nI * nB;
    f.uoff[t] = urows; urows += nB;
    f.flops_per_col += 8.0 * double(nI * nI + 2 * nB * nI);
  }
  f.urows = urows;
  f.fac.resize(size_t(tot));   // its pages are first written by the threads below
  Z* fac = reinterpret_cast<Z*>(f.fac.data());
  std::vector<std::vector<Z>> schur(nn);   // S of a node until its parent has used it
  std::vector<std::vector<int>> by_depth(maxd + 1);
  for (int t = 0; t < nn; ++t) by_depth[h.nd_depth[t]].push_back(t);
  std::mutex err_mu;
  std::string err;
  std::vector<std::vector<Z>> front(nn);
  auto assemble = [&](int t) {
    const int off = h.nd_off[t], nI = nI_of(t), nB = nB_of(t), nf = nI + nB;
    const int* B = h.nd_bnd.data() + h.nd_boff[t];
    auto pos = [&](int64_t g) -> int {
      if (g >= off && g < off + nI) return int(g - off);
      const int* it = std::lower_bound(B, B + nB, int(g));
      if (it == B + nB || *it != g) return -1;
      return nI + int(it - B);
    };
    std::vector<Z>& F = front[t];
    F.assign(size_t(nf) * nf, Z{0, 0});
    for (int64_t q : bucket[t]) {
      const int64_t col = kidx[q] / nK;
      const int a = pos(kidx[q] - col * nK), b = pos(col);
      if (a < 0 || b < 0) {
        std::lock_guard<std::mutex> g(err_mu);
        err = "coarse entry outside its nested-dissection front";
        return;
      }
      F[size_t(a) * nf + b].re += kval[q].x;
      F[size_t(a) * nf + b].im += kval[q].y;
    }
    for (int k = 0; k < 2; ++k) {
      const int c = h.nd_child[2 * size_t(t) + k];
      if (c < 0) continue;
      const int nc = nB_of(c);
      const int* Bc = h.nd_bnd.data() + h.nd_boff[c];
      std::vector<int> pc(nc);
      for (int a = 0; a < nc; ++a) {
        pc[a] = pos(Bc[a]);
        if (pc[a] < 0) {
          std::lock_guard<std::mutex> g(err_mu);
          err = "child boundary outside its parent's front";
          return;
        }
      }
      const std::vector<Z>& S = schur[c];
      for (int a = 0; a < nc; ++a)
        for (int b = 0; b < nc; ++b) {
          Z& x = F[size_t(pc[a]) * nf + pc[b]];
          x.re += S[size_t(a) * nc + b].re;
          x.im += S[size_t(a) * nc + b].im;
        }
      std::vector<Z>().swap(schur[c]);
    }
    Z* D = fac + f.mD[t];
    for (int i = 0; i < nI; ++i)
      for (int j = 0; j < nI; ++j) D[size_t(i) * nI + j] = F[size_t(i) * nf + j];
    if (!zinverse(nI, D)) {
      std::lock_guard<std::mutex> g(err_mu);
      err = "singular diagonal block in the nested-dissection coarse factor";
      return;
    }
    schur[t].resize(size_t(nB) * nB);
  };
  // rows b0 .. b1 - 1 of L and of S = F_BB - L F_IB
  auto eliminate = [&](int t, int b0, int b1) {
    const int nI = nI_of(t), nB = nB_of(t), nf = nI + nB, nb = b1 - b0;
    const Z* F = front[t].data();
    Z* L = fac + f.mL[t] + size_t(b0) * nI;
    std::fill(L, L + size_t(nb) * nI, Z{0, 0});
    zgemm_acc(nb, nI, nI, 1.0, F + size_t(nI + b0) * nf, nf, fac + f.mD[t], nI, L, nI);
    Z* Lt = fac + f.mLt[t] + b0;
    for (int i = 0; i < nI; ++i)
      for (int b = 0; b < nb; ++b) Lt[size_t(i) * nB + b] = L[size_t(b) * nI + i];
    Z* S = schur[t].data() + size_t(b0) * nB;
    for (int b = 0; b < nb; ++b) std::copy_n(F + size_t(nI + b0 + b) * nf + nI, nB, S + size_t(b) * nB);
    zgemm_acc(nb, nB, nI, -1.0, L, nI, F + nI, nf, S, nB);
  };
  // depth by depth: a thread per node, then a thread per 16 rows below a node's block,
  // so that the few large fronts near the root keep the team busy
  constexpr int ND_ROWS = 16;
  struct Rows { int t, b0, b1; };
  for (int dpt = maxd; dpt >= 0; --dpt) {
    const std::vector<int>& lv = by_depth[dpt];
    team.run(int(lv.size()), [&](int q) { assemble(lv[q]); });
    if (!err.empty()) fail(HDP_E_COARSE, err);
    std::vector<Rows> rows;
    for (int t : lv)
      for (int b = 0; b < nB_of(t); b += ND_ROWS) rows.push_back(Rows{t, b, std::min(b + ND_ROWS, nB_of(t))});
    team.run(int(rows.size()), [&](int q) { eliminate(rows[q].t, rows[q].b0, rows[q].b1); });
    for (int t : lv) std::vector<Z>().swap(front[t]);
  }
  // where each update row goes in the parent's front: slot k of the parent's rows
  // for child k (interior rows first, then update rows from nK on)
  std::vector<int> parent(nn, -1);
  for (int t = 0; t < nn; ++t)
    for (int k = 0; k < 2; ++k)
      if (h.nd_child[2 * size_t(t) + k] >= 0) parent[h.nd_child[2 * size_t(t) + k]] = t;
  f.push2.assign(size_t(std::max<int64_t>(1, urows)), 0);
  const int64_t srows = nK + urows;
  if (2 * srows >= (int64_t(1) << 31)) fail(HDP_E_COARSE, "nested-dissection slot index overflows");
  for (int t = 0; t < nn; ++t) {
    const int p = parent[t];
    if (nB_of(t) > 0 && p < 0) fail(HDP_E_COARSE, "nested-dissection root with a boundary");
    const int k = p >= 0 && h.nd_child[2 * size_t(p)] == t ? 0 : 1;
    const int* Bt = h.nd_bnd.data() + h.nd_boff[t];
    for (int a = 0; a < nB_of(t); ++a) {
      const int g = Bt[a];
      if (g >= h.nd_off[p] && g < h.nd_off[p + 1]) {
        f.push2[f.uoff[t] + a] = int(k * srows + g);
      } else {
        const int* Bp = h.nd_bnd.data() + h.nd_boff[p];
        const int* it = std::lower_bound(Bp, Bp + nB_of(p), g);
        if (it == Bp + nB_of(p) || *it != g) fail(HDP_E_COARSE, "child boundary outside its parent's front");
        f.push2[f.uoff[t] + a] = int(k * srows + nK + f.uoff[p] + (it - Bp));
      }
    }
  }
  nd_tasks(h, f, 1024);
}

// Row tasks of the device sweeps, depth by depth.  Several columns: tiles of
// ND_TILE outputs; a depth with few tiles splits each tile's sum so that about `target`
// workgroups run (the set-up autotuner tries several targets).
void nd_tasks(const Handle& h, NDHost& f, int target) {
  const int nn = int(h.nd_off.size()) - 1;
  int maxd = 0;
  for (int t = 0; t < nn; ++t) maxd = std::max(maxd, h.nd_depth[t]);
  std::vector<std::vector<int>> by_depth(maxd + 1);
  for (int t = 0; t < nn; ++t) by_depth[h.nd_depth[t]].push_back(t);
  auto nI_of = [&](int t) { return h.nd_off[t + 1] - h.nd_off[t]; };
  auto nB_of = [&](int t) { return int(h.nd_boff[t + 1] - h.nd_boff[t]); };
  f.levels.assign(maxd + 1, NDLevel{});
  f.tRf.clear();
  f.tRb.clear();
  f.part_tasks = 0;
  for (int dpt = 0; dpt <= maxd; ++dpt) {
    NDLevel& L = f.levels[dpt];
    for (int bwd = 0; bwd < 2; ++bwd) {
      int ntiles = 0, kmax = 0;
      for (int t : by_depth[dpt]) {
        const int nout = bwd ? nI_of(t) : nB_of(t);
        ntiles += (nout + ND_TILE - 1) / ND_TILE;
        if (nout > 0) kmax = std::max(kmax, bwd ? nI_of(t) + nB_of(t) : nI_of(t));
      }
      int S = 1;
      if (ntiles > 0) S = std::max(1, std::min((target + ntiles - 1) / ntiles, (kmax + 63) / 64));   // ranges of the longest sums keep more than 32 rows
      std::vector<int4>& T = bwd ? f.tRb : f.tRf;
      const int first = int(T.size());
      // nodes with the longest sums first: a depth whose tiles overflow one round
      // of workgroups leaves its shortest ones for the last round (each output's
      // tasks stay together, so every sum is the same)
      std::vector<int> order = by_depth[dpt];
      std::stable_sort(order.begin(), order.end(), [&](int a, int c) {
        const int ka = bwd ? nI_of(a) + nB_of(a) : nI_of(a), kc = bwd ? nI_of(c) + nB_of(c) : nI_of(c);
        return ka > kc;
      });
      for (int t : order) {
        const int nout = bwd ? nI_of(t) : nB_of(t);
        const int K = bwd ? nI_of(t) + nB_of(t) : nI_of(t);
        const int chunk = (K + S - 1) / S;
        for (int j = 0; j < nout; j += ND_TILE)
          for (int c = 0; c < S; ++c) {
            const int i0 = std::min(K, c * chunk), i1 = std::min(K, (c + 1) * chunk);
            T.push_back(make_int4(t, j, i0, i1));
          }
      }
      if (S > 1) f.part_tasks = std::max<int64_t>(f.part_tasks, int64_t(ntiles) * S);
      if (bwd) { L.bR = first; L.nbR = ntiles; L.Sb = S; }
      else { L.fR = first; L.nfR = ntiles; L.Sf = S; }
    }
  }
}

// One-column sweeps.  A depth whose sums are at least ND1_ROW long on average (a
// wave's lanes) runs a wave per output: 32 / 64 / 128 gave 6.63 / 5.60 / 5.67 ms per
// solve of the 80x80 layered scatterer and 17.8 / 16.9 / 17.9 ms of the refined disk.
// The other depths, near the leaves, run in units of ND1_P outputs,
// and consecutive ones become the stages of one launch, a workgroup per subtree rooted
// at the shallowest of them, while there are ND1_MIN_ROOTS subtrees (half the compute
// units) and none holds more than ND1_MAX_WORK factor entries (0.6 MB, some 5 us for
// a compute unit at 0.13 MB per us, about what the merged launches save).  Backward,
// where sums are longer by the boundary, only such stages do: a single depth in units
// took 4.3 us, by rows 3.7 (96x96 elements, l = 1).  They come with the small leaves of
// a requested factor: 545 us in stages, 582 by rows, for the 15 backward sweeps of a
// solve on 64x64 elements, l = 2.
//
// Backward units read D by columns; so that they use the same inverse as the rows
// (the computed D is symmetric only up to its own error, which a nearly singular
// front makes large), their D is transposed in the factor.  The sweeps at several
// columns read D by rows, so a handle for more than one column runs rows here.
void nd_units(const Handle& h, NDHost& f, bool bwd, ND1Plan& p) {
  constexpr int ND1_ROW = 64, ND1_MIN_ROOTS = 128;
  constexpr double ND1_MAX_WORK = 40000;
  const int nn = int(h.nd_off.size()) - 1;
  int maxd = 0;
  for (int t = 0; t < nn; ++t) maxd = std::max(maxd, h.nd_depth[t]);
  std::vector<std::vector<int>> by_depth(maxd + 1);
  for (int t = 0; t < nn; ++t) by_depth[h.nd_depth[t]].push_back(t);
  auto nI = [&](int t) { return h.nd_off[t + 1] - h.nd_off[t]; };
  auto nB = [&](int t) { return int(h.nd_boff[t + 1] - h.nd_boff[t]); };
  auto outs = [&](int t) { return bwd ? nI(t) : nB(t); };
  auto sums = [&](int t) { return bwd ? nI(t) + nB(t) : nI(t); };
  auto work = [&](int t) { return double(outs(t)) * sums(t); };
  auto long_sums = [&](int d) {
    if (bwd && h.max_rhs > 1) return true;   // the blocks D are not transposed (below)
    double o = 0, k = 0;
    for (int t : by_depth[d]) {
      o += outs(t);
      k += work(t);
    }
    return k >= ND1_ROW * o;
  };
  auto node_units = [&](int t) {
    if (bwd) {
      double2* D = f.fac.data() + f.mD[t];
      for (int i = 0; i < nI(t); ++i)
        for (int j = 0; j < i; ++j) std::swap(D[size_t(i) * nI(t) + j], D[size_t(j) * nI(t) + i]);
    }
    for (int o0 = 0; o0 < outs(t); o0 += ND1_P)
      p.units.push_back(ND1Unit{bwd ? f.mD[t] : f.mLt[t], h.nd_boff[t], outs(t), o0, sums(t), nI(t), h.nd_off[t],
                                int(f.uoff[t])});
  };
  p = ND1Plan{};
  // the batches of depths [top, bottom], deepest first; sub[t]: work of t's subtree
  // within its batch
  std::vector<std::pair<int, int>> batches;
  std::vector<double> sub(nn, 0.0);
  for (int bottom = maxd; bottom >= 0;) {
    for (int t : by_depth[bottom]) sub[t] = work(t);
    int top = bottom;
    while (!long_sums(bottom) && top > 0 && !long_sums(top - 1) && int(by_depth[top - 1].size()) >= ND1_MIN_ROOTS) {
      double most = 0;
      for (int t : by_depth[top - 1]) {
        sub[t] = work(t);
        for (int k = 0; k < 2; ++k) {
          const int c = h.nd_child[2 * size_t(t) + k];
          if (c >= 0) sub[t] += sub[c];
        }
        most = std::max(most, sub[t]);
      }
      if (most > ND1_MAX_WORK) break;
      --top;
    }
    batches.push_back({top, bottom});
    bottom = top - 1;
  }
  if (bwd) std::reverse(batches.begin(), batches.end());
  for (auto& b : batches) {
    ND1Launch L;
    L.stages = b.second - b.first + 1;
    if (L.stages == 1 && (bwd || long_sums(b.first))) {
      L.rows = true;
      L.first = int64_t(p.rows.size());
      for (int t : by_depth[b.first])
        for (int j = 0; j < outs(t); ++j) {
          if (bwd)
            p.rows.push_back(ND1Row{f.mD[t] + int64_t(nI(t)) * j, f.mLt[t] + int64_t(nB(t)) * j, h.nd_boff[t], nI(t),
                                    nB(t), h.nd_off[t], h.nd_off[t] + j});
          else
            p.rows.push_back(ND1Row{f.mL[t] + int64_t(nI(t)) * j, 0, 0, nI(t), 0, h.nd_off[t], int(f.uoff[t]) + j});
        }
      L.groups = int(int64_t(p.rows.size()) - L.first);
    } else if (L.stages == 1) {
      L.first = int64_t(p.gptr.size());
      const int u0 = int(p.units.size());
      for (int t : by_depth[b.first]) node_units(t);
      const int n = int(p.units.size()) - u0;
      for (int u = 0; u < n; u += L.waves) {
        p.gptr.push_back(u0 + u);
        p.gptr.push_back(u0 + std::min(n, u + L.waves));
        ++L.groups;
      }
    } else {
      L.first = int64_t(p.gptr.size());
      L.waves = 8;
      for (int root : by_depth[b.first]) {
        std::vector<std::vector<int>> at(L.stages);
        at[0].push_back(root);
        for (int s = 0; s + 1 < L.stages; ++s)
          for (int t : at[s])
            for (int k = 0; k < 2; ++k)
              if (h.nd_child[2 * size_t(t) + k] >= 0) at[s + 1].push_back(h.nd_child[2 * size_t(t) + k]);
        for (int s = 0; s < L.stages; ++s) {
          p.gptr.push_back(int(p.units.size()));
          for (int t : at[bwd ? s : L.stages - 1 - s]) node_units(t);
        }
        p.gptr.push_back(int(p.units.size()));
        ++L.groups;
      }
    }
    p.launches.push_back(L);
  }
}

}  // namespace hdp
