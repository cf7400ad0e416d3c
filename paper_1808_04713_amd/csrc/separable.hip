// The separable element solves and the GLL sampling of the full-element arrays
// (gfx950, 64-wide waves).
//
// X = Ex [(Ex^T Y Ey) ./ D] Ey^T is four products over one mode index.  A
// workgroup holds n x n x (columns) coefficients in shared memory; a column is a
// right-hand side of an element, and all elements of a workgroup are of one
// class, so every column meets the same eigenbasis.  A line is the n entries
// along one index for one value of the other index and one column.  A wave takes
// 16 lines at a time: it reads them, forms their products on the FP64 matrix
// cores (16x16x4: rows of the eigenbasis by lines) and writes them back into the
// same places, so that one stage serves every product and only a barrier parts
// them.  (Near an element resonance 1 / D amplifies rounding by many digits, so the
// order of the products, x y x y, and of their sums is kept as it is.)  The eigenbasis stays in the wave's registers for a whole product.  Where
// n passes 16 or 32 by at most 4 (17 modes are the usual case) the rows
// beyond it are summed on the vector ALUs instead of filling another tile (at 21 and
// 22 modes a padded tile is the faster: the six rows took 285 registers).
//
// What bounds it: 16 n^3 flops per column with a real eigenbasis against 32 n^2
// bytes of HBM traffic; at n = 17 the two take about the same time, and a
// workgroup's chain of one load, four products and one store is hidden only by the
// other workgroups of its compute unit.  Measured, whole call, 32x32 elements of
// degree 16: 7 columns 145 -> 68 us, of which some 25 us are the call itself; 64
// columns 340 us (1.8 TB/s).  It took the place of two stages of a padded 32 x 32
// (3.5 times the products at n = 17).  Lines on the vector ALUs with the
// eigenbasis as scalar operands took 78 us: a scalar load's latency per row stays
// exposed (417 cycles a row of 34 multiply-adds).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.hpp"
#include "kernels.hpp"

namespace hdp {

namespace {

constexpr int SEP_EG = SEP_EG_MAX;   // elements per workgroup, at most
constexpr int SEP_FB = 16;           // entries per thread and batch of the staging loops

__device__ __forceinline__ double2 cfma2(double2 a, double2 b, double2 c) {
  return make_double2(c.x + a.x * b.x - a.y * b.y, c.y + a.x * b.y + a.y * b.x);
}

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double2 cmul2(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// A product's matrix in a wave's registers: M(m, k) at M[m ms + k ks], complex
// entries interleaved.  KS steps of four summation indices, MT tiles of 16 rows,
// XR further rows; entries past n are zero.
template <int KS, int MT, int XR, bool CPLX>
struct SepMat {
  double re[MT][KS], im[CPLX ? MT : 1][KS];
  double xre[XR ? XR : 1][KS], xim[CPLX && XR ? XR : 1][KS];

  __device__ __forceinline__ void load(const double* __restrict__ M, int n, int ms, int ks, int m0 = 0) {
    const int l = threadIdx.x & 63, c16 = l & 15, kq = l >> 4;
    constexpr int W = CPLX ? 2 : 1;
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      const int k = 4 * q + kq, kc = min(k, n - 1);
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const int m = m0 + 16 * t + c16;
        const double* p = M + W * (min(m, n - 1) * ms + kc * ks);
        const bool in = m < n && k < n;
        re[t][q] = in ? p[0] : 0.0;
        if (CPLX) im[t][q] = in ? p[1] : 0.0;
      }
#pragma unroll
      for (int x = 0; x < XR; ++x) {
        const int m = 16 * MT + x;
        const double* p = M + W * (min(m, n - 1) * ms + kc * ks);
        const bool in = m < n && k < n;
        xre[x][q] = in ? p[0] : 0.0;
        if (CPLX) xim[x][q] = in ? p[1] : 0.0;
      }
    }
  }
};

// out(m) = sum_k M(m, k) line(k) in place on the block's nl lines; line i has its
// entries st apart from at(i) on, read times scale(i, k) when given.
// SPLIT: 17 to 32 lines and four waves, of which wave w forms the 16 rows from
// 16 (w >> 1) on (M holds these) of the lines of tile w & 1.
template <bool SPLIT, int KS, int MT, int XR, bool CPLX, class At, class Sc>
__device__ __forceinline__ void tile_products(const SepMat<KS, MT, XR, CPLX>& M, int n, int nl, double2* A, int st,
                                              At at, Sc scale, bool scaled) {
  const int l = threadIdx.x & 63, c16 = l & 15, kq = l >> 4;
  const int w = threadIdx.x >> 6, nw = SPLIT ? 2 : blockDim.x >> 6;
  const int m0 = SPLIT ? 16 * (w >> 1) : 0;
#pragma unroll 1
  for (int t0 = SPLIT ? w & 1 : w; 16 * t0 < nl; t0 += nw) {
    const int i = min(16 * t0 + c16, nl - 1);   // lanes past the last line repeat it
    double2* line = A + at(i);
    double2 s[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) s[q] = line[min(4 * q + kq, n - 1) * st];
    if (scaled) {
#pragma unroll
      for (int q = 0; q < KS; ++q) s[q] = cmul2(s[q], scale(i, min(4 * q + kq, n - 1)));
    }
    d4 cr[MT], ci[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      cr[t] = (d4){0, 0, 0, 0};
      ci[t] = (d4){0, 0, 0, 0};
    }
#pragma unroll
    for (int q = 0; q < KS; ++q) {
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        cr[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(M.re[t][q], s[q].x, cr[t], 0, 0, 0);
        ci[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(M.re[t][q], s[q].y, ci[t], 0, 0, 0);
        if (CPLX) {
          cr[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(M.im[t][q], -s[q].y, cr[t], 0, 0, 0);
          ci[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(M.im[t][q], s[q].x, ci[t], 0, 0, 0);
        }
      }
    }
    // the rows past the tiles: each lane sums its k, then the four lanes of a line
    double2 xo[XR ? XR : 1];
#pragma unroll
    for (int x = 0; x < XR; ++x) {
      double ax = 0, ay = 0;
#pragma unroll
      for (int q = 0; q < KS; ++q) {
        ax = fma(M.xre[x][q], s[q].x, ax);
        ay = fma(M.xre[x][q], s[q].y, ay);
        if (CPLX) {
          ax = fma(-M.xim[x][q], s[q].y, ax);
          ay = fma(M.xim[x][q], s[q].x, ay);
        }
      }
      ax += __shfl_xor(ax, 16, 64);
      ay += __shfl_xor(ay, 16, 64);
      ax += __shfl_xor(ax, 32, 64);
      ay += __shfl_xor(ay, 32, 64);
      xo[x] = make_double2(ax, ay);
    }
    // lane l holds rows (l >> 4) + 4 v of line c16; every read of the tile is done,
    // another wave's too where it forms the lines' other rows
    if (SPLIT) __syncthreads();
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + 16 * t + kq + 4 * v;
        if (m < n) line[m * st] = make_double2(cr[t][v], ci[t][v]);
      }
#pragma unroll
    for (int x = 0; x < XR; ++x)
      if ((x & 3) == kq && 16 * MT + x < n) line[(16 * MT + x) * st] = xo[x];
  }
}

// The kernels whose one column a workgroup's four waves share by lines and rows: two
// tiles of each (21 to 32 modes).
constexpr bool sep_splits(int KS, int MT, int XR) { return MT == 2 && XR == 0 && KS <= 8; }

// One product on the stage A (entry (ix + n iy) ld + column): along x (the lines of
// (iy, column)) or y; M(m, k) at mat[m ms + k ks].  With dinv (along x) the entries
// are read times 1 / D (entry (k, j) of D at k + n j).
template <int KS, int MT, int XR, bool CPLX>
__device__ __forceinline__ void sep_product(const double* __restrict__ mat, int ms, int ks, bool along_x, int n,
                                            int ncol, int ld, double2* A, const double2* __restrict__ dinv = nullptr) {
  const int step = along_x ? n * ld : ld, st = along_x ? ld : n * ld;
  if constexpr (sep_splits(KS, MT, XR)) {
    if (ncol == 1 && blockDim.x == 256) {   // (n is past 16: two tiles of lines)
      SepMat<KS, 1, 0, CPLX> M;
      M.load(mat, n, ms, ks, 16 * (threadIdx.x >> 7));
      tile_products<true>(M, n, n, A, st, [&](int i) { return i * step; },
                          [&](int i, int k) { return dinv[k + n * i]; }, dinv != nullptr);
      return;
    }
  }
  SepMat<KS, MT, XR, CPLX> M;
  M.load(mat, n, ms, ks);
  const float inv = 1.0f / float(ncol);
  auto over = [&](int i) { return int((float(i) + 0.5f) * inv); };   // i / ncol (i below 2^15)
  tile_products<false>(M, n, n * ncol, A, st, [&](int i) { const int q = over(i); return q * step + (i - q * ncol); },
                       [&](int i, int k) { return dinv[k + n * over(i)]; }, dinv != nullptr);
}

template <int KS, int MT, int XR>
__device__ __forceinline__ void sep_product_any(bool real, const double* __restrict__ mat, int ms, int ks, bool along_x,
                                                int n, int ncol, int ld, double2* A,
                                                const double2* __restrict__ dinv = nullptr) {
  if (real) sep_product<KS, MT, XR, false>(mat, ms, ks, along_x, n, ncol, ld, A, dinv);
  else sep_product<KS, MT, XR, true>(mat, ms, ks, along_x, n, ncol, ld, A, dinv);
  __syncthreads();
}

// A thread's way through an element's (entry t, column r) pairs, pair threadIdx.x,
// threadIdx.x + blockDim.x, ..: the offsets in the global array (column stride R)
// and in the stage (ld), advanced without divisions or products.
struct SepWalk {
  int t, r, g, s;
  int rc, dt, dr, dg, ds, wg, ws;
  __device__ __forceinline__ SepWalk(int n2, int rc_, int R, int ld, int first) : rc(rc_) {
    t = threadIdx.x / rc;
    r = threadIdx.x - t * rc;
    g = t * R + r;
    s = t * ld + r + first;
    dt = blockDim.x / rc;
    dr = blockDim.x - dt * rc;
    dg = dt * R + dr;
    ds = dt * ld + dr;
    wg = R - rc;
    ws = ld - rc;
  }
  __device__ __forceinline__ void next() {
    t += dt;
    r += dr;
    g += dg;
    s += ds;
    if (r >= rc) {
      r -= rc;
      ++t;
      g += wg;
      s += ws;
    }
  }
};

struct SepArgs {
  const SepItem* items;   // runs of elements of one class, and the class's record
  const SepElem* elem;    // per element in class order: first coefficient, coarse mode and dual slot
  const int* r_modes;     // coarse modes, and dual-slot modes, of every class
  const int* gam_modes;
  const double2* in;
  double2* out;
  int R, nchunk, RC;      // column stride, chunks of RC columns
  const int* slot_row;    // with nu: C_1^T nu is subtracted at the dual slots
  const double* slot_coef;
  const double2* nu;
  double2* Xr;            // [coarse mode][R]
  double2* GL;
  const double2* kx;
  double2* xslot;         // [dual slot][R]
  int64_t rhs_stride;     // SEP_GLL: stride of a right-hand side's field
  int cols;               // columns in use (SEP_GLL: the fields asked for; else R)
};

// MODE SEP_SOLVE: out = A~^-1 in on every element.
// SEP_COARSE: the coarse pass of eq. block_matrix_inversion: y = in with the
//   coarse-mode rows zeroed and C_1^T nu subtracted; x_R of A~^-1 y to Xr, K_e x_R
//   to GL, and with xslot its dual-slot values.
// SEP_FULL: the full solve with the Woodbury correction folded in: the coarse
//   rows of y are -mu = -K_e Xr (Xr = x_R - T_e w), or with kx (Xr = -T_e w)
//   K_e T_e w - kx; out = A~^-1 (y - E_R mu) = A~^-1 y - G mu.
// SEP_GLL: field = V X V^T at the GLL nodes, one contiguous field per column.
template <int KS, int MT, int XR, int MODE>
__device__ __forceinline__ void sep_block(const SepArgs& g, const double* __restrict__ mats,
                                          const double2* __restrict__ Dinv, const double2* __restrict__ Kc,
                                          const double* __restrict__ gll, double2* sm, SepElem* se) {
  const SepItem I = g.items[blockIdx.x / g.nchunk];
  const int r0 = int(blockIdx.x % g.nchunk) * g.RC;
  const int R = g.R, rc = min(g.RC, g.cols - r0);
  const SepClass C = I.cls;
  const int n = C.n, n2 = n * n, nr = C.nr, ncol = I.count * rc;
  const int NTH = blockDim.x;
  // an odd column count keeps the reads that run over entries free of bank conflicts
  const bool padded = MODE == SEP_GLL || I.count > 1;
  const int ld = padded ? ncol | 1 : ncol;
  double2* A = sm;
  double2* xs = sm + n2 * ld;
  if (threadIdx.x < I.count) se[threadIdx.x] = g.elem[I.pos + threadIdx.x];
  __syncthreads();
  // stage the columns: batches of SEP_FB loads per thread (unconditional, so that a
  // batch is in flight at once)
  if (!padded && rc == R) {
    // all columns of one element: one contiguous run
    const double2* __restrict__ in = g.in + se[0].base * R;
    const int ny = n2 * rc;
    for (int i0 = threadIdx.x; i0 < ny; i0 += NTH * SEP_FB) {
      double2 v[SEP_FB];
#pragma unroll
      for (int u = 0; u < SEP_FB; ++u) v[u] = in[min(i0 + u * NTH, ny - 1)];
#pragma unroll
      for (int u = 0; u < SEP_FB; ++u)
        if (i0 + u * NTH < ny) A[i0 + u * NTH] = v[u];
    }
  } else {
    for (int el = 0; el < I.count; ++el) {
      const double2* __restrict__ in = g.in + se[el].base * R + r0;
      SepWalk w(n2, rc, R, ld, el * rc);
      while (w.t < n2) {
        double2 v[SEP_FB];
        SepWalk a = w;
#pragma unroll
        for (int u = 0; u < SEP_FB; ++u) {
          v[u] = in[a.t < n2 ? a.g : 0];
          a.next();
        }
#pragma unroll
        for (int u = 0; u < SEP_FB; ++u) {
          if (w.t < n2) A[w.s] = v[u];
          w.next();
        }
      }
    }
  }
  const int* rm = g.r_modes + C.roff;
  const int* gm = g.gam_modes + C.goff;
  if (MODE == SEP_FULL)
    for (int i = threadIdx.x; i < nr * ncol; i += NTH) {
      const int a = i / ncol, c = i - a * ncol, el = c / rc, r = c - el * rc;
      xs[i] = g.Xr[(int64_t)(se[el].cmo + a) * R + r0 + r];
    }
  __syncthreads();
  if (MODE == SEP_COARSE || MODE == SEP_FULL) {
    const double2* __restrict__ K = Kc + C.kc;
    for (int i = threadIdx.x; i < nr * ncol; i += NTH) {
      const int a = i / ncol, c = i - a * ncol;
      double2 y = make_double2(0, 0);
      if (MODE == SEP_FULL) {
        for (int b = 0; b < nr; ++b) y = cfma2(K[a + nr * b], xs[b * ncol + c], y);
        y.x = -y.x;
        y.y = -y.y;
        if (g.kx) {
          const int el = c / rc, r = c - el * rc;
          const double2 k = g.kx[(int64_t)(se[el].cmo + a) * R + r0 + r];
          y.x -= k.x;
          y.y -= k.y;
        }
      }
      A[rm[a] * ld + c] = y;
    }
    if (g.nu)   // the dual slots are distinct modes, none of them coarse
      for (int i = threadIdx.x; i < C.ns * ncol; i += NTH) {
        const int q = i / ncol, c = i - q * ncol, el = c / rc, r = c - el * rc, sl = se[el].s0 + q;
        const double2 a = g.nu[(int64_t)g.slot_row[sl] * R + r0 + r];
        const double cf = g.slot_coef[sl];
        double2& y = A[gm[q] * ld + c];
        y.x -= cf * a.x;
        y.y -= cf * a.y;
      }
    __syncthreads();
  }
  if (MODE == SEP_GLL) {
    const double* V = gll + C.voff;
    sep_product_any<KS, MT, XR>(true, V, n, 1, true, n, ncol, ld, A);
    sep_product_any<KS, MT, XR>(true, V, n, 1, false, n, ncol, ld, A);
    for (int c = 0; c < ncol; ++c) {
      const int el = c / rc, r = c - el * rc;
      double2* __restrict__ f = g.out + (int64_t)(r0 + r) * g.rhs_stride + se[el].base;
      for (int t = threadIdx.x; t < n2; t += NTH) f[t] = A[t * ld + c];
    }
    return;
  }
  // eigenbases by column: E(i, j) at i + n j
  sep_product_any<KS, MT, XR>(C.rx, mats + C.ex, n, 1, true, n, ncol, ld, A);
  sep_product_any<KS, MT, XR>(C.ry, mats + C.ey, n, 1, false, n, ncol, ld, A);
  sep_product_any<KS, MT, XR>(C.rx, mats + C.ex, 1, n, true, n, ncol, ld, A, Dinv + C.doff);
  sep_product_any<KS, MT, XR>(C.ry, mats + C.ey, 1, n, false, n, ncol, ld, A);
  if (MODE == SEP_COARSE) {
    const double2* __restrict__ K = Kc + C.kc;
    for (int i = threadIdx.x; i < nr * ncol; i += NTH) {
      const int a = i / ncol, c = i - a * ncol, el = c / rc, r = c - el * rc;
      const double2 x = A[rm[a] * ld + c];
      xs[i] = x;
      g.Xr[(int64_t)(se[el].cmo + a) * R + r0 + r] = x;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nr * ncol; i += NTH) {
      const int a = i / ncol, c = i - a * ncol, el = c / rc, r = c - el * rc;
      double2 y = make_double2(0, 0);
      for (int b = 0; b < nr; ++b) y = cfma2(K[a + nr * b], xs[b * ncol + c], y);
      g.GL[(int64_t)(se[el].cmo + a) * R + r0 + r] = y;
    }
    if (g.xslot)
      for (int i = threadIdx.x; i < C.ns * ncol; i += NTH) {
        const int q = i / ncol, c = i - q * ncol, el = c / rc, r = c - el * rc;
        g.xslot[(int64_t)(se[el].s0 + q) * R + r0 + r] = A[gm[q] * ld + c];
      }
    return;
  }
  if (!padded && rc == R) {
    double2* __restrict__ out = g.out + se[0].base * R;
    for (int i = threadIdx.x; i < n2 * rc; i += NTH) out[i] = A[i];
  } else {
    for (int el = 0; el < I.count; ++el) {
      double2* __restrict__ out = g.out + se[el].base * R + r0;
      for (SepWalk w(n2, rc, R, ld, el * rc); w.t < n2; w.next()) out[w.g] = A[w.s];
    }
  }
}

template <int KS, int MT, int XR, int MODE>
__global__ void __launch_bounds__(256) k_sep(SepArgs g, const double* __restrict__ mats, const double2* __restrict__ Dinv,
                                             const double2* __restrict__ Kc, const double* __restrict__ gll) {
  extern __shared__ double2 sm[];
  __shared__ SepElem se[SEP_EG];
  sep_block<KS, MT, XR, MODE>(g, mats, Dinv, Kc, gll, sm, se);
}

// The kernels: the largest n of each, its steps of 4 summation indices, tiles of 16 rows
// and rows beyond them.
#define HDP_SEP_TO_32(CASE) \
  CASE(4, 1, 1, 0) CASE(8, 2, 1, 0) CASE(12, 3, 1, 0) CASE(16, 4, 1, 0) CASE(18, 5, 1, 2) CASE(20, 5, 1, 4) \
  CASE(24, 6, 2, 0) CASE(28, 7, 2, 0) CASE(32, 8, 2, 0)
#define HDP_SEP_ABOVE_32(CASE) CASE(34, 9, 2, 2) CASE(36, 9, 2, 4) CASE(40, 10, 3, 0) CASE(44, 11, 3, 0)

// Elements of uneven degree, each by the kernel of its class: a launch per kernel leaves
// most of the chip idle where each has few workgroups (sep_mixes).
template <int MODE>
__global__ void __launch_bounds__(256) k_sep_mix(SepArgs g, const double* __restrict__ mats,
                                                 const double2* __restrict__ Dinv, const double2* __restrict__ Kc,
                                                 const double* __restrict__ gll) {
  extern __shared__ double2 sm[];
  __shared__ SepElem se[SEP_EG];
  switch (g.items[blockIdx.x / g.nchunk].cls.N) {
#define HDP_SEP_CASE(V, KS, MT, XR) \
  case V: sep_block<KS, MT, XR, MODE>(g, mats, Dinv, Kc, gll, sm, se); break;
    HDP_SEP_TO_32(HDP_SEP_CASE)
#undef HDP_SEP_CASE
  }
}

template <int MODE>
void launch_bucket(const SepBucket& b, SepArgs a, const SepCut& c, const Handle& h, hipStream_t s) {
  const auto& d = h.d;
  a.items = d.sep_items + b.first[c.eg - 1];
  a.nchunk = c.nchunk;
  a.RC = c.rc;
  const int64_t blocks = int64_t(b.count[c.eg - 1]) * c.nchunk;
  if (blocks > 0x7fffffff) fail(HDP_E_ARG, "element solve: too many columns");
  const dim3 grid{unsigned(blocks)}, block{unsigned(c.threads)};
  switch (b.N) {
#define HDP_SEP_CASE(V, KS, MT, XR)                                                                             \
  case V:                                                                                                       \
    hipLaunchKernelGGL((k_sep<KS, MT, XR, MODE>), grid, block, c.lds, s, a, d.sep_mat, d.Dinv, d.Kc, d.sep_gll); \
    break;
    HDP_SEP_TO_32(HDP_SEP_CASE) HDP_SEP_ABOVE_32(HDP_SEP_CASE)
#undef HDP_SEP_CASE
    default: hipLaunchKernelGGL(k_sep_mix<MODE>, grid, block, c.lds, s, a, d.sep_mat, d.Dinv, d.Kc, d.sep_gll);
  }
  HIPCHECK(hipGetLastError());
}

template <int MODE>
void launch_sep(const Handle& h, SepArgs a, int want, hipStream_t s) {
  const auto& d = h.d;
  a.elem = d.sep_elem;
  a.r_modes = d.r_modes;
  a.gam_modes = d.gam_modes;
  bool mixed = false;
  if (h.sep_mix.count[0] > 0) {
    const SepCut c = sep_cut(h.sep_mix, a.cols, want, MODE == SEP_GLL);
    mixed = sep_mixes(h.sep_mix, c);
    if (mixed) launch_bucket<MODE>(h.sep_mix, a, c, h, s);
  }
  for (const SepBucket& b : h.sep_buckets)
    if (!mixed || b.N > SEP_MIX_N) launch_bucket<MODE>(b, a, sep_cut(b, a.cols, want, MODE == SEP_GLL), h, s);
}

}  // namespace

bool sep_width_fits(const Handle& h, int rc) {
  for (const SepBucket& b : h.sep_buckets)
    if (!sep_fits(b, rc, false)) return false;
  return true;
}

// the kernel of a class of n modes per direction, by the largest n it takes
int sep_len(int n) {
  for (int N : {4, 8, 12, 16, 18, 20, 24, 28, 32, 34, 36, 40, 44})
    if (n <= N) return N;
  fail(HDP_E_UNSUPPORTED, "element solve: degree out of range");
}

void launch_sep_solve(const Handle& h, const double2* in, double2* out, int R, hipStream_t s) {
  SepArgs a{};
  a.in = in;
  a.out = out;
  a.R = a.cols = R;
  launch_sep<SEP_SOLVE>(h, a, h.fdm_rc, s);
}

void launch_sep_coarse(const Handle& h, const double2* in, int R, hipStream_t s, const double2* nu, double2* xslot,
                       int rc) {
  SepArgs a{};
  a.in = in;
  a.R = a.cols = R;
  a.nu = nu;
  a.slot_row = h.d.slot_row;
  a.slot_coef = h.d.slot_coef;
  a.Xr = h.d.cmX;
  a.GL = h.d.cmA;
  a.xslot = xslot;
  launch_sep<SEP_COARSE>(h, a, rc > 0 ? rc : h.fdm_rc, s);
}

void launch_sep_full(const Handle& h, const double2* in, double2* out, int R, hipStream_t s, const double2* nu,
                     const double2* kx, int rc) {
  SepArgs a{};
  a.in = in;
  a.out = out;
  a.R = a.cols = R;
  a.nu = nu;
  a.slot_row = h.d.slot_row;
  a.slot_coef = h.d.slot_coef;
  a.Xr = h.d.cmX;
  a.kx = kx;
  launch_sep<SEP_FULL>(h, a, rc > 0 ? rc : h.fdm_rc, s);
}

void launch_gll(const Handle& h, const double2* X, double2* field, int R, int64_t rhs_stride, int nrhs_out,
                hipStream_t s) {
  SepArgs a{};
  a.in = X;
  a.out = field;
  a.R = R;
  a.cols = nrhs_out;
  a.rhs_stride = rhs_stride;
  launch_sep<SEP_GLL>(h, a, 0, s);
}

}  // namespace hdp
