// Device kernels of the interface-problem solver for gfx950 (64-wide waves).
//
// Layouts: every vector family stores the right-hand-side index fastest
// (stride R).  Dual-slot arrays hold, per element, the type-1 edge modes that
// the jump operator C_1 touches; full-element arrays hold all n_e^2 vertex-
// basis coefficients of every element.
#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "kernels.hpp"

namespace hdp {

namespace {

constexpr int NT = 256;      // threads per block
constexpr int RC = 8;        // RHS columns per block in the slot kernels
constexpr int MMAX = 160;    // max dual slots per element (4 sides x 40 modes)
constexpr int NRMAX = 160;   // max coarse modes per element

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 c) {
  return make_double2(c.x + a.x * b.x - a.y * b.y, c.y + a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cfma(float2 a, float2 b, float2 c) {
  return make_float2(c.x + a.x * b.x - a.y * b.y, c.y + a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cconjmul(double2 a, double2 b) {  // conj(a) * b
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}

template <class T2> struct Scal;
template <> struct Scal<double2> { using T = double; };
template <> struct Scal<float2> { using T = float; };

template <class T2> __device__ __forceinline__ T2 mk(double x, double y);
template <> __device__ __forceinline__ double2 mk<double2>(double x, double y) { return make_double2(x, y); }
template <> __device__ __forceinline__ float2 mk<float2>(double x, double y) { return make_float2(float(x), float(y)); }

// Reduce a per-thread value over the threads of a block that share an RHS
// column (lanes with equal lane % R inside a wave, then the four waves).
__device__ __forceinline__ double2 block_sum_by_rhs(double2 v, int R, double2* red) {
  for (int off = 32; off >= R && off > 0; off >>= 1) {
    v.x += __shfl_xor(v.x, off, 64);
    v.y += __shfl_xor(v.y, off, 64);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane < R) red[wv * 64 + lane] = v;
  __syncthreads();
  double2 s = make_double2(0, 0);
  if (threadIdx.x < R)
    for (int q = 0; q < NT / 64; ++q) {
      s.x += red[q * 64 + threadIdx.x].x;
      s.y += red[q * 64 + threadIdx.x].y;
    }
  __syncthreads();
  return s;   // valid in threads 0..R-1
}

// ---------------------------------------------------------------------------
// Slot kernels: one block per element (class-grouped order), RC RHS per block.
template <class T2, int MODE>
__global__ void __launch_bounds__(NT) k_slot_apply(const SlotBlock* __restrict__ blk, const SlotIn* __restrict__ sin,
                                                   const T2* __restrict__ op1, const T2* __restrict__ se,
                                                   const T2* __restrict__ v, T2* __restrict__ X, T2* __restrict__ GL,
                                                   int R) {
  using S = typename Scal<T2>::T;
  __shared__ T2 y[MMAX * RC];
  const SlotBlock B = blk[blockIdx.x];
  const int m = B.m, nr = B.nr, so = B.so;
  const int r0 = blockIdx.y * RC;
  const int rc = min(RC, R - r0);
  for (int idx = threadIdx.x; idx < m * rc; idx += NT) {
    const int s = idx / rc, r = idx - s * rc;
    // MODE 0/1: v holds dual rows; MODE 2: dual slots, the row value being the
    // jump C_1 z of its two slots
    const SlotIn g = sin[so + s];
    S ax = 0, ay = 0;
    if (g.s0 >= 0) {
      const T2 z = v[(int64_t)g.s0 * R + r0 + r];
      ax += S(g.a0) * z.x;
      ay += S(g.a0) * z.y;
    }
    if (MODE == 2 && g.s1 >= 0) {
      const T2 z = v[(int64_t)g.s1 * R + r0 + r];
      ax += S(g.a1) * z.x;
      ay += S(g.a1) * z.y;
    }
    y[s * RC + r] = mk<T2>(ax, ay);
  }
  __syncthreads();
  if (MODE == 0) {
    const int nrow = m + nr;
    const T2* A = op1 + B.op1;
    for (int idx = threadIdx.x; idx < nrow * rc; idx += NT) {
      int i = idx / rc, r = idx - i * rc;
      T2 acc = mk<T2>(0, 0);
      for (int kk = 0; kk < m; ++kk) acc = cfma(A[i + (int64_t)nrow * kk], y[kk * RC + r], acc);
      if (i < m) X[(int64_t)(so + i) * R + r0 + r] = acc;
      else GL[(int64_t)(B.cmo + i - m) * R + r0 + r] = acc;
    }
  } else {
    const T2* A = se + B.se;
    for (int idx = threadIdx.x; idx < m * rc; idx += NT) {
      int i = idx / rc, r = idx - i * rc;
      T2 acc = mk<T2>(0, 0);
      for (int kk = 0; kk < m; ++kk) acc = cfma(A[i + (int64_t)m * kk], y[kk * RC + r], acc);
      X[(int64_t)(so + i) * R + r0 + r] = acc;
    }
  }
}

// One column: a thread per row of the element's matrix, its sum in order.  The chain of
// such a block is its cost (record, slot records, gathered rows, 60 matrix columns), so
// the matrix is read SLOT_AHEAD columns ahead of the sum, the first ones before the
// operand is gathered, and a block has no more waves than rows.  F and P^-1 of the
// point source (32x32 elements, 60 slots each) 7.2 -> 6.2 and 8.1 -> 7.0 us, of the
// refined disk 7.8 -> 6.5 and 7.6 -> 6.0.  (Phi read ahead in the same way in
// k_slot_coarse, whose other waves gather, took it from 12 to 23 us at 64x64 elements:
// its 155 registers leave three waves a SIMD.)
constexpr int SLOT_AHEAD = 16;

template <class T2>
struct ColumnSum {
  T2 a[SLOT_AHEAD];
  const T2* A;
  int ld, K;
  // columns of row i from k0 on (past the last one: the last, against zeros)
  __device__ __forceinline__ void load(int i, int k0) {
#pragma unroll
    for (int q = 0; q < SLOT_AHEAD; ++q) a[q] = A[i + (int64_t)ld * min(k0 + q, K - 1)];
  }
  // acc + sum_k A[i, k] y[k ys]; y is zero up to the next multiple of SLOT_AHEAD past K
  __device__ __forceinline__ T2 sum(int i, const T2* y, int ys, T2 acc) {
    for (int k0 = 0; k0 < K; k0 += SLOT_AHEAD) {
      T2 b[SLOT_AHEAD];
#pragma unroll
      for (int q = 0; q < SLOT_AHEAD; ++q) b[q] = a[q];
      if (k0 + SLOT_AHEAD < K) load(i, k0 + SLOT_AHEAD);
#pragma unroll
      for (int q = 0; q < SLOT_AHEAD; ++q) acc = cfma(b[q], y[(k0 + q) * ys], acc);
    }
    return acc;
  }
};

enum SlotKind { SLOT_F, SLOT_P, SLOT_JUMPS, SLOT_ROWS };

// SLOT_F: op1 on the gathered dual rows (X and the coarse modes' GL); SLOT_P: S_e on
// them (X); SLOT_JUMPS: S_e on the jumps of the slots (X); SLOT_ROWS: the same, added
// into the dual rows `out` as k_slot_apply_rows does
template <class T2, int KIND>
__global__ void __launch_bounds__(NT) k_slot_one(const SlotBlock* __restrict__ blk, const SlotIn* __restrict__ sin,
                                                 const SlotOut* __restrict__ sout, const T2* __restrict__ mat,
                                                 const T2* __restrict__ v, T2* __restrict__ X, T2* __restrict__ GL,
                                                 double2* __restrict__ out) {
  using S = typename Scal<T2>::T;
  __shared__ T2 y[MMAX + SLOT_AHEAD];
  const SlotBlock B = blk[blockIdx.x];
  const int m = B.m, so = B.so, i = threadIdx.x;
  const int nrow = KIND == SLOT_F ? m + B.nr : m;
  ColumnSum<T2> c{{}, mat + (KIND == SLOT_F ? B.op1 : B.se), nrow, m};
  const int row = min(i, nrow - 1);
  if (m > 0) c.load(row, 0);
  for (int s = i; s < m + SLOT_AHEAD; s += blockDim.x) {
    S ax = 0, ay = 0;
    if (s < m) {
      const SlotIn g = sin[so + s];
      if (g.s0 >= 0) {
        const T2 z = v[g.s0];
        ax += S(g.a0) * z.x;
        ay += S(g.a0) * z.y;
      }
      if (KIND >= SLOT_JUMPS && g.s1 >= 0) {
        const T2 z = v[g.s1];
        ax += S(g.a1) * z.x;
        ay += S(g.a1) * z.y;
      }
    }
    y[s] = mk<T2>(ax, ay);
  }
  SlotOut o{};
  if (KIND == SLOT_ROWS && i < m) o = sout[so + i];
  __syncthreads();
  const T2 acc = c.sum(row, y, 1, mk<T2>(0, 0));
  if (i >= nrow) return;
  if (KIND == SLOT_ROWS) {
    double2* p = out + o.row;
    unsafeAtomicAdd(&p->x, o.coef * double(acc.x));
    unsafeAtomicAdd(&p->y, o.coef * double(acc.y));
  } else if (i < m) {
    X[so + i] = acc;
  } else {
    GL[B.cmo + i - m] = acc;
  }
}

// The preconditioner on dual slots (S_e on the jumps C_1 z of each element's
// slots) with the row gather fused: every output slot adds its value times its
// row coefficient into the dual row.  A row has at most two slots and out is
// zero on entry, so the two additions give the same sum in either order.
__global__ void __launch_bounds__(NT) k_slot_apply_rows(const SlotBlock* __restrict__ blk,
                                                        const SlotIn* __restrict__ sin,
                                                        const SlotOut* __restrict__ sout,
                                                        const double2* __restrict__ se,
                                                        const double2* __restrict__ v, double2* __restrict__ out,
                                                        int R) {
  __shared__ double2 y[MMAX * RC];
  const SlotBlock B = blk[blockIdx.x];
  const int m = B.m, so = B.so;
  const int r0 = blockIdx.y * RC;
  const int rc = min(RC, R - r0);
  for (int idx = threadIdx.x; idx < m * rc; idx += NT) {
    const int sl = idx / rc, r = idx - sl * rc;
    const SlotIn g = sin[so + sl];
    double ax = 0, ay = 0;
    if (g.s0 >= 0) {
      const double2 z = v[(int64_t)g.s0 * R + r0 + r];
      ax += g.a0 * z.x;
      ay += g.a0 * z.y;
    }
    if (g.s1 >= 0) {
      const double2 z = v[(int64_t)g.s1 * R + r0 + r];
      ax += g.a1 * z.x;
      ay += g.a1 * z.y;
    }
    y[sl * RC + r] = make_double2(ax, ay);
  }
  __syncthreads();
  const double2* A = se + B.se;
  for (int idx = threadIdx.x; idx < m * rc; idx += NT) {
    const int i = idx / rc, r = idx - i * rc;
    double2 acc = make_double2(0, 0);
    for (int kk = 0; kk < m; ++kk) acc = cfma(A[i + (int64_t)m * kk], y[kk * RC + r], acc);
    const SlotOut o = sout[so + i];
    double2* p = out + (int64_t)o.row * R + r0 + r;
    unsafeAtomicAdd(&p->x, o.coef * acc.x);
    unsafeAtomicAdd(&p->y, o.coef * acc.y);
  }
}

template <class T2>
__global__ void __launch_bounds__(NT) k_slot_coarse(const SlotBlock* __restrict__ blk, const T2* __restrict__ phi,
                                                    const int* __restrict__ t_ptr, const int* __restrict__ t_dof,
                                                    const double* __restrict__ t_coef, const T2* __restrict__ X,
                                                    const double2* __restrict__ w, T2* __restrict__ Z, int R) {
  __shared__ T2 we[NRMAX * RC];
  const SlotBlock B = blk[blockIdx.x];
  const int m = B.m, nr = B.nr, co = B.cmo, so = B.so;
  const int r0 = blockIdx.y * RC;
  const int rc = min(RC, R - r0);
  if (rc == 1) {
    // one column: each coarse mode's expansion (long on hanging edges) is split
    // over RC threads whose partial sums sit in we[j RC .. j RC + RC) and are
    // added in order into we[j RC]
    for (int idx = threadIdx.x; idx < nr * RC; idx += NT) {
      const int j = idx / RC, q = idx - j * RC;
      double ax = 0, ay = 0;
      for (int t = t_ptr[co + j] + q; t < t_ptr[co + j + 1]; t += RC) {
        const double2 a = w[(int64_t)t_dof[t] * R + r0];
        ax += t_coef[t] * a.x;
        ay += t_coef[t] * a.y;
      }
      we[idx] = mk<T2>(ax, ay);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < nr; j += NT) {
      T2 sum = we[j * RC];
      for (int q = 1; q < RC; ++q) {
        const T2 p = we[j * RC + q];
        sum.x += p.x;
        sum.y += p.y;
      }
      we[j * RC] = sum;
    }
  } else {
    for (int idx = threadIdx.x; idx < nr * rc; idx += NT) {
      int j = idx / rc, r = idx - j * rc;
      double ax = 0, ay = 0;
      for (int t = t_ptr[co + j]; t < t_ptr[co + j + 1]; ++t) {
        double2 a = w[(int64_t)t_dof[t] * R + r0 + r];
        ax += t_coef[t] * a.x;
        ay += t_coef[t] * a.y;
      }
      we[j * RC + r] = mk<T2>(ax, ay);
    }
  }
  __syncthreads();
  const T2* P = phi + B.phi;
  for (int idx = threadIdx.x; idx < m * rc; idx += NT) {
    int i = idx / rc, r = idx - i * rc;
    T2 acc = X[(int64_t)(so + i) * R + r0 + r];
    for (int j = 0; j < nr; ++j) acc = cfma(P[i + (int64_t)m * j], we[j * RC + r], acc);
    Z[(int64_t)(so + i) * R + r0 + r] = acc;
  }
}

typedef double d4 __attribute__((ext_vector_type(4)));

// The slot operators at 16, 32 or 64 right-hand sides on the FP64 matrix
// cores.  Per element (block): the K x R operand (gathered dual slots, or the
// element's coarse values for MODE 3) goes to LDS with R fastest; out = Mat
// operand, Mat column-major nrow x K (op1 for MODE 0, S_e for MODEs 1/2, Phi for
// MODE 3, which also adds X).  Wave w owns output tiles (16 rows of Mat) x (16
// columns of R) in turn; a step of 4 summation rows is four real 16x16x4
// operations per complex tile (A operand: 16 columns of R x 4 rows from LDS, B
// operand: 4 rows x 16 rows of Mat).  Lane l holds result (column (l >> 4) + 4 v,
// row l & 15) in value v; the tiles are written back to the LDS buffer and
// copied out with R fastest.  The LDS buffer holds max(K, nrow) x R entries
// (at most the largest such count over the classes, times R).
constexpr int SLOT_MF_LDS = 65536;
constexpr int SLOT_GB = 4;   // gathered operand entries per thread and pass

// The coarse values (T_e w)[kk][r] of an element's coarse modes kk < K (their
// expansions over the coarse unknowns, from t_ptr[cmo + kk]) for the RB columns
// from r0, into out (K x RB, r fastest).  SLOT_GB entries per thread and pass:
// the first term of every expansion (pointer, then index and coefficient, then
// the row of w) is requested for all of them before any is used; further terms
// (modes on hanging edges) follow in expansion order.
template <class OT>
__device__ __forceinline__ void gather_coarse(const int* __restrict__ t_ptr, const int* __restrict__ t_dof,
                                              const double* __restrict__ t_coef, const double2* __restrict__ v,
                                              int cmo, int K, int RB, int R, int r0, OT* out) {
  for (int i0 = threadIdx.x; i0 < K * RB; i0 += NT * SLOT_GB) {
    int p0[SLOT_GB], p1[SLOT_GB];
#pragma unroll
    for (int u = 0; u < SLOT_GB; ++u) {
      const int co = cmo + min(i0 + u * NT, K * RB - 1) / RB;
      p0[u] = t_ptr[co];
      p1[u] = t_ptr[co + 1];
    }
    int d[SLOT_GB];
    double c[SLOT_GB];
#pragma unroll
    for (int u = 0; u < SLOT_GB; ++u) {
      const bool has = p1[u] > p0[u];
      d[u] = has ? t_dof[p0[u]] : -1;
      c[u] = has ? t_coef[p0[u]] : 0.0;
    }
    double2 z[SLOT_GB];
#pragma unroll
    for (int u = 0; u < SLOT_GB; ++u) {
      const int idx = i0 + u * NT, r = idx % RB;
      z[u] = make_double2(0, 0);
      if (idx < K * RB && d[u] >= 0) z[u] = v[(int64_t)d[u] * R + r0 + r];
    }
#pragma unroll
    for (int u = 0; u < SLOT_GB; ++u) {
      const int idx = i0 + u * NT, r = idx % RB;
      if (idx >= K * RB) break;
      double sx = c[u] * z[u].x, sy = c[u] * z[u].y;
      for (int t = p0[u] + 1; t < p1[u]; ++t) {
        const double2 a = v[(int64_t)t_dof[t] * R + r0 + r];
        sx += t_coef[t] * a.x;
        sy += t_coef[t] * a.y;
      }
      out[idx] = mk<OT>(sx, sy);
    }
  }
}

// (at most 128 registers: four blocks per compute unit where the shared memory
// allows them; unbounded the compiler took 146 and three)
template <int MODE>
__global__ void __launch_bounds__(NT, 4) k_slot_mfma(const SlotBlock* __restrict__ blk,
                                                  const SlotIn* __restrict__ sin, const double2* __restrict__ op1,
                                                  const double2* __restrict__ se, const double2* __restrict__ phi,
                                                  const int* __restrict__ t_ptr, const int* __restrict__ t_dof,
                                                  const double* __restrict__ t_coef, const double2* __restrict__ v,
                                                  const double2* __restrict__ Xin, double2* __restrict__ X,
                                                  double2* __restrict__ GL, int R, int RB) {
  extern __shared__ double2 buf[];
  const int r0 = blockIdx.y * RB;   // this block's RB columns of the R
  const SlotBlock B = blk[blockIdx.x];
  const int m = B.m, nr = B.nr, so = B.so;
  const int K = MODE == 3 ? nr : m;
  const int nrow = MODE == 0 ? m + nr : m;
  const double2* Mat = MODE == 0 ? op1 + B.op1 : (MODE == 3 ? phi + B.phi : se + B.se);
  // operand rows kk x R
  if (MODE == 3) {
    gather_coarse<double2>(t_ptr, t_dof, t_coef, v, B.cmo, K, RB, R, r0, buf);
  } else {
    // SLOT_GB entries per thread and pass: the slot records, then the gathered
    // rows, are all requested before any is used
    for (int i0 = threadIdx.x; i0 < K * RB; i0 += NT * SLOT_GB) {
      SlotIn g[SLOT_GB];
#pragma unroll
      for (int u = 0; u < SLOT_GB; ++u) {
        const int idx = min(i0 + u * NT, K * RB - 1);
        g[u] = sin[so + idx / RB];
      }
      double2 z0[SLOT_GB], z1[SLOT_GB];
#pragma unroll
      for (int u = 0; u < SLOT_GB; ++u) {
        const int idx = i0 + u * NT, r = idx % RB;
        z0[u] = z1[u] = make_double2(0, 0);
        if (idx < K * RB && g[u].s0 >= 0) z0[u] = v[(int64_t)g[u].s0 * R + r0 + r];
        if (MODE == 2 && idx < K * RB && g[u].s1 >= 0) z1[u] = v[(int64_t)g[u].s1 * R + r0 + r];
      }
#pragma unroll
      for (int u = 0; u < SLOT_GB; ++u) {
        const int idx = i0 + u * NT;
        if (idx >= K * RB) break;
        double ax = g[u].a0 * z0[u].x, ay = g[u].a0 * z0[u].y;
        if (MODE == 2) {
          ax += g[u].a1 * z1[u].x;
          ay += g[u].a1 * z1[u].y;
        }
        buf[idx] = make_double2(ax, ay);
      }
    }
  }
  __syncthreads();
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int jl = l & 15, kq = l >> 4;
  const int nit = (nrow + 15) >> 4, nrt = RB >> 4, ntile = nit * nrt;
  // at most 4 row tiles x 4 column tiles: each wave keeps up to 4 tiles
  d4 cr[4], ci[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    cr[q] = (d4){0, 0, 0, 0};
    ci[q] = (d4){0, 0, 0, 0};
  }
  // two steps of 4 summation rows per pass: the operator entries of both steps
  // (global, cached) are requested before their matrix operations (one step per
  // pass for MODE 3, whose gather of coarse values needs the occupancy more)
  constexpr int NS = MODE == 3 ? 1 : 2;
  for (int k0 = 0; k0 < K; k0 += 4 * NS) {
    double2 bq[NS][4];
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const int kk = k0 + 4 * st + kq;
      const bool kv = kk < K;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int tile = min(wv + 4 * q, ntile - 1);
        const int it = tile / nrt;
        const int i = 16 * it + jl;
        bq[st][q] = (kv && i < nrow) ? Mat[i + (int64_t)nrow * kk] : make_double2(0, 0);
      }
    }
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const int kk = k0 + 4 * st + kq;
      const bool kv = kk < K;
      if (k0 + 4 * st >= K) break;   // uniform: a step wholly past K
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int tile = wv + 4 * q;
        if (tile >= ntile) break;   // uniform over the wave
        const int rt = tile - (tile / nrt) * nrt;
        const double2 b = bq[st][q];
        const double2 a = kv ? buf[kk * RB + 16 * rt + jl] : make_double2(0, 0);
        cr[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, cr[q], 0, 0, 0);
        ci[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, ci[q], 0, 0, 0);
        cr[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, cr[q], 0, 0, 0);
        ci[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, ci[q], 0, 0, 0);
      }
    }
  }
  __syncthreads();   // every wave is done with the operand
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int tile = wv + 4 * q;
    if (tile >= ntile) break;
    const int it = tile / nrt, rt = tile - it * nrt;
    const int i = 16 * it + jl;
    if (i < nrow) {
#pragma unroll
      for (int vv = 0; vv < 4; ++vv) buf[i * RB + 16 * rt + kq + 4 * vv] = make_double2(cr[q][vv], ci[q][vv]);
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < nrow * RB; idx += NT) {
    const int i = idx / RB, r = idx - i * RB;
    double2 o = buf[idx];
    if (MODE == 3) {
      const double2 x = Xin[(int64_t)(so + i) * R + r0 + r];
      o.x += x.x;
      o.y += x.y;
    }
    if (MODE != 0 || i < m) X[(int64_t)(so + i) * R + r0 + r] = o;
    else GL[(int64_t)(B.cmo + i - m) * R + r0 + r] = o;
  }
}

typedef float f4 __attribute__((ext_vector_type(4)));

// The slot operators of the mixed-precision path at 16, 32 or 64 right-hand
// sides on the FP32 matrix cores (FP32 operators and operands, FP32
// accumulation), laid out as k_slot_mfma: the K x RB operand in shared memory
// with R fastest, out = Mat operand, a step of 4 summation rows as four real
// 16x16x4 FP32 operations per complex tile.  The FP32 operation returns, in lane
// l and value v, row 4 (l >> 4) + v (the operand column) and column l & 15 (the
// row of Mat) of its 16 x 16 tile.  VT is the operand source type: FP32 dual or
// slot values, or (MODE 3) the FP64 coarse solution gathered through T.
template <int MODE, class VT>
__global__ void __launch_bounds__(NT) k_slot_mfma32(const SlotBlock* __restrict__ blk,
                                                    const SlotIn* __restrict__ sin, const float2* __restrict__ op1,
                                                    const float2* __restrict__ se, const float2* __restrict__ phi,
                                                    const int* __restrict__ t_ptr, const int* __restrict__ t_dof,
                                                    const double* __restrict__ t_coef, const VT* __restrict__ v,
                                                    const float2* __restrict__ Xin, float2* __restrict__ X,
                                                    float2* __restrict__ GL, int R, int RB) {
  extern __shared__ float2 buf32[];
  const int r0 = blockIdx.y * RB;
  const SlotBlock B = blk[blockIdx.x];
  const int m = B.m, nr = B.nr, so = B.so;
  const int K = MODE == 3 ? nr : m;
  const int nrow = MODE == 0 ? m + nr : m;
  const float2* Mat = MODE == 0 ? op1 + B.op1 : (MODE == 3 ? phi + B.phi : se + B.se);
  if (MODE == 3) {
    if constexpr (std::is_same<VT, double2>::value) gather_coarse<float2>(t_ptr, t_dof, t_coef, v, B.cmo, K, RB, R, r0, buf32);
  } else {
    // as k_slot_mfma: the slot records, then the gathered rows, all requested
    // before any is used
    for (int i0 = threadIdx.x; i0 < K * RB; i0 += NT * SLOT_GB) {
      SlotIn g[SLOT_GB];
#pragma unroll
      for (int u = 0; u < SLOT_GB; ++u) {
        const int idx = min(i0 + u * NT, K * RB - 1);
        g[u] = sin[so + idx / RB];
      }
      VT z0[SLOT_GB], z1[SLOT_GB];
#pragma unroll
      for (int u = 0; u < SLOT_GB; ++u) {
        const int idx = i0 + u * NT, r = idx % RB;
        z0[u].x = z0[u].y = z1[u].x = z1[u].y = 0;
        if (idx < K * RB && g[u].s0 >= 0) z0[u] = v[(int64_t)g[u].s0 * R + r0 + r];
        if (MODE == 2 && idx < K * RB && g[u].s1 >= 0) z1[u] = v[(int64_t)g[u].s1 * R + r0 + r];
      }
#pragma unroll
      for (int u = 0; u < SLOT_GB; ++u) {
        const int idx = i0 + u * NT;
        if (idx >= K * RB) break;
        float ax = float(g[u].a0) * z0[u].x, ay = float(g[u].a0) * z0[u].y;
        if (MODE == 2) {
          ax += float(g[u].a1) * z1[u].x;
          ay += float(g[u].a1) * z1[u].y;
        }
        buf32[idx] = make_float2(ax, ay);
      }
    }
  }
  __syncthreads();
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int jl = l & 15, kq = l >> 4;
  const int nit = (nrow + 15) >> 4, nrt = RB >> 4, ntile = nit * nrt;
  f4 cr[4], ci[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    cr[q] = (f4){0, 0, 0, 0};
    ci[q] = (f4){0, 0, 0, 0};
  }
  constexpr int NS = MODE == 3 ? 1 : 2;   // steps per pass, operator loads first (as k_slot_mfma)
  for (int k0 = 0; k0 < K; k0 += 4 * NS) {
    float2 bq[NS][4];
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const int kk = k0 + 4 * st + kq;
      const bool kv = kk < K;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int tile = min(wv + 4 * q, ntile - 1);
        const int i = 16 * (tile / nrt) + jl;
        bq[st][q] = (kv && i < nrow) ? Mat[i + (int64_t)nrow * kk] : make_float2(0, 0);
      }
    }
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const int kk = k0 + 4 * st + kq;
      const bool kv = kk < K;
      if (k0 + 4 * st >= K) break;   // uniform: a step wholly past K
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int tile = wv + 4 * q;
        if (tile >= ntile) break;   // uniform over the wave
        const int rt = tile - (tile / nrt) * nrt;
        const float2 b = bq[st][q];
        const float2 a = kv ? buf32[kk * RB + 16 * rt + jl] : make_float2(0, 0);
        cr[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, cr[q], 0, 0, 0);
        ci[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.y, ci[q], 0, 0, 0);
        cr[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(-a.y, b.y, cr[q], 0, 0, 0);
        ci[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.x, ci[q], 0, 0, 0);
      }
    }
  }
  __syncthreads();   // every wave is done with the operand
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int tile = wv + 4 * q;
    if (tile >= ntile) break;
    const int it = tile / nrt, rt = tile - it * nrt;
    const int i = 16 * it + jl;
    if (i < nrow) {
#pragma unroll
      for (int vv = 0; vv < 4; ++vv) buf32[i * RB + 16 * rt + 4 * kq + vv] = make_float2(cr[q][vv], ci[q][vv]);
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < nrow * RB; idx += NT) {
    const int i = idx / RB, r = idx - i * RB;
    float2 o = buf32[idx];
    if (MODE == 3) {
      const float2 x = Xin[(int64_t)(so + i) * R + r0 + r];
      o.x += x.x;
      o.y += x.y;
    }
    if (MODE != 0 || i < m) X[(int64_t)(so + i) * R + r0 + r] = o;
    else GL[(int64_t)(B.cmo + i - m) * R + r0 + r] = o;
  }
}

// k_slot_coarse with the coarse solution taken straight from the partial sums
// of the tiled coarse apply (one right-hand side): w[d] = sum_J P[d / 64][J][d % 64],
// each coarse mode's sum split over SCP thread groups and added in a fixed
// order, so the row-sum kernel is not needed.
constexpr int SCP = 16;
constexpr int SYM_TILE = 64;   // tile edge of the symmetric coarse inverse

template <class T2>
__global__ void __launch_bounds__(NT) k_slot_coarse_sym(const SlotBlock* __restrict__ blk, const T2* __restrict__ phi,
                                                        const int* __restrict__ t_ptr, const int* __restrict__ t_dof,
                                                        const double* __restrict__ t_coef,
                                                        const T2* __restrict__ X, const double2* __restrict__ P,
                                                        int nt, T2* __restrict__ Z) {
  extern __shared__ double2 part[];   // nr x SCP partial sums of the largest class
  __shared__ T2 we[NRMAX];
  const SlotBlock B = blk[blockIdx.x];
  const int m = B.m, nr = B.nr, co = B.cmo, so = B.so;
  for (int idx = threadIdx.x; idx < nr * SCP; idx += NT) {
    const int j = idx / SCP, q = idx - j * SCP;
    double ax = 0, ay = 0;
    for (int t = t_ptr[co + j]; t < t_ptr[co + j + 1]; ++t) {
      const int dof = t_dof[t];
      const double2* Pr = P + (int64_t)(dof / SYM_TILE) * nt * SYM_TILE + dof % SYM_TILE;
      double sx = 0, sy = 0;
      for (int J = q; J < nt; J += SCP) {
        const double2 a = Pr[(int64_t)J * SYM_TILE];
        sx += a.x;
        sy += a.y;
      }
      ax += t_coef[t] * sx;
      ay += t_coef[t] * sy;
    }
    part[idx] = make_double2(ax, ay);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < nr; j += NT) {
    double ax = 0, ay = 0;
    for (int q = 0; q < SCP; ++q) {
      ax += part[j * SCP + q].x;
      ay += part[j * SCP + q].y;
    }
    we[j] = mk<T2>(ax, ay);
  }
  __syncthreads();
  const T2* Pm = phi + B.phi;
  for (int i = threadIdx.x; i < m; i += NT) {
    T2 acc = X[so + i];
    for (int j = 0; j < nr; ++j) acc = cfma(Pm[i + (int64_t)m * j], we[j], acc);
    Z[so + i] = acc;
  }
}

// scale_row * (sum coef * src[pos(slot)] + sum_{C_2} coef * w[dof])
template <class T2>
__device__ __forceinline__ double2 row_value(int row, int r, int R, const int* __restrict__ row_slot,
                                             const double* __restrict__ row_coef,
                                             const double* __restrict__ row_xinv, const int64_t* __restrict__ slot_pos,
                                             const T2* __restrict__ src, const int* __restrict__ c2_ptr,
                                             const int* __restrict__ c2_dof, const double* __restrict__ c2_coef,
                                             const double2* __restrict__ w) {
  double ax = 0, ay = 0;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    int slot = row_slot[2 * row + t];
    if (slot < 0) continue;
    int64_t pos = slot_pos ? slot_pos[slot] : slot;
    T2 a = src[pos * R + r];
    double cf = row_coef[2 * row + t];
    ax += cf * double(a.x);
    ay += cf * double(a.y);
  }
  if (w)
    for (int t = c2_ptr[row]; t < c2_ptr[row + 1]; ++t) {
      double2 a = w[(int64_t)c2_dof[t] * R + r];
      ax += c2_coef[t] * a.x;
      ay += c2_coef[t] * a.y;
    }
  if (row_xinv) {
    ax *= row_xinv[row];
    ay *= row_xinv[row];
  }
  return make_double2(ax, ay);
}

template <class T2>
__global__ void k_rowgather(int nlam, const int* __restrict__ row_slot, const double* __restrict__ row_coef,
                            const double* __restrict__ row_xinv, const int64_t* __restrict__ slot_pos,
                            const T2* __restrict__ src, const int* __restrict__ c2_ptr,
                            const int* __restrict__ c2_dof, const double* __restrict__ c2_coef,
                            const double2* __restrict__ w, double2* __restrict__ u, int R) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)nlam * R) return;
  int row = int(idx / R), r = int(idx - (int64_t)row * R);
  u[idx] = row_value<T2>(row, r, R, row_slot, row_coef, row_xinv, slot_pos, src, c2_ptr, c2_dof, c2_coef, w);
}

// The same at one right-hand side with one wave per coarse unknown, for meshes
// with hanging edges: the lanes split the unknown's expansion and C_2 entries
// (long there) and add them with shuffles, so no lane walks a long list alone.
// (On conforming meshes the lists hold one to four entries and a thread per
// unknown is faster.)
template <class T2>
__global__ void __launch_bounds__(NT) k_assemble1(int nK, const int* __restrict__ ptr, const int* __restrict__ list,
                                                  const double* __restrict__ coef, const T2* __restrict__ GL,
                                                  const int64_t* __restrict__ cm_pos,
                                                  const double2* __restrict__ Bfull, const int* __restrict__ c2t_ptr,
                                                  const int* __restrict__ c2t_row,
                                                  const double* __restrict__ c2t_coef, const double2* __restrict__ v,
                                                  double csign, double2* __restrict__ g) {
  const int lane = threadIdx.x & 63;
  const int d = blockIdx.x * (NT / 64) + (threadIdx.x >> 6);
  if (d >= nK) return;
  double ax = 0, ay = 0;
  for (int t = ptr[d] + lane; t < ptr[d + 1]; t += 64) {
    const int i = list[t];
    const double c = coef[t];
    if (GL) {
      const T2 a = GL[i];
      ax += c * double(a.x);
      ay += c * double(a.y);
    }
    if (Bfull) {
      const double2 b = Bfull[cm_pos[i]];
      ax += c * b.x;
      ay += c * b.y;
    }
  }
  if (v)
    for (int t = c2t_ptr[d] + lane; t < c2t_ptr[d + 1]; t += 64) {
      const double2 a = v[c2t_row[t]];
      ax += csign * c2t_coef[t] * a.x;
      ay += csign * c2t_coef[t] * a.y;
    }
  for (int off = 32; off > 0; off >>= 1) {
    ax += __shfl_xor(ax, off, 64);
    ay += __shfl_xor(ay, off, 64);
  }
  if (lane == 0) g[d] = make_double2(ax, ay);
}

// g[d] = sum_{(i, c) in T^T} c (GL[i] + Bfull[pos(i)]) + csign sum_{(row, c) in C_2^T} c v[row]
template <class T2>
__global__ void k_assemble(int nK, const int* __restrict__ ptr, const int* __restrict__ list,
                           const double* __restrict__ coef, const T2* __restrict__ GL,
                           const int64_t* __restrict__ cm_pos, const double2* __restrict__ Bfull,
                           const int* __restrict__ c2t_ptr, const int* __restrict__ c2t_row,
                           const double* __restrict__ c2t_coef, const double2* __restrict__ v, double csign,
                           double2* __restrict__ g, int R) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)nK * R) return;
  int d = int(idx / R), r = int(idx - (int64_t)d * R);
  double ax = 0, ay = 0;
  for (int t = ptr[d]; t < ptr[d + 1]; ++t) {
    int i = list[t];
    double c = coef[t];
    if (GL) {
      T2 a = GL[(int64_t)i * R + r];
      ax += c * double(a.x);
      ay += c * double(a.y);
    }
    if (Bfull) {
      double2 b = Bfull[cm_pos[i] * R + r];
      ax += c * b.x;
      ay += c * b.y;
    }
  }
  if (v)
    for (int t = c2t_ptr[d]; t < c2t_ptr[d + 1]; ++t) {
      double2 a = v[(int64_t)c2t_row[t] * R + r];
      ax += csign * c2t_coef[t] * a.x;
      ay += csign * c2t_coef[t] * a.y;
    }
  g[idx] = make_double2(ax, ay);
}

// Dense blocks over the dual rows that C_2 couples (hanging edges).  They hold a few
// rows of the many (4 of 9,698 on the refined disk), so a launch of theirs is the
// chain of its loads: X^-1 v shares the launch that copies the other rows, and
// X^-1 (u + Y_2 s) the one that gathers them, in workgroups of their own.
// X^-1 Y X^-1 of the disk at 12 columns: 73 us a call with six launches, of it 3 + 8 +
// 4 + 9 + 6 for these steps, which take 3.6 + 4.3 now; 49 us.

// sum_j M[il, j] x[at(j)] for one block row, on a wave: 64 / RB lanes per column split the
// sum (RB columns, a power of two); valid in the first RB lanes.  at(j) may be a gathered
// index, so a term is two loads in turn: each lane takes four terms at a time, their
// indices first, past the last one the last against zeros.  (With the value under a
// column test, index and value were waited for term by term: a block of 512 rows and 4
// columns took 19.4 us a launch, 9.7 with a wave's 64 lanes along the sum; now 7.4.)
template <class At>
__device__ __forceinline__ double2 hblock_row(const double* __restrict__ Mb, int nb, int il, int RB, const double2* x,
                                              At&& at) {
  const int lane = threadIdx.x & 63, step = 64 / RB;
  double sx = 0, sy = 0;
  for (int j0 = lane / RB; j0 < nb; j0 += 4 * step) {
    double m[4];
    int64_t i[4];
    double2 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = min(j0 + q * step, nb - 1);
      i[q] = at(j);
      m[q] = Mb[il + (int64_t)nb * j];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = x[i[q]];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double f = j0 + q * step < nb ? m[q] : 0.0;
      sx += f * v[q].x;
      sy += f * v[q].y;
    }
  }
  for (int off = 32; off >= RB; off >>= 1) {
    sx += __shfl_xor(sx, off, 64);
    sy += __shfl_xor(sy, off, 64);
  }
  return make_double2(sx, sy);
}

// y = v, X^-1 v on the blocks' rows (hb_of: the row's number among them, or -1):
// workgroups of entries, then, from block `copies` on, a wave per block row and HB_R columns
constexpr int HB_R = 4;   // 16 lanes a column: sums of 16 rows in one step, of 64 in four loads in flight

__global__ void __launch_bounds__(NT) k_hcopy(int64_t count, int copies, const int* __restrict__ hb_of, int nh,
                                              const int* __restrict__ blk, const int* __restrict__ off,
                                              const int* __restrict__ rows, const int64_t* __restrict__ moff,
                                              const double* __restrict__ M, const double2* __restrict__ v,
                                              double2* __restrict__ y, int R, int RB) {
  if ((int)blockIdx.x < copies) {
    const int64_t idx = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (idx < count && hb_of[idx / R] < 0) y[idx] = v[idx];
    return;
  }
  const int nch = (R + RB - 1) / RB;
  const int t = ((int)blockIdx.x - copies) * (NT / 64) + (threadIdx.x >> 6), i = t / nch, r0 = (t - i * nch) * RB;
  if (i >= nh) return;
  const int b = blk[i], o = off[b], nb = off[b + 1] - o;
  const int lane = threadIdx.x & 63, r = min(r0 + (lane & (RB - 1)), R - 1);   // (columns past R are not stored)
  const double2 s = hblock_row(M + moff[b], nb, i - o, RB, v, [&](int j) { return (int64_t)rows[o + j] * R + r; });
  if (lane < RB && r0 + lane < R) y[(int64_t)rows[i] * R + r0 + lane] = s;
}

// u = the row gather of src; on the blocks' rows X^-1 (that + Y_2 s): workgroups of
// entries, then one per block and RB columns (the inner sums in shared memory)
template <class T2>
__global__ void __launch_bounds__(NT) k_hgather(int64_t count, int copies, const int* __restrict__ hb_of,
                                                const int* __restrict__ row_slot, const double* __restrict__ row_coef,
                                                const double* __restrict__ row_xinv, const T2* __restrict__ src,
                                                const int* __restrict__ off, const int* __restrict__ rows,
                                                const int64_t* __restrict__ moff, const double* __restrict__ Xi,
                                                const double* __restrict__ Y2, const double2* __restrict__ sv,
                                                double2* __restrict__ u, int R, int RB) {
  extern __shared__ double2 hbt[];   // [nb][RB]
  auto gather = [&](int row, int r) {
    return row_value<T2>(row, r, R, row_slot, row_coef, row_xinv, nullptr, src, nullptr, nullptr, nullptr, nullptr);
  };
  if ((int)blockIdx.x < copies) {
    const int64_t idx = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (idx >= count) return;
    const int row = int(idx / R);
    if (hb_of[row] < 0) u[idx] = gather(row, int(idx - (int64_t)row * R));
    return;
  }
  const int nch = (R + RB - 1) / RB, q = (int)blockIdx.x - copies;
  const int b = q / nch, r0 = (q - b * nch) * RB, o = off[b], nb = off[b + 1] - o;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, r = r0 + lane;
  const bool mine = lane < RB && r < R;
  const int rl = lane & (RB - 1), rc = min(r0 + rl, R - 1);
  for (int i = wv; i < nb; i += NT / 64) {
    const double2 a = mine ? gather(rows[o + i], r) : make_double2(0, 0);
    const double2 s = hblock_row(Y2 + moff[b], nb, i, RB, sv, [&](int j) { return (int64_t)rows[o + j] * R + rc; });
    if (lane < RB) hbt[i * RB + lane] = make_double2(s.x + a.x, s.y + a.y);
  }
  __syncthreads();
  for (int i = wv; i < nb; i += NT / 64) {
    const double2 s = hblock_row(Xi + moff[b], nb, i, RB, hbt, [&](int j) { return (int64_t)(j * RB + rl); });
    if (mine) u[(int64_t)rows[o + i] * R + r] = s;
  }
}

// Blocks too large for that: a wave per block row i and RB columns,
//   out_i = (add ? add[row_i] : 0) + sum_j M_b[i, j] in_j
// in_j is x[row_j] (gather) or x[off_b + j] (compact); out_i goes to
// y[row_i] (scatter) or y[off_b + i] (compact).
__global__ void __launch_bounds__(NT) k_hblock(int nh, const int* __restrict__ blk, const int* __restrict__ off,
                                               const int* __restrict__ rows, const int64_t* __restrict__ moff,
                                               const double* __restrict__ M, const double2* __restrict__ x,
                                               int in_gather, const double2* __restrict__ add,
                                               double2* __restrict__ y, int out_scatter, int R, int RB) {
  const int nch = (R + RB - 1) / RB;
  const int t = blockIdx.x * (NT / 64) + (threadIdx.x >> 6), i = t / nch, r0 = (t - i * nch) * RB;
  if (i >= nh) return;
  const int b = blk[i], o = off[b], nb = off[b + 1] - o;
  const int lane = threadIdx.x & 63, r = min(r0 + (lane & (RB - 1)), R - 1);
  double2 s = in_gather
      ? hblock_row(M + moff[b], nb, i - o, RB, x, [&](int j) { return (int64_t)rows[o + j] * R + r; })
      : hblock_row(M + moff[b], nb, i - o, RB, x, [&](int j) { return (int64_t)(o + j) * R + r; });
  if (lane >= RB || r0 + lane >= R) return;
  if (add) {
    const double2 a = add[(int64_t)rows[i] * R + r0 + lane];
    s.x += a.x;
    s.y += a.y;
  }
  y[(out_scatter ? (int64_t)rows[i] : (int64_t)i) * R + r0 + lane] = s;
}

// The top depths of the tree as one dense block (several columns): the
// right-hand side of the top unknowns once every deeper node is eliminated,
// r[i] = g[x_i] plus both child slots of each front row listed for x_i
// (its own row in a front of the deepest top depth, and the update rows of
// those fronts that couple to it); x_i = idx[i]; [n][R] and [nK][R] arrays.
__global__ void k_nd_top_gather(int n, const int* __restrict__ idx, const int64_t* __restrict__ gptr,
                                const int* __restrict__ grow, const double2* __restrict__ g,
                                const double2* __restrict__ slot, int64_t ld, int64_t sst, double2* __restrict__ r,
                                int R) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * R) return;
  const int i = int(e / R), c = int(e - (int64_t)i * R);
  double2 v = g[(int64_t)idx[i] * R + c];
  for (int64_t q = gptr[i]; q < gptr[i + 1]; ++q) {
    const double2* p = slot + (int64_t)grow[q] * ld + c;
    const double2 a = p[0], b = p[sst];
    v.x += a.x + b.x;
    v.y += a.y + b.y;
  }
  r[e] = v;
}

// w[x_i] = x[i] for the top unknowns ([n][R] into [nK][R]).
__global__ void k_nd_top_scatter(int n, const int* __restrict__ idx, const double2* __restrict__ x,
                                 double2* __restrict__ w, int R) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * R) return;
  const int i = int(e / R), c = int(e - (int64_t)i * R);
  w[(int64_t)idx[i] * R + c] = x[e];
}

// Set-up of the dense top block: columns k0 .. k0 + cols - 1 of (K^-1) restricted
// to the top unknowns, from the coarse solutions w ([nK][R]) of the unit vectors
// at x_k0 .., into the row-major n x n block M.
__global__ void k_nd_top_collect(int n, const int* __restrict__ idx, const double2* __restrict__ w, int R, int k0,
                                 int cols, double2* __restrict__ M) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * cols) return;
  const int i = int(e / cols), c = int(e - (int64_t)i * cols);
  M[(int64_t)i * n + k0 + c] = w[(int64_t)idx[i] * R + c];
}

// r = g - K x with K in CSR by row: one wave per row; at one column the lanes
// take the row's entries, otherwise the lanes are the columns.
__global__ void __launch_bounds__(NT) k_csr_residual(int n, const int64_t* __restrict__ ptr,
                                                     const int* __restrict__ col, const double2* __restrict__ val,
                                                     const double2* __restrict__ x, const double2* __restrict__ g,
                                                     double2* __restrict__ r, int R) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * (NT / 64) + (threadIdx.x >> 6);
  if (i >= n) return;
  const int64_t a = ptr[i], b = ptr[i + 1];
  if (R == 1) {
    double ax = 0, ay = 0;
    for (int64_t t = a + lane; t < b; t += 64) {
      const double2 m = val[t], v = x[col[t]];
      ax += m.x * v.x - m.y * v.y;
      ay += m.x * v.y + m.y * v.x;
    }
    for (int sh = 32; sh > 0; sh >>= 1) {
      ax += __shfl_xor(ax, sh, 64);
      ay += __shfl_xor(ay, sh, 64);
    }
    if (lane == 0) r[i] = make_double2(g[i].x - ax, g[i].y - ay);
    return;
  }
  for (int c = lane; c < R; c += 64) {
    double ax = 0, ay = 0;
    for (int64_t t = a; t < b; ++t) {
      const double2 m = val[t], v = x[(int64_t)col[t] * R + c];
      ax += m.x * v.x - m.y * v.y;
      ay += m.x * v.y + m.y * v.x;
    }
    const double2 gg = g[(int64_t)i * R + c];
    r[(int64_t)i * R + c] = make_double2(gg.x - ax, gg.y - ay);
  }
}

// w = K^-1 g: one wavefront per row of the (symmetric) inverse, RHS in chunks of 8.
__global__ void __launch_bounds__(NT) k_coarse_gemv(int nK, const double2* __restrict__ Kinv,
                                                    const double2* __restrict__ g, double2* __restrict__ w,
                                                    int R) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * (NT / 64) + (threadIdx.x >> 6);
  if (row >= nK) return;
  const double2* Kr = Kinv + (int64_t)row * nK;
  for (int r0 = 0; r0 < R; r0 += 8) {
    int rc = min(8, R - r0);
    double ax[8] = {0}, ay[8] = {0};
    for (int j = lane; j < nK; j += 64) {
      double2 a = Kr[j];
      for (int r = 0; r < rc; ++r) {
        double2 b = g[(int64_t)j * R + r0 + r];
        ax[r] += a.x * b.x - a.y * b.y;
        ay[r] += a.x * b.y + a.y * b.x;
      }
    }
    for (int r = 0; r < rc; ++r) {
      double sx = ax[r], sy = ay[r];
      for (int off = 32; off > 0; off >>= 1) {
        sx += __shfl_down(sx, off, 64);
        sy += __shfl_down(sy, off, 64);
      }
      if (lane == 0) w[(int64_t)row * R + r0 + r] = make_double2(sx, sy);
    }
  }
}

// ---------------------------------------------------------------------------
// One right-hand side against the symmetric inverse held as its upper 64 x 64
// tiles (I <= J): every tile is read once and serves both the block row I
// (y_I += T x_J) and, transposed, the block row J (y_J += T^T x_I), so the
// coarse step streams half of the dense inverse.  Tile t writes its two
// contributions to fixed places of a partial buffer P[row tile][column tile][64];
// a second kernel adds them per row in a fixed order (no atomics, so repeated
// solves give identical results).

// Packs the upper tiles of K^-1 from the dense row-major inverse, taking
// (A_ij + A_ji) / 2 (the computed inverse is symmetric up to rounding) and
// zero outside n_K.
__global__ void __launch_bounds__(NT) k_pack_sym_tiles(int nK, const double2* __restrict__ A,
                                                       const int2* __restrict__ tij, double2* __restrict__ tiles) {
  const int t = blockIdx.x;
  const int2 IJ = tij[t];
  double2* T = tiles + (int64_t)t * SYM_TILE * SYM_TILE;
  for (int e = threadIdx.x; e < SYM_TILE * SYM_TILE; e += NT) {
    const int i = IJ.x * SYM_TILE + e / SYM_TILE, j = IJ.y * SYM_TILE + e % SYM_TILE;
    double2 v = make_double2(0, 0);
    if (i < nK && j < nK) {
      const double2 a = A[(int64_t)i * nK + j], b = A[(int64_t)j * nK + i];
      v = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y + b.y));
    }
    T[e] = v;
  }
}

// SYM_WAVES waves per tile, rows in batches of SYM_KB: lane = column, the
// batch's loads all in flight at once.
constexpr int SYM_KB = 8;

// Exchange steps of the transposed row reduction: with M values per lane the
// partner is the lane across bit 32 M / SYM_KB, and that bit chooses the half
// of the values a lane keeps (and adds the partner's copy to).  The choice is
// made with weights 0 / 1 (exact for finite values) rather than selects, so
// that the values stay in fixed registers.
template <int M>
__device__ __forceinline__ void halve(double* vx, double* vy, int lane) {
  if constexpr (M > 1) {
    constexpr int o = 32 * M / SYM_KB;
    const double fh = (lane & o) ? 1.0 : 0.0, fl = 1.0 - fh;
#pragma unroll
    for (int i = 0; i < M / 2; ++i) {
      const double sx = fh * vx[i] + fl * vx[i + M / 2], sy = fh * vy[i] + fl * vy[i + M / 2];
      const double kx = fl * vx[i] + fh * vx[i + M / 2], ky = fl * vy[i] + fh * vy[i + M / 2];
      vx[i] = kx + __shfl_xor(sx, o, 64);
      vy[i] = ky + __shfl_xor(sy, o, 64);
    }
    halve<M / 2>(vx, vy, lane);
  }
}

// value of lane l (uniform l) in every lane
__device__ __forceinline__ double bcast_lane(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}

constexpr int SYM_WAVES = 4;   // waves per tile, each taking SYM_TILE / SYM_WAVES rows

__global__ void __launch_bounds__(SYM_WAVES * 64) k_coarse_symv_tiles(int nK, int nt, const int2* __restrict__ tij,
                                                                      const double2* __restrict__ tiles,
                                                                      const double2* __restrict__ g,
                                                                      double2* __restrict__ P) {
  __shared__ double2 red[SYM_WAVES][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int t = blockIdx.x;
  const double2* T = tiles + (int64_t)t * SYM_TILE * SYM_TILE;
  const int2 IJ = tij[t];
  const int jc = IJ.y * SYM_TILE + lane;
  const double2 xJ = jc < nK ? g[jc] : make_double2(0, 0);
  const int ir = IJ.x * SYM_TILE + lane;
  const double2 xIl = ir < nK ? g[ir] : make_double2(0, 0);   // x_I[lane], broadcast per row below
  double cx = 0, cy = 0;
  double2* Prow = P + ((int64_t)IJ.x * nt + IJ.y) * SYM_TILE;
  constexpr int rows = SYM_TILE / SYM_WAVES;
#pragma unroll 1
  for (int r0 = wv * rows; r0 < (wv + 1) * rows; r0 += SYM_KB) {
    double2 a[SYM_KB];
#pragma unroll
    for (int k = 0; k < SYM_KB; ++k) a[k] = T[(r0 + k) * SYM_TILE + lane];
    double vx[SYM_KB], vy[SYM_KB];
#pragma unroll
    for (int k = 0; k < SYM_KB; ++k) {
      vx[k] = a[k].x * xJ.x - a[k].y * xJ.y;
      vy[k] = a[k].x * xJ.y + a[k].y * xJ.x;
      const double xx = bcast_lane(xIl.x, r0 + k), xy = bcast_lane(xIl.y, r0 + k);
      cx += a[k].x * xx - a[k].y * xy;
      cy += a[k].x * xy + a[k].y * xx;
    }
    // row sums over the 64 lanes for the batch's rows at once: recursive halving
    // (each exchange keeps half of the rows, chosen by one bit of the lane), then
    // plain butterfly steps over the low lane bits; lane l ends with row
    // l / (64 / SYM_KB) of the batch
    halve<SYM_KB>(vx, vy, lane);
#pragma unroll
    for (int o = 32 / SYM_KB; o > 0; o >>= 1) {
      vx[0] += __shfl_xor(vx[0], o, 64);
      vy[0] += __shfl_xor(vy[0], o, 64);
    }
    constexpr int low = 64 / SYM_KB;   // lanes sharing one row sum
    if ((lane & (low - 1)) == 0) Prow[r0 + lane / low] = make_double2(vx[0], vy[0]);
  }
  if (IJ.x == IJ.y) return;   // a diagonal tile serves its own block row only
  red[wv][lane] = make_double2(cx, cy);
  __syncthreads();
  if (wv == 0) {
    double sx = 0, sy = 0;
#pragma unroll
    for (int q = 0; q < SYM_WAVES; ++q) {
      sx += red[q][lane].x;
      sy += red[q][lane].y;
    }
    P[((int64_t)IJ.y * nt + IJ.x) * SYM_TILE + lane] = make_double2(sx, sy);
  }
}

// w[I*64 + r] = sum_J P[I][J][r], J in increasing order within each wave's
// share, the four shares added in a fixed order.
__global__ void __launch_bounds__(NT) k_coarse_symv_reduce(int nK, int nt, const double2* __restrict__ P,
                                                           double2* __restrict__ w) {
  __shared__ double2 red[NT / 64][SYM_TILE];
  const int I = blockIdx.x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  double sx = 0, sy = 0;
  for (int J = wv; J < nt; J += NT / 64) {
    const double2 v = P[((int64_t)I * nt + J) * SYM_TILE + lane];
    sx += v.x;
    sy += v.y;
  }
  red[wv][lane] = make_double2(sx, sy);
  __syncthreads();
  if (wv == 0) {
    double tx = 0, ty = 0;
#pragma unroll
    for (int q = 0; q < NT / 64; ++q) {
      tx += red[q][lane].x;
      ty += red[q][lane].y;
    }
    const int row = I * SYM_TILE + lane;
    if (row < nK) w[row] = make_double2(tx, ty);
  }
}

// Xr[i][r] -= sum_t T(i, t) w[t][r] for every coarse mode i (its expansion over
// the coarse unknowns): the x_R - T_e w of the corrected element solve (-T_e w
// with from_zero).
__global__ void __launch_bounds__(NT) k_coarse_minus_tw(int ncm, int R, const int* __restrict__ t_ptr,
                                                        const int* __restrict__ t_dof,
                                                        const double* __restrict__ t_coef,
                                                        const double2* __restrict__ w, double2* __restrict__ Xr,
                                                        int from_zero) {
  const int64_t idx = (int64_t)blockIdx.x * NT + threadIdx.x;
  if (idx >= (int64_t)ncm * R) return;
  const int i = int(idx / R), r = int(idx - (int64_t)i * R);
  double2 x = from_zero ? make_double2(0, 0) : Xr[idx];
  for (int t = t_ptr[i]; t < t_ptr[i + 1]; ++t) {
    const double2 ww = w[(int64_t)t_dof[t] * R + r];
    x.x -= t_coef[t] * ww.x;
    x.y -= t_coef[t] * ww.y;
  }
  Xr[idx] = x;
}

// ---------------------------------------------------------------------------
// Vector kernels.
__global__ void k_axpby(const double2* __restrict__ x, const double2* __restrict__ y, double2* __restrict__ z,
                        int64_t count, double a, double b) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= count) return;
  double2 p = x[idx], q = y ? y[idx] : make_double2(0, 0);
  z[idx] = make_double2(a * p.x + b * q.x, a * p.y + b * q.y);
}

__global__ void k_cast_f(const double2* __restrict__ x, float2* __restrict__ y, int64_t count) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < count) y[idx] = make_float2(float(x[idx].x), float(x[idx].y));
}

// Far field, step 1: trace u and normal derivative d_n' u at the Gauss nodes of
// every boundary side of the enclosed region (Sec. 3.3.1), one block per
// (side, RHS).  For a side normal to x the trace row of the vertex-basis
// coefficients is X[a0, b] (a0 = 0 at x = +1, 1 at x = -1) and the normal
// derivative uses dN~_a(+-1); sides normal to y swap the roles.
__global__ void __launch_bounds__(NT) k_far_trace(const int* __restrict__ elem, const int* __restrict__ side,
                                                  const int* __restrict__ node_off, const int64_t* __restrict__ tab_off,
                                                  const double* __restrict__ tab, const double* __restrict__ dscale,
                                                  const int* __restrict__ elem_cls, const int* __restrict__ cls_n,
                                                  const int64_t* __restrict__ dof_off, const double2* __restrict__ X,
                                                  int R, double2* __restrict__ U, double2* __restrict__ DU) {
  __shared__ double2 tv[64], dv[64];
  const int g = blockIdx.x, r = blockIdx.y;
  const int e = elem[g], sd = side[g];
  const int n = cls_n[elem_cls[e]];
  const int64_t base = dof_off[e];
  // tab for this side: [q][n] basis values at the nodes, then dN~(end) (n values)
  const int q0 = node_off[g], nq = node_off[g + 1] - q0;
  const double* Nq = tab + tab_off[g];
  const double* dend = Nq + (int64_t)nq * n;
  const bool xside = sd <= 2;
  const int a0 = (sd == 2 || sd == 4) ? 0 : 1;
  for (int b = threadIdx.x; b < n; b += NT) {
    double2 t = xside ? X[(base + a0 + (int64_t)n * b) * R + r] : X[(base + b + (int64_t)n * a0) * R + r];
    double dx = 0, dy = 0;
    for (int a = 0; a < n; ++a) {
      double2 c = xside ? X[(base + a + (int64_t)n * b) * R + r] : X[(base + b + (int64_t)n * a) * R + r];
      dx += dend[a] * c.x;
      dy += dend[a] * c.y;
    }
    tv[b] = t;
    dv[b] = make_double2(dx * dscale[g], dy * dscale[g]);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < nq; q += NT) {
    double ux = 0, uy = 0, vx = 0, vy = 0;
    for (int b = 0; b < n; ++b) {
      double w = Nq[(int64_t)q * n + b];
      ux += w * tv[b].x;
      uy += w * tv[b].y;
      vx += w * dv[b].x;
      vy += w * dv[b].y;
    }
    U[(int64_t)(q0 + q) * R + r] = make_double2(ux, uy);
    DU[(int64_t)(q0 + q) * R + r] = make_double2(vx, vy);
  }
}

// Far field, step 2: E[r][phi] = sum_q w_q e^{-i k xhat.x_q} [(xhat.n'_q) U_q + (i k)^-1 DU_q].
// A workgroup takes FAR_A angles and FAR_R columns: w_q e^{-i k xhat.x_q} and xhat.n'_q
// of FAR_Q nodes are formed once (a sine and a cosine each) and shared by its columns,
// and a node's U and DU are read once for its angles.  360 angles and 64 columns on
// the boundary of a 64x64-element box: 316 us with a workgroup per angle and the
// phases formed by every column's thread, 77 now.
constexpr int FAR_A = 4, FAR_R = 16, FAR_Q = 64;

__global__ void __launch_bounds__(NT) k_far_sum(int nq, const double* __restrict__ px, const double* __restrict__ py,
                                                const double* __restrict__ pw, const double* __restrict__ pnx,
                                                const double* __restrict__ pny, const double* __restrict__ ang,
                                                double k, const double2* __restrict__ U, const double2* __restrict__ DU,
                                                int R, int nrhs_out, int nfar, double2* __restrict__ E) {
  __shared__ double2 red[NT];
  __shared__ double2 ph[FAR_A][FAR_Q];
  __shared__ double xn[FAR_A][FAR_Q];
  const int f0 = blockIdx.x * FAR_A, nf = min(FAR_A, nfar - f0);
  const int RB = min(R, FAR_R), r0 = blockIdx.y * RB;   // R is a power of two
  const int rl = threadIdx.x % RB, ql = threadIdx.x / RB, step = NT / RB;
  // the angle whose phases this thread forms
  const int tf = threadIdx.x / FAR_Q, tq = threadIdx.x % FAR_Q;
  static_assert(FAR_A * FAR_Q == NT, "one phase per thread");
  const double cx = cos(ang[f0 + min(tf, nf - 1)]), cy = sin(ang[f0 + min(tf, nf - 1)]);
  double2 acc[FAR_A];
#pragma unroll
  for (int f = 0; f < FAR_A; ++f) acc[f] = make_double2(0, 0);
  const double ik = 1.0 / k;
  for (int q0 = 0; q0 < nq; q0 += FAR_Q) {
    const int q = min(q0 + tq, nq - 1);
    const double a = -k * (cx * px[q] + cy * py[q]), w = q0 + tq < nq ? pw[q] : 0.0;
    __syncthreads();
    ph[tf][tq] = make_double2(w * cos(a), w * sin(a));
    xn[tf][tq] = cx * pnx[q] + cy * pny[q];
    __syncthreads();
    for (int t = ql; t < min(FAR_Q, nq - q0); t += step) {
      const double2 u = U[(int64_t)(q0 + t) * R + r0 + rl], du = DU[(int64_t)(q0 + t) * R + r0 + rl];
      const double2 v = make_double2(du.y * ik, -du.x * ik);   // (i k)^-1 du
#pragma unroll
      for (int f = 0; f < FAR_A; ++f) {
        const double2 c = ph[f][t];
        const double x = xn[f][t], tx = x * u.x + v.x, ty = x * u.y + v.y;
        acc[f].x += c.x * tx - c.y * ty;
        acc[f].y += c.x * ty + c.y * tx;
      }
    }
  }
#pragma unroll
  for (int f = 0; f < FAR_A; ++f) {
    if (f >= nf) break;   // uniform
    const double2 t = block_sum_by_rhs(acc[f], RB, red);
    if (threadIdx.x < RB && r0 + threadIdx.x < nrhs_out) E[(int64_t)(r0 + threadIdx.x) * nfar + f0 + f] = t;
  }
}

// The adjoint of the two far-field steps at one angle: the element vectors
// dE/dphi of the outside elements along the boundary (G is zero elsewhere, cleared
// before).  One workgroup per element: the sides of an element follow each other in
// the list, the first one's workgroup adds them all, in their order.  With
// T_b = sum_q w_q e^{-i k xhat.x_q} N~_b(t_q) a side's entry (a across it, b along it)
// is T_b ((xhat.n') [a = a0] + (i k)^-1 dscale dN~_a).  Formed on the host, with a
// whole zero vector to allocate and to send, it took 1.8 ms on 64x64 elements.
__global__ void __launch_bounds__(NT) k_far_adjoint(int nsides, const int* __restrict__ elem,
                                                    const int* __restrict__ side, const int* __restrict__ node_off,
                                                    const int64_t* __restrict__ tab_off,
                                                    const double* __restrict__ tab, const double* __restrict__ dscale,
                                                    const int* __restrict__ elem_cls, const int* __restrict__ cls_n,
                                                    const int64_t* __restrict__ dof_off,
                                                    const double* __restrict__ px, const double* __restrict__ py,
                                                    const double* __restrict__ pw, const double* __restrict__ pnx,
                                                    const double* __restrict__ pny, const double* __restrict__ ang,
                                                    double k, double2* __restrict__ G) {
  __shared__ double2 c[128], T[64];
  const int e = elem[blockIdx.x];
  if (blockIdx.x > 0 && elem[blockIdx.x - 1] == e) return;
  const int n = cls_n[elem_cls[e]];
  double2* __restrict__ g = G + dof_off[e];
  const double cx = cos(ang[0]), cy = sin(ang[0]);
  for (int s = blockIdx.x; s < nsides && elem[s] == e; ++s) {
    const int q0 = node_off[s], nq = node_off[s + 1] - q0, sd = side[s];
    const double* Nq = tab + tab_off[s];
    const double* dend = Nq + (int64_t)nq * n;
    for (int q = threadIdx.x; q < nq; q += NT) {
      const double a = -k * (cx * px[q0 + q] + cy * py[q0 + q]), w = pw[q0 + q];
      c[q] = make_double2(w * cos(a), w * sin(a));
    }
    __syncthreads();
    for (int b = threadIdx.x; b < n; b += NT) {
      double2 t = make_double2(0, 0);
      for (int q = 0; q < nq; ++q) {
        const double N = Nq[(int64_t)q * n + b];
        t.x += c[q].x * N;
        t.y += c[q].y * N;
      }
      T[b] = t;
    }
    __syncthreads();
    const bool xside = sd <= 2;
    const int a0 = (sd == 2 || sd == 4) ? 0 : 1;
    const double xn = cx * pnx[q0] + cy * pny[q0], ds = dscale[s] / k;
    for (int t = threadIdx.x; t < n * n; t += NT) {
      const int ix = t % n, iy = t / n, a = xside ? ix : iy, b = xside ? iy : ix;
      const double2 v = cmul(T[b], make_double2(a == a0 ? xn : 0.0, -ds * dend[a]));
      double2 o = s == (int)blockIdx.x ? make_double2(0, 0) : g[t];
      o.x += v.x;
      o.y += v.y;
      g[t] = o;
    }
    __syncthreads();
  }
}

// Plane-wave loads in the vertex basis:
// scattered field, f = k^2 (eps - 1) e^{ik d.x} (separable: b = f0 a (x) b);
// total field, impedance data g = ik(d.n - 1) e^{ik d.x} on the boundary sides.
// N holds the vertex basis at the element degree's Gauss nodes ([q][64]).
// One workgroup per (listed element, RB columns): the phases of its nodes are formed
// once per column (2 q or 4 q of them, in shared memory), then every basis function's
// integral, then the element's block in runs of RB columns.  With a workgroup per
// column and the phases formed again for every basis function, 256 elements of degree
// 12 and 64 angles took 330 us, nearly all of it sines and cosines; now 38.
constexpr int PW_R = 8;

__global__ void __launch_bounds__(NT) k_plane_wave_loads(
    int kind, const int* __restrict__ elems, const int* __restrict__ elem_cls, const int* __restrict__ cls_n,
    const int64_t* __restrict__ dof_off, const int* __restrict__ cls_q, const int64_t* __restrict__ cls_qoff,
    const double* __restrict__ qx, const double* __restrict__ qw, const double* __restrict__ qN,
    const double* __restrict__ ox, const double* __restrict__ oy, const double* __restrict__ hx,
    const double* __restrict__ hy, const double* __restrict__ eps, const int* __restrict__ bmask,
    const double* __restrict__ angles, double k, double2* __restrict__ B, int nrhs, int R, int RB) {
  extern __shared__ double2 sm[];
  const int e = elems[blockIdx.x], r0 = blockIdx.y * RB, nr = min(RB, nrhs - r0);
  const int c = elem_cls[e], n = cls_n[c], q = cls_q[c];
  const double* xq = qx + cls_qoff[c];
  const double* wq = qw + cls_qoff[c];
  const double* N = qN + cls_qoff[c] * 64;   // [q][64], basis padded to 64 columns
  const double X0 = ox[e], Y0 = oy[e], HX = hx[e], HY = hy[e];
  const int64_t base = dof_off[e];
  const int ns = kind == 2 ? 2 : 4;   // directions, or sides
  double2* ph = sm;                   // [ns][q][nr]: weighted phases
  double2* sv = sm + ns * q * nr;     // [ns][n][nr]: integrals against the basis
  for (int i = threadIdx.x; i < ns * q * nr; i += NT) {
    const int r = i % nr, st = i / nr, sd = st / q, t = st - sd * q;
    const double dx = cos(angles[r0 + r]), dy = sin(angles[r0 + r]);
    double2 v = make_double2(0, 0);
    if (kind == 2) {
      const double pos = sd ? Y0 + (xq[t] + 1) * HY / 2 : X0 + (xq[t] + 1) * HX / 2;
      const double p = k * (sd ? dy : dx) * pos;
      v = make_double2(cos(p), sin(p));
    } else if (bmask[e] & (1 << sd)) {
      const double nx = sd == 0 ? -1 : sd == 1 ? 1 : 0, ny = sd == 2 ? -1 : sd == 3 ? 1 : 0;
      const double gy = k * (dx * nx + dy * ny - 1.0);   // ik(d.n - 1)
      double x, y;
      if (sd <= 1) { x = sd == 0 ? X0 : X0 + HX; y = Y0 + (xq[t] + 1) * HY / 2; }
      else { y = sd == 2 ? Y0 : Y0 + HY; x = X0 + (xq[t] + 1) * HX / 2; }
      const double p = k * (dx * x + dy * y);
      v = make_double2(-gy * sin(p), gy * cos(p));
    }
    ph[i] = v;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < ns * n * nr; i += NT) {
    const int r = i % nr, st = i / nr, sd = st / n, m = st - sd * n;
    const double hl = kind == 2 ? 1.0 : (sd <= 1 ? HY : HX) / 2;
    double sx = 0, sy = 0;
    for (int t = 0; t < q; ++t) {
      const double wn = wq[t] * hl * N[(int64_t)t * 64 + m];
      const double2 v = ph[(sd * q + t) * nr + r];
      sx += wn * v.x;
      sy += wn * v.y;
    }
    sv[i] = make_double2(sx, sy);
  }
  __syncthreads();
  const double f0 = k * k * (eps[e] - 1.0) * (HX / 2) * (HY / 2);
  const int mask = kind == 2 ? 0 : bmask[e];
  for (int i = threadIdx.x; i < n * n * nr; i += NT) {
    const int r = i % nr, t = i / nr, ix = t % n, iy = t / n;
    double2 v = make_double2(0, 0);
    if (kind == 2) {
      const double2 p = cmul(sv[ix * nr + r], sv[(n + iy) * nr + r]);
      v = make_double2(f0 * p.x, f0 * p.y);
    } else {
      // the side vectors on the trace modes (left: ix=1, right: ix=0, bottom: iy=1,
      // top: iy=0); corners receive two contributions
      for (int sd = 0; sd < 4; ++sd) {
        const int across = sd <= 1 ? ix : iy, along = sd <= 1 ? iy : ix;
        if (!(mask & (1 << sd)) || across != (sd & 1 ? 0 : 1)) continue;
        const double2 a = sv[(sd * n + along) * nr + r];
        v.x += a.x;
        v.y += a.y;
      }
    }
    B[(base + t) * R + r0 + r] = v;
  }
}

// Adjoint gradient with respect to each element's relative permittivity:
//   dJ/d eps_e = 2 Re( conj(E) [ lambda_e^T db_e + k^2 (h_x h_y / 4) lambda_e^T (M~ (x) M~) u_e ] )
// with db_e = k^2 (h_x/2)(h_y/2) a (x) b the scattered-field load per unit (eps_e - 1)
// (a, b: the 1-D integrals of N~ e^{ik d x} as in the plane-wave loads).  One block per element.
__global__ void __launch_bounds__(NT) k_eps_grad(
    const int* __restrict__ elem_cls, const int* __restrict__ cls_n, const int64_t* __restrict__ dof_off,
    const int* __restrict__ cls_q, const int64_t* __restrict__ cls_qoff, const double* __restrict__ qx,
    const double* __restrict__ qw, const double* __restrict__ qN, const double* __restrict__ cls_M,
    const int64_t* __restrict__ cls_Moff, const double* __restrict__ ox, const double* __restrict__ oy,
    const double* __restrict__ hx, const double* __restrict__ hy, const double2* __restrict__ mass_fac,
    const double2* __restrict__ U, const double2* __restrict__ Lam, double2 E, double k, double dx, double dy,
    double* __restrict__ grad) {
  extern __shared__ double2 sm[];
  __shared__ double2 red[NT], ph[192];   // two directions of n + 40 <= 81 nodes
  const int e = blockIdx.x;
  const int c = elem_cls[e], n = cls_n[c], n2 = n * n, q = cls_q[c];
  double2* su = sm;
  double2* sT = sm + n2;
  double2* sa = sm + 2 * n2;
  double2* sb = sa + 64;
  const double* M = cls_M + cls_Moff[c];
  const double* xq = qx + cls_qoff[c];
  const double* wq = qw + cls_qoff[c];
  const double* N = qN + cls_qoff[c] * 64;
  const double X0 = ox[e], Y0 = oy[e], HX = hx[e], HY = hy[e];
  const int64_t base = dof_off[e];
  for (int t = threadIdx.x; t < n2; t += NT) su[t] = U[base + t];
  // the phases of the nodes in both directions, once (for every basis function the
  // kernel took 109 us at 64x64 elements, now 40)
  for (int i = threadIdx.x; i < 2 * q; i += NT) {
    const int t = i % q;
    const double pos = i >= q ? Y0 + (xq[t] + 1) * HY / 2 : X0 + (xq[t] + 1) * HX / 2;
    const double p = k * (i >= q ? dy : dx) * pos;
    ph[i] = make_double2(cos(p), sin(p));
  }
  __syncthreads();
  for (int m = threadIdx.x; m < 2 * n; m += NT) {
    const bool yd = m >= n;
    const int mm = yd ? m - n : m;
    double sx = 0, sy = 0;
    for (int t = 0; t < q; ++t) {
      const double wn = wq[t] * N[(int64_t)t * 64 + mm];
      const double2 e = ph[yd ? q + t : t];
      sx += wn * e.x;
      sy += wn * e.y;
    }
    if (yd) sb[mm] = make_double2(sx, sy); else sa[mm] = make_double2(sx, sy);
  }
  __syncthreads();
  // T = U M^T (U[c][d] = u[c + n d])
  for (int t = threadIdx.x; t < n2; t += NT) {
    const int cc = t % n, b = t / n;
    double ax = 0, ay = 0;
    for (int dd = 0; dd < n; ++dd) {
      const double m = M[b + n * dd];
      ax += m * su[cc + n * dd].x;
      ay += m * su[cc + n * dd].y;
    }
    sT[t] = make_double2(ax, ay);
  }
  __syncthreads();
  const double f0 = k * k * (HX / 2) * (HY / 2);
  const double fm = k * k * (HX * HY / 4);
  double vx = 0, vy = 0;
  for (int t = threadIdx.x; t < n2; t += NT) {
    const int a = t % n, b = t / n;
    double wx = 0, wy = 0;   // (M U M^T)[a][b]
    for (int cc = 0; cc < n; ++cc) {
      const double m = M[a + n * cc];
      wx += m * sT[cc + n * b].x;
      wy += m * sT[cc + n * b].y;
    }
    const double2 l = Lam[base + t];
    const double2 db = cmul(sa[a], sb[b]);
    double2 mw = make_double2(wx, wy);
    if (mass_fac) mw = cmul(mass_fac[e], mw);   // layers: the mass term carries s_x s_y
    const double px = f0 * db.x + fm * mw.x, py = f0 * db.y + fm * mw.y;
    vx += l.x * px - l.y * py;
    vy += l.x * py + l.y * px;
  }
  red[threadIdx.x] = make_double2(vx, vy);
  __syncthreads();
  for (int off = NT / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) {
      red[threadIdx.x].x += red[threadIdx.x + off].x;
      red[threadIdx.x].y += red[threadIdx.x + off].y;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) grad[e] = 2.0 * (E.x * red[0].x + E.y * red[0].y);
}

__global__ void k_fill_zero(double2* __restrict__ x, int64_t count) {
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < count) x[idx] = make_double2(0.0, 0.0);
}

// Scatter packed element blocks into a zeroed full-element array.
__global__ void k_block_scatter(const int* __restrict__ elems, const int64_t* __restrict__ src_off,
                                const int64_t* __restrict__ dof_off, const double2* __restrict__ src,
                                double2* __restrict__ full, int R) {
  const int b = blockIdx.x;
  const int e = elems[b];
  const int64_t len = src_off[b + 1] - src_off[b];
  const double2* sp = src + src_off[b];
  double2* dp = full + dof_off[e] * R;
  for (int64_t t = threadIdx.x; t < len; t += blockDim.x) dp[t] = sp[t];
}

__global__ void k_dense_scatter(const int64_t* __restrict__ idx, const double2* __restrict__ val, int64_t nnz,
                                double2* __restrict__ M) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < nnz) M[idx[t]] = val[t];
}

// ---------------------------------------------------------------------------
// Device-resident GMRES.  The iteration index j lives in device memory so every
// launch has a fixed shape; R (RHS count) divides 64 and thread t owns RHS
// column t % R.  nvec = j + 1 Arnoldi vectors take part in an iteration.

// w[row][r] += sign * sum_{i < nvec} V_i[row][r] h[i][r]; when npart is given the
// block also writes the partial squared norms of the updated w (per RHS column).
__global__ void __launch_bounds__(NT) k_mupdate(const double2* __restrict__ V, int64_t vs, const int* __restrict__ jptr,
                                                const double2* __restrict__ hc, double2* __restrict__ w,
                                                int n, int R, double sign, double* __restrict__ npart) {
  __shared__ double2 red[NT];
  const int nvec = *jptr;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int r = threadIdx.x % R;   // NT is a multiple of R, so idx % R == threadIdx.x % R
  double nx = 0;
  if (idx < (int64_t)n * R) {
    double ax = 0, ay = 0;
#pragma unroll 4
    for (int i = 0; i < nvec; ++i) {
      double2 a = V[(int64_t)i * vs + idx], b = hc[i * R + r];
      ax += a.x * b.x - a.y * b.y;
      ay += a.x * b.y + a.y * b.x;
    }
    double2 c = w[idx];
    double2 o = make_double2(c.x + sign * ax, c.y + sign * ay);
    w[idx] = o;
    nx = o.x * o.x + o.y * o.y;
  }
  if (npart) {
    double2 t = block_sum_by_rhs(make_double2(nx, 0), R, red);
    if (threadIdx.x < R) npart[blockIdx.x * R + threadIdx.x] = t.x;
  }
}

// The same update for short vectors (few rows x RHS): a workgroup owns 64
// entries and its four waves take every fourth Arnoldi vector, so that the
// chip holds four times as many waves and each lane has fewer loads in a row.
constexpr int UPD_SPLIT_MAX = 1 << 20;   // entries (rows x RHS) up to which the split form is used

__global__ void __launch_bounds__(NT) k_mupdate_split(const double2* __restrict__ V, int64_t vs,
                                                      const int* __restrict__ jptr,
                                                      const double2* __restrict__ hc, double2* __restrict__ w, int n,
                                                      int R, double sign, double* __restrict__ npart) {
  __shared__ double2 red[NT / 64][64];
  const int nvec = *jptr;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t idx = (int64_t)blockIdx.x * 64 + lane;
  const bool live = idx < (int64_t)n * R;
  const int r = lane % R;   // 64 is a multiple of R
  double ax = 0, ay = 0;
  if (live) {
#pragma unroll 4
    for (int i = wv; i < nvec; i += NT / 64) {
      const double2 a = V[(int64_t)i * vs + idx], b = hc[i * R + r];
      ax += a.x * b.x - a.y * b.y;
      ay += a.x * b.y + a.y * b.x;
    }
  }
  red[wv][lane] = make_double2(ax, ay);
  __syncthreads();
  if (wv == 0) {
    double nx = 0;
    if (live) {
      double sx = 0, sy = 0;
      for (int q = 0; q < NT / 64; ++q) {
        sx += red[q][lane].x;
        sy += red[q][lane].y;
      }
      const double2 c = w[idx];
      const double2 o = make_double2(c.x + sign * sx, c.y + sign * sy);
      w[idx] = o;
      nx = o.x * o.x + o.y * o.y;
    }
    if (npart) {
      for (int off = 32; off >= R && off > 0; off >>= 1) nx += __shfl_xor(nx, off, 64);
      if (lane < R) npart[(int64_t)blockIdx.x * R + lane] = nx;
    }
  }
}

// Partial squared norms of w per block and RHS column.
// With blockIdx.y = 1 those of w2, behind them.
__global__ void __launch_bounds__(NT) k_norm2_part(const double2* __restrict__ w1, const double2* __restrict__ w2,
                                                   int n, int R, double* __restrict__ part) {
  __shared__ double2 red[NT];
  const double2* __restrict__ w = blockIdx.y ? w2 : w1;
  const int r = threadIdx.x % R, rl = threadIdx.x / R, step = NT / R;
  double acc = 0;
  for (int64_t row = (int64_t)blockIdx.x * step + rl; row < n; row += (int64_t)gridDim.x * step) {
    double2 a = w[row * R + r];
    acc += a.x * a.x + a.y * a.y;
  }
  double2 s = block_sum_by_rhs(make_double2(acc, 0), R, red);
  if (threadIdx.x < R) part[(blockIdx.y * gridDim.x + blockIdx.x) * R + threadIdx.x] = s.x;
}

// nrm[r] = sqrt(sum_b part[b][r]): one block per RHS column (and vector: the second
// one's partials and norms follow the first's).
__global__ void __launch_bounds__(NT) k_norm_reduce(const double* __restrict__ part, int nblk, int R,
                                                    double* __restrict__ nrm) {
  __shared__ double2 red[NT];
  const int r = blockIdx.x;
  part += (int64_t)blockIdx.y * nblk * R;
  double acc = 0;
  for (int b = threadIdx.x; b < nblk; b += NT) acc += part[(int64_t)b * R + r];
  double2 t = block_sum_by_rhs(make_double2(acc, 0), 1, red);
  if (threadIdx.x == 0) nrm[blockIdx.y * R + r] = sqrt(t.x);
}

// out = w / nrm (zero where nrm = 0); out2 (optional) receives the same vector.
// The destination is V_kry + (j + 1) * vs when jptr is given, else out directly.
__global__ void __launch_bounds__(NT) k_normalize(const double2* __restrict__ w, const double* __restrict__ nrm,
                                                  int n, int R, double2* __restrict__ out,
                                                  const int* __restrict__ jptr, int64_t vs,
                                                  double2* __restrict__ out2) {
  __shared__ double inv[64];
  if (threadIdx.x < R) {
    double nv = nrm[threadIdx.x];
    inv[threadIdx.x] = nv > 0 ? 1.0 / nv : 0.0;
  }
  __syncthreads();
  double2* dst = out + (jptr ? (int64_t)(*jptr + 1) * vs : 0);
  for (int64_t idx = (int64_t)blockIdx.x * NT + threadIdx.x; idx < (int64_t)n * R; idx += (int64_t)gridDim.x * NT) {
    double f = inv[idx % R];
    double2 a = w[idx];
    double2 o = make_double2(a.x * f, a.y * f);
    dst[idx] = o;
    if (out2) out2[idx] = o;
  }
}

__device__ __forceinline__ double2 shfl_up2(double2 v, int d) {
  return make_double2(__shfl_up(v.x, d, 64), __shfl_up(v.y, d, 64));
}

// Column j of the Hessenberg matrix for system r: entries 0..j in hc and the
// subdiagonal entry sub (real, >= 0); the earlier rotations in csl, snl and
// g_j in gj, all in shared memory or registers.  Applies the earlier
// rotations, forms rotation j, updates g and the residual estimate.  Called
// by every thread of the block; xj_sh is block-shared scratch.
//
// The j earlier rotations form a chain: with x_0 = h_0 and h_i the new column,
// rotation i maps (x_i, h_{i+1}) to the rotated entry t_i = c_i x_i + s_i h_{i+1}
// and the carried value x_{i+1} = -conj(s_i) x_i + c_i h_{i+1}.  The carry is a
// first-order affine recurrence, so the first wave resolves it as a prefix scan
// of affine maps (each lane composes a segment of consecutive rotations, the
// segments are combined across lanes in six shuffle steps) instead of a chain
// of j dependent steps on one lane.
__device__ void givens_column(int j, int r, const double2* hc, double sub, const double2* csl, const double2* snl,
                              double2 gj, double2* __restrict__ H, double2* __restrict__ cs, double2* __restrict__ sn,
                              double2* __restrict__ g, const double* __restrict__ beta, int* __restrict__ done,
                              int* __restrict__ iters, double* __restrict__ resid, double tol, int maxvec, int R,
                              double* __restrict__ hist, double2* xj_sh) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    const int seg = (j + 63) / 64;
    const int s0 = min(j, lane * seg), s1 = min(j, s0 + seg);
    // this lane's segment as one map x -> A x + B
    double2 A = make_double2(1, 0), B = make_double2(0, 0);
    for (int i = s0; i < s1; ++i) {
      const double2 c = csl[i], s = snl[i], hb = hc[i + 1];
      const double2 al = make_double2(-s.x, s.y);   // -conj(s)
      B = cfma(c, hb, cmul(al, B));
      A = cmul(al, A);
    }
    // inclusive scan over the lanes, earlier segments applied first
    for (int d = 1; d < 64; d <<= 1) {
      const double2 Ap = shfl_up2(A, d), Bp = shfl_up2(B, d);
      if (lane >= d) {
        B = cfma(A, Bp, B);
        A = cmul(A, Ap);
      }
    }
    double2 Ae = shfl_up2(A, 1), Be = shfl_up2(B, 1);
    if (lane == 0) {
      Ae = make_double2(1, 0);
      Be = make_double2(0, 0);
    }
    const double2 x0 = hc[0];
    double2 x = cfma(Ae, x0, Be);   // carried value entering this lane's segment
    for (int i = s0; i < s1; ++i) {
      const double2 c = csl[i], s = snl[i], hb = hc[i + 1];
      H[((int64_t)j * maxvec + i) * R + r] = cfma(c, x, cmul(s, hb));
      x = cfma(c, hb, cmul(make_double2(-s.x, s.y), x));
    }
    if (j == 0 && lane == 0) *xj_sh = x0;
    if (j > 0 && s0 < s1 && s1 == j) *xj_sh = x;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double2 a = *xj_sh, b = make_double2(sub, 0.0);
    double aa = sqrt(a.x * a.x + a.y * a.y), bb = sqrt(b.x * b.x + b.y * b.y);
    double den = sqrt(aa * aa + bb * bb);
    double2 c, s;
    if (den == 0) { c = make_double2(1, 0); s = make_double2(0, 0); }
    else if (aa == 0) { c = make_double2(0, 0); s = make_double2(b.x / den, -b.y / den); }
    else {
      c = make_double2(aa / den, 0);
      double2 ph = make_double2(a.x / aa, a.y / aa);          // a / |a|
      s = make_double2((ph.x * b.x + ph.y * b.y) / den, (ph.y * b.x - ph.x * b.y) / den);  // ph conj(b) / den
    }
    cs[j * R + r] = c;
    sn[j * R + r] = s;
    H[((int64_t)j * maxvec + j) * R + r] =
        make_double2(c.x * a.x + s.x * b.x - s.y * b.y, c.x * a.y + s.x * b.y + s.y * b.x);
    const double2 gn = make_double2(-(s.x * gj.x + s.y * gj.y), -(s.x * gj.y - s.y * gj.x));
    g[(j + 1) * R + r] = gn;
    g[j * R + r] = make_double2(c.x * gj.x, c.x * gj.y);
    double res = sqrt(gn.x * gn.x + gn.y * gn.y) / beta[r];
    resid[r] = res;
    if (hist) hist[(int64_t)(j + 1) * R + r] = res;
    iters[r] = j + 1;
    if (res <= tol || sub == 0.0) done[r] = 1;
  }
}

// End of an iteration's scalar step: the last block to finish publishes
// status = {all converged, jnext} and sets j = jnext.  The status goes to
// host-mapped coherent memory (slot jnext - 1 mod STATUS_SLOTS), so the host
// reads it without a copy in the stream.
__device__ void publish_step(int jnext, int* __restrict__ jptr, const int* __restrict__ done, int R,
                             int* __restrict__ counter, int* __restrict__ status) {
  __syncthreads();
  int* st = status + 2 * ((jnext - 1) % STATUS_SLOTS);
  if (threadIdx.x == 0 && gridDim.x == 1) {
    // a single system: no other block to wait for (device-wide fences are costly
    // across the chip's separate L2 caches)
    st[0] = done[0];
    st[1] = jnext;
    *jptr = jnext;
  } else if (threadIdx.x == 0) {
    __threadfence();
    int prev = atomicAdd(counter, 1);
    if (prev == gridDim.x - 1) {
      __threadfence();
      int all = 1;
      for (int q = 0; q < R; ++q) all &= __hip_atomic_load(done + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      st[0] = all;
      st[1] = jnext;
      *jptr = jnext;
      *counter = 0;
    }
  }
}

// ---------------------------------------------------------------------------
// Arnoldi with delayed reorthogonalisation (one multi-dot and one update per
// iteration).  At iteration j the basis q_0..q_{j-1} is final and V_j holds a
// tentative vector u (projected once, scaled); z = P^-1 F u has just been
// formed.  One pass over the basis gives s = Q^H u, t = Q^H z, u^H z, |u|^2 and
// |z|^2, from which
//   q_j   = (u - Q s) / nu,                 nu^2 = |u|^2 - |s|^2,
//   column j-1 of H: h' + rho s on rows 0..j-1 and rho nu on row j, where h'
//          and rho are the first-pass coefficients and scale of u,
//   A q_j = (z - Q_{j+1} H s) / nu, so the first-pass coefficients of column j
//          are ([t; tau] - H s) / nu with tau = q_j^H z = (u^H z - s^H t) / nu,
//   u_next = (z - Q t - q_j tau) / sigma,   sigma^2 = |z|^2 - |t|^2 - |tau|^2,
//          and its scale rho_next = sigma / nu.
// The norms come from the dot products (exact for orthonormal Q); the scale of
// u only has to be the one used, since nu and the column entries are formed
// from the dots of the stored u itself.  Dot entries per chunk: s at 0..j-1, t
// at j..2j-1, then u^H z, |u|^2, |z|^2.

__device__ __forceinline__ void cdot_acc(double2 a, double2 b, double& x, double& y) {  // += conj(a) b
  x += a.x * b.x + a.y * b.y;
  y += a.x * b.y - a.y * b.x;
}

// Sums of N values (a power of two) over the lanes of equal lane % R: at each step a
// lane passes on the half of its values that its partner keeps, so four values take seven
// exchanges and not 24.  Lane l then
// holds value `which`, in v[0].
template <int N>
__device__ __forceinline__ int lane_sums(double (&v)[N], int R) {
  const int lane = threadIdx.x & 63;
  int which = 0, off = 32;
#pragma unroll
  for (int half = N / 2; half >= 1; half >>= 1, off >>= 1) {
    const bool up = lane & off;
#pragma unroll
    for (int q = 0; q < half; ++q) {
      const double keep = up ? v[half + q] : v[q], send = up ? v[q] : v[half + q];
      v[q] = keep + __shfl_xor(send, off, 64);
    }
    which += up ? half : 0;
  }
  for (; off >= R; off >>= 1) v[0] += __shfl_xor(v[0], off, 64);
  return which;
}

// few right-hand sides (R <= 4): one wave per (row chunk, basis vector or the extra
// item).  Point source, 27,776 unknowns, one column, 96 vectors on average: 11.6 us
// a launch for 43 MB of basis (12.6 with a butterfly over all six sums); groups of 2
// and 4 vectors, which share the reads of u and z, took 14.5 and 21.6, with too few
// loads in flight.
__global__ void __launch_bounds__(NT) k_dmdot_wave(const double2* __restrict__ V, int64_t vs,
                                                   const int* __restrict__ jptr, const double2* __restrict__ z, int n,
                                                   int R, int chunk, int nchunks, int dstride,
                                                   double2* __restrict__ part) {
  const int j = *jptr;
  const int nitems = nchunks * (j + 1);
  const int lane = threadIdx.x & 63;
  const int wave = blockIdx.x * (NT / 64) + (threadIdx.x >> 6);
  const int nwaves = gridDim.x * (NT / 64);
  const double2* u = V + (int64_t)j * vs;
  for (int item = wave; item < nitems; item += nwaves) {
    const int c = item % nchunks, i = item / nchunks;
    const int64_t lo = (int64_t)c * chunk * R, hi = min((int64_t)n, (int64_t)(c + 1) * chunk) * R;
    double2* pc = part + (int64_t)c * dstride * R + lane % R;
    double v[4] = {0, 0, 0, 0};
    if (i < j) {
      const double2* q = V + (int64_t)i * vs;   // q^H u, q^H z
#pragma unroll 4
      for (int64_t e = lo + lane; e < hi; e += 64) {
        const double2 a = q[e];
        cdot_acc(a, u[e], v[0], v[1]);
        cdot_acc(a, z[e], v[2], v[3]);
      }
    } else {
#pragma unroll 4
      for (int64_t e = lo + lane; e < hi; e += 64) {   // u^H z, |u|^2, |z|^2
        const double2 a = u[e], b = z[e];
        cdot_acc(a, b, v[0], v[1]);
        v[2] += a.x * a.x + a.y * a.y;
        v[3] += b.x * b.x + b.y * b.y;
      }
    }
    const int k = lane_sums(v, R);   // (lanes that hold the same value write it alike)
    if (i < j) {
      reinterpret_cast<double*>(pc + (int64_t)(k < 2 ? i : j + i) * R)[k & 1] = v[0];
    } else {
      double* o = reinterpret_cast<double*>(pc + (int64_t)(2 * j + max(0, k - 1)) * R);
      o[k == 1] = v[0];
      if (k >= 2) o[1] = 0;
    }
  }
}

// many right-hand sides: one block per (row chunk, group of DGV basis vectors
// or the extra item), threads own RHS column t % R; grouping the vectors reads
// the long u and z once per group instead of once per vector
constexpr int DGV = 4;

__global__ void __launch_bounds__(NT) k_dmdot_blk(const double2* __restrict__ V, int64_t vs,
                                                  const int* __restrict__ jptr, const double2* __restrict__ z, int n,
                                                  int R, int chunk, int nchunks, int dstride,
                                                  double2* __restrict__ part) {
  __shared__ double2 red[NT];
  const int j = *jptr;
  const int ng = (j + DGV - 1) / DGV;   // vector groups; group ng is the extra item
  const int nitems = nchunks * (ng + 1);
  const int r = threadIdx.x % R, rl = threadIdx.x / R, step = NT / R;
  const double2* u = V + (int64_t)j * vs;
  for (int item = blockIdx.x; item < nitems; item += gridDim.x) {
    const int c = item % nchunks, gi = item / nchunks;
    const int64_t lo = (int64_t)c * chunk, hi = min((int64_t)n, lo + chunk);
    double2* pc = part + (int64_t)c * dstride * R + r;
    if (gi < ng) {
      const int i0 = gi * DGV;
      double sx[DGV], sy[DGV], tx[DGV], ty[DGV];
#pragma unroll
      for (int t = 0; t < DGV; ++t) sx[t] = sy[t] = tx[t] = ty[t] = 0;
      for (int64_t row = lo + rl; row < hi; row += step) {
        const int64_t o = row * R + r;
        const double2 uo = u[o], zo = z[o];
#pragma unroll
        for (int t = 0; t < DGV; ++t) {
          if (i0 + t < j) {
            const double2 a = V[(int64_t)(i0 + t) * vs + o];
            cdot_acc(a, uo, sx[t], sy[t]);
            cdot_acc(a, zo, tx[t], ty[t]);
          }
        }
      }
#pragma unroll
      for (int t = 0; t < DGV; ++t) {
        if (i0 + t >= j) break;   // uniform over the block
        const double2 s0 = block_sum_by_rhs(make_double2(sx[t], sy[t]), R, red);
        const double2 s1 = block_sum_by_rhs(make_double2(tx[t], ty[t]), R, red);
        if (threadIdx.x < R) {
          pc[(int64_t)(i0 + t) * R] = s0;
          pc[(int64_t)(j + i0 + t) * R] = s1;
        }
      }
    } else {
      double x0 = 0, y0 = 0, x1 = 0, x2 = 0;
      for (int64_t row = lo + rl; row < hi; row += step) {
        const int64_t o = row * R + r;
        const double2 a = u[o], b = z[o];
        cdot_acc(a, b, x0, y0);
        x1 += a.x * a.x + a.y * a.y;
        x2 += b.x * b.x + b.y * b.y;
      }
      const double2 s0 = block_sum_by_rhs(make_double2(x0, y0), R, red);
      const double2 s1 = block_sum_by_rhs(make_double2(x1, x2), R, red);
      if (threadIdx.x < R) {
        pc[(int64_t)(2 * j) * R] = s0;
        pc[(int64_t)(2 * j + 1) * R] = make_double2(s1.x, 0);
        pc[(int64_t)(2 * j + 2) * R] = make_double2(s1.y, 0);
      }
    }
  }
}

// D[k][r] = sum_c part[c][k][r] for k < 2j + 3: one wave per (k, r)
__global__ void __launch_bounds__(NT) k_dmdot_reduce(const double2* __restrict__ part, int nchunks,
                                                     const int* __restrict__ jptr, int dstride, int R,
                                                     double2* __restrict__ D) {
  const int j = *jptr;
  const int lane = threadIdx.x & 63;
  const int idx = blockIdx.x * (NT / 64) + (threadIdx.x >> 6);   // k * R + r
  if (idx >= (2 * j + 3) * R) return;
  double ax = 0, ay = 0;
  for (int c = lane; c < nchunks; c += 64) {
    const double2 a = part[(int64_t)c * dstride * R + idx];
    ax += a.x;
    ay += a.y;
  }
  for (int off = 32; off > 0; off >>= 1) {
    ax += __shfl_xor(ax, off, 64);
    ay += __shfl_xor(ay, off, 64);
  }
  if (lane == 0) D[idx] = make_double2(ax, ay);
}

// block-wide sums of four values over all threads; valid in every thread
__device__ __forceinline__ void block_sum4(double (&v)[4], double (*red)[4]) {
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] += __shfl_xor(v[q], off, 64);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) red[wv][q] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    v[q] = 0;
    for (int u = 0; u < NT / 64; ++u) v[q] += red[u][q];
  }
}

// The scalar step of an iteration, one block per system r: finishes column j-1
// of H (stored unrotated in Hraw, then rotated by givens_column), forms the
// update coefficients uc = [s (j), t (j), tau, 1/nu, 1/sigma] and advances j.
// The first-pass coefficients of column j, which need H s, are formed by the
// update kernel that follows (they are first used in the next scalar step).
// Every global value the step needs is loaded up front; the column and the
// earlier rotations are kept in shared memory ((3 maxvec + 1) entries).
// D: the reduced dots, or with nch > 1 the partials of that many row chunks, cstride
// apart, which each thread adds for its entries.  A step is a chain of some 5 us
// (j, dots, two reductions, the rotation's square roots and quotients) at any j, so a
// reduction launch ahead of it is worth its 2 to 4 us only where one block's loads
// would take longer (DOTS_FOLD).
__global__ void __launch_bounds__(NT) k_dcgs_scalar(int* __restrict__ jptr, const double2* __restrict__ D, int nch,
                                                    int64_t cstride,
                                                    double2* __restrict__ Hraw, const double2* __restrict__ hprev,
                                                    double* __restrict__ rho, double2* __restrict__ uc,
                                                    double2* __restrict__ H, double2* __restrict__ cs,
                                                    double2* __restrict__ sn, double2* __restrict__ g,
                                                    const double* __restrict__ beta, int* __restrict__ done,
                                                    int* __restrict__ iters, double* __restrict__ resid, double tol,
                                                    int maxvec, int R, int* __restrict__ counter,
                                                    int* __restrict__ status, double* __restrict__ hist) {
  extern __shared__ double2 shm[];
  double2* col = shm;                  // column j-1: maxvec + 1 entries
  double2* csl = col + maxvec + 1;     // rotations 0..j-2
  double2* snl = csl + maxvec;
  __shared__ double red[NT / 64][4];
  __shared__ double2 xj_sh;
  const int r = blockIdx.x;
  const int j = *jptr;
  auto dot = [&](int k) {
    double2 a = D[(int64_t)k * R + r];
#pragma unroll 4
    for (int c = 1; c < nch; ++c) {
      const double2 b = D[c * cstride + (int64_t)k * R + r];
      a.x += b.x;
      a.y += b.y;
    }
    return a;
  };
  const double rho_prev = rho[r];
  const int is_done = done[r];
  const double2 gj = j >= 1 ? g[(j - 1) * R + r] : make_double2(0, 0);
  const double2 uz = dot(2 * j);
  const double uu = dot(2 * j + 1).x, zz = dot(2 * j + 2).x;
  double ss = 0, tt = 0, stx = 0, sty = 0;
  for (int i = threadIdx.x; i < j; i += NT) {
    const double2 a = dot(i), b = dot(j + i);
    const double2 hp = hprev[(int64_t)i * R + r];
    if (i < j - 1) {
      csl[i] = cs[(int64_t)i * R + r];
      snl[i] = sn[(int64_t)i * R + r];
    }
    uc[(int64_t)i * R + r] = a;
    uc[(int64_t)(j + i) * R + r] = b;
    col[i] = make_double2(hp.x + rho_prev * a.x, hp.y + rho_prev * a.y);
    ss += a.x * a.x + a.y * a.y;
    tt += b.x * b.x + b.y * b.y;
    cdot_acc(a, b, stx, sty);   // s^H t
  }
  double sums[4] = {ss, tt, stx, sty};
  block_sum4(sums, red);
  const double2 st = make_double2(sums[2], sums[3]);
  const double nu2 = uu - sums[0];
  const double nu = nu2 > 0 ? sqrt(nu2) : 0.0;
  const double inu = nu > 0 ? 1.0 / nu : 0.0;
  if (j >= 1) {
    // column j-1, unrotated, to Hraw (rows 0..j), then rotated
    if (threadIdx.x == 0) col[j] = make_double2(rho_prev * nu, 0);
    __syncthreads();
    for (int i = threadIdx.x; i <= j; i += NT) Hraw[((int64_t)(j - 1) * maxvec + i) * R + r] = col[i];
    if (!is_done) givens_column(j - 1, r, col, rho_prev * nu, csl, snl, gj, H, cs, sn, g, beta, done, iters, resid,
                                tol, maxvec, R, hist, &xj_sh);
  }
  if (threadIdx.x == 0) {
    // tau = (u^H z - s^H t) / nu; sigma^2 = |z|^2 - |t|^2 - |tau|^2
    const double2 tau = make_double2((uz.x - st.x) * inu, (uz.y - st.y) * inu);
    const double sg2 = zz - sums[1] - (tau.x * tau.x + tau.y * tau.y);
    const double sg = sg2 > 0 ? sqrt(sg2) : 0.0;
    const double isg = sg > 0 ? 1.0 / sg : 0.0;
    uc[(int64_t)(2 * j) * R + r] = tau;
    uc[(int64_t)(2 * j + 1) * R + r] = make_double2(inu, 0);
    uc[(int64_t)(2 * j + 2) * R + r] = make_double2(isg, 0);
    rho[r] = sg * inu;
  }
  publish_step(j + 1, jptr, done, R, counter, status);
}

// First-pass coefficients of column j, hprev = ([t; tau] - H s) / nu with H the
// unrotated (j+1) x j Hessenberg matrix: one (row, system) item per wave in turn.
// Every wave of the update kernels takes part, the last blocks first, so that the
// rows cost no launch of their own (with a block-wide dot per item the 33 rows of
// three blocks, 168 unknowns, took 8 of the 13 us of that update).
__device__ void first_pass_rows(int j, int R, int maxvec, const double2* __restrict__ Hraw,
                                const double2* __restrict__ uc, double2* __restrict__ hprev) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int item = (gridDim.x - 1 - blockIdx.x) * nw + wv; item < (j + 1) * R; item += gridDim.x * nw) {
    const int i = item / R, r = item - i * R;
    double x = 0, y = 0;
    for (int k = max(0, i - 1) + lane; k < j; k += 64) {
      const double2 a = Hraw[((int64_t)k * maxvec + i) * R + r], b = uc[(int64_t)k * R + r];
      x += a.x * b.x - a.y * b.y;
      y += a.x * b.y + a.y * b.x;
    }
    for (int off = 32; off > 0; off >>= 1) {
      x += __shfl_xor(x, off, 64);
      y += __shfl_xor(y, off, 64);
    }
    if (lane == 0) {
      const double2 c = uc[(int64_t)(i < j ? j + i : 2 * j) * R + r];
      const double inu = uc[(int64_t)(2 * j + 1) * R + r].x;
      hprev[(int64_t)i * R + r] = make_double2((c.x - x) * inu, (c.y - y) * inu);
    }
  }
}

// The update of iteration j (read as *jptr - 1, after the scalar step):
// V_j = q_j = (u - Q s) / nu and V_{j+1} = out2 = (z - Q t - q_j tau) / sigma.
// Short vectors: a workgroup owns 64 entries and its UW waves take every UW-th basis
// vector (a wave's loads, four in flight, are a chain: with four waves the update of
// the point source, 27,776 unknowns and 96 vectors on average, took 12.2 us).
constexpr int UW = 8;

__global__ void __launch_bounds__(64 * UW) k_dupdate_split(double2* __restrict__ V, int64_t vs,
                                                      const int* __restrict__ jptr, const double2* __restrict__ uc,
                                                      double2* __restrict__ z, int n, int R,
                                                      double2* __restrict__ out2, const double2* __restrict__ Hraw,
                                                      double2* __restrict__ hprev, int maxvec) {
  __shared__ double2 red[2][UW][64];
  const int j = *jptr - 1;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t idx = (int64_t)blockIdx.x * 64 + lane;
  const bool live = idx < (int64_t)n * R;
  const int r = lane % R;   // 64 is a multiple of R
  double sx = 0, sy = 0, tx = 0, ty = 0;
  if (live) {
#pragma unroll 4
    for (int i = wv; i < j; i += UW) {
      const double2 a = V[(int64_t)i * vs + idx], b = uc[(int64_t)i * R + r], c = uc[(int64_t)(j + i) * R + r];
      sx += a.x * b.x - a.y * b.y;
      sy += a.x * b.y + a.y * b.x;
      tx += a.x * c.x - a.y * c.y;
      ty += a.x * c.y + a.y * c.x;
    }
  }
  red[0][wv][lane] = make_double2(sx, sy);
  red[1][wv][lane] = make_double2(tx, ty);
  __syncthreads();
  if (wv == 0 && live) {
    double ax = 0, ay = 0, bx = 0, by = 0;
    for (int q = 0; q < UW; ++q) {
      ax += red[0][q][lane].x;
      ay += red[0][q][lane].y;
      bx += red[1][q][lane].x;
      by += red[1][q][lane].y;
    }
    const double2 tau = uc[(int64_t)(2 * j) * R + r];
    const double inu = uc[(int64_t)(2 * j + 1) * R + r].x, isg = uc[(int64_t)(2 * j + 2) * R + r].x;
    const double2 u = V[(int64_t)j * vs + idx], zv = z[idx];
    const double2 q = make_double2((u.x - ax) * inu, (u.y - ay) * inu);
    const double2 un = make_double2((zv.x - bx - (q.x * tau.x - q.y * tau.y)) * isg,
                                    (zv.y - by - (q.x * tau.y + q.y * tau.x)) * isg);
    V[(int64_t)j * vs + idx] = q;
    V[(int64_t)(j + 1) * vs + idx] = un;
    if (out2) out2[idx] = un;
    z[idx] = make_double2(0, 0);   // cleared for the next operator output (added into)
  }
  first_pass_rows(j, R, maxvec, Hraw, uc, hprev);
}

// the same for long vectors: one thread per entry over all basis vectors
__global__ void __launch_bounds__(NT) k_dupdate(double2* __restrict__ V, int64_t vs, const int* __restrict__ jptr,
                                                const double2* __restrict__ uc, double2* __restrict__ z, int n,
                                                int R, double2* __restrict__ out2, const double2* __restrict__ Hraw,
                                                double2* __restrict__ hprev, int maxvec) {
  const int j = *jptr - 1;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < (int64_t)n * R) {
    const int r = threadIdx.x % R;   // NT is a multiple of R
    double ax = 0, ay = 0, bx = 0, by = 0;
#pragma unroll 4
    for (int i = 0; i < j; ++i) {
      const double2 a = V[(int64_t)i * vs + idx], b = uc[(int64_t)i * R + r], c = uc[(int64_t)(j + i) * R + r];
      ax += a.x * b.x - a.y * b.y;
      ay += a.x * b.y + a.y * b.x;
      bx += a.x * c.x - a.y * c.y;
      by += a.x * c.y + a.y * c.x;
    }
    const double2 tau = uc[(int64_t)(2 * j) * R + r];
    const double inu = uc[(int64_t)(2 * j + 1) * R + r].x, isg = uc[(int64_t)(2 * j + 2) * R + r].x;
    const double2 u = V[(int64_t)j * vs + idx], zv = z[idx];
    const double2 q = make_double2((u.x - ax) * inu, (u.y - ay) * inu);
    const double2 un = make_double2((zv.x - bx - (q.x * tau.x - q.y * tau.y)) * isg,
                                    (zv.y - by - (q.x * tau.y + q.y * tau.x)) * isg);
    V[(int64_t)j * vs + idx] = q;
    V[(int64_t)(j + 1) * vs + idx] = un;
    if (out2) out2[idx] = un;
    z[idx] = make_double2(0, 0);
  }
  first_pass_rows(j, R, maxvec, Hraw, uc, hprev);
}

// End of a GMRES run: H y = g (upper triangular, one block per system) for the
// columns the system took, zero beyond; block 0 leaves the largest column count of
// all systems in jptr, and each its iteration count behind its residual in res
// ([2][rstride], ahead of the residual history), so that one copy carries all the
// host reads.  Blocks of EB columns, from the last: one wave solves the block's
// triangle out of shared memory, all threads take its columns off the rows above.
// With H copied to the host instead (the whole rectangle of maxvec rows a column, in
// pageable memory) and four more synchronous copies this end took 0.25 ms at one
// column and 0.45 ms at 64.
constexpr int EB = 32;

__global__ void __launch_bounds__(NT) k_gmres_end(const double2* __restrict__ H, const double2* __restrict__ g,
                                                  const int* __restrict__ iters, int maxvec, int R,
                                                  double2* __restrict__ y, int* __restrict__ jptr,
                                                  double* __restrict__ res, int rstride) {
  extern __shared__ double2 b[];           // right-hand side, then solution: the system's columns
  __shared__ double2 T[EB][EB + 1];        // T[c][l] = H(b0 + l, b0 + c)
  const int r = blockIdx.x, k = iters[r];
  int kmax = 0;
  for (int q = 0; q < R; ++q) kmax = max(kmax, iters[q]);
  auto at = [&](int i, int c) { return H[((int64_t)c * maxvec + i) * R + r]; };
  for (int i = threadIdx.x; i < k; i += NT) b[i] = g[(int64_t)i * R + r];
  for (int b0 = k > 0 ? (k - 1) / EB * EB : -1; b0 >= 0; b0 -= EB) {
    const int nb = min(EB, k - b0);
    for (int q = threadIdx.x; q < nb * EB; q += NT) {
      const int c = q / EB, l = q - c * EB;
      if (l <= c) T[c][l] = at(b0 + l, b0 + c);
    }
    __syncthreads();
    if (threadIdx.x < 64) {
      const int l = min((int)threadIdx.x, nb - 1);
      // 1 / T_ll, scaled by the larger part
      const double2 d = T[l][l];
      double2 inv;
      if (fabs(d.x) >= fabs(d.y)) {
        const double q = d.y / d.x, den = d.x + d.y * q;
        inv = make_double2(1.0 / den, -q / den);
      } else {
        const double q = d.x / d.y, den = d.x * q + d.y;
        inv = make_double2(q / den, -1.0 / den);
      }
      double2 v = b[b0 + l];
      for (int c = nb - 1; c >= 0; --c) {
        const double2 yl = cmul(v, inv);
        const double2 yc = make_double2(__shfl(yl.x, c, 64), __shfl(yl.y, c, 64));
        if (l < c) {
          const double2 t = T[c][l];
          v.x -= t.x * yc.x - t.y * yc.y;
          v.y -= t.x * yc.y + t.y * yc.x;
        }
      }
      if (threadIdx.x < nb) b[b0 + l] = cmul(v, inv);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < b0; i += NT) {
      double2 v = b[i];
#pragma unroll 8
      for (int c = 0; c < nb; ++c) {
        const double2 t = at(i, b0 + c), yc = b[b0 + c];
        v.x -= t.x * yc.x - t.y * yc.y;
        v.y -= t.x * yc.y + t.y * yc.x;
      }
      b[i] = v;
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < kmax; i += NT) y[(int64_t)i * R + r] = i < k ? b[i] : make_double2(0, 0);
  if (threadIdx.x == 0) {
    res[rstride + r] = k;
    if (r == 0) *jptr = kmax;
  }
}

// Start of a GMRES run: g_0 = beta = ||P^-1 rhs||, flags cleared, j = 0.
__global__ void k_gmres_init(const double* __restrict__ nrm, double* __restrict__ beta, double2* __restrict__ g,
                             int* __restrict__ done, int* __restrict__ iters, double* __restrict__ resid,
                             int* __restrict__ jptr, int* __restrict__ counter, int* __restrict__ status, int R,
                             double* __restrict__ hist) {
  int r = threadIdx.x;
  if (r < R) {
    double b = nrm[r];
    beta[r] = b;
    g[r] = make_double2(b, 0);
    done[r] = b > 0 ? 0 : 1;
    iters[r] = 0;
    resid[r] = b > 0 ? 1.0 : 0.0;
    if (hist) hist[r] = resid[r];
  }
  if (r == 0) {
    *jptr = 0;
    *counter = 0;
    status[0] = 0;
    status[1] = 0;
  }
}

inline unsigned nblocks(int64_t n, int t = NT) { return unsigned((n + t - 1) / t); }
inline int pow2_at_least(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

}  // namespace

// ---------------------------------------------------------------------------
// shared memory of the matrix-core slot kernels at R columns, or 0 when they do
// not apply (R not a multiple of 16, or an element's operand or output rows do not
// fit: at most 64 KB and 16 output tiles per element)

// columns per block of the matrix-core slot operators: the handle's choice
// (16, 32 or 64; 32 unless tuned), at most R and a divisor of it (R is a multiple of 16)
static int slot_rb(const Handle& h, int R) {
  int rb = std::min(R, h.slot_rb);
  while (R % rb) rb -= 16;
  return rb;
}

static size_t slot_mfma_lds(const Handle& h, int R, int mode) {
  if (R < 16 || R % 16 != 0) return 0;
  const int rb = slot_rb(h, R);
  int rows = 0;   // operand and output rows: m + nr (interface operator) or max(m, nr)
  for (auto& C : h.classes) rows = std::max(rows, mode == 0 ? C.m + C.nr : std::max(C.m, C.nr));
  const size_t lds = size_t(rows) * rb * sizeof(double2);
  if (lds > SLOT_MF_LDS || ((rows + 15) / 16) * (rb / 16) > 16) return 0;
  return lds;
}

// threads of the one-column slot kernels: the waves that hold the longest class's rows
static int slot_one_threads(const Handle& h, bool f) {
  int rows = 1;
  for (auto& C : h.classes) rows = std::max(rows, f ? C.m + C.nr : C.m);
  return (rows + 63) / 64 * 64;
}

bool slot_rows_fused(const Handle& h, int R) { return !h.nonconforming && R < 16; }

void launch_slot_apply_rows(const Handle& h, const double2* v, double2* out, int R, hipStream_t s) {
  const auto& d = h.d;
  if (R == 1)
    hipLaunchKernelGGL((k_slot_one<double2, SLOT_ROWS>), dim3(h.E), dim3(slot_one_threads(h, false)), 0, s, d.slot_blk,
                       d.slot_in[2], d.slot_out, d.se, v, nullptr, nullptr, out);
  else
    hipLaunchKernelGGL(k_slot_apply_rows, dim3(h.E, (R + RC - 1) / RC), dim3(NT), 0, s, d.slot_blk, d.slot_in[2],
                       d.slot_out, d.se, v, out, R);
  HIPCHECK(hipGetLastError());
}

template <class T2>
void launch_slot_apply(const Handle& h, int mode, const T2* v, T2* X, T2* GL, int R, hipStream_t s) {
  dim3 grid(h.E, (R + RC - 1) / RC);
  const auto& d = h.d;
  if constexpr (std::is_same<T2, double2>::value) {
    if (const size_t lds = slot_mfma_lds(h, R, mode)) {
      const int rb = slot_rb(h, R);
      const dim3 g(h.E, R / rb);
#define HDP_MF_ARGS d.slot_blk, d.slot_in[mode], d.op1, d.se, d.phi, d.t_ptr, d.t_dof, d.t_coef, v, nullptr, X, GL, R, rb
      if (mode == 0) hipLaunchKernelGGL(k_slot_mfma<0>, g, dim3(NT), lds, s, HDP_MF_ARGS);
      else if (mode == 1) hipLaunchKernelGGL(k_slot_mfma<1>, g, dim3(NT), lds, s, HDP_MF_ARGS);
      else hipLaunchKernelGGL(k_slot_mfma<2>, g, dim3(NT), lds, s, HDP_MF_ARGS);
#undef HDP_MF_ARGS
      HIPCHECK(hipGetLastError());
      return;
    }
  }
  if constexpr (std::is_same<T2, float2>::value) {
    if (const size_t lds = slot_mfma_lds(h, R, mode)) {   // FP32 operands: half the bytes of the FP64 sizing
      const int rb = slot_rb(h, R);
      const dim3 g(h.E, R / rb);
#define HDP_MF32_ARGS d.slot_blk, d.slot_in[mode], d.op1_f, d.se_f, d.phi_f, d.t_ptr, d.t_dof, d.t_coef, v, nullptr, X, GL, R, rb
      if (mode == 0) hipLaunchKernelGGL((k_slot_mfma32<0, float2>), g, dim3(NT), lds / 2, s, HDP_MF32_ARGS);
      else if (mode == 1) hipLaunchKernelGGL((k_slot_mfma32<1, float2>), g, dim3(NT), lds / 2, s, HDP_MF32_ARGS);
      else hipLaunchKernelGGL((k_slot_mfma32<2, float2>), g, dim3(NT), lds / 2, s, HDP_MF32_ARGS);
#undef HDP_MF32_ARGS
      HIPCHECK(hipGetLastError());
      return;
    }
  }
  const T2* op1;
  const T2* se;
  if constexpr (std::is_same<T2, double2>::value) { op1 = d.op1; se = d.se; }
  else { op1 = d.op1_f; se = d.se_f; }
  if (R == 1) {
    const dim3 t(slot_one_threads(h, mode == 0));
#define HDP_SLOT_ONE(KIND, MAT) \
  hipLaunchKernelGGL((k_slot_one<T2, KIND>), dim3(h.E), t, 0, s, d.slot_blk, d.slot_in[mode], nullptr, MAT, v, X, GL, \
                     nullptr)
    if (mode == 0) HDP_SLOT_ONE(SLOT_F, op1);
    else if (mode == 1) HDP_SLOT_ONE(SLOT_P, se);
    else HDP_SLOT_ONE(SLOT_JUMPS, se);
#undef HDP_SLOT_ONE
    HIPCHECK(hipGetLastError());
    return;
  }
#define HDP_SLOT_ARGS d.slot_blk, d.slot_in[mode], op1, se, v, X, GL, R
  if (mode == 0)
    hipLaunchKernelGGL((k_slot_apply<T2, 0>), grid, dim3(NT), 0, s, HDP_SLOT_ARGS);
  else if (mode == 1)
    hipLaunchKernelGGL((k_slot_apply<T2, 1>), grid, dim3(NT), 0, s, HDP_SLOT_ARGS);
  else
    hipLaunchKernelGGL((k_slot_apply<T2, 2>), grid, dim3(NT), 0, s, HDP_SLOT_ARGS);
#undef HDP_SLOT_ARGS
  HIPCHECK(hipGetLastError());
}

bool slot_coarse_from_tiles(const Handle& h, int R) {
  return R == 1 && h.coarse_mode == 0 && h.d.Ksym && !h.coarse_refine && !h.nonconforming;
}

template <class T2>
void launch_slot_coarse_sym(const Handle& h, const T2* X, T2* Z, hipStream_t s) {
  const auto& d = h.d;
  const T2* phi;
  if constexpr (std::is_same<T2, double2>::value) phi = d.phi; else phi = d.phi_f;
  int nrmax = 1;
  for (auto& C : h.classes) nrmax = std::max(nrmax, C.nr);
  const size_t shm = size_t(nrmax) * SCP * sizeof(double2);
  hipLaunchKernelGGL((k_slot_coarse_sym<T2>), dim3(h.E), dim3(NT), shm, s, d.slot_blk, phi, d.t_ptr, d.t_dof,
                     d.t_coef, X, d.sym_part, h.sym_nt, Z);
  HIPCHECK(hipGetLastError());
}
template void launch_slot_coarse_sym<double2>(const Handle&, const double2*, double2*, hipStream_t);
template void launch_slot_coarse_sym<float2>(const Handle&, const float2*, float2*, hipStream_t);

template <class T2>
static void slot_coarse_impl(const Handle& h, const T2* X, const double2* w, T2* Z, int R, hipStream_t s,
                             const int* t_ptr, const int* t_dof, const double* t_coef);

template <class T2>
void launch_slot_coarse(const Handle& h, const T2* X, const double2* w, T2* Z, int R, hipStream_t s) {
  slot_coarse_impl(h, X, w, Z, R, s, h.d.t_ptr, h.d.t_dof, h.d.t_coef);
}

void launch_slot_coarse_cm(const Handle& h, const double2* X, const double2* cm, double2* Z, int R, hipStream_t s) {
  slot_coarse_impl(h, X, cm, Z, R, s, h.d.id_ptr, h.d.id_dof, h.d.id_coef);
}

template <class T2>
static void slot_coarse_impl(const Handle& h, const T2* X, const double2* w, T2* Z, int R, hipStream_t s,
                             const int* t_ptr, const int* t_dof, const double* t_coef) {
  dim3 grid(h.E, (R + RC - 1) / RC);
  const auto& d = h.d;
  if constexpr (std::is_same<T2, double2>::value) {
    if (const size_t lds = slot_mfma_lds(h, R, 3)) {
      const int rb = slot_rb(h, R);
      hipLaunchKernelGGL(k_slot_mfma<3>, dim3(h.E, R / rb), dim3(NT), lds, s, d.slot_blk, nullptr, d.op1, d.se,
                         d.phi, t_ptr, t_dof, t_coef, w, X, Z, nullptr, R, rb);
      HIPCHECK(hipGetLastError());
      return;
    }
  }
  if constexpr (std::is_same<T2, float2>::value) {
    if (const size_t lds = slot_mfma_lds(h, R, 3)) {
      const int rb = slot_rb(h, R);
      hipLaunchKernelGGL((k_slot_mfma32<3, double2>), dim3(h.E, R / rb), dim3(NT), lds / 2, s, d.slot_blk, nullptr,
                         d.op1_f, d.se_f, d.phi_f, t_ptr, t_dof, t_coef, w, X, Z, nullptr, R, rb);
      HIPCHECK(hipGetLastError());
      return;
    }
  }
  const T2* phi;
  if constexpr (std::is_same<T2, double2>::value) phi = d.phi; else phi = d.phi_f;
  hipLaunchKernelGGL((k_slot_coarse<T2>), grid, dim3(NT), 0, s, d.slot_blk, phi, t_ptr, t_dof, t_coef, X, w, Z, R);
  HIPCHECK(hipGetLastError());
}

template <class T2>
void launch_rowgather(const Handle& h, const T2* src, bool full, bool precond, const double2* w, double2* u, int R,
                      hipStream_t s) {
  const auto& d = h.d;
  if (!h.nonconforming) w = nullptr;
  hipLaunchKernelGGL((k_rowgather<T2>), dim3(nblocks(int64_t(h.nlam) * R)), dim3(NT), 0, s, h.nlam, d.row_slot,
                     d.row_coef, precond ? d.row_xinv : nullptr, full ? d.slot_pos : nullptr, src, d.c2_ptr,
                     d.c2_dof, d.c2_coef, w, u, R);
  HIPCHECK(hipGetLastError());
}

template <class T2>
void launch_assemble(const Handle& h, const T2* GL, const double2* Bfull, const double2* v, double vsign, double2* g,
                     int R, hipStream_t s) {
  const auto& d = h.d;
  if (!h.nonconforming) v = nullptr;
  if (R == 1 && h.nonconforming) {   // long expansion and C_2 lists on hanging edges
    hipLaunchKernelGGL((k_assemble1<T2>), dim3(nblocks(h.nK, NT / 64)), dim3(NT), 0, s, h.nK, d.cdof_ptr, d.cdof_list,
                       d.cdof_coef, GL, d.cm_pos, Bfull, d.c2t_ptr, d.c2t_row, d.c2t_coef, v, vsign, g);
    HIPCHECK(hipGetLastError());
    return;
  }
  hipLaunchKernelGGL((k_assemble<T2>), dim3(nblocks(int64_t(h.nK) * R)), dim3(NT), 0, s, h.nK, d.cdof_ptr,
                     d.cdof_list, d.cdof_coef, GL, d.cm_pos, Bfull, d.c2t_ptr, d.c2t_row, d.c2t_coef, v, vsign, g,
                     R);
  HIPCHECK(hipGetLastError());
}

static int hb_cols(int R) {   // columns a wave takes: a power of two, at most HB_R
  int rb = 1;
  while (rb < R && rb < HB_R) rb <<= 1;
  return rb;
}

void launch_hcopy(const Handle& h, const double2* v, double2* y, int R, hipStream_t s) {
  const auto& d = h.d;
  const int RB = hb_cols(R), nch = (R + RB - 1) / RB;
  const int64_t count = int64_t(h.nlam) * R;
  const int copies = int(nblocks(count));
  hipLaunchKernelGGL(k_hcopy, dim3(copies + nblocks(int64_t(h.nh) * nch, NT / 64)), dim3(NT), 0, s, count, copies,
                     d.hb_of, h.nh, d.hb_blk, d.hb_off, d.hb_rows, d.hb_moff, d.hb_xinv, v, y, R, RB);
  HIPCHECK(hipGetLastError());
}

template <class T2>
void launch_hgather(const Handle& h, const T2* src, const double2* sv, double2* u, int R, hipStream_t s) {
  const auto& d = h.d;
  const int nblk = int(h.hb_off.size()) - 1, RB = hb_cols(R), nch = (R + RB - 1) / RB;
  const size_t lds = size_t(h.hb_largest) * RB * sizeof(double2);
  const int64_t count = int64_t(h.nlam) * R;
  const int copies = int(nblocks(count));
  hipLaunchKernelGGL((k_hgather<T2>), dim3(copies + nblk * nch), dim3(NT), lds, s, count, copies, d.hb_of, d.row_slot,
                     d.row_coef, d.row_xinv, src, d.hb_off, d.hb_rows, d.hb_moff, d.hb_xinv, d.hb_y2, sv, u, R, RB);
  HIPCHECK(hipGetLastError());
}

void launch_hblock(const Handle& h, bool y2, const double2* x, bool in_gather, const double2* add, double2* y,
                   bool out_scatter, int R, hipStream_t s) {
  const auto& d = h.d;
  const int RB = hb_cols(R), nch = (R + RB - 1) / RB;
  hipLaunchKernelGGL(k_hblock, dim3(nblocks(int64_t(h.nh) * nch, NT / 64)), dim3(NT), 0, s, h.nh, d.hb_blk, d.hb_off,
                     d.hb_rows, d.hb_moff, y2 ? d.hb_y2 : d.hb_xinv, x, int(in_gather), add, y, int(out_scatter), R,
                     RB);
  HIPCHECK(hipGetLastError());
}

template void launch_hgather<double2>(const Handle&, const double2*, const double2*, double2*, int, hipStream_t);
template void launch_hgather<float2>(const Handle&, const float2*, const double2*, double2*, int, hipStream_t);
template void launch_slot_apply<double2>(const Handle&, int, const double2*, double2*, double2*, int, hipStream_t);
template void launch_slot_apply<float2>(const Handle&, int, const float2*, float2*, float2*, int, hipStream_t);
template void launch_slot_coarse<double2>(const Handle&, const double2*, const double2*, double2*, int, hipStream_t);
template void launch_slot_coarse<float2>(const Handle&, const float2*, const double2*, float2*, int, hipStream_t);
template void launch_rowgather<double2>(const Handle&, const double2*, bool, bool, const double2*, double2*, int,
                                        hipStream_t);
template void launch_rowgather<float2>(const Handle&, const float2*, bool, bool, const double2*, double2*, int,
                                       hipStream_t);
template void launch_assemble<double2>(const Handle&, const double2*, const double2*, const double2*, double,
                                       double2*, int, hipStream_t);
template void launch_assemble<float2>(const Handle&, const float2*, const double2*, const double2*, double, double2*,
                                      int, hipStream_t);

// The tiled symmetric inverse at one column: partial products, then their row sums.
void launch_coarse_symv_tiles(const Handle& h, const double2* g, hipStream_t s) {
  hipLaunchKernelGGL(k_coarse_symv_tiles, dim3(h.sym_ntiles), dim3(SYM_WAVES * 64), 0, s, h.nK, h.sym_nt,
                     h.d.sym_tij, h.d.Ksym, g, h.d.sym_part);
  HIPCHECK(hipGetLastError());
}

void launch_coarse_symv_reduce(const Handle& h, double2* w, hipStream_t s) {
  hipLaunchKernelGGL(k_coarse_symv_reduce, dim3(h.sym_nt), dim3(NT), 0, s, h.nK, h.sym_nt, h.d.sym_part, w);
  HIPCHECK(hipGetLastError());
}

void launch_coarse_solve(const Handle& h, const double2* g, double2* w, int R, hipStream_t s) {
  if (R == 1 && h.d.Ksym) {
    launch_coarse_symv_tiles(h, g, s);
    launch_coarse_symv_reduce(h, w, s);
    return;
  }
  hipLaunchKernelGGL(k_coarse_gemv, dim3(nblocks(h.nK, NT / 64)), dim3(NT), 0, s, h.nK, h.d.Kinv, g, w, R);
  HIPCHECK(hipGetLastError());
}

int sym_tile_size() { return SYM_TILE; }

void launch_pack_sym_tiles(const Handle& h, hipStream_t s) {
  hipLaunchKernelGGL(k_pack_sym_tiles, dim3(h.sym_ntiles), dim3(NT), 0, s, h.nK, h.d.Kinv, h.d.sym_tij, h.d.Ksym);
  HIPCHECK(hipGetLastError());
}

void launch_coarse_minus_tw(const Handle& h, const double2* w, int R, bool from_zero, hipStream_t s) {
  const auto& d = h.d;
  hipLaunchKernelGGL(k_coarse_minus_tw, dim3(nblocks(int64_t(h.ncm) * R)), dim3(NT), 0, s, h.ncm, R, d.t_ptr, d.t_dof,
                     d.t_coef, w, d.cmX, from_zero ? 1 : 0);
  HIPCHECK(hipGetLastError());
}

GmresDims gmres_dims(int n, int R, int maxvec) {
  GmresDims g;
  g.step = NT / R;
  g.wave = R < 8;
  if (g.wave) {
    // one wave per (chunk, basis vector): 256 entries per chunk (four per lane),
    // more when the partial buffer's 512 chunks would not cover the rows; a
    // grid of up to 4,096 workgroups (16,384 waves) strides over the items
    g.chunk = int(std::max<int64_t>(256 / R, (int64_t(n) + 511) / 512));
    g.nchunks = int((int64_t(n) + g.chunk - 1) / g.chunk);
    g.grid = int(std::max<int64_t>(1, std::min<int64_t>(4096, (int64_t(g.nchunks) * maxvec + 3) / 4)));
  } else {
    // up to 512 row chunks (the partial buffer holds 512) keep the chip busy with
    // many right-hand sides while only a few Arnoldi vectors exist
    g.chunk = int(std::max<int64_t>(g.step, (int64_t(n) + 511) / 512));
    g.nchunks = int((int64_t(n) + g.chunk - 1) / g.chunk);
    g.grid = int(std::max<int64_t>(1, std::min<int64_t>(2048, int64_t(g.nchunks) * ((maxvec + DGV - 1) / DGV + 1))));
  }
  g.nnorm = int(std::max<int64_t>(1, std::min<int64_t>(256, (int64_t(n) * R + NT - 1) / NT)));
  return g;
}

void launch_mupdate(const double2* V, int64_t vs, const int* jptr, const double2* hc, double2* w, int n,
                    int R, double sign, double* npart, hipStream_t s) {
  if (int64_t(n) * R <= UPD_SPLIT_MAX)
    hipLaunchKernelGGL(k_mupdate_split, dim3(nblocks(int64_t(n) * R, 64)), dim3(NT), 0, s, V, vs, jptr, hc, w, n,
                       R, sign, npart);
  else
    hipLaunchKernelGGL(k_mupdate, dim3(nblocks(int64_t(n) * R)), dim3(NT), 0, s, V, vs, jptr, hc, w, n, R, sign,
                       npart);
  HIPCHECK(hipGetLastError());
}

// nrm[r] = |w_r|, and with w2 nrm[R + r] = |w2_r|
void launch_norms(const double2* w, const double2* w2, int n, int R, const GmresDims& g, double* part, double* nrm,
                  hipStream_t s) {
  const int two = w2 ? 2 : 1;
  hipLaunchKernelGGL(k_norm2_part, dim3(g.nnorm, two), dim3(NT), 0, s, w, w2, n, R, part);
  hipLaunchKernelGGL(k_norm_reduce, dim3(R, two), dim3(NT), 0, s, part, g.nnorm, R, nrm);
  HIPCHECK(hipGetLastError());
}

void launch_normalize(const double2* w, int n, int R, const GmresDims& g, double* part, double* nrm, double2* out,
                      const int* jptr, int64_t vs, double2* out2, hipStream_t s) {
  launch_norms(w, nullptr, n, R, g, part, nrm, s);
  hipLaunchKernelGGL(k_normalize, dim3(g.nnorm), dim3(NT), 0, s, w, nrm, n, R, out, jptr, vs, out2);
  HIPCHECK(hipGetLastError());
}

void launch_dmdot(const double2* V, int64_t vs, const int* jptr, const double2* z, int n, int R, const GmresDims& g,
                  int dstride, double2* part, hipStream_t s) {
  if (g.wave)
    hipLaunchKernelGGL(k_dmdot_wave, dim3(g.grid), dim3(NT), 0, s, V, vs, jptr, z, n, R, g.chunk, g.nchunks, dstride,
                       part);
  else
    hipLaunchKernelGGL(k_dmdot_blk, dim3(g.grid), dim3(NT), 0, s, V, vs, jptr, z, n, R, g.chunk, g.nchunks, dstride,
                       part);
  HIPCHECK(hipGetLastError());
}

void launch_dmdot_reduce(const double2* part, const GmresDims& g, const int* jptr, int dstride, int R, double2* D,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_dmdot_reduce, dim3(nblocks(int64_t(dstride) * R, NT / 64)), dim3(NT), 0, s, part, g.nchunks,
                     jptr, dstride, R, D);
  HIPCHECK(hipGetLastError());
}

void launch_dcgs_scalar(int* jptr, const double2* D, int nch, int64_t cstride, double2* Hraw, const double2* hprev, double* rho, double2* uc,
                        double2* H, double2* cs, double2* sn, double2* g, const double* beta, int* done, int* iters,
                        double* resid, double tol, int maxvec, int R, int* counter, int* status, double* hist,
                        hipStream_t s) {
  const size_t shm = (3 * size_t(maxvec) + 1) * sizeof(double2);
  hipLaunchKernelGGL(k_dcgs_scalar, dim3(R), dim3(NT), shm, s, jptr, D, nch, cstride, Hraw, hprev, rho, uc, H, cs, sn, g, beta,
                     done, iters, resid, tol, maxvec, R, counter, status, hist);
  HIPCHECK(hipGetLastError());
}

void launch_dupdate(double2* V, int64_t vs, const int* jptr, const double2* uc, double2* z, int n, int R,
                    double2* out2, const double2* Hraw, double2* hprev, int maxvec, hipStream_t s) {
  if (int64_t(n) * R <= UPD_SPLIT_MAX)
    // (blocks past the entries take first-pass rows alone)
    hipLaunchKernelGGL(k_dupdate_split, dim3(std::max(nblocks(int64_t(n) * R, 64), 32u)), dim3(64 * UW), 0, s, V, vs, jptr, uc, z, n, R,
                       out2, Hraw, hprev, maxvec);
  else
    hipLaunchKernelGGL(k_dupdate, dim3(nblocks(int64_t(n) * R)), dim3(NT), 0, s, V, vs, jptr, uc, z, n, R, out2, Hraw,
                       hprev, maxvec);
  HIPCHECK(hipGetLastError());
}

void launch_gmres_end(const double2* H, const double2* g, const int* iters, int maxvec, int R, double2* y, int* jptr,
                      double* res, int rstride, hipStream_t s) {
  hipLaunchKernelGGL(k_gmres_end, dim3(R), dim3(NT), size_t(maxvec) * sizeof(double2), s, H, g, iters, maxvec, R, y,
                     jptr, res, rstride);
  HIPCHECK(hipGetLastError());
}

void launch_gmres_init(const double* nrm, double* beta, double2* g, int* done, int* iters, double* resid, int* jptr,
                       int* counter, int* status, int R, double* hist, hipStream_t s) {
  hipLaunchKernelGGL(k_gmres_init, dim3(1), dim3(64), 0, s, nrm, beta, g, done, iters, resid, jptr, counter, status,
                     R, hist);
  HIPCHECK(hipGetLastError());
}

void launch_axpby(const double2* x, const double2* y, double2* z, int64_t count, double a, double b, hipStream_t s) {
  hipLaunchKernelGGL(k_axpby, dim3(nblocks(count)), dim3(NT), 0, s, x, y, z, count, a, b);
  HIPCHECK(hipGetLastError());
}

void launch_cast_f(const double2* x, float2* y, int64_t count, hipStream_t s) {
  hipLaunchKernelGGL(k_cast_f, dim3(nblocks(count)), dim3(NT), 0, s, x, y, count);
  HIPCHECK(hipGetLastError());
}

void launch_block_scatter(const int* elems, const int64_t* src_off, int nblk, const int64_t* dof_off,
                          const double2* src, double2* full, int R, hipStream_t s) {
  if (nblk == 0) return;
  hipLaunchKernelGGL(k_block_scatter, dim3(nblk), dim3(NT), 0, s, elems, src_off, dof_off, src, full, R);
  HIPCHECK(hipGetLastError());
}

void launch_far_field(const Handle& h, const double2* X, int R, int nrhs_out, double2* E, hipStream_t s) {
  const auto& d = h.d;
  const auto& f = h.far;
  if (f.nsides == 0) {
    launch_fill_zero(E, int64_t(nrhs_out) * f.nfar, s);
    return;
  }
  hipLaunchKernelGGL(k_far_trace, dim3(f.nsides, R), dim3(NT), 0, s, f.elem, f.side, f.node_off, f.tab_off, f.tab,
                     f.dscale, d.elem_cls, d.cls_n, d.dof_off, X, R, f.U, f.DU);
  hipLaunchKernelGGL(k_far_sum, dim3((f.nfar + FAR_A - 1) / FAR_A, (R + FAR_R - 1) / FAR_R), dim3(NT), 0, s, f.nq, f.px, f.py, f.pw, f.pnx, f.pny, f.ang, h.k, f.U,
                     f.DU, R, nrhs_out, f.nfar, E);
  HIPCHECK(hipGetLastError());
}

// G (dof, cleared here) = dE/dphi at the first angle of the prepared boundary
void launch_far_adjoint(const Handle& h, double2* G, hipStream_t s) {
  const auto& d = h.d;
  const auto& f = h.far;
  launch_fill_zero(G, h.dof, s);
  if (f.nsides == 0) return;
  hipLaunchKernelGGL(k_far_adjoint, dim3(f.nsides), dim3(NT), 0, s, f.nsides, f.elem, f.side, f.node_off, f.tab_off,
                     f.tab, f.dscale, d.elem_cls, d.cls_n, d.dof_off, f.px, f.py, f.pw, f.pnx, f.pny, f.ang, h.k, G);
  HIPCHECK(hipGetLastError());
}

void launch_plane_wave_loads(const Handle& h, int kind, const int* elems, int nel, const double* angles, double2* B,
                             int nrhs, int R, hipStream_t s) {
  if (nel == 0 || nrhs == 0) return;
  if (nrhs > R) fail(HDP_E_ARG, "plane-wave loads: more right-hand sides than the stride");
  const auto& d = h.d;
  size_t rows = 0;   // nodes and basis functions of the largest class
  for (auto& C : h.classes) rows = std::max(rows, h.quad_x.at(C.n).size() + size_t(C.n));
  const int RB = std::min(nrhs, PW_R);
  const size_t lds = rows * (kind == 2 ? 2 : 4) * RB * sizeof(double2);
  hipLaunchKernelGGL(k_plane_wave_loads, dim3(nel, (nrhs + RB - 1) / RB), dim3(NT), lds, s, kind, elems, d.elem_cls, d.cls_n, d.dof_off,
                     d.cls_q, d.cls_qoff, d.qx, d.qw, d.qN, d.ox, d.oy, d.hx, d.hy, d.eps, d.bmask, angles, h.k, B, nrhs, R, RB);
  HIPCHECK(hipGetLastError());
}

void launch_eps_gradient(const Handle& h, const double2* U, const double2* Lam, double2 E, double incidence,
                         double* grad, hipStream_t s) {
  const auto& d = h.d;
  int nmax = 0;
  for (auto& C : h.classes) nmax = std::max(nmax, C.n);
  const size_t shm = (size_t(2) * nmax * nmax + 128) * sizeof(double2);
  hipLaunchKernelGGL(k_eps_grad, dim3(h.E), dim3(NT), shm, s, d.elem_cls, d.cls_n, d.dof_off, d.cls_q, d.cls_qoff,
                     d.qx, d.qw, d.qN, d.cls_M, d.cls_Moff, d.ox, d.oy, d.hx, d.hy, d.mass_fac, U, Lam, E, h.k,
                     std::cos(incidence), std::sin(incidence), grad);
  HIPCHECK(hipGetLastError());
}

void launch_fill_zero(double2* x, int64_t count, hipStream_t s) {
  if (count == 0) return;
  hipLaunchKernelGGL(k_fill_zero, dim3(nblocks(count)), dim3(NT), 0, s, x, count);
  HIPCHECK(hipGetLastError());
}

void launch_csr_residual(int n, const int64_t* ptr, const int* col, const double2* val, const double2* x,
                         const double2* g, double2* r, int R, hipStream_t s) {
  hipLaunchKernelGGL(k_csr_residual, dim3(nblocks(n, NT / 64)), dim3(NT), 0, s, n, ptr, col, val, x, g, r, R);
  HIPCHECK(hipGetLastError());
}

void launch_nd_top_gather(int n, const int* idx, const int64_t* gptr, const int* grow, const double2* g,
                          const double2* slot, int64_t ld, int64_t sst, double2* r, int R, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_nd_top_gather, dim3(nblocks(int64_t(n) * R)), dim3(NT), 0, s, n, idx, gptr, grow, g, slot, ld,
                     sst, r, R);
  HIPCHECK(hipGetLastError());
}

void launch_nd_top_scatter(int n, const int* idx, const double2* x, double2* w, int R, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_nd_top_scatter, dim3(nblocks(int64_t(n) * R)), dim3(NT), 0, s, n, idx, x, w, R);
  HIPCHECK(hipGetLastError());
}

void launch_nd_top_collect(int n, const int* idx, const double2* w, int R, int k0, int cols, double2* M,
                           hipStream_t s) {
  if (n == 0 || cols == 0) return;
  hipLaunchKernelGGL(k_nd_top_collect, dim3(nblocks(int64_t(n) * cols)), dim3(NT), 0, s, n, idx, w, R, k0, cols, M);
  HIPCHECK(hipGetLastError());
}

void launch_dense_scatter(const int64_t* idx, const double2* val, int64_t nnz, double2* M, hipStream_t s) {
  if (nnz == 0) return;
  hipLaunchKernelGGL(k_dense_scatter, dim3(nblocks(nnz)), dim3(NT), 0, s, idx, val, nnz, M);
  HIPCHECK(hipGetLastError());
}

}  // namespace hdp
