// Sweeps of the nested-dissection coarse factor (gfx950, 64-wide waves).
//
// Node t of the tree owns the coarse unknowns I (nI of them) and couples to the
// ancestor unknowns B (nB).  Forward, deepest first, with Y = g + the children's
// updates on I:  U = A - L Y (A: the children's updates on B), stored into t's slot
// of its parent's rows; backward, root first:  X_I = D Y - L^T X_B.  Every front row
// has two slots, one per child, so the updates are plain stores and a slot row that
// no child writes stays zero from set-up.
//
// One column.  What bounds it near the root is the chain record -> operands -> sums ->
// store of a launch, about 4 us for 5 to 30 MB of factor; near the leaves the number of waves,
// as fronts there own 10 to 60 unknowns.  So two forms:
//  - k_nd1_row, long sums: a wave per output, its lanes along the row;
//  - k_nd1, short sums and many outputs: the product as out(j) = sum_k M[k][j] z_k with
//    j fastest, M = L^T (nI x nB) forward and [D^T; L] ((nI + nB) x nI, back to back in
//    the factor) backward, z = [Y; -X_B].  A wave works P outputs, 64 / P
//    rows of M side by side, z through its own piece of shared memory.  (A wave per
//    output left most lanes idle here and launched tens of thousands of waves of one
//    or two loads: 70,000 for the leaves of an 80x80 mesh.)  A workgroup takes a whole
//    subtree: the stages of a launch are consecutive depths, with a barrier between
//    instead of a launch.
// nd_units (coarse_nd.cpp) has the rules.  One coarse solve of the 80x80 layered
// scatterer (n_K = 71,361), within its GMRES: 21 launches and a clearing, 177 us, with a
// wave per output at every depth and atomic updates; 19 launches, 131 us.
//
// Several columns: k_nd_tile, below, also for the dense inverse (a one-node tree).
#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "kernels.hpp"

namespace hdp {

namespace {

// The right-hand side of interior row `row`: g plus the two children's updates.
__device__ __forceinline__ double2 front_rhs(const double2* __restrict__ g, const double2* slot, int64_t srows, int row) {
  const double2 y = g[row], s0 = slot[row], s1 = slot[srows + row];
  return make_double2(y.x + (s0.x + s1.x), y.y + (s0.y + s1.y));
}

// units[gptr[b (stages + 1) + s] ..] are the units (P outputs each) of stage s of
// workgroup b; its waves take them in turn.
template <bool BWD, int P>
__global__ void __launch_bounds__(512) k_nd1(const ND1Unit* __restrict__ units, const int* __restrict__ gptr,
                                              int stages, const double2* __restrict__ fac,
                                              const int* __restrict__ bnd, const int* __restrict__ push,
                                              const double2* __restrict__ g, double2* slot, int64_t srows, int nK,
                                              double2* X) {
  constexpr int SUB = 64 / P;   // rows of M side by side; P loads per lane for 64 rows
  __shared__ double2 zs[8][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  const int ks = lane / P;
  const int* gp = gptr + (int64_t)blockIdx.x * (stages + 1);
  for (int st = 0; st < stages; ++st) {
    const int u1 = gp[st + 1];
    for (int q = gp[st] + wave; q < u1; q += nw) {
      const ND1Unit U = units[q];
      const int rem = min(P, U.n_out - U.o0), i = min(lane & (P - 1), rem - 1);
      const int K = U.K;
      const double2* M = fac + U.mat;
      const int step = SUB * U.n_out, last = (K - 1) * U.n_out + U.o0 + i;
      double2 m[P];
      auto rows = [&](int k0) {   // rows past the last repeat it (their z is zero)
        const int off = (k0 + ks) * U.n_out + U.o0 + i;
#pragma unroll
        for (int b = 0; b < P; ++b) m[b] = M[min(off + b * step, last)];
      };
      auto index = [&](int k0) { return BWD ? bnd[U.bo + min(max(k0 + lane - U.nI, 0), K - 1 - U.nI)] : 0; };
      // the values of 64 rows: interior rows from the front, boundary rows from X
      auto value = [&](int k0, int at) {
        const int k = k0 + lane;
        double2 z = make_double2(0, 0);
        if (k < U.nI) z = front_rhs(g, slot, srows, U.o + k);
        else if (BWD && k < K) {
          const double2 x = X[at];
          z = make_double2(-x.x, -x.y);
        }
        return z;
      };
      rows(0);
      const bool bound = BWD && K > U.nI;
      int at = bound ? index(0) : 0;
      double2 a0 = make_double2(0, 0), a1 = a0;
      int dst = 0;
      if (!BWD) {   // the finishing lanes' operands
        const int64_t row = (int64_t)nK + U.u + U.o0 + i;
        dst = push[U.u + U.o0 + i];
        a0 = slot[row];
        a1 = slot[srows + row];
      }
      double2 z = value(0, at);
      at = bound ? index(64) : 0;
      double ax = 0, ay = 0;
      for (int k0 = 0; k0 < K; k0 += 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        zs[wave][lane] = z;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (k0 + 64 < K) {
          z = value(k0 + 64, at);
          if (bound) at = index(k0 + 128);
        }
#pragma unroll
        for (int b = 0; b < P; ++b) {
          const double2 zz = zs[wave][b * SUB + ks];
          ax += m[b].x * zz.x - m[b].y * zz.y;
          ay += m[b].x * zz.y + m[b].y * zz.x;
        }
        if (k0 + 64 < K) rows(k0 + 64);
      }
#pragma unroll
      for (int off = P; off < 64; off <<= 1) {
        ax += __shfl_xor(ax, off, 64);
        ay += __shfl_xor(ay, off, 64);
      }
      if (lane < rem) {
        if (BWD) X[U.o + U.o0 + lane] = make_double2(ax, ay);
        else slot[dst] = make_double2(a0.x + a1.x - ax, a0.y + a1.y - ay);
      }
    }
    if (st + 1 < stages) __syncthreads();   // the next stage reads what this one stored
  }
}

// One wave per output row, lanes along the row.
template <bool BWD>
__global__ void __launch_bounds__(256) k_nd1_row(const ND1Row* __restrict__ task, int ntask,
                                                 const double2* __restrict__ fac, const int* __restrict__ bnd,
                                                 const int* __restrict__ push, const double2* __restrict__ g,
                                                 double2* slot, int64_t srows, int nK, double2* X) {
  const int lane = threadIdx.x & 63;
  const int q = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (q >= ntask) return;
  const ND1Row T = task[q];
  double ax = 0, ay = 0;
  double2 m0 = make_double2(0, 0), x0 = m0, a0 = m0, a1 = m0;
  int dst = 0;
  if (BWD) {   // the first boundary gather (index, then value) is the longest chain: start it first
    if (lane < T.n1) {
      m0 = fac[T.m1 + lane];
      x0 = X[bnd[T.bo + lane]];
    }
  } else if (lane == 0) {
    dst = push[T.out];
    a0 = slot[nK + T.out];
    a1 = slot[srows + nK + T.out];
  }
#pragma unroll 4
  for (int k = lane; k < T.n0; k += 64) {
    const double2 m = fac[T.m0 + k], y = front_rhs(g, slot, srows, T.o + k);
    ax += m.x * y.x - m.y * y.y;
    ay += m.x * y.y + m.y * y.x;
  }
  if (BWD) {
    ax -= m0.x * x0.x - m0.y * x0.y;
    ay -= m0.x * x0.y + m0.y * x0.x;
#pragma unroll 4
    for (int b = lane + 64; b < T.n1; b += 64) {
      const double2 m = fac[T.m1 + b], x = X[bnd[T.bo + b]];
      ax -= m.x * x.x - m.y * x.y;
      ay -= m.x * x.y + m.y * x.x;
    }
  }
  for (int sh = 32; sh > 0; sh >>= 1) {
    ax += __shfl_xor(ax, sh, 64);
    ay += __shfl_xor(ay, sh, 64);
  }
  if (lane == 0) {
    if (BWD) X[T.out] = make_double2(ax, ay);
    else slot[dst] = make_double2(a0.x + a1.x - ax, a0.y + a1.y - ay);
  }
}

// ---------------------------------------------------------------------------
// Several columns on the FP64 matrix cores: a workgroup forms 16 outputs of a node
// at all R columns over a range [i0, i1) of the summation (split ranges go to P, added
// by k_nd_reduce), its four waves each a quarter of the range, added through shared
// memory.  Per step of 4 rows a wave loads 16 x 4 entries of the factor block (read
// once in the workgroup) and 4 rows of CT x 16 columns, the next step's loads in flight
// during the 4 CT matrix operations of the present one; a boundary row's index is
// read a step before its values.  Lane l supplies M(l & 15, l >> 4) and
// x(l >> 4, 16 c + (l & 15)), and receives outputs (l >> 4) + 4 v, column l & 15.
// Columns past R repeat column R - 1 and are not stored.
//
// What bounds it: the factor's bytes at few columns (CT = 1: the 164 MB inverse of
// n_K = 3,201 at 5 columns in 44 us, 3.7 TB/s, where the vector ALUs took 237), the
// matrix operations (64 cycles each) at 64 (leaves, backward: 4.7 GFLOP in 107 us);
// before both the loads in flight, which is why the range is cut in four: the sums
// near the leaves are 40 to 200 rows long.  One 64-column solve of the 64x64
// scatterer (n_K = 45,825) takes 422 us; with 32 outputs per workgroup, every sum
// whole in one wave, it took 483.
constexpr int ND_J = ND_TILE;   // outputs per workgroup

typedef double d4 __attribute__((ext_vector_type(4)));

struct NDNodes {
  const int* off;          // [n + 1]
  const int64_t* boff;     // [n + 1] into bnd
  const int* bnd;
  const int64_t* uoff;     // first update row of node t
  const int64_t* mD;       // factor offsets
  const int64_t* mL;
  const int64_t* mLt;
  const double2* fac;
  // each front row has two slots (one per child) at a fixed column stride ld; update
  // row u of a node goes by a plain store to slot row push2[u] (slot k of the parent's
  // interior row, or of its update row nK + a); slot rows no child writes stay zero
  const int* push2;
  const int* child;      // [2 n], -1 where absent
  double2* slot;         // [2][nK + urows][ld]
  int64_t ld, srows;     // column stride, rows per slot (nK + urows)
  int nK;
};

// The sum of the child slots of front row `row` (interior rows [0, nK), update rows after).
__device__ __forceinline__ double2 nd_slots(const NDNodes& nd, bool leaf, int64_t row, int r) {
  if (leaf) return make_double2(0, 0);
  const double2* p = nd.slot + row * nd.ld + r;
  const double2 a = p[0], b = p[nd.srows * nd.ld];
  return make_double2(a.x + b.x, a.y + b.y);
}

__device__ __forceinline__ bool nd_leaf(const NDNodes& nd, int t) {
  return nd.child[2 * t] < 0 && nd.child[2 * t + 1] < 0;
}

// Output j of node t at column r: U = A - sum into t's slot of its parent's row, or X.
template <bool BWD>
__device__ __forceinline__ void nd_finish(const NDNodes& nd, int t, bool leaf, int o, int j, int r, int R, double2 sum,
                                          double2* X) {
  if (BWD) {
    X[((int64_t)o + j) * R + r] = sum;
  } else {
    const int64_t u = nd.uoff[t] + j;
    const double2 a = nd_slots(nd, leaf, nd.nK + u, r);
    nd.slot[(int64_t)nd.push2[u] * nd.ld + r] = make_double2(a.x - sum.x, a.y - sum.y);
  }
}

// Workgroups go to the eight XCDs in turn, each with an L2 of its own: the tasks of
// a node (consecutive in the list) read the same rows of columns, so every XCD takes
// runs of ND_RUN consecutive tasks.  Runs keep the list's order, longest sums first,
// which one range per XCD would not.
constexpr int ND_RUN = 32;
__device__ __forceinline__ int xcd_task(int b, int n) {
  const int block = 8 * ND_RUN, first = b / block * block, at = b - first;
  const int len = min(block, n - first);   // the last block may be short
  const int x = at & 7, q = len >> 3, rem = len & 7;
  return first + x * q + min(x, rem) + (at >> 3);
}

template <int CT, bool BWD>
__global__ void __launch_bounds__(256, 2) k_nd_tile(const int4* __restrict__ task, NDNodes nd,
                                                    const double2* __restrict__ g, double2* X, int R,
                                                    double2* __restrict__ P) {
  __shared__ double2 red[4][3][4][16 * CT];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6, jl = l & 15, kq = l >> 4;
  const int id = xcd_task(blockIdx.x, gridDim.x);
  const int4 tk = task[id];
  const int t = tk.x, j0 = tk.y, i0 = tk.z, i1 = tk.w;
  const int o = nd.off[t], nI = nd.off[t + 1] - o;
  const int64_t bo = nd.boff[t];
  const int nB = int(nd.boff[t + 1] - bo), n_out = BWD ? nI : nB;
  const bool leaf = nd_leaf(nd, t);
  const int q = ((i1 - i0 + 15) / 16) * 4;
  const int ks = i0 + w * q, ke = min(i1, ks + q);
  const int j = min(j0 + jl, n_out - 1);
  const double2* m0 = nd.fac + (BWD ? nd.mD[t] : nd.mL[t]) + (int64_t)nI * j;
  const double2* m1 = nd.fac + nd.mLt[t] + (int64_t)nB * j - nI;
  const int64_t sst = nd.srows * nd.ld;
  int col[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) col[c] = min(16 * c + jl, R - 1);
  // forward: where this lane's output goes and what its children sent there
  int64_t dst = 0;
  double2 a[CT];
  if (!BWD && !P) {
    const int64_t u = nd.uoff[t] + min(j0 + kq + 4 * w, n_out - 1);
    dst = nd.push2[u];
#pragma unroll
    for (int c = 0; c < CT; ++c) a[c] = nd_slots(nd, leaf, nd.nK + u, col[c]);
  }
  d4 cr[CT], ci[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    cr[c] = (d4){0, 0, 0, 0};
    ci[c] = (d4){0, 0, 0, 0};
  }
  // rows past the wave's range read its last row and are multiplied by zero
  auto index = [&](int k0) {
    const int k = min(k0 + kq, ke - 1);
    return BWD && k >= nI ? nd.bnd[bo + k - nI] : o + k;
  };
  auto load = [&](int k0, int row, double2& m, double2 (&x)[CT]) {
    const int k = min(k0 + kq, ke - 1);
    if (!BWD || k < nI) {
      m = m0[k];
#pragma unroll
      for (int c = 0; c < CT; ++c) x[c] = g[(int64_t)row * R + col[c]];
      if (!leaf) {
        const double2* s0 = nd.slot + (int64_t)row * nd.ld;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          const double2 a = s0[col[c]], b = s0[sst + col[c]];
          x[c].x += a.x + b.x;
          x[c].y += a.y + b.y;
        }
      }
    } else {
      const double2 v = m1[k];
      m = make_double2(-v.x, -v.y);
#pragma unroll
      for (int c = 0; c < CT; ++c) x[c] = X[(int64_t)row * R + col[c]];
    }
    if (k0 + kq >= ke) m = make_double2(0, 0);
  };
  if (ks < ke) {
    double2 m, x[CT];
    int row = index(ks);
    load(ks, row, m, x);
    row = index(ks + 4);
    for (int k = ks; k < ke; k += 4) {
      double2 mn = m, xn[CT];
#pragma unroll
      for (int c = 0; c < CT; ++c) xn[c] = x[c];
      if (k + 4 < ke) {   // uniform over the wave
        load(k + 4, row, mn, xn);
        row = index(k + 8);
      }
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        cr[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(m.x, x[c].x, cr[c], 0, 0, 0);
        ci[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(m.x, x[c].y, ci[c], 0, 0, 0);
        cr[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(m.y, -x[c].y, cr[c], 0, 0, 0);
        ci[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(m.y, x[c].x, ci[c], 0, 0, 0);
      }
      m = mn;
#pragma unroll
      for (int c = 0; c < CT; ++c) x[c] = xn[c];
    }
  }
  // wave v finishes outputs (l >> 4) + 4 v: the others hand it theirs
  double2 sum[CT];
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const double2 p = make_double2(cr[c][v], ci[c][v]);
      if (v == w) sum[c] = p;
      else red[v][w < v ? w : w - 1][kq][16 * c + jl] = p;
    }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 3; ++u)
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const double2 p = red[w][u][kq][16 * c + jl];
      sum[c].x += p.x;
      sum[c].y += p.y;
    }
  const int jj = kq + 4 * w;
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int r = 16 * c + jl;
    if (r >= R) continue;
    if (P) P[((int64_t)id * ND_J + jj) * 64 + r] = sum[c];
    else if (j0 + jj < n_out) {
      if (BWD) X[((int64_t)o + j0 + jj) * R + r] = sum[c];
      else nd.slot[dst * nd.ld + r] = make_double2(a[c].x - sum[c].x, a[c].y - sum[c].y);
    }
  }
}

// Adds the S partial tiles of each output tile (tasks q S .. q S + S - 1 share node
// and first output) and finishes the step.
template <bool BWD>
__global__ void __launch_bounds__(256) k_nd_reduce(const int4* __restrict__ task, int ntiles, int S,
                                                   const double2* __restrict__ P, NDNodes nd, double2* __restrict__ X,
                                                   int R) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)ntiles * ND_J * R) return;
  const int r = int(e % R);
  const int jj = int((e / R) % ND_J);
  const int q = int(e / ((int64_t)R * ND_J));
  const int4 tk = task[(int64_t)q * S];
  const int t = tk.x, j = tk.y + jj;
  const int o = nd.off[t];
  const int n_out = BWD ? nd.off[t + 1] - o : int(nd.boff[t + 1] - nd.boff[t]);
  if (j >= n_out) return;
  double2 sum = make_double2(0, 0);
  for (int c = 0; c < S; ++c) {
    const double2 v = P[(((int64_t)q * S + c) * ND_J + jj) * 64 + r];
    sum.x += v.x;
    sum.y += v.y;
  }
  nd_finish<BWD>(nd, t, nd_leaf(nd, t), o, j, r, R, sum, X);
}

template <bool BWD>
void launch_tiles(const int4* task, int ntiles, int S, const NDNodes& nd, const double2* g, double2* X, int R,
                  double2* part, hipStream_t s) {
  const dim3 grid{unsigned(ntiles) * unsigned(S)};
  const int ct = (R + 15) / 16;
  if (ct == 1) hipLaunchKernelGGL((k_nd_tile<1, BWD>), grid, dim3(256), 0, s, task, nd, g, X, R, part);
  else if (ct == 2) hipLaunchKernelGGL((k_nd_tile<2, BWD>), grid, dim3(256), 0, s, task, nd, g, X, R, part);
  else if (ct == 3) hipLaunchKernelGGL((k_nd_tile<3, BWD>), grid, dim3(256), 0, s, task, nd, g, X, R, part);
  else hipLaunchKernelGGL((k_nd_tile<4, BWD>), grid, dim3(256), 0, s, task, nd, g, X, R, part);
  if (S > 1)
    hipLaunchKernelGGL(k_nd_reduce<BWD>, dim3(unsigned((int64_t(ntiles) * ND_J * R + 255) / 256)), dim3(256), 0, s, task,
                       ntiles, S, part, nd, X, R);
}

}  // namespace

void launch_nd_tiles(bool bwd, const int4* task, int ntiles, int S, const NDView& v, const double2* g, double2* X,
                     int R, double2* P, hipStream_t s) {
  if (ntiles == 0) return;
  if (R > v.ld || R > 64) fail(HDP_E_ARG, "nested-dissection sweep: more columns than the slot stride");
  const NDNodes nd{v.off, v.boff, v.bnd, v.uoff, v.mD, v.mL, v.mLt, v.fac, v.push2, v.child, v.slot, v.ld, v.srows, v.nK};
  double2* part = S > 1 ? P : nullptr;
  if (bwd) launch_tiles<true>(task, ntiles, S, nd, g, X, R, part, s);
  else launch_tiles<false>(task, ntiles, S, nd, g, X, R, part, s);
  HIPCHECK(hipGetLastError());
}

void launch_nd1(bool bwd, const ND1Launch& l, const Handle& h, const double2* g, double2* X, hipStream_t s) {
  if (l.groups == 0) return;
  const auto& d = h.d;
  const int64_t srows = int64_t(h.nK) + d.nd_urows;
#define HDP_ND1_ARGS d.nd_fac, d.nd_bnd, d.nd_push2, g, d.nd_slot1, srows, h.nK, X
  if (l.rows) {
    const dim3 grid{unsigned((l.groups + 3) / 4)};
    if (bwd) hipLaunchKernelGGL(k_nd1_row<true>, grid, dim3(256), 0, s, d.nd_r1[1] + l.first, l.groups, HDP_ND1_ARGS);
    else hipLaunchKernelGGL(k_nd1_row<false>, grid, dim3(256), 0, s, d.nd_r1[0] + l.first, l.groups, HDP_ND1_ARGS);
  } else {
    const dim3 grid{unsigned(l.groups)}, block{unsigned(64 * l.waves)};
    if (bwd)
      hipLaunchKernelGGL((k_nd1<true, ND1_P>), grid, block, 0, s, d.nd_u1[1], d.nd_g1[1] + l.first, l.stages,
                         HDP_ND1_ARGS);
    else
      hipLaunchKernelGGL((k_nd1<false, ND1_P>), grid, block, 0, s, d.nd_u1[0], d.nd_g1[0] + l.first, l.stages,
                         HDP_ND1_ARGS);
  }
#undef HDP_ND1_ARGS
  HIPCHECK(hipGetLastError());
}

}  // namespace hdp
