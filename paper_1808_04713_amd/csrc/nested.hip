// One-column sweeps of the nested-dissection coarse factor (gfx950, 64-wide waves).
//
// Node t of the tree owns the coarse unknowns I (nI of them) and couples to the
// ancestor unknowns B (nB).  Forward, deepest first, with Y = g + the children's
// updates on I:  U = A - L Y (A: the children's updates on B), stored into t's slot
// of its parent's rows; backward, root first:  X_I = D Y - L^T X_B.  Every front row
// has two slots, one per child, so the updates are plain stores and a slot row that
// no child writes stays zero from set-up.
//
// What bounds it near the root is the chain record -> operands -> sums -> store of a
// launch, about 4 us for 5 to 30 MB of factor; near the leaves the number of waves,
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
// scatterer (n_K = 71,361): 23 launches and a clearing, 212 us, with a wave per output
// at every depth; 19 launches, 160 us, of which the subtrees' two take 41.
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

}  // namespace

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
