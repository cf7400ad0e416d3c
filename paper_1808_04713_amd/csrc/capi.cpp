// C ABI of the solver: device setup, operator entry points and the GMRES
// driver (paper Sec. 2.3.1 and 2.3.4; GMRES-IR for the mixed-precision path).
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <functional>
#include <map>
#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include "basis.hpp"
#include "internal.hpp"
#include "kernels.hpp"
#include "team.hpp"

struct hdp_handle {
  hdp::Handle h;
};

namespace hdp {

namespace {
thread_local std::string g_err;

int pow2ceil(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

template <class T>
T* dalloc(Handle& h, size_t count) {
  void* p = nullptr;
  if (count == 0) count = 1;
  const size_t bytes = count * sizeof(T);
  if (h.allocator.alloc) {
    p = h.allocator.alloc(bytes, h.allocator.ctx);
    if (!p) fail(HDP_E_NOMEM, "the caller's allocator returned no memory for " + std::to_string(bytes) + " bytes");
    if (reinterpret_cast<uintptr_t>(p) % 256 != 0) {
      h.allocator.free(p, h.allocator.ctx);
      fail(HDP_E_NOMEM, "the caller's allocator returned memory aligned to less than 256 bytes");
    }
  } else if (hipMalloc(&p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    fail(HDP_E_NOMEM, "device allocation of " + std::to_string(bytes) + " bytes failed");
  }
  h.allocations.push_back(p);
  return static_cast<T*>(p);
}

template <class T>
T* upload(Handle& h, const T* v, size_t count) {
  T* p = dalloc<T>(h, count);
  if (count) HIPCHECK(hipMemcpy(p, v, count * sizeof(T), hipMemcpyHostToDevice));
  return p;
}

template <class T>
T* upload(Handle& h, const std::vector<T>& v) {
  return upload(h, v.data(), v.size());
}

std::vector<double2> pack_c(const std::vector<cd>& v) {
  std::vector<double2> o(v.size());
  for (size_t i = 0; i < v.size(); ++i) o[i] = make_double2(v[i].real(), v[i].imag());
  return o;
}

}  // namespace

[[noreturn]] void fail(hdp_status s, const std::string& msg) { throw Error{s, msg}; }

const char* const KF_NAMES[KF_COUNT] = {"slot_apply_F", "slot_apply_P", "coarse_assemble", "coarse_gemv",
                                        "slot_coarse", "row_gather", "gmres_dots", "gmres_update",
                                        "gmres_norm_scale", "fdm_local_solve", "element_coarse_fix",
                                        "gll_sample", "precision_cast", "gmres_givens", "far_field",
                                        "hanging_blocks", "coarse_reduce"};

static hipEvent_t prof_event(Handle& h) {
  if (!h.prof.pool.empty()) {
    hipEvent_t e = h.prof.pool.back();
    h.prof.pool.pop_back();
    return e;
  }
  hipEvent_t e;
  HIPCHECK(hipEventCreate(&e));
  return e;
}

Timed::Timed(Handle& h_, int fam_, double bytes_, double flops_) : h(h_), fam(fam_), bytes(bytes_), flops(flops_) {
  if (!h.prof.on || h.prof.suspended) return;
  a = prof_event(h);
  HIPCHECK(hipEventRecord(a, h.stream));
}

Timed::~Timed() {
  if (!h.prof.on || !a) return;
  hipEvent_t b = prof_event(h);
  if (hipEventRecord(b, h.stream) != hipSuccess) return;
  h.prof.pend.push_back({fam, a, b, bytes, flops});
}

void prof_flush(Handle& h) {
  for (auto& p : h.prof.pend) {
    float ms = 0;
    if (hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
      h.prof.ms[p.fam] += ms;
      h.prof.n[p.fam] += 1;
      h.prof.bytes[p.fam] += p.bytes;
      h.prof.flops[p.fam] += p.flops;
    }
    h.prof.pool.push_back(p.a);
    h.prof.pool.push_back(p.b);
  }
  h.prof.pend.clear();
}

void release_allocations(Handle& h) {
  for (void* p : h.allocations) {
    if (h.allocator.free) h.allocator.free(p, h.allocator.ctx);
    else (void)hipFree(p);
  }
  h.allocations.clear();
}

void check_hip(hipError_t e, const char* what) {
  if (e != hipSuccess) fail(HDP_E_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

// Dense coarse inverse K^-1 (rocSOLVER getrf + getri), row-major n_K x n_K.
static void build_coarse_dense(Handle& h, const std::vector<int64_t>& kidx, const std::vector<double2>& kval) {
  auto& d = h.d;
  size_t nK = size_t(h.nK);
  // the dense coarse inverse is addressed with 32-bit sizes by the factorisation
  // routines: refuse coarse spaces whose square does not fit that range
  if (int64_t(h.nK) * int64_t(h.nK) >= (int64_t(1) << 31))
    fail(HDP_E_UNSUPPORTED, "coarse space too large for the dense coarse inverse (n_K = " +
                                std::to_string(h.nK) + ", n_K^2 >= 2^31)");
  d.Kinv = dalloc<double2>(h, nK * nK);
  HIPCHECK(hipMemsetAsync(d.Kinv, 0, nK * nK * sizeof(double2), h.stream));
  int64_t* didx = upload(h, kidx);
  double2* dval = upload(h, kval);
  launch_dense_scatter(didx, dval, int64_t(kidx.size()), d.Kinv, h.stream);
  rocblas_handle rb = static_cast<rocblas_handle>(h.rocblas);
  int* ipiv = dalloc<int>(h, nK);
  int* info = dalloc<int>(h, 1);
  rocblas_status st = rocsolver_zgetrf(rb, h.nK, h.nK, (rocblas_double_complex*)d.Kinv, h.nK, ipiv, info);
  int hinfo = 0;
  if (st == rocblas_status_success) {
    HIPCHECK(hipMemcpyAsync(&hinfo, info, sizeof(int), hipMemcpyDeviceToHost, h.stream));
    HIPCHECK(hipStreamSynchronize(h.stream));
  }
  if (st == rocblas_status_success && hinfo == 0)
    st = rocsolver_zgetri(rb, h.nK, (rocblas_double_complex*)d.Kinv, h.nK, ipiv, info);
  if (st == rocblas_status_success && hinfo == 0) {
    HIPCHECK(hipMemcpyAsync(&hinfo, info, sizeof(int), hipMemcpyDeviceToHost, h.stream));
    HIPCHECK(hipStreamSynchronize(h.stream));
  }
  if (st != rocblas_status_success) fail(HDP_E_DEVICE, "rocsolver failed on the coarse matrix");
  if (hinfo != 0) fail(HDP_E_COARSE, "coarse matrix K is singular");
  h.coarse_mode = 0;
  h.coarse_bytes = 16.0 * double(nK) * double(nK);
  h.coarse_flops = 8.0 * double(nK) * double(nK);
  // upper tiles for the one-RHS apply: each unique entry of the symmetric
  // inverse read once
  const int ts = sym_tile_size();
  h.sym_nt = int((nK + ts - 1) / ts);
  h.sym_ntiles = h.sym_nt * (h.sym_nt + 1) / 2;
  std::vector<int2> tij;
  tij.reserve(h.sym_ntiles);
  for (int I = 0; I < h.sym_nt; ++I)
    for (int J = I; J < h.sym_nt; ++J) tij.push_back(make_int2(I, J));
  d.sym_tij = upload(h, tij);
  d.Ksym = dalloc<double2>(h, size_t(h.sym_ntiles) * ts * ts);
  d.sym_part = dalloc<double2>(h, size_t(h.sym_nt) * h.sym_nt * ts);
  launch_pack_sym_tiles(h, h.stream);
  h.coarse_bytes1 = 16.0 * double(nK) * double(nK + 1) / 2;
  // several columns: w = K^-T g by the nested-dissection tile kernels, the inverse
  // taken as the diagonal block of a one-node tree (no boundary, no children);
  // each output tile's sum split so that about 1024 workgroups run
  if (pow2ceil(h.max_rhs) >= 4) {
    const int ntiles = int((nK + ND_TILE - 1) / ND_TILE);
    const int S = std::max(1, std::min((1024 + ntiles - 1) / ntiles, int(nK + 63) / 64));
    const int chunk = int((nK + S - 1) / S);
    std::vector<int4> tasks;
    for (int j = 0; j < int(nK); j += ND_TILE)
      for (int c = 0; c < S; ++c)
        tasks.push_back(make_int4(0, j, std::min(int(nK), c * chunk), std::min(int(nK), (c + 1) * chunk)));
    d.dn_tasks = upload(h, tasks);
    d.dn_off = upload(h, std::vector<int>{0, int(nK)});
    d.dn_boff = upload(h, std::vector<int64_t>{0, 0});
    d.dn_zero64 = upload(h, std::vector<int64_t>{0});
    d.dn_int = upload(h, std::vector<int>{-1, -1, 0});
    h.dn_ntiles = ntiles;
    h.dn_S = S;
    if (S > 1) d.dn_P = dalloc<double2>(h, size_t(ntiles) * S * ND_TILE * 64);
  }
}

// w = K^-T g at several columns with the tile kernels (see build_coarse_dense).
static void coarse_solve_dense_tiles(Handle& h, const double2* g, double2* w, int R) {
  auto& d = h.d;
  NDView v;
  v.off = d.dn_off; v.boff = d.dn_boff; v.bnd = d.dn_int + 2; v.uoff = d.dn_zero64;
  v.mD = d.dn_zero64; v.mL = d.dn_zero64; v.mLt = d.dn_zero64; v.fac = d.Kinv;
  v.push2 = d.dn_int + 2; v.child = d.dn_int; v.slot = nullptr; v.ld = pow2ceil(h.max_rhs); v.srows = 0; v.nK = h.nK;
  launch_nd_tiles(true, d.dn_tasks, h.dn_ntiles, h.dn_S, v, g, w, R, d.dn_P, h.stream);
}

// Nested-dissection factor: assembled on the host (coarse_nd.cpp), uploaded
// with its per-depth front-assembly entries and row tasks.
static void build_coarse_nd(Handle& h, const std::vector<int64_t>& kidx, const std::vector<double2>& kval,
                            Team& team) {
  auto& d = h.d;
  NDHost f;
  nd_factor(h, kidx, kval, f, &team);
  d.nd_off = upload(h, h.nd_off);
  d.nd_boff = upload(h, h.nd_boff);
  d.nd_bnd = upload(h, h.nd_bnd);
  d.nd_uoff = upload(h, f.uoff);
  d.nd_mD = upload(h, f.mD);
  d.nd_mL = upload(h, f.mL);
  d.nd_mLt = upload(h, f.mLt);
  for (int bwd = 0; bwd < 2; ++bwd) {
    ND1Plan p;
    nd_units(h, f, bwd != 0, p);   // (may transpose blocks of the factor)
    d.nd_u1[bwd] = upload(h, p.units);
    d.nd_r1[bwd] = upload(h, p.rows);
    d.nd_g1[bwd] = upload(h, p.gptr);
    h.nd_l1[bwd] = p.launches;
  }
  d.nd_fac = upload(h, static_cast<const double2*>(f.fac.data()), f.fac.size());
  const size_t Rp = size_t(pow2ceil(h.max_rhs));
  {
    // task lists and partial tiles sized for every split the autotuner may try
    size_t nf = f.tRf.size(), nb = f.tRb.size();
    int64_t most = f.part_tasks;
    if (Rp > 1)
      for (int target : ND_SPLITS) {
        NDHost g;
        nd_tasks(h, g, target);
        nf = std::max(nf, g.tRf.size());
        nb = std::max(nb, g.tRb.size());
        most = std::max(most, g.part_tasks);
      }
    d.nd_tRf = dalloc<int4>(h, std::max<size_t>(1, nf));
    d.nd_tRb = dalloc<int4>(h, std::max<size_t>(1, nb));
    h.nd_tR_cap[0] = nf;
    h.nd_tR_cap[1] = nb;
    if (!f.tRf.empty()) HIPCHECK(hipMemcpy(d.nd_tRf, f.tRf.data(), f.tRf.size() * sizeof(int4), hipMemcpyHostToDevice));
    if (!f.tRb.empty()) HIPCHECK(hipMemcpy(d.nd_tRb, f.tRb.data(), f.tRb.size() * sizeof(int4), hipMemcpyHostToDevice));
    h.nd_P_tasks = Rp > 1 ? most : 0;
    if (Rp > 1 && most > 0) d.nd_P = dalloc<double2>(h, size_t(most) * ND_TILE * 64);
  }
  d.nd_urows = f.urows;
  // the child slots, cleared once here (a slot row is either rewritten by every
  // solve or never): one column's, and those of several at their own stride
  d.nd_push2 = upload(h, f.push2);
  d.nd_slot1 = dalloc<double2>(h, 2 * size_t(h.nK + f.urows));
  HIPCHECK(hipMemsetAsync(d.nd_slot1, 0, 2 * size_t(h.nK + f.urows) * sizeof(double2), h.stream));
  if (Rp > 1) {
    d.nd_ld = int64_t(Rp);
    const size_t ns = 2 * size_t(h.nK + f.urows) * Rp;
    d.nd_slot = dalloc<double2>(h, ns);
    HIPCHECK(hipMemsetAsync(d.nd_slot, 0, ns * sizeof(double2), h.stream));
    d.nd_childv = upload(h, h.nd_child);
  }
  h.nd_levels = f.levels;
  h.coarse_mode = 2;
  h.coarse_bytes = 16.0 * double(f.fac.size());
  h.coarse_flops = f.flops_per_col;
  // several columns: the depths above D as one dense block of at most ND_TOP_MAX
  // unknowns (D >= 2, at least one depth below it).  Once every node deeper than
  // D - 1 is eliminated, a top unknown's right-hand side is g plus what those
  // nodes pushed into the fronts of depth D - 1: the child slots of its own row
  // there and of those fronts' update rows for it.  The block itself is filled
  // at the end of set-up (build_nd_top).
  const int nn = int(h.nd_off.size()) - 1, maxd = int(h.nd_levels.size()) - 1;
  if (Rp > 1 && maxd >= 2) {
    std::vector<int64_t> above(maxd + 2, 0);   // unknowns at depths < d
    for (int t = 0; t < nn; ++t) above[h.nd_depth[t] + 1] += h.nd_off[t + 1] - h.nd_off[t];
    for (int q = 1; q <= maxd + 1; ++q) above[q] += above[q - 1];
    int D = 0;
    for (int q = 2; q <= maxd; ++q)
      if (above[q] <= ND_TOP_MAX) D = q;
    if (D >= 2) {
      std::vector<int> tops;
      for (int t = 0; t < nn; ++t)
        if (h.nd_depth[t] < D)
          for (int x = h.nd_off[t]; x < h.nd_off[t + 1]; ++x) tops.push_back(x);
      std::sort(tops.begin(), tops.end());
      std::vector<std::vector<int>> rows(tops.size());
      auto pos = [&](int x) { return int(std::lower_bound(tops.begin(), tops.end(), x) - tops.begin()); };
      for (int t = 0; t < nn; ++t) {
        if (h.nd_depth[t] != D - 1) continue;
        for (int x = h.nd_off[t]; x < h.nd_off[t + 1]; ++x) rows[pos(x)].push_back(x);
        for (int64_t b = h.nd_boff[t]; b < h.nd_boff[t + 1]; ++b)
          rows[pos(h.nd_bnd[b])].push_back(int(h.nK + f.uoff[t] + (b - h.nd_boff[t])));
      }
      std::vector<int64_t> gptr(tops.size() + 1, 0);
      std::vector<int> grow;
      for (size_t i = 0; i < tops.size(); ++i) {
        grow.insert(grow.end(), rows[i].begin(), rows[i].end());
        gptr[i + 1] = int64_t(grow.size());
      }
      d.nd_top_idx = upload(h, tops);
      d.nd_top_gptr = upload(h, gptr);
      d.nd_top_grow = upload(h, grow.empty() ? std::vector<int>{0} : grow);
      h.nd_top_host = tops;
      h.nd_top_depth = D;
    }
  }
}

// Re-cut the several-column tasks for another split target (the factor and the
// one-column tasks do not depend on it).
static void set_nd_split(Handle& h, int target) {
  NDHost g;
  nd_tasks(h, g, target);
  if (g.part_tasks > h.nd_P_tasks || g.tRf.size() > h.nd_tR_cap[0] || g.tRb.size() > h.nd_tR_cap[1])
    fail(HDP_E_DEVICE, "nested-dissection split beyond its task or partial-tile buffers");
  auto put = [&](int4* dst, const std::vector<int4>& src) {
    if (!src.empty())
      HIPCHECK(hipMemcpyAsync(dst, src.data(), src.size() * sizeof(int4), hipMemcpyHostToDevice, h.stream));
  };
  put(h.d.nd_tRf, g.tRf);
  put(h.d.nd_tRb, g.tRb);
  HIPCHECK(hipStreamSynchronize(h.stream));
  h.nd_levels = g.levels;
  h.nd_split = target;
}

static void coarse_solve_nd(Handle& h, const double2* g, double2* w, int R) {
  auto& d = h.d;
  NDView v;
  v.off = d.nd_off; v.boff = d.nd_boff; v.bnd = d.nd_bnd; v.uoff = d.nd_uoff;
  v.mD = d.nd_mD; v.mL = d.nd_mL; v.mLt = d.nd_mLt; v.fac = d.nd_fac;
  const int nd = int(h.nd_levels.size());
  if (R == 1) {
    for (int bwd = 0; bwd < 2; ++bwd)
      for (const ND1Launch& l : h.nd_l1[bwd]) launch_nd1(bwd != 0, l, h, g, w, h.stream);
    return;
  }
  v.push2 = d.nd_push2; v.child = d.nd_childv; v.slot = d.nd_slot; v.ld = d.nd_ld;
  v.srows = int64_t(h.nK) + d.nd_urows; v.nK = h.nK;
  // with the dense top block the depths above nd_top_depth are one product
  const int top = h.nd_top_n > 0 ? h.nd_top_depth : 0;
  for (int L = nd - 1; L >= top; --L) {   // leaves first
    const NDLevel& lv = h.nd_levels[L];
    launch_nd_tiles(false, d.nd_tRf + lv.fR, lv.nfR, lv.Sf, v, g, w, R, d.nd_P, h.stream);
  }
  if (top > 0) {
    launch_nd_top_gather(h.nd_top_n, d.nd_top_idx, d.nd_top_gptr, d.nd_top_grow, g, d.nd_slot, d.nd_ld,
                         v.srows * d.nd_ld, d.nd_top_r, R, h.stream);
    NDView tv;
    tv.off = d.nd_top_off; tv.boff = d.nd_top_boff; tv.bnd = d.nd_top_int + 2; tv.uoff = d.nd_top_zero64;
    tv.mD = d.nd_top_zero64; tv.mL = d.nd_top_zero64; tv.mLt = d.nd_top_zero64;
    tv.fac = d.nd_top_inv; tv.push2 = d.nd_top_int + 2; tv.child = d.nd_top_int; tv.slot = nullptr;
    tv.ld = d.nd_ld; tv.srows = 0; tv.nK = h.nd_top_n;
    launch_nd_tiles(true, d.nd_top_tasks, h.nd_top_ntiles, h.nd_top_S, tv, d.nd_top_r, d.nd_top_x, R, d.nd_top_P,
                    h.stream);
    launch_nd_top_scatter(h.nd_top_n, d.nd_top_idx, d.nd_top_x, w, R, h.stream);
  }
  for (int L = top; L < nd; ++L) {   // root first
    const NDLevel& lv = h.nd_levels[L];
    launch_nd_tiles(true, d.nd_tRb + lv.bR, lv.nbR, lv.Sb, v, g, w, R, d.nd_P, h.stream);
  }
}

void coarse_solve(Handle& h, const double2* g, double2* w, int R);

// The dense top block of the nested-dissection sweeps at several columns: the
// rows of K^-1 at the top unknowns (the inverse of their Schur complement once
// the deeper nodes are eliminated), from the factor's own solves of the unit
// vectors at those unknowns; then a check of the sweeps that use it against the
// assembled K, which switches the block off if it fails.
static void build_nd_top(Handle& h, const std::vector<int64_t>& kidx, const std::vector<double2>& kval) {
  auto& d = h.d;
  const int n = int(h.nd_top_host.size());
  const int Rp = pow2ceil(h.max_rhs);
  const int64_t nK = h.nK;
  if (n == 0 || Rp < 2) return;
  d.nd_top_inv = dalloc<double2>(h, size_t(n) * n);
  d.nd_top_r = dalloc<double2>(h, size_t(n) * Rp);
  d.nd_top_x = dalloc<double2>(h, size_t(n) * Rp);
  int64_t* uidx = dalloc<int64_t>(h, Rp);
  double2* uval = dalloc<double2>(h, Rp);
  std::vector<int64_t> hidx(Rp);
  const std::vector<double2> ones(Rp, make_double2(1.0, 0.0));
  HIPCHECK(hipMemcpyAsync(uval, ones.data(), Rp * sizeof(double2), hipMemcpyHostToDevice, h.stream));
  for (int k0 = 0; k0 < n; k0 += Rp) {
    const int cols = std::min(Rp, n - k0);
    for (int c = 0; c < cols; ++c) hidx[c] = int64_t(h.nd_top_host[k0 + c]) * Rp + c;
    HIPCHECK(hipMemcpyAsync(uidx, hidx.data(), cols * sizeof(int64_t), hipMemcpyHostToDevice, h.stream));
    launch_fill_zero(d.gK, nK * Rp, h.stream);
    launch_dense_scatter(uidx, uval, cols, d.gK, h.stream);
    coarse_solve(h, d.gK, d.wK, Rp);
    launch_nd_top_collect(n, d.nd_top_idx, d.wK, Rp, k0, cols, d.nd_top_inv, h.stream);
    HIPCHECK(hipStreamSynchronize(h.stream));   // hidx is rewritten by the next batch
  }
  // each output tile's sum split so that about 1024 workgroups run
  const int ntiles = (n + ND_TILE - 1) / ND_TILE;
  const int S = std::max(1, std::min((1024 + ntiles - 1) / ntiles, (n + 63) / 64));
  const int chunk = (n + S - 1) / S;
  std::vector<int4> tasks;
  for (int j = 0; j < n; j += ND_TILE)
    for (int c = 0; c < S; ++c) tasks.push_back(make_int4(0, j, std::min(n, c * chunk), std::min(n, (c + 1) * chunk)));
  d.nd_top_tasks = upload(h, tasks);
  d.nd_top_off = upload(h, std::vector<int>{0, n});
  d.nd_top_boff = upload(h, std::vector<int64_t>{0, 0});
  d.nd_top_zero64 = upload(h, std::vector<int64_t>{0});
  d.nd_top_int = upload(h, std::vector<int>{-1, -1, 0});
  if (S > 1) d.nd_top_P = dalloc<double2>(h, size_t(ntiles) * S * ND_TILE * 64);
  h.nd_top_ntiles = ntiles;
  h.nd_top_S = S;
  h.nd_top_n = n;
  // check: two pseudo-random columns through the sweeps with the block
  std::vector<double2> b(size_t(nK) * Rp, make_double2(0, 0)), x(size_t(nK) * Rp);
  uint64_t state = 0x2545F4914F6CDD1Dull;
  auto next = [&]() {
    state = state * 6364136223846793005ull + 1442695040888963407ull;
    return double(state >> 11) * (2.0 / 9007199254740992.0) - 1.0;
  };
  const int nc = std::min(Rp, 2);
  for (int64_t i = 0; i < nK; ++i)
    for (int c = 0; c < nc; ++c) b[i * Rp + c] = make_double2(next(), next());
  HIPCHECK(hipMemcpyAsync(d.gK, b.data(), b.size() * sizeof(double2), hipMemcpyHostToDevice, h.stream));
  coarse_solve(h, d.gK, d.wK, Rp);
  HIPCHECK(hipMemcpyAsync(x.data(), d.wK, x.size() * sizeof(double2), hipMemcpyDeviceToHost, h.stream));
  HIPCHECK(hipStreamSynchronize(h.stream));
  double worst = 0;
  for (int c = 0; c < nc; ++c) {
    std::vector<cd> r(nK);
    for (int64_t i = 0; i < nK; ++i) r[i] = -cd(b[i * Rp + c].x, b[i * Rp + c].y);
    for (size_t t = 0; t < kidx.size(); ++t) {
      const int64_t i = kidx[t] % nK, j = kidx[t] / nK;
      r[i] += cd(kval[t].x, kval[t].y) * cd(x[j * Rp + c].x, x[j * Rp + c].y);
    }
    double rn = 0, bn = 0;
    for (int64_t i = 0; i < nK; ++i) {
      rn += std::norm(r[i]);
      bn += b[i * Rp + c].x * b[i * Rp + c].x + b[i * Rp + c].y * b[i * Rp + c].y;
    }
    worst = std::max(worst, std::sqrt(rn / bn));
  }
  h.nd_top_check = worst;
  if (!(worst <= std::max(1e-10, 10 * h.coarse_check))) h.nd_top_n = 0;
}

void coarse_solve(Handle& h, const double2* g, double2* w, int R);

// ||K x - b|| / ||b|| for x from the coarse solve of a fixed pseudo-random b,
// K applied on the host from its assembled entries.
static double coarse_residual(Handle& h, const std::vector<int64_t>& kidx, const std::vector<double2>& kval) {
  const int64_t nK = h.nK;
  std::vector<double2> b(nK), x(nK);
  uint64_t state = 0x9E3779B97F4A7C15ull;
  auto next = [&]() {
    state = state * 6364136223846793005ull + 1442695040888963407ull;
    return double(state >> 11) * (2.0 / 9007199254740992.0) - 1.0;
  };
  for (auto& v : b) { v.x = next(); v.y = next(); }
  HIPCHECK(hipMemcpyAsync(h.d.gK, b.data(), nK * sizeof(double2), hipMemcpyHostToDevice, h.stream));
  coarse_solve(h, h.d.gK, h.d.wK, 1);
  HIPCHECK(hipMemcpyAsync(x.data(), h.d.wK, nK * sizeof(double2), hipMemcpyDeviceToHost, h.stream));
  HIPCHECK(hipStreamSynchronize(h.stream));
  std::vector<cd> r(nK);
  for (int64_t i = 0; i < nK; ++i) r[i] = -cd(b[i].x, b[i].y);
  for (size_t t = 0; t < kidx.size(); ++t) {
    int64_t i = kidx[t] % nK, j = kidx[t] / nK;
    r[i] += cd(kval[t].x, kval[t].y) * cd(x[j].x, x[j].y);
  }
  double rn = 0, bn = 0;
  for (int64_t i = 0; i < nK; ++i) { rn += std::norm(r[i]); bn += b[i].x * b[i].x + b[i].y * b[i].y; }
  return std::sqrt(rn / bn);
}

void build_device(Handle& h, Team& team) {
  auto& d = h.d;
  int E = h.E;
  d.elem_cls = upload(h, h.cls);
  d.dof_off = upload(h, h.dof_off);
  d.row_slot = upload(h, h.row_slot);
  d.row_coef = upload(h, h.row_coef);
  d.row_xinv = upload(h, h.row_xinv);
  d.slot_row = upload(h, h.slot_row);
  d.slot_coef = upload(h, h.slot_coef);
  d.t_ptr = upload(h, h.t_ptr);
  d.t_dof = upload(h, h.t_dof);
  d.t_coef = upload(h, h.t_coef);
  {
    std::vector<int> ip(size_t(h.ncm) + 1), id(h.ncm);
    for (int i = 0; i <= h.ncm; ++i) ip[i] = i;
    for (int i = 0; i < h.ncm; ++i) id[i] = i;
    d.id_ptr = upload(h, ip);
    d.id_dof = upload(h, id);
    d.id_coef = upload(h, std::vector<double>(h.ncm, -1.0));
  }
  d.cdof_ptr = upload(h, h.cdof_ptr);
  d.cdof_list = upload(h, h.cdof_list);
  d.cdof_coef = upload(h, h.cdof_coef);
  d.c2_ptr = upload(h, h.c2_ptr);
  d.c2_dof = upload(h, h.c2_dof);
  d.c2_coef = upload(h, h.c2_coef);
  d.c2t_ptr = upload(h, h.c2t_ptr);
  d.c2t_row = upload(h, h.c2t_row);
  d.c2t_coef = upload(h, h.c2t_coef);
  if (h.nh > 0) {
    std::vector<int> blk(h.nh);
    for (size_t b = 0; b + 1 < h.hb_off.size(); ++b)
      for (int i = h.hb_off[b]; i < h.hb_off[b + 1]; ++i) blk[i] = int(b);
    std::vector<int> of(h.nlam, -1);   // dual row -> its number among the blocks' rows
    for (int i = 0; i < h.nh; ++i) of[h.hb_rows[i]] = i;
    d.hb_of = upload(h, of);
    d.hb_off = upload(h, h.hb_off);
    d.hb_rows = upload(h, h.hb_rows);
    d.hb_blk = upload(h, blk);
    d.hb_moff = upload(h, h.hb_moff);
    d.hb_xinv = upload(h, h.hb_xinv);
    d.hb_y2 = upload(h, h.hb_y2);
  }
  std::vector<int64_t> slot_pos(h.nslots), cm_pos(h.ncm);
  for (int e = 0; e < E; ++e) {
    for (int s = h.slot_off[e]; s < h.slot_off[e + 1]; ++s) slot_pos[s] = h.dof_off[e] + h.slot_mode[s];
    for (int i = h.cm_off[e]; i < h.cm_off[e + 1]; ++i) cm_pos[i] = h.dof_off[e] + h.cm_mode[i];
  }
  d.slot_pos = upload(h, slot_pos);
  d.cm_pos = upload(h, cm_pos);
  // class tables and operators
  int NC = int(h.classes.size());
  std::vector<int> cn(NC);
  std::vector<int64_t> o_op1(NC), o_phi(NC), o_se(NC);
  std::vector<double2> op1, phi, Dinv, Kc;
  std::vector<double2> se;
  std::vector<double> mats, V;
  std::vector<int> gam, rmod;
  std::vector<SepClass> sc(NC);
  for (int c = 0; c < NC; ++c) {
    const ElemClass& C = h.classes[c];
    cn[c] = C.n;
    o_op1[c] = op1.size(); o_phi[c] = phi.size(); o_se[c] = se.size();
    for (auto& v : C.Op1.a) op1.push_back(make_double2(v.real(), v.imag()));
    for (auto& v : C.Phi.a) phi.push_back(make_double2(v.real(), v.imag()));
    for (auto& v : C.Se.a) se.push_back(make_double2(v.real(), v.imag()));
    // a real pencil (no impedance or layer terms along its direction) gives an
    // exactly real eigenbasis; each by column
    int64_t at[2];
    int real[2];
    for (int dir = 0; dir < 2; ++dir) {
      const MatC& Eb = dir ? C.Ey : C.Ex;
      at[dir] = int64_t(mats.size());
      real[dir] = 1;
      for (auto& v : Eb.a)
        if (v.imag() != 0.0) real[dir] = 0;
      for (auto& v : Eb.a) {
        mats.push_back(v.real());
        if (!real[dir]) mats.push_back(v.imag());
      }
    }
    sc[c] = SepClass{at[0], at[1], int64_t(Dinv.size()), int64_t(Kc.size()), int64_t(V.size()), C.n, C.nr,
                     C.m, int(rmod.size()), int(gam.size()), real[0], real[1], sep_len(C.n)};
    for (auto& v : C.Dg) { cd iv = 1.0 / v; Dinv.push_back(make_double2(iv.real(), iv.imag())); }
    for (auto& v : C.Kc.a) Kc.push_back(make_double2(v.real(), v.imag()));
    std::vector<double> t = gll_nodes(C.n), row(C.n);
    for (int i = 0; i < C.n; ++i) {
      vertex_basis(C.n, t[i], row.data());
      V.insert(V.end(), row.begin(), row.end());
    }
    gam.insert(gam.end(), C.Gam.begin(), C.Gam.end());
    rmod.insert(rmod.end(), C.R.begin(), C.R.end());
  }
  d.cls_n = upload(h, cn);
  {
    // flattened per-block and per-slot tables of the slot kernels
    std::vector<SlotBlock> blk(E);
    for (int b = 0; b < E; ++b) {
      const int e = h.order[b], c = h.cls[e];
      blk[b] = SlotBlock{o_op1[c], o_se[c], o_phi[c], e, c, h.slot_off[e], h.cm_off[e], h.classes[c].m, h.classes[c].nr, 0, 0};
    }
    d.slot_blk = upload(h, blk);
    const size_t ns = h.slot_row.size();
    std::vector<SlotIn> in0(ns), in1(ns), in2(ns);
    for (size_t sl = 0; sl < ns; ++sl) {
      const int row = h.slot_row[sl];
      const double f = h.slot_coef[sl], fx = f * h.row_xinv[row];
      in0[sl] = SlotIn{f, 0.0, row, -1};
      in1[sl] = SlotIn{fx, 0.0, row, -1};
      in2[sl] = SlotIn{h.row_coef[2 * size_t(row)] * fx, h.row_coef[2 * size_t(row) + 1] * fx,
                       h.row_slot[2 * size_t(row)], h.row_slot[2 * size_t(row) + 1]};
    }
    d.slot_in[0] = upload(h, in0);
    d.slot_in[1] = upload(h, in1);
    d.slot_in[2] = upload(h, in2);
    // row scatter of the preconditioner output: row scaling times the row's
    // coefficient for this slot
    std::vector<SlotOut> out(ns);
    for (size_t sl = 0; sl < ns; ++sl) {
      const int row = h.slot_row[sl];
      double c = 0;
      for (int t = 0; t < 2; ++t)
        if (h.row_slot[2 * size_t(row) + t] == int(sl)) c = h.row_coef[2 * size_t(row) + t];
      out[sl] = SlotOut{h.row_xinv[row] * c, row, 0};
    }
    d.slot_out = upload(h, out);
  }
  {
    // separable element solves: records, and per bucket of classes of one kernel
    // the items for every number of elements per workgroup
    std::vector<SepElem> el(E);
    for (int b = 0; b < E; ++b) el[b] = SepElem{h.dof_off[h.order[b]], h.cm_off[h.order[b]], h.slot_off[h.order[b]]};
    // kernel -> (first position in order, class), the classes with complex
    // eigenbases (twice the products, or more) first so that none is left for the tail
    std::map<int, std::vector<std::pair<int, int>>> runs;
    for (int b = 0; b < E; ++b)
      if (b == 0 || h.cls[h.order[b]] != h.cls[h.order[b - 1]]) {
        const int c = h.cls[h.order[b]];
        runs[sep_len(h.classes[c].n)].push_back({b, c});
      }
    std::vector<SepItem> items;
    h.sep_buckets.clear();
    for (auto& kv : runs) {
      std::stable_sort(kv.second.begin(), kv.second.end(), [&](const std::pair<int, int>& a, const std::pair<int, int>& b) {
        return sc[a.second].rx + sc[a.second].ry < sc[b.second].rx + sc[b.second].ry;
      });
      SepBucket bk;
      bk.N = kv.first;
      for (int eg = 1; eg <= SEP_EG_MAX; ++eg) {
        bk.first[eg - 1] = int(items.size());
        for (auto& rn : kv.second) {
          const ElemClass& C = h.classes[rn.second];
          bk.n = std::max(bk.n, C.n);
          bk.nr = std::max(bk.nr, C.nr);
          const int ne = int(C.elems.size());
          for (int q = 0; q < ne; q += eg) items.push_back(SepItem{sc[rn.second], rn.first + q, std::min(eg, ne - q)});
        }
        bk.count[eg - 1] = int(items.size()) - bk.first[eg - 1];
      }
      h.sep_buckets.push_back(bk);
    }
    // the same of every kernel of up to SEP_MIX_N modes together, longest first
    h.sep_mix = SepBucket{};
    int kernels = 0;
    for (auto& kv : runs) kernels += kv.first <= SEP_MIX_N;
    if (kernels > 1) {
      SepBucket& bk = h.sep_mix;
      bk.first[0] = int(items.size());
      for (auto b = h.sep_buckets.rbegin(); b != h.sep_buckets.rend(); ++b) {
        if (b->N > SEP_MIX_N) continue;
        bk.n = std::max(bk.n, b->n);
        bk.nr = std::max(bk.nr, b->nr);
        for (int q = 0; q < b->count[0]; ++q) items.push_back(SepItem(items[b->first[0] + q]));
        bk.count[0] += b->count[0];
      }
    }
    d.sep_elem = upload(h, el);
    d.sep_items = upload(h, items);
  }
  d.gam_modes = upload(h, gam);
  d.r_modes = upload(h, rmod);
  // plane-wave load tables
  {
    std::vector<int> cq(NC);
    std::vector<int64_t> cqo(NC);
    std::vector<double> qx, qw, qN;
    int64_t acc = 0;
    for (int c = 0; c < NC; ++c) {
      const ElemClass& C = h.classes[c];
      const auto& xs = h.quad_x.at(C.n);
      const auto& ws = h.quad_w.at(C.n);
      const auto& Ns = h.quad_N.at(C.n);
      cq[c] = int(xs.size());
      cqo[c] = acc;
      acc += int64_t(xs.size());
      qx.insert(qx.end(), xs.begin(), xs.end());
      qw.insert(qw.end(), ws.begin(), ws.end());
      for (size_t t = 0; t < xs.size(); ++t)
        for (int m = 0; m < 64; ++m) qN.push_back(m < C.n ? Ns[t * C.n + m] : 0.0);
    }
    d.cls_q = upload(h, cq);
    d.cls_qoff = upload(h, cqo);
    d.qx = upload(h, qx);
    d.qw = upload(h, qw);
    d.qN = upload(h, qN);
    d.ox = upload(h, h.ox);
    d.oy = upload(h, h.oy);
    d.hx = upload(h, h.hx);
    d.hy = upload(h, h.hy);
    d.eps = upload(h, h.eps);
    d.bmask = upload(h, h.bmask);
    d.angles = dalloc<double>(h, size_t(h.max_rhs));
    std::vector<double> Ms;
    std::vector<int64_t> Mo(NC);
    for (int c = 0; c < NC; ++c) {
      Mo[c] = int64_t(Ms.size());
      MatD M = mass_vertex(h.classes[c].n);
      Ms.insert(Ms.end(), M.a.begin(), M.a.end());
    }
    d.cls_M = upload(h, Ms);
    d.cls_Moff = upload(h, Mo);
  }
  d.op1 = upload(h, op1); d.phi = upload(h, phi); d.se = upload(h, se);
  std::vector<float2> op1f(op1.size()), phif(phi.size());
  std::vector<float2> sef(se.size());
  for (size_t i = 0; i < op1.size(); ++i) op1f[i] = make_float2(float(op1[i].x), float(op1[i].y));
  for (size_t i = 0; i < phi.size(); ++i) phif[i] = make_float2(float(phi[i].x), float(phi[i].y));
  for (size_t i = 0; i < se.size(); ++i) sef[i] = make_float2(float(se[i].x), float(se[i].y));
  d.op1_f = upload(h, op1f); d.phi_f = upload(h, phif); d.se_f = upload(h, sef);
  if (h.pml) {   // s_x s_y per element: the layers' factor on the mass term (adjoint gradient)
    std::vector<double2> mf(E);
    for (int e = 0; e < E; ++e) {
      const cd f = cd(1.0, h.sigx[e] / h.k) * cd(1.0, h.sigy[e] / h.k);
      mf[e] = make_double2(f.real(), f.imag());
    }
    d.mass_fac = upload(h, mf);
  }
  d.sep_mat = upload(h, mats);
  d.sep_gll = upload(h, V);
  d.Dinv = upload(h, Dinv);
  d.Kc = upload(h, Kc);
  std::vector<int64_t> kidx;
  std::vector<double2> kval;
  coarse_coo(h, kidx, kval, &team);
  size_t nK = size_t(h.nK);
  h.coarse_band_bytes = coarse_band_bytes(h.nK, kidx);
  rocblas_handle rb;
  if (rocblas_create_handle(&rb) != rocblas_status_success) fail(HDP_E_DEVICE, "rocblas_create_handle");
  rocblas_set_stream(rb, h.stream);
  h.rocblas = rb;   // rocSOLVER's factorisation of the dense coarse inverse at set-up
  // the coarse factor chosen at set-up: dense inverse (0) or nested dissection (2)
  const auto tk = std::chrono::steady_clock::now();
  if (h.coarse_mode == 2) build_coarse_nd(h, kidx, kval, team);
  else build_coarse_dense(h, kidx, kval);
  h.setup_coarse_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - tk).count();
  // work buffers sized for the largest RHS batch (padded to a power of two)
  size_t Rp = size_t(pow2ceil(h.max_rhs));
  size_t nl = size_t(h.nlam);
  d.slotA = dalloc<double2>(h, size_t(h.nslots) * Rp);
  d.slotB = dalloc<double2>(h, size_t(h.nslots) * Rp);
  d.slotA_f = dalloc<float2>(h, size_t(h.nslots) * Rp);
  d.slotB_f = dalloc<float2>(h, size_t(h.nslots) * Rp);
  d.cmA = dalloc<double2>(h, size_t(h.ncm) * Rp);
  d.cmX = dalloc<double2>(h, size_t(h.ncm) * Rp);
  d.cmA_b = dalloc<double2>(h, size_t(h.ncm) * Rp);
  d.cmA_f = dalloc<float2>(h, size_t(h.ncm) * Rp);
  d.gK = dalloc<double2>(h, nK * Rp);
  d.wK = dalloc<double2>(h, nK * Rp);
  d.full0 = dalloc<double2>(h, size_t(h.dof) * Rp);
  d.full1 = dalloc<double2>(h, size_t(h.dof) * Rp);
  // basis vectors q_0..q_{max_iter} and one tentative vector beyond them
  d.V_kry = dalloc<double2>(h, (size_t(h.max_iter) + 2) * nl * Rp);
  d.w = dalloc<double2>(h, nl * Rp);
  d.t0 = dalloc<double2>(h, nl * Rp);
  d.t1 = dalloc<double2>(h, nl * Rp);
  d.t2 = dalloc<double2>(h, nl * Rp);
  d.vf = dalloc<float2>(h, nl * Rp);
  // multi-dot partials: up to 512 row chunks x (2 max_iter + 4) entries
  const size_t dstride = 2 * (size_t(h.max_iter) + 1) + 2;
  d.part = dalloc<double2>(h, size_t(512) * dstride * Rp);
  d.dots = dalloc<double2>(h, dstride * Rp);
  d.ucoef = dalloc<double2>(h, dstride * Rp);
  // partial norms: at most one per 64 entries of a dual vector, or 512 blocks
  d.npart = dalloc<double>(h, size_t((nl * Rp + 63) / 64 + 512) * Rp);
  size_t mv = size_t(h.max_iter) + 1;
  d.vcur = dalloc<double2>(h, nl * Rp);
  d.Hdev = dalloc<double2>(h, size_t(h.max_iter) * mv * Rp);
  d.Hraw = dalloc<double2>(h, size_t(h.max_iter) * mv * Rp);
  d.hprev = dalloc<double2>(h, (mv + 1) * Rp);
  d.rho = dalloc<double>(h, Rp);
  d.cs = dalloc<double2>(h, mv * Rp);
  d.sn = dalloc<double2>(h, mv * Rp);
  d.gvec = dalloc<double2>(h, (mv + 1) * Rp);
  d.beta = dalloc<double>(h, Rp);
  const size_t nres = (mv + 3) * Rp;
  d.resid = dalloc<double>(h, nres);
  d.hist = d.resid + 2 * Rp;
  d.jdev = dalloc<int>(h, 1);
  d.counter = dalloc<int>(h, 1);
  d.status = dalloc<int>(h, 2);
  d.done = dalloc<int>(h, Rp);
  d.iters = dalloc<int>(h, Rp);
  // the iteration status: written by the device straight into coherent pinned
  // host memory, read by the host after the iteration's event; behind it what the
  // host reads at the end of a run and the angles it sends
  void* ph = nullptr;
  const size_t status_bytes = (2 * STATUS_SLOTS * sizeof(int) + 63) / 64 * 64;
  HIPCHECK(hipHostMalloc(&ph, status_bytes + (nres + 3 * size_t(Rp)) * sizeof(double),
                         hipHostMallocMapped | hipHostMallocCoherent));
  d.status_host = static_cast<int*>(ph);
  d.res_host = reinterpret_cast<double*>(static_cast<char*>(ph) + status_bytes);
  d.nrm_host = d.res_host + nres;
  d.ang_host = d.nrm_host + 2 * Rp;
  void* pd = nullptr;
  HIPCHECK(hipHostGetDevicePointer(&pd, ph, 0));
  d.status_hdev = static_cast<int*>(pd);
  d.nrm = dalloc<double>(h, 2 * size_t(Rp));
  d.ycoef = dalloc<double2>(h, (size_t(h.max_iter) + 1) * Rp);
  // a gross failure of the factor (an unstable pivot sequence) shows here; a
  // residual at the level of cond(K) * eps is reported in the stats
  h.coarse_check = coarse_residual(h, kidx, kval);
  if (h.coarse_check > 1e-10) {
    // an ill-conditioned K costs the factor accuracy (the explicit inverse, or
    // block elimination that pivots only inside each block): every coarse solve
    // is then refined once against the assembled K
    std::vector<int64_t> ptr(size_t(h.nK) + 1, 0);
    for (int64_t key : kidx) ptr[key % h.nK + 1]++;
    for (int i = 0; i < h.nK; ++i) ptr[i + 1] += ptr[i];
    std::vector<int> col(kidx.size());
    std::vector<double2> val(kidx.size());
    std::vector<int64_t> fill(ptr.begin(), ptr.end() - 1);
    for (size_t t = 0; t < kidx.size(); ++t) {
      const int64_t at = fill[kidx[t] % h.nK]++;
      col[at] = int(kidx[t] / h.nK);
      val[at] = kval[t];
    }
    d.k_ptr = upload(h, ptr);
    d.k_col = upload(h, col);
    d.k_val = upload(h, val);
    d.nd_r = dalloc<double2>(h, size_t(h.nK) * Rp);
    d.nd_dx = dalloc<double2>(h, size_t(h.nK) * Rp);
    h.coarse_refine = true;
    h.coarse_bytes = 2 * h.coarse_bytes + 20.0 * double(kidx.size()) + 8.0 * (h.nK + 1);
    if (h.coarse_bytes1 > 0) h.coarse_bytes1 = 2 * h.coarse_bytes1 + 20.0 * double(kidx.size()) + 8.0 * (h.nK + 1);
    h.coarse_flops = 2 * h.coarse_flops + 8.0 * double(kidx.size());
    h.coarse_check = coarse_residual(h, kidx, kval);
  }
  if (!(h.coarse_check < 1e-6)) {
    char msg[96];
    std::snprintf(msg, sizeof msg, "coarse factor inaccurate (relative residual %.3e)", h.coarse_check);
    fail(HDP_E_COARSE, msg);
  }
  if (h.nh > 0) d.hb_tmp = dalloc<double2>(h, size_t(h.nh) * Rp);
  if (h.nonconforming) {
    d.fv = dalloc<double2>(h, nl * Rp);
    d.pv = dalloc<double2>(h, nl * Rp);
  }
  if (h.coarse_mode == 2 && h.nd_top_depth > 0) build_nd_top(h, kidx, kval);
  HIPCHECK(hipStreamSynchronize(h.stream));
}

// ---------------------------------------------------------------------------
// Operators on dual vectors ([nlam][R]).
// w = K^-1 g for R right-hand sides ([n_K][R]): a streaming GEMV kernel for a
// few columns, the tile kernels (matrix cores at 16-64 columns) from 4 on.
static void coarse_solve_once(Handle& h, const double2* g, double2* w, int R) {
  if (h.coarse_mode == 2) {
    coarse_solve_nd(h, g, w, R);
    return;
  }
  if (R < 4) {
    launch_coarse_solve(h, g, w, R, h.stream);
    return;
  }
  coarse_solve_dense_tiles(h, g, w, R);
}

// The coarse solve inside the operator applications, timed per kernel family:
// the one-RHS symmetric-tile apply as its two kernels, everything else as one.
static void coarse_solve_timed(Handle& h, const double2* g, double2* w, int R) {
  const double vec = 32.0 * double(h.nK) * R;
  if (R == 1 && h.coarse_mode == 0 && h.d.Ksym && !h.coarse_refine) {
    {
      Timed t(h, KF_COARSE, h.coarse_bytes1 + vec / 2, h.coarse_flops);
      launch_coarse_symv_tiles(h, g, h.stream);
    }
    Timed t(h, KF_COARSE_RED, 16.0 * double(h.sym_nt) * h.sym_nt * sym_tile_size() + vec / 2, 0);
    launch_coarse_symv_reduce(h, w, h.stream);
    return;
  }
  Timed t(h, KF_COARSE, (R == 1 && h.coarse_bytes1 > 0 ? h.coarse_bytes1 : h.coarse_bytes) + vec, h.coarse_flops * R);
  coarse_solve(h, g, w, R);
}

void coarse_solve(Handle& h, const double2* g, double2* w, int R) {
  coarse_solve_once(h, g, w, R);
  if (h.coarse_refine) {   // w += K^-1 (g - K w), once, against the assembled K
    auto& d = h.d;
    launch_csr_residual(h.nK, d.k_ptr, d.k_col, d.k_val, w, g, d.nd_r, R, h.stream);
    coarse_solve_once(h, d.nd_r, d.nd_dx, R);
    launch_axpby(w, d.nd_dx, w, int64_t(h.nK) * R, 1.0, 1.0, h.stream);
  }
}

// F up to the element slots: z = A_11^-1 y + Phi K^-1 Phi^T y with y = C_1^T v,
// left in slotB (FP64) or slotB_f (FP32).
static void apply_F_slots(Handle& h, const double2* v, int R, int prec) {
  auto& d = h.d;
  hipStream_t s = h.stream;
  const double c = 16.0 * R, nsl = h.nslots, ncm = h.ncm, nl = h.nlam, nK = h.nK;
  const double cw = prec == HDP_FP64 ? 16.0 * R : 8.0 * R;   // bytes per value of the local operators
  const double ob = prec == HDP_FP64 ? 1.0 : 0.5;
  if (prec != HDP_FP64) {
    Timed t(h, KF_CAST, nl * (c + cw), 0);
    launch_cast_f(v, d.vf, int64_t(h.nlam) * R, s);
  }
  {
    Timed t(h, KF_SLOT_F, nsl * cw * 2 + ncm * cw + ob * h.op1_bytes, h.flops_F * R);
    if (prec == HDP_FP64) launch_slot_apply<double2>(h, 0, v, d.slotA, d.cmA, R, s);
    else launch_slot_apply<float2>(h, 0, d.vf, d.slotA_f, d.cmA_f, R, s);
  }
  {
    Timed t(h, KF_ASSEMBLE, ncm * cw + nK * c, 0);
    // g = Phi^T y_1 + C_2^T v
    if (prec == HDP_FP64) launch_assemble<double2>(h, d.cmA, nullptr, v, 1.0, d.gK, R, s);
    else launch_assemble<float2>(h, d.cmA_f, nullptr, v, 1.0, d.gK, R, s);
  }
  {
    if (slot_coarse_from_tiles(h, R)) {
      // the tiled coarse apply's partial sums go straight into the coarse
      // correction of the slots (no row-sum kernel)
      {
        Timed t(h, KF_COARSE, h.coarse_bytes1 + 16.0 * nK, h.coarse_flops);
        launch_coarse_symv_tiles(h, d.gK, s);
      }
      Timed t(h, KF_SLOT_COARSE, nsl * cw * 2 + ncm * c + ob * h.phi_bytes, h.flops_coarse * R);
      if (prec == HDP_FP64) launch_slot_coarse_sym<double2>(h, d.slotA, d.slotB, s);
      else launch_slot_coarse_sym<float2>(h, d.slotA_f, d.slotB_f, s);
      return;
    }
    coarse_solve_timed(h, d.gK, d.wK, R);
  }
  {
    Timed t(h, KF_SLOT_COARSE, nsl * cw * 2 + ncm * c + ob * h.phi_bytes, h.flops_coarse * R);
    if (prec == HDP_FP64) launch_slot_coarse<double2>(h, d.slotA, d.wK, d.slotB, R, s);
    else launch_slot_coarse<float2>(h, d.slotA_f, d.wK, d.slotB_f, R, s);
  }
}

void apply_F(Handle& h, const double2* v, double2* u, int R, int prec) {
  auto& d = h.d;
  const double c = 16.0 * R, nsl = h.nslots, nl = h.nlam;
  const double cw = prec == HDP_FP64 ? 16.0 * R : 8.0 * R;
  apply_F_slots(h, v, R, prec);
  Timed t(h, KF_ROWGATHER, nsl * cw + nl * c, 0);
  // u = C_1 z + C_2 w
  if (prec == HDP_FP64) launch_rowgather<double2>(h, d.slotB, false, false, d.wK, u, R, h.stream);
  else launch_rowgather<float2>(h, d.slotB_f, false, false, d.wK, u, R, h.stream);
}

void apply_P(Handle& h, const double2* v, double2* u, int R, int prec);

// w = P^-1 F v with the preconditioner's gather reading F's slot values directly.
void apply_PF(Handle& h, const double2* v, double2* w, int R, int prec) {
  auto& d = h.d;
  if (h.nonconforming) {
    // C_2 terms enter both operators: apply them one after the other
    apply_F(h, v, d.fv, R, prec);
    apply_P(h, d.fv, w, R, prec);
    return;
  }
  hipStream_t s = h.stream;
  const double c = 16.0 * R, nsl = h.nslots, nl = h.nlam;
  const double cw = prec == HDP_FP64 ? 16.0 * R : 8.0 * R;
  const double ob = prec == HDP_FP64 ? 1.0 : 0.5;
  apply_F_slots(h, v, R, prec);
  if (prec == HDP_FP64 && slot_rows_fused(h, R)) {
    // preconditioner with the row gather fused: w must be zero on entry (the
    // GMRES update clears it after its last read)
    Timed t(h, KF_SLOT_P, nsl * cw * 2 + ob * h.se_bytes + nl * c, h.flops_P * R);
    launch_slot_apply_rows(h, d.slotB, w, R, s);
    return;
  }
  {
    Timed t(h, KF_SLOT_P, nsl * cw * 2 + ob * h.se_bytes, h.flops_P * R);
    if (prec == HDP_FP64) launch_slot_apply<double2>(h, 2, d.slotB, d.slotA, nullptr, R, s);
    else launch_slot_apply<float2>(h, 2, d.slotB_f, d.slotA_f, nullptr, R, s);
  }
  {
    Timed t(h, KF_ROWGATHER, nsl * cw + nl * c, 0);
    if (prec == HDP_FP64) launch_rowgather<double2>(h, d.slotA, false, true, nullptr, w, R, s);
    else launch_rowgather<float2>(h, d.slotA_f, false, true, nullptr, w, R, s);
  }
}

// P^-1 v with the work buffers of w (the handle's own, or the caller-free
// scratch of the allocation-free entry point).
void apply_P_ws(Handle& h, const double2* v, double2* u, int R, int prec, const PWork& w) {
  auto& d = h.d;
  hipStream_t s = h.stream;
  const double c = 16.0 * R, nsl = h.nslots, nl = h.nlam, nh = h.nh;
  const double cw = prec == HDP_FP64 ? 16.0 * R : 8.0 * R;
  const double ob = prec == HDP_FP64 ? 1.0 : 0.5;
  const double hb_bytes = 8.0 * h.hb_xinv.size();
  if (h.nh > 0) {
    // P^-1 = X^-1 Y X^-1: X is diagonal except for dense blocks on the hanging
    // rows, whose scale factor is 1 in row_xinv; first s = X^-1 v there
    Timed t(h, KF_HBLOCK, hb_bytes + 2 * nh * c + nl * 2 * c, 2.0 * h.hb_xinv.size() * 2 * R);
    launch_hcopy(h, v, w.pv, R, s);
    v = w.pv;
  }
  if (prec != HDP_FP64) {
    Timed t(h, KF_CAST, nl * (c + cw), 0);
    launch_cast_f(v, w.vf, int64_t(h.nlam) * R, s);
  }
  {
    Timed t(h, KF_SLOT_P, nsl * cw * 2 + ob * h.se_bytes, h.flops_P * R);
    if (prec == HDP_FP64) launch_slot_apply<double2>(h, 1, v, w.slot, nullptr, R, s);
    else launch_slot_apply<float2>(h, 1, w.vf, w.slot_f, nullptr, R, s);
  }
  if (h.nh > 0 && h.hb_largest <= HB_GATHER) {
    // hanging rows: u = X^-1 (C_1 S C_1^T s + Y_2 s)
    Timed t(h, KF_HBLOCK, nsl * cw + nl * c + 2 * hb_bytes + 2 * nh * c, 2.0 * 2 * h.hb_xinv.size() * 2 * R);
    if (prec == HDP_FP64) launch_hgather<double2>(h, w.slot, w.pv, u, R, s);
    else launch_hgather<float2>(h, w.slot_f, w.pv, u, R, s);
    return;
  }
  {
    Timed t(h, KF_ROWGATHER, nsl * cw + nl * c, 0);
    if (prec == HDP_FP64) launch_rowgather<double2>(h, w.slot, false, true, nullptr, u, R, s);
    else launch_rowgather<float2>(h, w.slot_f, false, true, nullptr, u, R, s);
  }
  if (h.nh > 0) {
    Timed t(h, KF_HBLOCK, 2 * hb_bytes + 6 * nh * c, 2.0 * 2 * h.hb_xinv.size() * 2 * R);
    launch_hblock(h, true, w.pv, true, u, w.hb_tmp, false, R, s);
    launch_hblock(h, false, w.hb_tmp, false, nullptr, u, true, R, s);
  }
}

void apply_P(Handle& h, const double2* v, double2* u, int R, int prec) {
  auto& d = h.d;
  apply_P_ws(h, v, u, R, prec, PWork{d.slotA, d.slotA_f, d.vf, d.pv, d.hb_tmp});
}

// Solve A^ [x_I; x_R] = [y_I; y_R] element-wise (eq. block_matrix_inversion):
// y_I is read from Y (coarse modes ignored; with nu, C_1^T nu subtracted at the
// dual slots); X receives the element solution; y_R is assembled from Y's coarse
// modes, minus C_2^T nu when nu is given.  A coarse pass (x_R and K_e x_R) and,
// after the coarse solve, the full solve of y - E_R mu, which folds the Woodbury
// correction into the separable solve.
void element_solve(Handle& h, double2* X, const double2* Y, const double2* nu, int R) {
  auto& d = h.d;
  hipStream_t s = h.stream;
  const double c = 16.0 * R, dof = double(h.dof), ncm = h.ncm, nK = h.nK;
  {
    Timed t(h, KF_FDM, dof * c + 2 * ncm * c, h.flops_fdm_coarse * R);
    launch_sep_coarse(h, Y, R, s, nu);
  }
  {
    Timed t(h, KF_ASSEMBLE, 2 * ncm * c + nK * c, 0);
    launch_assemble<double2>(h, d.cmA, Y, nu, -1.0, d.gK, R, s);
  }
  coarse_solve_timed(h, d.gK, d.wK, R);
  Timed t(h, KF_FDM, 2 * dof * c + ncm * c + nK * c, h.flops_fdm * R);
  launch_coarse_minus_tw(h, d.wK, R, false, s);
  launch_sep_full(h, Y, X, R, s, nu);
}

// Interface right-hand side g = C_1 x_1 + C_2 x_2 of x = A^-1 b^ with the element
// loads in full0 (eq. block_matrix_inversion).  Only the dual-slot values of x are
// formed: the first pass of the element solve keeps
// the slot values x_S and coarse-mode values x_R of A~^-1 b (coarse rows of b
// zeroed), and the Woodbury correction restricted to the slots is
// x_1 = x_S - Phi (x_R - T_e w) (Phi = G_S K_e, G = A~^-1 E_R), which the slot
// coarse correction applies; the full corrected solve is left to the recovery.
void interface_rhs(Handle& h, double2* g, int R) {
  auto& d = h.d;
  hipStream_t s = h.stream;
  const double c = 16.0 * R, nsl = h.nslots, ncm = h.ncm, nK = h.nK, dof = double(h.dof);
  {
    Timed t(h, KF_FDM, dof * c + 2 * ncm * c + nsl * c, h.flops_fdm_coarse * R);
    launch_sep_coarse(h, d.full0, R, s, nullptr, d.slotA);   // x_S, x_R, K_e x_R
  }
  {
    // K_e x_R of the loads, for the recovery of the same loads
    Timed t(h, KF_ELEMENT_MISC, 2 * ncm * c, 0);
    HIPCHECK(hipMemcpyAsync(d.cmA_b, d.cmA, size_t(h.ncm) * R * sizeof(double2), hipMemcpyDeviceToDevice, s));
    h.cmA_b_R = R;
  }
  {
    Timed t(h, KF_ASSEMBLE, 2 * ncm * c + nK * c, 0);
    launch_assemble<double2>(h, d.cmA, d.full0, nullptr, -1.0, d.gK, R, s);
  }
  coarse_solve_timed(h, d.gK, d.wK, R);
  {
    Timed t(h, KF_SLOT_COARSE, nsl * c * 2 + 2 * ncm * c + h.phi_bytes, h.flops_coarse * R);
    launch_coarse_minus_tw(h, d.wK, R, false, s);               // cmX = x_R - T_e w
    launch_slot_coarse_cm(h, d.slotA, d.cmX, d.slotB, R, s);    // x_1 = x_S - Phi cmX
  }
  Timed t(h, KF_ROWGATHER, nsl * c + h.nlam * c, 0);
  launch_rowgather<double2>(h, d.slotB, false, false, d.wK, g, R, s);   // C_1 x_1 + C_2 x_2
}

// Recovery phi = A^-1 (b^ - C^T nu) of the loads in full0 after interface_rhs
// (Sec. 2.3.1).  The element solve's coarse pass is linear in the load, and on
// a load y on the dual slots K_e x_R(y) = Phi^T y (A~ and K_e are complex
// symmetric), which the slot operators give.  So K_e x_R of b - C_1^T nu is the
// right-hand side pass's K_e x_R(b) minus Phi^T C_1^T nu, and only the coarse
// solve and the corrected full solve run again.
void recover(Handle& h, double2* X, const double2* nu, int R) {
  auto& d = h.d;
  hipStream_t s = h.stream;
  if (h.cmA_b_R != R) {
    element_solve(h, X, d.full0, nu, R);
    return;
  }
  const double c = 16.0 * R, nsl = h.nslots, ncm = h.ncm, nK = h.nK, dof = double(h.dof);
  {
    Timed t(h, KF_SLOT_F, nsl * c * 2 + ncm * c + h.op1_bytes, h.flops_F * R);
    launch_slot_apply<double2>(h, 0, nu, d.slotA, d.cmA, R, s);   // cmA = Phi^T C_1^T nu
  }
  {
    Timed t(h, KF_ELEMENT_MISC, 3 * ncm * c, 0);
    launch_axpby(d.cmA_b, d.cmA, d.cmA, int64_t(h.ncm) * R, 1.0, -1.0, s);
  }
  {
    Timed t(h, KF_ASSEMBLE, 2 * ncm * c + nK * c, 0);
    launch_assemble<double2>(h, d.cmA, d.full0, nu, -1.0, d.gK, R, s);
  }
  coarse_solve_timed(h, d.gK, d.wK, R);
  {
    Timed t(h, KF_FDM, 2 * dof * c + 2 * ncm * c + nK * c, h.flops_fdm * R);
    launch_coarse_minus_tw(h, d.wK, R, true, s);
    launch_sep_full(h, d.full0, X, R, s, nu, d.cmA);
  }
}

struct GmresResult {
  std::vector<int> iters;
  std::vector<double> rel;
};

// Left-preconditioned GMRES on R systems at once (x0 = 0); stops each system
// when ||P^-1 r_k|| / ||P^-1 r_0|| <= tol.  x receives the iterate.  The
// Arnoldi basis is orthogonalised twice (classical Gram-Schmidt with one
// reorthogonalisation), the second pass delayed into the next iteration so that
// each iteration makes one pass over the basis for dots and one for updates.
// The Arnoldi step, the Hessenberg column and the Givens rotations stay on the
// device; the host reads a two-word status one iteration behind the GPU.
GmresResult gmres(Handle& h, const double2* rhs, double2* x, int R, int prec, double tol, int max_iter) {
  auto& d = h.d;
  hipStream_t s = h.stream;
  const int n = h.nlam;
  const int64_t vs = int64_t(n) * R;
  const int maxvec = h.max_iter + 1;
  max_iter = std::min(max_iter, h.max_iter);
  GmresDims gd = gmres_dims(n, R, maxvec);
  const double vb = 16.0 * double(vs);
  const int Rmax = pow2ceil(h.max_rhs);   // the widest run: rows of the result block
  GmresResult res;
  res.iters.assign(R, 0);
  res.rel.assign(R, 1.0);
  HIPCHECK(hipMemsetAsync(x, 0, size_t(vs) * sizeof(double2), s));
  apply_P(h, rhs, d.w, R, prec);
  {
    Timed t(h, KF_NORM_SCALE, 3 * vb, 6.0 * double(vs));
    launch_normalize(d.w, n, R, gd, d.npart, d.nrm, d.V_kry, nullptr, vs, d.vcur, s);
  }
  launch_gmres_init(d.nrm, d.beta, d.gvec, d.done, d.iters, d.resid, d.jdev, d.counter, d.status, R, d.hist, s);
  for (int q = 0; q < 2 * STATUS_SLOTS; ++q) d.status_host[q] = 0;   // no kernel of this stream writes it yet
  // the fused preconditioner adds into w; later iterations find it cleared by the update
  HIPCHECK(hipMemsetAsync(d.w, 0, size_t(vs) * sizeof(double2), s));
  // up to `ahead` iterations are queued beyond the one whose status the host
  // reads; the device writes the status of iteration j to slot j mod
  // STATUS_SLOTS (more slots than iterations in flight)
  const int ahead = vs >= GMRES_LONG ? 0 : GMRES_AHEAD;
  hipEvent_t ev[STATUS_SLOTS];
  for (int q = 0; q < STATUS_SLOTS; ++q) HIPCHECK(hipEventCreateWithFlags(&ev[q], hipEventDisableTiming));
  int launched = 0;
  try {
    const int dstride = 2 * maxvec + 2;
    const bool fold = gd.nchunks <= DOTS_FOLD;
    // one Arnoldi step with delayed reorthogonalisation; nv - 1 = j basis
    // vectors are final when it starts
    auto issue = [&](int nv) {
      const double jv = nv - 1;
      apply_PF(h, d.vcur, d.w, R, prec);
      {
        Timed t(h, KF_DOTS, (jv + 2) * vb, (16.0 * jv + 24.0) * double(vs));
        launch_dmdot(d.V_kry, vs, d.jdev, d.w, n, R, gd, dstride, d.part, s);
        if (!fold) launch_dmdot_reduce(d.part, gd, d.jdev, dstride, R, d.dots, s);
      }
      {
        Timed t(h, KF_GIVENS, 0, 0);
        launch_dcgs_scalar(d.jdev, fold ? d.part : d.dots, fold ? gd.nchunks : 1, int64_t(dstride) * R, d.Hraw, d.hprev, d.rho, d.ucoef, d.Hdev, d.cs, d.sn, d.gvec, d.beta,
                           d.done, d.iters, d.resid, tol, maxvec, R, d.counter, d.status_hdev, d.hist, s);
      }
      {
        Timed t(h, KF_UPDATE, (jv + 5) * vb, (16.0 * jv + 20.0) * double(vs));
        launch_dupdate(d.V_kry, vs, d.jdev, d.ucoef, d.w, n, R, d.vcur, d.Hraw, d.hprev, maxvec, s);
      }
    };
    // one GMRES iteration as a captured graph (every launch reads j on the device)
    hipGraphExec_t exec = nullptr;
    // captured at fewer than 4 columns (no library routine is in any solve; the
    // replay test covers one column)
    const bool graph = h.use_graphs && !h.prof.on && (h.coarse_mode == 0 || h.coarse_mode == 2) && R < 4;
    if (graph) {
      auto key = std::make_tuple(R, prec, tol);
      auto itg = h.graphs.find(key);
      if (itg == h.graphs.end()) {
        hipGraph_t gr;
        HIPCHECK(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
        issue(1);
        HIPCHECK(hipStreamEndCapture(s, &gr));
        hipGraphExec_t ex;
        hipError_t ie = hipGraphInstantiate(&ex, gr, nullptr, nullptr, 0);
        (void)hipGraphDestroy(gr);
        HIPCHECK(ie);
        itg = h.graphs.emplace(key, ex).first;
      }
      exec = itg->second;
    }
    using clk = std::chrono::steady_clock;
    // column j - 1 of H is completed in iteration j: max_iter + 1 iterations
    for (int it = 0; it <= max_iter; ++it) {
      auto t0 = clk::now();
      if (graph) HIPCHECK(hipGraphLaunch(exec, s));
      else issue(it + 1);
      HIPCHECK(hipEventRecord(ev[it % STATUS_SLOTS], s));
      auto t1 = clk::now();
      h.t_launch += std::chrono::duration<double, std::milli>(t1 - t0).count();
      launched = it + 1;
      if (it >= ahead) {
        HIPCHECK(hipEventSynchronize(ev[(it - ahead) % STATUS_SLOTS]));
        h.t_wait += std::chrono::duration<double, std::milli>(clk::now() - t1).count();
        if (d.status_host[2 * ((it - ahead) % STATUS_SLOTS)]) break;
      }
    }
    // x = sum_i V_i y_i with H y = g
    launch_gmres_end(d.Hdev, d.gvec, d.iters, maxvec, R, d.ycoef, d.jdev, d.resid, Rmax, s);
    launch_mupdate(d.V_kry, vs, d.jdev, d.ycoef, x, n, R, 1.0, nullptr, s);
    HIPCHECK(hipMemcpyAsync(d.res_host, d.resid, (2 * size_t(Rmax) + size_t(launched + 1) * R) * sizeof(double),
                            hipMemcpyDeviceToHost, s));
    HIPCHECK(hipStreamSynchronize(s));
  } catch (...) {
    (void)hipStreamSynchronize(s);
    for (int q = 0; q < STATUS_SLOTS; ++q) (void)hipEventDestroy(ev[q]);
    throw;
  }
  for (int q = 0; q < STATUS_SLOTS; ++q) (void)hipEventDestroy(ev[q]);
  prof_flush(h);
  int kmax = 0;
  for (int r = 0; r < R; ++r) {
    res.iters[r] = int(d.res_host[Rmax + r]);
    res.rel[r] = d.res_host[r];
    kmax = std::max(kmax, res.iters[r]);
  }
  h.last_hist.assign(d.res_host + 2 * Rmax, d.res_host + 2 * Rmax + size_t(kmax + 1) * R);
  h.last_hist_R = R;
  h.last_hist_len = kmax + 1;
  return res;
}

// Geometry of the far-field integral over the boundary of the leaves marked
// inside (Sec. 3.3.1): every side of an outside leaf whose neighbour is inside,
// Gauss-Legendre with n+12 nodes per side.
void far_prepare(Handle& h, int n_far, const double* angles, const uint8_t* inside, int R) {
  auto& f = h.far;
  std::vector<uint8_t> in(inside, inside + h.E);
  std::vector<double> an(angles, angles + n_far);
  if (f.elem && in == f.inside && an == f.angles && f.capR >= R) return;
  std::vector<int> el, sd, noff{0};
  std::vector<int64_t> toff{0};
  std::vector<double> tab, dsc, px, py, pw, pnx, pny;
  struct Rule {
    std::vector<double> x, w, N, d0, d1;   // nodes, weights, [q][n] basis, derivatives at -1 and 1
  };
  std::map<int, Rule> rules;   // by n
  for (int e = 0; e < h.E; ++e) {
    if (in[e]) continue;
    for (int s = 1; s <= 4; ++s) {
      const int si = 4 * e + s - 1;
      bool facing_inside = false;
      if (h.side_type[si] == 1 || h.side_type[si] == 2) {
        facing_inside = in[h.nb_e[si]] != 0;
      } else if (h.side_type[si] == 3) {
        int n_in = 0;
        for (int f : h.side_nbrs[si]) n_in += in[f] != 0;
        if (n_in != 0 && n_in != int(h.side_nbrs[si].size()))
          fail(HDP_E_ARG, "far-field boundary must follow whole element sides of the outside elements");
        facing_inside = n_in != 0;
      }
      if (!facing_inside) continue;
      const int n = h.deg[e] + 1, q = n + 12;
      Rule& u = rules[n];
      if (u.x.empty()) {
        gauss_legendre(q, u.x, u.w);
        u.N.resize(size_t(q) * n);
        for (int t = 0; t < q; ++t) vertex_basis(n, u.x[t], u.N.data() + size_t(t) * n);
        u.d0.resize(n);
        u.d1.resize(n);
        vertex_basis_dx(n, -1.0, u.d0.data());
        vertex_basis_dx(n, 1.0, u.d1.data());
      }
      const std::vector<double>&xq = u.x, &wq = u.w;
      double ox = h.ox[e], oy = h.oy[e], hx = h.hx[e], hy = h.hy[e];
      double nx = s == 1 ? 1 : s == 2 ? -1 : 0, ny = s == 3 ? 1 : s == 4 ? -1 : 0;   // into e
      tab.insert(tab.end(), u.N.begin(), u.N.end());
      for (int t = 0; t < q; ++t) {
        double x, y;
        if (s <= 2) { x = s == 1 ? ox : ox + hx; y = oy + (xq[t] + 1) * hy / 2; }
        else { y = s == 3 ? oy : oy + hy; x = ox + (xq[t] + 1) * hx / 2; }
        px.push_back(x);
        py.push_back(y);
        pw.push_back(wq[t] * (s <= 2 ? hy : hx) / 2);
        pnx.push_back(nx);
        pny.push_back(ny);
      }
      const auto& dend = (s == 2 || s == 4) ? u.d1 : u.d0;
      tab.insert(tab.end(), dend.begin(), dend.end());
      dsc.push_back(s <= 2 ? nx * 2.0 / hx : ny * 2.0 / hy);
      el.push_back(e);
      sd.push_back(s);
      noff.push_back(noff.back() + q);
      toff.push_back(int64_t(tab.size()));
    }
  }
  f.nsides = int(el.size());
  f.nq = noff.back();
  f.nfar = n_far;
  f.inside = in;
  f.angles = an;
  f.capR = std::max(f.capR, R);
  f.elem = upload(h, el);
  f.side = upload(h, sd);
  f.node_off = upload(h, noff);
  f.tab_off = upload(h, toff);
  f.tab = upload(h, tab);
  f.dscale = upload(h, dsc);
  f.px = upload(h, px);
  f.py = upload(h, py);
  f.pw = upload(h, pw);
  f.pnx = upload(h, pnx);
  f.pny = upload(h, pny);
  f.ang = upload(h, an);
  f.U = dalloc<double2>(h, size_t(std::max(1, f.nq)) * f.capR);
  f.DU = dalloc<double2>(h, size_t(std::max(1, f.nq)) * f.capR);
}

// Set-up autotuner: each candidate tile width of the separable element solve
// and of the slot operators runs three times on the handle's own mesh at max_rhs
// columns (after one untimed launch); the fastest is kept.  The element solve
// is timed as its two passes (coarse pass and corrected solve) on a zero input
// (its time does not depend on the values), the slot operators as the interface
// operator's first product.
static void set_nd_split(Handle& h, int target);
static void coarse_solve_nd(Handle& h, const double2* g, double2* w, int R);

static void autotune(Handle& h, bool fdm, bool slot) {
  auto& d = h.d;
  hipStream_t s = h.stream;
  const int R = pow2ceil(h.max_rhs);
  hipEvent_t a, b;
  HIPCHECK(hipEventCreate(&a));
  HIPCHECK(hipEventCreate(&b));
  auto time3 = [&](auto&& launch) {
    launch();
    HIPCHECK(hipEventRecord(a, s));
    for (int q = 0; q < 3; ++q) launch();
    HIPCHECK(hipEventRecord(b, s));
    HIPCHECK(hipEventSynchronize(b));
    float ms = 0;
    HIPCHECK(hipEventElapsedTime(&ms, a, b));
    return double(ms) / 3.0;
  };
  try {
    launch_fill_zero(d.full0, int64_t(h.dof) * R, s);
    launch_fill_zero(d.w, int64_t(h.nlam) * R, s);
    if (fdm) {
      int best = 0;
      double tbest = 1e300;
      const size_t first = h.tune.size();
      for (int rc : {1, 2, 4, 8, 16}) {
        if (rc > std::min(16, R) || !sep_width_fits(h, rc)) break;
        launch_fill_zero(d.cmX, int64_t(h.ncm) * R, s);
        const double ms = time3([&] {
          launch_sep_coarse(h, d.full0, R, s, nullptr, nullptr, rc);
          launch_sep_full(h, d.full0, d.full1, R, s, nullptr, nullptr, rc);
        });
        h.tune.push_back({"fdm_element_solve", rc, ms, false});
        if (ms < tbest) { tbest = ms; best = rc; }
      }
      h.fdm_rc = best;
      for (size_t i = first; i < h.tune.size(); ++i) h.tune[i].chosen = h.tune[i].cols == best;
    }
    if (slot && R >= 16) {
      int best = h.slot_rb;
      double tbest = 1e300;
      const size_t first = h.tune.size();
      for (int rb : {16, 32, 64}) {
        if (rb > R) break;
        h.slot_rb = rb;
        const double ms = time3([&] { launch_slot_apply<double2>(h, 0, d.w, d.slotA, d.cmA, R, s); });
        h.tune.push_back({"slot_operator", rb, ms, false});
        if (ms < tbest) { tbest = ms; best = rb; }
      }
      h.slot_rb = best;
      for (size_t i = first; i < h.tune.size(); ++i) h.tune[i].chosen = h.tune[i].cols == best;
    }
    if (h.coarse_mode == 2 && R > 1) {
      // nested-dissection split target: one coarse solve at max_rhs columns
      int best = h.nd_split;
      double tbest = 1e300;
      const size_t first = h.tune.size();
      launch_fill_zero(d.gK, int64_t(h.nK) * R, s);
      for (int target : ND_SPLITS) {
        set_nd_split(h, target);
        const double ms = time3([&] { coarse_solve_nd(h, d.gK, d.wK, R); });
        h.tune.push_back({"coarse_nd_split", target, ms, false});
        if (ms < tbest) { tbest = ms; best = target; }
      }
      set_nd_split(h, best);
      for (size_t i = first; i < h.tune.size(); ++i) h.tune[i].chosen = h.tune[i].cols == best;
    }
  } catch (...) {
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    throw;
  }
  HIPCHECK(hipEventDestroy(a));
  HIPCHECK(hipEventDestroy(b));
}

// Order the handle's stream after everything already issued on the caller's stream.
void after_user(Handle& h) {
  HIPCHECK(hipEventRecord(h.order_ev, h.user_stream));
  HIPCHECK(hipStreamWaitEvent(h.stream, h.order_ev, 0));
}

}  // namespace hdp

using namespace hdp;

#define API_BEGIN try {
#define API_END                                  \
  }                                              \
  catch (const Error& e) {                       \
    g_err = e.msg;                               \
    return e.status;                             \
  }                                              \
  catch (const std::exception& e) {              \
    g_err = e.what();                            \
    return HDP_E_ARG;                            \
  }

extern "C" {

hdp_status hdp_setup(const hdp_mesh* mesh, const hdp_problem* prob, const hdp_options* opt, hdp_handle** out) {
  API_BEGIN
  if (!out || !opt) fail(HDP_E_ARG, "null output or options");
  *out = nullptr;
  if (opt->max_rhs < 1 || opt->max_rhs > 64) fail(HDP_E_ARG, "max_rhs must lie in 1..64");
  if (opt->max_iter < 1 || opt->max_iter > 1000) fail(HDP_E_ARG, "max_iter must lie in 1..1000");
  if (!(opt->tol > 0) || !(opt->tol < 1)) fail(HDP_E_ARG, "tol must lie in (0,1)");
  if (opt->precision != HDP_FP64 && opt->precision != HDP_MIXED) fail(HDP_E_ARG, "unknown precision");
  auto t0 = std::chrono::steady_clock::now();
  hdp_handle* H = new hdp_handle();
  Handle& h = H->h;
  h.max_rhs = opt->max_rhs;
  h.max_iter = opt->max_iter;
  h.tol = opt->tol;
  h.precision = opt->precision;
  h.user_stream = static_cast<hipStream_t>(opt->stream);
  h.use_graphs = (opt->flags & HDP_FLAG_GRAPH) != 0;
  if (opt->tile_fdm != 0 && opt->tile_fdm != 1 && opt->tile_fdm != 2 && opt->tile_fdm != 4 && opt->tile_fdm != 8 &&
      opt->tile_fdm != 16)
    fail(HDP_E_ARG, "tile_fdm must be 0, 1, 2, 4, 8 or 16");
  if (opt->tile_slot != 0 && opt->tile_slot != 16 && opt->tile_slot != 32 && opt->tile_slot != 64)
    fail(HDP_E_ARG, "tile_slot must be 0, 16, 32 or 64");
  h.fdm_rc = opt->tile_fdm;
  if (opt->tile_slot) h.slot_rb = opt->tile_slot;
  if ((opt->allocator.alloc == nullptr) != (opt->allocator.free == nullptr))
    fail(HDP_E_ARG, "hdp_allocator: set both alloc and free, or neither");
  h.allocator = opt->allocator;
  if (opt->flags & HDP_FLAG_COARSE_BLOCK)
    fail(HDP_E_ARG, "HDP_FLAG_COARSE_BLOCK: the strip factor is no longer provided (use HDP_FLAG_COARSE_ND)");
  if ((opt->flags & HDP_FLAG_COARSE_DENSE) && (opt->flags & HDP_FLAG_COARSE_ND))
    fail(HDP_E_ARG, "HDP_FLAG_COARSE_DENSE and HDP_FLAG_COARSE_ND are exclusive");
  h.coarse_mode = (opt->flags & HDP_FLAG_COARSE_DENSE) ? 0 : (opt->flags & HDP_FLAG_COARSE_ND) ? 2 : -1;
  try {
    HIPCHECK(hipGetDevice(&h.device));
    scratch_init(h.device);   // the allocation-free entry point's array on this device
    // a stream of the handle's own (default priority): capturable, unlike the null stream
    HIPCHECK(hipStreamCreateWithFlags(&h.stream, hipStreamNonBlocking));
    HIPCHECK(hipEventCreateWithFlags(&h.order_ev, hipEventDisableTiming));
    HIPCHECK(hipEventRecord(h.order_ev, h.user_stream));
    HIPCHECK(hipStreamWaitEvent(h.stream, h.order_ev, 0));
    Team team;
    {
      const auto th = std::chrono::steady_clock::now();
      build_host(h, mesh, prob, &team);
      h.setup_host_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - th).count();
    }
    build_device(h, team);
    if (opt->flags & HDP_FLAG_AUTOTUNE) autotune(h, opt->tile_fdm == 0, opt->tile_slot == 0);
  } catch (...) {
    if (h.stream) (void)hipStreamSynchronize(h.stream);
    release_allocations(h);
    if (h.d.status_host) (void)hipHostFree(h.d.status_host);
    if (h.order_ev) (void)hipEventDestroy(h.order_ev);
    if (h.rocblas) rocblas_destroy_handle(static_cast<rocblas_handle>(h.rocblas));
    if (h.stream) (void)hipStreamDestroy(h.stream);
    delete H;
    throw;
  }
  h.setup_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  *out = H;
  return HDP_OK;
  API_END
}

hdp_status hdp_inspect(const hdp_mesh* mesh, const hdp_problem* prob, hdp_stats* st) {
  API_BEGIN
  if (!st) fail(HDP_E_ARG, "null stats");
  hdp_handle H;
  build_host(H.h, mesh, prob);
  {
    std::vector<int64_t> kidx;
    std::vector<double2> kval;
    coarse_coo(H.h, kidx, kval);
    H.h.coarse_band_bytes = coarse_band_bytes(H.h.nK, kidx);
  }
  return hdp_get_stats(&H, st);
  API_END
}

hdp_status hdp_get_stats(const hdp_handle* H, hdp_stats* st) {
  API_BEGIN
  if (!H || !st) fail(HDP_E_ARG, "null handle or stats");
  const Handle& h = H->h;
  std::memset(st, 0, sizeof(*st));
  st->dof = h.dof;
  st->n_elements = h.E;
  st->n_lambda = h.nlam;
  st->n_coarse = h.nK;
  st->l = h.l;
  st->n_classes = int(h.classes.size());
  st->min_element_margin = h.min_margin;
  st->setup_ms = h.setup_ms;
  st->coarse_residual = h.coarse_check;
  st->coarse_mode = h.coarse_mode >= 0 ? h.coarse_mode : (h.nK > 6000 ? 2 : 0);
  st->coarse_band_bytes = h.coarse_band_bytes;
  st->setup_host_ms = h.setup_host_ms;
  st->setup_classes_ms = h.setup_classes_ms;
  st->setup_coarse_ms = h.setup_coarse_ms;
  st->coarse_factor_bytes = h.coarse_bytes;
  st->coarse_blocks = st->coarse_mode == 2 ? int(h.nd_off.size()) - 1 : 1;
  st->coarse_top_unknowns = h.nd_top_n;
  st->coarse_top_check = h.nd_top_check;
  return HDP_OK;
  API_END
}

hdp_status hdp_apply_interface(hdp_handle* H, const hdp_c64* v, hdp_c64* u, int32_t n_rhs, int32_t precision) {
  API_BEGIN
  if (!H || !v || !u) fail(HDP_E_ARG, "null argument");
  Handle& h = H->h;
  if (n_rhs < 1 || n_rhs > pow2ceil(h.max_rhs)) fail(HDP_E_ARG, "n_rhs out of range");
  after_user(h);
  apply_F(h, reinterpret_cast<const double2*>(v), reinterpret_cast<double2*>(u), n_rhs, precision);
  HIPCHECK(hipStreamSynchronize(h.stream));
  prof_flush(h);
  return HDP_OK;
  API_END
}

hdp_status hdp_apply_precond(hdp_handle* H, const hdp_c64* v, hdp_c64* u, int32_t n_rhs, int32_t precision) {
  API_BEGIN
  if (!H || !v || !u) fail(HDP_E_ARG, "null argument");
  Handle& h = H->h;
  if (n_rhs < 1 || n_rhs > pow2ceil(h.max_rhs)) fail(HDP_E_ARG, "n_rhs out of range");
  after_user(h);
  apply_P(h, reinterpret_cast<const double2*>(v), reinterpret_cast<double2*>(u), n_rhs, precision);
  HIPCHECK(hipStreamSynchronize(h.stream));
  prof_flush(h);
  return HDP_OK;
  API_END
}

hdp_status hdp_apply_precond_noalloc(hdp_handle* H, const hdp_c64* v, hdp_c64* u, int32_t n_rhs,
                                     int32_t precision) {
  API_BEGIN
  if (!H || !v || !u) fail(HDP_E_ARG, "null argument");
  Handle& h = H->h;
  if (n_rhs < 1 || n_rhs > pow2ceil(h.max_rhs)) fail(HDP_E_ARG, "n_rhs out of range");
  if (precision != HDP_FP64 && precision != HDP_MIXED) fail(HDP_E_ARG, "unknown precision");
  // carve the work buffers out of the device's scratch array, 256-byte aligned
  const size_t R = size_t(n_rhs);
  const bool mixed = precision == HDP_MIXED, hanging = h.nh > 0;
  const size_t sizes[5] = {mixed ? 0 : size_t(h.nslots) * R * sizeof(double2),
                           mixed ? size_t(h.nslots) * R * sizeof(float2) : 0,
                           mixed ? size_t(h.nlam) * R * sizeof(float2) : 0,
                           hanging ? size_t(h.nlam) * R * sizeof(double2) : 0,
                           hanging ? size_t(h.nh) * R * sizeof(double2) : 0};
  size_t off[5], need = 0;
  for (int i = 0; i < 5; ++i) {
    off[i] = need;
    need += (sizes[i] + 255) / 256 * 256;
  }
  if (need > SCRATCH_BYTES) {
    char msg[160];
    std::snprintf(msg, sizeof msg, "hdp_apply_precond_noalloc needs %zu bytes of scratch at n_rhs = %d; the limit is %zu",
                  need, n_rhs, SCRATCH_BYTES);
    fail(HDP_E_ARG, msg);
  }
  char* base = static_cast<char*>(scratch_ptr(h.device));
  if (!base) fail(HDP_E_DEVICE, "scratch array not resolved on the handle's device");
  auto at = [&](int i) { return sizes[i] ? static_cast<void*>(base + off[i]) : nullptr; };
  const PWork w{static_cast<double2*>(at(0)), static_cast<float2*>(at(1)), static_cast<float2*>(at(2)),
                static_cast<double2*>(at(3)), static_cast<double2*>(at(4))};
  after_user(h);
  h.prof.suspended = true;   // no profiling events inside this call
  try {
    apply_P_ws(h, reinterpret_cast<const double2*>(v), reinterpret_cast<double2*>(u), n_rhs, precision, w);
  } catch (...) {
    h.prof.suspended = false;
    throw;
  }
  h.prof.suspended = false;
  HIPCHECK(hipStreamSynchronize(h.stream));
  return HDP_OK;
  API_END
}

hdp_status hdp_local_solve(hdp_handle* H, const hdp_c64* y, hdp_c64* x, int32_t n_rhs) {
  API_BEGIN
  if (!H || !y || !x) fail(HDP_E_ARG, "null argument");
  Handle& h = H->h;
  if (n_rhs < 1) fail(HDP_E_ARG, "n_rhs out of range");
  after_user(h);
  launch_sep_solve(h, reinterpret_cast<const double2*>(y), reinterpret_cast<double2*>(x), n_rhs, h.stream);
  HIPCHECK(hipStreamSynchronize(h.stream));
  return HDP_OK;
  API_END
}

static void check_rhs(const Handle& h, const hdp_rhs* rhs) {
  if (!rhs) fail(HDP_E_ARG, "null rhs");
  if (rhs->n_rhs < 1 || rhs->n_rhs > h.max_rhs) fail(HDP_E_ARG, "n_rhs out of range");
  if (rhs->kind == HDP_RHS_POINT) {
    if (!rhs->points) fail(HDP_E_ARG, "points missing");
    for (int i = 0; i < 2 * rhs->n_rhs; ++i)
      if (!std::isfinite(rhs->points[i])) fail(HDP_E_ARG, "non-finite source point");
  } else if (rhs->kind == HDP_RHS_PLANE_WAVE_TOTAL || rhs->kind == HDP_RHS_PLANE_WAVE_SCATTERED) {
    if (!rhs->angles) fail(HDP_E_ARG, "angles missing");
    for (int i = 0; i < rhs->n_rhs; ++i)
      if (!std::isfinite(rhs->angles[i])) fail(HDP_E_ARG, "non-finite angle");
  } else if (rhs->kind == HDP_RHS_ELEMENT_LOADS) {
    if (!rhs->loads) fail(HDP_E_ARG, "element loads missing");
  } else {
    fail(HDP_E_ARG, "unknown rhs kind");
  }
}

// Loads of all RHS into full0 with stride Rp (zero-padded columns): packed
// non-zero element blocks are uploaded and scattered into a zeroed array.
static void load_rhs(Handle& h, const hdp_rhs* rhs, int Rp) {
  auto& d = h.d;
  hipStream_t s = h.stream;
  if (rhs->kind == HDP_RHS_ELEMENT_LOADS) {
    // caller's [dof][n_rhs] loads into the [dof][Rp] work array (padding zeroed)
    if (rhs->n_rhs < Rp) launch_fill_zero(d.full0, h.dof * Rp, s);
    HIPCHECK(hipMemcpy2DAsync(d.full0, size_t(Rp) * sizeof(double2), rhs->loads, size_t(rhs->n_rhs) * sizeof(double2),
                              size_t(rhs->n_rhs) * sizeof(double2), size_t(h.dof), hipMemcpyDeviceToDevice, s));
    return;
  }
  if (rhs->kind == HDP_RHS_PLANE_WAVE_TOTAL || rhs->kind == HDP_RHS_PLANE_WAVE_SCATTERED) {
    // computed on the device for the elements that carry a load
    const int kind = rhs->kind;
    if (d.pw_kind != kind) {
      std::vector<int> el;
      for (int e = 0; e < h.E; ++e)
        if (kind == HDP_RHS_PLANE_WAVE_TOTAL ? h.bmask[e] != 0 : h.eps[e] != 1.0) el.push_back(e);
      d.pw_elems = upload(h, el);
      d.n_pw_elems = int(el.size());
      d.pw_kind = kind;
    }
    // (pinned, read before the call that wrote it ends: nothing to wait for here)
    for (int r = 0; r < rhs->n_rhs; ++r) d.ang_host[r] = rhs->angles[r];
    HIPCHECK(hipMemcpyAsync(d.angles, d.ang_host, rhs->n_rhs * sizeof(double), hipMemcpyHostToDevice, s));
    launch_fill_zero(d.full0, h.dof * Rp, s);
    launch_plane_wave_loads(h, kind, d.pw_elems, d.n_pw_elems, d.angles, d.full0, rhs->n_rhs, Rp, s);
    return;
  }
  std::vector<int> elems;
  std::vector<cd> vals;
  compute_loads(h, rhs, Rp, elems, vals);
  int nb = int(elems.size());
  std::vector<int64_t> off(nb + 1, 0);
  for (int b = 0; b < nb; ++b) {
    int n = h.deg[elems[b]] + 1;
    off[b + 1] = off[b] + int64_t(n) * n * Rp;
  }
  size_t need_blocks = size_t(nb), need_vals = vals.size();
  if (need_blocks > h.load_cap_blocks || need_vals > h.load_cap_vals) {
    // staging grows on demand; freed with the handle
    h.load_cap_blocks = std::max(need_blocks, h.load_cap_blocks);
    h.load_cap_vals = std::max(need_vals, h.load_cap_vals);
    d.load_elems = dalloc<int>(h, h.load_cap_blocks);
    d.load_off = dalloc<int64_t>(h, h.load_cap_blocks + 1);
    d.load_vals = dalloc<double2>(h, h.load_cap_vals);
  }
  launch_fill_zero(d.full0, h.dof * Rp, s);
  if (nb) {
    std::vector<double2> pv(vals.size());
    for (size_t i = 0; i < vals.size(); ++i) pv[i] = make_double2(vals[i].real(), vals[i].imag());
    HIPCHECK(hipMemcpyAsync(d.load_elems, elems.data(), nb * sizeof(int), hipMemcpyHostToDevice, s));
    HIPCHECK(hipMemcpyAsync(d.load_off, off.data(), (nb + 1) * sizeof(int64_t), hipMemcpyHostToDevice, s));
    HIPCHECK(hipMemcpyAsync(d.load_vals, pv.data(), pv.size() * sizeof(double2), hipMemcpyHostToDevice, s));
    launch_block_scatter(d.load_elems, d.load_off, nb, d.dof_off, d.load_vals, d.full0, Rp, s);
  }
  HIPCHECK(hipStreamSynchronize(s));
}

hdp_status hdp_interface_rhs(hdp_handle* H, const hdp_rhs* rhs, hdp_c64* g) {
  API_BEGIN
  if (!H || !g) fail(HDP_E_ARG, "null argument");
  Handle& h = H->h;
  check_rhs(h, rhs);
  int R = rhs->n_rhs;
  after_user(h);
  load_rhs(h, rhs, R);
  interface_rhs(h, reinterpret_cast<double2*>(g), R);
  HIPCHECK(hipStreamSynchronize(h.stream));
  return HDP_OK;
  API_END
}

// The preconditioned residual (the stopping test) can reach tol while the true
// interface residual ||g - F nu|| / ||g|| stays large: rows of tiny scale (the
// decayed change of basis on hanging edges) dominate X^-1.  A solve whose true
// residual exceeds this bound is reported as HDP_W_TRUE_RESIDUAL.
static double true_residual_bound(double tol) { return std::max(1e3 * tol, 1e-6); }

static hdp_status solve_status(bool conv, bool true_ok) {
  if (!conv) return HDP_W_NOT_CONVERGED;
  return true_ok ? HDP_OK : HDP_W_TRUE_RESIDUAL;
}

struct SolveOut {
  int iters = 0, refinements = 0;
  double rel = 0, true_res = 0, t_rhs = 0, t_gmres = 0;
  bool conv = true, true_ok = true;
  std::chrono::steady_clock::time_point t_rec0;   // start of the recovery
};

// One solve of n_rhs systems: loads, interface right-hand side, GMRES (FP64 or
// GMRES-IR), true residual and recovery; leaves the element coefficients of the
// solutions in full1 ([dof][Rp], vertex basis) and nu in t2.  tail: the caller's own
// launches on the solution, issued before the host waits for the residual's norms.
static SolveOut solve_core(Handle& h, const hdp_rhs* rhs, int R, int Rp, const std::function<void()>& tail) {
  SolveOut o;
  auto& d = h.d;
  hipStream_t s = h.stream;
  auto t0 = std::chrono::steady_clock::now();
  auto ms_since = [](std::chrono::steady_clock::time_point a) {
    return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - a).count();
  };
  int64_t vs = int64_t(h.nlam) * Rp;
  load_rhs(h, rhs, Rp);
  interface_rhs(h, d.t0, Rp);                       // g
  HIPCHECK(hipStreamSynchronize(s));
  double t_rhs = ms_since(t0);
  auto tg = std::chrono::steady_clock::now();
  int iters = 0, refinements = 0;
  double rel = 0;
  bool conv = true;
  if (h.precision == HDP_FP64) {
    GmresResult gr = gmres(h, d.t0, d.t2, Rp, HDP_FP64, h.tol, h.max_iter);
    for (int r = 0; r < R; ++r) {
      iters = std::max(iters, gr.iters[r]);
      rel = std::max(rel, gr.rel[r]);
      if (gr.rel[r] > h.tol) conv = false;
    }
  } else {
    // GMRES-IR: inner GMRES on FP32 local operators, FP64 residual and update
    GmresDims gd = gmres_dims(h.nlam, Rp, h.max_iter + 1);
    HIPCHECK(hipMemsetAsync(d.t2, 0, size_t(vs) * sizeof(double2), s));
    apply_P(h, d.t0, d.w, Rp, HDP_FP64);
    launch_norms(d.w, nullptr, h.nlam, Rp, gd, d.npart, d.nrm, s);
    std::vector<double> s0(Rp);
    HIPCHECK(hipMemcpyAsync(d.nrm_host, d.nrm, Rp * sizeof(double), hipMemcpyDeviceToHost, s));
    HIPCHECK(hipStreamSynchronize(s));
    std::copy(d.nrm_host, d.nrm_host + Rp, s0.begin());
    HIPCHECK(hipMemcpyAsync(d.t1, d.t0, size_t(vs) * sizeof(double2), hipMemcpyDeviceToDevice, s));  // r = g
    double2* delta = nullptr;
    delta = d.full1;   // scratch of at least nlam * Rp (dof >= nlam)
    int budget = h.max_iter;
    conv = false;
    rel = 1.0;
    // inner tolerance: as far as the FP32 operator usefully goes on the first
    // pass, then only the reduction the outer residual still needs (on the
    // 32x32 point source a floor of 3e-7 took 185 iterations in all, 5e-8 took
    // 192 and 5e-9 took 200)
    const double floor32 = 3e-7;
    for (int outer = 0; outer < 30 && budget > 0; ++outer) {
      double inner = std::min(0.1, std::max(floor32, 0.5 * h.tol / std::max(rel, 1e-300)));
      GmresResult gr = gmres(h, d.t1, delta, Rp, HDP_MIXED, inner, budget);
      int used = 0;
      for (int r = 0; r < R; ++r) used = std::max(used, gr.iters[r]);
      iters += used;
      budget -= std::max(used, 1);
      ++refinements;
      launch_axpby(d.t2, delta, d.t2, vs, 1.0, 1.0, s);   // nu += delta
      apply_F(h, d.t2, d.t1, Rp, HDP_FP64);                // F nu
      launch_axpby(d.t0, d.t1, d.t1, vs, 1.0, -1.0, s);   // r = g - F nu
      apply_P(h, d.t1, d.w, Rp, HDP_FP64);
      launch_norms(d.w, nullptr, h.nlam, Rp, gd, d.npart, d.nrm, s);
      HIPCHECK(hipMemcpyAsync(d.nrm_host, d.nrm, Rp * sizeof(double), hipMemcpyDeviceToHost, s));
      HIPCHECK(hipStreamSynchronize(s));
      const double* sk = d.nrm_host;
      rel = 0;
      for (int r = 0; r < R; ++r) rel = std::max(rel, s0[r] > 0 ? sk[r] / s0[r] : 0.0);
      if (rel <= h.tol) { conv = true; break; }
    }
  }
  HIPCHECK(hipStreamSynchronize(s));
  double t_gmres = ms_since(tg);
  o.t_rec0 = std::chrono::steady_clock::now();
  // recovery phi = A^-1 (b^ - C^T nu) (Sec. 2.3.1)
  recover(h, d.full1, d.t2, Rp);
  // true interface residual ||g - F nu|| / ||g|| in FP64 (reported, not a stopping
  // test): g - F nu = C^ A^-1 (b^ - C^T nu), the constraint rows applied to the
  // recovered partially assembled solution, so one row gather of what the
  // recovery left (element values, coarse solution in wK) gives it
  double true_res = 0;
  {
    GmresDims gd = gmres_dims(h.nlam, Rp, h.max_iter + 1);
    {
      Timed t(h, KF_ROWGATHER, h.nslots * 16.0 * Rp + h.nlam * 16.0 * Rp, 0);
      launch_rowgather<double2>(h, d.full1, true, false, d.wK, d.t1, Rp, s);   // C_1 x_1 + C_2 x_2
    }
    launch_norms(d.t0, d.t1, h.nlam, Rp, gd, d.npart, d.nrm, s);
    HIPCHECK(hipMemcpyAsync(d.nrm_host, d.nrm, 2 * size_t(Rp) * sizeof(double), hipMemcpyDeviceToHost, s));
    tail();
    HIPCHECK(hipStreamSynchronize(s));
    const double *gn = d.nrm_host, *rn = gn + Rp;
    for (int r = 0; r < R; ++r) true_res = std::max(true_res, gn[r] > 0 ? rn[r] / gn[r] : 0.0);
  }
  o.iters = iters;
  o.refinements = refinements;
  o.rel = rel;
  o.conv = conv;
  o.true_res = true_res;
  o.true_ok = true_res <= true_residual_bound(h.tol);
  o.t_rhs = t_rhs;
  o.t_gmres = t_gmres;
  return o;
}

hdp_status hdp_solve(hdp_handle* H, const hdp_rhs* rhs, hdp_c64* field, int32_t n_far, const double* far_angles,
                     const uint8_t* far_inside, hdp_c64* far, hdp_stats* stats) {
  API_BEGIN
  if (!H) fail(HDP_E_ARG, "null handle");
  Handle& h = H->h;
  check_rhs(h, rhs);
  if (far && (n_far < 1 || !far_angles || !far_inside)) fail(HDP_E_ARG, "far-field arguments incomplete");
  auto t0 = std::chrono::steady_clock::now();
  auto& d = h.d;
  hipStream_t s = h.stream;
  int R = rhs->n_rhs, Rp = pow2ceil(R);
  h.t_launch = h.t_wait = 0;
  after_user(h);
  SolveOut so = solve_core(h, rhs, R, Rp, [&] {
    if (field) {
      Timed t(h, KF_GLL, 2.0 * h.dof * 16.0 * R, h.flops_gll * R);
      launch_gll(h, d.full1, reinterpret_cast<double2*>(field), Rp, h.dof, R, s);
    }
    if (far) {
      far_prepare(h, n_far, far_angles, far_inside, Rp);
      Timed t(h, KF_FAR, 0, 0);
      launch_far_field(h, d.full1, Rp, R, reinterpret_cast<double2*>(far), s);
    }
  });
  prof_flush(h);
  double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  if (stats) {
    hdp_get_stats(H, stats);
    stats->iterations = so.iters;
    stats->refinements = so.refinements;
    stats->rel_residual = so.rel;
    stats->solve_ms = ms;
    stats->rhs_ms = so.t_rhs;
    stats->gmres_ms = so.t_gmres;
    stats->gmres_launch_ms = h.t_launch;
    stats->gmres_wait_ms = h.t_wait;
    stats->recover_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - so.t_rec0).count();
    stats->true_residual = so.true_res;
  }
  return solve_status(so.conv, so.true_ok);
  API_END
}

hdp_status hdp_far_intensity_gradient(hdp_handle* H, double incidence, double far_angle, const uint8_t* far_inside,
                                      double* J, double* grad, hdp_stats* stats) {
  API_BEGIN
  if (!H) fail(HDP_E_ARG, "null handle");
  if (!far_inside || !J || !grad) fail(HDP_E_ARG, "null far_inside, J or grad");
  if (!std::isfinite(incidence) || !std::isfinite(far_angle)) fail(HDP_E_ARG, "non-finite angle");
  Handle& h = H->h;
  auto& d = h.d;
  hipStream_t s = h.stream;
  auto t0 = std::chrono::steady_clock::now();
  h.t_launch = h.t_wait = 0;
  if (!d.adj_u) {
    d.adj_u = dalloc<double2>(h, size_t(h.dof));
    d.adj_g = dalloc<double2>(h, size_t(h.dof));
    d.adj_grad = dalloc<double>(h, size_t(h.E));
    d.adj_E = dalloc<double2>(h, 1);
  }
  after_user(h);
  // forward: scattered field for the incidence, its far field E
  hdp_rhs fw{};
  fw.kind = HDP_RHS_PLANE_WAVE_SCATTERED;
  fw.n_rhs = 1;
  fw.angles = &incidence;
  double2 E;
  SolveOut so = solve_core(h, &fw, 1, 1, [&] {
    HIPCHECK(hipMemcpyAsync(d.adj_u, d.full1, size_t(h.dof) * sizeof(double2), hipMemcpyDeviceToDevice, s));
    far_prepare(h, 1, &far_angle, far_inside, 1);
    launch_far_field(h, d.full1, 1, 1, d.adj_E, s);
    HIPCHECK(hipMemcpyAsync(&E, d.adj_E, sizeof(double2), hipMemcpyDeviceToHost, s));
  });
  // adjoint: A lambda = dE/dphi with the same solver (A is complex symmetric).  The far
  // field is linear in the coefficients of the outside elements along Gamma,
  // E = sum_q c_q [(xhat.n') u(x_q) + (ik)^-1 d_n' u(x_q)], c_q = w_q e^{-ik xhat.x_q}.
  launch_far_adjoint(h, d.adj_g, s);
  hdp_rhs ad{};
  ad.kind = HDP_RHS_ELEMENT_LOADS;
  ad.n_rhs = 1;
  ad.loads = reinterpret_cast<const hdp_c64*>(d.adj_g);
  SolveOut sa = solve_core(h, &ad, 1, 1, [] {});
  launch_eps_gradient(h, d.adj_u, d.full1, E, incidence, d.adj_grad, s);
  HIPCHECK(hipMemcpyAsync(grad, d.adj_grad, size_t(h.E) * sizeof(double), hipMemcpyDeviceToHost, s));
  HIPCHECK(hipStreamSynchronize(s));
  prof_flush(h);
  *J = E.x * E.x + E.y * E.y;
  if (stats) {
    hdp_get_stats(H, stats);
    stats->iterations = so.iters;
    stats->refinements = so.refinements;
    stats->rel_residual = std::max(so.rel, sa.rel);
    stats->true_residual = std::max(so.true_res, sa.true_res);
    stats->solve_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    stats->rhs_ms = so.t_rhs;
    stats->gmres_ms = so.t_gmres + sa.t_gmres;
  }
  return solve_status(so.conv && sa.conv, so.true_ok && sa.true_ok);
  API_END
}

hdp_status hdp_residual_history(const hdp_handle* H, int32_t rhs, double* out, int32_t max, int32_t* count) {
  API_BEGIN
  if (!H || !count) fail(HDP_E_ARG, "null argument");
  const Handle& h = H->h;
  if (rhs < 0 || (h.last_hist_R && rhs >= h.last_hist_R)) fail(HDP_E_ARG, "rhs index out of range");
  *count = h.last_hist_len;
  for (int i = 0; i < h.last_hist_len && i < max && out; ++i) out[i] = h.last_hist[size_t(i) * h.last_hist_R + rhs];
  return HDP_OK;
  API_END
}

hdp_status hdp_autotune_table(const hdp_handle* H, hdp_tune_entry* out, int32_t max, int32_t* count) {
  API_BEGIN
  if (!H || !count) fail(HDP_E_ARG, "null handle or count");
  const Handle& h = H->h;
  *count = int32_t(h.tune.size());
  for (int32_t i = 0; i < std::min<int32_t>(max, *count); ++i) {
    std::memset(&out[i], 0, sizeof(out[i]));
    std::snprintf(out[i].kernel, sizeof(out[i].kernel), "%s", h.tune[size_t(i)].kernel.c_str());
    out[i].cols = h.tune[size_t(i)].cols;
    out[i].ms = h.tune[size_t(i)].ms;
    out[i].chosen = h.tune[size_t(i)].chosen ? 1 : 0;
  }
  return HDP_OK;
  API_END
}

hdp_status hdp_profile(hdp_handle* H, int32_t enable) {
  API_BEGIN
  if (!H) fail(HDP_E_ARG, "null handle");
  Handle& h = H->h;
  HIPCHECK(hipStreamSynchronize(h.stream));
  prof_flush(h);
  if (enable) {
    for (int f = 0; f < KF_COUNT; ++f) h.prof.ms[f] = h.prof.bytes[f] = h.prof.flops[f] = 0, h.prof.n[f] = 0;
  }
  h.prof.on = enable != 0;
  return HDP_OK;
  API_END
}

hdp_status hdp_profile_read(const hdp_handle* H, hdp_kernel_time* out, int32_t max, int32_t* count) {
  API_BEGIN
  if (!H || !count) fail(HDP_E_ARG, "null argument");
  const Handle& h = H->h;
  *count = KF_COUNT;
  for (int f = 0; f < KF_COUNT && f < max && out; ++f) {
    std::memset(&out[f], 0, sizeof(out[f]));
    std::strncpy(out[f].name, KF_NAMES[f], sizeof(out[f].name) - 1);
    out[f].launches = h.prof.n[f];
    out[f].total_ms = h.prof.ms[f];
    out[f].bytes = h.prof.bytes[f];
    out[f].flops = h.prof.flops[f];
  }
  return HDP_OK;
  API_END
}

void hdp_destroy(hdp_handle* H) {
  if (!H) return;
  (void)hipStreamSynchronize(H->h.stream);
  for (auto& p : H->h.prof.pend) {
    (void)hipEventDestroy(p.a);
    (void)hipEventDestroy(p.b);
  }
  for (auto e : H->h.prof.pool) (void)hipEventDestroy(e);
  if (H->h.d.status_host) (void)hipHostFree(H->h.d.status_host);
  for (auto& kv : H->h.graphs) (void)hipGraphExecDestroy(kv.second);
  if (H->h.order_ev) (void)hipEventDestroy(H->h.order_ev);
  if (H->h.stream) (void)hipStreamDestroy(H->h.stream);
  release_allocations(H->h);
  delete H;
}

const char* hdp_status_string(hdp_status s) {
  switch (s) {
    case HDP_OK: return "ok";
    case HDP_W_NOT_CONVERGED: return "not converged";
    case HDP_W_TRUE_RESIDUAL: return "true residual above bound";
    case HDP_E_ARG: return "invalid argument";
    case HDP_E_MESH: return "invalid mesh";
    case HDP_E_RESONANCE: return "element resonance";
    case HDP_E_COARSE: return "singular coarse matrix";
    case HDP_E_DEVICE: return "device error";
    case HDP_E_NOMEM: return "out of device memory";
    case HDP_E_UNSUPPORTED: return "unsupported input";
  }
  return "unknown status";
}

const char* hdp_last_error_detail(void) { return g_err.c_str(); }

}  // extern "C"
