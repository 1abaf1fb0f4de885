// Poisson solve on the free nodes (Eq. poisson with Eq. poisson_bc in the
// Galerkin form of App. B): Jacobi-preconditioned CG in the single-
// reduction (Chronopoulos-Gear) ordering, warm started, with the stopping
// test re-checked on the true residual, and the nodal field E = R phi.
//
// The solve is a chain of ordinary kernel launches (a launch costs ~3 us on
// MI355X, a device-wide barrier inside a persistent kernel 12-19 us):
//   resfield: one pass over phi: b on the fly, r = b - K phi, x = phi on
//             free nodes, E = R phi on every node, phi = 0 on Dirichlet
//             nodes; (b,b), (r,r)
//   start   : convergence test on that true residual; stats; when not
//             converged, u = D^-1 r, w = K u, (r,u), (w,u)
//   iter(i) : one iteration in one launch: its scalars, the p, s, x, r, u
//             updates and w = K u; (r,r), (r,u), (w,u); or in two, the updates
//             and the product (see jacobi_split)
//   scatter : phi = x on free nodes, before the re-check (a resfield pass)
// K and R share the sparsity of the free rows, so the field of phi comes out
// of the same pass that tests phi: when the warm start already meets the
// tolerance (no iteration), the step's solve is two launches, and whenever
// the solver stops, E belongs to the final phi.
// Each kernel writes one partial sum per workgroup; the next kernel reduces
// all partials in a fixed order in every workgroup (deterministic, same
// values everywhere), so no cross-workgroup synchronization is needed
// inside a kernel.  A control word in device memory carries the state
// (ITER, RECHECK, DONE, NOCONV); kernels whose state does not apply return
// at once, which lets the host launch iterations in batches.  The last
// kernel before each host wait also writes the state, with a sequence
// number, into host-mapped memory that the host polls.
//
// Storage is sliced ELLPACK (64 rows per slice, column-major in the slice):
// one row per lane, so every load of a wave is contiguous.  Slices are split
// into contiguous blocks per workgroup, grouped so that each of the 8 XCDs
// (workgroup g runs on XCD g mod 8) sweeps one contiguous eighth of the
// matrix, which keeps neighbour gathers in one L2.
#include "amg.h"

#include <algorithm>
#include <cstring>
#include <type_traits>
#include "common.h"
#include "solver.h"

namespace fp {

namespace {

struct Range {
  int64_t lo, hi;
};

__device__ inline Range my_range(int64_t n, VB vb) {
  const int G = vb.n;
  const int g = vb.id;
  int chunk = g;
  if ((G & 7) == 0) chunk = (g & 7) * (G >> 3) + (g >> 3);
  const int64_t per = (n + G - 1) / G;
  Range r;
  r.lo = (int64_t)chunk * per;
  if (r.lo > n) r.lo = n;
  r.hi = r.lo + per < n ? r.lo + per : n;
  return r;
}

// Deterministic block sum; result valid in every thread.
template <int NQ>
__device__ inline void block_sum(double (&v)[NQ]) {
  __shared__ double lds[NQ][16];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int nw = blockDim.x >> 6;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double x = v[q];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
    if (lane == 0) lds[q][wave] = x;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += lds[q][w];
    v[q] = s;
  }
  __syncthreads();
}

// Totals of partial sums written by the previous kernel: part[q*stride + j].
template <int NQ>
__device__ inline void totals(const double* part, int P, int stride,
                              double (&t)[NQ]) {
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double s = 0.0;
    for (int j = threadIdx.x; j < P; j += blockDim.x) s += part[q * stride + j];
    t[q] = s;
  }
  block_sum<NQ>(t);
}

template <int NQ>
__device__ inline void write_partials(double* part, int stride,
                                      double (&v)[NQ], VB vb) {
  block_sum<NQ>(v);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) part[q * stride + vb.id] = v[q];
  }
}

template <typename T>
__device__ inline const T* sell_val(const SellView& M) {
  if constexpr (std::is_same<T, float>::value) return M.val32;
  else return M.val;
}
template <typename T>
__device__ inline const T* sell_dict(const SellView& M) {
  if constexpr (std::is_same<T, float>::value) return M.dict32;
  else return M.dict;
}

// The table of a packed matrix in LDS (synchronizes; null when plain).
template <typename T>
__device__ inline const T* sell_table(const SellView& M) {
  if (!M.code) return nullptr;
  __shared__ T dict[kDictMax];
  const T* __restrict__ gd = sell_dict<T>(M);
  for (int k = threadIdx.x; k < kDictMax; k += blockDim.x) dict[k] = gd[k];
  __syncthreads();
  return dict;
}

// sum_j val_rj ev(ld(col_rj)) of this lane's row r of slice s, in the
// arithmetic of T and in entry order.  Up to eight entries per trip (slice
// widths are uniform across the wave): their words, then their gathers ld,
// are in flight together.  The packed form looks its values up in dict.
template <typename T, typename Lf, typename Vf>
__device__ inline T sell_sum(const SellView& M, const T* dict, int64_t s,
                             int lane, Lf&& ld, Vf&& ev) {
  using X = decltype(ld(0));
  const int32_t p0 = M.sptr[s], p1 = M.sptr[s + 1];
  T acc = T(0);
  if (dict) {
    const uint32_t* __restrict__ code = M.code;
    for (int32_t p = p0 + lane; p < p1; p += 8 * kSell) {
      const int32_t left = p1 - (p - lane);
      uint32_t c[8];
      X xv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (u * kSell < left) c[u] = code[p + u * kSell];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (u * kSell < left) xv[u] = ld((int32_t)(c[u] & ((1u << kColBits) - 1)));
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (u * kSell < left) acc += dict[c[u] >> kColBits] * ev(xv[u]);
    }
    return acc;
  }
  const int32_t* __restrict__ col = M.col;
  const T* __restrict__ val = sell_val<T>(M);
  for (int32_t p = p0 + lane; p < p1; p += 4 * kSell) {
    const int32_t left = p1 - (p - lane);
    int32_t c[4];
    T v[4];
    X xv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u * kSell < left) {
        c[u] = col[p + u * kSell];
        v[u] = val[p + u * kSell];
      }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u * kSell < left) xv[u] = ld(c[u]);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u * kSell < left) acc += v[u] * ev(xv[u]);
  }
  return acc;
}

// emit(r, sum_j val_rj ev(ld(col_rj))) for every row r of M in this
// workgroup's share (see sell_sum).
template <typename T, typename Lf, typename Vf, typename Ef>
__device__ inline void sell_rows(const SellView& M, int64_t nslices,
                                 int64_t nrows, VB vb, Lf&& ld, Vf&& ev,
                                 Ef&& emit) {
  const T* dict = sell_table<T>(M);
  const Range sl = my_range(nslices, vb);
  const int lane = threadIdx.x & (kSell - 1);
  for (int64_t s = sl.lo + threadIdx.x / kSell; s < sl.hi; s += blockDim.x / kSell) {
    const T acc = sell_sum<T>(M, dict, s, lane, ld, ev);
    const int64_t r = s * kSell + lane;
    if (r < nrows) emit(r, acc);
  }
}

// Record of one row in the Jacobi recursion: residual, w = K u, s, and the
// inverse diagonal.
template <typename T>
struct alignas(4 * sizeof(T)) CgRec {
  T r, w, s, d;
};

}  // namespace

// Partial-sum slots (each [G] doubles): 0 bb, 1 rr(resid), 2-3 start (ru, wu),
// 4-5 (rr, ru) of the even iterations, 6-7 of the odd, 8 and 9 (wu) alike.
__device__ inline double* slot(const CgArgs& a, int k) {
  return a.part + (size_t)k * a.G;
}

__device__ inline void ctrl_reset(CgCtrl* c) {
  CgCtrl z;
  z.state = CG_ITER;
  z.zero_rhs = 0;
  z.iters = 0;
  z.iters_final = 0;
  z.restarts = 0;
  z.bb = 0.0;
  z.relres = 0.0;
  z.rstart = 0.0;
  z.alpha[0] = z.alpha[1] = 0.0;
  z.gamma[0] = z.gamma[1] = 0.0;
  z.it_a = z.it_b = 0;
  z.rc_gate = z.pad = 0;
  z.stop[0] = z.stop[1] = 0;
  *c = z;
}

// Copy of the control state to host-mapped memory; the sequence number is
// stored last with system-scope release so the host sees a complete record.
__device__ inline void report(const CgCtrl* c, CgReport* r, int64_t seq,
                              int32_t state) {
  r->state = state;
  r->iters = state == CG_RECHECK ? c->iters_final : c->iters;
  __hip_atomic_store(&r->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The pass over phi (see the file comment).  reset != 0 starts a new solve
// (control word cleared by workgroup 0; no other workgroup reads it here).
// Bound: the matrix bytes, 36 per entry plain (77 us on the production tip,
// 278 MB of them) and 4 packed (33 us).
// FP32 field (e32): E = R phi in the difference form
//   E_i = sum_j R_ij (phi_j - phi_i) + S_i phi_i,   S_i = sum_j R_ij (FP64),
// with R in FP32: the differences are of the size of E h, so rounding R
// costs a relative error of about 2^-24 in E, while R_ij phi_j alone would
// lose the ratio |phi| / (|E| h) to cancellation.
// dev_gate (re-check passes only): run only if the recursion has stopped;
// workgroup 0 records the decision for the start pass that follows.
__device__ inline void k_cg_resfield_body(const CgArgs& a, int reset, VB vb,
                                          int dev_gate = 0) {
  if (dev_gate) {
    const bool on = a.ctrl->state == CG_RECHECK;
    if (vb.id == 0 && threadIdx.x == 0) a.ctrl->rc_gate = on ? 1 : 0;
    if (!on) return;
  }
  const DevMesh& m = a.m;
  if (reset && vb.id == 0 && threadIdx.x == 0) ctrl_reset(a.ctrl);
  if (reset && a.acc_rows)
    for (int k = vb.id; k < kStepCounters; k += vb.n) {
      step_counter_sum(a.acc_rows, a.acc_n, a.step_stats, k);
      __syncthreads();
    }
  const int lane = threadIdx.x & (kSell - 1);
  const int sub = threadIdx.x / kSell;
  const int nsub = blockDim.x / kSell;
  const bool withE = a.E != nullptr && !(reset && a.keep_field);
  const bool e32 = a.e32 != 0;
  const int64_t np = m.k_np;
  double v[2] = {0.0, 0.0};
  // packed: the table of (K, R) quadruples in LDS
  __shared__ double quad[4 * kDictMax];
  if (m.kr_code) {
    const double* __restrict__ gd = e32 ? m.kr_dict32 : m.kr_dict;
    for (int k = threadIdx.x; k < 4 * kDictMax; k += blockDim.x) quad[k] = gd[k];
    __syncthreads();
  }
  {
    const Range sl = my_range(m.k_nslices, vb);
    for (int64_t s = sl.lo + sub; s < sl.hi; s += nsub) {
      const int64_t r = s * kSell + lane;
      const bool row = r < m.n_free;
      const int32_t nd = row ? m.free2node[r] : 0;
      const double pi = row ? a.phi[nd] : 0.0;
      const int32_t p0 = m.k_sptr[s], p1 = m.k_sptr[s + 1];
      double kx = 0.0, ex = 0.0, ey = 0.0, ez = 0.0;
      // four entries per trip where the slice allows (uniform across the
      // wave): their loads are in flight together; sums in entry order
      int32_t p = p0 + lane;
      if (m.kr_code) {
        // eight entries per trip; the sums as below, in entry order
        for (; p < p1; p += 8 * kSell) {
          const int32_t left = p1 - (p - lane);
          uint32_t c[8];
          double xj[8];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (u * kSell < left) c[u] = m.kr_code[p + u * kSell];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (u * kSell < left) xj[u] = a.phi[c[u] & ((1u << kColBits) - 1)];
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (u * kSell < left) {
              const double* t = quad + 4 * (c[u] >> kColBits);
              kx += t[0] * xj[u];
              if (withE) {
                const double d = e32 ? xj[u] - pi : xj[u];
                ex += t[1] * d;
                ey += t[2] * d;
                ez += t[3] * d;
              }
            }
        }
      } else if (!withE) {
        for (; p + 3 * kSell < p1; p += 4 * kSell) {
          int32_t c[4];
          double kv[4], xj[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            c[u] = m.k_ncol[p + u * kSell];
            kv[u] = m.k_sval[p + u * kSell];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) xj[u] = a.phi[c[u]];
#pragma unroll
          for (int u = 0; u < 4; ++u) kx += kv[u] * xj[u];
        }
        for (; p < p1; p += kSell)
          kx += m.k_sval[p] * a.phi[m.k_ncol[p]];
      } else if (!e32) {
        for (; p + 3 * kSell < p1; p += 4 * kSell) {
          int32_t c[4];
          double kv[4], rx[4], ry[4], rz[4], xj[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int32_t q = p + u * kSell;
            c[u] = m.k_ncol[q];
            kv[u] = m.k_sval[q];
            rx[u] = m.r_sval[q];
            ry[u] = m.r_sval[np + q];
            rz[u] = m.r_sval[2 * np + q];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) xj[u] = a.phi[c[u]];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            kx += kv[u] * xj[u];
            ex += rx[u] * xj[u];
            ey += ry[u] * xj[u];
            ez += rz[u] * xj[u];
          }
        }
        for (; p < p1; p += kSell) {
          const double xj = a.phi[m.k_ncol[p]];
          kx += m.k_sval[p] * xj;
          ex += m.r_sval[p] * xj;
          ey += m.r_sval[np + p] * xj;
          ez += m.r_sval[2 * np + p] * xj;
        }
      } else {
        for (; p + 3 * kSell < p1; p += 4 * kSell) {
          int32_t c[4];
          double kv[4], xj[4];
          float rx[4], ry[4], rz[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int32_t q = p + u * kSell;
            c[u] = m.k_ncol[q];
            kv[u] = m.k_sval[q];
            rx[u] = m.r_sval32[q];
            ry[u] = m.r_sval32[np + q];
            rz[u] = m.r_sval32[2 * np + q];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) xj[u] = a.phi[c[u]];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            kx += kv[u] * xj[u];
            const double d = xj[u] - pi;
            ex += (double)rx[u] * d;
            ey += (double)ry[u] * d;
            ez += (double)rz[u] * d;
          }
        }
        for (; p < p1; p += kSell) {
          const double xj = a.phi[m.k_ncol[p]];
          kx += m.k_sval[p] * xj;
          const double d = xj - pi;
          ex += (double)m.r_sval32[p] * d;
          ey += (double)m.r_sval32[np + p] * d;
          ez += (double)m.r_sval32[2 * np + p] * d;
        }
      }
      if (!row) continue;
      double bi;
      if (a.rhs) {
        bi = a.rhs[r];
      } else if (a.b_saved) {
        bi = a.bprev[r];  // the same value, formed by the solve's first pass
      } else {
        const double c = a.charge ? (double)a.charge[nd] : 0.0;
        bi = a.coef * c + a.E0 * m.g_unit[r];
      }
      const double ri = bi - kx;
      a.x[r] = pi;
      if (a.bprev) a.bprev[r] = bi;
      a.r[r] = ri;  // (also kept for an incremental next pass)
      v[0] += bi * bi;
      v[1] += ri * ri;
      if (withE) {
        if (e32) {
          const double4 S = m.f_rowsum[nd];
          reinterpret_cast<float4*>(a.E)[nd] =
              make_float4((float)(ex + S.x * pi), (float)(ey + S.y * pi),
                          (float)(ez + S.z * pi), 0.0f);
        } else {
          reinterpret_cast<double4*>(a.E)[nd] = make_double4(ex, ey, ez, 0.0);
        }
      }
    }
  }
  // Dirichlet rows: phi = 0 there (never read above: columns are free
  // nodes), E = R phi
  {
    const Range dr = my_range(a.n_dir, vb);
    for (int64_t i = dr.lo + threadIdx.x; i < dr.hi; i += blockDim.x)
      a.phi[a.dir_nodes[i]] = 0.0;
  }
  if (withE) {
    const int64_t dnp = m.d_np;
    const Range sl = my_range(m.d_nslices, vb);
    for (int64_t s = sl.lo + sub; s < sl.hi; s += nsub) {
      const int64_t r = s * kSell + lane;
      const int32_t p0 = m.d_sptr[s], p1 = m.d_sptr[s + 1];
      double ex = 0.0, ey = 0.0, ez = 0.0;
      if (!e32) {
        for (int32_t p = p0 + lane; p < p1; p += kSell) {
          const double xj = a.phi[m.d_ncol[p]];
          ex += m.d_sval[p] * xj;
          ey += m.d_sval[dnp + p] * xj;
          ez += m.d_sval[2 * dnp + p] * xj;
        }
      } else {
        for (int32_t p = p0 + lane; p < p1; p += kSell) {
          const double xj = a.phi[m.d_ncol[p]];
          ex += (double)m.d_sval32[p] * xj;
          ey += (double)m.d_sval32[dnp + p] * xj;
          ez += (double)m.d_sval32[2 * dnp + p] * xj;
        }
      }
      if (r >= a.n_dir) continue;
      const int32_t nd = a.dir_nodes[r];
      if (e32)
        reinterpret_cast<float4*>(a.E)[nd] =
            make_float4((float)ex, (float)ey, (float)ez, 0.0f);
      else
        reinterpret_cast<double4*>(a.E)[nd] = make_double4(ex, ey, ez, 0.0);
    }
  }
  write_partials<2>(slot(a, 0), a.G, v, vb);
}

// First pass of a solve whose previous solve (same system, phi unchanged
// since) ended with the true residual r and right-hand side b_prev: r =
// (b - b_prev) + r, the same quantity as b - K phi without the product with
// K; x = phi, (b,b), (r,r) as in the full pass.  The field is
// that of phi already.
__device__ inline void k_cg_resinc_body(const CgArgs& a, VB vb) {
  const DevMesh& m = a.m;
  if (vb.id == 0 && threadIdx.x == 0) ctrl_reset(a.ctrl);
  if (a.acc_rows)
    for (int k = vb.id; k < kStepCounters; k += vb.n) {
      step_counter_sum(a.acc_rows, a.acc_n, a.step_stats, k);
      __syncthreads();
    }
  const Range rows = my_range(m.n_free, vb);
  double v[2] = {0.0, 0.0};
  for (int64_t i = rows.lo + threadIdx.x; i < rows.hi; i += blockDim.x) {
    const int32_t nd = m.free2node[i];
    const double c = a.charge ? (double)a.charge[nd] : 0.0;
    const double bi = a.coef * c + a.E0 * m.g_unit[i];
    const double ri = (bi - a.bprev[i]) + a.r[i];
    a.r[i] = ri;
    a.bprev[i] = bi;
    if (a.lean) {
      a.clear_charge[nd] = 0;  // (read above; b stays in bprev)
    } else {
      a.x[i] = a.phi[nd];
    }
    v[0] += bi * bi;
    v[1] += ri * ri;
  }
  if (a.lean) {
    // the Dirichlet nodes' charges (never part of b) cleared as well
    const Range dr = my_range(a.n_dir, vb);
    for (int64_t i = dr.lo + threadIdx.x; i < dr.hi; i += blockDim.x)
      a.clear_charge[a.dir_nodes[i]] = 0;
  }
  write_partials<2>(slot(a, 0), a.G, v, vb);
}

// D^-1 r of a row for the V-cycle, in its arithmetic: gathered on the way
// up the finest level in place of r and the diagonal.
__device__ inline void amg_put_z(const CgArgs& a, int64_t i, double ri) {
  if (a.amg32)
    ((float*)a.z)[i] = (float)ri * a.m.invdiag32[i];
  else
    ((double*)a.z)[i] = ri * a.m.invdiag[i];
}

// x of a lean first pass whose test asked for iterations.
__device__ inline void k_cg_prep_body(const CgArgs& a, VB vb) {
  const DevMesh& m = a.m;
  const Range rows = my_range(m.n_free, vb);
  for (int64_t i = rows.lo + threadIdx.x; i < rows.hi; i += blockDim.x) {
    a.x[i] = a.phi[m.free2node[i]];
    if (a.amg) amg_put_z(a, i, a.r[i]);
  }
}

// The stopping test on the recursive residual after it iterations of the
// current (re)start, whose (r,r) is rr (every workgroup decides alike).
__device__ inline bool recursion_stops(const CgArgs& a, const CgCtrl* c, int it,
                                       double rr) {
  const double bn = sqrt(c->bb);
  double thr = a.tol * (a.bref ? fmax(bn, *a.bref) : bn);
  if (a.mixed) thr = fmax(thr, a.inner_tol * c->rstart);
  return sqrt(rr) <= thr || c->iters + it >= a.max_iter;
}

// phi = x on the free nodes (before a re-check pass; dev_gate: only if the
// recursion has stopped).  The conditional form ends a round of iterations,
// so it also makes the stopping test that the next iteration would open
// with: a solve that needs just the iterations of its round ends in it.
__device__ inline void k_cg_scatter_body(const CgArgs& a, VB vb, int dev_gate = 0) {
  if (dev_gate) {
    CgCtrl* c = a.ctrl;
    const int32_t state = c->state;
    const int it = c->it_a;
    if (state == CG_DONE || state == CG_NOCONV) return;
    // (workgroup 0 may set RECHECK while others start: the same decision)
    double t[1] = {0.0};
    if (it > 0) totals<1>(slot(a, 4 + 2 * ((it - 1) & 1)), a.G, 1, t);
    if (state == CG_ITER) {
      if (it == 0 || !recursion_stops(a, c, it, t[0])) return;
      if (vb.id == 0 && threadIdx.x == 0) {
        c->state = CG_RECHECK;
        c->iters_final = c->iters + it;
      }
    }
  }
  const DevMesh& m = a.m;
  const Range rows = my_range(m.n_free, vb);
  // a Jacobi recursion that stopped after an even iteration has left its x to
  // the odd one (see cg_iter); the counters tell (no launch writes them here)
  const bool pending = !a.amg && a.ctrl->it_b > a.ctrl->it_a;
  const double alpha = a.ctrl->alpha[0];
  for (int64_t i = rows.lo + threadIdx.x; i < rows.hi; i += blockDim.x) {
    double x = a.x[i];
    if (pending) x += alpha * (a.mixed ? (double)((const float*)a.p)[i] : a.p[i]);
    a.phi[m.free2node[i]] = x;
  }
}

// u = D^-1 r at the (re)start of a Jacobi recursion, from the FP64 residual
// (rounded to FP32 in mixed precision).
template <typename T>
__device__ inline T start_u(const CgArgs& a, int64_t i) {
  return (T)(a.r[i] * a.m.invdiag[i]);
}

// The records of a (re)started Jacobi recursion: w = K u, s = 0 (u is not
// stored: it is D^-1 r); (r,u) and (w,u).
template <typename T>
__device__ inline void start_records(const CgArgs& a, VB vb) {
  const DevMesh& m = a.m;
  const T* __restrict__ d = std::is_same<T, float>::value ? (const T*)m.invdiag32
                                                          : (const T*)m.invdiag;
  CgRec<T>* __restrict__ out = (CgRec<T>*)a.rec0;
  double v[2] = {0.0, 0.0};
  sell_rows<T>(m.kz, m.k_nslices, m.n_free, vb,
               [&](int32_t c) { return start_u<T>(a, c); }, [](T x) { return x; },
               [&](int64_t i, T w) {
                 const T r = (T)a.r[i];
                 const T u = start_u<T>(a, i);
                 out[i] = CgRec<T>{r, w, T(0), d[i]};
                 v[0] += (double)r * (double)u;
                 v[1] += (double)w * (double)u;
               });
  write_partials<2>(slot(a, 2), a.G, v, vb);
}

// The same with the vectors u, w, s of an iteration in two launches.
__device__ inline void start_vectors(const CgArgs& a, VB vb) {
  const DevMesh& m = a.m;
  double v[2] = {0.0, 0.0};
  sell_rows<double>(m.kz, m.k_nslices, m.n_free, vb,
                    [&](int32_t c) { return start_u<double>(a, c); },
                    [](double x) { return x; },
                    [&](int64_t i, double w) {
                      const double u = start_u<double>(a, i);
                      a.u[i] = u;
                      a.w[i] = w;
                      v[0] += a.r[i] * u;
                      v[1] += w * u;
                    });
  write_partials<2>(slot(a, 2), a.G, v, vb);
}

__device__ inline void start_product(const CgArgs& a, VB vb) {
  if (a.split)
    start_vectors(a, vb);
  else if (a.mixed)
    start_records<float>(a, vb);
  else
    start_records<double>(a, vb);
}

// Convergence test on the true residual of the last resfield pass; when the
// solve ends, its statistics; when not converged, the first product w = K u
// of a (re)started CG.  Fields written here by workgroup 0 (state, iters,
// bb, relres, rstart, restarts) are never read by other workgroups of this
// launch; they read iters_final, which is stable here.  A zero right-hand
// side gives phi = 0 and E = 0, written by every workgroup.
// dev_gate 1: only where the resfield pass before it ran (rc_gate; the
// state itself is rewritten by workgroup 0 here); 2: the product only,
// after a lean first pass's test (state CG_ITER) and k_cg_prep; 3: the test
// of a lean first pass only (one workgroup).
__device__ inline void k_cg_start_body(const CgArgs& a, int64_t seq, VB vb,
                                       int dev_gate = 0) {
  CgCtrl* c = a.ctrl;
  if (dev_gate == 1 && !c->rc_gate) return;
  if (dev_gate == 2) {
    if (c->state == CG_ITER && !a.amg) start_product(a, vb);
    return;
  }
  double t[2];
  totals<2>(slot(a, 0), a.G, a.G, t);
  const double bn = sqrt(t[0]);
  const double rn = sqrt(t[1]);
  const int64_t done_iters = c->iters_final;
  const double bs = a.bref ? fmax(bn, *a.bref) : bn;
  const bool done = bn == 0.0 || rn <= a.tol * bs;
  const bool noconv = !done && done_iters >= a.max_iter;
  if (vb.id == 0 && threadIdx.x == 0) {
    c->bb = t[0];
    c->iters = done_iters;
    const double relres = bn > 0.0 ? rn / bn : 0.0;
    c->relres = relres;
    c->rstart = rn;
    const int32_t state = done ? CG_DONE : (noconv ? CG_NOCONV : CG_ITER);
    c->state = state;
    c->stop[0] = c->stop[1] = state != CG_ITER;
    c->it_a = 0;
    if (!done && !noconv) c->restarts += 1;
    if (bn == 0.0) c->zero_rhs = 1;
    if (done || noconv) {
      const int64_t st = noconv ? PIC_E_NOCONV : 0;
      if (a.stats) {
        a.stats->iters = done_iters;
        a.stats->status = st;
        a.stats->restarts = c->restarts;
        a.stats->relres = relres;
        a.stats->bnorm = bn;
      }
      if (a.step_stats) {
        a.step_stats->cg_iters = done_iters;
        a.step_stats->cg_relres = relres;
        if (st != 0 && a.step_stats->status == 0) a.step_stats->status = st;
      }
    }
    if (seq) {
      __threadfence_system();
      report(c, a.report, seq, state);
    }
  }
  if (bn == 0.0) {
    const DevMesh& m = a.m;
    // phi = 0 solves it; its residual (b = 0) is 0, which is what the next
    // solve's incremental first pass builds on
    const Range fr = my_range(m.n_free, vb);
    for (int64_t i = fr.lo + threadIdx.x; i < fr.hi; i += blockDim.x) a.r[i] = 0.0;
    const Range nr = my_range(m.n_nodes, vb);
    for (int64_t i = nr.lo + threadIdx.x; i < nr.hi; i += blockDim.x) {
      a.phi[i] = 0.0;
      if (a.E && a.e32)
        reinterpret_cast<float4*>(a.E)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      else if (a.E)
        reinterpret_cast<double4*>(a.E)[i] = make_double4(0.0, 0.0, 0.0, 0.0);
    }
  }
  if ((done || noconv) && a.next_stats) {
    // the start of the next step (as k_begin does it)
    if (vb.id == 0) {
      int64_t* s64 = reinterpret_cast<int64_t*>(a.next_stats);
      const int ns = (int)(sizeof(pic_step_stats) / sizeof(int64_t));
      if (threadIdx.x < ns) s64[threadIdx.x] = 0;
      int32_t* c32 = reinterpret_cast<int32_t*>(a.next_scratch);
      const int nc = (int)(sizeof(StepScratch) / sizeof(int32_t));
      static_assert(sizeof(StepScratch) / sizeof(int32_t) <= kCgBlock, "one word per thread");
      if (threadIdx.x < nc) c32[threadIdx.x] = 0;
      __syncthreads();
      if (threadIdx.x == 0) a.next_scratch->inj_base = *a.n_slots;
    }
    if (!a.b_saved) {  // (else the lean first pass cleared them)
      const Range cr = my_range(a.n_clear, vb);
      for (int64_t i = cr.lo + threadIdx.x; i < cr.hi; i += blockDim.x)
        a.clear_charge[i] = 0;
    }
  }
  if (done || noconv) return;
  if (dev_gate == 3) return;  // the test of a lean first pass only
  if (a.amg) {  // its iterations start with the V-cycle
    const Range rows = my_range(a.m.n_free, vb);
    for (int64_t i = rows.lo + threadIdx.x; i < rows.hi; i += blockDim.x)
      amg_put_z(a, i, a.r[i]);
    return;
  }
  start_product(a, vb);
}

// Iteration it (0-based since the last (re)start; par = it & 1) in one
// launch.  With the scalars of the previous sums, w = K u_new of row i needs
// u_new at its neighbours j, which only needs their old records:
//   s_j' = w_j + beta s_j,  r_j' = r_j - alpha s_j',  u_j' = d_j r_j',
// so every row forms its neighbours' u' again (three multiply-adds per
// entry on a 32-byte record out of L2) instead of waiting for a launch that
// writes it; the new records go to the other array.  The row-local part (p,
// x, (r,r), (r,u)) runs over even row ranges in a second loop, so that all
// sums keep the order, and all values the bits, of separate update and
// product launches.  x takes its share of two iterations in the odd one, which
// reads the direction of the even one anyway (the same sums in the same
// order): 8 bytes per row and iteration less.
// Bound: latency of the record gathers, then the Infinity Cache.  The first
// slice's words and records are in flight before the scalars are reduced, and
// the first rows of the row-local part before the products.
// An FP64 iteration on the production tip (515k rows, 60 MB) takes 16.3 us;
// an update launch and a product over all 15 entries per row took 14 + 19,
// this kernel without the early loads of the products 22, without those of
// the row-local part 17, with x in every iteration 16.5, with three waves per
// SIMD (136 registers) 22.
template <typename T, bool PK>
__device__ inline void cg_iter(const CgArgs& a, int par, VB vb) {
  CgCtrl* c = a.ctrl;
  if (c->stop[par]) {
    if (vb.id == 0 && threadIdx.x == 0) c->stop[par ^ 1] = 1;
    return;
  }
  const int it = par ? c->it_b : c->it_a;
  const DevMesh& m = a.m;
  const SellView& K = m.kz;
  const CgRec<T>* __restrict__ in = (const CgRec<T>*)(par ? a.rec1 : a.rec0);
  CgRec<T>* __restrict__ out = (CgRec<T>*)(par ? a.rec0 : a.rec1);
  const uint32_t* __restrict__ code = K.code;
  const int32_t* __restrict__ col = K.col;
  const T* __restrict__ val = sell_val<T>(K);
  constexpr uint32_t kMask = (1u << kColBits) - 1;
  constexpr int W = PK ? 8 : 4;   // entries in flight
  __shared__ T dict[PK ? kDictMax : 1];
  const int lane = threadIdx.x & (kSell - 1);
  const int nsub = blockDim.x / kSell;
  const Range sl = my_range(m.k_nslices, vb);
  int64_t s = sl.lo + threadIdx.x / kSell;
  // the first W entries of this lane's row
  uint32_t cw[W];
  T vv[W];
  CgRec<T> q[W], own;
  int32_t p = 0, left = 0;
  auto open = [&]() {
    const int32_t p0 = K.sptr[s];
    left = K.sptr[s + 1] - p0;
    p = p0 + lane;
    const int64_t r = s * kSell + lane;
    own = in[r < m.n_free ? r : m.n_free - 1];
#pragma unroll
    for (int u = 0; u < W; ++u)
      if (u * kSell < left) {
        cw[u] = PK ? code[p + u * kSell] : (uint32_t)col[p + u * kSell];
        if (!PK) vv[u] = val[p + u * kSell];
      }
#pragma unroll
    for (int u = 0; u < W; ++u)
      if (u * kSell < left) q[u] = in[PK ? cw[u] & kMask : cw[u]];
  };
  if (s < sl.hi) open();
  if (PK) {
    const T* __restrict__ gd = sell_dict<T>(K);
    for (int k = threadIdx.x; k < kDictMax; k += blockDim.x) dict[k] = gd[k];
  }
  double alpha, beta, gamma, a_prev = 0.0;
  if (it == 0) {
    double t[2];
    totals<2>(slot(a, 2), a.G, a.G, t);
    gamma = t[0];
    alpha = gamma / t[1];
    beta = 0.0;
  } else {
    const int pb = par ^ 1;
    double t[3];
    {
      const double* p2 = slot(a, 4 + 2 * pb);
      const double* p1 = slot(a, 8 + pb);
      t[0] = t[1] = t[2] = 0.0;
      for (int j = threadIdx.x; j < a.G; j += blockDim.x) {
        t[0] += p2[j];
        t[1] += p2[a.G + j];
        t[2] += p1[j];
      }
      block_sum<3>(t);
    }
    // it iterations done since the (re)start; c->iters is stable while
    // iterating, so every workgroup takes the same decision
    if (recursion_stops(a, c, it, t[0])) {
      if (vb.id == 0 && threadIdx.x == 0) {
        c->state = CG_RECHECK;
        c->stop[par ^ 1] = 1;
        c->iters_final = c->iters + it;
      }
      return;
    }
    const double g_prev = c->gamma[pb];
    a_prev = c->alpha[pb];
    gamma = t[1];
    beta = gamma / g_prev;
    alpha = gamma / (t[2] - beta * gamma / a_prev);
  }
  if (vb.id == 0 && threadIdx.x == 0) {
    c->gamma[par] = gamma;
    c->alpha[par] = alpha;
    (par ? c->it_a : c->it_b) = it + 1;
  }
  const T al = (T)alpha, be = (T)beta;
  auto step = [&](const CgRec<T>& o, T& sn, T& rn) {
    sn = o.w + be * o.s;
    rn = o.r - al * sn;
  };
  double v[3] = {0.0, 0.0, 0.0};
  // the row-local part's first rows are in flight during the products
  const bool first = it == 0;
  T* __restrict__ pv = (T*)a.p;
  double* __restrict__ x = a.x;
  const Range rows = my_range(m.n_free, vb);
  int64_t i = rows.lo + threadIdx.x;
  CgRec<T> o;
  T po = T(0);
  double xo = 0.0;
  auto fetch = [&]() {
    o = in[i];
    po = first ? start_u<T>(a, i) : pv[i];
    if (par) xo = x[i];
  };
  if (i < rows.hi) fetch();
  while (s < sl.hi) {
    T acc = T(0);
    auto add = [&](T k, const CgRec<T>& o) {
      T sj, rj;
      step(o, sj, rj);
      acc += k * (rj * o.d);
    };
#pragma unroll
    for (int u = 0; u < W; ++u)
      if (u * kSell < left) add(PK ? dict[cw[u] >> kColBits] : vv[u], q[u]);
    // longer rows: the rest four entries at a time (packed: one, to stay
    // within the registers of four waves per SIMD)
    for (int e = W; PK && e * kSell < left; ++e) {
      const uint32_t cu = code[p + e * kSell];
      add(dict[cu >> kColBits], in[cu & kMask]);
    }
    for (int e = W; !PK && e * kSell < left; e += 4) {
      uint32_t c[4];
      T k[4];
      CgRec<T> o[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if ((e + u) * kSell < left) {
          c[u] = (uint32_t)col[p + (e + u) * kSell];
          k[u] = val[p + (e + u) * kSell];
        }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if ((e + u) * kSell < left) o[u] = in[c[u]];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if ((e + u) * kSell < left) add(k[u], o[u]);
    }
    const int64_t r = s * kSell + lane;
    if (r < m.n_free) {
      T si, ri;
      step(own, si, ri);
      out[r] = CgRec<T>{ri, acc, si, own.d};
      v[2] += (double)acc * (double)(ri * own.d);
    }
    s += nsub;
    if (s < sl.hi) open();
  }
  while (i < rows.hi) {
    const T pi = first ? po : o.r * o.d + be * po;
    T si, ri;
    step(o, si, ri);
    pv[i] = pi;
    if (par) x[i] = (xo + a_prev * (double)po) + alpha * (double)pi;
    v[0] += (double)ri * (double)ri;
    v[1] += (double)ri * (double)(ri * o.d);
    i += blockDim.x;
    if (i < rows.hi) fetch();
  }
  block_sum<3>(v);
  if (threadIdx.x == 0) {
    slot(a, 4 + 2 * par)[vb.id] = v[0];
    slot(a, 5 + 2 * par)[vb.id] = v[1];
    slot(a, 8 + par)[vb.id] = v[2];
  }
}

__device__ inline void k_cg_iter_body(const CgArgs& a, int par, VB vb) {
  if (a.m.kz.code) {
    if (a.mixed)
      cg_iter<float, true>(a, par, vb);
    else
      cg_iter<double, true>(a, par, vb);
  } else {
    if (a.mixed)
      cg_iter<float, false>(a, par, vb);
    else
      cg_iter<double, false>(a, par, vb);
  }
}

// An iteration in two launches, the same operations in the same order: the
// update of p, s, x, r and u, then w = K u.  The update reads it_a and its
// stop word and writes it_b, the product the reverse.  Bound: the vectors'
// and the matrix's bytes.
__device__ inline void jacobi_update(const CgArgs& a, VB vb) {
  CgCtrl* c = a.ctrl;
  if (c->stop[0]) {
    if (vb.id == 0 && threadIdx.x == 0) c->stop[1] = 1;
    return;
  }
  const int it = c->it_a, par = it & 1;
  double alpha, beta, gamma;
  if (it == 0) {
    double t[2];
    totals<2>(slot(a, 2), a.G, a.G, t);
    gamma = t[0];
    alpha = gamma / t[1];
    beta = 0.0;
  } else {
    const int pb = par ^ 1;
    const double g_prev = c->gamma[pb], a_prev = c->alpha[pb];
    double t[2], tw[1];
    totals<2>(slot(a, 4 + 2 * pb), a.G, a.G, t);
    totals<1>(slot(a, 8 + pb), a.G, 1, tw);
    if (recursion_stops(a, c, it, t[0])) {
      if (vb.id == 0 && threadIdx.x == 0) {
        c->state = CG_RECHECK;
        c->stop[1] = 1;
        c->iters_final = c->iters + it;
      }
      return;
    }
    gamma = t[1];
    beta = gamma / g_prev;
    alpha = gamma / (tw[0] - beta * gamma / a_prev);
  }
  if (vb.id == 0 && threadIdx.x == 0) {
    c->gamma[par] = gamma;
    c->alpha[par] = alpha;
    c->it_b = it;
  }
  const double* __restrict__ d = a.m.invdiag;
  const Range rows = my_range(a.m.n_free, vb);
  const bool first = it == 0;
  double v[2] = {0.0, 0.0};
  for (int64_t i = rows.lo + threadIdx.x; i < rows.hi; i += blockDim.x) {
    const double pi = first ? a.u[i] : a.u[i] + beta * a.p[i];
    const double si = first ? a.w[i] : a.w[i] + beta * a.s[i];
    a.p[i] = pi;
    a.s[i] = si;
    a.x[i] += alpha * pi;
    const double ri = a.r[i] - alpha * si;
    a.r[i] = ri;
    const double ui = ri * d[i];
    a.u[i] = ui;
    v[0] += ri * ri;
    v[1] += ri * ui;
  }
  write_partials<2>(slot(a, 4 + 2 * par), a.G, v, vb);
}

__device__ inline void jacobi_product(const CgArgs& a, VB vb) {
  CgCtrl* c = a.ctrl;
  if (c->stop[1]) {
    if (vb.id == 0 && threadIdx.x == 0) c->stop[0] = 1;
    return;
  }
  const int it = c->it_b;
  if (vb.id == 0 && threadIdx.x == 0) c->it_a = it + 1;
  const DevMesh& m = a.m;
  const double* __restrict__ u = a.u;
  double v[1] = {0.0};
  sell_rows<double>(m.kz, m.k_nslices, m.n_free, vb,
                    [&](int32_t c) { return u[c]; }, [](double x) { return x; },
                    [&](int64_t i, double w) {
                      a.w[i] = w;
                      v[0] += w * u[i];
                    });
  write_partials<1>(slot(a, 8 + (it & 1)), a.G, v, vb);
}

// Single-instance kernels.
__global__ void __launch_bounds__(kCgBlock) k_cg_resfield(CgArgs a, int reset,
                                                         int dev_gate) {
  k_cg_resfield_body(a, reset, VB{(int)blockIdx.x, (int)gridDim.x}, dev_gate);
}
__global__ void __launch_bounds__(kCgBlock) k_cg_scatter(CgArgs a, int dev_gate) {
  k_cg_scatter_body(a, VB{(int)blockIdx.x, (int)gridDim.x}, dev_gate);
}
__global__ void __launch_bounds__(kCgBlock) k_cg_resinc(CgArgs a) {
  k_cg_resinc_body(a, VB{(int)blockIdx.x, (int)gridDim.x});
}
__global__ void __launch_bounds__(kCgBlock) k_cg_prep(CgArgs a) {
  k_cg_prep_body(a, VB{(int)blockIdx.x, (int)gridDim.x});
}
__global__ void __launch_bounds__(kCgBlock) k_cg_start(CgArgs a, int64_t seq,
                                                      int dev_gate) {
  k_cg_start_body(a, seq, VB{(int)blockIdx.x, (int)gridDim.x}, dev_gate);
}
template <typename T, bool PK>
__global__ void __launch_bounds__(kCgBlock, 4) k_cg_iter(CgArgs a, int par) {
  cg_iter<T, PK>(a, par, VB{(int)blockIdx.x, (int)gridDim.x});
}

__global__ void __launch_bounds__(kCgBlock) k_jacobi_update(CgArgs a) {
  jacobi_update(a, VB{(int)blockIdx.x, (int)gridDim.x});
}
__global__ void __launch_bounds__(kCgBlock) k_jacobi_product(CgArgs a) {
  jacobi_product(a, VB{(int)blockIdx.x, (int)gridDim.x});
}

__global__ void k_cg_report(CgArgs a, int64_t seq) {
  if (threadIdx.x != 0) return;
  __threadfence_system();
  report(a.ctrl, a.report, seq, a.ctrl->state);
}

// Batched kernels: block -> (instance, virtual block) by the schedule.
// gated (re-check launches): 1 skips the instances outside the mask, 2
// leaves the decision to each instance's state (conditional re-check).
__global__ void __launch_bounds__(kCgBlock) k_cg_resfield_b(CgBatch b, int reset,
                                                           int gated) {
  int i;
  const VB vb = batch_block(b.map, i);
  if (gated == 1 && !((b.mask >> i) & 1ull)) return;
  const CgArgs a = batch_args(b.args, i);
  k_cg_resfield_body(a, reset, vb, gated == 2);
}
__global__ void __launch_bounds__(kCgBlock) k_cg_resinc_b(CgBatch b) {
  int i;
  const VB vb = batch_block(b.map, i);
  const CgArgs a = batch_args(b.args, i);
  k_cg_resinc_body(a, vb);
}
__global__ void __launch_bounds__(kCgBlock) k_cg_scatter_b(CgBatch b, int gated) {
  int i;
  const VB vb = batch_block(b.map, i);
  if (gated == 1 && !((b.mask >> i) & 1ull)) return;
  const CgArgs a = batch_args(b.args, i);
  k_cg_scatter_body(a, vb, gated == 2);
}
// seq: as k_cg_start's, or 0
__global__ void __launch_bounds__(kCgBlock) k_cg_start_b(CgBatch b, int64_t seq, int gated) {
  int i;
  const VB vb = batch_block(b.map, i);
  if (gated == 1 && !((b.mask >> i) & 1ull)) return;
  const CgArgs a = batch_args(b.args, i);
  k_cg_start_body(a, seq, vb, gated == 2);
}
__global__ void __launch_bounds__(kCgBlock, 4) k_cg_iter_b(CgBatch b, int par) {
  int i;
  const VB vb = batch_block(b.map, i);
  const CgArgs a = batch_args(b.args, i);
  k_cg_iter_body(a, par, vb);
}
// One thread per instance: report the control state with sequence seq.
__global__ void k_cg_report_b(CgBatch b, int n, int64_t seq) {
  const int i = threadIdx.x;
  if (i >= n) return;
  const CgArgs& a = b.args[i];
  __threadfence_system();
  report(a.ctrl, a.report, seq, a.ctrl->state);
}

// ---------------------------------------------------------------------------
// CG preconditioned by one smoothed-aggregation V(1,1)-cycle (FP64).  Each
// iteration is [V-cycle u = M r, w = K u, update], the Chronopoulos-Gear
// recurrences being the same for any symmetric positive definite M.
// Partial-sum slots of parity p = it & 1: 4 + 2p (r,r) from the update,
// 5 + 2p (r,u) from the last V-cycle kernel, 8 + p (w,u) from the product.
// Counters: the V-cycle and the product read it_a, the product copies it to
// it_b, the update reads it_b and sets it_a = it_b + 1.  The first V-cycle
// kernel of every iteration after the first applies the stopping test to
// the recursive residual.  Every kernel returns at once unless the state is
// ITER.
// ---------------------------------------------------------------------------
namespace {

// sum over this lane's share of CSR row r (lpr lanes per row, this one sub):
// every lpr-th entry, up to eight per trip with their loads in flight
// together (a remainder summed one by one was a chain of loads per entry).
// The lanes past the row's end load nothing: with loads of the row's first
// entry in their place a level's way up on a moved 92^2 x 184 lattice took
// 124 us (a solve 14.6 ms, 13.6 so; of a 51^2 x 102 lattice 1.75 and 1.70).
template <typename T, typename Gf>
__device__ inline T csr_part(const SellMat& M, int64_t r, int sub, Gf&& g) {
  const int lpr = M.lpr;
  const T* __restrict__ val = sell_val<T>(M.v);
  const int32_t* __restrict__ col = M.v.col;
  const int32_t p1 = M.v.sptr[r + 1];
  T acc = 0;
  for (int32_t p = M.v.sptr[r] + sub; p < p1; p += 8 * lpr) {
    int32_t c[8];
    T v[8], xv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (p + u * lpr < p1) {
        c[u] = col[p + u * lpr];
        v[u] = val[p + u * lpr];
      }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (p + u * lpr < p1) xv[u] = g(c[u]);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (p + u * lpr < p1) acc += v[u] * xv[u];
  }
  return acc;
}

// emit(r, f(r, M's row sum over g, N's row sum over h)) for the rows of this
// workgroup's share; M and N have the same rows and lanes per row (N may be
// null: its sum is 0).  SELL (lpr = 1): one lane per row, see sell_sum.  CSR
// (lpr > 1): lpr lanes per row, f of the lanes' shares summed by a fixed
// shuffle tree (f is linear in the sums); every group of a workgroup makes
// the same number of trips, so the shuffles run on whole waves.
// gate() decides whether the launch does anything (false: nothing is
// emitted).  It is asked once the first rows' loads are under way, not
// ahead of them: the control word is written by another XCD just before,
// and waiting for it first cost every launch of a V-cycle close to 1 us.
// GB: the gate holds a barrier.
template <typename T, bool GB, typename Gf, typename Hf, typename Ff, typename Ef,
          typename Qf>
__device__ inline bool amg_rows(const SellMat& M, const SellMat* N, VB vb,
                                Gf&& g, Hf&& h, Ff&& f, Ef&& emit, Qf&& gate) {
  auto id = [](T v) { return v; };
  if (M.lpr == 1) {
    const T* dict = sell_table<T>(M.v);
    const Range sl = my_range(M.nslices, vb);
    const int lane = threadIdx.x & (kSell - 1);
    int64_t s = sl.lo + threadIdx.x / kSell;
    if (GB || s >= sl.hi) {
      if (!gate()) return false;
    }
    bool ask = !GB;
    for (; s < sl.hi; s += blockDim.x / kSell) {
      const int64_t r = s * kSell + lane;
      const T a = sell_sum<T>(M.v, dict, s, lane, g, id);
      const T b = N ? sell_sum<T>(N->v, (const T*)nullptr, s, lane, h, id) : T(0);
      if (ask) {
        if (!gate()) return false;
        ask = false;
      }
      if (r < M.nrows) emit(r, f(r, a, b));
    }
    return true;
  }
  const int lpr = M.lpr;
  const Range rows = my_range(M.nrows, vb);
  const int sub = threadIdx.x & (lpr - 1);
  const int grp = threadIdx.x / lpr, ngrp = blockDim.x / lpr;
  auto part = [&](int64_t r) {
    return r < rows.hi
               ? f(r, csr_part<T>(M, r, sub, g), N ? csr_part<T>(*N, r, sub, h) : T(0))
               : T(0);
  };
  T acc = part(rows.lo + grp);
  if (!gate()) return false;
  for (int64_t r0 = rows.lo; r0 < rows.hi; r0 += ngrp) {
    const int64_t r = r0 + grp;
    if (r0 > rows.lo) acc = part(r);
    for (int off = lpr >> 1; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, lpr);
    if (r < rows.hi && sub == 0) emit(r, acc);
  }
  return true;
}

// Vectors and diagonal of a level in the arithmetic of T.
template <typename T>
struct LevelVecs {
  const T* dinv;
  T *b, *t;
};
template <typename T>
__host__ __device__ inline LevelVecs<T> level_vecs(const AmgLevel& L) {
  if constexpr (std::is_same<T, float>::value)
    return LevelVecs<T>{L.invdiag32, L.b32, L.t32};
  else
    return LevelVecs<T>{L.invdiag, L.b, L.t};
}

}  // namespace

// Down a level: nb = Rs b, the next level's right-hand side.  On the finest
// level b is the CG residual (FP64; rounded once to T), and the launch opens
// with the stopping test.
template <typename T>
__device__ inline void amg_down_body(const CgArgs& a, const AmgLevel& L,
                                     int level, T* nb, VB vb) {
  CgCtrl* c = a.ctrl;
  const int32_t state = c->state;
  const double* __restrict__ r64 = a.r;
  const T* __restrict__ bl = level_vecs<T>(L).b;
  auto F = [](int64_t, T s, T) { return s; };
  auto put = [&](int64_t r, T v) { nb[r] = v; };
  if (level > 0) {
    auto B = [&](int32_t i) { return bl[i]; };
    amg_rows<T, false>(L.Rs, nullptr, vb, B, B, F, put, [&]() { return state == CG_ITER; });
    return;
  }
  // the partial sums of either parity, in flight ahead of the rows
  const int it = c->it_a;
  double t[2] = {0.0, 0.0};
  for (int j = threadIdx.x; j < a.G; j += blockDim.x) {
    t[0] += slot(a, 4)[j];
    t[1] += slot(a, 6)[j];
  }
  auto B = [&](int32_t i) { return (T)r64[i]; };
  amg_rows<T, true>(L.Rs, nullptr, vb, B, B, F, put, [&]() {
    block_sum<2>(t);
    if (state != CG_ITER) return false;
    if (it == 0 || !recursion_stops(a, c, it, t[(it - 1) & 1])) return true;
    if (vb.id == 0 && threadIdx.x == 0) {
      c->state = CG_RECHECK;
      c->iters_final = c->iters + it;
    }
    return false;
  });
}

// Coarsest level: x = M b with its dense matrix, one wave per row, eight
// entries per lane in flight.
template <typename T>
__device__ inline void amg_coarse_body(const CgArgs& a, int64_t n, const T* inv,
                                       const T* b, T* x, VB vb) {
  const int32_t state = a.ctrl->state;
  const Range rows = my_range(n, vb);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t i = rows.lo + wave; i < rows.hi; i += blockDim.x >> 6) {
    const T* __restrict__ m = inv + i * n;
    T s = 0;
    for (int64_t j0 = lane; j0 < n; j0 += 8 * 64) {
      T mv[8], bv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t j = j0 + 64 * u;
        mv[u] = j < n ? m[j] : T(0);
        bv[u] = j < n ? b[j] : T(0);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) s += mv[u] * bv[u];
    }
    if (state != CG_ITER) return;
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) x[i] = s;
  }
}

// Up a level: out = w D^-1 (2 b - w A D^-1 b) + Ps y, y the next level's
// result; on the finest level out is the CG vector u (FP64) and the
// workgroups write their share of (r,u).
template <typename T>
__device__ inline void amg_up_body(const CgArgs& a, const AmgLevel& L,
                                   int level, const T* __restrict__ y, VB vb) {
  const int32_t state = a.ctrl->state;
  const int it = a.ctrl->it_a;
  const LevelVecs<T> V = level_vecs<T>(L);
  const double* __restrict__ r64 = a.r;
  const T* __restrict__ bl = V.b;
  const T* __restrict__ dinv = V.dinv;
  const T omega = (T)L.omega;
  const T* __restrict__ z0 = (const T*)a.z;
  auto Z = [&](int64_t c) -> T { return level == 0 ? z0[c] : bl[c] * dinv[c]; };
  double v[1] = {0.0};
  const bool on = amg_rows<T, false>(
      L.A, &L.Ps, vb, [&](int32_t c) { return Z(c); },
      [&](int32_t c) { return y[c]; },
      [&](int64_t r, T ax, T py) { return py - (omega * omega) * (dinv[r] * ax); },
      [&](int64_t r, T s) {
        const T o = (T(2) * omega) * Z(r) + s;
        if (level == 0) {
          a.u[r] = (double)o;
          v[0] += r64[r] * (double)o;
        } else {
          V.t[r] = o;
        }
      },
      [&]() { return state == CG_ITER; });
  if (on && level == 0) write_partials<1>(slot(a, 5 + 2 * (it & 1)), a.G, v, vb);
}

// w = K u and (w,u); it_b = it_a.
__device__ inline void amg_spmv_body(const CgArgs& a, VB vb) {
  CgCtrl* c = a.ctrl;
  if (c->state != CG_ITER) return;
  const int it = c->it_a;
  if (vb.id == 0 && threadIdx.x == 0) c->it_b = it;
  const DevMesh& m = a.m;
  double v[1] = {0.0};
  const double* __restrict__ u = a.u;
  sell_rows<double>(m.kz, m.k_nslices, m.n_free, vb,
                    [&](int32_t c) { return u[c]; }, [](double v) { return v; },
                    [&](int64_t i, double s) {
                      a.w[i] = s;
                      v[0] += s * u[i];
                    });
  write_partials<1>(slot(a, 8 + (it & 1)), a.G, v, vb);
}

// Scalars of iteration it from (r,u) and (w,u), then p, s, x, r and (r,r);
// it_a = it + 1.
__device__ inline void amg_upd_body(const CgArgs& a, VB vb) {
  CgCtrl* c = a.ctrl;
  if (c->state != CG_ITER) return;
  const int it = c->it_b;
  const int pb = it & 1;
  const double g_prev = c->gamma[pb ^ 1], a_prev = c->alpha[pb ^ 1];
  double t[2] = {0.0, 0.0};
  for (int j = threadIdx.x; j < a.G; j += blockDim.x) {
    t[0] += slot(a, 5 + 2 * pb)[j];
    t[1] += slot(a, 8 + pb)[j];
  }
  // two rows per trip, the first trip's loads in flight ahead of the sums
  const Range rows = my_range(a.m.n_free, vb);
  const bool first = it == 0;
  double u[2], w[2], p[2], sv[2], x[2], r[2];
  auto fetch = [&](int64_t i0) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int64_t i = i0 + k * (int64_t)blockDim.x;
      if (i >= rows.hi) continue;
      u[k] = a.u[i];
      w[k] = a.w[i];
      x[k] = a.x[i];
      r[k] = a.r[i];
      if (!first) {
        p[k] = a.p[i];
        sv[k] = a.s[i];
      }
    }
  };
  const int64_t lo = rows.lo + threadIdx.x, step = 2 * (int64_t)blockDim.x;
  fetch(lo);
  block_sum<2>(t);
  const double gamma = t[0];
  double alpha, beta;
  if (first) {
    beta = 0.0;
    alpha = gamma / t[1];
  } else {
    beta = gamma / g_prev;
    alpha = gamma / (t[1] - beta * gamma / a_prev);
  }
  if (vb.id == 0 && threadIdx.x == 0) {
    c->gamma[pb] = gamma;
    c->alpha[pb] = alpha;
    c->it_a = it + 1;
  }
  double v[1] = {0.0};
  for (int64_t i0 = lo; i0 < rows.hi; i0 += step) {
    if (i0 > lo) fetch(i0);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int64_t i = i0 + k * (int64_t)blockDim.x;
      if (i >= rows.hi) continue;
      const double pi = first ? u[k] : u[k] + beta * p[k];
      const double si = first ? w[k] : w[k] + beta * sv[k];
      a.p[i] = pi;
      a.s[i] = si;
      a.x[i] = x[k] + alpha * pi;
      const double ri = r[k] - alpha * si;
      a.r[i] = ri;
      amg_put_z(a, i, ri);
      v[0] += ri * ri;
    }
  }
  write_partials<1>(slot(a, 4 + 2 * pb), a.G, v, vb);
}

// One instance: the level, matrix and vectors come as kernel arguments.
template <typename T>
__global__ void __launch_bounds__(kCgBlock) k_amg_down(CgArgs a, AmgLevel L,
                                                       int level, T* nb) {
  amg_down_body<T>(a, L, level, nb, VB{(int)blockIdx.x, (int)gridDim.x});
}
template <typename T>
__global__ void __launch_bounds__(kCgBlock) k_amg_coarse(CgArgs a, int64_t n,
                                                         const T* inv,
                                                         const T* b, T* x) {
  amg_coarse_body<T>(a, n, inv, b, x, VB{(int)blockIdx.x, (int)gridDim.x});
}
template <typename T>
__global__ void __launch_bounds__(kCgBlock) k_amg_up(CgArgs a, AmgLevel L,
                                                     int level, const T* y) {
  amg_up_body<T>(a, L, level, y, VB{(int)blockIdx.x, (int)gridDim.x});
}
__global__ void __launch_bounds__(kCgBlock) k_amg_spmv(CgArgs a) {
  amg_spmv_body(a, VB{(int)blockIdx.x, (int)gridDim.x});
}
__global__ void __launch_bounds__(kCgBlock) k_amg_upd(CgArgs a) {
  amg_upd_body(a, VB{(int)blockIdx.x, (int)gridDim.x});
}

// Several instances: block -> (instance, virtual block) by the schedule;
// each instance's hierarchy is read from the device copy of its AmgDev.
struct AmgBatch {
  const CgArgs* args;
  BatchMap map;
};

template <typename T>
__device__ inline T* coarse_vec(const AmgDev& D, int which) {
  if constexpr (std::is_same<T, float>::value)
    return global_ptr(which ? D.coarse_x32 : D.coarse_b32);
  else
    return global_ptr(which ? D.coarse_x : D.coarse_b);
}

template <typename T>
__global__ void __launch_bounds__(kCgBlock) k_amg_down_b(AmgBatch b, int level) {
  int i;
  const VB vb = batch_block(b.map, i);
  const CgArgs a = batch_args(b.args, i);
  const AmgDev* D = const_args((const AmgDev*)a.amg_dev);
  const AmgLevel L = batch_args(D->lv, level);
  T* nb = level + 1 < D->n_levels ? level_vecs<T>(batch_args(D->lv, level + 1)).b
                                  : coarse_vec<T>(*D, 0);
  amg_down_body<T>(a, L, level, nb, vb);
}
template <typename T>
__global__ void __launch_bounds__(kCgBlock) k_amg_up_b(AmgBatch b, int level) {
  int i;
  const VB vb = batch_block(b.map, i);
  const CgArgs a = batch_args(b.args, i);
  const AmgDev* D = const_args((const AmgDev*)a.amg_dev);
  const AmgLevel L = batch_args(D->lv, level);
  const T* y = level + 1 < D->n_levels ? level_vecs<T>(batch_args(D->lv, level + 1)).t
                                       : coarse_vec<T>(*D, 1);
  amg_up_body<T>(a, L, level, y, vb);
}
template <typename T>
__global__ void __launch_bounds__(kCgBlock) k_amg_coarse_b(AmgBatch b) {
  int i;
  const VB vb = batch_block(b.map, i);
  const CgArgs a = batch_args(b.args, i);
  const AmgDev* D = const_args((const AmgDev*)a.amg_dev);
  const T* inv;
  if constexpr (std::is_same<T, float>::value) inv = global_ptr(D->coarse_inv32);
  else inv = global_ptr(D->coarse_inv);
  amg_coarse_body<T>(a, D->n_coarse, inv, coarse_vec<T>(*D, 0),
                     coarse_vec<T>(*D, 1), vb);
}
__global__ void __launch_bounds__(kCgBlock) k_amg_spmv_b(AmgBatch b) {
  int i;
  const VB vb = batch_block(b.map, i);
  const CgArgs a = batch_args(b.args, i);
  amg_spmv_body(a, vb);
}
__global__ void __launch_bounds__(kCgBlock) k_amg_upd_b(AmgBatch b) {
  int i;
  const VB vb = batch_block(b.map, i);
  const CgArgs a = batch_args(b.args, i);
  amg_upd_body(a, vb);
}

namespace {

// The coarsest level's matrix and vectors in the arithmetic of T.
template <typename T>
struct CoarseVecs {
  const T* inv;
  T *b, *x;
};
template <typename T>
CoarseVecs<T> coarse_host(const AmgDev& d) {
  if constexpr (std::is_same<T, float>::value)
    return CoarseVecs<T>{d.coarse_inv32, d.coarse_b32, d.coarse_x32};
  else
    return CoarseVecs<T>{d.coarse_inv, d.coarse_b, d.coarse_x};
}

// Workgroups of a level kernel over the rows of M: one lane of work per
// thread (a row takes M.lpr lanes; the rows of a SELL slice share a lane
// column), at most the solver grid, so that the small coarse passes neither
// loop over row groups in one workgroup nor launch and drain hundreds of
// idle workgroups.  The finest level's way up keeps the solver grid (it also
// reduces over it).
int amg_grid(const CgArgs& a, int64_t lanes, int block) {
  // (rounded up to whole rounds of the XCDs: rounded down, a few rows make
  // every workgroup loop once more)
  const int64_t want = (lanes + block - 1) / block;
  const int64_t most = (int64_t)a.G * (kCgBlock / block);
  return (int)std::min<int64_t>(most, std::max<int64_t>(8, (want + 7) / 8 * 8));
}
int64_t lanes_of(const SellMat& M) { return M.nrows * (int64_t)M.lpr; }
// Threads of a level's workgroups: half as many below the finest level and in
// the dense coarsest one, whose hundred or two hundred workgroups of kCgBlock
// left CUs without one.  (The finest level's sum partials of the whole grid,
// each workgroup on its own.)  With the rounding above: an AMG solve a step at
// 40^2 x 80 4.19 -> 3.92 ms for five steps, an adjoint window at 32^2 x 64
// 17.6 -> 15.6 ms, a cold solve at 51^2 x 102 1.81 -> 1.73 ms.
constexpr int kAmgBlock = kCgBlock / 2;
int amg_block(int level) { return level > 0 ? kAmgBlock : kCgBlock; }
// one wave per row of the dense coarsest inverse
int coarse_grid(const CgArgs& a, int64_t n_coarse) {
  return amg_grid(a, n_coarse * 64, kAmgBlock);
}

template <typename T>
hipError_t amg_iters_t(const CgArgs& a, const AmgDev& d, int n, hipStream_t s) {
  const dim3 b(kCgBlock);
  const int L = d.n_levels;
  auto vec = [](const AmgLevel& lv) { return level_vecs<T>(lv); };
  const auto cv = coarse_host<T>(d);
  const int gc = coarse_grid(a, d.n_coarse);
  for (int k = 0; k < n; ++k) {
    for (int l = 0; l < L; ++l) {
      const AmgLevel& lv = d.lv[l];
      T* nb = l + 1 < L ? vec(d.lv[l + 1]).b : cv.b;
      hipLaunchKernelGGL(k_amg_down<T>, dim3(amg_grid(a, lanes_of(lv.Rs), amg_block(l))),
                         dim3(amg_block(l)), 0, s, a, lv, l, nb);
    }
    hipLaunchKernelGGL(k_amg_coarse<T>, dim3(gc), dim3(kAmgBlock), 0, s, a, d.n_coarse, cv.inv,
                       (const T*)cv.b, cv.x);
    for (int l = L - 1; l >= 0; --l) {
      const AmgLevel& lv = d.lv[l];
      const T* y = l + 1 < L ? vec(d.lv[l + 1]).t : cv.x;
      hipLaunchKernelGGL(k_amg_up<T>,
                         dim3(l == 0 ? a.G : amg_grid(a, lanes_of(lv.A), amg_block(l))),
                         dim3(amg_block(l)), 0, s, a, lv, l, y);
    }
    hipLaunchKernelGGL(k_amg_spmv, dim3(a.G), b, 0, s, a);
    hipLaunchKernelGGL(k_amg_upd, dim3(a.G), b, 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t amg_launch_iters(const CgArgs& a, const AmgDev& d, int n,
                            hipStream_t s) {
  return a.amg32 ? amg_iters_t<float>(a, d, n, s) : amg_iters_t<double>(a, d, n, s);
}

namespace {

// Schedule over the instances with on[i] and count(i) > 0 workgroups.
template <typename F>
BatchMap sched(const std::vector<char>& on, F&& count) {
  BatchMap m;
  std::memset(&m, 0, sizeof m);
  int j = 0;
  for (size_t i = 0; i < on.size(); ++i) {
    if (!on[i]) continue;
    const int c = count((int)i);
    if (c <= 0) continue;
    m.inst[j] = (int32_t)i;
    m.off[j + 1] = m.off[j] + c;
    ++j;
  }
  m.n_seg = j;
  return m;
}

template <typename T>
hipError_t amg_batch_t(const CgArgs* dargs, const std::vector<const CgArgs*>& hargs,
                       const std::vector<char>& on, int n, hipStream_t s) {
  const dim3 blk(kCgBlock);
  auto hier = [&](int i) -> const AmgDev& { return *(const AmgDev*)hargs[i]->amg; };
  int L = 0;
  for (size_t i = 0; i < on.size(); ++i)
    if (on[i]) L = std::max(L, hier((int)i).n_levels);
  BatchMap mA[kAmgMaxLevels], mR[kAmgMaxLevels];
  for (int l = 0; l < L; ++l) {
    mA[l] = sched(on, [&](int i) {
      const AmgDev& d = hier(i);
      return l >= d.n_levels ? 0 : l == 0 ? hargs[i]->G : amg_grid(*hargs[i], lanes_of(d.lv[l].A), amg_block(l));
    });
    mR[l] = sched(on, [&](int i) {
      const AmgDev& d = hier(i);
      return l >= d.n_levels ? 0 : amg_grid(*hargs[i], lanes_of(d.lv[l].Rs), amg_block(l));
    });
  }
  const BatchMap mC = sched(on, [&](int i) { return coarse_grid(*hargs[i], hier(i).n_coarse); });
  const BatchMap mG = sched(on, [&](int i) { return hargs[i]->G; });
  auto grid = [](const BatchMap& m) { return m.off[m.n_seg]; };
  auto B = [&](const BatchMap& m) { return AmgBatch{dargs, m}; };
  for (int k = 0; k < n; ++k) {
    for (int l = 0; l < L; ++l)
      if (grid(mR[l]))
        hipLaunchKernelGGL(k_amg_down_b<T>, dim3(grid(mR[l])), dim3(amg_block(l)), 0, s,
                           B(mR[l]), l);
    if (grid(mC))
      hipLaunchKernelGGL(k_amg_coarse_b<T>, dim3(grid(mC)), dim3(kAmgBlock), 0, s, B(mC));
    for (int l = L - 1; l >= 0; --l)
      if (grid(mA[l]))
        hipLaunchKernelGGL(k_amg_up_b<T>, dim3(grid(mA[l])), dim3(amg_block(l)), 0, s,
                           B(mA[l]), l);
    if (grid(mG)) {
      hipLaunchKernelGGL(k_amg_spmv_b, dim3(grid(mG)), blk, 0, s, B(mG));
      hipLaunchKernelGGL(k_amg_upd_b, dim3(grid(mG)), blk, 0, s, B(mG));
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t amg_batch_iters(const CgArgs* dargs, const std::vector<const CgArgs*>& hargs,
                           const std::vector<char>& on, int n, hipStream_t s) {
  int f32 = -1;
  for (size_t i = 0; i < on.size(); ++i) {
    if (!on[i]) continue;
    if (!hargs[i]->amg || !hargs[i]->amg_dev) return hipErrorInvalidValue;
    if (f32 >= 0 && f32 != hargs[i]->amg32) return hipErrorInvalidValue;
    f32 = hargs[i]->amg32;
  }
  if (f32 < 0 || n <= 0) return hipSuccess;
  return f32 ? amg_batch_t<float>(dargs, hargs, on, n, s)
             : amg_batch_t<double>(dargs, hargs, on, n, s);
}

#define LAUNCH(kern, ...)                                                   \
  do {                                                                      \
    hipLaunchKernelGGL(kern, dim3(a.G), dim3(kCgBlock), 0, s, __VA_ARGS__); \
    hipError_t e_ = hipGetLastError();                                      \
    if (e_ != hipSuccess) return e_;                                        \
  } while (0)

hipError_t cg_launch_begin(const CgArgs& a, int64_t seq, hipStream_t s) {
  const bool inc = a.incremental && !a.rhs && a.bprev;
  if (a.lean) {
    if (!inc || !a.next_stats || !a.charge ||
        (const int64_t*)a.clear_charge != a.charge)
      return hipErrorInvalidValue;
    LAUNCH(k_cg_resinc, a);
    // the test in one workgroup (no product to start)
    hipLaunchKernelGGL(k_cg_start, dim3(1), dim3(kCgBlock), 0, s, a, seq, 3);
    return hipGetLastError();
  }
  if (inc)
    LAUNCH(k_cg_resinc, a);
  else
    LAUNCH(k_cg_resfield, a, 1, 0);
  LAUNCH(k_cg_start, a, seq, 0);
  return hipSuccess;
}

hipError_t cg_launch_lean_iter(const CgArgs& a, hipStream_t s) {
  if (!a.lean) return hipErrorInvalidValue;
  LAUNCH(k_cg_prep, a);
  if (!a.amg) LAUNCH(k_cg_start, a, (int64_t)0, 2);
  return hipSuccess;
}

hipError_t cg_launch_report(const CgArgs& a, int64_t seq, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_report, dim3(1), dim3(64), 0, s, a, seq);
  return hipGetLastError();
}

hipError_t cg_launch_iters_dev(const CgArgs& a, int n, hipStream_t s) {
  if (n & 1) return hipErrorInvalidValue;
  if (a.split) {
    for (int k = 0; k < n; ++k) {
      LAUNCH(k_jacobi_update, a);
      LAUNCH(k_jacobi_product, a);
    }
    return hipSuccess;
  }
  const auto kern = a.m.kz.code
                        ? (a.mixed ? k_cg_iter<float, true> : k_cg_iter<double, true>)
                        : (a.mixed ? k_cg_iter<float, false> : k_cg_iter<double, false>);
  for (int k = 0; k < n; ++k) LAUNCH(kern, a, k & 1);
  return hipSuccess;
}

hipError_t cg_launch_recheck(const CgArgs& a, int64_t seq, hipStream_t s) {
  LAUNCH(k_cg_scatter, a, 0);
  LAUNCH(k_cg_resfield, a, 0, 0);
  LAUNCH(k_cg_start, a, seq, 0);
  return hipSuccess;
}

hipError_t cg_launch_recheck_if(const CgArgs& a, hipStream_t s) {
  LAUNCH(k_cg_scatter, a, 1);
  LAUNCH(k_cg_resfield, a, 0, 1);
  LAUNCH(k_cg_start, a, (int64_t)0, 1);
  return hipSuccess;
}

#define BLAUNCH(kern, ...)                                                    \
  do {                                                                        \
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kCgBlock), 0, s, __VA_ARGS__);  \
    hipError_t e_ = hipGetLastError();                                        \
    if (e_ != hipSuccess) return e_;                                          \
  } while (0)

hipError_t cg_batch_begin(const CgBatch& b, int grid, int incremental, int64_t seq,
                          hipStream_t s) {
  if (incremental)
    BLAUNCH(k_cg_resinc_b, b);
  else
    BLAUNCH(k_cg_resfield_b, b, 1, 0);
  BLAUNCH(k_cg_start_b, b, seq, 0);
  return hipSuccess;
}

hipError_t cg_batch_iters(const CgBatch& b, int grid, int n, hipStream_t s) {
  if (n & 1) return hipErrorInvalidValue;
  for (int k = 0; k < n; ++k) BLAUNCH(k_cg_iter_b, b, k & 1);
  return hipSuccess;
}

hipError_t cg_batch_recheck(const CgBatch& b, int grid, hipStream_t s) {
  BLAUNCH(k_cg_scatter_b, b, 1);
  BLAUNCH(k_cg_resfield_b, b, 0, 1);
  BLAUNCH(k_cg_start_b, b, (int64_t)0, 1);
  return hipSuccess;
}

hipError_t cg_batch_recheck_if(const CgBatch& b, int grid, hipStream_t s) {
  BLAUNCH(k_cg_scatter_b, b, 2);
  BLAUNCH(k_cg_resfield_b, b, 0, 2);
  BLAUNCH(k_cg_start_b, b, (int64_t)0, 2);
  return hipSuccess;
}

hipError_t cg_batch_report(const CgBatch& b, int n, int64_t seq, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_report_b, dim3(1), dim3(kMaxBatch), 0, s, b, n, seq);
  return hipGetLastError();
}

}  // namespace fp
