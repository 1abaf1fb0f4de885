// Particle side of the PIC cycle (Sec. II B 1-3): gather + leapfrog kick +
// drift + lateral wrap + absorption + neighbour-walk location + fixed-point
// deposition for the live particles; FN emission counts per face; injection
// of new particles; exact canonical location for the few particles the walk
// cannot certify.
//
// Particles are SoA arrays; every kernel runs a fixed grid-stride over the
// slot range read from device memory, so the host never waits for counts.
// Block b of the grid sweeps a contiguous slot range chosen so that the 8
// XCDs (block b runs on XCD b mod 8) each see one contiguous eighth of the
// slots; with particles sorted by tet, neighbouring tets then share an L2.
#include <type_traits>

#include "common.h"
#include "particles.h"
#include "solver.h"

namespace fp {

namespace {

constexpr int kMaxWalk = 256;
constexpr int kBlock = kParticleBlock;

struct Span {
  int64_t lo, hi;
};

// contiguous, XCD-grouped slot span of workgroup g of G
__device__ inline Span block_span(int64_t n, int G, int g) {
  int chunk = g;
  if ((G & 7) == 0) chunk = (g & 7) * (G >> 3) + (g >> 3);
  const int64_t per = (n + G - 1) / G;
  Span s;
  s.lo = (int64_t)chunk * per;
  s.hi = s.lo + per < n ? s.lo + per : n;
  if (s.lo > n) s.lo = n;
  return s;
}

// A launch gated on a solve whose outcome was not known when it was
// enqueued runs only if that solve has ended.
__device__ inline bool gate_closed(const int32_t* gate) {
  if (!gate) return false;
  const int32_t st = *gate;
  return st != CG_DONE && st != CG_NOCONV;
}

// Per-thread counters of one kernel, flushed once per block (a thread's
// counts fit 32 bits).
struct Acc {
  long long q_before, q_anode, q_after, q_cathode, q_inj;
  int n_before, n_anode, n_after, n_cathode, n_inj, walk_steps, walk_max;
};

__device__ inline void acc_zero(Acc& a) {
  a.q_before = a.q_anode = a.q_after = a.q_cathode = a.q_inj = 0;
  a.n_before = a.n_anode = a.n_after = a.n_cathode = a.n_inj = 0;
  a.walk_steps = a.walk_max = 0;
}

__device__ inline long long wave_sum(long long v) {
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ inline int wave_max(int v) {
  for (int off = 32; off >= 1; off >>= 1) {
    const int o = __shfl_xor(v, off, 64);
    v = o > v ? o : v;
  }
  return v;
}

// Block totals of the counters written to this block's row of the partials
// (no atomics: thousands of same-address atomics per step serialize); the
// stats kernel sums the rows at the end of the step.
__device__ inline void acc_flush(const Acc& a, int64_t* rows, int row,
                                 int stride) {
  __shared__ long long lds[kAccFields][kBlock / 64];
  const long long v[kAccFields] = {a.n_before, a.q_before, a.n_anode,
                                   a.q_anode,  a.n_after,  a.q_after,
                                   a.n_cathode, a.q_cathode, a.n_inj,
                                   a.q_inj,    a.walk_steps, a.walk_max};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < kAccFields; ++k) {
    long long s = v[k];
    if (k == kAccFields - 1) {
      s = wave_max((int)s);
    } else {
      s = wave_sum(s);
    }
    if (lane == 0) lds[k][wave] = s;
  }
  __syncthreads();
  if (threadIdx.x < kAccFields) {
    const int k = threadIdx.x;
    long long s = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w)
      s = k == kAccFields - 1 ? (lds[k][w] > s ? lds[k][w] : s) : s + lds[k][w];
    rows[(int64_t)k * stride + row] = s;  // field-major: coalesced sums
  }
}

// Nodal field at one node, widened to double when stored in float.
__device__ inline double4 ld_E(const void* E, int f32, int32_t node) {
  if (f32) {
    const float4 e = reinterpret_cast<const float4*>(E)[node];
    return make_double4(e.x, e.y, e.z, e.w);
  }
  return reinterpret_cast<const double4*>(E)[node];
}

// A tet's record in registers, from the mesh's 128-byte records or, where
// it has them, from the packed ones and the table of maps in LDS.  The two
// give the same bits everywhere; the kernels are compiled for either.
// Packed, the FP64 push needs fewer registers and gathers 17 words per
// particle where it gathered 28: see k_particles.
typedef __attribute__((address_space(3))) const double* lds_d;
typedef __attribute__((address_space(3))) const float* lds_f;

struct MapTable {
  double m[kMapMax * kMapLen];
};
struct MapTable32 : MapTable {  // with the FP32 maps of the mixed gather
  float m32[kMapMax * kMapLen];
};

// (the caller synchronizes)
__device__ inline void maps_load(const DevMesh& m, MapTable& M) {
  for (int k = threadIdx.x; k < kMapMax * kMapLen; k += blockDim.x) M.m[k] = m.maps[k];
}
__device__ inline void maps_load(const DevMesh& m, MapTable32& M) {
  maps_load(m, static_cast<MapTable&>(M));
  for (int k = threadIdx.x; k < kMapMax * kMapLen; k += blockDim.x) M.m32[k] = m.maps32[k];
}

template <bool PK>
struct Geo;

template <>
struct Geo<false> {
  TetGeom g;
  __device__ inline void load(const DevMesh& m, int t) { g = m.tg[t]; }
  __device__ inline const int32_t* node() const { return g.node; }
  __device__ inline void origin(double v[3]) const {
    v[0] = g.v0[0];
    v[1] = g.v0[1];
    v[2] = g.v0[2];
  }
  __device__ inline void map(const MapTable*, double r[9]) const {
#pragma unroll
    for (int k = 0; k < 9; ++k) r[k] = g.m[k];
  }
  // lam_c max_j |m_kj|
  __device__ inline double bound(const DevMesh& m, const MapTable*, int k) const {
    const double* r = g.m + 3 * (k - 1);
    return m.lam_c * fmax(fmax(fabs(r[0]), fabs(r[1])), fabs(r[2]));
  }
  // (selects, not an indexed load: the record stays in registers)
  __device__ inline uint32_t nbr(const DevMesh&, int, int f) const {
    return f == 0 ? g.nbr[0] : f == 1 ? g.nbr[1] : f == 2 ? g.nbr[2] : g.nbr[3];
  }
};

template <>
struct Geo<true> {
  double v0[3];
  uint32_t mp;
  int32_t nd[4];
  __device__ inline void load(const DevMesh& m, int t) {
    const TetPack* p = m.tc + t;
    v0[0] = p->v0[0];
    v0[1] = p->v0[1];
    v0[2] = p->v0[2];
    mp = p->map * kMapLen;
    const int4 n = *reinterpret_cast<const int4*>(p->node);
    nd[0] = n.x;
    nd[1] = n.y;
    nd[2] = n.z;
    nd[3] = n.w;
  }
  __device__ inline const int32_t* node() const { return nd; }
  __device__ inline void origin(double v[3]) const {
    v[0] = v0[0];
    v[1] = v0[1];
    v[2] = v0[2];
  }
  __device__ inline void map(const MapTable* M, double r[9]) const {
    const lds_d q = (lds_d)M->m + mp;
#pragma unroll
    for (int k = 0; k < 9; ++k) r[k] = q[k];
  }
  __device__ inline double bound(const DevMesh&, const MapTable* M, int k) const {
    return ((lds_d)M->m + mp)[8 + k];
  }
  __device__ inline uint32_t nbr(const DevMesh& m, int t, int f) const {
    return m.tc[t].nbr[f];
  }
};

// Barycentric coordinates of p in tet g (the fixed arithmetic of
// barycentric()).
template <bool PK>
__device__ inline void geo_lam(const Geo<PK>& g, const MapTable* M, double px,
                               double py, double pz, double lam[4]) {
  double v[3], r[9];
  g.origin(v);
  g.map(M, r);
  const double dx = px - v[0], dy = py - v[1], dz = pz - v[2];
  const double l1 = (r[0] * dx + r[1] * dy) + r[2] * dz;
  const double l2 = (r[3] * dx + r[4] * dy) + r[5] * dz;
  const double l3 = (r[6] * dx + r[7] * dy) + r[8] * dz;
  lam[0] = ((1.0 - l1) - l2) - l3;
  lam[1] = l1;
  lam[2] = l2;
  lam[3] = l3;
}

// Field at p inside tet g: sum_i lambda_i E_i in a fixed order.
template <bool PK>
__device__ inline void gather_field(const Geo<PK>& g, const MapTable* M,
                                    const void* E, double x, double y,
                                    double z, double& ex, double& ey,
                                    double& ez) {
  double lam[4];
  geo_lam<PK>(g, M, x, y, z, lam);
  const int32_t* nd = g.node();
  const double4 e0 = ld_E(E, 0, nd[0]);
  const double4 e1 = ld_E(E, 0, nd[1]);
  const double4 e2 = ld_E(E, 0, nd[2]);
  const double4 e3 = ld_E(E, 0, nd[3]);
  ex = ((lam[0] * e0.x + lam[1] * e1.x) + lam[2] * e2.x) + lam[3] * e3.x;
  ey = ((lam[0] * e0.y + lam[1] * e1.y) + lam[2] * e2.y) + lam[3] * e3.y;
  ez = ((lam[0] * e0.z + lam[1] * e1.z) + lam[2] * e2.z) + lam[3] * e3.z;
}

// Cell field of a tet (cell mode): E = -(grad phi)_t with grad lambda_k the
// rows m_k (k = 1..3) and grad lambda_0 = -(m_1 + m_2 + m_3), summed in a
// fixed order.
template <bool PK>
__device__ inline void cell_field(const Geo<PK>& g, const MapTable* M,
                                  const double* phi, double& ex, double& ey,
                                  double& ez) {
  const int32_t* nd = g.node();
  const double p0 = phi[nd[0]], p1 = phi[nd[1]], p2 = phi[nd[2]], p3 = phi[nd[3]];
  double r[9], e[3];
  g.map(M, r);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double g0 = -((r[k] + r[3 + k]) + r[6 + k]);
    e[k] = -(((p0 * g0 + p1 * r[k]) + p2 * r[3 + k]) + p3 * r[6 + k]);
  }
  ex = e[0];
  ey = e[1];
  ez = e[2];
}

// The cell field of an emitting face's tet.
__device__ inline void face_cell_field(const DevMesh& m, int t, const double* phi,
                                       double& ex, double& ey, double& ez) {
  Geo<false> g;
  g.load(m, t);
  cell_field<false>(g, nullptr, phi, ex, ey, ez);
}

// A place in a queue for every lane that calls (one atomic per wave).
__device__ inline int queue_slot(int32_t* count) {
  const unsigned long long here = __ballot(1);
  const int lane = threadIdx.x & 63;
  const int lead = __ffsll((long long)here) - 1;
  int base = 0;
  if (lane == lead) base = atomicAdd(count, __popcll(here));
  base = __shfl(base, lead, 64);
  return base + __popcll(here & ((1ull << lane) - 1));
}

__device__ inline void deposit_one(const TetGeom& g, double x, double y,
                                   double z, double w, int64_t* charge) {
  double lam[4];
  barycentric(g, x, y, z, lam);
  int64_t q[4];
  charge_split(lam, w, q);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    atomicAdd(reinterpret_cast<unsigned long long*>(charge + g.node[k]),
              (unsigned long long)q[k]);
}

// The seed tet of p's bucket (lowest-index tet whose centroid lies in the
// bucket), or -1: a walk start within about one cell of p.
__device__ inline int bucket_guess(const DevMesh& m, double x, double y,
                                   double z) {
  if (!(x >= m.b0[0] && x <= m.b1[0] && y >= m.b0[1] && y <= m.b1[1] &&
        z >= m.b0[2] && z <= m.b1[2]))
    return -1;
  const int bx = bucket_axis(x, m.b0[0], m.binv[0], m.nb[0]);
  const int by = bucket_axis(y, m.b0[1], m.binv[1], m.nb[1]);
  const int bz = bucket_axis(z, m.b0[2], m.binv[2], m.nb[2]);
  const int64_t id = ((int64_t)bx * m.nb[1] + by) * m.nb[2] + bz;
  return m.bseed[id];
}

// The fine-grid seed of p (the tet holding the centre of p's sub-cell).
__device__ inline int fine_seed(const DevMesh& m, double x, double y,
                                double z) {
  if (!(x >= m.b0[0] && x <= m.b1[0] && y >= m.b0[1] && y <= m.b1[1] &&
        z >= m.b0[2] && z <= m.b1[2]))
    return -1;
  const int bx = bucket_axis(x, m.b0[0], m.finv[0], m.fnb[0]);
  const int by = bucket_axis(y, m.b0[1], m.finv[1], m.fnb[1]);
  const int bz = bucket_axis(z, m.b0[2], m.finv[2], m.fnb[2]);
  return m.fseed[((int64_t)bx * m.fnb[1] + by) * m.fnb[2] + bz];
}

// Barycentric coordinates of p in tet g (the fixed arithmetic of
// barycentric()) with a certificate.  With d = p - v0 and
// M_k = max_j |m_kj|, each computed lambda_k (k = 1..3) lies within
// B_k = lam_c M_k |d|_1 of the exact barycentric coordinate of p in the tet
// of the exact vertices (lam_c bounds the rounding of the stored map, of d
// and of the dot product; it is set up with the mesh), and lambda_0 within
// B_0 = 3.01 u (1 + sum_k |lambda_k|) + sum_k B_k.  Returns true when every
// lambda_k > B_k, i.e. p is certainly strictly inside.  Otherwise exitf is
// the face (opposite vertex k) with the most negative lambda_k among those
// certainly negative (lambda_k < -B_k), or -1 when there is none.
template <bool PK>
__device__ inline bool lam_test(const DevMesh& m, const Geo<PK>& g,
                                const MapTable* M, double x, double y, double z,
                                double lam[4], int& exitf) {
  geo_lam<PK>(g, M, x, y, z, lam);
  double v[3];
  g.origin(v);
  const double dx = x - v[0], dy = y - v[1], dz = z - v[2];
  const double dn = (fabs(dx) + fabs(dy)) + fabs(dz);
  double B[4];
#pragma unroll
  for (int k = 1; k < 4; ++k) B[k] = g.bound(m, M, k) * dn;
  B[0] = 3.01 * 1.1102230246251565e-16 *
             (((1.0 + fabs(lam[1])) + fabs(lam[2])) + fabs(lam[3])) +
         1.0001 * ((B[1] + B[2]) + B[3]);
  bool inside = true;
  exitf = -1;
  double worst = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (lam[k] > B[k]) continue;
    inside = false;
    if (lam[k] < -B[k] && lam[k] < worst) {
      worst = lam[k];
      exitf = k;
    }
  }
  return inside;
}

// Neighbour walk from tet t with the point's frame offset (sx, sy) relative
// to t; G holds the record of t on entry.  A point that moved far (far =
// true), or is not in t, restarts from the fine-grid seed of its sub-cell.
// Returns the tet when the point is certified strictly inside it in its own
// frame (then no other tet holds it, so it is the canonical answer), with
// lam its barycentric coordinates there and G its record, or -1 when the
// exact bucket scan must decide.
template <bool PK>
__device__ inline int walk(const DevMesh& m, const MapTable* M, double x,
                           double y, double z, int t, int sx, int sy,
                           int& steps, bool far, Geo<PK>& G, double lam[4],
                           bool have_G = true) {
  bool jumped = false;
  for (steps = 0; steps < kMaxWalk; ++steps) {
    bool reload = steps > 0 || !have_G;
    if (!jumped && (far || steps == 1)) {
      jumped = true;
      int g = fine_seed(m, x, y, z);
      if (g < 0) g = bucket_guess(m, x, y, z);
      if (g >= 0 && !(g == t && sx == 0 && sy == 0)) {
        t = g;
        sx = 0;
        sy = 0;
        reload = true;
      }
    }
    if (reload) G.load(m, t);
    int exitf;
    if (lam_test<PK>(m, G, M, x + (double)sx * m.Lx, y + (double)sy * m.Ly, z,
                     lam, exitf))
      return (sx == 0 && sy == 0) ? t : -1;
    if (exitf < 0) return -1;
    const uint32_t nb = G.nbr(m, t, exitf);
    if ((nb & kNoNbr) == kNoNbr) return -1;
    sx += (int)((nb >> 28) & 3u) - 1;
    sy += (int)(nb >> 30) - 1;
    t = (int)(nb & kNoNbr);
  }
  return -1;
}

// Canonical location by exact predicates over the bucket's candidates
// (listed in ascending tet order, so the first hit is the lowest index).
__device__ int scan_locate(const DevMesh& m, double x, double y, double z) {
  if (!(x >= m.b0[0] && x <= m.b1[0] && y >= m.b0[1] && y <= m.b1[1] &&
        z >= m.b0[2] && z <= m.b1[2]))
    return -1;
  const int bx = bucket_axis(x, m.b0[0], m.binv[0], m.nb[0]);
  const int by = bucket_axis(y, m.b0[1], m.binv[1], m.nb[1]);
  const int bz = bucket_axis(z, m.b0[2], m.binv[2], m.nb[2]);
  const int64_t id = ((int64_t)bx * m.nb[1] + by) * m.nb[2] + bz;
  const double p[3] = {x, y, z};
  for (int q = m.bstart[id]; q < m.bstart[id + 1]; ++q) {
    const int t = m.bitem[q];
    const double* v = m.tw[t].v;
    if (vol6_sign(p, v + 3, v + 6, v + 9) < 0) continue;
    if (vol6_sign(v, p, v + 6, v + 9) < 0) continue;
    if (vol6_sign(v, v + 3, p, v + 9) < 0) continue;
    if (vol6_sign(v, v + 3, v + 6, p) < 0) continue;
    return t;
  }
  return -1;
}

// Whether the closed tet with vertices v holds p: no face sees p on its far
// side.  The four signs are filtered first and the exact predicate -- a long
// chain of dependent FP64 operations -- runs once per undecided sign, in one
// place: a point on a face, the usual case here, has one, where four
// predicates in a row cost a wave the exact path at each of them (the fallback
// launch of a mixed-precision step: 11.9 -> 9.8 us).
__device__ inline bool tet_holds(const double* v, const double p[3]) {
  double A[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) A[c] = v[c];
  unsigned open = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    double B[12], bound;
#pragma unroll
    for (int c = 0; c < 12; ++c) B[c] = c / 3 == k ? p[c % 3] : A[c];
    const double det = vol6_filtered(B, B + 3, B + 6, B + 9, bound);
    if (-det > bound) return false;
    if (!(det > bound)) open |= 1u << k;
  }
  while (open) {
    const int k = __ffs((int)open) - 1;
    open &= open - 1u;
    double B[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) B[c] = c / 3 == k ? p[c % 3] : A[c];
    if (vol6_sign_exact(B, B + 3, B + 6, B + 9) < 0) return false;
  }
  return true;
}

// The same canonical location with the 64 lanes of a wave testing 64
// candidates at a time (the point is uniform across the wave; every lane
// must call it).  The lowest lane holding the point gives the lowest index.
__device__ int scan_locate_wave(const DevMesh& m, double x, double y,
                                double z) {
  if (!(x >= m.b0[0] && x <= m.b1[0] && y >= m.b0[1] && y <= m.b1[1] &&
        z >= m.b0[2] && z <= m.b1[2]))
    return -1;
  const int bx = bucket_axis(x, m.b0[0], m.binv[0], m.nb[0]);
  const int by = bucket_axis(y, m.b0[1], m.binv[1], m.nb[1]);
  const int bz = bucket_axis(z, m.b0[2], m.binv[2], m.nb[2]);
  const int64_t id = ((int64_t)bx * m.nb[1] + by) * m.nb[2] + bz;
  const double p[3] = {x, y, z};
  const int lane = threadIdx.x & 63;
  const int q1 = m.bstart[id + 1];
  for (int base = m.bstart[id]; base < q1; base += 64) {
    const int q = base + lane;
    bool hit = false;
    if (q < q1) {
      const double* v = m.tw[m.bitem[q]].v;
      hit = tet_holds(v, p);
    }
    const unsigned long long mask = __ballot(hit);
    if (mask) return m.bitem[base + __ffsll((long long)mask) - 1];
  }
  return -1;
}

// After the drift: wrap, absorb at the anode, locate, deposit.
// Per-workgroup node-charge table in LDS (open addressing on the node id).
// Particles of one workgroup share few nodes, so accumulating their int64
// charges here and flushing one global atomic per distinct node removes
// the same-address contention of per-particle global atomics.  Integer
// addition is exact and order-free, so the result is unchanged.
constexpr int kTable = 2048;  // > 4 nodes x the particles of one block

struct ChargeTable {
  int32_t key[kTable];
  unsigned long long val[kTable];
  // the workgroup's absorbed superparticles (rare: kept out of the threads'
  // registers)
  unsigned long long n_anode, q_anode;
};

__device__ inline void table_clear(ChargeTable& T) {
  for (int k = threadIdx.x; k < kTable; k += blockDim.x) {
    T.key[k] = -1;
    T.val[k] = 0ull;
  }
  if (threadIdx.x == 0) T.n_anode = T.q_anode = 0ull;
  __syncthreads();
}

// 64-bit add into LDS.  The table reaches the helpers by reference, and
// through it the compiler emits a generic (flat) atomic, which takes the
// vector-memory path; the explicit LDS address space gives ds_add_u64.
__device__ inline void lds_add_u64(unsigned long long* p, unsigned long long v) {
  __atomic_fetch_add((__attribute__((address_space(3))) unsigned long long*)p, v,
                     __ATOMIC_RELAXED);
}

__device__ inline void table_add(ChargeTable& T, int32_t node, int64_t q,
                                 int64_t* charge) {
  uint32_t h = ((uint32_t)node * 2654435761u) >> 21;  // 11 bits
  // kept as a loop: unrolled at every inlined call site, the 64 probes
  // made the particle kernel tens of thousands of instructions long (an
  // instruction-cache and scalar-register-spill cost paid by every wave)
#pragma unroll 1
  for (int probe = 0; probe < 64; ++probe) {
    const int32_t old = atomicCAS(&T.key[h], -1, node);
    if (old == -1 || old == node) {
      lds_add_u64(&T.val[h], (unsigned long long)q);
      return;
    }
    h = (h + 1) & (kTable - 1);
  }
  atomicAdd(reinterpret_cast<unsigned long long*>(charge + node),
            (unsigned long long)q);
}

__device__ inline void table_flush(ChargeTable& T, int64_t* charge) {
  __syncthreads();
  for (int k = threadIdx.x; k < kTable; k += blockDim.x) {
    const int32_t node = T.key[k];
    const unsigned long long v = T.val[k];
    if (node >= 0 && v != 0ull)
      atomicAdd(reinterpret_cast<unsigned long long*>(charge + node), v);
  }
}

__device__ inline void deposit_table(const int32_t* node, const double lam[4],
                                     double w, ChargeTable& T,
                                     int64_t* charge) {
  int64_t q[4];
  charge_split(lam, w, q);
#pragma unroll
  for (int k = 0; k < 4; ++k) table_add(T, node[k], q[k], charge);
}

// G: the record of the hint tet (have_G), or to be loaded when needed.
// (tet: the slot's tet id; i: the slot)
template <bool PK>
__device__ inline void settle(const DevMesh& m, const MapTable* M,
                              const StepArgs& a, int32_t* tet, int32_t i,
                              double x, double y, double z, int sx, int sy,
                              int hint, Geo<PK>& G, double w, Acc& acc,
                              ChargeTable& T, bool far, bool have_G = true) {
  if (z >= m.z_top) {
    *tet = -1;
    lds_add_u64(&T.n_anode, 1ull);
    lds_add_u64(&T.q_anode, (unsigned long long)fx_round(w * kFx));
    return;
  }
  int steps = 0;
  double lam[4];
  const int t = walk<PK>(m, M, x, y, z, hint, sx, sy, steps, far, G, lam, have_G);
  acc.walk_steps += steps;
  if (steps > acc.walk_max) acc.walk_max = steps;
  if (t >= 0) {
    *tet = t;
    deposit_table(G.node(), lam, w, T, a.charge);
    acc.n_after += 1;
    acc.q_after += fx_round(w * kFx);
  } else {
    *tet = hint;
    const int slot = atomicAdd(&a.scratch->n_fallback, 1);
    a.queue[slot] = i;
  }
}

__device__ inline void wrap(const DevMesh& m, double& x, double& y, int& sx,
                            int& sy) {
  sx = 0;
  sy = 0;
  if (x >= m.Lx) {
    x = x - m.Lx;
    sx = 1;
  } else if (x < 0.0) {
    x = x + m.Lx;
    sx = -1;
  }
  if (y >= m.Ly) {
    y = y - m.Ly;
    sy = 1;
  } else if (y < 0.0) {
    y = y + m.Ly;
    sy = -1;
  }
}

}  // namespace

__device__ inline double fn_current(double F, double phi, const EmitConsts& c,
                                    int& clamped) {
  if (!(F > 1e-3)) return 0.0;
  double f = c.c_s * F / (phi * phi);
  if (f >= 1.0) {
    f = 1.0 - 1e-9;
    clamped = 1;
  }
  const double lf = log(f);
  const double v = 1.0 - f + (f / 6.0) * lf;
  const double t = 1.0 + f / 9.0 - (f / 18.0) * lf;
  const double Fsi = F * 1e9;
  return c.a_fn * Fsi * Fsi / (phi * t * t) *
         exp(-v * c.b_fn * (phi * sqrt(phi)) / F);
}

__device__ inline void face_field(const DevMesh& m, const void* E, int f32,
                                  int64_t f, double& ex, double& ey,
                                  double& ez) {
  const int32_t* nd = m.e_nodes + 3 * f;
  const double4 a = ld_E(E, f32, nd[0]);
  const double4 b = ld_E(E, f32, nd[1]);
  const double4 c = ld_E(E, f32, nd[2]);
  ex = ((a.x + b.x) + c.x) / 3.0;
  ey = ((a.y + b.y) + c.y) / 3.0;
  ez = ((a.z + b.z) + c.z) / 3.0;
}


// ---------------------------------------------------------------------------
// Emission counts: per emitting face the centroid field
// ((E_a + E_b) + E_c)/3, the FN current when the field pulls electrons out of
// the metal, Eq. nsp and the rounding of Eq. rnd_nsp; an exclusive scan of
// the counts gives every new particle its slot.
// ---------------------------------------------------------------------------
// PUB: the offsets and inj_fit are read by other workgroups of the same
// launch (see emit_publish), so they go past the caches.
template <bool PUB>
__device__ inline void emit_put(int32_t* p, int32_t v) {
  if (PUB)
    dev_put(p, v);
  else
    *p = v;
}

// Workgroup t of T: the faces are taken NT to a trip, the trips by the
// workgroups in turn.  Counts and currents of a trip are computed on their
// own; the running sums (counts, and currents and fields in a fixed order)
// then pass from trip to trip.
template <int NT, bool PUB>
__device__ void emit_block(const EmitArgs& a, int t, int T) {
  const DevMesh& m = a.m;
  __shared__ long long s_scan[NT / 64];
  __shared__ double s_red[3][NT / 64];
  __shared__ long long s_cl[NT / 64];
  __shared__ EmitSums s_sums;
  EmitSums sum{};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int trips = (int)((m.n_emit + NT - 1) / NT);
  for (int k = t; k < trips; k += T) {
    const int64_t f = k * (int64_t)NT + threadIdx.x;
    long long cnt = 0;
    double cur = 0.0, F = 0.0;
    int clamped = 0;
    if (f < m.n_emit) {
      double ex, ey, ez;
      if (a.cell)
        face_cell_field(m, m.e_tet[f], a.phi, ex, ey, ez);
      else
        face_field(m, a.E, a.f32, f, ex, ey, ez);
      F = sqrt((ex * ex + ey * ey) + ez * ez);
      const double* nr = m.e_nrm + 3 * f;
      const double en = (ex * nr[0] + ey * nr[1]) + ez * nr[2];
      double jd = 0.0;
      if (en < 0.0)
        jd = fn_current(F, a.phi_w, a.c, clamped) * a.c.j_unit;
      jd = jd * a.j_scale;
      cur = jd * m.e_area[f];
      if (a.counts) {
        const double nsp = cur * a.dt / a.w_sp;
        uint64_t r4[4];
        philox4x64_10(a.seed, a.instance, (uint64_t)a.step, (uint64_t)f, 0, 0,
                      r4);
        const double R = unit_double(r4[0]);
        const double fl = floor(nsp);
        double c = (R >= nsp - fl) ? fl : ceil(nsp);
        if (c > 2097152.0) c = 2097152.0;
        cnt = (long long)c;
        if (a.counts_in) {
          const int32_t ci = a.counts_in[f];
          cnt = ci < 0 ? 0 : (ci > 2097152 ? 2097152 : ci);
        }
        if (a.counts_out) a.counts_out[f] = (int32_t)cnt;
      }
      if (a.face_F) a.face_F[f] = F;
    }
    // exclusive scan of the counts: shuffle scan per wave, then waves
    long long inc = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const long long o = __shfl_up(inc, off, 64);
      if (lane >= off) inc += o;
    }
    if (lane == 63) s_scan[wave] = inc;
    // sums of current and |E|, max |E|, clamp count (fixed order)
    double v0 = cur, v1 = F, v2 = F;
    long long vc = clamped;
    for (int off = 32; off >= 1; off >>= 1) {
      v0 += __shfl_xor(v0, off, 64);
      v1 += __shfl_xor(v1, off, 64);
      const double o2 = __shfl_xor(v2, off, 64);
      v2 = o2 > v2 ? o2 : v2;
      vc += __shfl_xor(vc, off, 64);
    }
    if (lane == 0) {
      s_red[0][wave] = v0;
      s_red[1][wave] = v1;
      s_red[2][wave] = v2;
      s_cl[wave] = vc;
    }
    if (T > 1 && k > 0 && threadIdx.x == 0)
      sums_get(a.scratch->sums + (k - 1) % T, s_sums, k);
    __syncthreads();
    if (T > 1 && k > 0) sum = s_sums;
    const long long offset = sum.offset;
    long long before = 0;
    for (int w = 0; w < NT / 64; ++w) {
      if (w < wave) before += s_scan[w];
      sum.offset += s_scan[w];
      sum.cur += s_red[0][w];
      sum.F_sum += s_red[1][w];
      sum.F_max = s_red[2][w] > sum.F_max ? s_red[2][w] : sum.F_max;
      sum.n_clamp += s_cl[w];
    }
    if (T > 1 && k + 1 < trips && threadIdx.x == 0)
      sums_put(a.scratch->sums + k % T, sum, k + 1);
    if (f < m.n_emit && a.counts) {
      a.counts[f] = (int32_t)cnt;
      emit_put<PUB>(a.offsets + f, (int32_t)(offset + before + inc - cnt));
    }
    __syncthreads();
  }
  // the workgroup of the last trip ends the emission
  if (threadIdx.x == 0 && t == (trips > 0 ? (trips - 1) % T : 0)) {
    if (a.rate) *a.rate = sum.cur;
    if (a.stats) {
      pic_step_stats* st = a.stats;
      st->emit_current = sum.cur;
      st->mean_face_E = m.n_emit ? sum.F_sum / (double)m.n_emit : 0.0;
      st->max_face_E = sum.F_max;
      st->n_clamp = sum.n_clamp;
    }
    if (a.counts) {
      const long long base = *a.n_slots;
      const EmitEnd end = emit_end(sum, base, a.capacity);
      emit_put<PUB>(a.offsets + m.n_emit, (int32_t)end.total);
      a.scratch->inj_base = (int32_t)base;
      a.scratch->inj_total = (int32_t)end.total;
      emit_put<PUB>(&a.scratch->inj_fit, (int32_t)end.fit);
      *a.n_slots = (int32_t)(base + end.fit);
      if (a.stats) {
        a.stats->n_trunc = end.total - end.fit;
        if (end.status != PIC_OK) a.stats->status = end.status;
        a.stats->n_slots = base + end.fit;
      }
    }
  }
}

constexpr int kBeginBlock = 512;

__global__ void __launch_bounds__(kBlock) k_emit(EmitArgs a) {
  emit_block<kBlock, false>(a, 0, 1);
}

// Start of the first step of a call (the solve of a step starts the next):
// workgroup 0 clears the step's stats and counters, the others the node
// charges.
__device__ inline void begin_body(const EmitArgs& a, VB vb) {
  if (gate_closed(a.gate)) return;
  if (vb.id == 0) {
    int64_t* s64 = reinterpret_cast<int64_t*>(a.stats);
    const int ns = (int)(sizeof(pic_step_stats) / sizeof(int64_t));
    if (threadIdx.x < ns) s64[threadIdx.x] = 0;
    int32_t* c32 = reinterpret_cast<int32_t*>(a.scratch);
    const int nc = (int)(sizeof(StepScratch) / sizeof(int32_t));
    static_assert(sizeof(StepScratch) / sizeof(int32_t) <= kBeginBlock, "one word per thread");
    if (threadIdx.x < nc) c32[threadIdx.x] = 0;
    __syncthreads();
    // (the particle kernel emits; its pushing workgroups need the slot count
    // before injection now)
    if (threadIdx.x == 0) a.scratch->inj_base = *a.n_slots;
    return;
  }
  const int64_t G = vb.n - 1;
  for (int64_t i = (vb.id - 1) * (int64_t)blockDim.x + threadIdx.x;
       i < a.n_clear; i += G * blockDim.x)
    a.clear[i] = 0;
}

__global__ void __launch_bounds__(kBeginBlock) k_begin(EmitArgs a) {
  begin_body(a, VB{(int)blockIdx.x, (int)gridDim.x});
}

__global__ void __launch_bounds__(kBeginBlock) k_begin_b(const EmitArgs* E,
                                                         BatchMap map) {
  int i;
  const VB vb = batch_block(map, i);
  const EmitArgs a = batch_args(E, i);
  begin_body(a, vb);
}

// ---------------------------------------------------------------------------
// The particle kernel of a step.  Workgroups [0, g_push) advance the live
// particles (gather E_k, kick (v + QE) + QE, drift, wrap, absorb, walk,
// deposit); the remaining workgroups inject the new ones (Sec. II B 3,
// App. E: sample the face, Eq. sp_velocity, Eq. sp_displacement, drift,
// wrap, absorb, walk, deposit).  Both halves only read the slots below the
// pre-injection count, so they run side by side.
// ---------------------------------------------------------------------------
// Live particles, FP64 storage: the fixed arithmetic shared with the oracle.
// Element o of a stream read from the workgroup's base: the streams' bases
// advanced to the start of the workgroup's span are uniform (scalar
// registers), and one 32-bit byte offset per lane then addresses every
// stream (scalar base + vector offset) instead of a 64-bit address per
// stream and lane.  The FP64 push needed 142 VGPRs with per-stream
// addresses and spilled 9 dwords per lane at its 128-register bound; with
// the shared offset it fits in 124 (83.6 against 86.6 us per launch).
template <typename T>
__device__ inline T& at_off(const void* base, uint32_t bytes) {
  return *reinterpret_cast<T*>(reinterpret_cast<char*>(const_cast<void*>(base)) + bytes);
}

template <bool PK>
__device__ inline void push_role64(const StepArgs& a, const MapTable* M, int g,
                                   int G, Acc& acc, ChargeTable& T) {
  const DevMesh& m = a.m;
  const int64_t n = a.scratch->inj_base;
  const Span sp = block_span(n, G, g);
  const double Q = a.Q;
  const double dt = a.dt;
  // the span's streams (see at_off)
  double* X = (double*)a.x + sp.lo;
  double* Y = (double*)a.y + sp.lo;
  double* Z = (double*)a.z + sp.lo;
  double* VX = (double*)a.vx + sp.lo;
  double* VY = (double*)a.vy + sp.lo;
  double* VZ = (double*)a.vz + sp.lo;
  const double* W = a.w + sp.lo;
  int32_t* TT = a.tet + sp.lo;
  const uint32_t len = (uint32_t)(sp.hi - sp.lo), lo32 = (uint32_t)sp.lo;
  for (uint32_t j = threadIdx.x; j < len; j += blockDim.x) {
    const uint32_t o8 = j * 8u;
    const int t = at_off<const int32_t>(TT, j * 4u);
    if (t < 0) continue;
    const double w = at_off<const double>(W, o8);
    acc.n_before += 1;
    acc.q_before += fx_round(w * kFx);
    double x = at_off<double>(X, o8), y = at_off<double>(Y, o8), z = at_off<double>(Z, o8);
    double vx = at_off<double>(VX, o8), vy = at_off<double>(VY, o8),
           vz = at_off<double>(VZ, o8);
    Geo<PK> R;
    R.load(m, t);
    double ex, ey, ez;
    if (a.cell)
      cell_field<PK>(R, M, a.phi, ex, ey, ez);
    else
      gather_field<PK>(R, M, a.E, x, y, z, ex, ey, ez);
    const double qx = Q * ex, qy = Q * ey, qz = Q * ez;
    vx = (vx + qx) + qx;
    vy = (vy + qy) + qy;
    vz = (vz + qz) + qz;
    const double dx = dt * vx, dy = dt * vy, dz = dt * vz;
    const bool far = (dx * dx + dy * dy) + dz * dz > m.jump_len2;
    x = x + dx;
    y = y + dy;
    z = z + dz;
    int sx, sy;
    wrap(m, x, y, sx, sy);
    at_off<double>(X, o8) = x;
    at_off<double>(Y, o8) = y;
    at_off<double>(Z, o8) = z;
    at_off<double>(VX, o8) = vx;
    at_off<double>(VY, o8) = vy;
    at_off<double>(VZ, o8) = vz;
    settle<PK>(m, M, a, &at_off<int32_t>(TT, j * 4u), (int32_t)(lo32 + j), x, y, z, sx, sy, t,
               R, w, acc, T, far);
  }
}

// Live particles, mixed precision: FP32 position, velocity, field gather,
// kick and drift; the barycentric weights, the walk and the deposition take
// the stored FP32 position widened exactly to FP64.
template <bool PK>
__device__ inline void push_role32(const StepArgs& a, const MapTable* M, int g,
                                   int G, Acc& acc, ChargeTable& T) {
  const DevMesh& m = a.m;
  const int64_t n = a.scratch->inj_base;
  const Span sp = block_span(n, G, g);
  const float Q = (float)a.Q;
  const float dt = (float)a.dt;
  const float Lx = (float)m.Lx, Ly = (float)m.Ly;
  const float4* E = reinterpret_cast<const float4*>(a.E);
  // the span's streams (see at_off)
  float* X = (float*)a.x + sp.lo;
  float* Y = (float*)a.y + sp.lo;
  float* Z = (float*)a.z + sp.lo;
  float* VX = (float*)a.vx + sp.lo;
  float* VY = (float*)a.vy + sp.lo;
  float* VZ = (float*)a.vz + sp.lo;
  const double* W = a.w + sp.lo;
  int32_t* TT = a.tet + sp.lo;
  const uint32_t len = (uint32_t)(sp.hi - sp.lo), lo32 = (uint32_t)sp.lo;
  for (uint32_t j = threadIdx.x; j < len; j += blockDim.x) {
    const uint32_t o4 = j * 4u;
    const int t = at_off<const int32_t>(TT, o4);
    if (t < 0) continue;
    const double w = at_off<const double>(W, j * 8u);
    acc.n_before += 1;
    acc.q_before += fx_round(w * kFx);
    float x = at_off<float>(X, o4), y = at_off<float>(Y, o4), z = at_off<float>(Z, o4);
    float vx = at_off<float>(VX, o4), vy = at_off<float>(VY, o4), vz = at_off<float>(VZ, o4);
    // FP32 gather, from the packed record rounded to FP32, or from the FP32
    // record (half the bytes of the FP64 one, which the walk loads only
    // when it needs the hint tet itself)
    Geo<PK> R;
    float v0[3], r[9];
    int32_t nd[4];
    if constexpr (PK) {
      R.load(m, t);
      const lds_f q = (lds_f) static_cast<const MapTable32*>(M)->m32 + R.mp;
#pragma unroll
      for (int k = 0; k < 9; ++k) r[k] = q[k];
#pragma unroll
      for (int k = 0; k < 3; ++k) v0[k] = (float)R.v0[k];
#pragma unroll
      for (int k = 0; k < 4; ++k) nd[k] = R.nd[k];
    } else {
      const TetGeom32 G32 = m.tg32[t];
#pragma unroll
      for (int k = 0; k < 9; ++k) r[k] = G32.m[k];
#pragma unroll
      for (int k = 0; k < 3; ++k) v0[k] = G32.v0[k];
#pragma unroll
      for (int k = 0; k < 4; ++k) nd[k] = G32.node[k];
    }
    float ex, ey, ez;
    if (a.cell) {
      // -(grad phi)_t from the potential differences to vertex 0 (FP64
      // differences, FP32 products: no cancellation of the potential's size)
      const double p0 = a.phi[nd[0]];
      const float d1 = (float)(a.phi[nd[1]] - p0);
      const float d2 = (float)(a.phi[nd[2]] - p0);
      const float d3 = (float)(a.phi[nd[3]] - p0);
      ex = -((d1 * r[0] + d2 * r[3]) + d3 * r[6]);
      ey = -((d1 * r[1] + d2 * r[4]) + d3 * r[7]);
      ez = -((d1 * r[2] + d2 * r[5]) + d3 * r[8]);
    } else {
      const float4 e0 = E[nd[0]], e1 = E[nd[1]], e2 = E[nd[2]], e3 = E[nd[3]];
      const float dx0 = x - v0[0], dy0 = y - v0[1], dz0 = z - v0[2];
      const float l1 = (r[0] * dx0 + r[1] * dy0) + r[2] * dz0;
      const float l2 = (r[3] * dx0 + r[4] * dy0) + r[5] * dz0;
      const float l3 = (r[6] * dx0 + r[7] * dy0) + r[8] * dz0;
      const float l0 = ((1.0f - l1) - l2) - l3;
      ex = ((l0 * e0.x + l1 * e1.x) + l2 * e2.x) + l3 * e3.x;
      ey = ((l0 * e0.y + l1 * e1.y) + l2 * e2.y) + l3 * e3.y;
      ez = ((l0 * e0.z + l1 * e1.z) + l2 * e2.z) + l3 * e3.z;
    }
    const float qx = Q * ex, qy = Q * ey, qz = Q * ez;
    vx = (vx + qx) + qx;
    vy = (vy + qy) + qy;
    vz = (vz + qz) + qz;
    const float dx = dt * vx, dy = dt * vy, dz = dt * vz;
    const bool far = (double)((dx * dx + dy * dy) + dz * dz) > m.jump_len2;
    x = x + dx;
    y = y + dy;
    z = z + dz;
    int sx = 0, sy = 0;
    if (x >= Lx) {
      x = x - Lx;
      sx = 1;
    } else if (x < 0.0f) {
      x = x + Lx;
      sx = -1;
    }
    if (y >= Ly) {
      y = y - Ly;
      sy = 1;
    } else if (y < 0.0f) {
      y = y + Ly;
      sy = -1;
    }
    at_off<float>(X, o4) = x;
    at_off<float>(Y, o4) = y;
    at_off<float>(Z, o4) = z;
    at_off<float>(VX, o4) = vx;
    at_off<float>(VY, o4) = vy;
    at_off<float>(VZ, o4) = vz;
    settle<PK>(m, M, a, &at_off<int32_t>(TT, o4), (int32_t)(lo32 + j), x, y, z, sx, sy, t, R,
               w, acc, T, far, PK);
  }
}

constexpr int kEmitLds = 1024;  // emitting faces whose offsets fit in LDS

template <bool PK>
__device__ inline void inject_role(const StepArgs& a, const MapTable* M, int g,
                                   int G, Acc& acc, ChargeTable& T) {
  const DevMesh& m = a.m;
  const int64_t n = dev_get(&a.scratch->inj_fit);
  const int64_t base = a.scratch->inj_base;
  const double dt = a.dt;
  // the offsets for the search of a slot's face: in LDS where they fit (ten
  // dependent loads from LDS instead of memory)
  const int32_t* off = a.offsets;
  __shared__ int32_t s_off[kEmitLds];
  const bool in_lds = m.n_emit <= kEmitLds;
  if (g * (int64_t)blockDim.x >= n) return;  // (the whole workgroup)
  if (in_lds) {
    for (int f = threadIdx.x; f < (int)m.n_emit; f += blockDim.x) s_off[f] = dev_get(off + f);
    __syncthreads();
  }
  auto at = [&](int f) { return in_lds ? s_off[f] : dev_get(off + f); };
  for (int64_t s = g * (int64_t)blockDim.x + threadIdx.x; s < n;
       s += (int64_t)G * blockDim.x) {
    // face: last f with off[f] <= s
    int lo = 0, hi = (int)m.n_emit - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (at(mid) <= s) lo = mid; else hi = mid - 1;
    }
    const int f = lo;
    const int64_t o = s - at(f);
    uint64_t r4[4];
    philox4x64_10(a.seed, a.instance, (uint64_t)a.step, (uint64_t)f,
                  (uint64_t)o, 1, r4);
    double R1 = unit_double(r4[0]), R2 = unit_double(r4[1]);
    const double R = unit_double(r4[2]);
    if (R1 + R2 > 1.0) {
      R1 = 1.0 - R1;
      R2 = 1.0 - R2;
    }
    const double l0 = (1.0 - R1) - R2;
    const double* A = m.e_abc + 9 * (int64_t)f;
    const double px = (A[0] + R1 * (A[3] - A[0])) + R2 * (A[6] - A[0]);
    const double py = (A[1] + R1 * (A[4] - A[1])) + R2 * (A[7] - A[1]);
    const double pz = (A[2] + R1 * (A[5] - A[2])) + R2 * (A[8] - A[2]);
    double Ex, Ey, Ez;
    if (a.cell) {
      face_cell_field(m, m.e_tet[f], a.phi, Ex, Ey, Ez);
    } else {
      const int32_t* nd = m.e_nodes + 3 * (int64_t)f;
      const double4 ea = ld_E(a.E, a.f32, nd[0]);
      const double4 eb = ld_E(a.E, a.f32, nd[1]);
      const double4 ec = ld_E(a.E, a.f32, nd[2]);
      Ex = (l0 * ea.x + R1 * eb.x) + R2 * ec.x;
      Ey = (l0 * ea.y + R1 * eb.y) + R2 * ec.y;
      Ez = (l0 * ea.z + R1 * eb.z) + R2 * ec.z;
    }
    const double cv = a.qm_dt * (0.5 + R);
    const double vx = cv * Ex, vy = cv * Ey, vz = cv * Ez;
    double x = px + (vx * dt) * R;
    double y = py + (vy * dt) * R;
    double z = pz + (vz * dt) * R;
    x = x + dt * vx;
    y = y + dt * vy;
    z = z + dt * vz;
    int sx, sy;
    wrap(m, x, y, sx, sy);
    const int64_t i = base + s;
    const double w = a.s_face ? a.s_face[f] : 1.0;
    if (a.f32) {
      // stored in FP32; the walk and deposition use the stored values
      const float xf = (float)x, yf = (float)y, zf = (float)z;
      ((float*)a.x)[i] = xf;
      ((float*)a.y)[i] = yf;
      ((float*)a.z)[i] = zf;
      ((float*)a.vx)[i] = (float)vx;
      ((float*)a.vy)[i] = (float)vy;
      ((float*)a.vz)[i] = (float)vz;
      x = xf;
      y = yf;
      z = zf;
    } else {
      ((double*)a.x)[i] = x;
      ((double*)a.y)[i] = y;
      ((double*)a.z)[i] = z;
      ((double*)a.vx)[i] = vx;
      ((double*)a.vy)[i] = vy;
      ((double*)a.vz)[i] = vz;
    }
    a.w[i] = w;
    a.birth[i] = f;
    a.id[i] = (a.step << 42) | ((int64_t)f << 21) | o;
    acc.n_inj += 1;
    acc.q_inj += fx_round(w * kFx);
    const int h = m.e_tet[f];
    Geo<PK> H;
    H.load(m, h);
    settle<PK>(m, M, a, a.tet + i, (int32_t)i, x, y, z, sx, sy, h, H, w, acc, T, false);
  }
}

// The emission of the step computed inside the particle kernel: emitting
// workgroups compute the counts and offsets and publish them; the injecting
// workgroups (dispatched last) wait until all have.  The waits are bounded: a
// flag not seen in time (never expected) skips the injection and marks the
// step with a device error.
// The emitting workgroups are blocks 0, 8, 16, ... of a launch: all on the XCD
// of block 0, which takes its blocks in order, ahead of any block there that
// waits.  So wherever a waiting block holds a place of that XCD, the blocks it
// waits for have theirs, and launches of several streams cannot wait for one
// another's places.  (Spread over the XCDs, each of two launches could fill an
// XCD with waiting blocks while the other's emitting block for it had no
// place: two batches of 64 instances at 16 injecting blocks have 128 of them
// per XCD, as many as it has places.)  The seven blocks between two of them
// end at once.
// What is published (the sums, the offsets and inj_fit) goes past the caches
// (see handover.h), each wave's stores ahead of the barrier before the count.
// With fences of device scope instead, and the offsets not searched in LDS,
// the particle kernel of a small step (10k superparticles, 276 emitting faces)
// took 40 us, 30 so.  A trip of 256 faces takes 7 to 10 us, most of it
// dependent loads: one workgroup taking the trips in turn published 612 faces
// after 31 us, eight at once after 19.
constexpr int kXcds = 8;

__host__ __device__ inline int emitters(const DevMesh& m) {
  const int64_t trips = (m.n_emit + kBlock - 1) / kBlock;
  return trips < 1 ? 1 : (trips < kEmitters ? (int)trips : kEmitters);
}

__device__ inline void emit_publish(const EmitArgs& e, int t, int T) {
  emit_block<kBlock, true>(e, t, T);
  hand_over();
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_fetch_add(&e.scratch->emitted, 1, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline bool emit_wait(const StepArgs& a, int T) {
  __shared__ int seen;
  if (threadIdx.x == 0) {
    int ok = 0;
    for (int it = 0; it < kEmitSpin; ++it) {
      if (dev_get(&a.scratch->emitted) == T) {
        ok = 1;
        break;
      }
      __builtin_amdgcn_s_sleep(20);  // (128 workgroups poll one word)
    }
    take_over();
    if (!ok && a.stats) a.stats->status = PIC_E_DEVICE;
    seen = ok;
  }
  __syncthreads();
  return seen != 0;
}

// One instance per storage precision and record form, so that only one push
// is compiled in.  T_emit: emitting workgroups.
template <bool F32, bool PK>
__device__ inline void particles_body(const StepArgs& a, VB vb, int T_emit) {
  Acc acc;
  acc_zero(acc);
  __shared__ ChargeTable T;
  const MapTable* M = nullptr;
  if constexpr (PK) {
    __shared__ std::conditional_t<F32, MapTable32, MapTable> maps;
    maps_load(a.m, maps);
    M = &maps;
  }
  table_clear(T);  // (synchronizes)
  const int g_push = a.g_push;
  if (vb.id < g_push) {
    if (F32)
      push_role32<PK>(a, M, vb.id, g_push, acc, T);
    else
      push_role64<PK>(a, M, vb.id, g_push, acc, T);
  } else if (emit_wait(a, T_emit)) {
    inject_role<PK>(a, M, vb.id - g_push, vb.n - g_push, acc, T);
  }
  table_flush(T, a.charge);  // (synchronizes)
  if (threadIdx.x == 0) {
    acc.n_anode = (int)T.n_anode;
    acc.q_anode = (long long)T.q_anode;
  }
  acc_flush(acc, a.acc_rows, vb.id, a.acc_stride);
}

// The leading workgroups only emit (see emit_publish), the others push and
// inject, each on the XCD of its index among them.
// Bound: the load path and its latency (17 divergent 16-byte gathers per
// superparticle on packed records), so waves in flight count.  On packed
// records the push and the injection fit 96 registers without spills (maps
// in LDS, integer seed clamps, 32-bit counters, absorption counted in LDS)
// and five waves run per SIMD; only the emission spills then.
// Full records need 122 registers: four waves.  Ten steps of 1e6
// superparticles, re-sort included: 1098 us at four waves, 1067 at five; of
// 1e4, where the emission is the longest chain: 508 at four, 557 at five.
// So W = 5 only where the arrays have more slots than four waves have lanes
// (a fifth could not hold a superparticle otherwise).
template <bool F32, bool PK, int W>
__global__ void __launch_bounds__(kBlock, W) k_particles(StepArgs a, EmitArgs e) {
  if (gate_closed(a.gate)) return;
  const int T = emitters(a.m), lead = kXcds * T, g = (int)blockIdx.x;
  if (g < lead) {
    if (g % kXcds == 0) emit_publish(e, g / kXcds, T);
    return;
  }
  particles_body<F32, PK>(a, VB{g - lead, (int)gridDim.x - lead}, T);
}

// The emitting workgroups of all instances come first, one each (the other
// instances' pushes hide its trips; eight each took 1171 us instead of 1155
// for ten steps of six tips).
__host__ __device__ inline int batch_lead(const BatchMap& map) { return kXcds * map.n_seg; }

template <bool F32, bool PK>
__global__ void __launch_bounds__(kBlock, 4) k_particles_b(const StepArgs* A,
                                                            const EmitArgs* E,
                                                            BatchMap map) {
  const int lead = batch_lead(map);
  if ((int)blockIdx.x < lead) {
    if (blockIdx.x % kXcds) return;
    const EmitArgs e = batch_args(E, map.inst[blockIdx.x / kXcds]);
    if (!gate_closed(e.gate)) emit_publish(e, 0, 1);
    return;
  }
  int i;
  const VB vb = batch_block(map, i, lead);
  const StepArgs a = batch_args(A, i);
  if (gate_closed(a.gate)) return;
  particles_body<F32, PK>(a, vb, 1);
}

// ---------------------------------------------------------------------------
// Particles the walk could not certify: exact canonical location; those
// outside every tet (below the top plane) are absorbed by the cathode.
// ---------------------------------------------------------------------------
__device__ inline void fallback_body(const StepArgs& a, VB vb) {
  if (gate_closed(a.gate)) return;
  const DevMesh& m = a.m;
  const int64_t n = a.scratch->n_fallback;
  Acc acc;
  acc_zero(acc);
  // one wave per queued particle
  const int64_t waves = (int64_t)vb.n * (blockDim.x >> 6);
  const bool lead = (threadIdx.x & 63) == 0;
  for (int64_t j = vb.id * (int64_t)(blockDim.x >> 6) + (threadIdx.x >> 6);
       j < n; j += waves) {
    const int64_t i = a.queue[j];
    double x, y, z;
    if (a.f32) {
      x = ((const float*)a.x)[i];
      y = ((const float*)a.y)[i];
      z = ((const float*)a.z)[i];
    } else {
      x = ((const double*)a.x)[i];
      y = ((const double*)a.y)[i];
      z = ((const double*)a.z)[i];
    }
    const double w = a.w[i];
    const long long qfx = fx_round(w * kFx);
    const int t = scan_locate_wave(m, x, y, z);
    if (!lead) continue;
    if (t >= 0) {
      a.tet[i] = t;
      deposit_one(m.tg[t], x, y, z, w, a.charge);
      acc.n_after += 1;
      acc.q_after += qfx;
    } else {
      a.tet[i] = -1;
      acc.n_cathode += 1;
      acc.q_cathode += qfx;
    }
  }
  // counter rows after those of the particle kernel
  acc_flush(acc, a.acc_rows, a.n_blocks + vb.id, a.acc_stride);
  if (vb.id == 0 && threadIdx.x == 0) a.stats->n_fallback = n;
}

__global__ void __launch_bounds__(kBlock) k_fallback(StepArgs a) {
  fallback_body(a, VB{(int)blockIdx.x, (int)gridDim.x});
}

__global__ void __launch_bounds__(kBlock) k_fallback_b(const StepArgs* A,
                                                       BatchMap map) {
  int i;
  const VB vb = batch_block(map, i);
  const StepArgs a = batch_args(A, i);
  fallback_body(a, vb);
}

// ---------------------------------------------------------------------------
// Stand-alone location and deposition entry points.
// ---------------------------------------------------------------------------
template <bool PK>
__global__ void __launch_bounds__(kBlock) k_locate(LocateArgs a) {
  const DevMesh& m = a.m;
  const MapTable* M = nullptr;
  if constexpr (PK) {
    __shared__ MapTable maps;
    maps_load(m, maps);
    M = &maps;
    __syncthreads();
  }
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < a.n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double x = a.x[i], y = a.y[i], z = a.z[i];
    if (z >= m.z_top) {
      a.tet[i] = -1;
      a.where[i] = PIC_WHERE_ANODE;
      continue;
    }
    int h = a.tet[i];
    int t = -1, steps = 0;
    // without a hint the walk starts at the seed of the point's sub-cell (it
    // only answers when it is certain, so the answer does not depend on
    // where it starts), and only the points it cannot certify -- on a face,
    // in the metal, outside -- are left to the exact scan, a wave each.
    // Locating and depositing 300k points without hints: 475 us with every
    // one scanned (351 us, and 50 of atomics on the queue's counter), 126 so
    const bool hint = h >= 0 && h < m.n_tets;
    if (!hint) {
      h = fine_seed(m, x, y, z);
      if (h < 0) h = bucket_guess(m, x, y, z);
    }
    if (h >= 0) {
      Geo<PK> G;
      double lam[4];
      t = walk<PK>(m, M, x, y, z, h, 0, 0, steps, !hint, G, lam, false);
    }
    if (t >= 0) {
      a.tet[i] = t;
      a.where[i] = PIC_WHERE_INSIDE;
    } else {
      a.queue[queue_slot(a.n_queue)] = (int32_t)i;
    }
  }
}

__global__ void __launch_bounds__(kBlock) k_locate_scan(LocateArgs a) {
  const DevMesh& m = a.m;
  const int64_t n = *a.n_queue;
  // one wave per queued point
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t j = blockIdx.x * (int64_t)(blockDim.x >> 6) + (threadIdx.x >> 6);
       j < n; j += waves) {
    const int64_t i = a.queue[j];
    const int t = scan_locate_wave(m, a.x[i], a.y[i], a.z[i]);
    if ((threadIdx.x & 63) == 0) {
      a.tet[i] = t;
      a.where[i] = t >= 0 ? PIC_WHERE_INSIDE : PIC_WHERE_OUTSIDE;
    }
  }
}

__global__ void __launch_bounds__(kBlock) k_deposit(DepositArgs a) {
  const DevMesh& m = a.m;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < a.n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int t = a.tet[i];
    if (t < 0 || t >= m.n_tets) continue;
    deposit_one(m.tg[t], a.x[i], a.y[i], a.z[i], a.w[i], a.charge);
  }
}

// Fine walk seeds: the canonical tet of every sub-cell centre (exact scan),
// or the coarse seed where the centre lies in the metal.
__global__ void __launch_bounds__(kBlock) k_seed_build(DevMesh m) {
  const int64_t n = (int64_t)m.fnb[0] * m.fnb[1] * m.fnb[2];
  for (int64_t id = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; id < n;
       id += (int64_t)gridDim.x * blockDim.x) {
    const int64_t iz = id % m.fnb[2];
    const int64_t iy = (id / m.fnb[2]) % m.fnb[1];
    const int64_t ix = id / ((int64_t)m.fnb[2] * m.fnb[1]);
    const double x = m.b0[0] + ((double)ix + 0.5) / m.finv[0];
    const double y = m.b0[1] + ((double)iy + 0.5) / m.finv[1];
    const double z = m.b0[2] + ((double)iz + 0.5) / m.finv[2];
    int t = scan_locate(m, x, y, z);
    if (t < 0) t = bucket_guess(m, x, y, z);
    m.fseed[id] = t;
  }
}


// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_begin(const EmitArgs& a, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_begin, dim3(grid + 1), dim3(kBeginBlock), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_begin_b(const EmitArgs* E, const BatchMap& map, int grid,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_begin_b, dim3(grid), dim3(kBeginBlock), 0, s, E, map);
  return hipGetLastError();
}
hipError_t launch_particles_b(const StepArgs* A, const EmitArgs* E, const BatchMap& map,
                              int f32, int packed, hipStream_t s) {
  const auto kern = packed ? (f32 ? k_particles_b<true, true> : k_particles_b<false, true>)
                           : (f32 ? k_particles_b<true, false> : k_particles_b<false, false>);
  hipLaunchKernelGGL(kern, dim3(batch_lead(map) + map.off[map.n_seg]), dim3(kBlock), 0,
                     s, A, E, map);
  return hipGetLastError();
}
hipError_t launch_fallback_b(const StepArgs* A, const BatchMap& map, int grid,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_fallback_b, dim3(grid), dim3(kBlock), 0, s, A, map);
  return hipGetLastError();
}
using ParticlesKernel = void (*)(StepArgs, EmitArgs);

static ParticlesKernel particles_kernel(int f32, int packed, int waves) {
  if (!packed) return f32 ? k_particles<true, false, 4> : k_particles<false, false, 4>;
  if (waves == 5) return f32 ? k_particles<true, true, 5> : k_particles<false, true, 5>;
  return f32 ? k_particles<true, true, 4> : k_particles<false, true, 4>;
}

int particle_blocks_per_cu(int f32, int packed, int waves) {
  int n = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &n, particles_kernel(f32, packed, waves), kBlock, 0);
  return e == hipSuccess ? n : 0;
}

hipError_t launch_particles(const StepArgs& a, const EmitArgs& e, int g_push,
                            int g_inj, int waves, hipStream_t s) {
  StepArgs b = a;
  b.g_push = g_push;
  hipLaunchKernelGGL(particles_kernel(a.f32, a.m.tc != nullptr, waves),
                     dim3(kXcds * emitters(a.m) + g_push + g_inj), dim3(kBlock), 0, s, b, e);
  return hipGetLastError();
}
hipError_t launch_seed_build(const DevMesh& m, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_seed_build, dim3(grid), dim3(kBlock), 0, s, m);
  return hipGetLastError();
}
hipError_t launch_emit(const EmitArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_emit, dim3(1), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_fallback(const StepArgs& a, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_fallback, dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_locate(const LocateArgs& a, int grid, hipStream_t s) {
  hipLaunchKernelGGL(a.m.tc ? k_locate<true> : k_locate<false>, dim3(grid), dim3(kBlock), 0,
                     s, a);
  hipLaunchKernelGGL(k_locate_scan, dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_deposit(const DepositArgs& a, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_deposit, dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace fp
