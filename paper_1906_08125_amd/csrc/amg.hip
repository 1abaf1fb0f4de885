// Host setup of the smoothed-aggregation AMG hierarchy (Vanek, Mandel and
// Brezina 1996) used as a CG preconditioner for the FP64 Poisson solve:
//   strength  j is strongly coupled to i if |a_ij| >= theta sqrt(a_ii a_jj)
//             (theta = 0.08, halved on every coarser level);
//   aggregates three greedy phases in row order (root + its strong
//             neighbours when none of them is taken; leftovers join the
//             aggregate of a strong neighbour; the rest start new ones);
//   P         Jacobi-smoothed piecewise-constant prolongation
//             P = (I - omega D^-1 A) P0, omega = 4 / (3 lambda_max(D^-1 A))
//             with lambda_max from a power iteration;
//   coarse    A_c = P^T A P (symmetrized), down to at most kAmgCoarseMax
//             rows, whose dense inverse is applied exactly.
// Everything here runs once per mesh handle, on the first solve that asks
// for it; the V-cycle kernels are in solver.hip.
#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "amg.h"

namespace fp {

namespace {

struct HCsr {
  int64_t n = 0, m = 0;  // rows, columns
  std::vector<int64_t> rp;
  std::vector<int32_t> ci;
  std::vector<double> v;
};

std::vector<double> diag_of(const HCsr& A) {
  std::vector<double> d(A.n, 0.0);
  for (int64_t i = 0; i < A.n; ++i)
    for (int64_t p = A.rp[i]; p < A.rp[i + 1]; ++p)
      if (A.ci[p] == i) d[i] += A.v[p];
  return d;
}

HCsr transpose(const HCsr& A) {
  HCsr T;
  T.n = A.m;
  T.m = A.n;
  T.rp.assign(T.n + 1, 0);
  for (int64_t p = 0; p < A.rp[A.n]; ++p) T.rp[A.ci[p] + 1]++;
  for (int64_t i = 0; i < T.n; ++i) T.rp[i + 1] += T.rp[i];
  T.ci.resize(A.rp[A.n]);
  T.v.resize(A.rp[A.n]);
  std::vector<int64_t> fill(T.rp.begin(), T.rp.end() - 1);
  for (int64_t i = 0; i < A.n; ++i)  // rows in order: columns of T sorted
    for (int64_t p = A.rp[i]; p < A.rp[i + 1]; ++p) {
      const int64_t q = fill[A.ci[p]]++;
      T.ci[q] = (int32_t)i;
      T.v[q] = A.v[p];
    }
  return T;
}

// A row being summed: values by column, the columns in use sorted on demand.
class RowSum {
 public:
  explicit RowSum(int64_t columns) : at_(columns, Cell{-1, 0.0}) {}
  void open(int64_t row) {
    row_ = row;
    cols_.clear();
  }
  void add(int32_t j, double v) {
    Cell& c = at_[j];
    if (c.row != row_) {
      c = Cell{row_, 0.0};
      cols_.push_back(j);
    }
    c.v += v;
  }
  const std::vector<int32_t>& sorted() {
    std::sort(cols_.begin(), cols_.end());
    return cols_;
  }
  double operator[](int32_t j) const { return at_[j].v; }

 private:
  struct Cell {
    int64_t row;
    double v;
  };
  std::vector<Cell> at_;
  std::vector<int32_t> cols_;
  int64_t row_ = -1;
};

// Room for a matrix whose first rows are done, by their length.
void reserve_like(HCsr& M, int64_t done) {
  if (done != M.n / 32 || done == 0) return;
  const size_t want = M.ci.size() / (size_t)done * (size_t)M.n;
  M.ci.reserve(want + want / 8);
  M.v.reserve(want + want / 8);
}

// C = A B (Gustavson, dense accumulator over the columns of B).
HCsr multiply(const HCsr& A, const HCsr& B) {
  HCsr C;
  C.n = A.n;
  C.m = B.m;
  C.rp.assign(C.n + 1, 0);
  RowSum row(B.m);
  for (int64_t i = 0; i < A.n; ++i) {
    row.open(i);
    for (int64_t p = A.rp[i]; p < A.rp[i + 1]; ++p) {
      const int32_t k = A.ci[p];
      const double a = A.v[p];
      for (int64_t q = B.rp[k]; q < B.rp[k + 1]; ++q) row.add(B.ci[q], a * B.v[q]);
    }
    for (int32_t j : row.sorted()) {
      C.ci.push_back(j);
      C.v.push_back(row[j]);
    }
    C.rp[i + 1] = (int64_t)C.ci.size();
    reserve_like(C, i + 1);
  }
  return C;
}

// (A + A^T) / 2 for a structurally symmetric A (Galerkin products are).
HCsr symmetrize(const HCsr& A) {
  const HCsr T = transpose(A);
  HCsr S;
  S.n = A.n;
  S.m = A.m;
  S.rp.assign(S.n + 1, 0);
  S.ci.reserve(A.ci.size());
  S.v.reserve(A.v.size());
  for (int64_t i = 0; i < A.n; ++i) {
    int64_t p = A.rp[i], q = T.rp[i];
    const int64_t pe = A.rp[i + 1], qe = T.rp[i + 1];
    while (p < pe || q < qe) {
      int32_t j;
      double v = 0.0;
      if (q >= qe || (p < pe && A.ci[p] < T.ci[q])) {
        j = A.ci[p];
        v = 0.5 * A.v[p++];
      } else if (p >= pe || T.ci[q] < A.ci[p]) {
        j = T.ci[q];
        v = 0.5 * T.v[q++];
      } else {
        j = A.ci[p];
        v = 0.5 * (A.v[p++] + T.v[q++]);
      }
      S.ci.push_back(j);
      S.v.push_back(v);
    }
    S.rp[i + 1] = (int64_t)S.ci.size();
  }
  return S;
}

// Aggregate index of every row; nc receives the aggregate count.
std::vector<int32_t> aggregate(const HCsr& A, const std::vector<double>& d,
                               double theta, int64_t& nc) {
  const int64_t n = A.n;
  std::vector<int64_t> sp(n + 1, 0);
  std::vector<int32_t> sn;
  for (int64_t i = 0; i < n; ++i) {
    for (int64_t p = A.rp[i]; p < A.rp[i + 1]; ++p) {
      const int32_t j = A.ci[p];
      if (j != i && std::fabs(A.v[p]) >= theta * std::sqrt(std::fabs(d[i] * d[j])))
        sn.push_back(j);
    }
    sp[i + 1] = (int64_t)sn.size();
  }
  std::vector<int32_t> agg(n, -1);
  nc = 0;
  // 1: roots whose strong neighbourhood is untouched
  for (int64_t i = 0; i < n; ++i) {
    if (agg[i] != -1 || sp[i] == sp[i + 1]) continue;
    bool free = true;
    for (int64_t p = sp[i]; p < sp[i + 1] && free; ++p) free = agg[sn[p]] == -1;
    if (!free) continue;
    agg[i] = (int32_t)nc;
    for (int64_t p = sp[i]; p < sp[i + 1]; ++p) agg[sn[p]] = (int32_t)nc;
    ++nc;
  }
  // 2: join the phase-1 aggregate of the first strong neighbour
  const std::vector<int32_t> agg1 = agg;
  for (int64_t i = 0; i < n; ++i) {
    if (agg[i] != -1) continue;
    for (int64_t p = sp[i]; p < sp[i + 1]; ++p)
      if (agg1[sn[p]] != -1) {
        agg[i] = agg1[sn[p]];
        break;
      }
  }
  // 3: the rest start aggregates with their untaken strong neighbours
  for (int64_t i = 0; i < n; ++i) {
    if (agg[i] != -1) continue;
    agg[i] = (int32_t)nc;
    for (int64_t p = sp[i]; p < sp[i + 1]; ++p)
      if (agg[sn[p]] == -1) agg[sn[p]] = (int32_t)nc;
    ++nc;
  }
  return agg;
}

// Largest eigenvalue of D^-1 A (power iteration from a fixed start).
double lambda_max(const HCsr& A, const std::vector<double>& d) {
  std::vector<double> x(A.n), y(A.n);
  for (int64_t i = 0; i < A.n; ++i)
    x[i] = 1.0 + (double)((uint32_t)(i * 2654435761u) % 1024u) / 1024.0;
  double lam = 0.0;
  for (int it = 0; it < 30; ++it) {
    double nx = 0.0, ny = 0.0;
    for (int64_t i = 0; i < A.n; ++i) {
      double s = 0.0;
      for (int64_t p = A.rp[i]; p < A.rp[i + 1]; ++p) s += A.v[p] * x[A.ci[p]];
      y[i] = s / d[i];
      nx += x[i] * x[i];
      ny += y[i] * y[i];
    }
    lam = std::sqrt(ny / nx);
    const double sc = 1.0 / std::sqrt(ny);
    for (int64_t i = 0; i < A.n; ++i) x[i] = y[i] * sc;
  }
  return lam;
}

// P = (I - omega D^-1 A) P0 with P0 the aggregate indicator.
HCsr smoothed_p(const HCsr& A, const std::vector<double>& d,
                const std::vector<int32_t>& agg, int64_t nc, double omega) {
  HCsr P;
  P.n = A.n;
  P.m = nc;
  P.rp.assign(A.n + 1, 0);
  RowSum row(nc);
  for (int64_t i = 0; i < A.n; ++i) {
    row.open(i);
    row.add(agg[i], 1.0);
    const double s = omega / d[i];
    for (int64_t p = A.rp[i]; p < A.rp[i + 1]; ++p) row.add(agg[A.ci[p]], -s * A.v[p]);
    for (int32_t j : row.sorted()) {
      if (row[j] == 0.0) continue;
      P.ci.push_back(j);
      P.v.push_back(row[j]);
    }
    P.rp[i + 1] = (int64_t)P.ci.size();
    reserve_like(P, i + 1);
  }
  return P;
}

// (I - omega D^-1 A) P from P and AP = A P (rows sorted; the pattern of P
// lies in that of AP, whose rows hold a_ii P_i).
HCsr smooth_again(const HCsr& P, HCsr AP, const std::vector<double>& d, double omega) {
  HCsr S = std::move(AP);
  for (int64_t i = 0; i < S.n; ++i) {
    const double s = -omega / d[i];
    int64_t q = P.rp[i];
    const int64_t qe = P.rp[i + 1];
    for (int64_t p = S.rp[i]; p < S.rp[i + 1]; ++p) {
      S.v[p] *= s;
      if (q < qe && P.ci[q] == S.ci[p]) S.v[p] += P.v[q++];
    }
  }
  return S;
}

struct HSell {
  int64_t nrows = 0, nslices = 0;
  std::vector<int32_t> sptr, col;
  std::vector<double> val;
};

HSell to_sell(const HCsr& A) {
  HSell S;
  S.nrows = A.n;
  S.nslices = (A.n + kSell - 1) / kSell;
  S.sptr.assign(S.nslices + 1, 0);
  for (int64_t s = 0; s < S.nslices; ++s) {
    int64_t w = 0;
    for (int64_t r = s * kSell; r < std::min<int64_t>(A.n, (s + 1) * kSell); ++r)
      w = std::max(w, A.rp[r + 1] - A.rp[r]);
    S.sptr[s + 1] = (int32_t)(S.sptr[s] + w * kSell);
  }
  const int64_t np = S.sptr[S.nslices];
  S.col.assign(np, 0);
  S.val.assign(np, 0.0);
  for (int64_t s = 0; s < S.nslices; ++s)
    for (int64_t r = s * kSell; r < std::min<int64_t>(A.n, (s + 1) * kSell); ++r)
      for (int64_t k = A.rp[r]; k < A.rp[r + 1]; ++k) {
        const int64_t p = S.sptr[s] + (k - A.rp[r]) * kSell + (r - s * kSell);
        S.col[p] = A.ci[k];
        S.val[p] = A.v[k];
      }
  return S;
}

// Inverse of a dense SPD matrix (Cholesky, then the inverse from the
// factor); false when a pivot is not positive.
bool spd_inverse(std::vector<double>& a, int64_t n) {
  std::vector<double> L(n * n, 0.0);
  for (int64_t j = 0; j < n; ++j) {
    double s = a[j * n + j];
    for (int64_t k = 0; k < j; ++k) s -= L[j * n + k] * L[j * n + k];
    if (!(s > 0.0)) return false;
    const double ljj = std::sqrt(s);
    L[j * n + j] = ljj;
    for (int64_t i = j + 1; i < n; ++i) {
      double t = a[i * n + j];
      for (int64_t k = 0; k < j; ++k) t -= L[i * n + k] * L[j * n + k];
      L[i * n + j] = t / ljj;
    }
  }
  // columns of A^-1: solve L L^T x = e_c
  std::vector<double> y(n);
  for (int64_t c = 0; c < n; ++c) {
    for (int64_t i = 0; i < n; ++i) {
      double t = i == c ? 1.0 : 0.0;
      for (int64_t k = 0; k < i; ++k) t -= L[i * n + k] * y[k];
      y[i] = t / L[i * n + i];
    }
    for (int64_t i = n - 1; i >= 0; --i) {
      double t = y[i];
      for (int64_t k = i + 1; k < n; ++k) t -= L[k * n + i] * y[k];
      y[i] = t / L[i * n + i];
    }
    for (int64_t i = 0; i < n; ++i) a[i * n + c] = y[i];
  }
  // exact symmetry of the applied operator
  for (int64_t i = 0; i < n; ++i)
    for (int64_t j = i + 1; j < n; ++j) {
      const double v = 0.5 * (a[i * n + j] + a[j * n + i]);
      a[i * n + j] = a[j * n + i] = v;
    }
  return true;
}

// Host work allowed for a dense cycle (multiply-adds; a tenth of a second).
constexpr int64_t kDenseWork = 100000000;

// The V(1,1)-cycle of a level over the dense inverse inv of the next one as
// a dense matrix: 2 w D^-1 - w^2 D^-1 A D^-1 + Ps inv Rs.
std::vector<double> dense_cycle(const HCsr& A, const std::vector<double>& d,
                                double omega, const HCsr& Ps, const HCsr& Rs,
                                const std::vector<double>& inv) {
  const int64_t n = A.n, nc = Ps.m;
  std::vector<double> M(nc * n, 0.0);  // inv Rs
  for (int64_t k = 0; k < nc; ++k)
    for (int64_t q = 0; q < nc; ++q) {
      const double v = inv[k * nc + q];
      for (int64_t p = Rs.rp[q]; p < Rs.rp[q + 1]; ++p) M[k * n + Rs.ci[p]] += v * Rs.v[p];
    }
  // (symmetric: the upper half, then mirrored by blocks -- a column of the
  // whole matrix at a time misses the cache at every entry)
  std::vector<double> C(n * n, 0.0);
  for (int64_t i = 0; i < n; ++i) {
    double* c = &C[i * n];
    int64_t p = Ps.rp[i];
    const int64_t pe = Ps.rp[i + 1];
    auto row = [&](int64_t q) { return &M[(int64_t)Ps.ci[q] * n]; };
    for (; p + 4 <= pe; p += 4) {  // (four rows per pass over c)
      const double *m0 = row(p), *m1 = row(p + 1), *m2 = row(p + 2), *m3 = row(p + 3);
      const double v0 = Ps.v[p], v1 = Ps.v[p + 1], v2 = Ps.v[p + 2], v3 = Ps.v[p + 3];
      for (int64_t j = i; j < n; ++j)
        c[j] = (((c[j] + v0 * m0[j]) + v1 * m1[j]) + v2 * m2[j]) + v3 * m3[j];
    }
    for (; p < pe; ++p) {
      const double* m = row(p);
      for (int64_t j = i; j < n; ++j) c[j] += Ps.v[p] * m[j];
    }
    for (int64_t q = A.rp[i]; q < A.rp[i + 1]; ++q)
      if (A.ci[q] >= i) c[A.ci[q]] -= omega * omega * A.v[q] / (d[i] * d[A.ci[q]]);
    c[i] += 2.0 * omega / d[i];
  }
  constexpr int64_t kB = 64;
  for (int64_t i0 = 0; i0 < n; i0 += kB)
    for (int64_t j0 = i0; j0 < n; j0 += kB)
      for (int64_t i = i0; i < std::min(i0 + kB, n); ++i)
        for (int64_t j = std::max(j0, i + 1); j < std::min(j0 + kB, n); ++j)
          C[j * n + i] = C[i * n + j];
  return C;
}

}  // namespace

hipError_t amg_build(const DevMesh& m, hipStream_t s,
                     void* (*alloc)(void* ctx, size_t bytes), void* ctx,
                     AmgDev& d, std::string& msg) {
  d = AmgDev{};
  hipError_t e;
  // level 0: K on the free nodes without its zeros, from the device copy
  const int64_t ns = m.k_nslices;
  std::vector<int32_t> sptr(ns + 1);
  if ((e = hipMemcpyAsync(sptr.data(), m.kz.sptr, sizeof(int32_t) * (ns + 1),
                          hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  const int64_t np = sptr[ns];
  const bool packed = m.kz.code != nullptr;
  std::vector<int32_t> scol(np);   // (packed: the code words)
  std::vector<double> sval(packed ? kDictMax : np);
  if ((e = hipMemcpyAsync(scol.data(), packed ? (const void*)m.kz.code : m.kz.col,
                          sizeof(int32_t) * np, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipMemcpyAsync(sval.data(), packed ? m.kz.dict : m.kz.val,
                          sizeof(double) * sval.size(), hipMemcpyDeviceToHost, s)) !=
          hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return e;
  std::vector<HCsr> A(1);
  A[0].n = A[0].m = m.n_free;
  A[0].rp.assign(m.n_free + 1, 0);
  A[0].ci.reserve(np);
  A[0].v.reserve(np);
  for (int64_t r = 0; r < m.n_free; ++r) {
    const int64_t sl = r / kSell, lane = r % kSell;
    const int64_t w = (sptr[sl + 1] - sptr[sl]) / kSell;
    for (int64_t j = 0; j < w; ++j) {
      const int64_t p = sptr[sl] + j * kSell + lane;
      const uint32_t c = (uint32_t)scol[p];
      const double v = packed ? sval[c >> kColBits] : sval[p];
      if (v != 0.0) {  // (padding entries are zeros)
        A[0].ci.push_back((int32_t)(packed ? c & ((1u << kColBits) - 1) : c));
        A[0].v.push_back(v);
      }
    }
    A[0].rp[r + 1] = (int64_t)A[0].ci.size();
  }
  std::vector<HCsr> Ps, Rs;
  std::vector<std::vector<double>> diag;
  std::vector<double> omega;
  double theta = 0.08;
  // (at least one level with a smoother: its first kernel holds the
  // stopping test)
  while ((A.back().n > kAmgCoarseMax || Ps.empty()) &&
         (int)Ps.size() < kAmgMaxLevels) {
    const HCsr& Al = A.back();
    diag.push_back(diag_of(Al));
    const std::vector<double>& dl = diag.back();
    for (double v : dl)
      if (!(v > 0.0)) {
        msg = "amg: operator diagonal not positive";
        return hipErrorInvalidValue;
      }
    int64_t nc = 0;
    const std::vector<int32_t> agg = aggregate(Al, dl, theta, nc);
    if (nc >= Al.n) break;  // no coarsening possible
    omega.push_back(4.0 / (3.0 * lambda_max(Al, dl)));
    const HCsr P = smoothed_p(Al, dl, agg, nc, omega.back());
    HCsr AP = multiply(Al, P);
    HCsr next = symmetrize(multiply(transpose(P), AP));
    Ps.push_back(smooth_again(P, std::move(AP), dl, omega.back()));
    Rs.push_back(transpose(Ps.back()));
    A.push_back(std::move(next));  // (Al and dl end here)
    theta *= 0.5;
  }
  for (const auto* v : {&A, &Ps, &Rs})
    for (const HCsr& M : *v)
      if (M.rp[M.n] >= (int64_t)1 << 31) {
        msg = "amg: level matrix too large for 32-bit offsets";
        return hipErrorInvalidValue;
      }
  int L = (int)Ps.size();
  const HCsr& Ac = A.back();
  if (L == 0 || Ac.n > 4 * kAmgCoarseMax) {
    msg = "amg: the operator does not coarsen";
    return hipErrorInvalidValue;
  }
  std::vector<double> dense(Ac.n * Ac.n, 0.0);
  for (int64_t i = 0; i < Ac.n; ++i)
    for (int64_t p = Ac.rp[i]; p < Ac.rp[i + 1]; ++p) dense[i * Ac.n + Ac.ci[p]] = Ac.v[p];
  if (!spd_inverse(dense, Ac.n)) {
    msg = "amg: coarsest operator not positive definite";
    return hipErrorInvalidValue;
  }
  int64_t n_coarse = Ac.n;
  for (int l = 0; l <= L; ++l) d.rows[l] = A[l].n;
  if (L >= 2 && A[L - 1].n <= kAmgDenseMax &&
      Ps[L - 1].rp[A[L - 1].n] * A[L - 1].n <= kDenseWork) {
    --L;
    dense = dense_cycle(A[L], diag[L], omega[L], Ps[L], Rs[L], dense);
    n_coarse = A[L].n;
  }
  // upload
  auto up = [&](const void* src, size_t bytes) -> void* {
    void* p = alloc(ctx, bytes);
    if (p && bytes &&
        hipMemcpyAsync(p, src, bytes, hipMemcpyHostToDevice, s) != hipSuccess)
      return nullptr;
    return p;
  };
  // short rows: SELL, one lane per row; long rows: CSR with enough lanes
  // per row that each lane sums 3 to 6 entries, one trip with all its loads
  // in flight (lpr: as given, else by the row length)
  auto up_sell = [&](const HCsr& M, SellMat& out, int lpr = 0) -> bool {
    const double avg = M.n ? (double)M.rp[M.n] / (double)M.n : 0.0;
    out.nrows = M.n;
    out.lpr = lpr ? lpr : avg <= 24.0 ? 1 : avg <= 48.0 ? 8 : avg <= 96.0 ? 16 : avg <= 192.0 ? 32 : 64;
    if (out.lpr == 1) {
      const HSell S = to_sell(M);
      out.nslices = S.nslices;
      out.v.sptr = (const int32_t*)up(S.sptr.data(), sizeof(int32_t) * S.sptr.size());
      out.v.col = (const int32_t*)up(S.col.data(), sizeof(int32_t) * std::max<size_t>(S.col.size(), 1));
      out.v.val = (const double*)up(S.val.data(), sizeof(double) * std::max<size_t>(S.val.size(), 1));
      const std::vector<float> v32(S.val.begin(), S.val.end());
      out.v.val32 = (const float*)up(v32.data(), sizeof(float) * std::max<size_t>(v32.size(), 1));
      // (synchronized before the host copies go out of scope)
      return out.v.sptr && out.v.col && out.v.val && out.v.val32 &&
             hipStreamSynchronize(s) == hipSuccess;
    }
    std::vector<int32_t> rp(M.rp.begin(), M.rp.end());
    out.nslices = 0;
    out.v.sptr = (const int32_t*)up(rp.data(), sizeof(int32_t) * rp.size());
    out.v.col = (const int32_t*)up(M.ci.data(), sizeof(int32_t) * std::max<size_t>(M.ci.size(), 1));
    out.v.val = (const double*)up(M.v.data(), sizeof(double) * std::max<size_t>(M.v.size(), 1));
    const std::vector<float> v32(M.v.begin(), M.v.end());
    out.v.val32 = (const float*)up(v32.data(), sizeof(float) * std::max<size_t>(v32.size(), 1));
    return out.v.sptr && out.v.col && out.v.val && out.v.val32 &&
           hipStreamSynchronize(s) == hipSuccess;
  };
  d.n_levels = L;
  for (int l = 0; l < L; ++l) {
    AmgLevel& lv = d.lv[l];
    if (l == 0) {
      lv.A = SellMat{m.n_free, m.k_nslices, 1, m.kz};
      lv.invdiag = m.invdiag;
      lv.invdiag32 = m.invdiag32;
    } else {
      if (!up_sell(A[l], lv.A)) return hipErrorOutOfMemory;
      std::vector<double> inv(A[l].n);
      for (int64_t i = 0; i < A[l].n; ++i) inv[i] = 1.0 / diag[l][i];
      const std::vector<float> inv32(inv.begin(), inv.end());
      lv.invdiag = (const double*)up(inv.data(), sizeof(double) * inv.size());
      lv.invdiag32 = (const float*)up(inv32.data(), sizeof(float) * inv32.size());
      if (!lv.invdiag || !lv.invdiag32 || hipStreamSynchronize(s) != hipSuccess)
        return hipErrorOutOfMemory;
    }
    lv.omega = omega[l];
    // (one kernel sums a row of A and of Ps: the same lanes per row)
    if (!up_sell(Ps[l], lv.Ps, lv.A.lpr) || !up_sell(Rs[l], lv.Rs)) return hipErrorOutOfMemory;
    const size_t vb = sizeof(double) * (size_t)A[l].n;
    lv.b = l > 0 ? (double*)alloc(ctx, vb) : nullptr;
    lv.t = l > 0 ? (double*)alloc(ctx, vb) : nullptr;
    lv.b32 = l > 0 ? (float*)alloc(ctx, vb / 2) : nullptr;
    lv.t32 = l > 0 ? (float*)alloc(ctx, vb / 2) : nullptr;
    if (l > 0 && (!lv.b || !lv.t || !lv.b32 || !lv.t32)) return hipErrorOutOfMemory;
  }
  d.n_coarse = n_coarse;
  d.coarse_inv = (const double*)up(dense.data(), sizeof(double) * dense.size());
  const std::vector<float> dense32(dense.begin(), dense.end());
  d.coarse_inv32 = (const float*)up(dense32.data(), sizeof(float) * dense32.size());
  d.coarse_b = (double*)alloc(ctx, sizeof(double) * n_coarse);
  d.coarse_x = (double*)alloc(ctx, sizeof(double) * n_coarse);
  d.coarse_b32 = (float*)alloc(ctx, sizeof(float) * n_coarse);
  d.coarse_x32 = (float*)alloc(ctx, sizeof(float) * n_coarse);
  if (!d.coarse_inv || !d.coarse_b || !d.coarse_x || !d.coarse_inv32 ||
      !d.coarse_b32 || !d.coarse_x32)
    return hipErrorOutOfMemory;
  AmgDev* dd = (AmgDev*)alloc(ctx, sizeof(AmgDev));
  if (!dd) return hipErrorOutOfMemory;
  d.dev = dd;
  if ((e = hipMemcpyAsync(dd, &d, sizeof d, hipMemcpyHostToDevice, s)) != hipSuccess)
    return e;
  return hipStreamSynchronize(s);
}

}  // namespace fp
