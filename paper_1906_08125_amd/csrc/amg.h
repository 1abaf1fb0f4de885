// Smoothed-aggregation algebraic multigrid as a CG preconditioner for the
// FP64 solve (an alternative to Jacobi; the paper names no preconditioner).
#pragma once
#include <vector>

#include "common.h"
#include "solver.h"

namespace fp {

constexpr int kAmgMaxLevels = 8;
constexpr int kAmgCoarseMax = 512;  // the coarsest operator is inverted densely
// A last smoothed level of at most this many rows is applied with all below
// it as one dense matrix (see AmgDev): three dependent launches near the
// floor (18 us at 1,089 rows) against one product that reads 5 to 16 MB.
// The price is memory: 12 bytes an entry (FP64 and FP32), so up to 50 MB a
// handle where the inverse of at most 512 rows took 3.
constexpr int kAmgDenseMax = 2048;

// A sparse matrix of the hierarchy.  lpr = 1: the sliced ELLPACK layout of
// the solver (SellView, one lane per row), for short rows; packed on the
// finest level where K is.  lpr > 1 (a power of two up to 64): CSR with lpr
// lanes per row and a shuffle reduction, for the long rows of the Galerkin
// operators and restrictions.
struct SellMat {
  int64_t nrows, nslices;  // (nslices: SELL only)
  int lpr;
  SellView v;              // (CSR: sptr holds the row offsets [nrows + 1])
};

// One level of the hierarchy.  Level 0 is K on the free nodes; b of level 0
// is the CG residual and its smoothed output is the CG vector u.
//
// The V(1,1)-cycle with weighted-Jacobi smoothing is applied with its
// products folded at setup.  Pre-smoothing from zero, x = w D^-1 b, leaves
// the residual (I - w A D^-1) b, so the next level's right-hand side is
//   Rs b,  Rs = P^T (I - w A D^-1) = Ps^T,  Ps = (I - w D^-1 A) P,
// and post-smoothing x + P y gives
//   2 w D^-1 b - w D^-1 A (w D^-1 b) + Ps y.
// A level is then one launch down and one up (two and two before: the
// smoothing and the transfer each way), and stores neither x nor the
// residual.  Ps has the pattern of A P, which the Galerkin product forms
// anyway.
struct AmgLevel {
  SellMat A;
  const double* invdiag;
  double omega;   // Jacobi weight 4 / (3 lambda_max(D^-1 A))
  SellMat Ps;     // smoothed prolongation from the next level (rows: this)
  SellMat Rs;     // its transpose (rows: the next level)
  double* b;      // right-hand side (levels > 0)
  double* t;      // the cycle's result (levels > 0)
  // FP32 copies for the FP32 V-cycle (mixed precision)
  const float* invdiag32;
  float *b32, *t32;
};
__device__ inline void globalize(AmgLevel& a, const AmgLevel& from) {
  globalize(a.A.v, from.A.v);
  globalize(a.Ps.v, from.Ps.v);
  globalize(a.Rs.v, from.Rs.v);
  FP_GLOBAL(invdiag); FP_GLOBAL(b); FP_GLOBAL(t); FP_GLOBAL(invdiag32); FP_GLOBAL(b32);
  FP_GLOBAL(t32);
}

struct AmgDev {
  int n_levels;   // levels with a smoother; the dense coarsest level follows
  AmgLevel lv[kAmgMaxLevels];
  // The coarsest level: the inverse of its operator, or, where the last
  // smoothed level is small, that level's whole cycle
  // 2 w D^-1 - w^2 D^-1 A D^-1 + Ps inv Rs (the same preconditioner).
  int64_t n_coarse;
  const double* coarse_inv;  // [n_coarse][n_coarse], row-major
  double* coarse_b;
  double* coarse_x;
  const float* coarse_inv32;
  float* coarse_b32;
  float* coarse_x32;
  int64_t rows[kAmgMaxLevels + 1];  // rows per level (the coarsest last)
  // device copy of this descriptor (written last by amg_build), read by
  // the batched launches, which find each instance's hierarchy through
  // CgArgs::amg_dev
  const AmgDev* dev;
};

// Builds the hierarchy of the FP64 stiffness of m on the host (strength of
// connection, three-phase aggregation, Jacobi-smoothed prolongation,
// Galerkin products, dense inverse of the coarsest operator) and uploads it
// with alloc().  Returns hipSuccess and fills d, or an error.
hipError_t amg_build(const DevMesh& m, hipStream_t s,
                     void* (*alloc)(void* ctx, size_t bytes), void* ctx,
                     AmgDev& d, std::string& msg);

// n iterations of CG preconditioned by one V(1,1)-cycle, in the
// Chronopoulos-Gear ordering [V-cycle, w = K u, update], numbered by the
// device counters of the control word; no report.  The first V-cycle
// kernel of every iteration after the first tests the recursive residual.
// With a.amg32 the V-cycle runs in FP32 (level matrices, diagonals and
// vectors; the CG recursion stays FP64).  Levels below the finest launch
// grids sized to their rows.
hipError_t amg_launch_iters(const CgArgs& a, const AmgDev& d, int n,
                            hipStream_t s);

// n such iterations of several instances at once: every V-cycle stage (a
// level's smoothing, restriction, prolongation; the coarse solve; the
// product; the update) is one launch over all instances i with on[i], each
// getting the workgroups its own launch would have.  dargs: the instances'
// solver arguments in device memory (index i), hargs: the same on the host
// (their amg set, all alike in amg32).
hipError_t amg_batch_iters(const CgArgs* dargs, const std::vector<const CgArgs*>& hargs,
                           const std::vector<char>& on, int n, hipStream_t s);

}  // namespace fp
