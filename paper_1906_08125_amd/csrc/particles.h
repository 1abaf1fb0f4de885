// Launch interface of the particle kernels.
#pragma once
#include "common.h"

namespace fp {

constexpr int kAccFields = kStepCounters;  // counters per block row (see acc_flush)

struct EmitConsts {
  double a_fn, b_fn, c_s, j_unit;
};

constexpr int kParticleBlock = 256;  // threads of a particle workgroup

struct StepArgs {
  DevMesh m;
  void *x, *y, *z, *vx, *vy, *vz;  // double, or float when f32
  double* w;
  int32_t *tet, *birth;
  int64_t* id;
  int32_t* n_slots;
  const void* E;        // nodal field [4 n_nodes], double or float (f32)
  int f32;              // mixed precision: float particles and field
  int64_t* charge;      // [n_nodes]
  const double* s_face; // [n_emit] or null
  const int32_t* offsets;  // [n_emit + 1] exclusive scan of counts
  int32_t* queue;       // [capacity] fallback queue
  StepScratch* scratch;
  pic_step_stats* stats;
  int64_t* acc_rows;    // [kAccFields][acc_stride] per-block counters
  int acc_stride;       // rows of both kernels (field-major layout)
  double Q, dt, qm_dt;
  uint64_t seed;
  uint64_t instance;
  int64_t step;
  int g_push;           // workgroups of the push role (the rest inject)
  int n_blocks;         // workgroups of the particle kernel (the fallback
                        // kernel's counter rows follow theirs)
  // null, or the previous solve's control state: a launch enqueued before
  // that solve's outcome is known does nothing unless the solve has ended
  // (CG_DONE or CG_NOCONV)
  const int32_t* gate;
  // cell field mode: the field in tet t is -(grad phi)_t, from phi
  int cell;
  const double* phi;
};

struct EmitArgs {
  DevMesh m;
  const void* E;        // double [4 n_nodes], or float when f32
  int f32;
  EmitConsts c;
  double phi_w, j_scale, dt, w_sp;
  uint64_t seed, instance;
  int64_t step;
  int64_t capacity;
  int32_t* counts;   // [n_emit] or null (rate only)
  int32_t* offsets;  // [n_emit + 1]
  int32_t* n_slots;
  StepScratch* scratch;
  pic_step_stats* stats;  // or null
  double* rate;           // or null
  double* face_F;         // or null
  int64_t* clear;         // node charges cleared by k_begin, or null
  int64_t n_clear;
  const int32_t* gate;    // as StepArgs::gate
  int cell;               // as StepArgs::cell (face field of the face's tet)
  const double* phi;
  const int32_t* counts_in;  // frozen per-face counts (replace the rounding) or null
  int32_t* counts_out;       // the counts used, or null
};

__device__ inline void globalize(StepArgs& a, const StepArgs& from) {
  globalize(a.m, from.m);
  FP_GLOBAL(x); FP_GLOBAL(y); FP_GLOBAL(z); FP_GLOBAL(vx); FP_GLOBAL(vy); FP_GLOBAL(vz);
  FP_GLOBAL(w); FP_GLOBAL(tet); FP_GLOBAL(birth); FP_GLOBAL(id); FP_GLOBAL(n_slots);
  FP_GLOBAL(E); FP_GLOBAL(charge); FP_GLOBAL(s_face); FP_GLOBAL(offsets); FP_GLOBAL(queue);
  FP_GLOBAL(scratch); FP_GLOBAL(stats); FP_GLOBAL(acc_rows); FP_GLOBAL(gate); FP_GLOBAL(phi);
}
__device__ inline void globalize(EmitArgs& a, const EmitArgs& from) {
  globalize(a.m, from.m);
  FP_GLOBAL(E); FP_GLOBAL(counts); FP_GLOBAL(offsets); FP_GLOBAL(n_slots); FP_GLOBAL(scratch);
  FP_GLOBAL(stats); FP_GLOBAL(rate); FP_GLOBAL(face_F); FP_GLOBAL(clear); FP_GLOBAL(gate);
  FP_GLOBAL(phi); FP_GLOBAL(counts_in); FP_GLOBAL(counts_out);
}

struct LocateArgs {
  DevMesh m;
  int64_t n;
  const double *x, *y, *z;
  int32_t* tet;
  uint8_t* where;
  int32_t* queue;
  int32_t* n_queue;
};

struct DepositArgs {
  DevMesh m;
  int64_t n;
  const double *x, *y, *z, *w;
  const int32_t* tet;
  int64_t* charge;
};

hipError_t launch_begin(const EmitArgs& a, int grid, hipStream_t s);
// Workgroups of the particle kernel (FP64 or FP32 storage; packed tet records
// or not, built for so many waves per SIMD) resident on one compute unit at
// once, by the runtime's occupancy calculator (0 on error).
int particle_blocks_per_cu(int f32, int packed, int waves);
// e: the step's emission, computed by the first workgroups while the others
// push (the injecting ones wait for it).  waves: 4, or 5 (packed records only;
// else taken as 4).
hipError_t launch_particles(const StepArgs& a, const EmitArgs& e, int g_push,
                            int g_inj, int waves, hipStream_t s);
hipError_t launch_seed_build(const DevMesh& m, int grid, hipStream_t s);
hipError_t launch_emit(const EmitArgs& a, hipStream_t s);
hipError_t launch_fallback(const StepArgs& a, int grid, hipStream_t s);
hipError_t launch_locate(const LocateArgs& a, int grid, hipStream_t s);
hipError_t launch_deposit(const DepositArgs& a, int grid, hipStream_t s);

// Batched launches over the instances of device arrays E[] / A[] with the
// block schedules given (one schedule per kernel kind).
hipError_t launch_begin_b(const EmitArgs* E, const BatchMap& map, int grid,
                          hipStream_t s);
// (the instances of one launch all have packed tet records, or none has)
hipError_t launch_particles_b(const StepArgs* A, const EmitArgs* E, const BatchMap& map,
                              int f32, int packed, hipStream_t s);
hipError_t launch_fallback_b(const StepArgs* A, const BatchMap& map, int grid,
                             hipStream_t s);
}  // namespace fp
