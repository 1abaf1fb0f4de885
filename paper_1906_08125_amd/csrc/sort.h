// Launch interface of the particle re-sort (by tet, with compaction).
#pragma once
#include <vector>

#include "common.h"

namespace fp {

constexpr int kSortBins = 256;   // 8-bit digits
constexpr int kSortTile = 4096;  // items per workgroup of a pass

struct SortArgs {
  int64_t n_tets;
  int32_t* n_slots;       // in: slots in use, out: live particles
  int32_t* n_live;        // scratch scalar
  int ntiles;             // sort_tiles(capacity)
  pic_step_stats* stats;  // or null
  // particle arrays (x, y, z, vx, vy, vz of real_bytes each)
  void* real[6];
  int real_bytes;
  double* w;
  int32_t* tet;
  int32_t* birth;
  int64_t* id;
  // scratch
  uint32_t* key[2];
  uint32_t* val[2];
  uint32_t* hist;         // [kSortBins][sort_tiles(capacity)]
  uint32_t* total;        // [kSortBins]
  void* s_real[6];
  double* s_w;
  int32_t* s_tet;
  int32_t* s_birth;
  int64_t* s_id;
};

__device__ inline void globalize(SortArgs& a, const SortArgs& from) {
  for (int f = 0; f < 6; ++f) {
    FP_GLOBAL(real[f]);
    FP_GLOBAL(s_real[f]);
  }
  for (int k = 0; k < 2; ++k) {
    FP_GLOBAL(key[k]);
    FP_GLOBAL(val[k]);
  }
  FP_GLOBAL(n_slots); FP_GLOBAL(n_live); FP_GLOBAL(stats); FP_GLOBAL(w); FP_GLOBAL(tet);
  FP_GLOBAL(birth); FP_GLOBAL(id); FP_GLOBAL(hist); FP_GLOBAL(total); FP_GLOBAL(s_w);
  FP_GLOBAL(s_tet); FP_GLOBAL(s_birth); FP_GLOBAL(s_id);
}

// copyback: the sorted particles are copied back into the arrays they came
// from (real, w, ...); else they stay in the scratch arrays (s_real, s_w,
// ...), which the caller then uses as the particle arrays, and only the
// slot count is set.
hipError_t sort_particles(const SortArgs& a, int n_cu, hipStream_t s,
                          bool copyback = true);
// the s_* arrays copied into real, w, ... for the *n_slots slots in use
hipError_t copy_particles(const SortArgs& a, int n_cu, hipStream_t s);
// The re-sorts (with the copy back) of the instances due[i] of a batch of one
// precision, in shared launches; A: their arguments on the device, host: the
// same on the host.  Ten steps of six tips with one re-sort each: 1959 us with
// 66 launches of the re-sorts one after another, 1529 so.
hipError_t sort_particles_b(const SortArgs* A, const std::vector<const SortArgs*>& host,
                            const std::vector<char>& due, int n_cu, hipStream_t s);
size_t sort_scratch_bytes(int64_t capacity, int real_bytes);
int sort_tiles(int64_t capacity);

}  // namespace fp
