// Data handed from one workgroup to another inside a launch: device-scope
// accesses, which go past the per-XCD caches, with the fences that the memory
// model asks for between the data and the flag.  The fences are of workgroup
// scope: they order the compiler's accesses and cost nothing, where ones of
// device scope would write back or invalidate an L2 that the other workgroups
// are using (in the particle kernel of a small step 10 us).  What they leave
// to the hardware, that a wave's stores have arrived before its flag goes out,
// is the wait between them; a wave's loads return in order.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/femocs_pic.h"

namespace fp {

template <typename T>
__device__ inline void dev_put(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline T dev_get(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Ahead of a flag: this wave's stores have arrived.
__device__ inline void hand_over() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
}
// Behind a flag that has been seen.
__device__ inline void take_over() {
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The running sums of a step's emission, in the order of the faces, after
// one trip of its workgroups (lost: without those of a trip that was waited
// for in vain).
struct EmitSums {
  long long offset, n_clamp, lost;
  double cur, F_sum, F_max;
};
// The same in memory, with that trip's number plus one as the flag.
constexpr int kEmitWords = sizeof(EmitSums) / sizeof(unsigned long long);
struct EmitSlot {
  unsigned long long word[kEmitWords];
  int32_t flag, pad;
};

// What a trip hands to the next (one lane).
__device__ inline void sums_put(EmitSlot* p, const EmitSums& v, int32_t flag) {
  unsigned long long w[kEmitWords];
  __builtin_memcpy(w, &v, sizeof v);
#pragma unroll
  for (int k = 0; k < kEmitWords; ++k) dev_put(p->word + k, w[k]);
  hand_over();
  dev_put(&p->flag, flag);
}

// A wait is bounded: a flag not seen in time (never expected) ends it.
constexpr int kEmitSpin = 1 << 22;

// What a trip takes from the one before (one lane); lost when it does not
// come.
__device__ inline void sums_get(const EmitSlot* p, EmitSums& v, int32_t flag,
                                int spin = kEmitSpin) {
  for (int it = 0; it < spin; ++it) {
    if (dev_get(&p->flag) == flag) {
      take_over();
      unsigned long long w[kEmitWords];
#pragma unroll
      for (int k = 0; k < kEmitWords; ++k) w[k] = dev_get(p->word + k);
      __builtin_memcpy(&v, w, sizeof v);
      return;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  v = EmitSums{};  // (offsets stay within the arrays)
  v.lost = 1;
}

// What a step injects, by the sums of all its trips: total superparticles, of
// which fit have a slot behind the base slots in use.  After a lost trip the
// offsets of the faces are not those of one scan, so nothing is injected.
struct EmitEnd {
  long long total, fit;
  int32_t status;
};
__host__ __device__ inline EmitEnd emit_end(const EmitSums& sum, long long base,
                                            long long capacity) {
  EmitEnd e;
  e.total = sum.lost ? 0 : sum.offset;
  e.fit = capacity - base;
  if (e.fit > e.total) e.fit = e.total;
  if (e.fit < 0) e.fit = 0;
  e.status = sum.lost ? PIC_E_DEVICE : e.total > e.fit ? PIC_E_CAPACITY : PIC_OK;
  return e;
}

}  // namespace fp
