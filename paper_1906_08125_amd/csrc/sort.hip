// Particle re-sort by containing tet with compaction: a stable LSD radix
// sort of (key = tet, or n_tets for a free slot; value = slot index) with
// 8-bit digits, then a gather of every particle array into scratch and a
// copy back.
//
// One pass over a digit is three launches (two up to kFoldTiles tiles):
//   k_sort_hist     digit counts of every tile of kSortTile items;
//   k_sort_scan     one workgroup per digit: exclusive scan of that digit's
//                   counts over the tiles, and the digit's total;
//   k_sort_scatter  every wave ranks the 64 items of a round among the
//                   lanes with the same digit (eight ballots; lanes are in
//                   item order, so the rank is stable), per-wave digit
//                   counters in LDS carry the rank across rounds and waves,
//                   the tile is reordered by digit in LDS and written out in
//                   runs that are contiguous in the destination.
// The first pass takes its keys from the tets themselves (its values are the
// slot indices).  No atomic operation decides an order, so the permutation
// (and everything computed after it) is deterministic.
//
// The re-sorts of a batch share their launches: the workgroups of the
// instances that are due follow one another (BatchMap), each instance with
// its own arguments and counts.
#include <algorithm>

#include "common.h"
#include "sort.h"

namespace fp {

namespace {

constexpr int kBins = kSortBins;
// A tile is ranked by 16 waves of four rounds: a pass is bound by the
// latency of its phases (about one workgroup per CU at 1e6 items), and a
// round's rank waits for the one before it.  (1e6 superparticles, three
// passes: 27 us a pass with 4 waves of sixteen rounds, 26 so; with the keys
// from the tets and the count left to the gather the re-sort takes two
// launches less: ten steps of 1e4 superparticles 493 -> 472 us.)
constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kRounds = kSortTile / kThreads;  // rounds of 64 items per wave
static_assert(kThreads % kBins == 0, "kParts threads per digit in the tile sums");
static_assert(kSortTile == kWaves * kRounds * 64, "tile = waves x rounds x 64");
constexpr int kParts = kThreads / kBins;
constexpr int kScanThreads = 256;
constexpr int kMoveThreads = 256;
// Up to this many tiles the scatter sums the tiles' counts itself: a
// workgroup then reads 64 KB of counts at most, against a launch of 5 us.
constexpr int kFoldTiles = 64;

// Exclusive prefix of v over the threads of the workgroup (thread order);
// *total receives the sum.  Every thread must call it.
template <int W>
__device__ inline uint32_t block_exscan(uint32_t v, uint32_t* wsum,
                                        uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = __shfl_up(inc, off, 64);
    if (lane >= off) inc += o;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    if (w < wave) before += wsum[w];
    all += wsum[w];
  }
  __syncthreads();
  *total = all;
  return before + inc - v;
}

// Buffer src of a pair.  (A selection: an index that the compiler does not
// know would put a batch's arguments into scratch memory.)
__device__ inline uint32_t* buffer(uint32_t* const* pair, int src) {
  return src ? pair[1] : pair[0];
}

// Which pass: FIRST keys are the tets, else those of buffer src; the digit
// is the eight bits from shift on; the output goes to buffer src ^ 1.
template <bool FIRST>
__device__ inline uint32_t sort_key(const SortArgs& a, int src, int64_t i) {
  if constexpr (FIRST) {
    const int32_t t = a.tet[i];
    return t < 0 ? (uint32_t)a.n_tets : (uint32_t)t;
  } else {
    return buffer(a.key, src)[i];
  }
}

// Digit counts of tile b: hist[digit * ntiles + b].  (Integer counts: the
// order of the LDS additions does not matter.)  The first pass also leaves
// the incoming slot count in n_live, from which the gather takes it: the
// gather sets n_slots.
template <bool FIRST>
__device__ inline void hist_body(const SortArgs& a, VB vb, int src, int shift) {
  __shared__ uint32_t cnt[kBins];
  const int64_t n = *a.n_slots;
  if (FIRST && vb.id == 0 && threadIdx.x == 0) *a.n_live = (int32_t)n;
  if (threadIdx.x < kBins) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)vb.id * kSortTile + threadIdx.x;
  uint32_t k[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int64_t i = base + r * kThreads;
    k[r] = i < n ? sort_key<FIRST>(a, src, i) : 0u;
  }
#pragma unroll
  for (int r = 0; r < kRounds; ++r)
    if (base + r * kThreads < n) atomicAdd(&cnt[(k[r] >> shift) & (kBins - 1)], 1u);
  __syncthreads();
  if (threadIdx.x < kBins)
    a.hist[(int64_t)threadIdx.x * vb.n + vb.id] = cnt[threadIdx.x];
}

// Workgroup d: exclusive scan of hist[d][0..ntiles) in place, total[d].
__device__ inline void scan_body(const SortArgs& a, VB vb) {
  __shared__ uint32_t wsum[kScanThreads / 64];
  uint32_t* row = a.hist + (int64_t)vb.id * a.ntiles;
  uint32_t carry = 0;
  for (int j0 = 0; j0 < a.ntiles; j0 += kScanThreads) {
    const int j = j0 + threadIdx.x;
    const uint32_t v = j < a.ntiles ? row[j] : 0u;
    uint32_t chunk;
    const uint32_t ex = block_exscan<kScanThreads / 64>(v, wsum, &chunk);
    if (j < a.ntiles) row[j] = carry + ex;
    carry += chunk;
  }
  if (threadIdx.x == 0) a.total[vb.id] = carry;
}

template <bool FIRST>
__device__ inline void scatter_body(const SortArgs& a, VB vb, int src, int shift) {
  __shared__ uint32_t wc[kWaves][kBins];  // per-wave digit counts, then bases
  __shared__ uint32_t part[2][kParts][kBins];
  __shared__ uint32_t tstart[kBins];      // first slot of a digit in the tile
  __shared__ uint32_t gbase[kBins];       // destination of that slot
  __shared__ uint32_t s_key[kSortTile];
  __shared__ uint32_t s_val[kSortTile];
  __shared__ uint32_t wsum[kWaves];
  const int64_t n = *a.n_slots;
  const int64_t base = (int64_t)vb.id * kSortTile;
  if (base >= n) return;  // the whole workgroup: no barrier is skipped
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool fold = vb.n <= kFoldTiles;
  // wave w owns items [w, w + 1) * kRounds * 64 of the tile, round r the
  // 64 items from r * 64 on: lane order is item order
  const int64_t w0 = base + (int64_t)wave * kRounds * 64 + lane;
  uint32_t kr[kRounds], vr[kRounds], rk[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int64_t i = w0 + r * 64;
    kr[r] = i < n ? sort_key<FIRST>(a, src, i) : 0u;
    vr[r] = i < n ? (FIRST ? (uint32_t)i : buffer(a.val, src)[i]) : 0u;
  }
  for (int b = lane; b < kBins; b += 64) wc[wave][b] = 0;
  const int dig = threadIdx.x % kBins;
  if (fold) {
    // kParts threads per digit: its counts in the tiles before this one, and
    // in all of them
    const int p = threadIdx.x / kBins;
    const uint32_t* row = a.hist + (int64_t)dig * vb.n;
    uint32_t before = 0, all = 0;
    for (int j = p; j < vb.n; j += kParts) {
      const uint32_t c = row[j];
      before += j < vb.id ? c : 0u;
      all += c;
    }
    part[0][p][dig] = before;
    part[1][p][dig] = all;
  }
  __syncthreads();
  const uint64_t below_me = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const bool ok = w0 + r * 64 < n;
    const uint32_t d = (kr[r] >> shift) & (kBins - 1);
    // lanes holding an item with the same digit as this lane
    uint64_t peers = __ballot(ok);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const bool one = (d >> bit) & 1u;
      const uint64_t m = __ballot(one);
      peers &= one ? m : ~m;
    }
    const uint32_t prev = wc[wave][d];
    rk[r] = prev + (uint32_t)__popcll(peers & below_me);
    // the highest lane of each digit group advances the wave's counter
    // (after every lane of the wave has read it: LDS keeps a wave's order)
    if (ok && (peers >> lane) == 1ull)
      wc[wave][d] = prev + (uint32_t)__popcll(peers);
  }
  __syncthreads();
  {
    // thread b < kBins: the digit's wave bases inside the tile, its first
    // slot in the tile and the destination of that slot
    const int b = threadIdx.x;
    const bool on = b < kBins;
    uint32_t cnt = 0, tot = 0, before = 0;
    if (on) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = wc[w][b];
        wc[w][b] = cnt;
        cnt += c;
      }
      if (fold) {
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
          before += part[0][p][b];
          tot += part[1][p][b];
        }
      } else {
        before = a.hist[(int64_t)b * vb.n + vb.id];
        tot = a.total[b];
      }
    }
    uint32_t all;
    const uint32_t ts = block_exscan<kWaves>(cnt, wsum, &all);
    const uint32_t bb = block_exscan<kWaves>(tot, wsum, &all);
    if (on) {
      tstart[b] = ts;
      gbase[b] = bb + before;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    if (w0 + r * 64 >= n) continue;
    const uint32_t d = (kr[r] >> shift) & (kBins - 1);
    const uint32_t p = tstart[d] + wc[wave][d] + rk[r];
    s_key[p] = kr[r];
    s_val[p] = vr[r];
  }
  __syncthreads();
  const int m = n - base < kSortTile ? (int)(n - base) : kSortTile;
  uint32_t* okey = buffer(a.key, src ^ 1);
  uint32_t* oval = buffer(a.val, src ^ 1);
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int j = r * kThreads + (int)threadIdx.x;
    if (j < m) {
      const uint32_t kk = s_key[j];
      const uint32_t d = (kk >> shift) & (kBins - 1);
      const uint32_t pos = gbase[d] + ((uint32_t)j - tstart[d]);
      okey[pos] = kk;
      oval[pos] = s_val[j];
    }
  }
}

// One superparticle, all of its loads before its stores.
template <typename T>
__device__ inline void move_one(void* const* to, double* to_w, int32_t* to_t, int32_t* to_b,
                                int64_t* to_i, int64_t j, void* const* from,
                                const double* w, const int32_t* t, const int32_t* b,
                                const int64_t* id, int64_t s) {
  T r[6];
#pragma unroll
  for (int f = 0; f < 6; ++f) r[f] = reinterpret_cast<const T*>(from[f])[s];
  const double w_ = w[s];
  const int32_t t_ = t[s], b_ = b[s];
  const int64_t i_ = id[s];
#pragma unroll
  for (int f = 0; f < 6; ++f) reinterpret_cast<T*>(to[f])[j] = r[f];
  to_w[j] = w_;
  to_t[j] = t_;
  to_b[j] = b_;
  to_i[j] = i_;
}

// Gather every particle array into scratch in sorted order; the last live
// position sets the new slot count.  The sorted order is close to the
// previous one, so the sources of a run of outputs lie in a narrow window:
// each XCD (block index mod 8) takes one contiguous eighth of the outputs,
// so that a source line is fetched into one XCD's L2 rather than into
// every XCD whose blocks interleave over it.
template <typename T>
__device__ inline void gather_body(const SortArgs& a, VB vb, int src) {
  const int64_t n = *a.n_live;  // (the incoming slot count, see hist_body)
  const uint32_t* key = buffer(a.key, src);
  const uint32_t* val = buffer(a.val, src);
  const int parts = vb.n % 8 == 0 ? 8 : 1;
  const int part = vb.id % parts;
  const int64_t per_part = parts == 8 ? (n + 7) >> 3 : n;
  const int64_t lo = part * per_part;
  const int64_t hi = lo + per_part < n ? lo + per_part : n;
  const int64_t stride = (int64_t)(vb.n / parts) * blockDim.x;
  auto count = [&](int64_t c) {
    *a.n_slots = (int32_t)c;
    if (a.stats) a.stats->n_slots = c;
  };
  if (n == 0 && vb.id == 0 && threadIdx.x == 0) count(0);
  for (int64_t j = lo + (int64_t)(vb.id / parts) * blockDim.x + threadIdx.x;
       j < hi; j += stride) {
    const bool live = key[j] < (uint32_t)a.n_tets;
    const bool last = live && (j + 1 == n || key[j + 1] >= (uint32_t)a.n_tets);
    if (last) count(j + 1);
    if (j == 0 && !live) count(0);
    if (!live) continue;
    move_one<T>(a.s_real, a.s_w, a.s_tet, a.s_birth, a.s_id, j, a.real, a.w, a.tet,
                a.birth, a.id, val[j]);
  }
}

// The s_* arrays copied into real, w, ... for the *n_slots slots in use.
template <typename T>
__device__ inline void copy_body(const SortArgs& a, VB vb) {
  const int64_t n = *a.n_slots;
  for (int64_t j = vb.id * (int64_t)blockDim.x + threadIdx.x; j < n;
       j += (int64_t)vb.n * blockDim.x)
    move_one<T>(a.real, a.w, a.tet, a.birth, a.id, j, a.s_real, a.s_w, a.s_tet, a.s_birth,
                a.s_id, j);
}

__device__ inline VB grid_block() { return VB{(int)blockIdx.x, (int)gridDim.x}; }

}  // namespace

template <bool FIRST>
__global__ void __launch_bounds__(kThreads) k_sort_hist(SortArgs a, int src, int shift) {
  hist_body<FIRST>(a, grid_block(), src, shift);
}
__global__ void __launch_bounds__(kScanThreads) k_sort_scan(SortArgs a) {
  scan_body(a, grid_block());
}
template <bool FIRST>
__global__ void __launch_bounds__(kThreads) k_sort_scatter(SortArgs a, int src, int shift) {
  scatter_body<FIRST>(a, grid_block(), src, shift);
}
template <typename T>
__global__ void __launch_bounds__(kMoveThreads) k_sort_gather(SortArgs a, int src) {
  gather_body<T>(a, grid_block(), src);
}
template <typename T>
__global__ void __launch_bounds__(kMoveThreads) k_particles_copy(SortArgs a) {
  copy_body<T>(a, grid_block());
}

// Batched: the arguments of instance i are A[i].
template <bool FIRST>
__global__ void __launch_bounds__(kThreads) k_sort_hist_b(const SortArgs* A, BatchMap map,
                                                          int src, int shift) {
  int i;
  const VB vb = batch_block(map, i);
  hist_body<FIRST>(batch_args(A, i), vb, src, shift);
}
__global__ void __launch_bounds__(kScanThreads) k_sort_scan_b(const SortArgs* A,
                                                              BatchMap map) {
  int i;
  const VB vb = batch_block(map, i);
  const SortArgs a = batch_args(A, i);
  if (a.ntiles > kFoldTiles) scan_body(a, vb);
}
template <bool FIRST>
__global__ void __launch_bounds__(kThreads) k_sort_scatter_b(const SortArgs* A,
                                                             BatchMap map, int src,
                                                             int shift) {
  int i;
  const VB vb = batch_block(map, i);
  scatter_body<FIRST>(batch_args(A, i), vb, src, shift);
}
template <typename T>
__global__ void __launch_bounds__(kMoveThreads) k_sort_gather_b(const SortArgs* A,
                                                                BatchMap map, int src) {
  int i;
  const VB vb = batch_block(map, i);
  const SortArgs a = batch_args(A, i);
  gather_body<T>(a, vb, src);
}
template <typename T>
__global__ void __launch_bounds__(kMoveThreads) k_sort_copy_b(const SortArgs* A,
                                                              BatchMap map) {
  int i;
  const VB vb = batch_block(map, i);
  const SortArgs a = batch_args(A, i);
  copy_body<T>(a, vb);
}

int sort_tiles(int64_t capacity) {
  return (int)((capacity + kSortTile - 1) / kSortTile);
}

namespace {

// digits of the keys 0 .. n_tets
int sort_passes(int64_t n_tets) {
  int bits = 1;
  while ((1ll << bits) <= n_tets) ++bits;
  return (bits + 7) / 8;
}

}  // namespace

hipError_t sort_particles(const SortArgs& a, int n_cu, hipStream_t s, bool copyback) {
  const int grid = n_cu * 4, passes = sort_passes(a.n_tets);
  int src = 1;  // (the first pass reads the tets and writes buffer 0)
  for (int k = 0; k < passes; ++k) {
    hipLaunchKernelGGL(k == 0 ? k_sort_hist<true> : k_sort_hist<false>, dim3(a.ntiles),
                       dim3(kThreads), 0, s, a, src, 8 * k);
    if (a.ntiles > kFoldTiles)
      hipLaunchKernelGGL(k_sort_scan, dim3(kBins), dim3(kScanThreads), 0, s, a);
    hipLaunchKernelGGL(k == 0 ? k_sort_scatter<true> : k_sort_scatter<false>,
                       dim3(a.ntiles), dim3(kThreads), 0, s, a, src, 8 * k);
    src ^= 1;
  }
  hipLaunchKernelGGL(a.real_bytes == 8 ? k_sort_gather<double> : k_sort_gather<float>,
                     dim3(grid), dim3(kMoveThreads), 0, s, a, src);
  if (copyback) return copy_particles(a, n_cu, s);
  return hipGetLastError();
}

hipError_t copy_particles(const SortArgs& a, int n_cu, hipStream_t s) {
  hipLaunchKernelGGL(a.real_bytes == 8 ? k_particles_copy<double> : k_particles_copy<float>,
                     dim3(n_cu * 4), dim3(kMoveThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t sort_particles_b(const SortArgs* A, const std::vector<const SortArgs*>& host,
                            const std::vector<char>& due, int n_cu, hipStream_t s) {
  // the workgroups of each kind of launch, instance after instance
  BatchMap tiles{}, bins{}, moves{};
  int j = 0, passes = 0, real_bytes = 8;
  bool scan = false;
  for (size_t i = 0; i < host.size(); ++i) {
    if (!due[i]) continue;
    const SortArgs& a = *host[i];
    tiles.inst[j] = bins.inst[j] = moves.inst[j] = (int32_t)i;
    tiles.off[j + 1] = tiles.off[j] + a.ntiles;
    bins.off[j + 1] = bins.off[j] + kBins;
    // one slot per thread, in whole rounds of the XCDs
    moves.off[j + 1] = moves.off[j] + std::min(std::max(n_cu * 4 / 8 * 8, 8),
                                               a.ntiles * (kSortTile / kMoveThreads));
    // (an instance whose keys have fewer digits than another's is sorted by
    // zeros in the passes beyond its own: its order stays)
    passes = std::max(passes, sort_passes(a.n_tets));
    scan = scan || a.ntiles > kFoldTiles;
    real_bytes = a.real_bytes;  // (one precision per batch)
    ++j;
  }
  if (j == 0) return hipSuccess;
  tiles.n_seg = bins.n_seg = moves.n_seg = j;
  int src = 1;
  for (int k = 0; k < passes; ++k) {
    hipLaunchKernelGGL(k == 0 ? k_sort_hist_b<true> : k_sort_hist_b<false>,
                       dim3(tiles.off[j]), dim3(kThreads), 0, s, A, tiles, src, 8 * k);
    if (scan)
      hipLaunchKernelGGL(k_sort_scan_b, dim3(bins.off[j]), dim3(kScanThreads), 0, s, A, bins);
    hipLaunchKernelGGL(k == 0 ? k_sort_scatter_b<true> : k_sort_scatter_b<false>,
                       dim3(tiles.off[j]), dim3(kThreads), 0, s, A, tiles, src, 8 * k);
    src ^= 1;
  }
  const bool f64 = real_bytes == 8;
  hipLaunchKernelGGL(f64 ? k_sort_gather_b<double> : k_sort_gather_b<float>,
                     dim3(moves.off[j]), dim3(kMoveThreads), 0, s, A, moves, src);
  hipLaunchKernelGGL(f64 ? k_sort_copy_b<double> : k_sort_copy_b<float>,
                     dim3(moves.off[j]), dim3(kMoveThreads), 0, s, A, moves);
  return hipGetLastError();
}

size_t sort_scratch_bytes(int64_t capacity, int real_bytes) {
  const int64_t ntiles = sort_tiles(capacity);
  return (size_t)capacity * (16 + 6 * (size_t)real_bytes + 8 + 4 + 4 + 8) +
         (size_t)kBins * ntiles * 4 + kBins * 4 + 8192;
}

}  // namespace fp
