// A workgroup's neighbour-community table in LDS, for one vertex whose edges
// are all in the workgroup's registers (PER per thread).
#pragma once
#include "device.hpp"
#include "kernels.hpp"

namespace lk {

template <int T, int PER, int SLOTS>
struct BlockTable {
  static_assert(T * PER < SLOTS, "more slots than distinct communities");
  int keys[SLOTS];
  double vals[SLOTS];
  double rd[T / kWave], rs[T / kWave];
  int rc[T / kWave];
};

// Sum over the workgroup, in every thread.
template <int T>
__device__ __forceinline__ double block_total(double v, double *r) {
  v = wave_sum(v);
  if (lane() == 0) r[threadIdx.x / kWave] = v;
  __syncthreads();
  v = r[0];
#pragma unroll
  for (int k = 1; k < T / kWave; ++k) v += r[k];
  return v;
}

// Adds w to key's slot; the slot when this call took it, else -1.
__device__ __forceinline__ int block_slot(int *keys, double *vals, uint32_t mask, int key, double w) {
  uint32_t h = mix32((uint32_t)key) & mask;
  for (uint32_t probe = 0; probe <= mask; ++probe) {
    const int old = atomicCAS(&keys[h], kEmpty, key);
    if (old == kEmpty || old == key) {
      atomicAdd(&vals[h], w);
      return old == kEmpty ? (int)h : -1;
    }
    h = (h + 1) & mask;
  }
  return -1;
}

// Best positive-gain community over a vertex's edges (community c, kEmpty for
// edges that do not count, and weight x; deg edges in all), own community d:
// its weight, usually most of the edges, is summed in registers, the others in
// the table, and each slot is scored by the thread that took it.  In every
// thread: the gain bg and the community bc (kNoComm when no gain is positive).
template <int T, int PER, int SLOTS>
__device__ __forceinline__ void block_best(BlockTable<T, PER, SLOTS> &l, int deg, int (&c)[PER],
                                           const float (&x)[PER], int d, double M2, double Ki, double Sd,
                                           const double *Sig, double &bg, int &bc) {
  uint32_t cap = 64;
  while (cap < 2u * (uint32_t)deg && cap < (uint32_t)SLOTS) cap <<= 1;
  for (uint32_t s = threadIdx.x; s < cap; s += T) { l.keys[s] = kEmpty; l.vals[s] = 0.0; }
  double b = 0.0;
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (c[u] == d) {
      b += (double)x[u];
      c[u] = kEmpty;
    }
  b = block_total<T>(b, l.rs);  // its barrier also ends the clearing
  int own[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) own[u] = c[u] != kEmpty ? block_slot(l.keys, l.vals, cap - 1, c[u], (double)x[u]) : -1;
  double S[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) S[u] = own[u] >= 0 ? Sig[c[u]] : 0.0;
  __syncthreads();
  bg = 0.0;
  bc = kNoComm;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (own[u] < 0) continue;
    const double g = move_score(M2, l.vals[own[u]], b, Ki, S[u], Sd);
    if (g > 0.0 && better(g, c[u], bg, bc)) { bg = g; bc = c[u]; }
  }
  wave_argmax(bg, bc);
  const int wv = threadIdx.x / kWave;
  if (lane() == 0) { l.rd[wv] = bg; l.rc[wv] = bc; }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < T / kWave; ++k)
    if (k == 0 || better(l.rd[k], l.rc[k], bg, bc)) { bg = l.rd[k]; bc = l.rc[k]; }
}

// The chunked hubs' scoring: every segment's workgroup leaves its best (gain,
// community; thread 0's values) and the last of the hub's learns that it is
// (in every thread), so that it can reduce them.  The counter is back at 0 after that.
__device__ __forceinline__ bool hub_last_segment(const HubPlan &p, int h, int64_t q, double bg, int bc) {
  __shared__ int last;
  if (threadIdx.x == 0) {
    __hip_atomic_store(&p.pg[q], bg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p.pc[q], bc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int n = (int)(p.hsg[h + 1] - p.hsg[h]);
    // the stores above have reached memory before the count (a wait; a release
    // at device scope would write the L2 back, for every workgroup)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    const int done = __hip_atomic_fetch_add(&p.done[h], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = done == n - 1;
    if (last) p.done[h] = 0;
  }
  __syncthreads();
  return last != 0;
}
// Best of the hub's segments, in thread 0; the hub's sums are ready for the
// next iteration.
__device__ __forceinline__ void hub_reduce_segments(const HubPlan &p, int h, double &bg, int &bc) {
  if (threadIdx.x >= kWave) return;
  bg = 0.0;
  bc = kNoComm;
  for (int64_t q = p.hsg[h] + lane(); q < p.hsg[h + 1]; q += kWave) {
    const double g = __hip_atomic_load(&p.pg[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int c = __hip_atomic_load(&p.pc[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (better(g, c, bg, bc)) { bg = g; bc = c; }
  }
  wave_argmax(bg, bc);
  if (lane() == 0) {
    p.own[h] = 0.0;
    p.flag[h] = 0;
  }
}

}  // namespace lk
