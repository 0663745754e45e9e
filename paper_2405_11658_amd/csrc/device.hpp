// Device-side building blocks shared by the HIP kernels of the library:
// wave64 primitives, wave-aggregated atomics, an open-addressing
// community -> weight table (LDS or global memory), and the move score.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <limits.h>

namespace lk {

constexpr int kWave = 64;
constexpr int kNoComm = INT_MAX;  // "no candidate" in argmax reductions
constexpr int kEmpty = -1;        // empty table slot

__device__ __forceinline__ int lane() { return (int)__lane_id(); }

// Eq. 2 scaled by 2m^2 (so Delta-Q = g / (M2^2 / 2)):
//   g = M2*(K_{i->c} - K_{i->d}) - K_i*(K_i + Sigma_c - Sigma_d),
// Sigma_d including K_i.  Exact parenthesisation, no contraction, so the
// value is bit-identical to any other IEEE evaluation of the same expression.
__device__ __forceinline__ double move_score(double M2, double a, double b, double Ki, double Sc,
                                             double Sd) {
#pragma clang fp contract(off)
  double t1 = M2 * (a - b);
  double t2 = Ki * ((Ki + Sc) - Sd);
  return t1 - t2;
}

// Total order used by every argmax: larger gain first, then smaller id.
__device__ __forceinline__ bool better(double g1, int c1, double g2, int c2) {
  return g1 > g2 || (g1 == g2 && c1 < c2);
}

template <int W>
__device__ __forceinline__ void group_argmax(double &g, int &c) {
#pragma unroll
  for (int off = W / 2; off > 0; off >>= 1) {
    double og = __shfl_xor(g, off, W);
    int oc = __shfl_xor(c, off, W);
    if (better(og, oc, g, c)) { g = og; c = oc; }
  }
}

template <int W>
__device__ __forceinline__ double group_sum(double v) {
#pragma unroll
  for (int off = W / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, W);
  return v;
}

template <int W>
__device__ __forceinline__ long long group_sum_ll(long long v) {
#pragma unroll
  for (int off = W / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, W);
  return v;
}

// Reductions over the whole wavefront without LDS permutes (each of those is
// a round trip of ~100 cycles through the LDS pipe, three per step of a
// (gain, id) argmax): four steps inside the rows of 16 lanes with DPP moves,
// then the four rows' results through scalar registers.  Called by all 64
// lanes; every lane gets the result.
template <int CTRL>
__device__ __forceinline__ int dpp_move(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = dpp_move<CTRL>((int)b), hi = dpp_move<CTRL>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;           // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;  // within 8 and 16 lanes
__device__ __forceinline__ int lane_value(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
__device__ __forceinline__ double lane_value(double x, int l) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ int64_t lane_value64(int64_t x, int l) {
  const int lo = __builtin_amdgcn_readlane((int)x, l), hi = __builtin_amdgcn_readlane((int)(x >> 32), l);
  return ((int64_t)hi << 32) | (unsigned int)lo;
}
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_move<kDppXor1>(v);
  v += dpp_move<kDppXor2>(v);
  v += dpp_move<kDppHalfMirror>(v);
  v += dpp_move<kDppMirror>(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}
// x of the lane ^ J, the lane before (0 in lane 0) and the lane after (0 in
// lane 63), without the LDS pipe.
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
  if constexpr (J == 1) {
    return (uint32_t)dpp_move<kDppXor1>((int)x);
  } else if constexpr (J == 2) {
    return (uint32_t)dpp_move<kDppXor2>((int)x);
  } else if constexpr (J == 4) {
    return (uint32_t)dpp_move<0x1B>(dpp_move<kDppHalfMirror>((int)x));  // (l ^ 7) ^ 3
  } else if constexpr (J == 8) {
    return (uint32_t)dpp_move<0x128>((int)x);  // row_ror:8
  } else if constexpr (J == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return (lane() & 16) ? r[0] : r[1];
  } else {
    static_assert(J == 32, "a power of two below the wavefront");
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return (lane() & 32) ? r[0] : r[1];
  }
}
template <int J>
__device__ __forceinline__ float lane_xor(float x) {
  return __uint_as_float(lane_xor<J>(__float_as_uint(x)));
}
constexpr int kDppWaveShr1 = 0x138, kDppWaveShl1 = 0x130;
template <class T>
__device__ __forceinline__ T lane_before(T x) {
  return (T)dpp_move<kDppWaveShr1>((int)x);
}
__device__ __forceinline__ double lane_before(double x) { return dpp_move<kDppWaveShr1>(x); }
template <class T>
__device__ __forceinline__ T lane_after(T x) {
  return (T)dpp_move<kDppWaveShl1>((int)x);
}
constexpr int kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118;
// Inclusive prefix sum over the lanes; *tot the wavefront's.
__device__ __forceinline__ int wave_scan(int x, int *tot) {
  x += dpp_move<kDppRowShr1>(x);
  x += dpp_move<kDppRowShr2>(x);
  x += dpp_move<kDppRowShr4>(x);
  x += dpp_move<kDppRowShr8>(x);
  const int a = lane_value(x, 15), b = a + lane_value(x, 31), c = b + lane_value(x, 47);
  *tot = c + lane_value(x, 63);
  const int r = lane() >> 4;
  return x + (r == 0 ? 0 : r == 1 ? a : r == 2 ? b : c);
}
template <int CTRL>
__device__ __forceinline__ int64_t dpp_move(int64_t x) {
  const int lo = dpp_move<CTRL>((int)x), hi = dpp_move<CTRL>((int)(x >> 32));
  return ((int64_t)hi << 32) | (unsigned int)lo;
}
__device__ __forceinline__ int64_t wave_scan(int64_t x, int64_t *tot) {
  x += dpp_move<kDppRowShr1>(x);
  x += dpp_move<kDppRowShr2>(x);
  x += dpp_move<kDppRowShr4>(x);
  x += dpp_move<kDppRowShr8>(x);
  const int64_t a = lane_value64(x, 15), b = a + lane_value64(x, 31), c = b + lane_value64(x, 47);
  *tot = c + lane_value64(x, 63);
  const int r = lane() >> 4;
  return x + (r == 0 ? 0 : r == 1 ? a : r == 2 ? b : c);
}
template <int CTRL>
__device__ __forceinline__ void dpp_seg_add(double &x, int &f) {
  const double y = dpp_move<CTRL>(x);
  const int yf = dpp_move<CTRL>(f);
  if (!f) x += y;
  f |= yf;
}
// Segmented inclusive sum over the lanes (f: the lane starts a segment); on
// return f says whether any lane up to this one does.
__device__ __forceinline__ void wave_seg_scan(double &x, int &f) {
  dpp_seg_add<kDppRowShr1>(x, f);
  dpp_seg_add<kDppRowShr2>(x, f);
  dpp_seg_add<kDppRowShr4>(x, f);
  dpp_seg_add<kDppRowShr8>(x, f);
  const unsigned long long fl = __ballot(f);
  // sums open at the ends of the rows before
  const double a = lane_value(x, 15);
  const double b = (fl >> 31) & 1ull ? lane_value(x, 31) : a + lane_value(x, 31);
  const double c = (fl >> 47) & 1ull ? lane_value(x, 47) : b + lane_value(x, 47);
  const int r = lane() >> 4;
  if (!f) x += r == 0 ? 0.0 : r == 1 ? a : r == 2 ? b : c;
  f = (fl & (~0ull >> (63 - lane()))) != 0;
}
template <int CTRL>
__device__ __forceinline__ void dpp_argmax(double &g, int &c) {
  const double og = dpp_move<CTRL>(g);
  const int oc = dpp_move<CTRL>(c);
  if (better(og, oc, g, c)) { g = og; c = oc; }
}
__device__ __forceinline__ void wave_argmax(double &g, int &c) {
  dpp_argmax<kDppXor1>(g, c);
  dpp_argmax<kDppXor2>(g, c);
  dpp_argmax<kDppHalfMirror>(g, c);
  dpp_argmax<kDppMirror>(g, c);
  const double g0 = g;
  const int c0 = c;
#pragma unroll
  for (int r = 0; r < kWave; r += 16) {
    const double og = lane_value(g0, r);
    const int oc = lane_value(c0, r);
    if (r == 0 || better(og, oc, g, c)) { g = og; c = oc; }
  }
}

// 32-bit integer finaliser "lowbias32" (xorshift-multiply; constants from
// C. Wellons' published hash-prospector search).
__device__ __forceinline__ uint32_t mix32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}
__device__ __forceinline__ uint32_t mix64(uint64_t x) {
  return mix32((uint32_t)x ^ mix32((uint32_t)(x >> 32)));
}

// Argmax over a team of TEAM threads (TEAM a multiple of the wavefront or
// smaller); the result is valid in the team's first thread.  With TEAM >
// kWave every thread of the workgroup must call it.
template <int TEAM, int BLOCK>
__device__ __forceinline__ void team_argmax(double &g, int &c, double *rg, int *rc) {
  group_argmax<kWave>(g, c);
  if (TEAM > kWave) {
    const int w = threadIdx.x / kWave;
    if (lane() == 0) { rg[w] = g; rc[w] = c; }
    __syncthreads();
    if ((threadIdx.x % TEAM) == 0) {
      for (int k = 1; k < TEAM / kWave; ++k)
        if (better(rg[w + k], rc[w + k], g, c)) { g = rg[w + k]; c = rc[w + k]; }
    }
    __syncthreads();
  }
}

// Open addressing with linear probing.  keys[] holds kEmpty for free slots,
// vals[] starts at 0.  Capacity (mask+1) must exceed the number of distinct
// keys inserted; the probe loop is bounded by the capacity in any case.
__device__ __forceinline__ void table_add(int *keys, double *vals, uint32_t mask, int key,
                                          double w) {
  uint32_t h = mix32((uint32_t)key) & mask;
  for (uint32_t probe = 0; probe <= mask; ++probe) {
    int k = __atomic_load_n(&keys[h], __ATOMIC_RELAXED);
    if (k == key) { atomicAdd(&vals[h], w); return; }
    if (k == kEmpty) {
      int old = atomicCAS(&keys[h], kEmpty, key);
      if (old == kEmpty || old == key) { atomicAdd(&vals[h], w); return; }
    }
    h = (h + 1) & mask;
  }
}

// Workgroup-level merge of (key, value) additions before they reach global
// memory: the block inserts into an LDS table (capacity above the number of
// distinct keys it inserts) and then issues one atomic per distinct key, so a
// key shared by many items (a giant community) costs one global atomic per
// workgroup instead of one per item.  Called by the whole block.
template <int SLOTS>
__device__ __forceinline__ void block_merge_clear(int *tk, double *tv) {
  for (int s = threadIdx.x; s < SLOTS; s += blockDim.x) { tk[s] = kEmpty; tv[s] = 0.0; }
  __syncthreads();
}
template <int SLOTS>
__device__ __forceinline__ void block_merge_flush(int *tk, double *tv, double *out) {
  __syncthreads();
  for (int s = threadIdx.x; s < SLOTS; s += blockDim.x) {
    if (tk[s] != kEmpty) {
      unsafeAtomicAdd(&out[tk[s]], tv[s]);
      tk[s] = kEmpty;
      tv[s] = 0.0;
    }
  }
  __syncthreads();
}

__device__ __forceinline__ double table_get(const int *keys, const double *vals, uint32_t mask,
                                            int key) {
  uint32_t h = mix32((uint32_t)key) & mask;
  for (uint32_t probe = 0; probe <= mask; ++probe) {
    int k = keys[h];
    if (k == key) return vals[h];
    if (k == kEmpty) return 0.0;
    h = (h + 1) & mask;
  }
  return 0.0;
}

// Wave-aggregated counter increment: lanes with equal keys share one atomic.
// Returns, for each active lane, old counter value + rank among equal keys.
// Must be called by the whole wave (inactive lanes pass active = false).
__device__ __forceinline__ int wave_peel_inc(int *ctr, int key, bool active) {
  unsigned long long pending = __ballot(active);
  int result = 0;
  const int ln = lane();
  while (pending) {
    int leader = __ffsll((unsigned long long)pending) - 1;
    int k = __shfl(key, leader);
    unsigned long long grp = __ballot(active && key == k) & pending;
    int base = 0;
    if (ln == leader) base = atomicAdd(&ctr[k], (int)__popcll(grp));
    base = __shfl(base, leader);
    if ((grp >> ln) & 1ull) result = base + (int)__popcll(grp & ((1ull << ln) - 1ull));
    pending &= ~grp;
  }
  return result;
}

// Wave-aggregated append to one of `nb` lists: lanes with equal bucket share
// one atomic on counts[bucket].  Returns the slot index inside the bucket.
__device__ __forceinline__ int wave_append(int *counts, int bucket, bool active) {
  return wave_peel_inc(counts, bucket, active);
}

// Wave-aggregated FP64 scatter-add arr[key] += v.  The most frequent keys of
// the wave are combined first (up to 4 rounds), the rest use direct atomics.
__device__ __forceinline__ void wave_peel_add_f64(double *arr, int key, double v, bool active) {
  unsigned long long pending = __ballot(active);
  const int ln = lane();
  for (int round = 0; round < 4 && pending; ++round) {
    int leader = __ffsll((unsigned long long)pending) - 1;
    int k = __shfl(key, leader);
    bool mine = ((pending >> ln) & 1ull) && key == k;
    unsigned long long grp = __ballot(mine);
    double s = group_sum<kWave>(mine ? v : 0.0);
    if (ln == leader) atomicAdd(&arr[k], s);
    pending &= ~grp;
  }
  if ((pending >> ln) & 1ull) atomicAdd(&arr[key], v);
}

// Block-wide sum (blockDim.x <= 1024, multiple of 64); result valid in all threads.
__device__ __forceinline__ double block_sum(double v, double *scratch /* >= 16 */) {
  v = group_sum<kWave>(v);
  const int w = threadIdx.x / kWave;
  const int nw = blockDim.x / kWave;
  __syncthreads();
  if (lane() == 0) scratch[w] = v;
  __syncthreads();
  double t = 0.0;
  for (int k = 0; k < nw; ++k) t += scratch[k];
  __syncthreads();
  return t;
}

__device__ __forceinline__ long long block_sum_ll(long long v, long long *scratch /* >= 16 */) {
  v = group_sum_ll<kWave>(v);
  const int w = threadIdx.x / kWave;
  const int nw = blockDim.x / kWave;
  __syncthreads();
  if (lane() == 0) scratch[w] = v;
  __syncthreads();
  long long t = 0;
  for (int k = 0; k < nw; ++k) t += scratch[k];
  __syncthreads();
  return t;
}

__device__ __forceinline__ int64_t lower_bound_i32(const int32_t *a, int64_t lo, int64_t hi, int32_t x) {
  while (lo < hi) {
    int64_t mid = lo + ((hi - lo) >> 1);
    if (a[mid] < x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Exclusive max-scan across the block (blockDim.x multiple of 64, <= 1024).
__device__ __forceinline__ int block_excl_max_scan(int v, int *sh /* >= 16 ints */) {
  int x = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    int y = __shfl_up(x, off);
    if (lane() >= off) x = max(x, y);
  }
  const int w = threadIdx.x / kWave;
  __syncthreads();
  if (lane() == kWave - 1) sh[w] = x;
  __syncthreads();
  int pre = -1;
  for (int k = 0; k < w; ++k) pre = max(pre, sh[k]);
  int incl = max(x, pre);
  int ex = __shfl_up(incl, 1);
  if (lane() == 0) ex = pre;
  __syncthreads();
  return ex;
}

// Row mapping for a chunk of CSR positions [q0, q0 + len), len <= CH:
// rowof[t] receives the row owning position q0 + t.  lo is the row owning q0
// and hi an upper bound on the row owning q0 + len - 1 (both precomputed by
// chunk_start_rows).  Empty rows are handled.  Called by the whole block.
template <int CH>
__device__ __forceinline__ void chunk_rows(const int64_t *off, int64_t q0, int len, int lo, int hi,
                                           int *rowof, int *sh) {
  for (int t = threadIdx.x; t < CH; t += blockDim.x) rowof[t] = -1;
  __syncthreads();
  // the start of every non-empty row (an empty row starts where the next
  // non-empty one does, and that one owns the slot): one plain store per
  // slot, no atomics
  for (int r = lo + (int)threadIdx.x; r <= hi; r += blockDim.x) {
    int64_t s = off[r] - q0;
    if (s < 0) s = 0;
    if (s < len && (r == hi || off[r + 1] > off[r])) rowof[s] = r;
  }
  __syncthreads();
  const int per = CH / (int)blockDim.x;
  const int t0 = threadIdx.x * per;
  int m = -1;
  for (int t = t0; t < t0 + per; ++t) m = max(m, rowof[t]);
  int acc = block_excl_max_scan(m, sh);
  for (int t = t0; t < t0 + per; ++t) {
    acc = max(acc, rowof[t]);
    rowof[t] = acc;
  }
  __syncthreads();
}

}  // namespace lk
