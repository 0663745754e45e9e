// Local-moving phase (Alg. "leidenMove" with "scanCommunities", self=false),
// executed on the GPU as sweeps over S vertex slices (hash of the id); the
// slices of an iteration run in order, each synchronously:
//   frontier  - unprocessed in-range vertices of the slice are marked
//               processed (vertex pruning) and bucketed by degree;
//   propose   - each frontier vertex builds its neighbour-community weight
//               table and picks the community of best Eq. 2 gain (strictly
//               positive, ties to the smaller id);
//   apply     - a proposal d -> c is dropped when a neighbour of the same
//               slice proposes the exact reverse move c -> d with priority
//               (larger gain, then smaller id); accepted moves update C,
//               Sigma (atomics), flag
//               source and target communities as changed (dynamic runs) and
//               mark the mover's neighbours unprocessed; dropped proposers stay
//               unprocessed.
// Degree buckets pick the table: registers of a 4/8/32-lane group (all-pairs
// combine), an LDS table per wavefront or workgroup, or a global-memory table
// per workgroup for hubs.
#include "block_table.hpp"
#include "device.hpp"
#include "kernels.hpp"

namespace lk {

__device__ __forceinline__ int bucket_of_d(int64_t deg, int64_t hubdeg) {
  return deg > hubdeg ? 5 : deg <= 4 ? 0 : deg <= 8 ? 1 : deg <= 32 ? 2 : deg <= 256 ? 3 : 4;
}

// Keyed appends are aggregated per workgroup: a tile of kTile vertices is
// counted into LDS counters, one global atomic per non-empty key reserves
// the workgroup's range, and a second pass places the items.
constexpr int kTile = 4096;
constexpr int kMaxKeys = 2048;  // >= 256 slices * (kNB + 1)

__global__ __launch_bounds__(256) void k_slice_hist(const int64_t *off, int64_t n, int S, int64_t hubdeg,
                                                    int32_t *counts, int32_t *slice_cnt) {
  __shared__ int cnt[kMaxKeys];
  const int K = S * kNB + S;  // bucket keys, then slice keys
  for (int k = threadIdx.x; k < K; k += blockDim.x) cnt[k] = 0;
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t deg = off[i + 1] - off[i];
    const int sl = slice_of(i, S);
    atomicAdd(&cnt[S * kNB + sl], 1);
    if (deg > 0) atomicAdd(&cnt[sl * kNB + bucket_of_d(deg, hubdeg)], 1);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < K; k += blockDim.x) {
    const int c = cnt[k];
    if (c) atomicAdd(k < S * kNB ? &counts[k] : &slice_cnt[k - S * kNB], c);
  }
}
void slice_hist(const int64_t *off, int64_t n, int S, int64_t hubdeg, int32_t *counts, int32_t *slice_cnt,
                hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_slice_hist, flat_grid(n, 256, 1024), 256, 0, s, off, n, S, hubdeg, counts, slice_cnt);
}

__global__ __launch_bounds__(256) void k_slice_scatter(int64_t n, int S, const int32_t *slice_off,
                                                       int32_t *slice_fill, int32_t *vbyslice) {
  __shared__ int cnt[kMaxKeys];
  __shared__ int base[kMaxKeys];
  for (int64_t t0 = (int64_t)blockIdx.x * kTile; t0 < n; t0 += (int64_t)gridDim.x * kTile) {
    const int64_t t1 = min(t0 + (int64_t)kTile, n);
    for (int k = threadIdx.x; k < S; k += blockDim.x) cnt[k] = 0;
    __syncthreads();
    for (int64_t i = t0 + threadIdx.x; i < t1; i += blockDim.x) atomicAdd(&cnt[slice_of(i, S)], 1);
    __syncthreads();
    for (int k = threadIdx.x; k < S; k += blockDim.x) {
      const int c = cnt[k];
      base[k] = c ? atomicAdd(&slice_fill[k], c) : 0;
      cnt[k] = 0;
    }
    __syncthreads();
    for (int64_t i = t0 + threadIdx.x; i < t1; i += blockDim.x) {
      const int sl = slice_of(i, S);
      vbyslice[slice_off[sl] + base[sl] + atomicAdd(&cnt[sl], 1)] = (int32_t)i;
    }
    __syncthreads();
  }
}
void slice_scatter(int64_t n, int S, const int32_t *slice_off, int32_t *slice_fill, int32_t *vbyslice,
                   hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_slice_scatter, flat_grid(ceil_div(n, kTile), 1, 2048), 256, 0, s, n, S,
                                slice_off, slice_fill, vbyslice);
}

// Frontier of slice s: its unprocessed vertices become processed; in-range
// ones with edges are bucketed by degree.  Proposals of the slice are reset.
// A thread's vertices of a tile stay in its registers between the count and
// the placing.  The slices of small graphs are a tile or two, and a launch in
// the chain of slices lasts as long as its longest workgroup (4096 vertices,
// each read twice: 19 us, 1024: 6.5).
constexpr int kFrontPer = 4;
constexpr int kFrontTile = 256 * kFrontPer;
__global__ __launch_bounds__(256) void k_frontier(MoveArgs a) {
  __shared__ int cnt[kNB];
  __shared__ int base[kNB];
  int32_t *counts = a.counts + a.s * kNB;
  const int32_t *region = a.region + a.s * kNB;
  for (int64_t t0 = a.vbeg + (int64_t)blockIdx.x * kFrontTile; t0 < a.vend; t0 += (int64_t)gridDim.x * kFrontTile) {
    if (threadIdx.x < kNB) cnt[threadIdx.x] = 0;
    int i[kFrontPer], key[kFrontPer], at[kFrontPer];
    uint8_t u[kFrontPer], r[kFrontPer];
    int64_t deg[kFrontPer];
#pragma unroll
    for (int k = 0; k < kFrontPer; ++k) {
      const int64_t t = t0 + threadIdx.x + k * 256;
      i[k] = t < a.vend ? a.vbyslice[t] : -1;
    }
#pragma unroll
    for (int k = 0; k < kFrontPer; ++k) {
      u[k] = i[k] >= 0 ? a.U[i[k]] : 0;
      r[k] = i[k] >= 0 ? a.rng[i[k]] : 0;
      deg[k] = i[k] >= 0 ? a.off[i[k] + 1] - a.off[i[k]] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kFrontPer; ++k) {
      key[k] = u[k] && r[k] && deg[k] > 0 ? bucket_of_d(deg[k], a.hubdeg) : -1;
      at[k] = key[k] >= 0 ? atomicAdd(&cnt[key[k]], 1) : 0;
    }
    __syncthreads();
    if (threadIdx.x < kNB) {
      const int c = cnt[threadIdx.x];
      base[threadIdx.x] = c ? atomicAdd(&counts[threadIdx.x], c) : 0;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kFrontPer; ++k) {
      if (i[k] < 0) continue;
      a.prop[i[k]] = -1;
      a.U[i[k]] = 0;
      if (a.act && deg[k] > a.hubdeg) a.act[i[k]] = key[k] >= 0;
      if (key[k] >= 0) a.lists[region[key[k]] + base[key[k]] + at[k]] = i[k];
    }
    __syncthreads();
  }
}

// ---- propose: small-degree groups (deg <= G), all-pairs combine in registers
// (by workgroups blk of nblk, as in the other buckets)
template <int G>
__device__ __forceinline__ void propose_small(const MoveArgs &a, int b, int blk, int nblk) {
  const int count = a.counts[a.s * kNB + b];
  const int32_t *list = a.lists + a.region[a.s * kNB + b];
  const int gl = threadIdx.x & (G - 1);
  // the loop runs in step for the whole wavefront (collectives stay uniform)
  const int64_t wave = ((int64_t)blk * 256 + threadIdx.x) / kWave;
  const int64_t nwave = (int64_t)nblk * 256 / kWave;
  const int gin = lane() / G;
  for (int64_t v0 = wave * (kWave / G); v0 < count; v0 += nwave * (kWave / G)) {
    const int64_t v = v0 + gin;
    const bool valid = v < count;
    const int i = valid ? list[v] : 0;
    int deg = 0, d = 0;
    int64_t e0 = 0;
    if (valid) {
      e0 = a.off[i];
      deg = (int)(a.off[i + 1] - e0);
      d = a.C[i];
    }
    int key = -1;
    float wt = 0.0f;
    if (gl < deg) {
      const int j = a.idx[e0 + gl];
      if (j != i) { key = a.C[j]; wt = a.w[e0 + gl]; }
    }
    double sum = 0.0;
    bool first = true;
#pragma unroll
    for (int s = 0; s < G; ++s) {
      const int ks = __shfl(key, s, G);
      const float ws = __shfl(wt, s, G);
      if (ks == key) {
        sum += (double)ws;
        if (s < gl) first = false;
      }
    }
    const double bown = group_sum<G>((key == d && first) ? sum : 0.0);
    double g = 0.0;
    int c = kNoComm;
    if (key >= 0 && key != d && first) {
      const double x = move_score(a.M2, sum, bown, a.K[i], a.Sig[key], a.Sig[d]);
      if (x > 0.0) { g = x; c = key; }
    }
    group_argmax<G>(g, c);
    if (valid && gl == 0) {
      a.from[i] = d;
      a.prop[i] = (c == kNoComm) ? -1 : c;
      a.gp[i] = g;
    }
  }
}


__device__ __forceinline__ uint32_t pow2_at_least(uint64_t x) {
  uint32_t c = 2;
  while (c < x) c <<= 1;
  return c;
}

// ---- propose: a team (wavefront or workgroup) per vertex, hash table of T
// slots per team in LDS.
template <int TEAM, int T, int BLOCK>
struct TeamLds {
  static constexpr int NT = BLOCK / TEAM;
  double svals[NT * T];
  double sb[NT];
  double rg[BLOCK / kWave];
  int skeys[NT * T];
  int rc[BLOCK / kWave];
};
template <int TEAM, int T, int BLOCK>
__device__ __forceinline__ void propose_team(const MoveArgs &a, int b, int blk, int nblk,
                                             TeamLds<TEAM, T, BLOCK> &l) {
  constexpr int NT = BLOCK / TEAM;
  const int team = threadIdx.x / TEAM;
  const int t = threadIdx.x % TEAM;
  const int count = a.counts[a.s * kNB + b];
  const int32_t *list = a.lists + a.region[a.s * kNB + b];
  for (int64_t base = (int64_t)blk * NT; base < count; base += (int64_t)nblk * NT) {
    const int64_t v = base + team;
    const bool valid = v < count;
    const int i = valid ? list[v] : 0;
    int64_t e0 = 0, e1 = 0;
    int d = 0;
    if (valid) { e0 = a.off[i]; e1 = a.off[i + 1]; d = a.C[i]; }
    int *keys = l.skeys + team * T;
    double *vals = l.svals + team * T;
    const uint32_t mask = T - 1;
    for (uint32_t s = t; s <= mask; s += TEAM) { keys[s] = kEmpty; vals[s] = 0.0; }
    if (t == 0) l.sb[team] = 0.0;
    __syncthreads();
    if (valid) {
      for (int64_t e = e0 + t; e < e1; e += TEAM) {
        const int j = a.idx[e];
        if (j != i) table_add(keys, vals, mask, a.C[j], (double)a.w[e]);
      }
    }
    __syncthreads();
    if (valid)
      for (uint32_t s = t; s <= mask; s += TEAM)
        if (keys[s] == d) l.sb[team] = vals[s];
    __syncthreads();
    double bg = 0.0;
    int bc = kNoComm;
    if (valid) {
      const double bown = l.sb[team];
      const double Ki = a.K[i];
      const double Sd = a.Sig[d];
      for (uint32_t s = t; s <= mask; s += TEAM) {
        const int c = keys[s];
        if (c == kEmpty || c == d) continue;
        const double x = move_score(a.M2, vals[s], bown, Ki, a.Sig[c], Sd);
        if (x > 0.0 && better(x, c, bg, bc)) { bg = x; bc = c; }
      }
    }
    team_argmax<TEAM, BLOCK>(bg, bc, l.rg, l.rc);
    if (valid && t == 0) {
      a.from[i] = d;
      a.prop[i] = (bc == kNoComm) ? -1 : bc;
      a.gp[i] = bg;
    }
    __syncthreads();
  }
}

template <int TEAM, int T, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_propose_team(MoveArgs a, int b) {
  __shared__ TeamLds<TEAM, T, BLOCK> l;
  propose_team<TEAM, T, BLOCK>(a, b, blockIdx.x, gridDim.x, l);
}
template <int G>
__global__ __launch_bounds__(256) void k_propose_small(MoveArgs a, int b) {
  propose_small<G>(a, b, blockIdx.x, gridDim.x);
}
// All buckets but the hubs in one launch.  Its workgroups all have the largest
// table's LDS, three to a compute unit: for the slices whose workgroups all
// run at once that way, a slice being a chain of launches of which each lasts
// as long as its slowest workgroup (R-MAT scale 17, 1/32 of 100k vertices: five
// launches 35 us, this one 12).
__global__ __launch_bounds__(256) void k_propose_slice(MoveArgs a, BucketSpan sp) {
  __shared__ union {
    TeamLds<64, 512, 256> wave;
    TeamLds<256, 4096, 256> block;
  } l;
  int b = 0;
  while ((int)blockIdx.x >= sp.first[b + 1]) ++b;
  const int blk = blockIdx.x - sp.first[b], nblk = sp.first[b + 1] - sp.first[b];
  switch (b) {
    case 0: propose_small<4>(a, b, blk, nblk); break;
    case 1: propose_small<8>(a, b, blk, nblk); break;
    case 2: propose_small<32>(a, b, blk, nblk); break;
    case 3: propose_team<64, 512, 256>(a, b, blk, nblk, l.wave); break;
    default: propose_team<256, 4096, 256>(a, b, blk, nblk, l.block); break;
  }
}

// ---- propose: hubs, several workgroups per vertex --------------------------
struct HubGatherLds {
  int keys[2 * kHubEC];
  double vals[2 * kHubEC];
  int used[kHubEC];  // slots taken (at most one per edge)
  int nused;
};
// gather: a workgroup merges one edge chunk of a frontier hub in an LDS
// table, then adds its distinct communities into the hub's global table (the
// hub's own community into `own`).
__device__ __forceinline__ void hub_gather_chunk(const MoveArgs &a, int64_t q, HubGatherLds &l) {
  constexpr int T = 2 * kHubEC;
  constexpr int PER = kHubEC / 256;  // edges per thread
  static_assert(kHubEC % 256 == 0, "edge chunk must be a multiple of the workgroup size");
  int *keys = l.keys, *used = l.used;
  double *vals = l.vals;
  int &nused = l.nused;
  const int h = a.hp.chub[q];
  const int i = a.hp.hubv[h];
  if (a.hub_front) {
    // The hub enters the frontier of its slice: every chunk takes the same
    // decision from the processed flag, which the scoring clears; the first
    // chunk records it and resets the proposal.
    const bool go = a.U[i] && a.rng[i];
    if (q == a.hp.hch[h] && threadIdx.x == 0) {
      a.prop[i] = -1;
      a.act[i] = go;
    }
    if (!go) return;
  } else if (!a.act[i]) {
    return;
  }
  const int64_t e0 = a.off[i] + (q - a.hp.hch[h]) * kHubEC;
  const int64_t e1 = min(e0 + (int64_t)kHubEC, a.off[i + 1]);
  if (a.hub_scanned && threadIdx.x == 0) atomicAdd(a.hub_scanned, (unsigned long long)(e1 - e0));
  for (int s = threadIdx.x; s < T; s += blockDim.x) { keys[s] = kEmpty; vals[s] = 0.0; }
  if (threadIdx.x == 0) nused = 0;
  // this thread's edges: all ids first, then all communities
  int j[PER], c[PER];
  float x[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t e = e0 + threadIdx.x + u * 256;
    j[u] = i;
    x[u] = 0.0f;
    if (e < e1) { j[u] = a.idx[e]; x[u] = a.w[e]; }
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) c[u] = j[u] != i ? a.C[j[u]] : kEmpty;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (c[u] != kEmpty) table_add(keys, vals, T - 1, c[u], (double)x[u]);
  __syncthreads();
  // list the taken slots, so that the merge into the hub's global table is
  // spread evenly over the threads
  for (int s0 = 0; s0 < T; s0 += blockDim.x) {
    const int s = s0 + threadIdx.x;
    const bool taken = keys[s] != kEmpty;
    const unsigned long long m = __ballot(taken);
    int base = 0;
    if (lane() == 0 && m) base = atomicAdd(&nused, (int)__popcll(m));
    base = __shfl(base, 0);
    if (taken) used[base + (int)__popcll(m & ((1ull << lane()) - 1ull))] = s;
  }
  __syncthreads();
  const int nu = nused;
  const int d = a.C[i];
  const int64_t t0 = a.hp.htab[h];
  const uint32_t mask = (uint32_t)(a.hp.hcap[h] - 1);
  for (int k = threadIdx.x; k < nu; k += blockDim.x) {
    const int s = used[k];
    const int cs = keys[s];
    if (cs == d) unsafeAtomicAdd(&a.hp.own[h], vals[s]);
    else table_add(a.hp.keys + t0, a.hp.vals + t0, mask, cs, vals[s]);
  }
}
__global__ __launch_bounds__(256) void k_hub_gather(MoveArgs a) {
  __shared__ HubGatherLds l;
  hub_gather_chunk(a, a.qbeg + blockIdx.x, l);
}

// score: a workgroup scans one table segment of a frontier hub, frees the
// slots it reads, and leaves the segment's best (gain, community).
// Result (gain bg, community bc) valid in thread 0.
__device__ __forceinline__ void hub_score_segment(const MoveArgs &a, int64_t q, int h, int i, double &bg, int &bc) {
  __shared__ double rg[256 / kWave];
  __shared__ int rc[256 / kWave];
  const int64_t s0 = a.hp.htab[h] + (q - a.hp.hsg[h]) * kHubSeg;
  const int64_t s1 = s0 + min((int64_t)kHubSeg, a.hp.hcap[h]);
  const int d = a.C[i];
  const double Ki = a.K[i], Sd = a.Sig[d], bown = a.hp.own[h];
  bg = 0.0;
  bc = kNoComm;
  // the thread's slots in three rounds of loads: keys, then weights and Sigma,
  // each round's together
  constexpr int PER = kHubSeg / 256;
  int c[PER];
  double v[PER], S[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t s = s0 + threadIdx.x + u * 256;
    c[u] = s < s1 ? a.hp.keys[s] : kEmpty;
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t s = s0 + threadIdx.x + u * 256;
    v[u] = c[u] != kEmpty ? a.hp.vals[s] : 0.0;
    S[u] = c[u] != kEmpty ? a.Sig[c[u]] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (c[u] == kEmpty) continue;
    const int64_t s = s0 + threadIdx.x + u * 256;
    a.hp.keys[s] = kEmpty;
    a.hp.vals[s] = 0.0;
    const double x = move_score(a.M2, v[u], bown, Ki, S[u], Sd);
    if (x > 0.0 && better(x, c[u], bg, bc)) { bg = x; bc = c[u]; }
  }
  team_argmax<256, 256>(bg, bc, rg, rc);
}
// ---- hub plan -------------------------------------------------------------------
// Each workgroup takes a contiguous range of vertices, counts its hubs per
// slice in LDS, reserves each slice's places with one global atomic and then
// writes them: one atomic per workgroup and slice instead of one per hub (a
// level has up to millions of hubs but only S counters, and device-scope
// atomics on one address are performed one after another).  S <= 256.
constexpr int kHubFindBlocks = 1024;
__global__ __launch_bounds__(256) void k_hub_find(const int64_t *off, int64_t n, int S, int64_t hubdeg,
                                                  const int32_t *hub_soff, int32_t *hub_fill, int32_t *hubv) {
  __shared__ int cnt[256];
  __shared__ int base[256];
  const int64_t per = ceil_div(n, (int64_t)gridDim.x);
  const int64_t v0 = (int64_t)blockIdx.x * per;
  const int64_t v1 = min(v0 + per, n);
  for (int k = threadIdx.x; k < S; k += blockDim.x) cnt[k] = 0;
  __syncthreads();
  for (int64_t i = v0 + threadIdx.x; i < v1; i += blockDim.x)
    if (off[i + 1] - off[i] > hubdeg) atomicAdd(&cnt[slice_of(i, S)], 1);
  __syncthreads();
  for (int k = threadIdx.x; k < S; k += blockDim.x) {
    base[k] = cnt[k] ? atomicAdd(&hub_fill[k], cnt[k]) : 0;
    cnt[k] = 0;
  }
  __syncthreads();
  for (int64_t i = v0 + threadIdx.x; i < v1; i += blockDim.x) {
    if (off[i + 1] - off[i] <= hubdeg) continue;
    const int sl = slice_of(i, S);
    hubv[hub_soff[sl] + base[sl] + atomicAdd(&cnt[sl], 1)] = (int32_t)i;
  }
}
void hub_find(const int64_t *off, int64_t n, int S, int64_t hubdeg, const int32_t *hub_soff, int32_t *hub_fill,
              int32_t *hubv, hipStream_t s) {
  if (n > 0)
    hipLaunchKernelGGL(k_hub_find, (int)std::min<int64_t>(kHubFindBlocks, ceil_div(n, (int64_t)256)), 256, 0, s,
                       off, n, S, hubdeg, hub_soff, hub_fill, hubv);
}

__global__ void k_hub_sizes(const int64_t *off, const int32_t *hubv, int64_t nhub, int64_t *nch, int64_t *ncap,
                            int64_t *nseg, int64_t *nbig) {
  for (int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; h <= nhub; h += (int64_t)gridDim.x * blockDim.x) {
    if (h == nhub) { nch[h] = 0; ncap[h] = 0; nseg[h] = 0; nbig[h] = 0; continue; }
    const int i = hubv[h];
    const int64_t deg = off[i + 1] - off[i];
    nbig[h] = deg > kWideDeg ? (int64_t)1 << 32 : deg > kHubDeg;
    if (deg <= kHubDeg) { nch[h] = 0; ncap[h] = 0; nseg[h] = 0; continue; }
    int64_t cap = kHubMinCap;
    while (cap < 2 * deg) cap <<= 1;
    nch[h] = ceil_div(deg, (int64_t)kHubEC);
    ncap[h] = cap;
    nseg[h] = ceil_div(cap, (int64_t)kHubSeg);
  }
}
void hub_sizes(const int64_t *off, const int32_t *hubv, int64_t nhub, int64_t *nch, int64_t *ncap, int64_t *nseg,
               int64_t *nbig, hipStream_t s) {
  hipLaunchKernelGGL(k_hub_sizes, flat_grid(nhub + 1), 256, 0, s, off, hubv, nhub, nch, ncap, nseg, nbig);
}

// Table offsets counted from the start of each hub's slice: the slices run
// one after another and scoring frees every slot it reads, so all slices
// share one table area of the largest slice's size.
__global__ void k_hub_rel(int64_t *htab, int64_t nhub, const int32_t *hub_soff, int S, const int64_t *slice_base) {
  for (int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; h < nhub; h += (int64_t)gridDim.x * blockDim.x) {
    int lo = 0, hi = S;  // the slice s with hub_soff[s] <= h < hub_soff[s + 1]
    while (hi - lo > 1) {
      const int mid = (lo + hi) / 2;
      if (hub_soff[mid] <= h) lo = mid;
      else hi = mid;
    }
    htab[h] -= slice_base[lo];
  }
}
void hub_rel(int64_t *htab, int64_t nhub, const int32_t *hub_soff, int S, const int64_t *slice_base, hipStream_t s) {
  if (nhub > 0) hipLaunchKernelGGL(k_hub_rel, flat_grid(nhub), 256, 0, s, htab, nhub, hub_soff, S, slice_base);
}

__global__ void k_hub_expand(HubPlan p, int64_t nhub) {
  for (int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; h < nhub; h += (int64_t)gridDim.x * blockDim.x) {
    for (int64_t q = p.hch[h]; q < p.hch[h + 1]; ++q) p.chub[q] = (int32_t)h;
    for (int64_t q = p.hsg[h]; q < p.hsg[h + 1]; ++q) p.shub[q] = (int32_t)h;
  }
}
void hub_expand(const HubPlan &h, int64_t nhub, hipStream_t s) {
  if (nhub > 0) hipLaunchKernelGGL(k_hub_expand, flat_grid(nhub), 256, 0, s, h, nhub);
}

__global__ void k_gather_bounds(const int64_t *arr, const int32_t *at, int count, int64_t *out) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < count; k += gridDim.x * blockDim.x) out[k] = arr[at[k]];
}
void gather_bounds(const int64_t *arr, const int32_t *at, int count, int64_t *out, hipStream_t s) {
  if (count > 0) hipLaunchKernelGGL(k_gather_bounds, flat_grid(count), 256, 0, s, arr, at, count, out);
}

// ---- apply: reverse-move resolution and move application ------------------
__device__ __forceinline__ bool reverse_wins(const MoveArgs &a, int j, int i, int fi, int p, double gi) {
  const int pj = a.prop[j];
  return pj >= 0 && pj == fi && a.from[j] == p && slice_of(j, a.nsl) == a.s && better(a.gp[j], j, gi, i);
}

__device__ __forceinline__ void flush_gain(const MoveArgs &a, double gsum, long long mv) {
  __shared__ double sd[16];
  __shared__ long long sl[16];
  const double g = block_sum(gsum, sd);
  const long long m = block_sum_ll(mv, sl);
  if (threadIdx.x == 0) {
    if (g != 0.0 && a.gain) unsafeAtomicAdd(a.gain, g);
    if (m) atomicAdd(a.moves, (unsigned long long)m);
  }
}

__device__ __forceinline__ void do_move(const MoveArgs &a, int i, int fi, int p, double g, double &gsum,
                                        long long &mv) {
  a.C[i] = p;
  const double k = a.K[i];
  unsafeAtomicAdd(&a.Sig[fi], -k);
  unsafeAtomicAdd(&a.Sig[p], k);
  if (a.track) { a.dC[fi] = 1; a.dC[p] = 1; }
  if (a.gi) a.gi[i] = g;
  else gsum += g;
  mv += 1;
}

template <int G>
__device__ __forceinline__ void apply_small(const MoveArgs &a, int b, int blk, int nblk) {
  const int count = a.counts[a.s * kNB + b];
  const int32_t *list = a.lists + a.region[a.s * kNB + b];
  const int gl = threadIdx.x & (G - 1);
  const int64_t wave = ((int64_t)blk * 256 + threadIdx.x) / kWave;
  const int64_t nwave = (int64_t)nblk * 256 / kWave;
  const int gin = lane() / G;
  double gsum = 0.0;
  long long mv = 0;
  const unsigned long long gm =
      (G == kWave) ? ~0ull : (((1ull << G) - 1ull) << (unsigned)(lane() & ~(G - 1)));
  for (int64_t v0 = wave * (kWave / G); v0 < count; v0 += nwave * (kWave / G)) {
    const int64_t v = v0 + gin;
    const int i = v < count ? list[v] : 0;
    const int p = v < count ? a.prop[i] : -1;
    bool blocked = false;
    int j = -1;
    int fi = 0;
    double g = 0.0;
    int deg = 0;
    if (p >= 0) {
      fi = a.from[i];
      g = a.gp[i];
      const int64_t e0 = a.off[i];
      deg = (int)(a.off[i + 1] - e0);
      if (gl < deg) {
        j = a.idx[e0 + gl];
        if (j != i) blocked = reverse_wins(a, j, i, fi, p, g);
      }
    }
    const bool any = (__ballot(blocked) & gm) != 0ull;
    if (p >= 0) {
      if (!any) {
        if (gl < deg && j != i) a.U[j] = 1;
        if (gl == 0) do_move(a, i, fi, p, g, gsum, mv);
      } else if (gl == 0) {
        a.U[i] = 1;
      }
    }
  }
  flush_gain(a, gsum, mv);
}

template <int TEAM, int BLOCK>
__device__ __forceinline__ void apply_team(const MoveArgs &a, int b, int blk, int nblk) {
  constexpr int NT = BLOCK / TEAM;
  __shared__ int sany[NT];
  const int team = threadIdx.x / TEAM;
  const int t = threadIdx.x % TEAM;
  const int count = a.counts[a.s * kNB + b];
  const int32_t *list = a.lists + a.region[a.s * kNB + b];
  double gsum = 0.0;
  long long mv = 0;
  for (int64_t base = (int64_t)blk * NT; base < count; base += (int64_t)nblk * NT) {
    const int64_t v = base + team;
    const bool valid = v < count;
    const int i = valid ? list[v] : 0;
    const int p = valid ? a.prop[i] : -1;
    int fi = 0;
    double g = 0.0;
    int64_t e0 = 0, e1 = 0;
    bool blocked = false;
    if (p >= 0) {
      fi = a.from[i];
      g = a.gp[i];
      e0 = a.off[i];
      e1 = a.off[i + 1];
      for (int64_t e = e0 + t; e < e1 && !blocked; e += TEAM) {
        const int j = a.idx[e];
        if (j != i && reverse_wins(a, j, i, fi, p, g)) blocked = true;
      }
    }
    bool any;
    if (TEAM == kWave) {
      any = __ballot(blocked) != 0ull;
    } else {
      if (t == 0) sany[team] = 0;
      __syncthreads();
      if (blocked) sany[team] = 1;
      __syncthreads();
      any = sany[team] != 0;
    }
    if (p >= 0) {
      if (!any) {
        for (int64_t e = e0 + t; e < e1; e += TEAM) {
          const int j = a.idx[e];
          if (j != i) a.U[j] = 1;
        }
        if (t == 0) do_move(a, i, fi, p, g, gsum, mv);
      } else if (t == 0) {
        a.U[i] = 1;
      }
    }
    if (TEAM != kWave) __syncthreads();
  }
  flush_gain(a, gsum, mv);
}

// ---- apply for hubs, chunk-parallel --------------------------------------------
// The same rule as the other buckets, with the hub's edge chunks spread over
// workgroups: (1) a chunk that finds a same-slice neighbour proposing the
// exact reverse move with priority flags the hub blocked; (2) every chunk of
// an unblocked hub marks its neighbours unprocessed and the first one moves
// the hub, while the first chunk of a blocked hub leaves it unprocessed.
__device__ __forceinline__ void hub_rev_chunk(const MoveArgs &a, int64_t q) {
  const int h = a.hp.chub[q];
  const int i = a.hp.hubv[h];
  if (!a.act[i]) return;
  const int p = a.prop[i];
  if (p < 0) return;
  const int fi = a.from[i];
  const double g = a.gp[i];
  const int64_t e0 = a.off[i] + (q - a.hp.hch[h]) * kHubEC;
  const int64_t e1 = min(e0 + (int64_t)kHubEC, a.off[i + 1]);
  bool blocked = false;
  for (int64_t e = e0 + threadIdx.x; e < e1 && !blocked; e += blockDim.x) {
    const int j = a.idx[e];
    if (j != i && reverse_wins(a, j, i, fi, p, g)) blocked = true;
  }
  if (blocked) a.hp.flag[h] = 1;
}
// All buckets of a slice but the hubs, and the reverse checks of the hubs'
// chunks (the first `chunks` workgroups): nothing that one of them reads is
// written by another.
__global__ __launch_bounds__(256) void k_apply_slice(MoveArgs a, BucketSpan sp, int chunks) {
  if ((int)blockIdx.x < chunks) {
    hub_rev_chunk(a, a.qbeg + blockIdx.x);
    return;
  }
  const int at = blockIdx.x - chunks;
  int b = 0;
  while (at >= sp.first[b + 1]) ++b;
  const int blk = at - sp.first[b], nblk = sp.first[b + 1] - sp.first[b];
  switch (b) {
    case 0: apply_small<4>(a, b, blk, nblk); break;
    case 1: apply_small<8>(a, b, blk, nblk); break;
    case 2: apply_small<32>(a, b, blk, nblk); break;
    case 3: apply_team<64, 256>(a, b, blk, nblk); break;
    default: apply_team<256, 256>(a, b, blk, nblk); break;
  }
}

__global__ __launch_bounds__(256) void k_hub_mark(MoveArgs a) {
  const int64_t q = a.qbeg + blockIdx.x;
  const int h = a.hp.chub[q];
  const int i = a.hp.hubv[h];
  if (!a.act[i]) return;
  const int p = a.prop[i];
  if (p < 0) return;
  const bool lead = q == a.hp.hch[h] && threadIdx.x == 0;
  if (a.hp.flag[h] == 1) {
    if (lead) a.U[i] = 1;
    return;
  }
  if (lead) {
    double gsum = 0.0;
    long long mv = 0;
    do_move(a, i, a.from[i], p, a.gp[i], gsum, mv);
    if (gsum != 0.0 && a.gain) unsafeAtomicAdd(a.gain, gsum);
    atomicAdd(a.moves, 1ull);
  }
  const int64_t e0 = a.off[i] + (q - a.hp.hch[h]) * kHubEC;
  const int64_t e1 = min(e0 + (int64_t)kHubEC, a.off[i + 1]);
  for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
    const int j = a.idx[e];
    if (j != i) a.U[j] = 1;
  }
}

// ---- the hub slices of the asynchronous mode -------------------------------------
// A level's hubs move in up to 256 slices, one after another, and most slices
// hold a handful of hubs of a few hundred to a few thousand edges: a slice is
// a chain of launches, each bound by its own latency.  A hub that a workgroup
// can read at once gets one workgroup, with its table in LDS and its edges in
// registers, so that the chain is two launches of ~7 us (propose; reverse
// check and apply) instead of the five of the chunked kernels above (gather
// 11, score 10, final, rev and mark 3 each).  A slice with hubs beyond a
// workgroup's reach is four launches: its chunks ride with the other hubs'
// workgroups, and the last segment of a hub to be scored picks the hub's
// best.  The rule is that of the sliced sweep: the proposals of a slice all
// read the state before it.  (Moving 1/64 of the hubs at a time without the
// slices, each applied at once, was faster still, but cost 5e-3 to 7e-3 of
// modularity on R-MAT graphs of scale 16 to 22.)
template <int T, int PER, int SLOTS>
__device__ __forceinline__ void hub_propose(const MoveArgs &a, int64_t h, int64_t lo, int64_t hi,
                                            BlockTable<T, PER, SLOTS> &l) {
  const int i = a.hp.hubv[h];
  const int64_t e0 = a.off[i];
  const int deg = (int)min(a.off[i + 1] - e0, (int64_t)INT_MAX);
  if (deg <= lo || deg > hi) return;
  // only this workgroup writes the hub's flag in this launch, after the
  // barriers of block_best
  const bool go = a.U[i] && a.rng[i];
  if (!go) {
    if (threadIdx.x == 0) a.prop[i] = -1;
    return;
  }
  int j[PER], c[PER];
  float x[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int e = threadIdx.x + u * T;
    j[u] = i;
    x[u] = 0.0f;
    if (e < deg) { j[u] = a.idx[e0 + e]; x[u] = a.w[e0 + e]; }
  }
  const int d = a.C[i];
  const double Ki = a.K[i], Sd = a.Sig[d];
#pragma unroll
  for (int u = 0; u < PER; ++u) c[u] = j[u] != i ? a.C[j[u]] : kEmpty;
  double bg;
  int bc;
  block_best(l, deg, c, x, d, a.M2, Ki, Sd, a.Sig, bg, bc);
  if (threadIdx.x == 0) {
    a.U[i] = 0;
    a.from[i] = d;
    a.prop[i] = bc == kNoComm ? -1 : bc;
    a.gp[i] = bg;
    if (a.hub_scanned) atomicAdd(a.hub_scanned, (unsigned long long)deg);
  }
}

// Hubs of degree <= kHubDeg; the first `chunks` workgroups gather the chunks
// of the others.
__global__ __launch_bounds__(256) void k_hub_propose(MoveArgs a, int chunks) {
  __shared__ union {
    HubGatherLds gather;
    BlockTable<256, 8, 4096> table;
  } l;
  if ((int)blockIdx.x < chunks) hub_gather_chunk(a, a.qbeg + blockIdx.x, l.gather);
  else hub_propose<256, 8, 4096>(a, a.hbeg + blockIdx.x - chunks, 0, kHubDeg, l.table);
}
// One kind of hub of a large slice: degree in (lo, hi].
template <int PER, int SLOTS>
__global__ __launch_bounds__(256) void k_hub_propose_kind(MoveArgs a, int64_t lo, int64_t hi) {
  __shared__ BlockTable<256, PER, SLOTS> l;
  hub_propose<256, PER, SLOTS>(a, a.hbeg + blockIdx.x, lo, hi, l);
}
__global__ __launch_bounds__(kWideT) void k_hub_propose_wide(MoveArgs a, int64_t lo) {
  __shared__ BlockTable<kWideT, kWidePer, 8192> l;
  hub_propose<kWideT, kWidePer, 8192>(a, a.hbeg + blockIdx.x, lo, kWideDeg, l);
}

// Scores the segments of the chunked hubs; a hub's last one to finish reduces
// them all to the hub's proposal.
__global__ __launch_bounds__(256) void k_hub_score_final(MoveArgs a) {
  const int64_t q = a.gbeg + blockIdx.x;
  const int h = a.hp.shub[q];
  const int i = a.hp.hubv[h];
  if (!a.act[i]) return;
  double bg;
  int bc;
  hub_score_segment(a, q, h, i, bg, bc);
  if (!hub_last_segment(a.hp, h, q, bg, bc)) return;
  hub_reduce_segments(a.hp, h, bg, bc);
  if (threadIdx.x == 0) {
    a.from[i] = a.C[i];
    a.prop[i] = bc == kNoComm ? -1 : bc;
    a.gp[i] = bg;
    a.U[i] = 0;  // the gather has read it
  }
}

// Reverse check of the slice's proposals; hubs of degree <= hi (a workgroup
// each) then move, the chunked ones in k_hub_mark.
__global__ __launch_bounds__(256) void k_hub_apply(MoveArgs a, int chunks, int64_t hi) {
  if ((int)blockIdx.x < chunks) {
    hub_rev_chunk(a, a.qbeg + blockIdx.x);
    return;
  }
  const int i = a.hp.hubv[a.hbeg + blockIdx.x - chunks];
  const int64_t e0 = a.off[i], e1 = a.off[i + 1];
  if (e1 - e0 > hi) return;
  const int p = a.prop[i];
  if (p < 0) return;
  const int fi = a.from[i];
  const double g = a.gp[i];
  int blocked = 0;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
    const int j = a.idx[e];
    if (j != i && reverse_wins(a, j, i, fi, p, g)) blocked = 1;
  }
  if (__syncthreads_or(blocked)) {
    if (threadIdx.x == 0) a.U[i] = 1;
    return;
  }
  if (threadIdx.x == 0) {
    double gsum = 0.0;
    long long mv = 0;
    do_move(a, i, fi, p, g, gsum, mv);
    if (gsum != 0.0 && a.gain) unsafeAtomicAdd(a.gain, gsum);
    atomicAdd(a.moves, 1ull);
  }
  for (int64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
    const int j = a.idx[e];
    if (j != i) a.U[j] = 1;
  }
}

// ---- launchers -----------------------------------------------------------------
void move_frontier(const MoveArgs &a, hipStream_t s) {
  if (a.vend > a.vbeg)
    hipLaunchKernelGGL(k_frontier, flat_grid(ceil_div(a.vend - a.vbeg, kFrontTile), 1, 2048), 256, 0, s, a);
}

void move_propose(const MoveArgs &a, const int64_t *region_h, hipStream_t s) {
  const BucketSpan sp = bucket_span(region_h + a.s * kNB);
  if (sp.first[kNB - 1] == 0) return;
  if (sp.first[kNB - 1] <= kShareLaunch) {
    hipLaunchKernelGGL(k_propose_slice, sp.first[kNB - 1], 256, 0, s, a, sp);
    return;
  }
  for (int b = 0; b + 1 < kNB; ++b) {
    const int g = sp.first[b + 1] - sp.first[b];
    if (g == 0) continue;
    switch (b) {
      case 0: hipLaunchKernelGGL(k_propose_small<4>, g, 256, 0, s, a, b); break;
      case 1: hipLaunchKernelGGL(k_propose_small<8>, g, 256, 0, s, a, b); break;
      case 2: hipLaunchKernelGGL(k_propose_small<32>, g, 256, 0, s, a, b); break;
      case 3: hipLaunchKernelGGL((k_propose_team<64, 512, 256>), g, 256, 0, s, a, b); break;
      default: hipLaunchKernelGGL((k_propose_team<256, 4096, 256>), g, 256, 0, s, a, b); break;
    }
  }
}

void move_hub_gather(const MoveArgs &a, hipStream_t s) {
  if (a.qend > a.qbeg) hipLaunchKernelGGL(k_hub_gather, (int)(a.qend - a.qbeg), 256, 0, s, a);
}

void move_hub_score(const MoveArgs &a, hipStream_t s) {
  if (a.qend > a.qbeg) hipLaunchKernelGGL(k_hub_score_final, (int)(a.gend - a.gbeg), 256, 0, s, a);
}

void move_apply(const MoveArgs &a, const int64_t *region_h, hipStream_t s) {
  const BucketSpan sp = bucket_span(region_h + a.s * kNB);
  const int nq = (int)(a.qend - a.qbeg);
  if (nq + sp.first[kNB - 1] > 0)
    hipLaunchKernelGGL(k_apply_slice, nq + sp.first[kNB - 1], 256, 0, s, a, sp, nq);
  if (nq > 0) hipLaunchKernelGGL(k_hub_mark, nq, 256, 0, s, a);
}

void move_hubs(const MoveArgs &a, bool wide, hipStream_t s) {
  const int nh = (int)(a.hend - a.hbeg), nq = (int)(a.qend - a.qbeg);
  if (nh <= 0) return;
  // the large workgroups, one a CU, take all hubs of a slice while they find
  // a CU each
  const bool all = nq == 0 && wide && nh <= kWideAll;
  if (nq + nh > kShareLaunch) {
    move_hub_gather(a, s);
    hipLaunchKernelGGL((k_hub_propose_kind<2, 1024>), nh, 256, 0, s, a, (int64_t)0, kSmallHubDeg);
    hipLaunchKernelGGL((k_hub_propose_kind<8, 4096>), nh, 256, 0, s, a, kSmallHubDeg, kHubDeg);
  } else if (!all) {
    hipLaunchKernelGGL(k_hub_propose, nq + nh, 256, 0, s, a, nq);
  }
  if (nq > 0) hipLaunchKernelGGL(k_hub_score_final, (int)(a.gend - a.gbeg), 256, 0, s, a);
  else if (wide) hipLaunchKernelGGL(k_hub_propose_wide, nh, kWideT, 0, s, a, all ? 0 : kHubDeg);
  hipLaunchKernelGGL(k_hub_apply, nq + nh, 256, 0, s, a, nq, nq > 0 ? kHubDeg : kWideDeg);
  if (nq > 0) hipLaunchKernelGGL(k_hub_mark, nq, 256, 0, s, a);
}

// ---- fixed-order gain total (synchronous mode) ------------------------------------
// Sums of 256 values in order.  A workgroup reads the values of kTilesPer tiles
// together and a thread then adds each tile's from LDS: with a thread's loads
// one after another 28 us for 391 tiles, now below 10.
constexpr int kTilesPer = 16;
__global__ __launch_bounds__(256) void k_tile_sums(const double *x, int64_t n, double *tiles) {
  __shared__ double v[kTilesPer][257];
  const int64_t ntiles = ceil_div(n, 256);
  for (int64_t t0 = (int64_t)blockIdx.x * kTilesPer; t0 < ntiles; t0 += (int64_t)gridDim.x * kTilesPer) {
#pragma unroll
    for (int k = 0; k < kTilesPer; ++k) {
      const int64_t q = (t0 + k) * 256 + threadIdx.x;
      v[k][threadIdx.x] = q < n ? x[q] : 0.0;
    }
    __syncthreads();
    const int64_t t = t0 + threadIdx.x;
    if (threadIdx.x < kTilesPer && t < ntiles) {
      const int m = (int)min((int64_t)256, n - t * 256);
      double s = 0.0;
#pragma unroll 16
      for (int k = 0; k < m; ++k) s += v[threadIdx.x][k];
      tiles[t] = s;
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(64) void k_tiles_total(const double *tiles, int64_t ntiles, double *out) {
  __shared__ double buf[64];
  double total = 0.0;
  for (int64_t base = 0; base < ntiles; base += 64) {
    const int64_t k = base + threadIdx.x;
    buf[threadIdx.x] = k < ntiles ? tiles[k] : 0.0;
    __syncthreads();
    if (threadIdx.x == 0) {
      const int64_t m = min((int64_t)64, ntiles - base);
      for (int64_t q = 0; q < m; ++q) total += buf[q];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = total;
}

void tiled_sum(const double *gi, int64_t n, double *tiles, double *out, hipStream_t s) {
  const int64_t ntiles = ceil_div(n, 256);
  if (ntiles > 0) hipLaunchKernelGGL(k_tile_sums, flat_grid(ceil_div(ntiles, (int64_t)kTilesPer), 1, 2048), 256, 0, s, gi, n, tiles);
  hipLaunchKernelGGL(k_tiles_total, 1, 64, 0, s, tiles, ntiles, out);
}

}  // namespace lk
