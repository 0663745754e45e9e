// Device-wide primitives of the library: exclusive prefix scans and a stable
// least-significant-digit radix sort of (key, value) pairs over independent
// segments.  Both work in tiles of 4096 items (256 threads x 16 rounds); no
// vendor primitive library is used.
//
// Scan: tile totals (one workgroup per tile), a scan of the totals (the same
// routine, recursively), then each tile scans its items with the tile's prefix
// as carry, a wavefront 16 rounds of 64.  In-place use (in == out) is allowed.
//
// Radix sort: per pass (digits of at most 9 bits) a digit histogram per tile,
// an exclusive scan of the histograms laid out segment-major, digit-major,
// tile-minor (so the scanned value of (segment, digit, tile) is where the
// tile's items of that digit go), and a stable scatter that ranks the items of
// each 256-item round with wavefront ballots (lanes with the same digit) plus
// per-wavefront counts into a digit-sorted copy of the tile in LDS, written
// out in order (coalesced runs per digit).  Tiles never cross a segment.
#include <algorithm>

#include "device.hpp"
#include "kernels.hpp"

namespace lk {

// exclusive prefix over the workgroup of one value per thread, in thread
// order; *tot receives the workgroup total.  All threads must call it.
template <class T>
__device__ __forceinline__ T blk_excl(T x, T *tot, T *sw /* >= kPT / kWave */) {
  T incl = x;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const T y = __shfl_up(incl, o);
    if (lane() >= o) incl += y;
  }
  const int w = (int)threadIdx.x / kWave;
  if (lane() == kWave - 1) sw[w] = incl;
  __syncthreads();
  T pre = 0, all = 0;
#pragma unroll
  for (int k = 0; k < kPT / kWave; ++k) {
    if (k < w) pre += sw[k];
    all += sw[k];
  }
  __syncthreads();
  *tot = all;
  return pre + incl - x;
}

// ---- scan ----------------------------------------------------------------------
template <class I, class O>
__global__ __launch_bounds__(kPT) void k_scan_reduce(const I *in, int64_t n, O *tsum) {
  __shared__ O sw[kPT / kWave];
  const int64_t b = (int64_t)blockIdx.x * kPTile;
  O x[kPR];
#pragma unroll
  for (int r = 0; r < kPR; ++r) {
    const int64_t p = b + r * kPT + threadIdx.x;
    x[r] = p < n ? (O)in[p] : (O)0;
  }
  O s = 0;
#pragma unroll
  for (int r = 0; r < kPR; ++r) s += x[r];
  O tot;
  (void)wave_scan(s, &tot);
  if (lane() == 0) sw[threadIdx.x / kWave] = tot;
  __syncthreads();
  if (threadIdx.x == 0) {
    tot = 0;
#pragma unroll
    for (int w = 0; w < kPT / kWave; ++w) tot += sw[w];
    tsum[blockIdx.x] = tot;
  }
}

// Most scans here are of one tile or a few and lie in a chain of launches: the
// items are loaded together and the rounds' prefixes taken with lane moves,
// with one barrier (16 rounds of 256 one after another, two barriers each and
// the prefix through LDS permutes: 12 us a tile, now 4.5).
template <class I, class O>
__global__ __launch_bounds__(kPT) void k_scan_apply(const I *in, O *out, int64_t n, const O *tpre) {
  __shared__ O sw[kPT / kWave];
  const int wv = threadIdx.x / kWave;
  const int64_t b = (int64_t)blockIdx.x * kPTile + wv * (kPTile / (kPT / kWave));
  O x[kPR], ex[kPR], tot[kPR], sum = 0;
#pragma unroll
  for (int r = 0; r < kPR; ++r) {
    const int64_t p = b + r * kWave + lane();
    x[r] = p < n ? (O)in[p] : (O)0;
  }
#pragma unroll
  for (int r = 0; r < kPR; ++r) {
    ex[r] = wave_scan(x[r], &tot[r]) - x[r];
    sum += tot[r];
  }
  if (lane() == 0) sw[wv] = sum;
  __syncthreads();
  O carry = tpre ? tpre[blockIdx.x] : (O)0;
#pragma unroll
  for (int w = 0; w < kPT / kWave; ++w)
    if (w < wv) carry += sw[w];
#pragma unroll
  for (int r = 0; r < kPR; ++r) {
    const int64_t p = b + r * kWave + lane();
    if (p < n) out[p] = carry + ex[r];
    carry += tot[r];
  }
}

int64_t scan_tmp_elems(int64_t n) {
  int64_t t = 0;
  while (n > kPTile) {
    n = ceil_div(n, kPTile);
    t += n;
  }
  return t;
}

template <class I, class O>
void scan_rec(const I *in, O *out, int64_t n, O *tmp, hipStream_t s) {
  if (n <= 0) return;
  if (n <= kPTile) {
    hipLaunchKernelGGL((k_scan_apply<I, O>), 1, kPT, 0, s, in, out, n, (const O *)nullptr);
    return;
  }
  const int64_t nt = ceil_div(n, kPTile);
  hipLaunchKernelGGL((k_scan_reduce<I, O>), (int)nt, kPT, 0, s, in, n, tmp);
  scan_rec<O, O>(tmp, tmp, nt, tmp + nt, s);
  hipLaunchKernelGGL((k_scan_apply<I, O>), (int)nt, kPT, 0, s, in, out, n, (const O *)tmp);
}

static size_t scan_bytes(int64_t n, size_t osize) {
  return std::max<size_t>(256, (size_t)scan_tmp_elems(n) * osize);
}
size_t scan_excl_i32(void *temp, size_t tbytes, const int32_t *in, int32_t *out, int64_t n, hipStream_t s) {
  const size_t need = scan_bytes(n, sizeof(int32_t));
  if (temp && tbytes >= need) scan_rec<int32_t, int32_t>(in, out, n, (int32_t *)temp, s);
  return need;
}
size_t scan_excl_i64(void *temp, size_t tbytes, const int64_t *in, int64_t *out, int64_t n, hipStream_t s) {
  const size_t need = scan_bytes(n, sizeof(int64_t));
  if (temp && tbytes >= need) scan_rec<int64_t, int64_t>(in, out, n, (int64_t *)temp, s);
  return need;
}
size_t scan_excl_i32_to_i64(void *temp, size_t tbytes, const int32_t *in, int64_t *out, int64_t n,
                            hipStream_t s) {
  const size_t need = scan_bytes(n, sizeof(int64_t));
  if (temp && tbytes >= need) scan_rec<int32_t, int64_t>(in, out, n, (int64_t *)temp, s);
  return need;
}

// ---- radix sort ------------------------------------------------------------------
constexpr int kRadixBits = 9;            // digits of at most 9 bits
constexpr int kDig = 1 << kRadixBits;    // 512 digit values
constexpr int kDPT = kDig / kPT;         // digits per thread

// Sorted are the key's `low` low bits and, above them, its bits from 32 on
// (keys of two ids of fewer bits each; low = 32: the whole key).
template <class K>
__device__ __forceinline__ int rs_digit(K key, int low, int shift, int bits) {
  if constexpr (sizeof(K) == 8) key = ((key >> 32) << low) | (key & (((K)1 << low) - 1));
  return (int)((key >> shift) & (K)((1u << bits) - 1u));
}

// hist: scan layout (segment, digit, tile) over the pass's 2^bits digits.
template <class K>
__global__ __launch_bounds__(kPT) void k_rs_hist(const K *keys, RsSeg g, int low, int shift, int bits, int64_t *hist) {
  __shared__ int h[kDig];
  const int64_t t = blockIdx.x;
  const TileSpan ts = tile_span(g, t);
  for (int d = threadIdx.x; d < kDig; d += kPT) h[d] = 0;
  __syncthreads();
  // all of the thread's loads issued together, then the counts
  K kr[kPR];
#pragma unroll
  for (int r = 0; r < kPR; ++r) {
    const int64_t p = ts.lo + r * kPT + threadIdx.x;
    kr[r] = p < ts.hi ? keys[p] : (K)0;
  }
#pragma unroll
  for (int r = 0; r < kPR; ++r)
    if (ts.lo + r * kPT + threadIdx.x < ts.hi) atomicAdd(&h[rs_digit(kr[r], low, shift, bits)], 1);
  __syncthreads();
  const int nd = 1 << bits;
  for (int d = threadIdx.x; d < nd; d += kPT) hist[nd * ts.f0 + (int64_t)d * ts.nt + (t - ts.f0)] = h[d];
}

// Each tile ranks its items stably by digit into a local digit-sorted copy in
// LDS, then writes it out in order: the items of one digit go to consecutive
// places, so consecutive threads write consecutive addresses.  hs: the scanned
// histograms (null: the sort is of this one tile, whose order is final).  Each
// wavefront ranks its own contiguous quarter of the tile (16 rounds of 64
// items, in order) against digit counters that only it uses, so the rounds
// need no workgroup barrier; one prefix over the digits and the four
// wavefronts' counts then gives every item its place.  Items are ordered by
// (wavefront, round, lane), which is their order in the tile: stable.
template <class K, class V>
__global__ __launch_bounds__(kPT) void k_rs_scatter(const K *ki, const V *vi, K *ko, V *vo, RsSeg g, int low,
                                                    int shift, int bits, const int64_t *hs) {
  constexpr int W = kPT / kWave;
  constexpr int QW = kPTile / W;  // items per wavefront
  __shared__ K sk[kPTile];
  __shared__ V sv[kPTile];
  __shared__ int64_t gbase[kDig];
  __shared__ int cnt[W][kDig];
  __shared__ int sw[W];
  const int64_t t = blockIdx.x;
  const TileSpan ts = tile_span(g, t);
  const int nd = 1 << bits;
  const int64_t seg0 = hs ? hs[nd * ts.f0] : 0;
  const int wid = (int)threadIdx.x / kWave;
  for (int d = threadIdx.x; d < kDig; d += kPT) {
#pragma unroll
    for (int w = 0; w < W; ++w) cnt[w][d] = 0;
  }
  // the wavefront's items in registers first (all loads in flight together)
  const int64_t q0 = ts.lo + (int64_t)wid * QW;
  K kr[kPR];
  V vr[kPR];
#pragma unroll
  for (int r = 0; r < kPR; ++r) {
    const int64_t p = q0 + r * kWave + lane();
    kr[r] = (K)0;
    vr[r] = V();
    if (p < ts.hi) {
      kr[r] = ki[p];
      vr[r] = vi[p];
    }
  }
  __syncthreads();  // counters cleared
  const unsigned long long below = lane() == 0 ? 0ull : (~0ull >> (64 - lane()));
  int rk[kPR];
#pragma unroll
  for (int r = 0; r < kPR; ++r) {
    const int64_t p = q0 + r * kWave + lane();
    const bool act = p < ts.hi;
    const int dg = act ? rs_digit(kr[r], low, shift, bits) : 0;
    unsigned long long same = __ballot(act);
    for (int bit = 0; bit < bits; ++bit) {
      const unsigned long long on = __ballot(act && ((dg >> bit) & 1));
      same &= ((dg >> bit) & 1) ? on : ~on;
    }
    const int rank_w = __popcll(same & below);
    // every lane reads the count before the group's first lane adds to it
    // (one wavefront's LDS operations execute in order)
    const int old = act ? cnt[wid][dg] : 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    if (act && rank_w == 0) cnt[wid][dg] = old + __popcll(same);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    rk[r] = old + rank_w;
  }
  __syncthreads();
  {
    // digit d's items start at the total of the smaller digits; wavefront w's
    // after those of the wavefronts before it.  Each thread owns kDPT digits.
    int c[kDPT][W], sum = 0;
#pragma unroll
    for (int k = 0; k < kDPT; ++k) {
      const int d = threadIdx.x * kDPT + k;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        c[k][w] = cnt[w][d];
        sum += c[k][w];
      }
    }
    int tot;
    int pre = blk_excl<int>(sum, &tot, sw);  // barriers: every count read above
#pragma unroll
    for (int k = 0; k < kDPT; ++k) {
      const int d = threadIdx.x * kDPT + k;
      if (d < nd) gbase[d] = ts.sb + (hs ? hs[nd * ts.f0 + (int64_t)d * ts.nt + (t - ts.f0)] - seg0 - pre : 0);
#pragma unroll
      for (int w = 0; w < W; ++w) {
        cnt[w][d] = pre;
        pre += c[k][w];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kPR; ++r) {
    const int64_t p = q0 + r * kWave + lane();
    if (p < ts.hi) {
      const int dg = rs_digit(kr[r], low, shift, bits);
      const int q = cnt[wid][dg] + rk[r];
      sk[q] = kr[r];
      sv[q] = vr[r];
    }
  }
  __syncthreads();
  const int m = (int)(ts.hi - ts.lo);
  for (int j = threadIdx.x; j < m; j += kPT) {
    const K key = sk[j];
    const int dg = rs_digit(key, low, shift, bits);
    const int64_t q = gbase[dg] + j;
    ko[q] = key;
    vo[q] = sv[j];
  }
}

int rs_passes(int bits) { return bits <= 0 ? 0 : (bits + kRadixBits - 1) / kRadixBits; }

size_t rs_tmp_bytes(int64_t ntiles) {
  const int64_t nh = (int64_t)kDig * std::max<int64_t>(ntiles, 1);
  return (size_t)nh * sizeof(int64_t) + scan_bytes(nh, sizeof(int64_t));
}

template <class K, class V>
int rsort(K *k0, V *v0, K *k1, V *v1, const RsSeg &g, int bits, void *tmp, hipStream_t s, int low) {
  const int np = rs_passes(bits);
  if (np == 0 || g.ntiles <= 0) return 0;
  const int wd = (bits + np - 1) / np;
  const int64_t nhmax = (int64_t)kDig * g.ntiles;
  int64_t *hist = (int64_t *)tmp;
  int64_t *stmp = hist + nhmax;
  K *ks = k0, *kd = k1;
  V *vs = v0, *vd = v1;
  int shift = 0;
  for (int p = 0; p < np; ++p) {
    const int b = std::min(wd, bits - shift);
    const bool one = g.ntiles == 1;
    if (!one) {
      hipLaunchKernelGGL((k_rs_hist<K>), (int)g.ntiles, kPT, 0, s, (const K *)ks, g, low, shift, b, hist);
      scan_rec<int64_t, int64_t>(hist, hist, ((int64_t)1 << b) * g.ntiles, stmp, s);
    }
    hipLaunchKernelGGL((k_rs_scatter<K, V>), (int)g.ntiles, kPT, 0, s, (const K *)ks, (const V *)vs, kd, vd, g,
                       low, shift, b, one ? (const int64_t *)nullptr : (const int64_t *)hist);
    std::swap(ks, kd);
    std::swap(vs, vd);
    shift += b;
  }
  return np & 1;
}

template int rsort<uint32_t, int32_t>(uint32_t *, int32_t *, uint32_t *, int32_t *, const RsSeg &, int, void *,
                                      hipStream_t, int);
template int rsort<uint32_t, float>(uint32_t *, float *, uint32_t *, float *, const RsSeg &, int, void *,
                                    hipStream_t, int);

RsSeg rs_plain(int64_t n) {
  RsSeg g;
  g.ntiles = ceil_div(n, kPTile);
  g.n = n;
  g.tseg = nullptr;
  g.tfirst = nullptr;
  g.sbeg = nullptr;
  g.send = nullptr;
  return g;
}

int key_bits(unsigned long long x) {
  int b = 0;
  while (b < 64 && (x >> b) != 0ull) ++b;
  return b;
}

template int rsort<unsigned long long, int32_t>(unsigned long long *, int32_t *, unsigned long long *, int32_t *,
                                                 const RsSeg &, int, void *, hipStream_t, int);
template int rsort<unsigned long long, double>(unsigned long long *, double *, unsigned long long *, double *,
                                                const RsSeg &, int, void *, hipStream_t, int);
template int rsort<unsigned long long, float>(unsigned long long *, float *, unsigned long long *, float *,
                                               const RsSeg &, int, void *, hipStream_t, int);

// Rows sorted by column id: (row << 32 | column) keys over the bits in use.
// By chunks of positions: with a row a thread, the longest row's thread was the
// kernel (R-MAT scale 17, 1.75 ms).
__global__ __launch_bounds__(256) void k_row_keys(const int64_t *off, int64_t nnz, const int32_t *crow,
                                                  const int32_t *col, unsigned long long *keys) {
  __shared__ int rowof[kChunk];
  __shared__ int sh[16];
  const int64_t q0 = (int64_t)blockIdx.x * kChunk;
  const int len = (int)min((int64_t)kChunk, nnz - q0);
  chunk_rows<kChunk>(off, q0, len, crow[blockIdx.x], crow[blockIdx.x + 1], rowof, sh);
  for (int t = threadIdx.x; t < len; t += blockDim.x)
    keys[q0 + t] = ((unsigned long long)rowof[t] << 32) | (unsigned long long)(uint32_t)col[q0 + t];
}
__global__ void k_low_words(const unsigned long long *keys, int64_t n, int32_t *col) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    col[e] = (int32_t)(uint32_t)keys[e];
}
size_t seg_sort_i32_f32(void *temp, size_t tbytes, const int32_t *kin, int32_t *kout, const float *vin, float *vout,
                        int64_t nnz, int64_t nseg, const int64_t *off, const int32_t *crow, hipStream_t s) {
  const RsSeg g = rs_plain(nnz);
  const size_t kb = ((size_t)std::max<int64_t>(nnz, 1) * 8 + 255) & ~(size_t)255;
  const size_t vb = ((size_t)std::max<int64_t>(nnz, 1) * 4 + 255) & ~(size_t)255;
  const size_t need = 2 * kb + vb + rs_tmp_bytes(g.ntiles);
  if (!temp || tbytes < need || nnz <= 0) return need;
  char *t = (char *)temp;
  unsigned long long *k0 = (unsigned long long *)t, *k1 = (unsigned long long *)(t + kb);
  float *v1 = (float *)(t + 2 * kb);
  hipLaunchKernelGGL(k_row_keys, (int)ceil_div(nnz, (int64_t)kChunk), 256, 0, s, off, nnz, crow, kin, k0);
  const int low = key_bits((unsigned long long)std::max<int64_t>(nseg - 1, 0)), bits = 2 * low;
  const bool odd = rs_passes(bits) & 1;  // values end in vout either way
  (void)hipMemcpyAsync(odd ? v1 : vout, vin, sizeof(float) * nnz, hipMemcpyDeviceToDevice, s);
  const int r = odd ? rsort<unsigned long long, float>(k0, v1, k1, vout, g, bits, t + 2 * kb + vb, s, low)
                    : rsort<unsigned long long, float>(k0, vout, k1, v1, g, bits, t + 2 * kb + vb, s, low);
  hipLaunchKernelGGL(k_low_words, flat_grid(nnz), 256, 0, s, r ? k1 : k0, nnz, kout);
  return need;
}

}  // namespace lk
