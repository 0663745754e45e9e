// Modularity, Eq. 1: Q = sum_c [sigma_c / 2m - (Sigma_c / 2m)^2], with sigma_c the
// weight of stored entries inside c and Sigma_c the total weight of c.  One
// chunked pass over the CSR accumulates the internal weight and the row sums,
// merged by community within the chunk before they are added to Sigma (FP64); a second pass over communities sums Sigma_c and
// (Sigma_c / 2m)^2.
#include "device.hpp"
#include "kernels.hpp"

namespace lk {

// The pass is a few times the workgroups that the device holds, each with a range of
// chunks, its internal weight in registers and its sums by community in a
// table that it empties when that fills and at its end: atomics on one address
// are performed one after another, ~14 ns each, and with a workgroup a chunk
// those on the internal weight alone (and on the large communities) took as
// long as the whole pass.  A community that finds no slot near its own goes to
// memory at once.  R-MAT scale 22, 128M entries: 1.78 -> 1.31 ms (2048
// workgroups 1.45; a million labels, in the L2, 1.11; 4096 labels 0.79).
constexpr int kModBlocks = 8192;
constexpr int kModSlots = 512;
constexpr int kModProbes = 16;
__global__ __launch_bounds__(256) void k_mod_edges(const int64_t *off, const int32_t *idx, const float *w,
                                                   const int32_t *crow, int64_t nnz, const int32_t *C,
                                                   double *acc, double *S) {
  __shared__ int rowof[kChunk];
  __shared__ int tk[kModSlots];
  __shared__ double tv[kModSlots];
  __shared__ int sh[16];
  __shared__ double sd[16];
  __shared__ int taken;
  block_merge_clear<kModSlots>(tk, tv);
  if (threadIdx.x == 0) taken = 0;
  const int64_t nch = ceil_div(nnz, (int64_t)kChunk), per = ceil_div(nch, (int64_t)gridDim.x);
  const int64_t b1 = min(nch, per * (blockIdx.x + 1));
  double sig = 0.0;
  for (int64_t b = per * blockIdx.x; b < b1; ++b) {
    const int64_t q0 = b * kChunk;
    const int len = (int)min((int64_t)kChunk, nnz - q0);
    __syncthreads();
    chunk_rows<kChunk>(off, q0, len, crow[b], crow[b + 1], rowof, sh);
    // a wavefront's round is 64 entries in row order, whose row sums are taken
    // with lane moves: one addition in LDS a row and round
    constexpr int PER = kChunk / 256;
    int j[PER], r[PER];
    float x[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int t = threadIdx.x + k * 256;
      j[k] = 0;
      r[k] = -1;
      x[k] = 0.0f;
      if (t < len) {
        j[k] = idx[q0 + t];
        x[k] = w[q0 + t];
        r[k] = rowof[t];
      }
    }
    int c[PER], cr[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      c[k] = 0;
      cr[k] = -1;
      if (r[k] >= 0) {
        c[k] = C[j[k]];
        cr[k] = C[r[k]];
      }
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if (c[k] == cr[k]) sig += (double)x[k];
      const int before = lane_before(r[k]);  // by all lanes, not behind the ||
      int f = lane() == 0 || before != r[k];
      const unsigned long long starts = __ballot(f);
      double row = (double)x[k];
      wave_seg_scan(row, f);
      const bool last = lane() == kWave - 1 || ((starts >> (lane() + 1)) & 1ull);
      if (!last || r[k] < 0) continue;
      uint32_t h = mix32((uint32_t)cr[k]);
      int probe = 0;
      for (; probe < kModProbes; ++probe, ++h) {
        const int old = atomicCAS(&tk[h & (kModSlots - 1)], kEmpty, cr[k]);
        if (old == kEmpty) atomicAdd(&taken, 1);
        if (old == kEmpty || old == cr[k]) break;
      }
      if (probe < kModProbes) atomicAdd(&tv[h & (kModSlots - 1)], row);
      else unsafeAtomicAdd(&S[cr[k]], row);
    }
    __syncthreads();
    if (taken > kModSlots / 2) {
      block_merge_flush<kModSlots>(tk, tv, S);
      if (threadIdx.x == 0) taken = 0;
    }
  }
  sig = block_sum(sig, sd);
  if (threadIdx.x == 0 && sig != 0.0) unsafeAtomicAdd(&acc[0], sig);
  block_merge_flush<kModSlots>(tk, tv, S);
}

static int mod_blocks(int64_t nnz) { return (int)std::min<int64_t>(kModBlocks, ceil_div(nnz, (int64_t)kChunk)); }

// Internal weight only (acc[0] += sum of entries inside a community): used
// when Sigma and 2m are already known.  W: float for a stored graph, double
// for the FP64 weights of an aggregated level.
template <class W>
__global__ __launch_bounds__(256) void k_mod_intra(const int64_t *off, const int32_t *idx, const W *w,
                                                   const int32_t *crow, int64_t nnz, const int32_t *C,
                                                   double *acc) {
  __shared__ int rowof[kChunk];
  __shared__ int sh[16];
  __shared__ double sd[16];
  const int64_t nch = ceil_div(nnz, (int64_t)kChunk);
  double sig = 0.0;
  for (int64_t b = blockIdx.x; b < nch; b += gridDim.x) {
    const int64_t q0 = b * kChunk;
    const int len = (int)min((int64_t)kChunk, nnz - q0);
    __syncthreads();
    chunk_rows<kChunk>(off, q0, len, crow[b], crow[b + 1], rowof, sh);
    // loads in two rounds, each issued together: ids, weights and row ids;
    // then both communities
    constexpr int PER = kChunk / 256;
    int j[PER], r[PER];
    W x[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int t = threadIdx.x + k * 256;
      j[k] = 0;
      r[k] = 0;
      x[k] = W(0);
      if (t < len) {
        j[k] = idx[q0 + t];
        x[k] = w[q0 + t];
        r[k] = rowof[t];
      }
    }
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (threadIdx.x + k * 256 < len && C[j[k]] == C[r[k]]) sig += (double)x[k];
  }
  sig = block_sum(sig, sd);
  if (threadIdx.x == 0 && sig != 0.0) unsafeAtomicAdd(&acc[0], sig);
}
void modularity_intra(const int64_t *off, const int32_t *idx, const float *w, const int32_t *crow, int64_t nnz,
                      const int32_t *C, double *acc, hipStream_t s) {
  if (nnz > 0)
    hipLaunchKernelGGL(k_mod_intra<float>, mod_blocks(nnz), 256, 0, s, off, idx, w, crow, nnz, C, acc);
}
void modularity_intra64(const int64_t *off, const int32_t *idx, const double *w, const int32_t *crow, int64_t nnz,
                        const int32_t *C, double *acc, hipStream_t s) {
  if (nnz > 0)
    hipLaunchKernelGGL(k_mod_intra<double>, mod_blocks(nnz), 256, 0, s, off, idx, w, crow, nnz, C, acc);
}

__global__ void k_scatter_labels(const int32_t *to, const int32_t *val, int64_t n, int32_t *out) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
    out[to[v]] = val[v];
}
void scatter_labels(const int32_t *to, const int32_t *val, int64_t n, int32_t *out, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_scatter_labels, flat_grid(n), 256, 0, s, to, val, n, out);
}

void modularity_edges(const int64_t *off, const int32_t *idx, const float *w, const int32_t *crow,
                      int64_t n, int64_t nnz, const int32_t *C, double *acc, double *S, hipStream_t s) {
  (void)n;
  if (nnz > 0) hipLaunchKernelGGL(k_mod_edges, mod_blocks(nnz), 256, 0, s, off, idx, w, crow, nnz, C, acc, S);
}

__global__ __launch_bounds__(256) void k_mod_comm(const double *S, int64_t n, double *acc) {
  __shared__ double sd[16];
  double t = 0.0;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (int64_t)gridDim.x * blockDim.x) t += S[c];
  t = block_sum(t, sd);
  if (threadIdx.x == 0 && t != 0.0) unsafeAtomicAdd(&acc[1], t);
}
void modularity_comm(const double *S, int64_t n, double *acc, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_mod_comm, flat_grid(n, 256, 512), 256, 0, s, S, n, acc);
}

__global__ __launch_bounds__(256) void k_mod_comm_sq(const double *S, int64_t n, double M2, double *acc) {
  __shared__ double sd[16];
  double t = 0.0;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n; c += (int64_t)gridDim.x * blockDim.x) {
    const double a = S[c] / M2;
    t += a * a;
  }
  t = block_sum(t, sd);
  if (threadIdx.x == 0 && t != 0.0) unsafeAtomicAdd(&acc[2], t);
}
void modularity_comm_sq(const double *S, int64_t n, double M2, double *acc, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_mod_comm_sq, flat_grid(n, 256, 512), 256, 0, s, S, n, M2, acc);
}

}  // namespace lk
