// The move of one vertex by one wavefront with its edges in registers, shared
// by the asynchronous sweeps and the serial sweeps of the fused engine.
#pragma once
#include "device.hpp"

namespace lk {

// Orders the wavefront's LDS accesses only: LDS executes one wavefront's
// instructions in issue order, so a compiler barrier suffices for an LDS
// table that only this wavefront uses, and outstanding global stores (the
// previous vertex's move and marks) are not waited for.
__device__ __forceinline__ void lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Maximum over the wavefront (uniform).
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  x = max(x, (uint32_t)dpp_move<kDppXor1>((int)x));
  x = max(x, (uint32_t)dpp_move<kDppXor2>((int)x));
  x = max(x, (uint32_t)dpp_move<kDppHalfMirror>((int)x));
  x = max(x, (uint32_t)dpp_move<kDppMirror>((int)x));
  return max(max((uint32_t)lane_value((int)x, 0), (uint32_t)lane_value((int)x, 16)),
             max((uint32_t)lane_value((int)x, 32), (uint32_t)lane_value((int)x, 48)));
}

// Best positive-gain community other than d among NU edges per lane (community
// c, kEmpty for none; weight x; S the community's Sigma): summed by community
// in the LDS table, each slot scored and cleared by the lane that took it; the
// weight to d is summed apart.  Uniform results, as best_move.  Where few
// wavefronts run this chain of dependent steps bounds the sweep, so the table
// is used at its whole size (64 edges in 512 slots: hardly a second probe),
// and the argmax compares the bits of the positive gains, whose order is the
// gains': high words first, which nearly always decides.
template <int NU, int LDSCAP>
__device__ __forceinline__ void edge_move(int *keys, double *vals, const int (&c)[NU], const float (&x)[NU],
                                          const double (&S)[NU], double M2, int d, double Ki, double Sd, double &bg,
                                          int &bc, double &bs) {
  static_assert(NU * kWave < LDSCAP, "more slots than distinct communities");
  unsigned long long own[NU], any = 0, others = 0;
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    own[u] = __ballot(c[u] == d);
    any |= own[u];
    others |= __ballot(c[u] != kEmpty && c[u] != d);
  }
  bg = 0.0;
  bc = kNoComm;
  bs = 0.0;
  if (!others) return;
  double b = 0.0;
  if (any) {
    if (NU == 1) {
      // equal weights: their number times the weight is their exact sum
      const float x0 = __int_as_float(lane_value(__float_as_int(x[0]), __ffsll(own[0]) - 1));
      if (__ballot(c[0] == d && x[0] != x0)) b = wave_sum(c[0] == d ? (double)x[0] : 0.0);
      else b = (double)__popcll(own[0]) * (double)x0;
    } else {
#pragma unroll
      for (int u = 0; u < NU; ++u)
        if (c[u] == d) b += (double)x[u];
      b = wave_sum(b);
    }
  }
  constexpr uint32_t mask = LDSCAP - 1u;
  int slot[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    slot[u] = -1;
    if (c[u] == kEmpty || c[u] == d) continue;
    uint32_t h = ((uint32_t)c[u] * 0x9E3779B1u) >> (32 - __builtin_ctz(LDSCAP));
    for (uint32_t probe = 0; probe <= mask; ++probe) {
      const int old = atomicCAS(&keys[h], kEmpty, c[u]);
      if (old == kEmpty || old == c[u]) {
        atomicAdd(&vals[h], (double)x[u]);
        if (old == kEmpty) slot[u] = (int)h;
        break;
      }
      h = (h + 1) & mask;
    }
  }
  lds_fence();
  double g = 0.0, sg = 0.0;
  int cg = kNoComm;
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    if (slot[u] < 0) continue;
    const double q = move_score(M2, vals[slot[u]], b, Ki, S[u], Sd);
    keys[slot[u]] = kEmpty;
    vals[slot[u]] = 0.0;
    if (q > 0.0 && better(q, c[u], g, cg)) { g = q; cg = c[u]; sg = S[u]; }
  }
  lds_fence();
  unsigned long long win = __ballot(g > 0.0);
  if (!win) return;
  if (win & (win - 1)) {
    const unsigned long long bits = (unsigned long long)__double_as_longlong(g);
    const uint32_t hi = (uint32_t)(bits >> 32);
    const uint32_t mh = wave_max(hi);
    win = __ballot(hi == mh);
    if (win & (win - 1)) {
      const uint32_t ml = wave_max(hi == mh ? (uint32_t)bits : 0u);
      const bool top = hi == mh && (uint32_t)bits == ml;
      win = __ballot(top);
      if (win & (win - 1)) {
        // equal gains: the smallest community id (the reduction in all lanes,
        // not behind the && of the comparison)
        const uint32_t mc = ~wave_max(top ? ~(uint32_t)cg : 0u);
        win = __ballot(top && (uint32_t)cg == mc);
      }
    }
  }
  const int k = __ffsll(win) - 1;
  bg = lane_value(g, k);
  bc = lane_value(cg, k);
  bs = lane_value(sg, k);
}

template <int N>
struct Const {
  static constexpr int value = N;
};

}  // namespace lk
