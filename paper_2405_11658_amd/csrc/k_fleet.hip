// Fused many-graph engine (see fleet_kernels.hpp): one persistent launch in
// which each workgroup runs whole graph updates, one job after another.
#include "device.hpp"
#include "fleet_kernels.hpp"
#include "wave_move.hpp"

#pragma clang fp contract(off)

namespace lk {
namespace {

// Loads of words that other threads of the workgroup update with atomics
// (performed in L2): read past the CU's L1.
template <class V>
__device__ __forceinline__ V ldx(const V *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr unsigned long long kNoKey = ~0ull;

// Edges of a vertex that one wavefront visits from registers, and vertices
// whose edges it holds at a time.
constexpr int kWaveEdges = 256;
constexpr int kGroup = 2;

// Sums of weights are taken in an order that follows from the graph and the
// batch alone, not from the number of wavefronts or their timing, so that the
// last bits of K, Sigma and the aggregated weights are the same on every run
// and in every launch variant also where sums in 64 bits are rounded: passes
// over items are split into kParts ranges for any number of wavefronts (a
// divisor of kParts), and sums by community are added by one wavefront (one a
// community), in the items' order.
// 512 graphs of up to 30,000 vertices: 165 ms, as the wavefronts came 162.
constexpr int kParts = 8;

// LDS of one workgroup.
template <int T, int SLOTS>
struct FSh {
  static constexpr int W = T / kWave;
  // reductions and broadcasts
  double rd[W];
  int ri[W];
  long long rl[W];
  double partd[kParts];
  long long partl[kParts];
  int flag;
  int cnt;
  int wide;             // the sweep's next vertex for the whole workgroup
  // radix sort
  int hist[256];
  int wcnt[W][256];
  // neighbour-community table
  int tkeys[SLOTS];
  double tvals[SLOTS];
  int tlist[SLOTS];
  int tcnt;
  uint16_t mine[W][T];  // a wavefront's entries of a wide vertex's T
  // job state broadcast
  FleetJob job;
  FleetGraph g;
};

template <int T, int SLOTS>
struct Blk {
  using Sh = FSh<T, SLOTS>;
  static constexpr int W = T / kWave;

  static __device__ __forceinline__ int tid() { return (int)threadIdx.x; }
  static __device__ __forceinline__ int wid() { return (int)threadIdx.x / kWave; }

  static __device__ __forceinline__ double sum_d(double v, Sh &s) {
    v = wave_sum(v);
    __syncthreads();
    if (lane() == 0) s.rd[wid()] = v;
    __syncthreads();
    double t = 0.0;
    for (int k = 0; k < W; ++k) t += s.rd[k];
    __syncthreads();
    return t;
  }
  static __device__ __forceinline__ long long sum_l(long long v, Sh &s) {
    v = group_sum_ll<kWave>(v);
    __syncthreads();
    if (lane() == 0) s.rl[wid()] = v;
    __syncthreads();
    long long t = 0;
    for (int k = 0; k < W; ++k) t += s.rl[k];
    __syncthreads();
    return t;
  }
  static __device__ __forceinline__ int or_i(int v, Sh &s) {
    __syncthreads();
    if (tid() == 0) s.flag = 0;
    __syncthreads();
    if (v) atomicOr(&s.flag, v);
    __syncthreads();
    const int r = s.flag;
    __syncthreads();
    return r;
  }
  // best (larger gain, then smaller id) over the block; valid in all threads
  static __device__ __forceinline__ void argmax(double &g, int &c, Sh &s) {
    wave_argmax(g, c);
    __syncthreads();
    if (lane() == 0) {
      s.rd[wid()] = g;
      s.ri[wid()] = c;
    }
    __syncthreads();
    g = s.rd[0];
    c = s.ri[0];
    for (int k = 1; k < W; ++k)
      if (better(s.rd[k], s.ri[k], g, c)) { g = s.rd[k]; c = s.ri[k]; }
    __syncthreads();
  }
  // The items [lo, hi) of this wavefront when n items are split into W ranges
  // of whole tiles of 64.  Passes over a graph's entries give each wavefront
  // such a range, so that no barrier stands between its tiles: with one
  // barrier a tile the passes ran at the latency of a load per T items.
  static __device__ __forceinline__ int64_t range_lo(int64_t n) {
    const int64_t per = ((n + kWave - 1) / kWave + W - 1) / W * kWave;
    return min(n, per * wid());
  }
  static __device__ __forceinline__ int64_t range_hi(int64_t n) {
    const int64_t per = ((n + kWave - 1) / kWave + W - 1) / W * kWave;
    return min(n, per * (wid() + 1));
  }
  // The parts of n items (of whole tiles of 64 too), this wavefront's being
  // [kParts / W * wid(), kParts / W * (wid() + 1)).
  static constexpr int kOwnParts = kParts / W;
  static __device__ __forceinline__ int64_t part_lo(int64_t n, int p) {
    const int64_t per = ((n + kWave - 1) / kWave + kParts - 1) / kParts * kWave;
    return min(n, per * p);
  }
  // Sum of f(k) over k in [0, n), in every thread: each part by the lanes of
  // one wavefront, then the parts in order.
  template <class F>
  static __device__ __forceinline__ double ordered_sum(int64_t n, Sh &s, F f) {
    __syncthreads();
    for (int p = kOwnParts * wid(); p < kOwnParts * (wid() + 1); ++p) {
      double v = 0.0;
      for (int64_t k = part_lo(n, p) + lane(); k < part_lo(n, p + 1); k += kWave) v += f(k);
      v = wave_sum(v);
      if (lane() == 0) s.partd[p] = v;
    }
    __syncthreads();
    double t = 0.0;
    for (int p = 0; p < kParts; ++p) t += s.partd[p];
    __syncthreads();
    return t;
  }
  // add(k, get(k)) for k in [0, n) in order, by the calling wavefront: four
  // tiles' reads are issued together.
  template <class G, class A>
  static __device__ __forceinline__ void in_order(int64_t n, G get, A add) {
    constexpr int kAhead = 4;
    for (int64_t b = 0; b < n; b += kAhead * kWave) {
      decltype(get((int64_t)0)) x[kAhead];
#pragma unroll
      for (int q = 0; q < kAhead; ++q) x[q] = get(min(b + q * kWave + lane(), n - 1));
#pragma unroll
      for (int q = 0; q < kAhead; ++q)
        if (b + q * kWave + lane() < n) add(x[q]);
    }
  }
  // Sum of x (uniform in each wavefront) over the wavefronts before this one;
  // the total in *tot.
  static __device__ __forceinline__ long long before(long long x, long long *tot, Sh &s) {
    __syncthreads();
    if (lane() == 0) s.rl[wid()] = x;
    __syncthreads();
    long long pre = 0, all = 0;
    for (int k = 0; k < W; ++k) {
      if (k < wid()) pre += s.rl[k];
      all += s.rl[k];
    }
    *tot = all;
    return pre;
  }
  // out[k] = sum of in[0..k) for k in [0, n] (counts: below 2^31 in total);
  // returns the total.  in and out may be the same array.
  template <class I, class O>
  static __device__ __forceinline__ long long scan(const I *in, O *out, int64_t n, Sh &s) {
    const int64_t lo = range_lo(n), hi = range_hi(n);
    long long mine = 0;
    for (int64_t k = lo + lane(); k < hi; k += kWave) mine += (long long)ldx(&in[k]);
    long long tot;
    long long carry = before(group_sum_ll<kWave>(mine), &tot, s);
    for (int64_t b = lo; b < hi; b += kWave) {
      const int64_t k = b + lane();
      const int x = k < hi ? (int)ldx(&in[k]) : 0;
      int all;
      const int incl = wave_scan(x, &all);
      if (k < hi) out[k] = (O)(carry + (incl - x));
      carry += all;
    }
    if (tid() == 0) out[n] = (O)tot;
    __syncthreads();
    return tot;
  }

  // f(width, u, e0, e1, first, there) for every row u of a CSR, called by
  // `width` lanes that share the row's entries [e0, e1) (the calling lane's
  // first is `first`): 8 lanes for rows of up to 64 entries, a wavefront for
  // longer ones.  there: the lanes hold a row.  A wavefront a row, most rows
  // being of a few dozen entries, waited out three loads a row: copying 30000
  // rows 37 -> 5.7 ms, their modularity 40 -> 2.8 ms (8 rows at a time, and 8
  // wavefronts).
  template <class F>
  static __device__ __forceinline__ void rows(int64_t n, const int64_t *off, F f) {
    constexpr int kSub = 8;
    for (int64_t b = (int64_t)wid() * (kWave / kSub); b < n; b += (int64_t)W * (kWave / kSub)) {
      const int64_t u = b + lane() / kSub;
      int64_t e0 = 0, e1 = 0;
      if (u < n) {
        e0 = off[u];
        e1 = off[u + 1];
      }
      const bool wide = e1 - e0 > kWave;
      unsigned long long m = __ballot(wide && lane() % kSub == 0);
      f(Const<kSub>{}, u, e0, e1, e0 + lane() % kSub, u < n && !wide);
      for (; m; m &= m - 1) {
        const int l = __ffsll(m) - 1;
        const int64_t r0 = lane_value64(e0, l), r1 = lane_value64(e1, l);
        f(Const<kWave>{}, b + l / kSub, r0, r1, r0 + lane(), true);
      }
    }
  }

  // Stable LSD radix sort of (key, payload) pairs by the low `bits` key bits;
  // returns the buffer (0 / 1) holding the result.  Each wavefront counts and
  // then places the pairs of its own range, in order, with its own counters.
  static __device__ __forceinline__ int sort(unsigned long long *key[2], int32_t *pay[2], int64_t n, int bits, Sh &s) {
    const int64_t lo = range_lo(n), hi = range_hi(n);
    int *cnt = s.wcnt[wid()];
    int src = 0;
    for (int shift = 0; shift < bits; shift += 8) {
      const unsigned long long *ki = key[src];
      const int32_t *pi = pay[src];
      unsigned long long *ko = key[src ^ 1];
      int32_t *po = pay[src ^ 1];
      for (int d = lane(); d < 256; d += kWave) cnt[d] = 0;
      lds_fence();
      for (int64_t k = lo + lane(); k < hi; k += kWave) atomicAdd(&cnt[(int)((ki[k] >> shift) & 255ull)], 1);
      __syncthreads();
      // counts -> pairs of the digit in the wavefronts before; digit totals
      for (int d = tid(); d < 256; d += T) {
        int t = 0;
        for (int k = 0; k < W; ++k) {
          const int c = s.wcnt[k][d];
          s.wcnt[k][d] = t;
          t += c;
        }
        s.hist[d] = t;
      }
      __syncthreads();
      if (wid() == 0) {
        int c[4], all, sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          c[q] = s.hist[4 * lane() + q];
          sum += c[q];
        }
        int pre = wave_scan(sum, &all) - sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          s.hist[4 * lane() + q] = pre;
          pre += c[q];
        }
      }
      __syncthreads();
      for (int d = lane(); d < 256; d += kWave) cnt[d] += s.hist[d];
      lds_fence();
      // tiles of this range, the next one's pairs loaded ahead
      unsigned long long nkey = 0;
      int32_t npay = 0;
      if (lo + lane() < hi) {
        nkey = ki[lo + lane()];
        npay = pi[lo + lane()];
      }
      for (int64_t b = lo; b < hi; b += kWave) {
        const bool act = b + lane() < hi;
        const unsigned long long kk = nkey;
        const int32_t p = npay;
        const int64_t nx = b + kWave + lane();
        if (nx < hi) {
          nkey = ki[nx];
          npay = pi[nx];
        }
        const int dg = (int)((kk >> shift) & 255ull);
        // lanes of this wavefront with the same digit
        unsigned long long same = __ballot(act);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
          const unsigned long long on = __ballot(act && ((dg >> bit) & 1));
          same &= ((dg >> bit) & 1) ? on : ~on;
        }
        const unsigned long long below = (lane() == 0) ? 0ull : (~0ull >> (64 - lane()));
        const int rank = __popcll(same & below);
        if (act) {
          const int at = cnt[dg];
          ko[at + rank] = kk;
          po[at + rank] = p;
          lds_fence();
          if (rank == 0) cnt[dg] = at + __popcll(same);
        }
        lds_fence();
      }
      __syncthreads();
      src ^= 1;
    }
    return src;
  }
};

__device__ __forceinline__ int bits_for(unsigned long long top) {
  int b = 1;
  while (b < 64 && (top >> b) != 0) ++b;
  return b;
}

__device__ __forceinline__ int64_t lower_bound_u64(const unsigned long long *a, int64_t lo, int64_t hi,
                                                   unsigned long long x) {
  while (lo < hi) {
    const int64_t mid = lo + ((hi - lo) >> 1);
    if (a[mid] < x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Neighbouring-community table of one vertex (or community): the LDS table
// when the number of entries to insert is at most SLOTS/2, else the graph's
// dense global table (value per community id, touched ids listed).  Slots
// taken are listed, so reading and clearing cost the number of distinct keys.
template <int T, int SLOTS>
struct Tab {
  using Sh = FSh<T, SLOTS>;
  bool dense;
  double *dv;    // dense values
  int32_t *df;   // dense taken flags
  int32_t *dl;   // dense list

  __device__ __forceinline__ void add(Sh &s, int key, double x) const {
    if (dense) {
      unsafeAtomicAdd(&dv[key], x);
      if (atomicExch(&df[key], 1) == 0) dl[atomicAdd(&s.tcnt, 1)] = key;
      return;
    }
    uint32_t h = mix32((uint32_t)key) & (uint32_t)(SLOTS - 1);
    for (int probe = 0; probe < SLOTS; ++probe) {
      const int k = __atomic_load_n(&s.tkeys[h], __ATOMIC_RELAXED);
      if (k == key) { atomicAdd(&s.tvals[h], x); return; }
      if (k == kEmpty) {
        const int old = atomicCAS(&s.tkeys[h], kEmpty, key);
        if (old == kEmpty) {
          atomicAdd(&s.tvals[h], x);
          s.tlist[atomicAdd(&s.tcnt, 1)] = (int)h;
          return;
        }
        if (old == key) { atomicAdd(&s.tvals[h], x); return; }
      }
      h = (h + 1) & (uint32_t)(SLOTS - 1);
    }
  }
  // entry q < s.tcnt (after a barrier following the inserts)
  __device__ __forceinline__ void get(const Sh &s, int q, int &key, double &x) const {
    if (dense) {
      key = dl[q];
      x = ldx(&dv[key]);
    } else {
      const int h = s.tlist[q];
      key = s.tkeys[h];
      x = s.tvals[h];
    }
  }
  // the sum of a key (after a barrier following the inserts)
  __device__ __forceinline__ double find(const Sh &s, int key) const {
    if (dense) return ldx(&dv[key]);
    uint32_t h = mix32((uint32_t)key) & (uint32_t)(SLOTS - 1);
    for (int probe = 0; probe < SLOTS; ++probe) {
      const int k = s.tkeys[h];
      if (k == key) return s.tvals[h];
      if (k == kEmpty) return 0.0;
      h = (h + 1) & (uint32_t)(SLOTS - 1);
    }
    return 0.0;
  }
  // clears what was taken; ends with the table empty and a barrier
  __device__ __forceinline__ void clear(Sh &s) const {
    const int n = s.tcnt;
    for (int q = (int)threadIdx.x; q < n; q += T) {
      if (dense) {
        const int key = dl[q];
        dv[key] = 0.0;
        df[key] = 0;
      } else {
        const int h = s.tlist[q];
        s.tkeys[h] = kEmpty;
        s.tvals[h] = 0.0;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) s.tcnt = 0;
    __syncthreads();
  }
};

// Level graph of the pass loop.
struct FLevel {
  int64_t n, nnz;
  const int64_t *off;
  const int32_t *idx;
  const float *w;
};

template <int T, int SLOTS>
struct FleetRun {
  using Sh = FSh<T, SLOTS>;
  using B = Blk<T, SLOTS>;
  Sh &s;
  FleetGraph &g;
  const FleetJob &job;
  FleetResult *res;
  const FleetParams &prm;
  int br = 0;  // buffer of the sorted batch

  // of a vertex with `entries` entries in a level of n vertices
  __device__ __forceinline__ Tab<T, SLOTS> table(int64_t entries, int64_t n) const {
    Tab<T, SLOTS> t;
    t.dense = min(entries, n) > SLOTS / 2;
    t.dv = g.dense;
    t.df = g.tflag;
    t.dl = g.tlist;
    return t;
  }

  // ---------------- the serial sweeps ---------------------------------------
  // Vertices of up to kWaveEdges edges, by the first wavefront alone: from
  // vertex `pos` on, in ascending order, each one decided on the state that
  // the previous ones left.  Returns the first wider vertex that is to be
  // visited (the whole workgroup's: move_vertex, refine_vertex), or -1 at the
  // end of the level.  REFINE: the sweep of Alg. "leidenRefine".
  //
  // A visit is a chain of dependent steps and nothing else runs in the
  // workgroup, so the chain is what the sweep costs.  A tile of 64 vertices is
  // kept in registers, one per lane (row, community, K, Sigma of its
  // community), and the edges of the next kGroup candidates with their
  // communities and those communities' Sigma: three rounds of loads a group
  // instead of six a vertex.  A move is written to memory and into these
  // registers, so that each visit sees what memory holds.  Refinement of the
  // 20786 singletons of a graph of 29703 vertices: 79 -> 31 ms (3.8 -> 1.5 us
  // a vertex: 0.8 for the loads, 0.5 for the choice); its first local moving,
  // 12565 visits: 11.6 -> 5.3 ms.  Groups of 4 and 8 are no faster: what they
  // save of the loads they lose on what a move writes into their registers.
  // (Everything here is inlined: in a function of its own the tables are
  // reached by generic addresses, 1.7 times the time.)
  template <bool REFINE>
  __device__ __forceinline__ int sweep(const FLevel &L, int pos, bool use_rng, double M2, bool track, double &gsum, long long &moves) {
    const int64_t *off = L.off;
    const int32_t *idx = L.idx;
    const float *w = L.w;
    int32_t *Cl = g.Cl;
    const int32_t *CB = g.CB;
    double *Sl = g.Sl;
    const double *Kl = g.Kl;
    uint8_t *U = g.U, *dC = g.dC;
    const uint8_t *rng = g.rng;
    const int n = (int)L.n;
    for (int b0 = pos & ~(kWave - 1); b0 < n; b0 += kWave) {
      const int i = b0 + lane();
      bool cand = i < n && i >= pos;
      if (cand) cand = REFINE ? dC[CB[i]] != 0 : U[i] != 0;
      // positions the move sweep may visit
      unsigned long long may = ~0ull;
      if (!REFINE && use_rng) may = __ballot(i < n && rng[i]);
      unsigned long long pend = __ballot(cand) & may;
      if (!pend) continue;
      int64_t o = 0;
      int deg = 0, d = -1, cb = -1;
      double Ki = 0.0, Sd = 0.0;
      if (i < n) {
        o = off[i];
        deg = (int)min(off[i + 1] - o, (int64_t)INT_MAX);
        d = Cl[i];
        Ki = Kl[i];
        Sd = Sl[d];
        if (REFINE) cb = CB[i];
      }
      if (REFINE) pend &= __ballot(Sd == Ki);
      const unsigned long long one = __ballot(deg <= kWave);
      // Visits the next G candidates of at most NU wavefronts of edges.
      auto visits = [&](auto nu, auto ng) __attribute__((always_inline)) {
        constexpr int NU = decltype(nu)::value, G = decltype(ng)::value;
        int p[G];
        {
          unsigned long long m = pend;
          const unsigned long long wider = NU == 1 ? pend & ~one : 0;
          if (wider) m &= (wider & (0ull - wider)) - 1ull;
#pragma unroll
          for (int q = 0; q < G; ++q) {
            p[q] = m ? __ffsll(m) - 1 : -1;
            m &= m - 1;
          }
        }
        int j[G][NU], c[G][NU];
        float x[G][NU];
        double S[G][NU];
        bool ok[G][NU];  // refinement: the community's own vertex is in it
#pragma unroll
        for (int q = 0; q < G; ++q) {
          const int64_t e0 = p[q] >= 0 ? lane_value64(o, p[q]) : 0;
          const int dg = p[q] >= 0 ? lane_value(deg, p[q]) : 0;
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            j[q][u] = -1;
            x[q][u] = 0.0f;
            const int e = u * kWave + lane();
            if (e < dg) {
              j[q][u] = idx[e0 + e];
              x[q][u] = w[e0 + e];
            }
          }
        }
        // (each round's loads are issued for the whole group before the first
        // is used)
        int aux[G][NU];  // refinement: community bound of the neighbour, then the community's own vertex's community
#pragma unroll
        for (int q = 0; q < G; ++q)
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            if (j[q][u] == b0 + p[q]) j[q][u] = -1;  // self-loops do not count
            c[q][u] = kEmpty;
            aux[q][u] = 0;
            if (j[q][u] >= 0) {
              c[q][u] = Cl[j[q][u]];
              if (REFINE) aux[q][u] = CB[j[q][u]];
            }
          }
#pragma unroll
        for (int q = 0; q < G; ++q) {
          const int cbv = REFINE && p[q] >= 0 ? lane_value(cb, p[q]) : 0;
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            if (REFINE && aux[q][u] != cbv) {
              j[q][u] = -1;
              c[q][u] = kEmpty;
            }
            S[q][u] = 0.0;
            if (c[q][u] != kEmpty) {
              S[q][u] = Sl[c[q][u]];
              if (REFINE) aux[q][u] = Cl[c[q][u]];
            }
          }
        }
#pragma unroll
        for (int q = 0; q < G; ++q)
#pragma unroll
          for (int u = 0; u < NU; ++u) ok[q][u] = !REFINE || aux[q][u] == c[q][u];
        bool live = true;
#pragma unroll
        for (int q = 0; q < G; ++q) {
          if (p[q] < 0 || !live) continue;
          const unsigned long long bit = 1ull << p[q];
          // a vertex in between that a move has marked comes first
          if (pend & (bit - 1)) { live = false; continue; }
          if (!(pend & bit)) continue;  // joined since
          pend &= ~bit;
          const int v = b0 + p[q], dv = lane_value(d, p[q]);
          const double Kv = lane_value(Ki, p[q]), Sv = lane_value(Sd, p[q]);
          if (!REFINE && lane() == 0) U[v] = 0;
          double bg, bs;
          int bc;
          edge_move<NU, SLOTS>(s.tkeys, s.tvals, c[q], x[q], S[q], M2, dv, Kv, Sv, bg, bc, bs);
          if (bc == kNoComm) continue;
          if (REFINE) {
            bool gone = false;
#pragma unroll
            for (int u = 0; u < NU; ++u) gone |= c[q][u] == bc && !ok[q][u];
            if (__ballot(gone)) continue;
          }
          const double nd = REFINE ? 0.0 : Sv - Kv, nb = bs + Kv;
          if (lane() == 0) {
            Cl[v] = bc;
            Sl[dv] = nd;
            Sl[bc] = nb;
            if (!REFINE && track) {
              dC[dv] = 1;
              dC[bc] = 1;
            }
          }
          if (d == dv) Sd = nd;
          if (d == bc) Sd = nb;
          if (lane() == p[q]) {
            d = bc;
            Sd = nb;
          }
          if (REFINE) {
            pend &= __ballot(Sd == Ki);
          } else {
            gsum += bg;
            moves += 1;
            const unsigned long long later = p[q] < kWave - 1 ? ~0ull << (p[q] + 1) : 0ull;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
              if (j[q][u] >= 0) U[j[q][u]] = 1;
              const int t = j[q][u] - b0;
              for (unsigned long long r = __ballot(j[q][u] >= 0 && t >= 0 && t < kWave); r; r &= r - 1)
                pend |= (1ull << lane_value(t, __ffsll(r) - 1)) & may & later;
            }
          }
#pragma unroll
          for (int q2 = q + 1; q2 < G; ++q2)
#pragma unroll
            for (int u = 0; u < NU; ++u) {
              if (c[q2][u] == kEmpty) continue;
              if (c[q2][u] == dv) S[q2][u] = nd;
              if (c[q2][u] == bc) S[q2][u] = nb;
              if (REFINE && c[q2][u] == v) ok[q2][u] = false;
              if (j[q2][u] == v) {
                c[q2][u] = bc;
                S[q2][u] = nb;
                ok[q2][u] = true;
              }
            }
          lds_fence();
        }
      };
      while (pend) {
        const int p = __ffsll(pend) - 1;
        if ((one >> p) & 1ull) {
          visits(Const<1>{}, Const<kGroup>{});
        } else if (lane_value(deg, p) <= kWaveEdges) {
          visits(Const<kWaveEdges / kWave>{}, Const<1>{});
        } else {
          return b0 + p;
        }
      }
    }
    return -1;
  }

  // Weights of a wide vertex's edges by the neighbours' communities into the
  // table (REFINE: of the neighbours inside the bound cb); returns the weight
  // to d.  The workgroup loads T edges at a time and leaves them in LDS, where
  // each wavefront lists those of its communities and adds them in order: a
  // community's sum is one wavefront's.
  template <bool REFINE>
  __device__ __forceinline__ double table_row(const FLevel &L, const Tab<T, SLOTS> &t, int64_t e0, int64_t e1, int i,
                                              int d, int cb) {
    constexpr int W = T / kWave;
    static_assert(sizeof(s.wcnt) >= 2 * T * sizeof(int), "staging");
    int *sc = &s.wcnt[0][0];
    float *sx = (float *)(sc + T);
    const unsigned long long below = lane() == 0 ? 0ull : (~0ull >> (64 - lane()));
    for (int64_t b = e0; b < e1; b += T) {
      const int64_t e = b + B::tid();
      int c = kEmpty;
      float x = 0.0f;
      if (e < e1) {
        const int j = L.idx[e];
        if (j != i && (!REFINE || g.CB[j] == cb)) {
          c = g.Cl[j];
          x = L.w[e];
        }
      }
      sc[B::tid()] = c;
      sx[B::tid()] = x;
      __syncthreads();
      int cnt = 0;
#pragma unroll
      for (int r = 0; r < W; ++r) {
        const int k = r * kWave + lane();
        const int ck = sc[k];
        const bool mine = ck != kEmpty && (int)((mix32((uint32_t)ck) >> 16) % W) == B::wid();
        const unsigned long long m = __ballot(mine);
        if (mine) s.mine[B::wid()][cnt + __popcll(m & below)] = (uint16_t)k;
        cnt += __popcll(m);
      }
      lds_fence();
      for (int q = lane(); q < cnt; q += kWave) {
        const int k = s.mine[B::wid()][q];
        t.add(s, sc[k], (double)sx[k]);
      }
      __syncthreads();
    }
    return t.find(s, d);
  }

  // ---------------- Alg. "leidenMove" (serial sweep) -----------------------
  // One wider vertex: best community by Eq. 2, applied at once.  Returns true
  // if it moved, with its gain in *gain.
  __device__ __forceinline__ bool move_vertex(const FLevel &L, int i, double M2, bool track, double *gain) {
    const int64_t e0 = L.off[i], e1 = L.off[i + 1];
    const int d = g.Cl[i];
    const double Ki = g.Kl[i];
    const Tab<T, SLOTS> t = table(e1 - e0, L.n);
    const double b = table_row<false>(L, t, e0, e1, i, d, 0);
    const int nk = s.tcnt;
    const double Sd = g.Sl[d];
    double bg = 0.0;
    int bc = kNoComm;
    for (int q = B::tid(); q < nk; q += T) {
      int c;
      double a;
      t.get(s, q, c, a);
      if (c == d) continue;
      const double sc = move_score(M2, a, b, Ki, g.Sl[c], Sd);
      if (sc > 0.0 && better(sc, c, bg, bc)) { bg = sc; bc = c; }
    }
    B::argmax(bg, bc, s);
    t.clear(s);
    if (bc == kNoComm) return false;
    if (B::tid() == 0) {
      g.Cl[i] = bc;
      g.Sl[d] -= Ki;
      g.Sl[bc] += Ki;
      if (track) {
        g.dC[d] = 1;
        g.dC[bc] = 1;
      }
    }
    for (int64_t e = e0 + B::tid(); e < e1; e += T) {
      const int j = L.idx[e];
      if (j != i) g.U[j] = 1;
    }
    __syncthreads();
    *gain = bg;
    return true;
  }

  // Iterations of the local-moving phase; returns l (iterations executed).
  __device__ __forceinline__ int move(const FLevel &L, bool use_rng, double M2, double Tp, bool track, long long &moves_out) {
    int l = 0;
    long long moves = 0;
    for (int it = 0; it < prm.max_iter; ++it) {
      double gsum = 0.0;  // first wavefront: the moves' gains in visiting order
      for (int pos = 0;;) {
        if (B::wid() == 0) {
          const int v = sweep<false>(L, pos, use_rng, M2, track, gsum, moves);
          if (lane() == 0) {
            s.wide = v;
            if (v >= 0) g.U[v] = 0;
          }
        }
        __syncthreads();
        const int v = s.wide;
        if (v < 0) break;
        double bg;
        if (move_vertex(L, v, M2, track, &bg)) {
          gsum += bg;
          moves += 1;
        }
        pos = v + 1;
      }
      l = it + 1;
      if (B::tid() == 0) s.rd[0] = gsum;
      __syncthreads();
      const double gs = s.rd[0];
      __syncthreads();
      if (gs <= Tp) break;
    }
    moves_out = moves;
    return l;
  }

  // ---------------- Alg. "leidenRefine" (serial sweep) ---------------------
  __device__ __forceinline__ void refine_vertex(const FLevel &L, int i, double M2) {
    const int64_t e0 = L.off[i], e1 = L.off[i + 1];
    const int c = g.Cl[i];
    const int cb = g.CB[i];
    const double Ki = g.Kl[i];
    const Tab<T, SLOTS> t = table(e1 - e0, L.n);
    const double b = table_row<true>(L, t, e0, e1, i, c, cb);
    const int nk = s.tcnt;
    const double Sd = g.Sl[c];
    double bg = 0.0;
    int bc = kNoComm;
    for (int q = B::tid(); q < nk; q += T) {
      int cj;
      double a;
      t.get(s, q, cj, a);
      if (cj == c) continue;
      const double sc = move_score(M2, a, b, Ki, g.Sl[cj], Sd);
      if (sc > 0.0 && better(sc, cj, bg, bc)) { bg = sc; bc = cj; }
    }
    B::argmax(bg, bc, s);
    t.clear(s);
    if (bc == kNoComm) return;
    if (g.Cl[bc] != bc) return;
    if (B::tid() == 0) {
      g.Sl[c] = 0.0;
      g.Sl[bc] += Ki;
      g.Cl[i] = bc;
    }
    __syncthreads();
  }

  __device__ __forceinline__ void refine(const FLevel &L, double M2) {
    double gsum = 0.0;
    long long moves = 0;
    for (int pos = 0;;) {
      if (B::wid() == 0) {
        const int v = sweep<true>(L, pos, false, M2, false, gsum, moves);
        if (lane() == 0) s.wide = v;
      }
      __syncthreads();
      const int v = s.wide;
      if (v < 0) break;
      refine_vertex(L, v, M2);
      pos = v + 1;
    }
    __syncthreads();
  }

  // ---------------- Alg. "leidenSubsetRenumber", break, renumber -----------
  __device__ __forceinline__ void subset_renumber(int64_t n) {
    int32_t *rep = g.tmpi;
    for (int64_t c = B::tid(); c < n; c += T) rep[c] = INT_MAX;
    __syncthreads();
    for (int64_t i = B::tid(); i < n; i += T) atomicMin(&rep[g.Cl[i]], (int)i);
    __syncthreads();
    for (int64_t c = B::tid(); c < n; c += T) {
      g.S2[c] = 0.0;
      g.dC2[c] = 0;
    }
    __syncthreads();
    for (int64_t c = B::tid(); c < n; c += T) {
      const int r = ldx(&rep[c]);
      if (r != INT_MAX) {
        g.S2[r] = g.Sl[c];
        g.dC2[r] = g.dC[c];
      }
    }
    __syncthreads();
    for (int64_t i = B::tid(); i < n; i += T) g.Cl[i] = ldx(&rep[g.Cl[i]]);
    __syncthreads();
    if (B::tid() == 0) {
      double *ts = g.Sl;
      g.Sl = g.S2;
      g.S2 = ts;
      uint8_t *tc = g.dC;
      g.dC = g.dC2;
      g.dC2 = tc;
    }
    __syncthreads();
  }

  __device__ __forceinline__ void break_changed(int64_t n) {
    for (int64_t i = B::tid(); i < n; i += T) {
      if (g.dC[g.Cl[i]]) {
        g.Cl[i] = (int)i;
        g.Sl[i] = g.Kl[i];
      }
    }
    __syncthreads();
  }

  // Dense ascending relabel of lab[0..n) (labels < bound); returns the count.
  __device__ __forceinline__ int64_t renumber(int32_t *lab, int64_t n, int64_t bound) {
    int32_t *map = g.tmpi;
    for (int64_t c = B::tid(); c <= bound; c += T) map[c] = 0;
    __syncthreads();
    for (int64_t i = B::tid(); i < n; i += T) map[lab[i]] = 1;
    __syncthreads();
    const long long k = B::scan(map, map, bound, s);
    for (int64_t i = B::tid(); i < n; i += T) lab[i] = map[lab[i]];
    __syncthreads();
    return k;
  }

  // ---------------- Alg. "leidenAggregate" ---------------------------------
  // Super-vertex CSR of L under dense labels Cl (< nc) into level buffer ob,
  // K' (row sums of the stored float weights, in row order) into Kl.
  // Entries are sorted by (C[u], C[v]) with a stable sort: a pair's entries
  // in member-then-CSR order, summed in FP64.  The entries are read five times
  // (three passes of the sort, one to count the pairs, one to write them), each
  // time at the latency of a few loads a wavefront: all levels of an update of
  // 420k entries 160 -> 14 ms with 8 wavefronts.
  __device__ __forceinline__ FLevel aggregate(const FLevel &L, int64_t nc, int ob) {
    unsigned long long *key[2] = {g.akey[0], g.akey[1]};
    int32_t *pay[2] = {g.apay[0], g.apay[1]};
    const int32_t *Cl = g.Cl;
    const int kb = bits_for((unsigned long long)max(nc - 1, (int64_t)1));
    B::rows(L.n, L.off, [&](auto width, int64_t u, int64_t, int64_t e1, int64_t first, bool there) {
      if (!there) return;
      const unsigned long long cu = (unsigned long long)Cl[u] << kb;
      for (int64_t e = first; e < e1; e += decltype(width)::value) {
        key[0][e] = cu | (unsigned long long)Cl[L.idx[e]];
        pay[0][e] = (int32_t)e;
      }
    });
    __syncthreads();
    const int r = B::sort(key, pay, L.nnz, nc > 1 ? 2 * kb : 0, s);
    const unsigned long long *sk = key[r];
    const int32_t *sp = pay[r];
    // distinct keys of each part, and of those before it
    auto head = [&](int64_t t, int64_t hi) { return t < hi && (t == 0 || sk[t] != sk[t - 1]); };
    const int p0 = B::kOwnParts * B::wid(), p1 = p0 + B::kOwnParts;
    for (int p = p0; p < p1; ++p) {
      const int64_t hi = B::part_lo(L.nnz, p + 1);
      long long heads = 0;
      for (int64_t b = B::part_lo(L.nnz, p); b < hi; b += kWave) heads += __popcll(__ballot(head(b + lane(), hi)));
      if (lane() == 0) s.partl[p] = heads;
    }
    __syncthreads();
    auto heads_before = [&](int p) {
      int64_t k = 0;
      for (int q = 0; q < p; ++q) k += s.partl[q];
      return k;
    };
    const int64_t nu = heads_before(kParts);
    int64_t *off = g.loff[ob];
    int32_t *idx = g.lidx[ob];
    float *w = g.lw[ob];
    double *sum = g.asum;
    for (int64_t o = B::tid(); o < nu; o += T) sum[o] = 0.0;
    __syncthreads();
    // entries of the new rows: a part's entries of a key are summed in order;
    // the key that a part goes on with is left to the end
    for (int p = p0; p < p1; ++p) {
      const int64_t hi = B::part_lo(L.nnz, p + 1), first_own = heads_before(p);
      int64_t at = first_own;
      double lead = 0.0;
      for (int64_t b = B::part_lo(L.nnz, p); b < hi; b += kWave) {
        const int64_t t = b + lane();
        const bool in = t < hi;
        const unsigned long long kk = in ? sk[t] : 0ull;
        double x = in ? (double)L.w[sp[t]] : 0.0;
        const bool first = head(t, hi);
        const unsigned long long hm = __ballot(first);
        const int64_t o = at + __popcll(hm & (~0ull >> (63 - lane()))) - 1;
        if (first) {
          idx[o] = (int32_t)(kk & ((1ull << kb) - 1ull));
          const int64_t row = (int64_t)(kk >> kb);
          for (int64_t c = t == 0 ? 0 : (int64_t)(sk[t - 1] >> kb) + 1; c <= row; ++c) off[c] = o;
        }
        int f = first || lane() == 0;
        wave_seg_scan(x, f);
        const bool last = in && (lane() == kWave - 1 || t + 1 >= hi || ((hm >> (lane() + 1)) & 1ull));
        if (last) {
          if (o < first_own) lead += x;
          else unsafeAtomicAdd(&sum[o], x);
        }
        at += __popcll(hm);
      }
      lead = wave_sum(lead);
      if (lane() == 0) s.partd[p] = lead;
    }
    __syncthreads();
    if (B::tid() == 0)
      for (int p = 1; p < kParts; ++p)
        if (s.partd[p] != 0.0) unsafeAtomicAdd(&sum[heads_before(p) - 1], s.partd[p]);
    // rows after the last one with an entry
    const int64_t past = L.nnz > 0 ? (int64_t)(sk[L.nnz - 1] >> kb) + 1 : 0;
    for (int64_t c = past + B::tid(); c <= nc; c += T) off[c] = nu;
    __syncthreads();
    for (int64_t o = B::tid(); o < nu; o += T) w[o] = (float)ldx(&sum[o]);
    __syncthreads();
    for (int64_t c = B::tid(); c < nc; c += T) {
      double k = 0.0;
      for (int64_t e = off[c]; e < off[c + 1]; ++e) k += (double)w[e];
      g.Kl[c] = k;
    }
    __syncthreads();
    FLevel o{nc, nu, off, idx, w};
    return o;
  }

  // ---------------- the pass loop of Alg. "leiden" --------------------------
  // On entry Cl, Kl, Sl, dC, U, rng hold the level-0 state; result: dense
  // labels in g.C.
  __device__ __forceinline__ void core(const FLevel &L0, double M2, bool track) {
    const int64_t n0 = L0.n;
    for (int64_t i = B::tid(); i < n0; i += T) g.Ctop[i] = (int)i;
    if (prm.refine_variant == 1) {
      for (int64_t i = B::tid(); i < n0; i += T) g.dC[i] = 1;
      track = false;
    }
    __syncthreads();
    FLevel L = L0;
    int buf = 0;
    double tau = prm.tau0;
    int pass;
    for (pass = 0; pass < prm.max_passes; ++pass) {
      const int64_t nl = L.n;
      const double Tp = tau * M2 * M2 / 2.0;
      long long mv = 0;
      const int li = move(L, pass == 0, M2, Tp, track && pass == 0, mv);
      if (B::tid() == 0 && pass < 16) {
        res->move_iters[pass] = li;
        res->level_vertices[pass] = nl;
      }
      if (pass == 0) {
        long long ch = 0;
        for (int64_t c = B::tid(); c < nl; c += T) ch += g.dC[c] ? 1 : 0;
        ch = B::sum_l(ch, s);
        if (B::tid() == 0) {
          res->moves_pass0 = mv;
          res->changed = ch;
        }
      }
      subset_renumber(nl);
      for (int64_t i = B::tid(); i < nl; i += T) g.CB[i] = g.Cl[i];
      __syncthreads();
      break_changed(nl);
      refine(L, M2);
      if (B::tid() == 0) res->passes = pass + 1;
      if ((pass > 0 || prm.refine_variant == 2) && li <= 1) break;
      const int64_t nc = renumber(g.Cl, nl, nl);
      if (B::tid() == 0 && pass < 16) res->communities[pass] = nc;
      if (prm.agg_tol < 1.0 && (double)nc / (double)nl > prm.agg_tol) break;
      for (int64_t i = B::tid(); i < n0; i += T) g.Ctop[i] = g.Cl[g.Ctop[i]];
      __syncthreads();
      L = aggregate(L, nc, buf);
      buf ^= 1;
      for (int64_t i = B::tid(); i < nc; i += T) {
        g.Sl[i] = g.Kl[i];
        g.U[i] = 1;
        g.Cl[i] = (int)i;
        g.dC[i] = 1;
      }
      __syncthreads();
      tau = tau / prm.tol_drop;
    }
    if (pass >= prm.max_passes && B::tid() == 0) res->passes = prm.max_passes;
    for (int64_t i = B::tid(); i < n0; i += T) g.Ctop[i] = g.Cl[g.Ctop[i]];
    __syncthreads();
    renumber(g.Ctop, n0, n0);
    for (int64_t i = B::tid(); i < n0; i += T) g.C[i] = g.Ctop[i];
    __syncthreads();
  }

  // ---------------- graph update (Sec. 3.5, 5.1.4) ------------------------
  // Validates the batch against the current CSR and writes G^t into the other
  // buffer.  Returns the error bits (0: applied; the graph then switches).
  __device__ __forceinline__ int apply_batch() {
    const int64_t n = g.n;
    const int64_t nd = job.nd, ni = job.ni;
    const int64_t E = 2 * (nd + ni);
    const int cur = g.cur;
    const int64_t *off = g.off[cur];
    const int32_t *idx = g.idx[cur];
    const float *w = g.w[cur];
    unsigned long long *key[2] = {job.bkey[0], job.bkey[1]};
    int32_t *pay[2] = {job.bpay[0], job.bpay[1]};
    int err = 0;
    for (int64_t t = B::tid(); t < E; t += T) {
      const int64_t k = t >> 1;
      const bool del = k < nd;
      const int a = del ? job.du[k] : job.iu[k - nd];
      const int b = del ? job.dv[k] : job.iv[k - nd];
      const int u = (t & 1) ? b : a, v = (t & 1) ? a : b;
      float x = 0.0f;
      if (!del) {
        x = job.iw[k - nd];
        if (!(x > 0.0f) || !isfinite(x)) err |= 32;
      }
      if (u < 0 || u >= n || v < 0 || v >= n) {
        err |= 1;
        key[0][t] = kNoKey;
      } else {
        if (u == v) err |= 2;
        key[0][t] = (unsigned long long)u * (unsigned long long)n + (unsigned long long)v;
      }
      pay[0][t] = (int32_t)t;
      job.bw[t] = x;
    }
    err = B::or_i(err, s);
    if (err) return err;
    const unsigned long long top = (unsigned long long)n * (unsigned long long)n - 1ull;
    const int r = (E > 0) ? B::sort(key, pay, E, bits_for(top), s) : 0;
    br = r;
    const unsigned long long *sk = key[r];
    const int32_t *sp = pay[r];
    int32_t *pre = job.bpre;
    int32_t *seg0 = g.CB;    // first sorted position of each row's batch entries (-1: none)
    for (int64_t u = B::tid(); u < n; u += T) seg0[u] = -1;
    __syncthreads();
    for (int64_t t = B::tid(); t < E; t += T) {
      const unsigned long long kk = sk[t];
      const int u = (int)(kk / (unsigned long long)n), v = (int)(kk % (unsigned long long)n);
      const bool del = sp[t] < 2 * nd;
      if (t > 0 && sk[t - 1] == kk) err |= 4;
      if (t == 0 || sk[t - 1] / (unsigned long long)n != (unsigned long long)u) seg0[u] = (int)t;
      const int64_t p = lower_bound_i32(idx, off[u], off[u + 1], v);
      const bool found = p < off[u + 1] && idx[p] == v;
      if (del && !found) err |= 8;
      if (!del && found) err |= 16;
      if (del && found) job.bw[sp[t]] = w[p];
      pre[t] = del ? 1 : 0;
      atomicAdd(&g.rowd[u], del ? -1 : 1);
    }
    err = B::or_i(err, s);
    if (err) {
      for (int64_t u = B::tid(); u < n; u += T) g.rowd[u] = 0;
      __syncthreads();
      return err;
    }
    B::scan(pre, pre, E, s);
    // new offsets
    const int nb = cur ^ 1;
    int64_t *noff = g.off[nb];
    int32_t *nidx = g.idx[nb];
    float *nw = g.w[nb];
    for (int64_t u = B::tid(); u < n; u += T) {
      g.mcnt[u] = off[u + 1] - off[u] + ldx(&g.rowd[u]);
      g.rowd[u] = 0;
    }
    __syncthreads();
    const int64_t nnz_new = B::scan(g.mcnt, noff, n, s);
    // surviving old entries
    B::rows(n, off, [&](auto width, int64_t u, int64_t o0, int64_t o1, int64_t first, bool there) {
      if (!there) return;
      const int64_t to = noff[u];
      const int s0 = seg0[u];
      if (s0 < 0) {
        for (int64_t e = first; e < o1; e += decltype(width)::value) {
          nidx[to + (e - o0)] = idx[e];
          nw[to + (e - o0)] = w[e];
        }
        return;
      }
      const unsigned long long lo = (unsigned long long)u * (unsigned long long)n;
      const int64_t s1 = lower_bound_u64(sk, s0, E, lo + (unsigned long long)n);
      for (int64_t e = first; e < o1; e += decltype(width)::value) {
        const int v = idx[e];
        const int64_t p = lower_bound_u64(sk, s0, s1, lo + (unsigned long long)v);
        const int64_t dels = pre[p] - pre[s0];
        const int64_t inss = (p - s0) - dels;
        if (p < s1 && sk[p] == lo + (unsigned long long)v) continue;  // deleted (an insertion cannot match)
        const int64_t o = to + (e - o0) - dels + inss;
        nidx[o] = v;
        nw[o] = w[e];
      }
    });
    // inserted entries
    for (int64_t t = B::tid(); t < E; t += T) {
      if (sp[t] < 2 * nd) continue;
      const unsigned long long kk = sk[t];
      const int u = (int)(kk / (unsigned long long)n), v = (int)(kk % (unsigned long long)n);
      const int s0 = seg0[u];
      const int64_t olds = lower_bound_i32(idx, off[u], off[u + 1], v) - off[u];
      const int64_t dels = pre[t] - pre[s0];
      const int64_t inss = (t - s0) - dels;
      const int64_t o = noff[u] + olds - dels + inss;
      nidx[o] = v;
      nw[o] = job.bw[sp[t]];
    }
    __syncthreads();
    if (B::tid() == 0) {
      g.cur = nb;
      g.nnz = nnz_new;
    }
    __syncthreads();
    return 0;
  }

  // ---------------- marking, changedCommunities, updateWeights -------------
  // On the sorted batch (key / payload buffer r) and G^t; previous C, K,
  // Sigma, M2.  Leaves U = affected, rng = in range, dC = changed.
  __device__ __forceinline__ void mark(int mode, int r) {
    const int64_t n = g.n;
    const int64_t nd = job.nd, ni = job.ni;
    const int64_t E = 2 * (nd + ni);
    const unsigned long long *sk = job.bkey[r];
    const int32_t *sp = job.bpay[r];
    const int64_t *off = g.off[g.cur];
    const int32_t *idx = g.idx[g.cur];
    for (int64_t i = B::tid(); i < n; i += T) {
      g.U[i] = (mode == 1) ? 1 : 0;
      g.dC[i] = 0;
      g.dE[i] = 0;
      g.dCm[i] = 0;
    }
    __syncthreads();
    for (int64_t t = B::tid(); t < E; t += T) {
      const unsigned long long kk = sk[t];
      const int u = (int)(kk / (unsigned long long)n), v = (int)(kk % (unsigned long long)n);
      const bool del = sp[t] < 2 * nd;
      const bool same = g.C[u] == g.C[v];
      if (same) g.dC[g.C[u]] = 1;  // changedCommunities
      if (mode == 3 && ((del && same) || (!del && !same))) g.U[u] = 1;
      if (mode == 2 && del && same) {
        g.U[u] = 1;
        g.dE[u] = 1;
        g.dCm[g.C[v]] = 1;
      }
    }
    if (mode == 2) {
      // per unique source of insertions: the community of the best score
      // over its cross-community insertions (previous K, Sigma, M2)
      for (int64_t t = B::tid(); t < E; t += T) {
        const unsigned long long kk = sk[t];
        const int u = (int)(kk / (unsigned long long)n);
        if (t > 0 && sk[t - 1] / (unsigned long long)n == (unsigned long long)u) continue;
        int64_t t1 = t;
        while (t1 < E && sk[t1] / (unsigned long long)n == (unsigned long long)u) ++t1;
        const int cu = g.C[u];
        int best = -1;
        double bestg = 0.0;
        for (int64_t a = t; a < t1; ++a) {
          if (sp[a] < 2 * nd) continue;
          const int ca = g.C[(int)(sk[a] % (unsigned long long)n)];
          if (ca == cu) continue;
          bool seen = false;
          for (int64_t q = t; q < a && !seen; ++q)
            if (sp[q] >= 2 * nd && g.C[(int)(sk[q] % (unsigned long long)n)] == ca) seen = true;
          if (seen) continue;
          double h = 0.0;
          for (int64_t q = a; q < t1; ++q)
            if (sp[q] >= 2 * nd && g.C[(int)(sk[q] % (unsigned long long)n)] == ca)
              h += (double)job.bw[sp[q]];
          const double sc = (g.M2 * h) - (g.K[u] * g.Sig[ca]);
          if (best < 0 || sc > bestg || (sc == bestg && ca < best)) { best = ca; bestg = sc; }
        }
        if (best >= 0) {
          g.U[u] = 1;
          g.dE[u] = 1;
          g.dCm[best] = 1;
        }
      }
      __syncthreads();
      B::rows(n, off, [&](auto width, int64_t u, int64_t, int64_t e1, int64_t first, bool there) {
        if (!there || !g.dE[u]) return;
        for (int64_t e = first; e < e1; e += decltype(width)::value) g.U[idx[e]] = 1;
      });
      __syncthreads();
      for (int64_t i = B::tid(); i < n; i += T)
        if (g.dCm[g.C[i]]) g.U[i] = 1;
    }
    __syncthreads();
    for (int64_t i = B::tid(); i < n; i += T) g.rng[i] = (mode == 2) ? g.U[i] : 1;
    // updateWeights: K and Sigma of the previous membership, and 2m
    auto change = [&](int64_t t) { return sp[t] < 2 * nd ? -(double)job.bw[sp[t]] : (double)job.bw[sp[t]]; };
    if (B::wid() == 0) {
      struct Item {
        int u, c;
        double x;
      };
      B::in_order(
          E,
          [&](int64_t t) {
            const int u = (int)(sk[t] / (unsigned long long)n);
            return Item{u, g.C[u], change(t)};
          },
          [&](const Item &m) {
            unsafeAtomicAdd(&g.K[m.u], m.x);
            unsafeAtomicAdd(&g.Sig[m.c], m.x);
          });
    }
    const double dm = B::ordered_sum(E, s, change);
    if (B::tid() == 0) g.M2 = g.M2 + dm;
    __syncthreads();
    long long aff = 0;
    for (int64_t i = B::tid(); i < n; i += T) aff += g.U[i] ? 1 : 0;
    aff = B::sum_l(aff, s);
    if (B::tid() == 0) res->affected = aff;
    __syncthreads();
  }

  // Eq. 1 of the current graph and g.C (dense labels); also Sigma^t.
  __device__ __forceinline__ double modularity() {
    const int64_t n = g.n;
    const int64_t *off = g.off[g.cur];
    const int32_t *idx = g.idx[g.cur];
    const float *w = g.w[g.cur];
    double *sig = g.dense;   // holds 0 between uses
    double *inside = g.S2;   // of each row (free after the pass loop)
    for (int64_t c = B::tid(); c < n; c += T) g.Sig[c] = 0.0;
    const int32_t *C = g.C;
    B::rows(n, off, [&](auto width, int64_t u, int64_t, int64_t e1, int64_t first, bool there) {
      constexpr int N = decltype(width)::value;
      const int cu = there ? C[u] : 0;
      double in = 0.0;
      if (there)
        for (int64_t e = first; e < e1; e += N)
          if (C[idx[e]] == cu) in += (double)w[e];
      if constexpr (N == kWave) {
        in = wave_sum(in);
      } else {
        in += dpp_move<kDppXor1>(in);
        in += dpp_move<kDppXor2>(in);
        in += dpp_move<kDppHalfMirror>(in);
      }
      if (there && lane() % N == 0) inside[u] = in;
    });
    __syncthreads();
    // the communities' sums: two wavefronts where there are two
    struct Item {
      int c;
      double x;
    };
    if (B::wid() == 0)
      B::in_order(
          n, [&](int64_t i) { return Item{C[i], ldx(&g.K[i])}; },
          [&](const Item &m) { unsafeAtomicAdd(&g.Sig[m.c], m.x); });
    if (B::wid() == (B::W > 1 ? 1 : 0))
      B::in_order(
          n, [&](int64_t i) { return Item{C[i], ldx(&inside[i])}; },
          [&](const Item &m) {
            if (m.x != 0.0) unsafeAtomicAdd(&sig[m.c], m.x);
          });
    const double M2 = g.M2;
    const double q = B::ordered_sum(n, s, [&](int64_t c) {
      const double sc = ldx(&sig[c]);
      const double a = ldx(&g.Sig[c]) / M2;
      sig[c] = 0.0;
      return M2 > 0.0 ? sc / M2 - a * a : 0.0;
    });
    return M2 > 0.0 ? q : 0.0;
  }

  __device__ __forceinline__ void run() {
    const int mode = job.mode;
    const int64_t n = g.n;
    if (B::tid() == 0) {
      res->status = 0;
      res->err = 0;
      res->passes = 0;
      res->q = 0.0;
      res->affected = res->changed = res->moves_pass0 = 0;
      for (int k = 0; k < 16; ++k) {
        res->move_iters[k] = 0;
        res->level_vertices[k] = 0;
        res->communities[k] = 0;
      }
    }
    if (mode != 0 && !g.has_state) {
      if (B::tid() == 0) res->status = 3;
      return;
    }
    double M2;
    bool track;
    if (mode == 0) {
      const int64_t *off = g.off[g.cur];
      const float *w = g.w[g.cur];
      for (int64_t i = B::tid(); i < n; i += T) {
        double k = 0.0;
        for (int64_t e = off[i]; e < off[i + 1]; ++e) k += (double)w[e];
        g.K[i] = k;
        g.Kl[i] = k;
        g.Sl[i] = k;
        g.Cl[i] = (int)i;
        g.dC[i] = 1;
        g.U[i] = 1;
        g.rng[i] = 1;
      }
      const double m2 = B::ordered_sum(n, s, [&](int64_t i) { return g.K[i]; });
      if (B::tid() == 0) g.M2 = m2;
      __syncthreads();
      M2 = m2;
      track = false;
      if (B::tid() == 0) res->affected = n;
    } else {
      const int err = apply_batch();
      if (err) {
        if (B::tid() == 0) {
          res->status = 1;
          res->err = err;
        }
        return;
      }
      mark(mode, br);
      for (int64_t i = B::tid(); i < n; i += T) {
        g.Cl[i] = g.C[i];
        g.Kl[i] = ldx(&g.K[i]);
        g.Sl[i] = ldx(&g.Sig[i]);
      }
      __syncthreads();
      M2 = g.M2;
      track = true;
    }
    FLevel L0{n, g.nnz, g.off[g.cur], g.idx[g.cur], g.w[g.cur]};
    if (n > 0) core(L0, M2, track);
    const double q = modularity();
    if (job.out)
      for (int64_t i = B::tid(); i < n; i += T) job.out[i] = g.C[i];
    if (B::tid() == 0) {
      res->q = q;
      g.has_state = 1;
    }
    __syncthreads();
  }
};

// Four wavefronts a SIMD, so that two workgroups of 8 share a compute unit.
template <int T, int SLOTS>
__global__ __launch_bounds__(T, 4) void k_fleet(FleetLaunch a) {
  __shared__ FSh<T, SLOTS> s;
  for (int k = threadIdx.x; k < SLOTS; k += T) {
    s.tkeys[k] = kEmpty;
    s.tvals[k] = 0.0;
  }
  if (threadIdx.x == 0) s.tcnt = 0;
  __syncthreads();
  const int njobs = *a.njobs;
  for (;;) {
    if (threadIdx.x == 0) s.cnt = (int)atomicAdd(a.next, 1ull);
    __syncthreads();
    const int j = s.cnt;
    __syncthreads();
    if (j >= njobs) break;
    if (threadIdx.x == 0) {
      s.job = a.jobs[j];
      s.g = a.graphs[s.job.graph];
    }
    __syncthreads();
    // the graph record and the job stay in LDS: fields every thread reads,
    // written by thread 0 between barriers
    FleetRun<T, SLOTS> run{s, s.g, s.job, &a.results[j], a.prm};
    run.run();
    __syncthreads();
    if (threadIdx.x == 0) {
      FleetGraph *dst = &a.graphs[s.job.graph];
      dst->nnz = s.g.nnz;
      dst->cur = s.g.cur;
      dst->M2 = s.g.M2;
      dst->has_state = s.g.has_state;
    }
    __syncthreads();
  }
}

}  // namespace

hipError_t fleet_launch(const FleetLaunch &L, int variant, int blocks, hipStream_t s) {
  switch (variant) {
    case kFleetWide: hipLaunchKernelGGL((k_fleet<512, 2048>), blocks, 512, 0, s, L); break;
    case 0: hipLaunchKernelGGL((k_fleet<64, 512>), blocks, 64, 0, s, L); break;
    case 1: hipLaunchKernelGGL((k_fleet<128, 512>), blocks, 128, 0, s, L); break;
    case 2: hipLaunchKernelGGL((k_fleet<256, 512>), blocks, 256, 0, s, L); break;
    case 3: hipLaunchKernelGGL((k_fleet<64, 2048>), blocks, 64, 0, s, L); break;
    case 4: hipLaunchKernelGGL((k_fleet<128, 2048>), blocks, 128, 0, s, L); break;
    default: hipLaunchKernelGGL((k_fleet<256, 2048>), blocks, 256, 0, s, L); break;
  }
  return hipGetLastError();
}

}  // namespace lk
