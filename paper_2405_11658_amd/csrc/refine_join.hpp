// The join of one isolated vertex in the asynchronous refinement sweep, as the
// sequence of its operations on the community totals (Sigma) that other
// vertices' joins interleave with.  M makes them (atomics on the device); a
// host build explores their interleavings.
//
// Every vertex of a changed bound starts alone, in the community of its own
// id with Sigma = K.  The vertex claims its own community first (Sigma K -> 0)
// and adds itself to the target only then, so that an addition is never taken
// back and a target's total says what has happened to it:
//   K of its representative   the representative is there, alone;
//   0                         it has left, or its claim is being decided;
//   anything else             someone has joined it, so its representative's
//                             own claim can no longer succeed: it stays, and
//                             the community never empties.
// A lone target is therefore joined by a compare-and-swap from that K, which
// excludes the representative's claim; one with members by an addition.  (To
// add first and look at the total afterwards saves a round trip, but then a
// total that is neither K nor 0 may be an addition about to be taken back, and
// two vertices that share only a vertex that has left could end together.)
#pragma once

#if defined(__HIPCC__)
#define LK_JOIN __device__ __forceinline__
#else
#define LK_JOIN inline
#endif

namespace lk {

enum class Join {
  kDone,
  kTaken,  // someone has joined the vertex: it stays, for good
  kEmpty,  // the target's representative has left or is about to: look again
};

// Vertex of community c and weight kc, alone there, into community `to`, whose
// representative weighs kt.  held: `to` is known to have another member than
// its representative (on return also when its total has shown so).  later: a
// held target's addition is the caller's to make.
template <class M>
LK_JOIN Join join_singleton(M &m, int c, double kc, int to, double kt, bool &held, bool later) {
  double seen = held ? 0.0 : m.load(to);  // beside the claim: one round trip
  if (m.swap(c, kc, 0.0) != kc) return Join::kTaken;
  if (!held) {
    if (seen == kt) {
      seen = m.swap(to, kt, kt + kc);
      if (seen == kt) return Join::kDone;
    }
    if (seen == 0.0) {
      m.store(c, kc);  // nobody adds to an emptied community
      return Join::kEmpty;
    }
    held = true;
  }
  if (!later) m.add(to, kc);
  return Join::kDone;
}

}  // namespace lk
