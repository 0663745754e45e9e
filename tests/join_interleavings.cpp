// Every interleaving of the refinement joins of the vertices of a small graph
// (refine_join.hpp, each operation on shared memory one step).  A vertex reads
// its neighbours' labels one after another, chooses any of the communities it
// has seen (every choice is explored), joins, and looks again up to TRIES times
// when the target had emptied.  When all have ended, every community must be
// connected, hold its representative, and have its members' weight as total.
// Prints the number of final states; "bad" lines and exit status 1 otherwise.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <string>
#include <unordered_set>
#include <utility>
#include <vector>

#include "refine_join.hpp"

using Log = std::vector<double>;  // results of a vertex's steps so far
struct State {
  std::vector<double> sig;
  std::vector<int> label;
  std::vector<Log> log;
  std::vector<char> done;
};
struct Stop {};

int n;
std::vector<std::vector<int>> adj;
std::vector<double> K;
int tries;

// Replays a vertex up to its next step and takes that one.
struct Run {
  State &s;
  int v;
  int choice;      // of the next step, if it is a choice
  int options = 0;  // of the next step, if it is a choice (0: it is not)
  size_t at = 0;
  bool stepped = false;
  template <class F>
  double step(F f) {
    Log &l = s.log[v];
    if (at < l.size()) return l[at++];
    if (stepped) throw Stop{};
    stepped = true;
    l.push_back(f());
    return l[at++];
  }
  int choose(int k) {
    Log &l = s.log[v];
    if (at < l.size()) return (int)l[at++];
    if (stepped) throw Stop{};
    options = k;
    if (choice >= k) throw Stop{};
    stepped = true;
    l.push_back(choice);
    return (int)l[at++];
  }
  double load(int c) { return step([&] { return s.sig[c]; }); }
  double swap(int c, double from, double to) {
    return step([&] {
      const double old = s.sig[c];
      if (old == from) s.sig[c] = to;
      return old;
    });
  }
  void store(int c, double x) {
    step([&] { return s.sig[c] = x; });
  }
  void add(int c, double x) {
    step([&] { return s.sig[c] += x; });
  }
};

void vertex(Run &r) {
  const int v = r.v;
  if (r.load(v) != K[v]) return;  // not isolated
  for (int t = 0; t < tries; ++t) {
    std::vector<int> seen;
    std::set<int> to;
    for (int u : adj[v]) {
      seen.push_back((int)r.step([&] { return (double)r.s.label[u]; }));
      if (seen.back() != v) to.insert(seen.back());
    }
    const int c = r.choose((int)to.size() + 1);
    if (c == (int)to.size()) return;  // no gain is positive
    const int target = *std::next(to.begin(), c);
    bool held = false;
    for (size_t k = 0; k < seen.size(); ++k) held |= seen[k] == target && adj[v][k] != target;
    const lk::Join end = lk::join_singleton(r, v, K[v], target, K[target], held, false);
    if (end == lk::Join::kDone) r.step([&] { return (double)(r.s.label[v] = target); });
    if (end != lk::Join::kEmpty) return;
  }
}

std::string key(const State &s) {
  std::string k;
  for (double x : s.sig) k.append((const char *)&x, sizeof x);
  k.append((const char *)s.label.data(), sizeof(int) * s.label.size());
  for (auto &l : s.log) {
    k.push_back((char)l.size());
    for (double x : l) k.append((const char *)&x, sizeof x);
  }
  k.append(s.done.begin(), s.done.end());
  return k;
}

std::unordered_set<std::string> visited;
std::set<std::string> finals;
long bad = 0;

void finish(const State &s) {
  std::string why;
  std::vector<double> tot(n, 0.0);
  for (int v = 0; v < n; ++v) {
    tot[s.label[v]] += K[v];
    if (s.label[s.label[v]] != s.label[v]) why = "representative is elsewhere";
  }
  for (int v = 0; v < n; ++v)
    if (s.sig[v] != tot[v]) why = "total is not the members' weight";
  for (int c = 0; c < n; ++c) {
    std::vector<int> stack, in(n, 0);
    for (int v = 0; v < n && stack.empty(); ++v)
      if (s.label[v] == c) { stack.push_back(v); in[v] = 1; }
    while (!stack.empty()) {
      const int v = stack.back();
      stack.pop_back();
      for (int u : adj[v])
        if (s.label[u] == c && !in[u]) { in[u] = 1; stack.push_back(u); }
    }
    for (int v = 0; v < n; ++v)
      if (s.label[v] == c && !in[v]) why = "community is not connected";
  }
  std::string f;
  for (int v = 0; v < n; ++v) f += std::to_string(s.label[v]) + " ";
  finals.insert(f);
  if (!why.empty()) {
    if (bad++ < 5) std::printf("bad: %s, labels %s\n", why.c_str(), f.c_str());
  }
}

void explore(const State &s) {
  if (!visited.insert(key(s)).second) return;
  bool all = true;
  for (int v = 0; v < n; ++v) {
    if (s.done[v]) continue;
    all = false;
    for (int choice = 0;; ++choice) {
      State t = s;
      Run r{t, v, choice};
      bool over = false;
      try {
        vertex(r);
        over = true;
      } catch (Stop &) {
      }
      if (r.options && choice >= r.options) break;
      if (over) t.done[v] = 1;
      explore(t);
      if (!r.options) break;
    }
  }
  if (all) finish(s);
}

// argv: tries, vertices, then pairs of vertices
int main(int argc, char **argv) {
  tries = std::atoi(argv[1]);
  n = std::atoi(argv[2]);
  adj.resize(n);
  for (int k = 3; k + 1 < argc; k += 2) {
    const int u = std::atoi(argv[k]), v = std::atoi(argv[k + 1]);
    adj[u].push_back(v);
    adj[v].push_back(u);
  }
  State s;
  for (int v = 0; v < n; ++v) {
    K.push_back((double)(1 << v));  // sums of different sets differ
    s.label.push_back(v);
  }
  s.sig = K;
  s.log.resize(n);
  s.done.assign(n, 0);
  explore(s);
  std::printf("%zu states, %zu final labellings, %ld bad\n", visited.size(), finals.size(), bad);
  return bad != 0;
}
