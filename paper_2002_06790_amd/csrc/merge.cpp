// The merge program of a graph (host): a fixed instruction list, the same for
// every scenario, that computes the first-in-first-out replay whenever the
// order of most ops on their resource is the same in every scenario.
//
// Facts that hold in every scenario (durations >= 1, any gaps and delays).
// An op's arrival A is its finish plus its resource's output delay; its ready
// time is the largest arrival over its predecessors; a resource runs its ops
// in (ready time, compact id) key order.  So
//   - A(p) < A(q) when p is a predecessor of q, or when p comes before q in
//     key order on one resource (same delay, later finish), and transitively;
//   - key(v) < key(z) when every predecessor p of v has A(p) <= ready(z)
//     because p is a predecessor of z or A(p) < A(q) for a predecessor q of z,
//     and either the inequality is strict for every p or v has the lower id.
// Every resource's ops are split into chains whose key order is proved this
// way.  A resource with one chain has the same order in every scenario.  On
// the others one chain is the *spine* and the rest are *deferred*: which spine
// op a deferred op follows differs between scenarios.
//
// A cluster is a set of resources whose deferred ops feed each other, with
// one spine chain.  The program visits ops in one order shared by all
// scenarios; before it runs a visited op with key K it runs, per scenario and
// in key order, the cluster's deferred ops whose keys are below K.  This is
// exact when every other op of the cluster whose ready time is not known at
// that point has a key proved above K, and so has the next spine op.  Any op
// for which that can be proved is visited; one for which it cannot is
// deferred: a release instruction hands over its ready time once its
// predecessors' arrivals are known to the program, unless it is the partner of
// a deferred op (its one predecessor), whose run releases it (a chain's ops
// release those of another chain place by place, all of them or none).  A force
// instruction runs a cluster's deferred ops up to one of them in every
// scenario, so that its arrival is known to the program.  The builder emits an
// instruction only when its condition is proved, and gives up (the replay
// then uses the event list) when it can prove no next one.
#include <algorithm>
#include <map>
#include <numeric>
#include <vector>

#include "sim.hpp"

namespace mlsim {

namespace {

constexpr int kChainsPerRes = 4;   // more chains on one resource: no program
constexpr int kChainsMax = 256;    // more chains in all: no program
constexpr int kInsertScan = 64;    // places tried from a chain's end for one op
constexpr int64_t kWorkMax = 64 << 20;  // steps of the search for the chains, and of that for the program

struct Builder {
  int n, R;
  const std::vector<std::vector<int32_t>> &succ, &pred;
  const std::vector<int32_t> &res;

  // chains and the facts proved about arrivals
  int nch = 0, W = 0;                        // chains, row width of the tables below
  bool late = false;                         // an op came before one placed earlier
  int64_t work = 0;                          // table entries and predecessors looked at
  std::vector<std::vector<int32_t>> chain;   // ops in key order
  std::vector<std::vector<int32_t>> of_res;  // chains of each resource
  std::vector<int32_t> ch, pos;              // chain of an op, its place
  // per op and chain, the last op x of the chain with A(x) <= ready(op)
  // (rdy) and with A(x) < A(op) (arr); -1: none.  Rows by place in the order
  // the ops are looked at, and made as they are: a graph whose chains are soon
  // too many pays only for the rows so far.
  std::vector<int32_t> rdy, arr, row;

  Builder(int n_, int R_, const std::vector<std::vector<int32_t>> &s, const std::vector<std::vector<int32_t>> &p,
          const std::vector<int32_t> &r)
      : n(n_), R(R_), succ(s), pred(p), res(r) {}

  void raise(int32_t &x, int32_t y) const {  // x, y in one chain
    if (y >= 0 && (x < 0 || pos[y] > pos[x])) x = y;
  }
  void raise_all(int32_t *to, const int32_t *from) const {
    for (int c = 0; c < nch; ++c) raise(to[c], from[c]);
  }
  // (fresh: v's rows are still empty)
  void learn_ready(int v, bool fresh) {
    int32_t *r = &rdy[(size_t)row[v] * W];
    for (int32_t p : pred[v]) {
      const int32_t *a = &arr[(size_t)row[p] * W];
      if (fresh)
        std::copy_n(a, nch, r);
      else
        raise_all(r, a);
      fresh = false;
      raise(r[ch[p]], p);
    }
  }
  void learn_arrival(int v, bool fresh) {
    int32_t *a = &arr[(size_t)row[v] * W];
    if (fresh)
      std::copy_n(&rdy[(size_t)row[v] * W], nch, a);
    else
      raise_all(a, &rdy[(size_t)row[v] * W]);
    if (pos[v] > 0) {
      const int32_t t = chain[ch[v]][pos[v] - 1];
      if (pred[v].size() == 1 && pred[v][0] == t) return;  // known with the ready time
      raise_all(a, &arr[(size_t)row[t] * W]);
      raise(a[ch[t]], t);
    }
  }
  // key(v) < key(z) in every scenario
  bool before(int v, int z) const {
    if (v == z) return false;
    if (pred[v].empty() && pred[z].empty()) return v < z;
    if (pred[z].empty()) return false;
    if (ch[v] >= 0 && ch[v] == ch[z]) return pos[v] < pos[z];
    bool strict = true;
    const int32_t *r = &rdy[(size_t)row[z] * W];
    for (int32_t p : pred[v]) {
      const int32_t x = r[ch[p]];
      if (x < 0 || pos[p] > pos[x]) return false;
      if (p == x && std::binary_search(pred[z].begin(), pred[z].end(), p)) strict = false;
    }
    return strict || v < z;
  }

  bool place(int v) {  // into a chain of its resource
    auto &list = of_res[res[v]];
    for (int c : list) {
      auto &C = chain[c];
      int i = (int)C.size() - 1, scan = kInsertScan;
      for (; i >= 0 && scan > 0; --i, --scan) {
        if (before(C[i], v)) break;
        if (!before(v, C[i])) {
          scan = 0;
          break;
        }
      }
      if (scan == 0) continue;
      late = late || i + 1 < (int)C.size();
      C.insert(C.begin() + i + 1, v);
      ch[v] = c;
      for (int k = i + 1; k < (int)C.size(); ++k) pos[C[k]] = k;
      return true;
    }
    if ((int)list.size() >= kChainsPerRes || nch >= kChainsMax) return false;
    if (nch == W) widen();
    list.push_back(nch);
    chain.push_back({v});
    ch[v] = nch++;
    pos[v] = 0;
    return true;
  }

  void widen() {  // rows of twice the width
    const int wide = std::min(2 * W, kChainsMax);
    for (std::vector<int32_t> *t : {&rdy, &arr}) {
      const size_t rows = t->size() / W;
      std::vector<int32_t> x(rows * wide, -1);
      for (size_t i = 0; i < rows; ++i) std::copy_n(t->begin() + i * W, W, x.begin() + i * wide);
      t->swap(x);
    }
    W = wide;
  }

  bool chains(const std::vector<int32_t> &topo) {
    W = std::min(kChainsMax, 2 * R);  // (a device's own ops, and those that others release)
    nch = 0;
    late = false;
    work = 0;
    chain.clear();
    of_res.assign(R, {});
    ch.assign(n, -1);
    pos.assign(n, 0);
    row.assign(n, -1);
    rdy.clear();
    arr.clear();
    rdy.reserve((size_t)n * W);
    arr.reserve((size_t)n * W);
    int32_t rows = 0;
    for (int32_t v : topo) {
      row[v] = rows++;
      rdy.resize((size_t)rows * W, -1);
      arr.resize((size_t)rows * W, -1);
      learn_ready(v, true);
      work += (int64_t)pred[v].size() * (nch + kInsertScan);
      if (work > kWorkMax || !place(v)) return false;
      learn_arrival(v, true);
    }
    for (int32_t v : topo) {  // once more where an op was inserted into a chain late
      if (!late) break;
      learn_ready(v, false);
      learn_arrival(v, false);
    }
    return true;
  }
};

}  // namespace

namespace {
// the chains of a graph's ops; false: too many
bool find_chains(Builder &B, const std::vector<int32_t> &topo) {
  const int32_t n = B.n;
  if (n < 1 || n > kMergeMaxOps) return false;
  // ids are usually a topological order in which one device's ops follow one
  // another, which keeps its long chain whole
  bool ids = true;
  for (int32_t v = 0; v < n && ids; ++v)
    for (int32_t w : B.succ[v]) ids = ids && w > v;
  std::vector<int32_t> order(topo);
  if (ids) std::iota(order.begin(), order.end(), 0);
  return B.chains(order) || (ids && B.chains(topo));
}

bool build(const Builder &B, const std::vector<int32_t> &row_of, bool partners, MergeProgram &P) {
  P = MergeProgram{};
  const int32_t n = B.n, R = B.R;
  const std::vector<std::vector<int32_t>> &succ = B.succ, &pred = B.pred;
  const std::vector<int32_t> &res = B.res;

  // clusters: resources with several chains, united where a deferred op feeds
  // another one's; one spine chain each (the longest), and every resource
  // with one chain a cluster of its own without deferred ops
  std::vector<int32_t> uf(R);
  std::iota(uf.begin(), uf.end(), 0);
  auto root = [&](int32_t r) {
    while (uf[r] != r) r = uf[r] = uf[uf[r]];
    return r;
  };
  std::vector<int32_t> spine(R);  // per cluster root: its spine chain, -1 none
  std::vector<char> deferred(n);
  for (bool again = true; again;) {
    again = false;
    std::fill(spine.begin(), spine.end(), -1);
    for (int c = 0; c < B.nch; ++c) {
      int32_t &s = spine[root(res[B.chain[c][0]])];
      if (s < 0 || B.chain[c].size() > B.chain[s].size()) s = c;
    }
    for (int32_t v = 0; v < n; ++v) deferred[v] = B.ch[v] != spine[root(res[v])];
    for (int32_t v = 0; v < n; ++v)
      if (deferred[v])
        for (int32_t p : pred[v])
          if (deferred[p] && root(res[p]) != root(res[v])) {
            uf[root(res[p])] = root(res[v]);
            again = true;
          }
  }

  // cluster numbers (by lowest resource), their spines and other chains
  std::vector<int32_t> cl(R, -1), cspine;
  std::vector<std::vector<int32_t>> dchains;
  for (int32_t r = 0; r < R; ++r) {
    if (B.of_res[r].empty()) continue;
    const int32_t t = root(r);
    if (cl[t] < 0) {
      cl[t] = (int32_t)cspine.size();
      cspine.push_back(spine[t]);
      dchains.emplace_back();
    }
    for (int c : B.of_res[r])
      if (c != spine[t]) dchains[cl[t]].push_back(c);
  }
  const int32_t K = (int32_t)cspine.size();
  P.cluster.assign(K, MergeCluster{0, 0, -1});

  // Partners: a chain's ops each release one op of another chain of the
  // cluster.  A chain has at most one such follower, the one that waits for
  // most of its ops.
  std::vector<int32_t> partner(n, -1), leader(n, -1);
  if (partners)
    for (int32_t k = 0; k < K; ++k)
      for (int c : dchains[k]) {
        std::map<int32_t, std::vector<int32_t>> to;
        for (int32_t x : B.chain[c])
          for (int32_t y : succ[x])
            if (deferred[y] && pred[y].size() == 1 && B.ch[y] != c) to[B.ch[y]].push_back(y);
        const std::vector<int32_t> *most = nullptr;
        for (const auto &e : to)
          if (!most || e.second.size() > most->size()) most = &e.second;
        if (!most) continue;
        bool fresh = true;  // one leader per chain
        for (int32_t y : B.chain[B.ch[(*most)[0]]]) fresh = fresh && leader[y] < 0;
        if (!fresh) continue;
        for (int32_t y : *most)
          if (partner[pred[y][0]] < 0) {
            partner[pred[y][0]] = y;
            leader[y] = pred[y][0];
          }
      }

  // the program; operands are value numbers: ops, then maxima n, n + 1, ...
  enum { kOpen = 0, kVisited = 1, kReleased = 2, kFollows = 3 };
  std::vector<char> state(n, kOpen), known(n, 0);
  std::vector<int32_t> latest(K, -1);          // the op visited last in each cluster (-1: none, or a force came after)
  std::vector<char> defers(B.nch, 0);          // chains with a released op
  std::vector<size_t> at(K, 0), un(B.nch, 0);  // next spine op; first open op of each other chain
  int32_t values = n;
  auto emit = [&](int32_t kind, int32_t v, int32_t k) -> MergeIns & {
    MergeIns I{};
    I.kind = kind;
    I.row = v < 0 ? -1 : row_of[v];
    I.res = v < 0 ? 0 : res[v];
    I.out = -1;
    std::fill(I.p, I.p + 4, -1);
    I.cluster = k;
    I.x = I.id = std::max(v, 0);
    P.ins.push_back(I);
    return P.ins.back();
  };
  // Operands of op v: its predecessors, or, for more than four, the maximum
  // that the ops with these predecessors share (four at a time).
  struct Maximum {
    int32_t value;  // -1 until all are known
    size_t left;    // predecessors not yet known
  };
  std::map<std::vector<int32_t>, int32_t> set_of;
  std::vector<Maximum> sets;
  std::vector<std::vector<int32_t>> in_sets(n);
  std::vector<const std::vector<int32_t> *> members;
  for (int32_t v = 0; v < n; ++v)
    if (pred[v].size() > 4 && set_of.emplace(pred[v], (int32_t)sets.size()).second) {
      for (int32_t p : pred[v]) in_sets[p].push_back((int32_t)sets.size());
      sets.push_back({-1, pred[v].size()});
      members.push_back(&pred[v]);
    }
  auto learn = [&](int32_t v) {  // v's arrival is known to the program
    known[v] = 1;
    for (int32_t i : in_sets[v]) {
      if (--sets[i].left > 0) continue;
      std::vector<int32_t> w(*members[i]), up;
      for (; w.size() > 1; w.swap(up)) {
        up.clear();
        for (size_t a = 0; a < w.size(); a += 4) {
          MergeIns &I = emit(kMgMax, -1, -1);
          std::copy(w.begin() + a, w.begin() + std::min(a + 4, w.size()), I.p);
          I.out = values;
          up.push_back(values++);
        }
      }
      sets[i].value = w[0];
    }
  };
  auto operands = [&](int32_t v) {
    return pred[v].size() > 4 ? std::vector<int32_t>(1, sets[set_of[pred[v]]].value) : pred[v];
  };
  auto all_known = [&](int32_t v) {
    for (int32_t p : pred[v])
      if (!known[p]) return false;
    return true;
  };
  // an open op that only another open one can release comes after that one
  // (once that one has been released, or is itself released by a leader's run,
  // it may have run already)
  auto follows = [&](int32_t v) { return leader[v] >= 0 && state[leader[v]] == kOpen; };
  int64_t budget = kWorkMax;  // ops looked at; a graph that needs more gets no program
  auto first_open = [&](int c) -> int32_t {  // -1: none
    const auto &C = B.chain[c];
    --budget;
    while (un[c] < C.size() && state[C[un[c]]] != kOpen) ++un[c];
    for (size_t i = un[c]; i < C.size(); ++i, --budget)
      if (state[C[i]] == kOpen && !follows(C[i])) return C[i];
    return -1;
  };
  // v's key is below those of cluster k's next spine op and of every op whose
  // ready time some scenario may not know yet (later ones of a chain follow
  // its first)
  auto clear = [&](int32_t k, int32_t v) {
    const auto &S = B.chain[cspine[k]];
    if (at[k] < S.size() && S[at[k]] != v && !B.before(v, S[at[k]])) return false;
    for (int c : dchains[k]) {
      const int32_t z = first_open(c);
      if (z >= 0 && z != v && !B.before(v, z)) return false;
    }
    return true;
  };
  auto visit = [&](int32_t k, int32_t v) {
    const std::vector<int32_t> q = operands(v);
    // an operand that is the finish time of the op its resource ran last is
    // there as the resource's free time
    const bool after = pred[v].size() == 1 && latest[k] == pred[v][0] && res[pred[v][0]] == res[v];
    MergeIns &I = emit(kMgVisit, v, dchains[k].empty() ? -1 : k);
    for (size_t j = 0; j < q.size(); ++j) I.p[j] = q[j];
    I.out = v;
    I.local = 1;
    for (int32_t p : pred[v]) I.local = I.local && res[p] == res[v];
    I.next = after;
    state[v] = kVisited;
    latest[k] = v;
    learn(v);
  };
  // hands over the ready times of chain c (of cluster k) that are known, but
  // that no scenario-independent place fits; in the chain's order
  auto release = [&](int32_t k, int c, bool any) {
    bool done = false;
    for (int32_t z; (z = first_open(c)) >= 0 && B.pos[z] == (int32_t)un[c] && all_known(z) && (any || !clear(k, z));
         done = true) {
      defers[c] = 1;
      state[z] = kReleased;
      if (partner[z] >= 0) {
        emit(kMgLoad, partner[z], k);
        state[partner[z]] = kFollows;
      }
      const std::vector<int32_t> q = operands(z);
      MergeIns &I = emit(kMgRelease, z, k);
      for (size_t j = 0; j < q.size(); ++j) I.p[j] = q[j];
    }
    return done;
  };
  for (bool progress = true; progress;) {
    progress = false;
    if ((budget -= K) < 0) return false;
    for (int32_t k = 0; k < K; ++k) {  // everything that can be visited: spines first
      const auto &S = B.chain[cspine[k]];
      for (; at[k] < S.size() && all_known(S[at[k]]) && clear(k, S[at[k]]); progress = true) visit(k, S[at[k]++]);
    }
    for (int32_t k = 0; k < K; ++k)
      for (int c : dchains[k])
        for (int32_t z; (z = first_open(c)) >= 0 && all_known(z) && clear(k, z); progress = true) visit(k, z);
    if (progress) continue;
    // clusters that wait for a ready time: of chains that defer ops already,
    // and only if there are none of one more
    for (int32_t k = 0; k < K; ++k)
      for (int c : dchains[k])
        if (defers[c]) progress = release(k, c, false) || progress;
    for (int32_t k = 0; k < K && !progress; ++k)
      for (int c : dchains[k])
        if (!progress) progress = release(k, c, true);
    if (progress) continue;
    for (int32_t k = 0; k < K; ++k)  // deferred ops whose arrivals others wait for
      for (int c : dchains[k])
        for (int32_t x : B.chain[c]) {
          --budget;
          if (state[x] == kOpen) break;
          if (known[x]) continue;
          bool read = false;
          for (int32_t y : succ[x]) read = read || state[y] == kOpen;
          if (!read) continue;
          if (!clear(k, x)) break;
          emit(kMgForce, x, k).out = x;
          latest[k] = -1;
          learn(x);
          progress = true;
        }
  }
  for (int32_t v = 0; v < n; ++v)
    if (state[v] == kOpen) return false;

  // deferred chains: the released ops, and partners' chains in the same order
  std::vector<int32_t> dx(n, -1), mchain(B.nch, -1);
  for (int32_t k = 0; k < K; ++k) {
    P.cluster[k].beg = (int32_t)P.chain.size();
    for (int c : dchains[k]) {
      const int32_t beg = (int32_t)P.def.size();
      for (int32_t v : B.chain[c])
        if (state[v] != kVisited) {
          dx[v] = (int32_t)P.def.size();
          P.def.push_back({row_of[v], v, (int32_t)P.chain.size(), -1});
        }
      if ((int32_t)P.def.size() == beg) continue;
      mchain[c] = (int32_t)P.chain.size();
      P.chain.push_back({beg, res[B.chain[c][0]], -1, (int32_t)P.def.size() - beg, -1});
    }
    P.cluster[k].end = (int32_t)P.chain.size();
    if (P.cluster[k].end > P.cluster[k].beg) emit(kMgDrain, -1, k);
  }
  // a chain's ops release those of another place by place, or none of them does
  for (int32_t v = 0; v < n; ++v) {
    if (state[v] != kFollows) continue;
    P.def[dx[leader[v]]].partner = dx[v];
    P.chain[mchain[B.ch[leader[v]]]].follow = mchain[B.ch[v]];
    P.chain[mchain[B.ch[v]]].lead = mchain[B.ch[leader[v]]];
  }
  for (const MergeChain &C : P.chain) {
    if (C.lead >= 0 && &P.chain[P.chain[C.lead].follow] != &C) return false;
    if (C.follow < 0) continue;
    const MergeChain &D = P.chain[C.follow];
    if (D.len != C.len) return false;
    for (int32_t i = 0; i < C.len; ++i)
      if (P.def[C.beg + i].partner != D.beg + i) return false;
  }
  for (MergeIns &I : P.ins) {
    if (I.kind == kMgRelease || I.kind == kMgLoad || I.kind == kMgForce) I.x = dx[I.id];
    if (I.cluster >= 0 && P.cluster[I.cluster].beg == P.cluster[I.cluster].end) I.cluster = -1;
  }

  P.values = values;
  return (int32_t)P.chain.size() < 2048;
}
}  // namespace

// Slots: a resource's free time, a deferred chain's first ready time and
// duration (and its partner's, when there are any), a cluster's least ready
// time (its chain's own with one chain), 0, infinity, a slot nobody reads, then
// the values, each from its instruction to its last reader.  Without a device
// model a next reads no operand.
bool merge_slots(MergeProgram &P, int32_t R, bool device_model) {
  const int32_t NC = (int32_t)P.chain.size();
  bool aux = false;
  for (const MergeChain &c : P.chain) aux = aux || c.follow >= 0;
  P.head_slot = R;
  int32_t s = R + (aux ? 3 : 2) * NC;
  for (auto &k : P.cluster) k.min_slot = k.end - k.beg == 1 ? P.head_slot + k.beg : k.end > k.beg ? s++ : -1;
  P.zero_slot = s++;
  P.inf_slot = s++;
  P.sink_slot = s++;
  std::vector<int32_t> last(P.values, -1), slot(P.values, -1), pool;
  for (size_t i = 0; i < P.ins.size(); ++i)
    for (int32_t &p : P.ins[i].p) {
      if (P.ins[i].next && !device_model) p = -1;
      if (p >= 0) last[p] = (int32_t)i;
    }
  for (size_t i = 0; i < P.ins.size(); ++i) {
    MergeIns &I = P.ins[i];
    int32_t freed[4], nf = 0;
    for (int32_t &p : I.p) {
      if (p < 0) {
        p = P.zero_slot;
        continue;
      }
      const int32_t v = p;
      p = slot[v];
      if (last[v] == (int32_t)i) {
        last[v] = -1;
        freed[nf++] = slot[v];
      }
    }
    pool.insert(pool.end(), freed, freed + nf);
    if (I.out < 0 || last[I.out] < 0) {
      I.out = P.sink_slot;
      continue;
    }
    const int32_t v = I.out;
    if (pool.empty()) {
      slot[v] = s++;
    } else {
      slot[v] = pool.back();
      pool.pop_back();
    }
    I.out = slot[v];
  }
  P.slots = s;
  return s < kMergeMaxSlots;
}

// A deferred op of a cluster with three chains or more costs a search over
// the chains' first ready times, about 0.55 us and 0.3 us a chain, which few
// deferred ops hide: replays of 16384 scenarios by the program take 53 us where
// the event list takes 36 (19 ops, 9 of them deferred in one cluster of 5
// chains), 79 / 52 (23 ops, 12 in 7), 42 / 44 (24 ops, 7 in 3) and 50 / 77 (42
// ops, 4 in 3).  On 172 measured graphs of 1 to 250 ops (each by the mean over
// plain, device-model, generated and attribution calls) the faster one is taken
// on all but 4, where the other gains up to 20 %; the program on every graph
// would lose on 29, up to 1.54 times.  Deferred ops of one chain or two stay in
// registers: graphs of only such clusters are faster by the program throughout,
// from 1 to 12000 ops, 64 to 262144 scenarios and up to the 64 KB of LDS that a
// block may take (4.8 / 17.6 ms on ResNet-50, 16 workers, 58 KB, 16384
// scenarios; 9.8 / 21.9 ms at 65536).
bool merge_pays(const MergeProgram &P, int32_t n) {
  int64_t cost = 0;
  for (const MergeCluster &k : P.cluster)
    for (int32_t c = k.beg; c < k.end && k.end - k.beg > 2; ++c)
      cost += (int64_t)P.chain[c].len * (8 + k.end - k.beg);
  return cost < 4 * (int64_t)n;
}

bool build_merge(int32_t n, int32_t R, const std::vector<std::vector<int32_t>> &succ,
                 const std::vector<std::vector<int32_t>> &pred, const std::vector<int32_t> &res,
                 const std::vector<int32_t> &row_of, const std::vector<int32_t> &topo, MergeProgram &P) {
  P = MergeProgram{};
  Builder B(n, R, succ, pred, res);
  return find_chains(B, topo) && (build(B, row_of, true, P) || build(B, row_of, false, P));
}

}  // namespace mlsim
