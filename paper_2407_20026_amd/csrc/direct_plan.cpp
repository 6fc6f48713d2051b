// Plan of the sparse direct solver (host): nested dissection, fronts, work lists.
//
// Sec. 2.2.2 of the paper solves K u = f with direct solvers.  Here the node graph of K (one
// vertex per node, an edge where two nodes share an element) is split by vertex separators,
// recursively, and every separator is eliminated after the two parts that it separates.  A
// surface structure of n nodes then fills about n log n blocks and takes about n^1.5 operations.
//
// Splitting uses graph distances only.  Four landmarks far from each other (breadth-first
// search, farthest point next) give every node four distances; sums and differences of them are
// integer coordinates, and on a grid numbered in any way (members along grid lines, or quads)
// with its corners as landmarks they are the grid's own x and y.  A part is cut at the median of
// each candidate coordinate, the nodes of one side that touch the other form the separator, and
// the candidate with the smallest one is taken.
#include "direct_plan.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <exception>
#include <map>
#include <memory>
#include <system_error>
#include <thread>

namespace sso {
namespace {

// Parts of at most this many nodes are eliminated whole: 60 own DOFs, one panel.  8 took 2.0 ms
// instead of 2.2 on a 120 x 120 shell, but 0.43 instead of 0.40 on a 16 x 16 one and 11.0 instead of
// 10.8 on a 300 x 300 one; 14 fill more than direct_max_bytes allows small structures.
constexpr int LEAF_NODES = 10;
// Parts of fewer nodes keep the coordinates of the part they were cut from.
constexpr int LANDMARK_NODES = 120;
// A part that has fallen into more pieces than this (where a node with many spokes was taken out) is
// no longer cut but taken apart piece by piece: 300 ribs of 20 nodes under one crown have 12 levels
// instead of 152, 20,000 single members 15 instead of some 10,000.  A few pieces a cut
// still tells apart, one or two levels deeper at most.
constexpr int MAX_PIECES = 8;
// Small pieces share a front of at most this many nodes: fewer fronts, but a square of values each.
constexpr int PIECE_NODES = 4;
// After this many cuts in a row that each leave more than 7/8 of a part on one side, the rest is
// eliminated whole: nothing separates it (the members between every two of 300 nodes took 189
// levels).  A few nodes joined to all others are still taken out of a part one by one.
constexpr int MAX_POOR = 12;
// Parts of at least this many nodes hand one half to another thread, up to MAX_THREADS at once.
constexpr int MAX_THREADS = 8;
constexpr int THREAD_NODES = 4000;

// A part of the node graph, renumbered 0 .. n - 1 (no self edges).
struct Part {
  std::vector<int32_t> id;      // global node numbers
  std::vector<int32_t> rp, col;
  std::vector<int32_t> coord[4];
  int n() const { return (int)id.size(); }
};

struct Tree {                   // a front of the elimination: own nodes, then up to two subtrees
  std::vector<int32_t> own;
  std::unique_ptr<Tree> child[2];
  int level = 0;                // of the front: above its children's
  void raise() {
    for (const auto& c : child)
      if (c) level = std::max(level, c->level + 1);
  }
};

// Ends the build where nobody waits for the plan any more.
struct Stopped {};
void go_on(const std::atomic<bool>* stop) {
  if (stop && stop->load(std::memory_order_relaxed)) throw Stopped();
}

// Breadth-first distances from src (d: -1 everywhere on entry); queue: the nodes reached, in order.
void bfs(const Part& g, int src, std::vector<int32_t>& d, std::vector<int32_t>& queue) {
  queue.clear();
  queue.push_back(src);
  d[src] = 0;
  for (size_t h = 0; h < queue.size(); ++h) {
    const int v = queue[h], dv = d[v] + 1;
    for (int e = g.rp[v]; e < g.rp[v + 1]; ++e) {
      const int w = g.col[e];
      if (d[w] < 0) {
        d[w] = dv;
        queue.push_back(w);
      }
    }
  }
}

// The part's coordinates.  Landmark 0 is a node farthest from the first node, each next one the
// node farthest from those before (largest smallest distance, then largest sum of distances, so
// that on a grid the corners come before the middles of its edges); ties go to the lower degree,
// then to the lower number.  A node that a landmark does not reach counts as farther than any
// other (a part may fall into a few pieces).
void coordinates(Part& g, const std::atomic<bool>* stop) {
  const int n = g.n();
  std::vector<int32_t> dist[4], queue;
  queue.reserve(n);
  auto distances = [&](int src, std::vector<int32_t>& d) {
    go_on(stop);
    d.assign(n, -1);
    bfs(g, src, d, queue);
    if ((int)queue.size() < n)
      for (int32_t& v : d)
        if (v < 0) v = n;
  };
  auto farthest = [&](int k) {      // from landmarks 0 .. k - 1
    int best = 0;
    int64_t kb = -1;
    for (int v = 0; v < n; ++v) {
      int64_t lo = dist[0][v], sum = lo;
      for (int q = 1; q < k; ++q) {
        lo = std::min<int64_t>(lo, dist[q][v]);
        sum += dist[q][v];
      }
      const int64_t key = lo * (4 * (int64_t)n + 1) + sum;
      const int dv = g.rp[v + 1] - g.rp[v], db = g.rp[best + 1] - g.rp[best];
      if (key > kb || (key == kb && dv < db)) {
        best = v;
        kb = key;
      }
    }
    return best;
  };
  distances(0, dist[0]);
  const int first = farthest(1);
  distances(first, dist[0]);
  for (int k = 1; k < 4; ++k) distances(farthest(k), dist[k]);
  for (auto& c : g.coord) c.resize(n);
  for (int v = 0; v < n; ++v) {
    const int a = dist[0][v], b = dist[1][v], c = dist[2][v], d = dist[3][v];
    g.coord[0][v] = (a + b) - (c + d);
    g.coord[1][v] = (a + c) - (b + d);
    g.coord[2][v] = (a + d) - (b + c);
    g.coord[3][v] = a - b;
  }
}

// A cut of a part at a value of one coordinate (side 0: below at; by_list: the first half of the
// list instead) and its separator: the nodes of one side that touch the other.
struct Cut {
  int k = 0, at = 0;
  bool by_list = false;
  int from = 1;                 // the side that the separator is taken from
  int size = 0, n0 = 0, n1 = 0;
};

// The most balanced cut along coordinate k.  A distance changes by at most 1 along an edge, so a
// coordinate (sums and differences of at most four of them) by at most 4: only nodes that close
// to the cut can touch the other side, and only their edges are looked at.
Cut try_split(const Part& g, int k, std::vector<int32_t>& hist) {
  const int n = g.n();
  const std::vector<int32_t>& c = g.coord[k];
  int lo = c[0], hi = c[0];
  for (int v : c) {
    lo = v < lo ? v : lo;
    hi = v > hi ? v : hi;
  }
  Cut t;
  t.k = k;
  int left = n / 2;
  if (lo < hi) {
    hist.assign(hi - lo + 2, 0);
    for (int v : c) ++hist[v - lo + 1];
    int below = 0, best = n + 1;
    for (int q = 1; q <= hi - lo; ++q) {       // side 0: values below lo + q
      below += hist[q];
      const int off = std::abs(n - 2 * below);
      if (off < best) {
        best = off;
        left = below;
        t.at = lo + q;
      }
    }
  } else {
    t.by_list = true;
  }
  int touch[2] = {0, 0};
  for (int v = 0; v < n; ++v) {
    if (!t.by_list && (c[v] < t.at - 4 || c[v] > t.at + 3)) continue;
    const bool s = t.by_list ? v >= left : c[v] >= t.at;
    for (int e = g.rp[v]; e < g.rp[v + 1]; ++e) {
      const int w = g.col[e];
      if ((t.by_list ? w >= left : c[w] >= t.at) != s) {
        ++touch[s];
        break;
      }
    }
  }
  t.from = touch[1] < touch[0] || (touch[1] == touch[0] && left <= n - left) ? 1 : 0;
  t.size = touch[t.from];
  t.n0 = left - (t.from == 0 ? touch[0] : 0);
  t.n1 = n - left - (t.from == 1 ? touch[1] : 0);
  return t;
}

// Each node's side (0, 1) under the cut, 2 in the separator.
void take_split(const Part& g, const Cut& t, std::vector<int8_t>& side) {
  const int n = g.n();
  const std::vector<int32_t>& c = g.coord[t.k];
  auto of = [&](int v) { return (int8_t)(t.by_list ? v >= n / 2 : c[v] >= t.at); };
  for (int v = 0; v < n; ++v) side[v] = of(v);
  for (int v = 0; v < n; ++v) {
    if (side[v] != t.from) continue;
    if (!t.by_list && (c[v] < t.at - 4 || c[v] > t.at + 3)) continue;
    for (int e = g.rp[v]; e < g.rp[v + 1]; ++e)
      if (of(g.col[e]) != t.from) {
        side[v] = 2;
        break;
      }
  }
}

Part sub_part(const Part& g, const std::vector<int8_t>& side, int which, int n,
              std::vector<int32_t>& local) {
  Part s;
  s.id.reserve(n);
  const bool keep = g.n() >= LANDMARK_NODES ? n < LANDMARK_NODES : true;
  size_t edges = 0;
  for (int v = 0; v < g.n(); ++v) {
    local[v] = -1;
    if (side[v] != which) continue;
    local[v] = (int32_t)s.id.size();
    s.id.push_back(g.id[v]);
    edges += g.rp[v + 1] - g.rp[v];
  }
  s.rp.reserve(n + 1);
  s.col.reserve(edges);
  s.rp.push_back(0);
  for (int v = 0; v < g.n(); ++v) {
    if (side[v] != which) continue;
    for (int e = g.rp[v]; e < g.rp[v + 1]; ++e)
      if (local[g.col[e]] >= 0) s.col.push_back(local[g.col[e]]);
    s.rp.push_back((int32_t)s.col.size());
  }
  if (keep && n > LEAF_NODES)
    for (int k = 0; k < 4; ++k) {
      s.coord[k].reserve(n);
      for (int v = 0; v < g.n(); ++v)
        if (side[v] == which) s.coord[k].push_back(g.coord[k][v]);
    }
  return s;
}

// The connected pieces of a part, each with its nodes in the part's order; none if there are at
// most `few`.
std::vector<Part> pieces(const Part& g, int few) {
  const int n = g.n();
  std::vector<int32_t> piece(n, -1), list, local(n);   // list: the nodes, piece by piece
  std::vector<size_t> start;
  list.reserve(n);
  for (int v0 = 0; v0 < n; ++v0) {
    if (piece[v0] >= 0) continue;
    start.push_back(list.size());
    piece[v0] = 0;
    list.push_back(v0);
    for (size_t h = start.back(); h < list.size(); ++h)
      for (int e = g.rp[list[h]]; e < g.rp[list[h] + 1]; ++e)
        if (piece[g.col[e]] < 0) {
          piece[g.col[e]] = 0;
          list.push_back(g.col[e]);
        }
  }
  std::vector<Part> out;
  if (start.size() <= (size_t)few) return out;
  start.push_back(list.size());
  out.resize(start.size() - 1);
  for (size_t c = 0; c < out.size(); ++c) {
    const auto first = list.begin() + start[c], last = list.begin() + start[c + 1];
    std::sort(first, last);
    Part& p = out[c];
    p.id.reserve(last - first);
    p.rp.reserve(last - first + 1);
    p.rp.push_back(0);
    for (auto v = first; v != last; ++v) {
      local[*v] = (int32_t)p.id.size();
      p.id.push_back(g.id[*v]);
    }
    for (auto v = first; v != last; ++v) {
      for (int e = g.rp[*v]; e < g.rp[*v + 1]; ++e) p.col.push_back(local[g.col[e]]);
      p.rp.push_back((int32_t)p.col.size());
    }
    if (!g.coord[0].empty() && p.n() < LANDMARK_NODES && p.n() > LEAF_NODES)
      for (int k = 0; k < 4; ++k) {
        p.coord[k].reserve(last - first);
        for (auto v = first; v != last; ++v) p.coord[k].push_back(g.coord[k][*v]);
      }
  }
  return out;
}

std::unique_ptr<Tree> dissect(Part g, int threads, const std::atomic<bool>* stop, int poor = 0);

// Pieces that do not touch each other under fronts without own nodes: small ones together, up to
// PIECE_NODES in a front, and always the two lowest trees under one, so that no more levels come on
// top of the highest than their number makes necessary.
std::unique_ptr<Tree> dissect_pieces(std::vector<Part> parts, int threads,
                                     const std::atomic<bool>* stop) {
  std::vector<std::unique_ptr<Tree>> trees;
  Tree* leaf = nullptr;
  for (Part& p : parts) {
    if (p.n() > PIECE_NODES) {
      trees.push_back(dissect(std::move(p), threads, stop));
      continue;
    }
    if (!leaf || (int)leaf->own.size() + p.n() > PIECE_NODES) {
      trees.push_back(std::make_unique<Tree>());
      leaf = trees.back().get();
    }
    leaf->own.insert(leaf->own.end(), p.id.begin(), p.id.end());
  }
  std::multimap<int, std::unique_ptr<Tree>> by_level;    // equal ones in the order they came
  for (auto& t : trees) {
    const int h = t->level;
    by_level.emplace(h, std::move(t));
  }
  while (by_level.size() > 1) {
    auto t = std::make_unique<Tree>();
    for (auto& c : t->child) {
      c = std::move(by_level.begin()->second);
      by_level.erase(by_level.begin());
    }
    t->raise();
    const int h = t->level;
    by_level.emplace(h, std::move(t));
  }
  return std::move(by_level.begin()->second);
}

// threads: how many this call may use, itself included; poor: the cuts in a row before this one that
// left nearly all of a part on one side
std::unique_ptr<Tree> dissect(Part g, int threads, const std::atomic<bool>* stop, int poor) {
  const int n = g.n();
  if (n == 0) return nullptr;
  go_on(stop);
  auto t = std::make_unique<Tree>();
  if (n <= LEAF_NODES) {
    t->own = std::move(g.id);
    return t;
  }
  if (g.coord[0].empty()) coordinates(g, stop);
  std::vector<int8_t> side(n);
  std::vector<int32_t> hist;
  double cost = 0.0;
  Cut best;
  for (int k = 0; k < 4; ++k) {
    const Cut t = try_split(g, k, hist);
    const double balance = (double)std::max(t.n0, t.n1) / n;
    const double ck = t.size * (1.0 + 2.0 * std::max(0.0, balance - 0.55)) + 1e-6 * balance;
    if (k == 0 || ck < cost) {
      cost = ck;
      best = t;
    }
  }
  poor = 8 * std::max(best.n0, best.n1) > 7 * n ? poor + 1 : 0;
  if (best.size == 0 || poor > 0) {      // the cuts of a part that has fallen into pieces
    std::vector<Part> parts = pieces(g, MAX_PIECES);
    if (!parts.empty()) {
      g = Part();
      return dissect_pieces(std::move(parts), threads, stop);
    }
  }
  if (poor > MAX_POOR) {
    t->own = std::move(g.id);
    return t;
  }
  take_split(g, best, side);
  std::vector<int32_t>& local = hist;
  local.resize(n);
  for (int v = 0; v < n; ++v)
    if (side[v] == 2) t->own.push_back(g.id[v]);
  Part left = sub_part(g, side, 0, best.n0, local);
  Part right = sub_part(g, side, 1, best.n1, local);
  g = Part();
  if (threads > 1 && n >= THREAD_NODES) {
    std::exception_ptr err[2];
    auto half = [&](Part& part, int k, int th) {
      try {
        t->child[k] = dissect(std::move(part), th, stop, poor);
      } catch (...) {
        err[k] = std::current_exception();
      }
    };
    std::thread other;
    try {
      other = std::thread([&] { half(right, 1, threads / 2); });
    } catch (const std::system_error&) {   // no thread to be had: both halves here
    }
    half(left, 0, threads - threads / 2);
    if (other.joinable())
      other.join();
    else
      half(right, 1, 1);
    for (const std::exception_ptr& e : err)
      if (e) std::rethrow_exception(e);
  } else {
    t->child[0] = dissect(std::move(left), 1, stop, poor);
    t->child[1] = dissect(std::move(right), 1, stop, poor);
  }
  t->raise();
  return t;
}

struct Front0 {            // a front while the plan is built
  int own_off, own_cnt;    // own nodes: range of `order`
  int child[2];
  int level;
};

struct Dissection {
  std::vector<int32_t> order;       // nodes in elimination order
  std::vector<Front0> fronts;       // children before parents

  int flatten(const Tree* t) {
    if (!t) return -1;
    Front0 f;
    f.level = t->level;
    for (int c = 0; c < 2; ++c) f.child[c] = flatten(t->child[c].get());
    f.own_off = (int)order.size();
    f.own_cnt = (int)t->own.size();
    order.insert(order.end(), t->own.begin(), t->own.end());
    fronts.push_back(f);
    return (int)fronts.size() - 1;
  }

  void run(int n, const int32_t* rp, const int32_t* col, int threads,
           const std::atomic<bool>* stop) {
    Part g;
    g.id.resize(n);
    g.rp.reserve(n + 1);
    g.rp.push_back(0);
    for (int v = 0; v < n; ++v) {
      g.id[v] = v;
      for (int e = rp[v]; e < rp[v + 1]; ++e)
        if (col[e] != v) g.col.push_back(col[e]);
      g.rp.push_back((int32_t)g.col.size());
    }
    order.reserve(n);
    std::vector<Part> parts = pieces(g, 1);
    flatten((parts.empty() ? dissect(std::move(g), threads, stop)
                           : dissect_pieces(std::move(parts), threads, stop))
                .get());
  }
};

// Offsets for arrays that live from one level to a later one: first fit over the free gaps.
struct Gaps {
  std::map<int64_t, int64_t> gaps;   // offset -> length
  int64_t top = 0;
  int64_t take(int64_t len) {
    if (len == 0) return 0;
    for (auto it = gaps.begin(); it != gaps.end(); ++it)
      if (it->second >= len) {
        const int64_t off = it->first, rest = it->second - len;
        gaps.erase(it);
        if (rest) gaps[off + len] = rest;
        return off;
      }
    const int64_t off = top;
    top += len;
    return off;
  }
  void give(int64_t off, int64_t len) {
    if (len == 0) return;
    auto next = gaps.lower_bound(off);
    if (next != gaps.begin()) {
      auto prev = std::prev(next);
      if (prev->first + prev->second == off) {
        off = prev->first;
        len += prev->second;
        gaps.erase(prev);
      }
    }
    if (next != gaps.end() && next->first == off + len) {
      len += next->second;
      gaps.erase(next);
    }
    gaps[off] = len;
  }
};

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline int64_t even(int64_t v) { return (v + 1) & ~(int64_t)1; }

}  // namespace

bool build_direct_plan(int n, const int32_t* rp, const int32_t* col, double max_bytes,
                       DirectPlan& plan, const std::atomic<bool>* stop) try {
  plan = DirectPlan();
  plan.n_nodes = n;
  Dissection ds;
  ds.run(n, rp, col, MAX_THREADS, stop);
  const int nf = (int)ds.fronts.size();

  // level by level, children's order within a level kept
  std::vector<int> order(nf), rank(nf);
  for (int i = 0; i < nf; ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return ds.fronts[a].level < ds.fronts[b].level; });
  for (int i = 0; i < nf; ++i) rank[order[i]] = i;
  const int nl = ds.fronts.back().level + 1;

  // elimination position of each node: fronts children-first, own nodes in their order
  std::vector<int32_t> pos(n), owner(n);
  {
    int p = 0;
    for (int f = 0; f < nf; ++f)
      for (int k = 0; k < ds.fronts[f].own_cnt; ++k) {
        const int v = ds.order[ds.fronts[f].own_off + k];
        pos[v] = p++;
        owner[v] = f;
      }
  }

  // boundaries, children first: the children's boundary nodes and the own nodes' neighbours that
  // are eliminated later
  std::vector<std::vector<int32_t>> bnd(nf);
  std::vector<int32_t> stamp(n, -1);
  double bytes = 0.0;
  for (int f = 0; f < nf; ++f) {
    go_on(stop);
    const Front0& F = ds.fronts[f];
    std::vector<int32_t>& b = bnd[f];
    auto add = [&](int v) {
      if (stamp[v] != f && owner[v] > f) {
        stamp[v] = f;
        b.push_back(v);
      }
    };
    for (int c : F.child)
      if (c >= 0)
        for (int v : bnd[c]) add(v);
    for (int k = 0; k < F.own_cnt; ++k) {
      const int q = ds.order[F.own_off + k];
      for (int e = rp[q]; e < rp[q + 1]; ++e) add(col[e]);
    }
    std::sort(b.begin(), b.end(), [&](int x, int y) { return pos[x] < pos[y]; });
    const double s = 6.0 * F.own_cnt, t = 6.0 * (double)b.size();
    bytes += 8.0 * (s + t) * s;
    if (bytes > max_bytes || s > DIRECT_MAX_OWN || t > DIRECT_MAX_BOUNDARY) return false;
  }

  plan.fronts.resize(nf);
  plan.level_off.resize(nl);
  plan.level_np.assign(nl, 0);
  plan.level_own.assign(nl, 0);
  std::vector<std::vector<int>> by_level(nl);
  for (int i = 0; i < nf; ++i) by_level[ds.fronts[order[i]].level].push_back(i);

  size_t n_list = 0;
  for (int f = 0; f < nf; ++f) n_list += ds.fronts[f].own_cnt + bnd[f].size();
  plan.nodes.reserve(n_list);
  plan.maps.reserve(2 * n_list);
  std::vector<int32_t> local(n, -1);    // position of a node in the front at hand
  Gaps schur;
  int64_t b_off = 0;

  for (int h = 0; h < nl; ++h) {
    int64_t work = 0, again = 0, w = 0;
    for (int i : by_level[h]) {
      go_on(stop);
      const int f0 = order[i];
      const Front0& F = ds.fronts[f0];
      DirectFront& D = plan.fronts[i];
      const int ns = F.own_cnt, nb = (int)bnd[f0].size();
      D.ns6 = 6 * ns;
      D.nb6 = 6 * nb;
      D.np = ceil_div(D.ns6, DIRECT_NB);
      D.nt = D.np + ceil_div(D.nb6, DIRECT_NB);
      D.level = h;
      for (int c = 0; c < 2; ++c) D.child[c] = F.child[c] < 0 ? -1 : rank[F.child[c]];
      D.nodes_off = (int32_t)plan.nodes.size();
      plan.nodes.insert(plan.nodes.end(), ds.order.begin() + F.own_off,
                        ds.order.begin() + F.own_off + ns);
      plan.nodes.insert(plan.nodes.end(), bnd[f0].begin(), bnd[f0].end());
      const int32_t* list = plan.nodes.data() + D.nodes_off;
      const int cnt = ns + nb;
      // maps into the children's boundaries
      D.map_off = (int32_t)plan.maps.size();
      for (int c = 0; c < 2; ++c) {
        const int ch = F.child[c];
        if (ch >= 0)
          for (size_t k = 0; k < bnd[ch].size(); ++k) local[bnd[ch][k]] = (int32_t)k;
        for (int k = 0; k < cnt; ++k) plan.maps.push_back(ch >= 0 ? local[list[k]] : -1);
        if (ch >= 0)
          for (int v : bnd[ch]) local[v] = -1;
      }
      D.fact_off = plan.fact_len;
      plan.fact_len += even((int64_t)(D.ns6 + D.nb6) * D.ns6);
      D.work_off = work;
      work += even((int64_t)(D.ns6 + D.nb6) * D.ns6);
      // a single panel goes straight into the factor; two panels need one copy between
      D.again_off = again;
      D.w_off = w;
      if (D.np > 1) {
        again += even((int64_t)(D.ns6 + D.nb6) * D.ns6);
        w += (int64_t)DIRECT_NB * DIRECT_NB * (3 * D.nt - D.np);
      }
      for (int c = 0; c < 2; ++c)
        D.child_u[c] = D.child[c] < 0 ? 0 : plan.fronts[D.child[c]].u_off;
      D.u_off = schur.take(direct_tri(D.nb6));
      D.v_off = plan.v_len;
      plan.v_len += D.nb6;
      D.b_off = b_off;
      b_off += D.ns6;
      plan.level_np[h] = std::max(plan.level_np[h], D.np);
      plan.level_own[h] = std::max(plan.level_own[h], D.ns6);
    }
    plan.work_len = std::max(plan.work_len, work);
    plan.again_len = std::max(plan.again_len, again);
    plan.w_len = std::max(plan.w_len, w);
    for (int i : by_level[h])
      for (int c : plan.fronts[i].child)
        if (c >= 0) {
          const DirectFront& C = plan.fronts[c];
          schur.give(C.u_off, direct_tri(C.nb6));
        }
  }
  plan.u_len = even(schur.top);
  if (8.0 * (double)plan.values() > max_bytes) return false;

  // work lists
  std::vector<int32_t> start;
  std::vector<int32_t> lo, hi, fill;
  std::vector<DirectItem> assemble, spare;
  for (int h = 0; h < nl; ++h) {
    const int np = plan.level_np[h];
    plan.level_off[h] = (int32_t)plan.steps.size();
    plan.steps.resize(plan.steps.size() + STEP_PANEL + np + 1, DirectRange{0, 0});
    DirectRange* st = plan.steps.data() + plan.level_off[h];
    auto open = [&](int s) { st[s].off = (int32_t)plan.items.size(); };
    auto close = [&](int s) { st[s].cnt = (int32_t)plan.items.size() - st[s].off; };
    // The items from `from` on so that an XCD gets a run of them: neighbours in the list read the
    // same rows of a front, from its L2 then.
    auto spread = [&](int s, int from) {
      const int cnt = (int)plan.items.size() - from, phase = (from - st[s].off) % DIRECT_XCDS;
      int at[DIRECT_XCDS], run = 0;
      for (int x = 0; x < DIRECT_XCDS; ++x) {
        const int p = (x + DIRECT_XCDS - phase) % DIRECT_XCDS;     // its first position
        at[x] = run;
        run += p < cnt ? (cnt - p - 1) / DIRECT_XCDS + 1 : 0;
      }
      spare.assign(plan.items.begin() + from, plan.items.end());
      for (int p = 0; p < cnt; ++p)
        plan.items[from + p] = spare[at[(phase + p) % DIRECT_XCDS]++];
    };
    int bnd_tiles = 0;
    for (int i : by_level[h])
      if (plan.fronts[i].np > 1)
        bnd_tiles += (plan.fronts[i].nt - plan.fronts[i].np) * plan.fronts[i].np;
    const bool gain = bnd_tiles >= DIRECT_GAIN_TILES;
    // row tiles of a front that its panel steps take
    for (int i : by_level[h]) plan.fronts[i].gain = gain && plan.fronts[i].np > 1;
    auto rows_of = [&](const DirectFront& D) { return D.gain ? D.np : D.nt; };
    // step 0: blocks of K with a column among the own nodes, bucketed by tile, first columns first
    assemble.clear();
    int at_once = 1;
    for (; at_once < DIRECT_FIRST_MOST; ++at_once) {
      int items = 0;
      for (int i : by_level[h])
        if (plan.fronts[i].np > 0) items += ceil_div(rows_of(plan.fronts[i]), at_once);
      if (items <= DIRECT_FIRST_ITEMS) break;
    }
    open(STEP_PANEL);
    for (int i : by_level[h]) {
      go_on(stop);
      DirectFront& D = plan.fronts[i];
      const int ns = D.ns6 / 6, cnt = ns + D.nb6 / 6;
      if (ns == 0) continue;
      const int32_t* list = plan.nodes.data() + D.nodes_off;
      for (int k = 0; k < cnt; ++k) local[list[k]] = k;
      start.assign(D.nt * D.np + 1, 0);
      lo.resize(cnt);                        // first and last row tile of a node
      hi.resize(cnt);
      for (int k = 0; k < cnt; ++k) {
        const int first = k < ns ? 0 : D.np, row = k < ns ? 6 * k : 6 * k - D.ns6;
        lo[k] = first + row / DIRECT_NB;
        hi[k] = first + (row + 5) / DIRECT_NB;
      }
      auto each = [&](auto&& f) {            // over K's blocks and the tiles they lie in
        for (int q = 0; q < ns; ++q) {
          const int v = list[q];
          const int b0 = 6 * q / DIRECT_NB, b1 = (6 * q + 5) / DIRECT_NB;
          for (int e = rp[v]; e < rp[v + 1]; ++e) {
            const int r = local[col[e]];
            if (r < 0) continue;             // eliminated below
            for (int a = lo[r]; a <= hi[r]; ++a)
              for (int b = b0; b <= b1 && b <= a; ++b) f(b * D.nt + a, a, b, q, r, e);
          }
        }
      };
      each([&](int k, int, int, int, int, int) { ++start[k + 1]; });
      start[0] = (int32_t)plan.entries.size();
      for (int k = 0; k < D.nt * D.np; ++k) start[k + 1] += start[k];
      plan.entries.resize(start.back());
      fill.assign(start.begin(), start.end() - 1);
      each([&](int k, int a, int b, int q, int r, int e) {
        const int off = a < D.np ? a * DIRECT_NB : D.ns6 + (a - D.np) * DIRECT_NB;
        plan.entries[fill[k]++] = {(6 * r - off + DIRECT_EDGE) << 16 |
                                       (6 * q - b * DIRECT_NB + DIRECT_EDGE),
                                   e};
      });
      D.e0 = start[0];
      D.e1 = start[1];
      D.tile_off = (int32_t)plan.tile_end.size();
      plan.tile_end.insert(plan.tile_end.end(), start.begin() + 1, start.begin() + 1 + D.nt);
      const int nr = rows_of(D);
      for (int a = 0; a < nr; a += at_once)
        plan.items.push_back({i, a, -std::min(at_once, nr - a), start[a], start[a + 1]});
      for (int b = 0; b < D.np; ++b)
        for (int a = b == 0 ? nr : b; a < D.nt; ++a)
          assemble.push_back({i, a, b, start[b * D.nt + a], start[b * D.nt + a + 1]});
      for (int k = 0; k < cnt; ++k) local[list[k]] = -1;
    }
    spread(STEP_PANEL, st[STEP_PANEL].off);
    const int from = (int)plan.items.size();                 // the longer work first
    plan.items.insert(plan.items.end(), assemble.begin(), assemble.end());
    spread(STEP_PANEL, from);
    close(STEP_PANEL);
    for (int q = 1; q <= np; ++q) {
      open(STEP_PANEL + q);
      for (int i : by_level[h]) {
        const DirectFront& D = plan.fronts[i];
        for (int r = 0; q < D.np && r < rows_of(D); ++r) plan.items.push_back({i, r, -1, 0, 0});
      }
      spread(STEP_PANEL + q, st[STEP_PANEL + q].off);
      const int updates = (int)plan.items.size();
      for (int i : by_level[h]) {
        const DirectFront& D = plan.fronts[i];
        // a single panel is done once scaled, the last one's update goes with the Schur step
        if (q > D.np || D.np == 1 || (q == D.np && !gain)) continue;
        for (int r = 0; r < rows_of(D); ++r)
          for (int c = 0; c < D.np; ++c) plan.items.push_back({i, r, c, 0, 0});
      }
      spread(STEP_PANEL + q, updates);
      close(STEP_PANEL + q);
    }
    open(STEP_GAIN);
    for (int i : by_level[h]) {
      const DirectFront& D = plan.fronts[i];
      for (int r = rows_of(D); r < D.nt; ++r)
        for (int c = 0; c < D.np; ++c) plan.items.push_back({i, r, c, 0, 0});
    }
    spread(STEP_GAIN, st[STEP_GAIN].off);
    close(STEP_GAIN);
    open(STEP_SCHUR);
    for (int i : by_level[h]) {
      const int t = ceil_div(plan.fronts[i].nb6, DIRECT_NB);
      for (int a = 0; a < t; ++a)
        for (int b = 0; b <= a; ++b) plan.items.push_back({i, a, b, 0, 0});
    }
    spread(STEP_SCHUR, st[STEP_SCHUR].off);
    const int last = (int)plan.items.size();
    for (int i : by_level[h]) {
      const DirectFront& D = plan.fronts[i];
      for (int r = 0; !gain && D.np > 1 && r < D.nt; ++r)
        for (int c = 0; c < D.np; ++c) plan.items.push_back({i, r, c, 1, 0});
    }
    spread(STEP_SCHUR, last);
    close(STEP_SCHUR);
    open(STEP_FWD);
    int passes = 0;
    for (int i : by_level[h]) passes += ceil_div(plan.fronts[i].nb6, DIRECT_FWD_ROWS);
    const int rows = DIRECT_FWD_ROWS *
                     std::min(DIRECT_FWD_MOST, std::max(1, passes / DIRECT_FWD_ITEMS));
    for (int i : by_level[h]) {
      const DirectFront& D = plan.fronts[i];
      if (D.nb6 == 0 && D.ns6 > 0) plan.items.push_back({i, 0, 0, 0, 0});
      for (int a = 0; a < D.nb6; a += rows)
        plan.items.push_back({i, a, 0, std::min(a + rows, D.nb6), 0});
    }
    spread(STEP_FWD, st[STEP_FWD].off);
    close(STEP_FWD);
    open(STEP_BWD);
    for (int i : by_level[h])
      for (int a = 0; a < ceil_div(plan.fronts[i].ns6, DIRECT_BWD_COLS); ++a)
        plan.items.push_back({i, a, 0, 0, 0});
    spread(STEP_BWD, st[STEP_BWD].off);
    close(STEP_BWD);
  }
  return true;
} catch (const Stopped&) {
  plan = DirectPlan();
  return false;
}

int check_direct_plan(int n, const int32_t* rp, const int32_t* col, const DirectPlan& plan,
                      char* msg, size_t len) {
  auto fail = [&](int code, const char* what, long long at) {
    std::snprintf(msg, len, "direct plan: %s (at %lld)", what, at);
    return code;
  };
  // every node is eliminated once, in a front whose list holds its neighbours eliminated later
  std::vector<int32_t> front(n, -1), at(n, -1);
  for (size_t f = 0; f < plan.fronts.size(); ++f) {
    const DirectFront& D = plan.fronts[f];
    for (int k = 0; k < D.ns6 / 6; ++k) {
      const int v = plan.nodes[D.nodes_off + k];
      if (v < 0 || v >= n || front[v] >= 0) return fail(1, "node eliminated twice", v);
      front[v] = (int32_t)f;
    }
  }
  for (int v = 0; v < n; ++v)
    if (front[v] < 0) return fail(1, "node never eliminated", v);
  size_t blocks = 0;
  for (size_t f = 0; f < plan.fronts.size(); ++f) {
    const DirectFront& D = plan.fronts[f];
    const int ns = D.ns6 / 6, cnt = ns + D.nb6 / 6;
    const int32_t* list = plan.nodes.data() + D.nodes_off;
    for (int k = 0; k < cnt; ++k) {
      if (at[list[k]] >= 0) return fail(2, "node listed twice in a front", list[k]);
      at[list[k]] = k;
      if (k >= ns && plan.fronts[front[list[k]]].level <= D.level)
        return fail(3, "boundary node eliminated too early", list[k]);
    }
    for (int k = 0; k < ns; ++k)
      for (int e = rp[list[k]]; e < rp[list[k] + 1]; ++e)
        if (at[col[e]] < 0) {
          if (plan.fronts[front[col[e]]].level >= D.level)
            return fail(4, "neighbour missing from a front", list[k]);
        } else {
          ++blocks;
        }
    // each child's boundary lies in this front, in the same order
    for (int c = 0; c < 2; ++c) {
      const int32_t* map = plan.maps.data() + D.map_off + c * cnt;
      int prev = -1, seen = 0;
      for (int k = 0; k < cnt; ++k) {
        if (map[k] < 0) continue;
        if (D.child[c] < 0) return fail(5, "map without a child", (long long)f);
        const DirectFront& C = plan.fronts[D.child[c]];
        if (map[k] <= prev || map[k] >= C.nb6 / 6 ||
            plan.nodes[C.nodes_off + C.ns6 / 6 + map[k]] != list[k])
          return fail(5, "child map", (long long)f);
        prev = map[k];
        ++seen;
      }
      if (D.child_u[c] != (D.child[c] < 0 ? 0 : plan.fronts[D.child[c]].u_off))
        return fail(5, "child's Schur complement", (long long)f);
      if (D.child[c] >= 0 && (seen != plan.fronts[D.child[c]].nb6 / 6 ||
                              plan.fronts[D.child[c]].level >= D.level))
        return fail(6, "child boundary lost", (long long)f);
    }
    for (int k = 0; k < cnt; ++k) at[list[k]] = -1;
    const int64_t panel = (int64_t)(D.ns6 + D.nb6) * D.ns6;
    if (D.fact_off + panel > plan.fact_len || D.work_off + panel > plan.work_len ||
        D.u_off + direct_tri(D.nb6) > plan.u_len || D.v_off + D.nb6 > plan.v_len ||
        D.b_off + D.ns6 > 6 * (int64_t)n ||
        (D.np > 1 && (D.again_off + panel > plan.again_len ||
                      D.w_off + (int64_t)DIRECT_NB * DIRECT_NB * (3 * D.nt - D.np) > plan.w_len)))
      return fail(7, "array too short", (long long)f);
  }
  // a front's boundary tiles are formed by the gain step or by the update with the last panel
  std::vector<int> formed(plan.fronts.size(), 0);
  for (int h = 0; h < plan.levels(); ++h)
    for (int q = STEP_SCHUR; q <= STEP_PANEL + plan.level_np[h]; ++q) {
      const DirectRange st = plan.steps[plan.level_off[h] + q];
      for (int k = 0; k < st.cnt; ++k) {
        const DirectItem& it = plan.items[st.off + k];
        const DirectFront& D = plan.fronts[it.front];
        if (q == STEP_GAIN ? it.i >= D.np
                           : it.i >= D.np && it.j >= 0 &&
                                 (q == STEP_SCHUR ? it.e0 == 1 : q - STEP_PANEL == D.np))
          ++formed[it.front];
      }
    }
  for (size_t f = 0; f < plan.fronts.size(); ++f) {
    const DirectFront& D = plan.fronts[f];
    if (D.np > 1 && formed[f] != (D.nt - D.np) * D.np)
      return fail(10, "boundary tiles", (long long)f);
  }
  // the first panel step's tiles hold every value of those blocks once
  size_t values = 0;
  auto count = [&](const DirectFront& D, int i, int j, int e0, int e1) {
    const DirectRows R = direct_rows(D, i);
    const int nc = std::min(DIRECT_NB, D.ns6 - j * DIRECT_NB);
    for (int e = e0; e < e1; ++e) {
      const int r = (plan.entries[e].rc >> 16) - DIRECT_EDGE;
      const int c = (plan.entries[e].rc & 0xffff) - DIRECT_EDGE;
      values += (i < D.np && i != j ? 2 : 1) *
                (size_t)std::max(0, std::min(r + 6, R.n) - std::max(r, 0)) *
                (size_t)std::max(0, std::min(c + 6, nc) - std::max(c, 0));
    }
  };
  for (int h = 0; h < plan.levels(); ++h) {
    const DirectRange st = plan.steps[plan.level_off[h] + STEP_PANEL];
    for (int k = 0; k < st.cnt; ++k) {
      const DirectItem& it = plan.items[st.off + k];
      const DirectFront& D = plan.fronts[it.front];
      if (D.e1 != plan.tile_end[D.tile_off]) return fail(8, "first tile's entries", it.front);
      for (int t = 0; t < (it.j < 0 ? -it.j : 1); ++t) {
        if (it.i + t >= D.nt || it.j > it.i) return fail(8, "row tile out of range", it.front);
        const int e0 = t == 0 ? it.e0 : plan.tile_end[D.tile_off + it.i + t - 1];
        const int e1 = t == 0 ? it.e1 : plan.tile_end[D.tile_off + it.i + t];
        if (e0 < 0 || e0 > e1 || e1 > (int)plan.entries.size())
          return fail(8, "entries out of range", it.front);
        count(D, it.i + t, it.j < 0 ? 0 : it.j, e0, e1);
      }
    }
  }
  if (36 * blocks != values) return fail(8, "blocks of K", (long long)blocks);
  // Schur complements alive at the same time do not overlap
  std::vector<int> parent(plan.fronts.size(), -1);
  for (size_t f = 0; f < plan.fronts.size(); ++f)
    for (int c : plan.fronts[f].child)
      if (c >= 0) parent[c] = (int)f;
  for (int h = 0; h < plan.levels(); ++h) {
    std::vector<std::pair<int64_t, int64_t>> live;
    for (size_t f = 0; f < plan.fronts.size(); ++f) {
      const DirectFront& D = plan.fronts[f];
      const int last = parent[f] < 0 ? D.level : plan.fronts[parent[f]].level;
      if (D.nb6 && D.level <= h && last >= h)
        live.emplace_back(D.u_off, D.u_off + direct_tri(D.nb6));
    }
    std::sort(live.begin(), live.end());
    for (size_t k = 1; k < live.size(); ++k)
      if (live[k].first < live[k - 1].second) return fail(9, "Schur complements overlap", h);
  }
  return 0;
}

}  // namespace sso
