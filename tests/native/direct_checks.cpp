// Host checks of the direct solver's plan (built with AddressSanitizer and
// UndefinedBehaviorSanitizer, run on the CPU): on node graphs of every kind that the solver meets,
// grids of members and quads in several numberings, chains, hubs, pieces, the plan's invariants
// hold (check_direct_plan), and eliminating with it -- the work lists walked as the kernels walk
// them, in plain loops over bounds-checked arrays -- solves a random symmetric positive definite
// block system.
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "direct_plan.h"

using namespace sso;

struct Graph {
  int n = 0;
  std::vector<std::set<int>> adj;
  explicit Graph(int n_) : n(n_), adj(n_) {
    for (int i = 0; i < n; ++i) adj[i].insert(i);
  }
  void edge(int a, int b) {
    adj[a].insert(b);
    adj[b].insert(a);
  }
};

static Graph quads(int mx, int my) {
  Graph g((mx + 1) * (my + 1));
  for (int j = 0; j < my; ++j)
    for (int i = 0; i < mx; ++i) {
      const int a = j * (mx + 1) + i, q[4] = {a, a + 1, a + mx + 2, a + mx + 1};
      for (int x : q)
        for (int y : q) g.edge(x, y);
    }
  return g;
}
static Graph members(int nx, int ny) {
  Graph g(nx * ny);
  for (int j = 0; j < ny; ++j)
    for (int i = 0; i < nx; ++i) {
      if (i + 1 < nx) g.edge(j * nx + i, j * nx + i + 1);
      if (j + 1 < ny) g.edge(j * nx + i, j * nx + i + nx);
    }
  return g;
}
static Graph hub(int spokes) {
  Graph g(spokes + 1);
  for (int i = 0; i < spokes; ++i) {
    g.edge(0, 1 + i);
    g.edge(1 + i, 1 + (i + 1) % spokes);
  }
  return g;
}
// Chains of `length` nodes from one node, each with two more where it branches.
static Graph ribs(int count, int length, int branches = 0) {
  Graph g(1 + count * length * (1 + branches));
  int next = 1;
  for (int i = 0; i < count; ++i)
    for (int k = 0, at = 0; k < length; ++k) {
      const int v = next++;
      g.edge(at, v);
      for (int b = 0; b < branches; ++b) g.edge(v, next++);
      at = v;
    }
  return g;
}
// Every one of m nodes joined to every one of n others.
static Graph joined(int m, int n) {
  Graph g(m + n);
  for (int i = 0; i < m; ++i)
    for (int j = 0; j < n; ++j) g.edge(i, m + j);
  return g;
}
static Graph complete(int n) {
  Graph g(n);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < i; ++j) g.edge(i, j);
  return g;
}
static Graph pieces(const std::vector<Graph>& parts) {
  int n = 0;
  for (const Graph& p : parts) n += p.n;
  Graph g(n);
  int o = 0;
  for (const Graph& p : parts) {
    for (int i = 0; i < p.n; ++i)
      for (int j : p.adj[i]) g.edge(o + i, o + j);
    o += p.n;
  }
  return g;
}
static Graph shuffled(const Graph& g, unsigned seed) {
  std::mt19937 r(seed);
  std::vector<int> p(g.n);
  for (int i = 0; i < g.n; ++i) p[i] = i;
  for (int i = g.n - 1; i > 0; --i) std::swap(p[i], p[r() % (i + 1)]);
  Graph s(g.n);
  for (int i = 0; i < g.n; ++i)
    for (int j : g.adj[i]) s.edge(p[i], p[j]);
  return s;
}

// Sum over the children of the entry (r, c), DOF rows of front f.
static double children(const DirectPlan& pl, const std::vector<double>& u, const DirectFront& F,
                       int r, int c) {
  const int cnt = (F.ns6 + F.nb6) / 6;
  double s = 0.0;
  for (int k = 0; k < 2; ++k) {
    if (F.child[k] < 0) continue;
    const DirectFront& C = pl.fronts.at(F.child[k]);
    const int mr = pl.maps.at(F.map_off + k * cnt + r / 6);
    const int mc = pl.maps.at(F.map_off + k * cnt + c / 6);
    if (mr < 0 || mc < 0) continue;
    const int a = 6 * mr + r % 6, b = 6 * mc + c % 6;
    s += u.at(C.u_off + direct_tri(std::max(a, b)) + std::min(a, b));
  }
  return s;
}

static int run(const std::string& name, const Graph& g, bool numeric) {
  std::vector<int32_t> rp{0}, col;
  for (const auto& a : g.adj) {
    col.insert(col.end(), a.begin(), a.end());
    rp.push_back((int32_t)col.size());
  }
  DirectPlan pl;
  char msg[256] = "";
  if (!build_direct_plan(g.n, rp.data(), col.data(), 1e12, pl) ||
      check_direct_plan(g.n, rp.data(), col.data(), pl, msg, sizeof msg) != 0) {
    std::printf("FAIL %s: %s\n", name.c_str(), msg);
    return 1;
  }
  // levels are launches in a chain: cuts halve a part, or nearly, and what no cut parts is not cut
  if (pl.levels() > 16 + std::log2((double)g.n)) {
    std::printf("FAIL %s: %d levels for %d nodes\n", name.c_str(), pl.levels(), g.n);
    return 1;
  }
  // the plan depends on the graph alone
  DirectPlan again;
  build_direct_plan(g.n, rp.data(), col.data(), 1e12, again);
  if (again.nodes != pl.nodes || again.maps != pl.maps) {
    std::printf("FAIL %s: two plans of one graph differ\n", name.c_str());
    return 1;
  }
  DirectPlan none;
  if (build_direct_plan(g.n, rp.data(), col.data(), 8.0 * (double)pl.values() - 1.0, none)) {
    std::printf("FAIL %s: limit not kept\n", name.c_str());
    return 1;
  }
  if (!numeric) return 0;
  // K: diagonally dominant, symmetric
  std::mt19937 rng(7);
  std::uniform_real_distribution<double> ud(-1.0, 1.0);
  const int n6 = 6 * g.n;
  std::vector<double> K(36 * col.size());
  auto slot = [&](int I, int J) {
    for (int e = rp[I]; e < rp[I + 1]; ++e)
      if (col[e] == J) return e;
    return -1;
  };
  for (int I = 0; I < g.n; ++I)
    for (int e = rp[I]; e < rp[I + 1]; ++e) {
      const int J = col[e];
      if (J > I) continue;
      const int m = slot(J, I);
      for (int a = 0; a < 6; ++a)
        for (int b = 0; b < 6; ++b) {
          if (I == J && b > a) continue;
          const double v = I == J && a == b ? 8.0 * (rp[I + 1] - rp[I]) : ud(rng);
          K[36 * (size_t)e + 6 * a + b] = v;
          K[36 * (size_t)m + 6 * b + a] = v;
        }
    }
  std::vector<double> f(n6), x(n6, 0.0);
  for (double& v : f) v = ud(rng);
  std::vector<double> fact(pl.fact_len), f0(pl.work_len), u(pl.u_len, NAN), v(pl.v_len),
      b(n6), seen(pl.fact_len, 0.0);
  for (int h = 0; h < pl.levels(); ++h) {
    const DirectRange* st = pl.steps.data() + pl.level_off[h];
    for (int q = 0; q < st[STEP_PANEL].cnt; ++q) {
      const DirectItem it = pl.items.at(st[STEP_PANEL].off + q);
      const DirectFront& F = pl.fronts.at(it.front);
      for (int t = 0; t < (it.j < 0 ? -it.j : 1); ++t) {
        const DirectRows R = direct_rows(F, it.i + t);
        const int r0 = R.r0, c0 = DIRECT_NB * std::max(it.j, 0);
        const int nr = R.n, nc = std::min(DIRECT_NB, F.ns6 - c0);
        for (int r = r0; r < r0 + nr; ++r)
          for (int c = c0; c < c0 + nc; ++c) {
            f0.at(F.work_off + (int64_t)r * F.ns6 + c) = children(pl, u, F, r, c);
            seen.at(F.fact_off + (int64_t)r * F.ns6 + c) += 1.0;
            if (r < F.ns6 && r0 != c0) seen.at(F.fact_off + (int64_t)c * F.ns6 + r) += 1.0;
          }
        const int e0 = t == 0 ? it.e0 : pl.tile_end.at(F.tile_off + it.i + t - 1);
        const int e1 = t == 0 ? it.e1 : pl.tile_end.at(F.tile_off + it.i + t);
        for (int e = e0; e < e1; ++e) {
          const DirectEntry en = pl.entries.at(e);
          const int er = (en.rc >> 16) - DIRECT_EDGE, ec = (en.rc & 0xffff) - DIRECT_EDGE;
          for (int cb = 0; cb < 6; ++cb)
            for (int ca = 0; ca < 6; ++ca) {
              const int r = er + ca, c = ec + cb;
              if (r >= 0 && r < nr && c >= 0 && c < nc)
                f0.at(F.work_off + (int64_t)(r0 + r) * F.ns6 + c0 + c) +=
                    K.at(36 * (size_t)en.slot + 6 * cb + ca);
            }
        }
        for (int r = r0; r < r0 + nr && r < F.ns6; ++r)     // the other half
          for (int c = c0; c < c0 + nc; ++c)
            f0.at(F.work_off + (int64_t)c * F.ns6 + r) = f0.at(F.work_off + (int64_t)r * F.ns6 + c);
      }
    }
    for (int i = 0; i < (int)pl.fronts.size(); ++i) {
      const DirectFront& F = pl.fronts[i];
      if (F.level != h) continue;
      const int s = F.ns6, m = F.ns6 + F.nb6;
      for (int64_t q = 0; q < (int64_t)m * s; ++q)
        if (seen[F.fact_off + q] != 1.0) {
          std::printf("FAIL %s: panel entry assembled %g times\n", name.c_str(),
                      seen[F.fact_off + q]);
          return 1;
        }
      // sweep column by column; the boundary rows follow
      std::vector<double> A(f0.begin() + F.work_off, f0.begin() + F.work_off + (int64_t)m * s);
      for (int k = 0; k < s; ++k) {
        const double d = 1.0 / A[k * s + k];
        std::vector<double> ck(m), rk(A.begin() + k * s, A.begin() + (k + 1) * s);
        for (int r = 0; r < m; ++r) ck[r] = A[r * s + k];
        for (int r = 0; r < m; ++r)
          for (int c = 0; c < s; ++c)
            A[r * s + c] = r == k ? (c == k ? -d : rk[c] * d)
                                  : (c == k ? ck[r] * d : A[r * s + c] - ck[r] * d * rk[c]);
      }
      std::copy(A.begin(), A.end(), fact.begin() + F.fact_off);
      for (int r = 0; r < F.nb6; ++r)
        for (int c = 0; c <= r; ++c) {
          double t = children(pl, u, F, s + r, s + c);
          for (int k = 0; k < s; ++k)
            t -= A[(s + r) * s + k] * f0[F.work_off + (int64_t)(s + c) * s + k];
          u.at(F.u_off + direct_tri(r) + c) = t;
        }
    }
  }
  auto up = [&](const DirectFront& F, int r) {
    const int cnt = (F.ns6 + F.nb6) / 6;
    double t = 0.0;
    for (int k = 0; k < 2; ++k) {
      const int mm = pl.maps.at(F.map_off + k * cnt + r / 6);
      if (mm >= 0) t += v.at(pl.fronts.at(F.child[k]).v_off + 6 * mm + r % 6);
    }
    return t;
  };
  for (int h = 0; h < pl.levels(); ++h) {
    const DirectRange r = pl.steps[pl.level_off[h] + STEP_FWD];
    for (int q = 0; q < r.cnt; ++q) {
      const DirectItem it = pl.items.at(r.off + q);
      const DirectFront& F = pl.fronts.at(it.front);
      for (int c = 0; c < F.ns6; ++c)
        b.at(F.b_off + c) = f.at(6 * pl.nodes.at(F.nodes_off + c / 6) + c % 6) + up(F, c);
      for (int k = it.i; k < it.e0; ++k) {
        double t = up(F, F.ns6 + k);
        for (int c = 0; c < F.ns6; ++c)
          t -= fact.at(F.fact_off + (int64_t)(F.ns6 + k) * F.ns6 + c) * b[F.b_off + c];
        v.at(F.v_off + k) = t;
      }
    }
  }
  for (int h = pl.levels() - 1; h >= 0; --h) {
    const DirectRange r = pl.steps[pl.level_off[h] + STEP_BWD];
    for (int q = 0; q < r.cnt; ++q) {
      const DirectItem it = pl.items.at(r.off + q);
      const DirectFront& F = pl.fronts.at(it.front);
      for (int c = it.i * DIRECT_BWD_COLS; c < std::min(F.ns6, (it.i + 1) * DIRECT_BWD_COLS); ++c) {
        double t = 0.0;
        for (int k = 0; k < F.ns6 + F.nb6; ++k) {
          const int node = pl.nodes.at(F.nodes_off + k / 6);
          t -= fact.at(F.fact_off + (int64_t)k * F.ns6 + c) *
               (k < F.ns6 ? b[F.b_off + k] : x.at(6 * node + k % 6));
        }
        x.at(6 * pl.nodes.at(F.nodes_off + c / 6) + c % 6) = t;
      }
    }
  }
  double worst = 0.0;
  for (int I = 0; I < g.n; ++I)
    for (int a = 0; a < 6; ++a) {
      double t = f[6 * I + a];
      for (int e = rp[I]; e < rp[I + 1]; ++e)
        for (int c = 0; c < 6; ++c) t -= K[36 * (size_t)e + 6 * a + c] * x[6 * col[e] + c];
      worst = std::fmax(worst, std::fabs(t));
    }
  // K is diagonally dominant with entries of order 1 to 1000: a backward stable solve leaves
  // some n_terms * eps * |K| |x|, far below 1e-11
  if (!(worst <= 1e-11)) {
    std::printf("FAIL %s: residual %g\n", name.c_str(), worst);
    return 1;
  }
  return 0;
}

// A build that nobody waits for any more ends early, without a plan.
static int stopped() {
  const Graph g = quads(260, 260);
  std::vector<int32_t> rp{0}, col;
  for (const auto& a : g.adj) {
    col.insert(col.end(), a.begin(), a.end());
    rp.push_back((int32_t)col.size());
  }
  int bad = 0;
  for (bool at_once : {true, false}) {
    std::atomic<bool> stop{at_once};
    DirectPlan pl;
    bool built = true;
    std::thread t([&] { built = build_direct_plan(g.n, rp.data(), col.data(), 1e12, pl, &stop); });
    if (!at_once) std::this_thread::sleep_for(std::chrono::milliseconds(20));   // it takes longer
    stop = true;
    t.join();
    if (built || !pl.fronts.empty() || !pl.items.empty()) {
      std::printf("FAIL a build that was stopped gave a plan\n");
      ++bad;
    }
  }
  return bad;
}

int main() {
  int bad = stopped();
  struct {
    const char* name;
    Graph g;
    bool numeric;
  } all[] = {
      {"one node", Graph(1), true},
      {"two nodes", members(2, 1), true},
      {"one quad", quads(1, 1), true},
      {"leaf", members(5, 2), true},
      {"leaf and one more", members(11, 1), true},
      {"quads 9x7", quads(9, 7), true},
      {"quads 16x16", quads(16, 16), true},
      {"quads 3x60", quads(3, 60), true},
      {"members 13x13", members(13, 13), true},
      {"chain", members(400, 1), true},
      {"chain, shuffled", shuffled(members(301, 1), 3), true},
      {"quads 11x14, shuffled", shuffled(quads(11, 14), 5), true},
      {"hub", hub(20), true},
      {"large hub", hub(90), true},
      {"complete", complete(25), true},
      {"no edges", Graph(9), true},
      {"pieces", pieces({quads(4, 4), Graph(1), members(30, 1), hub(12), quads(7, 2)}), true},
      {"spokes", ribs(50, 1), true},
      {"ribs", ribs(14, 15), true},
      {"branched ribs", shuffled(ribs(30, 4, 2), 6), true},
      {"nodes joined to all others", joined(3, 90), true},
      {"large clique", complete(60), true},
      {"spokes and a clique", pieces({ribs(40, 1), complete(30), Graph(3)}), true},
      {"96 ribs", ribs(96, 20), false},
      {"300 ribs", ribs(300, 20), false},
      {"5000 spokes", ribs(5000, 1), false},
      {"20000 spokes", shuffled(ribs(20000, 1), 2), false},
      {"3000 branched spokes", ribs(3000, 1, 3), false},
      {"2 nodes joined to 4000", joined(2, 4000), false},
      {"30 nodes joined to 100", joined(30, 100), false},
      {"clique of 300", complete(300), false},
      {"quads 60x60", quads(60, 60), false},
      {"quads 80x70, shuffled", shuffled(quads(80, 70), 9), false},
  };
  for (auto& c : all) bad += run(c.name, c.g, c.numeric);
  std::printf("%s (%d failures)\n", bad ? "failed" : "ok", bad);
  return bad ? 1 : 0;
}
