// Host analysis for the supernodal Cholesky of A = M + h B + h^2 K (Eq. 5):
// node graph of the tetrahedral mesh, nested-dissection ordering and the
// supernodal elimination structure that the dissection tree implies.
//
// Ordering: recursive coordinate bisection.  At each region the nodes, kept
// sorted along every axis, are taken along the axis of largest extent and cut near the median at the
// widest coordinate gap (between grid layers for the jittered grids); the
// vertex separator is the smaller of the two one-sided boundaries of the cut.
// Regions are numbered children first, separator last, so every supernode's
// subtree occupies a contiguous range of permuted nodes.
//
// Structure: the below-rows of a supernode are the nodes outside its region
// adjacent to it.  Because separators isolate sibling regions, these are all
// ancestor-separator nodes and contain the true fill of every column of the
// supernode; explicit zeros are stored and computed, which keeps the factor
// exact (relaxed supernodes = dissection tree nodes).
#include <algorithm>
#include <array>
#include <cmath>
#include <numeric>
#include <sstream>
#include <stdexcept>

#include "icr_internal.hpp"

namespace icr {

MeshGraph build_graph(int N, const int32_t *tets, int T) {
  MeshGraph g;
  g.N = N;
  // incidences by counting, ascending element order per node
  g.inc_ptr.assign(N + 1, 0);
  for (long e = 0; e < 4L * T; ++e) g.inc_ptr[tets[e] + 1]++;
  for (int i = 0; i < N; ++i) g.inc_ptr[i + 1] += g.inc_ptr[i];
  g.inc.resize(4L * T);
  {
    std::vector<int> at(g.inc_ptr.begin(), g.inc_ptr.end() - 1);
    for (long e = 0; e < 4L * T; ++e) g.inc[at[tets[e]]++] = (int)e;
  }
  // neighbours of a node: the distinct nodes of its elements (a stamp per
  // node tells which were met)
  g.ptr.assign(N + 1, 0);
  g.adj.reserve(16L * N);
  std::vector<int> met(N, -1);
  for (int i = 0; i < N; ++i) {
    const size_t first = g.adj.size();
    g.adj.push_back(i);
    met[i] = i;
    for (int e = g.inc_ptr[i]; e < g.inc_ptr[i + 1]; ++e) {
      const int32_t *tet = tets + 4L * (g.inc[e] / 4);
      for (int b = 0; b < 4; ++b)
        if (met[tet[b]] != i) {
          met[tet[b]] = i;
          g.adj.push_back(tet[b]);
        }
    }
    std::sort(g.adj.begin() + first, g.adj.end());
    g.ptr[i + 1] = (int)g.adj.size();
  }
  return g;
}

namespace {

struct ND {
  const double *xyz;
  const MeshGraph *g;
  int leaf_max;
  // longest edge along each axis; infinite if a coordinate is not finite
  double reach[3] = {0.0, 0.0, 0.0};
  std::vector<int> stamp;   // region marker
  int cur = 0;
  Symbolic *sym;
  int next_pos = 0;
  std::vector<std::vector<int>> kids;

  int make_sup(const std::vector<int> &nodes, const std::vector<int> &children) {
    int s = sym->nsup++;
    sym->col0.push_back(next_pos);
    sym->ncol.push_back((int)nodes.size());
    sym->parent.push_back(-1);
    sym->first_desc.push_back(children.empty() ? s : sym->first_desc[children[0]]);
    for (int c : children) sym->parent[c] = s;
    kids.push_back(children);
    for (int v : nodes) sym->perm[next_pos++] = v;
    return s;
  }

  // The region's nodes sorted along each axis (coordinate, then id; a NaN as
  // +infinity): the lists of the root are sorted once and split stably on the
  // way down.
  typedef std::array<std::vector<int>, 3> Sorted;

  // Extent of a sorted list along its axis, without the NaNs.
  double extent(const std::vector<int> &v, int a) const {
    double lo = 1e300, hi = -1e300;
    auto add = [&](int node) {
      lo = std::min(lo, xyz[3 * node + a]);
      hi = std::max(hi, xyz[3 * node + a]);
    };
    if (std::isinf(reach[a])) {
      for (int node : v) add(node);
    } else {
      add(v.front());
      add(v.back());
    }
    return hi - lo;
  }

  int rec(Sorted by) {
    const int n = (int)by[0].size();
    if (n <= leaf_max) {
      std::sort(by[0].begin(), by[0].end());
      return make_sup(by[0], {});
    }
    int ax = 0;
    double ext = extent(by[0], 0);
    for (int a = 1; a < 3; ++a) {
      const double e = extent(by[a], a);
      if (e > ext) {
        ax = a;
        ext = e;
      }
    }
    const std::vector<int> &nodes = by[ax];
    int k0 = std::max(1, (int)(0.35 * n)), k1 = std::min(n - 1, (int)(0.65 * n));
    int best = n / 2;
    double bgap = -1.0;
    for (int k = k0; k <= k1; ++k) {
      double gap = xyz[3 * nodes[k] + ax] - xyz[3 * nodes[k - 1] + ax];
      if (gap > bgap * (1.0 + 1e-9) ||
          (std::fabs(gap - bgap) <= 1e-9 * std::fabs(bgap) && std::abs(k - n / 2) < std::abs(best - n / 2))) {
        bgap = gap;
        best = k;
      }
    }
    // sides of the cut; the separator is the smaller one-sided boundary
    const int left = ++cur, right = ++cur;
    for (int k = 0; k < n; ++k) stamp[nodes[k]] = k < best ? left : right;
    // (no edge is longer along the axis than reach, so only nodes that close to
    // the other side can have a neighbour there; with an infinite reach all are
    // looked at, also those whose distance is a NaN)
    auto at_cut = [&](int v, int other, std::vector<int> &sep) {
      for (int e = g->ptr[v]; e < g->ptr[v + 1]; ++e)
        if (stamp[g->adj[e]] == other) {
          sep.push_back(v);
          return;
        }
    };
    std::vector<int> sepL, sepR;
    const double xl = xyz[3 * nodes[best - 1] + ax], xr = xyz[3 * nodes[best] + ax];
    for (int k = best - 1; k >= 0 && !(xr - xyz[3 * nodes[k] + ax] > reach[ax]); --k) at_cut(nodes[k], right, sepL);
    for (int k = best; k < n && !(xyz[3 * nodes[k] + ax] - xl > reach[ax]); ++k) at_cut(nodes[k], left, sepR);
    std::vector<int> S = sepL.size() <= sepR.size() ? std::move(sepL) : std::move(sepR);
    const int sepmark = ++cur;
    if (S.empty()) {   // disconnected halves: any single node separates them
      S.push_back(best > 0 ? nodes[best - 1] : nodes[n - 1]);
    }
    for (int v : S) stamp[v] = sepmark;
    Sorted A, B;
    for (int a = 0; a < 3; ++a) {
      A[a].reserve(best);
      B[a].reserve(n - best);
      for (int v : by[a]) {
        if (stamp[v] == left)
          A[a].push_back(v);
        else if (stamp[v] == right)
          B[a].push_back(v);
      }
      std::vector<int>().swap(by[a]);
    }
    std::sort(S.begin(), S.end());
    std::vector<int> children;
    if (!A[0].empty()) children.push_back(rec(std::move(A)));
    if (!B[0].empty()) children.push_back(rec(std::move(B)));
    return make_sup(S, children);
  }
};

}  // namespace

void analyze(const double *xyz, const MeshGraph &g, int leaf_max, Symbolic &sym) {
  const int N = g.N;
  sym = Symbolic();
  sym.N = N;
  sym.perm.assign(N, -1);
  ND nd;
  nd.xyz = xyz;
  nd.g = &g;
  nd.leaf_max = leaf_max;
  nd.stamp.assign(N, 0);
  for (int v = 0; v < N; ++v)
    for (int e = g.ptr[v]; e < g.ptr[v + 1]; ++e)
      for (int a = 0; a < 3; ++a) {   // (a node is its own neighbour: inf - inf)
        const double d = std::fabs(xyz[3 * v + a] - xyz[3 * g.adj[e] + a]);
        nd.reach[a] = std::max(nd.reach[a], std::isnan(d) ? HUGE_VAL : d);
      }
  nd.sym = &sym;
  // connected components are dissected separately and become sibling roots
  std::vector<int> comp(N, -1);
  std::vector<std::vector<int>> comps;
  for (int s = 0; s < N; ++s) {
    if (comp[s] >= 0) continue;
    std::vector<int> stack{s}, members;
    comp[s] = (int)comps.size();
    while (!stack.empty()) {
      int v = stack.back();
      stack.pop_back();
      members.push_back(v);
      for (int e = g.ptr[v]; e < g.ptr[v + 1]; ++e) {
        int u = g.adj[e];
        if (comp[u] < 0) {
          comp[u] = comp[s];
          stack.push_back(u);
        }
      }
    }
    comps.push_back(std::move(members));
  }
  std::vector<std::pair<double, int>> key;
  for (auto &c : comps) {
    ND::Sorted by;
    for (int a = 0; a < 3; ++a) {
      key.clear();
      for (int v : c) key.emplace_back(std::isnan(xyz[3 * v + a]) ? HUGE_VAL : xyz[3 * v + a], v);
      std::sort(key.begin(), key.end());
      by[a].reserve(c.size());
      for (const auto &k : key) by[a].push_back(k.second);
    }
    nd.rec(std::move(by));
  }
  sym.iperm.assign(N, -1);
  for (int p = 0; p < N; ++p) sym.iperm[sym.perm[p]] = p;

  const int ns = sym.nsup;
  sym.child_ptr.assign(ns + 1, 0);
  for (int s = 0; s < ns; ++s) sym.child_ptr[s + 1] = sym.child_ptr[s] + (int)nd.kids[s].size();
  sym.child.clear();
  for (int s = 0; s < ns; ++s)
    for (int c : nd.kids[s]) sym.child.push_back(c);

  // below rows: nodes outside the region adjacent to it (all later in the
  // order): those of the children that lie outside, and the outside neighbours
  // of the own columns
  sym.rows_ptr.assign(ns + 1, 0);
  sym.rows.clear();
  std::vector<int> mark(N, -1);
  for (int s = 0; s < ns; ++s) {
    const int rlo = sym.col0[sym.first_desc[s]], c0 = sym.col0[s], rhi = c0 + sym.ncol[s];
    const size_t first = sym.rows.size();
    for (int e = sym.child_ptr[s]; e < sym.child_ptr[s + 1]; ++e) {
      const int c = sym.child[e];
      for (int i = sym.rows_ptr[c]; i < sym.rows_ptr[c + 1]; ++i) {
        const int q = sym.rows[i];
        if (q >= rhi && mark[q] != s) {
          mark[q] = s;
          sym.rows.push_back(q);
        }
      }
    }
    for (int p = c0; p < rhi; ++p) {
      const int v = sym.perm[p];
      for (int e = g.ptr[v]; e < g.ptr[v + 1]; ++e) {
        const int q = sym.iperm[g.adj[e]];
        if (q >= rhi && mark[q] != s) {
          mark[q] = s;
          sym.rows.push_back(q);
        }
        if (q < rlo) throw std::runtime_error("dissection: region adjacent to an earlier node");
      }
    }
    std::sort(sym.rows.begin() + first, sym.rows.end());
    sym.rows_ptr[s + 1] = (int)sym.rows.size();
  }
  // heights and levels
  sym.height.assign(ns, 0);
  int H = 0;
  for (int s = 0; s < ns; ++s) {
    int h = 0;
    for (int e = sym.child_ptr[s]; e < sym.child_ptr[s + 1]; ++e) h = std::max(h, sym.height[sym.child[e]] + 1);
    sym.height[s] = h;
    H = std::max(H, h);
  }
  sym.nlevels = H + 1;
  sym.level_ptr.assign(H + 2, 0);
  for (int s = 0; s < ns; ++s) sym.level_ptr[sym.height[s] + 1]++;
  for (int l = 0; l <= H; ++l) sym.level_ptr[l + 1] += sym.level_ptr[l];
  sym.level_sup.assign(ns, 0);
  std::vector<int> fill(sym.level_ptr.begin(), sym.level_ptr.end() - 1);
  for (int s = 0; s < ns; ++s) sym.level_sup[fill[sym.height[s]]++] = s;
}

std::string check_symbolic(const MeshGraph &g, const Symbolic &sym) {
  std::ostringstream err;
  const int N = sym.N;
  std::vector<int> seen(N, 0);
  for (int p = 0; p < N; ++p) {
    int v = sym.perm[p];
    if (v < 0 || v >= N || seen[v]++) {
      err << "perm is not a permutation at " << p;
      return err.str();
    }
  }
  int pos = 0;
  for (int s = 0; s < sym.nsup; ++s) {
    if (sym.col0[s] != pos || sym.ncol[s] < 1) {
      err << "supernode " << s << " columns not contiguous";
      return err.str();
    }
    pos += sym.ncol[s];
    int p = sym.parent[s];
    if (p >= 0 && p <= s) {
      err << "parent not after child at " << s;
      return err.str();
    }
    if (p >= 0) {
      // child's below rows must be columns or below rows of the parent
      int pc0 = sym.col0[p], pc1 = pc0 + sym.ncol[p];
      int at = sym.rows_ptr[p];   // both row lists ascend
      for (int e = sym.rows_ptr[s]; e < sym.rows_ptr[s + 1]; ++e) {
        int r = sym.rows[e];
        while (at < sym.rows_ptr[p + 1] && sym.rows[at] < r) ++at;
        bool ok = (r >= pc0 && r < pc1) || (at < sym.rows_ptr[p + 1] && sym.rows[at] == r);
        if (!ok) {
          err << "row " << r << " of supernode " << s << " missing in parent " << p;
          return err.str();
        }
      }
    } else if (sym.rows_ptr[s + 1] != sym.rows_ptr[s]) {
      err << "root " << s << " has below rows";
      return err.str();
    }
  }
  if (pos != N) return "columns do not cover all nodes";
  (void)g;
  return std::string();
}

}  // namespace icr
