// Elimination plan of the coarsest inverse (host only).
//
// The coarsest operator couples a node only with its 26 neighbours (8 in the
// plane), so with the unknowns ordered plane by plane along the grid's longest
// axis it is block tridiagonal, and planes that are not neighbours can be
// pivoted in the same step.  The plan dissects the planes: a separator plane
// splits a run of planes in two independent halves, which are pivoted side by
// side before it.  Pivoting a block K touches only the rows it is coupled
// with by then: the contiguous range [lo, hi) from its run's left boundary
// plane to the right one.  The number of dependent block steps falls from
// n / 64 to about log2(planes) * (plane size / 64).
#pragma once

#include <algorithm>
#include <cstdint>
#include <utility>
#include <vector>

namespace aarmr {

constexpr int kInvBlock = 64;  // most rows of a block

// Order of the unknowns of the coarsest level: component c of node (i, j, k)
// is row c * sc + i * si + j * sj + k * sk.
struct CoarseOrder {
  int si = 0, sj = 0, sk = 0, sc = 0;
};

// The order for a grid of nxp * nyp * nzp nodes with `comps` unknowns each:
// slowest along the axis with the most nodes, then by component.  *plane
// receives the unknowns of one plane.
inline CoarseOrder make_coarse_order(int nxp, int nyp, int nzp, int comps, int* plane) {
  CoarseOrder o;
  if (nxp >= nyp && nxp >= nzp) {
    o.sj = 1, o.sk = nyp, o.sc = nyp * nzp, o.si = comps * o.sc;
    *plane = o.si;
  } else if (nyp >= nzp) {
    o.si = 1, o.sk = nxp, o.sc = nxp * nzp, o.sj = comps * o.sc;
    *plane = o.sj;
  } else {
    o.si = 1, o.sj = nxp, o.sc = nxp * nyp, o.sk = comps * o.sc;
    *plane = o.sk;
  }
  return o;
}

// What one workgroup of a step does.
enum InvKind : int16_t {
  kInvTile = 0,    // A_IJ -= sum over pivots of T_I c_J^T (none for a run's first pivot)
  kInvDiag = 1,    // A_KK = -P
  kInvCrossI = 2,  // I is the other block, J = K: A_IK = T_I
  kInvCrossJ = 3,  // J is the other block, I = K: A_KJ = T_J^T
  kInvPanel = 4,   // a first pivot's panel: C_next[p][j] = A[I + p][j], j in J
};

// p0, p1: slots of the step's pivots that contribute (-1: none) and their
// blocks [k0?, k0? + kb?); nrow, ncol: slot of the next step's pivot whose block
// I or J is (-1: none).  A tile with I = J and nrow >= 0 also inverts itself
// into that pivot.  Slots count a step's pivots in row order; a pivot's panel
// is its slot's parity, so neighbouring pivots, whose ranges share a boundary
// plane, use different panels.
struct InvTask {
  int16_t kind, i0, ni, j0, nj, p0, p1, nrow, ncol, k00, kb0, k01, kb1, pad[3];
};

struct InvStep {
  int task0 = 0, ntask = 0;  // in InvPlan::tasks
};

struct InvPlan {
  int n = 0;
  std::vector<InvTask> tasks;
  std::vector<InvStep> steps;  // steps[0] only prepares the first pivots
  int max_pivots = 0;          // most pivots of one step
  int max_rows = 0;            // most rows of a block
};

// n rows in planes of m rows each.
inline InvPlan make_inv_plan(int n, int m) {
  InvPlan plan;
  plan.n = n;
  // units: planes, or groups of thin planes of 32 to 64 rows
  const int unit = m >= kInvBlock / 2 ? m : m * (kInvBlock / m);
  const int nu = (n + unit - 1) / unit;
  auto row_of = [&](int u) { return std::min(u * unit, n); };
  auto steps_of = [&](int rows) { return (rows + kInvBlock - 1) / kInvBlock; };
  // cost[len]: fewest dependent steps to pivot `len` consecutive units, either
  // as one dense run or split by a separator unit in the middle
  std::vector<int> cost(nu + 1, 0);
  for (int len = 1; len <= nu; ++len) {
    cost[len] = steps_of(len * unit);
    if (len >= 2) {
      const int a = (len - 1) / 2, b = len - 1 - a;
      cost[len] = std::min(cost[len], std::max(cost[a], cost[b]) + steps_of(unit));
    }
  }
  struct Node {
    int r0, r1;   // rows pivoted by this node
    int lo, hi;   // rows coupled with them when they are pivoted
    int start;    // first step
    std::vector<std::pair<int, int>> blk;  // its blocks (k0, kb)
  };
  std::vector<Node> nodes;
  // every node ends just before its parent starts; steps count down from 0
  // (the root's last) and are shifted afterwards
  struct Item {
    int a, b, left, right, end;  // units [a, b), boundary units (-1, nu: none), step after its last
  };
  std::vector<Item> todo{{0, nu, -1, nu, 0}};
  int first = 0;
  while (!todo.empty()) {
    const Item it = todo.back();
    todo.pop_back();
    const int len = it.b - it.a;
    if (len <= 0) continue;
    Node nd;
    const int dense = steps_of(row_of(it.b) - row_of(it.a));
    int sa = it.a, sb = it.b;
    bool split = false;
    if (len >= 2) {
      const int a = (len - 1) / 2, b = len - 1 - a;
      split = std::max(cost[a], cost[b]) + steps_of(unit) <= dense;
      if (split) {
        sa = it.a + a;
        sb = sa + 1;
      }
    }
    nd.r0 = row_of(sa);
    nd.r1 = row_of(sb);
    nd.lo = it.left >= 0 ? row_of(it.left) : 0;
    nd.hi = it.right < nu ? row_of(it.right + 1) : n;
    for (int k = nd.r0; k < nd.r1; k += kInvBlock)
      nd.blk.push_back({k, std::min(kInvBlock, nd.r1 - k)});
    plan.max_rows = std::max(plan.max_rows, std::min(kInvBlock, nd.r1 - nd.r0));
    nd.start = it.end - (int)nd.blk.size();
    first = std::min(first, nd.start);
    if (split) {
      todo.push_back({it.a, sa, it.left, sa, nd.start});
      todo.push_back({sb, it.b, sa, it.right, nd.start});
    }
    nodes.push_back(nd);
  }
  std::sort(nodes.begin(), nodes.end(), [](const Node& a, const Node& b) { return a.r0 < b.r0; });
  std::vector<std::pair<int, int>> blocks;  // all blocks in row order
  for (const Node& nd : nodes) blocks.insert(blocks.end(), nd.blk.begin(), nd.blk.end());
  const int nsteps = -first, nb = (int)blocks.size();
  std::vector<int> seen((size_t)nb * nb);
  auto block_of = [&](int row) {  // index of the block that starts at `row`
    return (int)(std::lower_bound(blocks.begin(), blocks.end(), std::make_pair(row, 0)) - blocks.begin());
  };
  auto active = [&](int s) {  // nodes pivoting in step s, in row order
    std::vector<const Node*> v;
    for (const Node& nd : nodes)
      if (s >= nd.start - first && s < nd.start - first + (int)nd.blk.size()) v.push_back(&nd);
    return v;
  };
  auto block_at = [&](const Node* nd, int s) { return nd->blk[s - (nd->start - first)]; };
  // step -1 prepares the first pivots; step s pivots and prepares step s + 1
  for (int s = -1; s < nsteps; ++s) {
    InvStep st;
    st.task0 = (int)plan.tasks.size();
    const auto cur = s >= 0 ? active(s) : std::vector<const Node*>();
    const auto nxt = s + 1 < nsteps ? active(s + 1) : std::vector<const Node*>();
    plan.max_pivots = std::max(plan.max_pivots, (int)cur.size());
    std::vector<int> next_slot(nb, -1);  // block -> slot of the next step's pivots
    for (int q = 0; q < (int)nxt.size(); ++q)
      next_slot[block_of(block_at(nxt[q], s + 1).first)] = q;
    std::fill(seen.begin(), seen.end(), -1);  // tile -> task
    std::vector<InvTask> heavy, rest;         // tiles that invert a pivot go first
    std::vector<InvTask> tasks;
    for (int q = 0; q < (int)cur.size(); ++q) {
      const auto K = block_at(cur[q], s);
      const int b0 = block_of(cur[q]->lo), b1 = block_of(cur[q]->hi);
      for (int bi = b0; bi < b1; ++bi)
        for (int bj = bi; bj < b1; ++bj) {
          int& f = seen[(size_t)bi * nb + bj];
          if (f >= 0) {  // the boundary plane that two neighbouring pivots share
            tasks[f].p1 = (int16_t)q;
            tasks[f].k01 = (int16_t)K.first;
            tasks[f].kb1 = (int16_t)K.second;
            continue;
          }
          const auto I = blocks[bi], J = blocks[bj];
          InvTask t{};
          t.i0 = (int16_t)I.first;
          t.ni = (int16_t)I.second;
          t.j0 = (int16_t)J.first;
          t.nj = (int16_t)J.second;
          t.p0 = (int16_t)q;
          t.k00 = (int16_t)K.first;
          t.kb0 = (int16_t)K.second;
          t.p1 = -1;
          t.nrow = (int16_t)next_slot[bi];
          t.ncol = (int16_t)next_slot[bj];
          t.kind = I.first == K.first ? (J.first == K.first ? kInvDiag : kInvCrossJ)
                                      : (J.first == K.first ? kInvCrossI : kInvTile);
          f = (int)tasks.size();
          tasks.push_back(t);
        }
    }
    // next pivots that no pivot of this step touches yet: invert and copy from A
    for (const Node* nd : nxt) {
      const auto K = block_at(nd, s + 1);
      InvTask t{};
      t.i0 = t.j0 = (int16_t)K.first;
      t.ni = t.nj = (int16_t)K.second;
      t.p0 = t.p1 = -1;
      const int bk = block_of(K.first);
      t.nrow = t.ncol = (int16_t)next_slot[bk];
      t.kind = kInvTile;
      if (seen[(size_t)bk * nb + bk] < 0) tasks.push_back(t);
      t.kind = kInvPanel;
      const int b1 = block_of(nd->hi);
      for (int bj = block_of(nd->lo); bj < b1; ++bj) {
        if (bj == bk || seen[(size_t)std::min(bj, bk) * nb + std::max(bj, bk)] >= 0) continue;
        t.j0 = (int16_t)blocks[bj].first;
        t.nj = (int16_t)blocks[bj].second;
        tasks.push_back(t);
      }
    }
    for (const InvTask& t : tasks)
      (t.kind == kInvTile && t.i0 == t.j0 && t.nrow >= 0 ? heavy : rest).push_back(t);
    plan.tasks.insert(plan.tasks.end(), heavy.begin(), heavy.end());
    plan.tasks.insert(plan.tasks.end(), rest.begin(), rest.end());
    st.ntask = (int)plan.tasks.size() - st.task0;
    plan.steps.push_back(st);
  }
  return plan;
}

}  // namespace aarmr
