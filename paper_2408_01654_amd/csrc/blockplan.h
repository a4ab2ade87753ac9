// Elimination plan of the large reduced systems (DPV-SLAM Appendix A: the
// Cholesky of the pose block), built on the host from which poses are
// coupled; the kernels that follow it are in sparse.hip.
//
// The poses are ordered by nested dissection on top of a base order (the
// analysis' reverse Cuthill-McKee order, or the poses' own): a list of poses
// is cut in the middle, the poses of one side that touch the other become a
// separator, eliminated after both sides, and the sides are cut again while
// that shortens the chain of dependent steps.  Runs of the order become
// blocks of at most 64 rows that never straddle a separator, so the blocks of
// different parts are eliminated at the same time: what bounds the factor of
// such a system is the number of dependent block steps (levels), not its
// arithmetic.
//
// Storage: every structurally non-zero lower block (I, J), fill included, is
// a dense 64 x 64 array, block columns one after another, each with its
// diagonal block first.  Rows a block does not use are identity rows, so no
// kernel masks sizes.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace dpvba {

constexpr int kBlk = 64;  // rows of a block

// Child column J of a LevelTask (K, I): blocks (K, J) and (I, J) (-1: none).
struct LevelChild {
  int32_t kj, ij, J, pad;
};
// One block of block column K in its level's launch: target block `blk` (the
// diagonal block dblk of `size` used rows, or the block of a row of the
// column), and the columns of the level before that still have to be
// subtracted: child[j0 .. j0 + nj), the first of them here too (a task then
// has its first operands' places with its own record).
struct LevelTask {
  int32_t K, blk, dblk, size, j0, nj, pad[2];
  LevelChild first;
};
// One block (I, J') that the columns of the level before update and that is
// eliminated later: src[s0 .. s0 + ns); row = I for a diagonal block (whose
// right-hand side is updated with it), else -1.
struct UpdateTask {
  int32_t blk, s0, ns, row;
};
// Source column J of an UpdateTask: blocks (I, J) and (J', J).
struct UpdateSrc {
  int32_t ij, jj, J, pad;
};

struct BlockPlan {
  int bw = 0, n_pose = 0, nb = 0;       // rows of a pose, poses, block columns
  std::vector<int32_t> order;           // pose at each place of the elimination order
  std::vector<int32_t> row0;            // per pose: its first row in the padded vectors (64 nb rows)
  std::vector<int32_t> size;            // rows used of each block
  std::vector<int32_t> colptr, rowidx;  // block ids of each column (diagonal first) and their block rows
  std::vector<int32_t> level;
  int n_level = 0;
  // launches: level l's tasks, and the updates that ride along
  std::vector<int32_t> task_off, upd_off;  // [n_level + 1]
  std::vector<LevelTask> tasks;
  std::vector<LevelChild> children;
  std::vector<UpdateTask> updates;
  std::vector<UpdateSrc> srcs;
  // the update of a level whose predecessor is a single column is enumerated
  // by the kernel as the pairs of that column's rows (implicit[l] = the
  // column, else -1), so that a dense system needs no lists of pairs
  std::vector<int32_t> implicit_col;
  // triangular solves: columns by level, and each block row's columns
  // (J, id) by level
  std::vector<int32_t> by_level, rptr, rlist;
  int n_blocks() const { return colptr.empty() ? 0 : colptr.back(); }
  // id of block (I, K), -1 if structurally zero
  int find(int I, int K) const {
    const auto b = rowidx.begin() + colptr[K], e = rowidx.begin() + colptr[K + 1];
    const auto it = std::lower_bound(b, e, I);
    return it != e && *it == I ? (int)(it - rowidx.begin()) : -1;
  }
};

// Nested dissection of `list` (base order).  Appends groups of poses to
// `groups` in elimination order and returns the depth in blocks of at most
// `cap` poses.  where/tag: scratch marks per pose.
inline int dissect(const std::vector<std::vector<int32_t>>& adj, const std::vector<int32_t>& list, int cap,
                   std::vector<int32_t>& where, int32_t& tag, std::vector<std::vector<int32_t>>& groups) {
  const int m = (int)list.size();
  const int leaf = (m + cap - 1) / cap;
  if (leaf > 2) {
    const int32_t t0 = tag;
    tag += m;  // place of list[q] in this call: where = t0 + q
    for (int q = 0; q < m; ++q) where[list[q]] = t0 + q;
    auto place = [&](int v) { const int32_t w = where[v] - t0; return w >= 0 && w < m ? (int)w : -1; };
    // cut before place c: the poses at or after c with a neighbour before it,
    // or the ones before it with a neighbour after; the smaller set separates
    int best_c = 0, best_side = 0;
    size_t best = (size_t)m;
    std::vector<int32_t> lo(m), hi(m);  // least and largest neighbouring place
    for (int q = 0; q < m; ++q) {
      lo[q] = hi[q] = q;
      for (int u : adj[list[q]]) {
        const int w = place(u);
        if (w >= 0) {
          lo[q] = std::min(lo[q], (int32_t)w);
          hi[q] = std::max(hi[q], (int32_t)w);
        }
      }
    }
    for (int e = 3; e <= 5; ++e) {
      const int c = m * e / 8;
      size_t after = 0, before = 0;
      for (int q = c; q < m; ++q) after += lo[q] < c;
      for (int q = 0; q < c; ++q) before += hi[q] >= c;
      const size_t s = std::min(after, before);
      if (s < best || (s == best && e == 4)) {
        best = s;
        best_c = c;
        best_side = after <= before ? 1 : 0;
      }
    }
    if (best * 3 <= (size_t)m) {
      std::vector<int32_t> a, b, s;
      for (int q = 0; q < m; ++q) {
        const bool sep = best_side ? q >= best_c && lo[q] < best_c : q < best_c && hi[q] >= best_c;
        (sep ? s : (q < best_c ? a : b)).push_back(list[q]);
      }
      if (!a.empty() && !b.empty()) {
        std::vector<std::vector<int32_t>> g;
        const int da = dissect(adj, a, cap, where, tag, g), db = dissect(adj, b, cap, where, tag, g);
        const int d = std::max(da, db) + (int)((s.size() + cap - 1) / cap);
        if (d < leaf) {
          if (!s.empty()) g.push_back(s);
          for (auto& x : g) groups.push_back(std::move(x));
          return d;
        }
      }
    }
  }
  groups.push_back(list);
  return leaf;
}

// Plan of a system of adj.size() poses of bw rows each.  base: the base order;
// split: dissect it (else the blocks are eliminated one after another in the
// base order).
inline BlockPlan build_block_plan(const std::vector<std::vector<int32_t>>& adj, const std::vector<int32_t>& base,
                                  int bw, bool split) {
  constexpr size_t kMaxListed = (size_t)1 << 21;  // update pairs listed at most (beyond: no dissection)
  BlockPlan p;
  p.bw = bw;
  p.n_pose = (int)adj.size();
  const int cap = kBlk / bw;
  std::vector<std::vector<int32_t>> groups;
  if (split) {
    std::vector<int32_t> where(adj.size(), -1);
    int32_t tag = 0;
    dissect(adj, base, cap, where, tag, groups);
  } else {
    groups.push_back(base);
  }
  const bool chain = groups.size() == 1;  // one run: no independent parts to look for
  std::vector<int32_t> blk(adj.size());
  p.row0.assign(adj.size(), 0);
  for (const auto& g : groups) {
    const int m = (int)g.size(), k = (m + cap - 1) / cap;
    for (int q = 0; q < k; ++q) {
      const int a = (int)((long long)m * q / k), b = (int)((long long)m * (q + 1) / k);
      for (int x = a; x < b; ++x) {
        blk[g[x]] = p.nb;
        p.row0[g[x]] = kBlk * p.nb + bw * (x - a);
        p.order.push_back(g[x]);
      }
      p.size.push_back(bw * (b - a));
      ++p.nb;
    }
  }
  const int nb = p.nb;
  // structure: the coupled blocks, then the fill (a column's rows below its
  // first one are rows of that one's column too)
  std::vector<std::vector<int32_t>> st(nb);
  for (size_t v = 0; v < adj.size(); ++v)
    for (int u : adj[v])
      if (blk[u] > blk[v]) st[blk[v]].push_back(blk[u]);
  p.colptr.assign(1, 0);
  for (int K = 0; K < nb; ++K) {
    auto& s = st[K];
    std::sort(s.begin(), s.end());
    s.erase(std::unique(s.begin(), s.end()), s.end());
    if (s.size() > 1) st[s[0]].insert(st[s[0]].end(), s.begin() + 1, s.end());
    p.rowidx.push_back(K);
    p.rowidx.insert(p.rowidx.end(), s.begin(), s.end());
    p.colptr.push_back((int32_t)p.rowidx.size());
  }
  // levels: one past the deepest column that updates this one; a single run
  // is a chain of its own (every column after the one before)
  p.level.assign(nb, 0);
  for (int K = 0; K < nb; ++K) {
    if (chain) p.level[K] = K;
    for (int q = p.colptr[K] + 1; q < p.colptr[K + 1]; ++q)
      p.level[p.rowidx[q]] = std::max(p.level[p.rowidx[q]], p.level[K] + 1);
  }
  p.n_level = 0;
  for (int K = 0; K < nb; ++K) p.n_level = std::max(p.n_level, p.level[K] + 1);
  std::vector<std::vector<int32_t>> cols(p.n_level);
  for (int K = 0; K < nb; ++K) cols[p.level[K]].push_back(K);
  for (const auto& c : cols) p.by_level.insert(p.by_level.end(), c.begin(), c.end());
  std::vector<std::vector<int32_t>> rows(nb);  // per block row: (J, id), by level
  for (int J : p.by_level)
    for (int q = p.colptr[J] + 1; q < p.colptr[J + 1]; ++q) {
      rows[p.rowidx[q]].push_back(J);
      rows[p.rowidx[q]].push_back(q);
    }
  p.rptr.assign(1, 0);
  for (int K = 0; K < nb; ++K) {
    p.rlist.insert(p.rlist.end(), rows[K].begin(), rows[K].end());
    p.rptr.push_back((int32_t)(p.rlist.size() / 2));
  }
  // tasks
  p.task_off.assign(1, 0);
  p.upd_off.assign(1, 0);
  p.implicit_col.assign(p.n_level, -1);
  size_t listed = 0;
  for (int l = 0; l < p.n_level; ++l) {
    for (int K : cols[l]) {
      std::vector<int32_t> kids;  // (J, id of (K, J)) of the level before
      for (size_t q = 0; q < rows[K].size(); q += 2)
        if (p.level[rows[K][q]] == l - 1) {
          kids.push_back(rows[K][q]);
          kids.push_back(rows[K][q + 1]);
        }
      for (int q = p.colptr[K]; q < p.colptr[K + 1]; ++q) {
        LevelTask t{K, q, p.colptr[K], p.size[K], (int32_t)p.children.size(), (int32_t)(kids.size() / 2), {0, 0}, {-1, -1, -1, 0}};
        for (size_t x = 0; x < kids.size(); x += 2)
          p.children.push_back(LevelChild{kids[x + 1], p.find(p.rowidx[q], kids[x]), kids[x], 0});
        if (t.nj) t.first = p.children[t.j0];
        p.tasks.push_back(t);
      }
    }
    p.task_off.push_back((int32_t)p.tasks.size());
    if (l > 0 && cols[l - 1].size() == 1) {
      p.implicit_col[l] = cols[l - 1][0];
    } else if (l > 0) {
      struct Pair { int32_t tgt, row; UpdateSrc s; };
      std::vector<Pair> v;
      for (int J : cols[l - 1]) {
        const int c0 = p.colptr[J] + 1, c1 = p.colptr[J + 1];
        listed += (size_t)(c1 - c0) * (c1 - c0 + 1) / 2;
        if (listed > kMaxListed) return build_block_plan(adj, base, bw, false);
        for (int b = c0; b < c1; ++b) {
          if (p.level[p.rowidx[b]] <= l) continue;  // eliminated by this launch
          for (int a = b; a < c1; ++a)
            v.push_back(Pair{p.find(p.rowidx[a], p.rowidx[b]), a == b ? p.rowidx[a] : -1, UpdateSrc{a, b, J, 0}});
        }
      }
      std::stable_sort(v.begin(), v.end(), [](const Pair& x, const Pair& y) { return x.tgt < y.tgt; });
      for (size_t q = 0; q < v.size(); ++q) {
        if (q == 0 || v[q].tgt != v[q - 1].tgt) p.updates.push_back(UpdateTask{v[q].tgt, (int32_t)p.srcs.size(), 0, v[q].row});
        ++p.updates.back().ns;
        p.srcs.push_back(v[q].s);
      }
    }
    p.upd_off.push_back((int32_t)p.updates.size());
  }
  return p;
}

}  // namespace dpvba
