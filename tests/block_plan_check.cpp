// Executes a block elimination plan (csrc/blockplan.h) on the host in float64,
// launch by launch, with every read taken from the state before the launch
// (so a task that needed a value of its own launch would fail), and compares the
// solution with the system's residual.  Usage: prog; one line per plan, exit
// status 1 on a failure.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>

#include "blockplan.h"

using namespace dpvba;
typedef std::vector<double> V;

static int fail(const char* what) {
  std::printf("FAILED: %s\n", what);
  return 1;
}

static void mul_sub(V& t, const V& x, const V& y) {  // t -= x y^T
  for (int r = 0; r < 64; ++r)
    for (int c = 0; c < 64; ++c) {
      double s = 0;
      for (int k = 0; k < 64; ++k) s += x[r * 64 + k] * y[c * 64 + k];
      t[r * 64 + c] -= s;
    }
}

static int check(const std::vector<std::vector<int32_t>>& adj, const std::vector<int32_t>& base, int bw, bool split,
                 std::mt19937& gen, const char* name) {
  auto uni = [&]() { return std::uniform_real_distribution<double>(-0.5, 0.5)(gen); };
  const BlockPlan p = build_block_plan(adj, base, bw, split);
  const int n = (int)adj.size(), N = 64 * p.nb;
  std::vector<char> used(N, 0);
  for (int v = 0; v < n; ++v)
    for (int r = 0; r < bw; ++r) {
      if (p.row0[v] % 64 + bw > p.size[p.row0[v] / 64] || used[p.row0[v] + r]) return fail("row of a pose");
      used[p.row0[v] + r] = 1;
    }
  V D((size_t)N * N, 0.0), b(N, 0.0), x(N, 0.0);
  for (int r = 0; r < N; ++r) D[(size_t)r * N + r] = 1.0;
  auto set = [&](int r, int c, double a) { D[(size_t)r * N + c] = D[(size_t)c * N + r] = a; };
  for (int v = 0; v < n; ++v)
    for (int r = 0; r < bw; ++r) {
      b[p.row0[v] + r] = uni();
      for (int c = 0; c <= r; ++c) set(p.row0[v] + r, p.row0[v] + c, uni() + (r == c ? 60 + 6.0 * adj[v].size() : 0.0));
      for (int u : adj[v])
        if (u < v)
          for (int c = 0; c < bw; ++c) set(p.row0[v] + r, p.row0[u] + c, uni());
    }
  std::vector<V> A(p.n_blocks(), V(4096)), Li(p.nb, V(4096, 0.0));
  long long outside = 0;
  for (double a : D) outside += a != 0.0;
  for (int K = 0; K < p.nb; ++K)
    for (int q = p.colptr[K]; q < p.colptr[K + 1]; ++q)
      for (int r = 0; r < 64; ++r)
        for (int c = 0; c < 64; ++c) {
          const double a = D[(size_t)(64 * p.rowidx[q] + r) * N + 64 * K + c];
          A[q][r * 64 + c] = a;
          outside -= a != 0.0 ? (p.rowidx[q] == K ? 1 : 2) : 0;
        }
  if (outside) return fail("an entry outside the plan's blocks");
  V v = b;
  for (int l = 0; l < p.n_level; ++l) {
    const std::vector<V> A0 = A;
    const V v0 = v;
    for (int t = p.task_off[l]; t < p.task_off[l + 1]; ++t) {
      const LevelTask& T = p.tasks[t];
      if (p.level[T.K] != l) return fail("task's level");
      V d = A0[p.colptr[T.K]], m = A0[T.blk], rb(v0.begin() + 64 * T.K, v0.begin() + 64 * T.K + 64);
      for (int j = T.j0; j < T.j0 + T.nj; ++j) {
        const LevelChild& c = p.children[j];
        if (p.rowidx[c.kj] != T.K || (c.ij >= 0 && p.rowidx[c.ij] != p.rowidx[T.blk])) return fail("child's blocks");
        mul_sub(d, A0[c.kj], A0[c.kj]);
        if (c.ij >= 0) mul_sub(m, A0[c.ij], A0[c.kj]);
        for (int r = 0; r < 64; ++r)
          for (int k = 0; k < 64; ++k) rb[r] -= A0[c.kj][r * 64 + k] * v0[64 * c.J + k];
      }
      V L(4096, 0.0), inv(4096, 0.0);
      for (int c = 0; c < 64; ++c)
        for (int r = c; r < 64; ++r) {
          double s = d[r * 64 + c];
          for (int k = 0; k < c; ++k) s -= L[r * 64 + k] * L[c * 64 + k];
          if (r == c && !(s > 0)) return fail("not positive definite");
          L[r * 64 + c] = r == c ? std::sqrt(s) : s / L[c * 64 + c];
        }
      for (int c = 0; c < 64; ++c)
        for (int r = c; r < 64; ++r) {
          double s = r == c;
          for (int k = c; k < r; ++k) s -= L[r * 64 + k] * inv[k * 64 + c];
          inv[r * 64 + c] = s / L[r * 64 + r];
        }
      if (T.blk == p.colptr[T.K]) {
        Li[T.K] = inv;
        for (int r = 0; r < 64; ++r) {
          double s = 0;
          for (int k = 0; k <= r; ++k) s += inv[r * 64 + k] * rb[k];
          v[64 * T.K + r] = s;
        }
      } else {
        for (int r = 0; r < 64; ++r)
          for (int c = 0; c < 64; ++c) {
            double s = 0;
            for (int k = 0; k <= c; ++k) s += m[r * 64 + k] * inv[c * 64 + k];
            A[T.blk][r * 64 + c] = s;
          }
      }
    }
    if (l == 0) continue;
    std::vector<char> seen(p.n_blocks(), 0);
    auto update = [&](int blk, int row, const UpdateSrc* s, int ns) {
      if (blk < 0 || seen[blk]) return false;
      seen[blk] = 1;
      for (int q = 0; q < ns; ++q) {
        mul_sub(A[blk], A0[s[q].ij], A0[s[q].jj]);
        if (row >= 0)
          for (int r = 0; r < 64; ++r)
            for (int k = 0; k < 64; ++k) v[64 * row + r] -= A0[s[q].ij][r * 64 + k] * v0[64 * s[q].J + k];
      }
      return true;
    };
    if (p.implicit_col[l] >= 0) {
      const int J = p.implicit_col[l], c0 = p.colptr[J] + 1, c1 = p.colptr[J + 1];
      for (int q = c0; q < c1; ++q)
        for (int a = q; a < c1 && p.level[p.rowidx[q]] > l; ++a) {
          const UpdateSrc s{a, q, J, 0};
          if (!update(p.find(p.rowidx[a], p.rowidx[q]), a == q ? p.rowidx[a] : -1, &s, 1)) return fail("pair");
        }
    }
    for (int u = p.upd_off[l]; u < p.upd_off[l + 1]; ++u)
      if (!update(p.updates[u].blk, p.updates[u].row, &p.srcs[p.updates[u].s0], p.updates[u].ns)) return fail("update");
  }
  for (int q = p.nb - 1; q >= 0; --q) {
    const int K = p.by_level[q];
    V a(v.begin() + 64 * K, v.begin() + 64 * K + 64);
    for (int id = p.colptr[K] + 1; id < p.colptr[K + 1]; ++id)
      for (int c = 0; c < 64; ++c)
        for (int r = 0; r < 64; ++r) a[c] -= A[id][r * 64 + c] * x[64 * p.rowidx[id] + r];
    for (int c = 0; c < 64; ++c)
      for (int r = c; r < 64; ++r) x[64 * K + c] += Li[K][r * 64 + c] * a[r];
  }
  // forward by the row lists gives the factor's own y
  V y(N, 0.0);
  for (int q = 0; q < p.nb; ++q) {
    const int K = p.by_level[q];
    V a(b.begin() + 64 * K, b.begin() + 64 * K + 64);
    for (int e = p.rptr[K]; e < p.rptr[K + 1]; ++e)
      for (int r = 0; r < 64; ++r)
        for (int k = 0; k < 64; ++k) a[r] -= A[p.rlist[2 * e + 1]][r * 64 + k] * y[64 * p.rlist[2 * e] + k];
    for (int r = 0; r < 64; ++r)
      for (int k = 0; k <= r; ++k) y[64 * K + r] += Li[K][r * 64 + k] * a[k];
  }
  double err = 0, dy = 0;
  for (int r = 0; r < N; ++r) {
    double s = b[r];
    for (int c = 0; c < N; ++c) s -= D[(size_t)r * N + c] * x[c];
    err = std::max(err, std::fabs(s));
    dy = std::max(dy, std::fabs(y[r] - v[r]));
  }
  std::printf("%s poses %d rows %d split %d blocks %d levels %d residual %.2e\n", name, n, bw, (int)split, p.nb,
              p.n_level, err);
  return err < 1e-12 && dy < 1e-12 ? 0 : fail("residual");
}

int main() {
  std::mt19937 gen(1);
  const char* names[] = {"path", "band", "dense", "band+loops", "wide band", "pieces", "star", "edgeless"};
  for (int kind = 0; kind < 8; ++kind)
    for (int n : {1, 9, 10, 11, 41, 63, 120}) {
      std::vector<std::vector<int32_t>> adj(n);
      auto couple = [&](int a, int b) {
        if (a == b || a >= n || b >= n) return;
        adj[a].push_back(b);
        adj[b].push_back(a);
      };
      const int w = kind == 0 ? 1 : kind == 1 ? 5 : kind == 2 ? n : kind == 3 ? 3 : kind == 4 ? 8 : kind == 5 ? 2 : 0;
      for (int i = 0; i < n; ++i)
        for (int d = 1; d <= w; ++d)
          if (kind != 5 || (i % 17) + d < 17) couple(i, i + d);
      if (kind == 3)
        for (int q = 0; q < 4; ++q) couple((int)(gen() % n), (int)(gen() % n));
      if (kind == 6)
        for (int i = 1; i < n; ++i) couple(0, i);
      for (auto& a : adj) {
        std::sort(a.begin(), a.end());
        a.erase(std::unique(a.begin(), a.end()), a.end());
      }
      std::vector<int32_t> base(n);
      for (int i = 0; i < n; ++i) base[i] = i;
      if (n == 63) std::shuffle(base.begin(), base.end(), gen);
      for (int split = 0; split < 2; ++split)
        if (check(adj, base, kind % 2 ? 6 : 7, split, gen, names[kind])) return 1;
    }
  return 0;
}
