// Block-sparse Cholesky of the large reduced systems (DPV-SLAM Appendix A),
// following an elimination plan (blockplan.h): dense 64 x 64 blocks, one
// launch per level of block columns that do not depend on each other.
//
// A launch holds two kinds of workgroups, none of which waits for another:
//  * level tasks, one per non-zero block (I, K) of the level's columns: the
//    workgroup subtracts what the columns of the level before still owe
//    (A_KK - sum L_KJ L_KJ^T and A_IK - sum L_IJ L_KJ^T), factors the diagonal block
//    itself and forms L_IK = A_IK L_KK^-T.  Every block of a column repeats
//    the column's diagonal factor: the chip has CUs to spare at every level,
//    and a factor computed where it is used needs no second launch and no
//    publication;
//  * update tasks, one per block that is eliminated later: subtract the
//    products of the columns of the level before.
// The chain per level is one launch: loads, the diagonal block's update, four
// 16-column panels, one product; two dependent round trips to memory and the
// panels' pivot chain are what bounds it.  On 1000 keyframes with loop closures
// (5,994 unknowns) an iteration's factor and solve take 26 launches of 11.5 us
// and one of 35 us, against 94 dependent pairs of launches (10.4 + 5.5 us) and a
// triangular chain of 118 us when the blocks were eliminated one after another:
// 9.09 -> 2.43 ms for five iterations.  A Sim(3) pose graph of 1000 keyframes
// (float64) takes 8 levels of 13.8 us instead of 109 pairs of 22.4 + 5.0 us:
// 36.1 -> 2.1 ms for ten iterations.
//
// Blocks are staged in LDS by the whole workgroup (16 bytes a thread,
// coalesced) and the matrix-core operands read from there: straight from
// memory every wavefront loaded its own strips, three to six times a block
// (13.7 us a level in float32, 19.6 us in float64).
#include <algorithm>
#include <cfloat>

#include "common.h"
#include "mfma.h"
#include "packed.h"
#include "sparse.h"

namespace dpvba {

constexpr int kBB = kBlk * kBlk;
constexpr int kLevelThreads = 512;

// row stride of a staged block and of the diagonal factor's working matrix:
// 16-byte rows, and 16-row operand reads on different LDS banks
template <typename T>
__host__ __device__ constexpr int staged_ld() { return sizeof(T) == 4 ? kBlk + 4 : kBlk + 2; }

template <typename T>
__host__ __device__ constexpr int level_lds_elems() {
  return 4 * kBlk * staged_ld<T>() + kBlk + 8 * kBlk;
}

// A block on its way from memory to LDS: 16-byte vectors of 512 threads.
template <typename T>
struct Stage {
  static constexpr int V = 16 / (int)sizeof(T), N = kBB / V / kLevelThreads;
  typename V16<T>::type x[N];
  __device__ __forceinline__ void load(const T* blk) {
    const typename V16<T>::type* p = reinterpret_cast<const typename V16<T>::type*>(blk) + threadIdx.x;
#pragma unroll
    for (int u = 0; u < N; ++u) x[u] = p[u * kLevelThreads];
  }
  __device__ __forceinline__ void store(T* lds) const {
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int q = (int)threadIdx.x + u * kLevelThreads, r = q / (kBlk / V), c = V * (q % (kBlk / V));
      *reinterpret_cast<typename V16<T>::type*>(lds + r * staged_ld<T>() + c) = x[u];
    }
  }
};

// acc += X Y^T for rows rx .. of X and ry .. of Y (staged blocks).  A lane reads
// 16 bytes of its row, the operands of four (two) product steps at once: the
// steps take the columns in another order, the same one for X and Y.
template <typename T>
__device__ __forceinline__ typename Mfma<T>::acc_t staged_mma(const T* X, int rx, const T* Y, int ry,
                                                              typename Mfma<T>::acc_t acc) {
  constexpr int ld = staged_ld<T>(), V = 16 / (int)sizeof(T);
  typedef typename V16<T>::type vec_t;
  const int lane = threadIdx.x & 63;
  const T* x = X + (rx + (lane & 15)) * ld + V * (lane >> 4);
  const T* y = Y + (ry + (lane & 15)) * ld + V * (lane >> 4);
#pragma unroll
  for (int k = 0; k < kBlk; k += 4 * V) {
    const vec_t a = *reinterpret_cast<const vec_t*>(x + k), b = *reinterpret_cast<const vec_t*>(y + k);
#pragma unroll
    for (int u = 0; u < V; ++u) acc = Mfma<T>::step(a[u], b[u], acc);
  }
  return acc;
}

// Rank-16 update of the working matrix by panel p: the 16 x 16 blocks (bi, bk), bk =
// bk_lo .. bk_hi, bi = bk .. 4 + p (the rows whose panel-p entries can be non-zero),
// go to the wavefronts first, first + nwav, ...: W_(bi,bk) -= W_(bi,p) W_(bk,p)^T.
template <typename T>
__device__ __forceinline__ void diag_update_blocks(T* W, int p, int bk_lo, int bk_hi, int first, int nwav) {
  constexpr int kLd = staged_ld<T>();
  const int lane = threadIdx.x & 63, c0 = 16 * p;
  int count = 0;
  for (int bk = bk_lo; bk <= bk_hi; ++bk) count += 5 + p - bk;
  for (int q = first; q < count; q += nwav) {
    int bk = bk_lo, rem = q;
    while (rem >= 5 + p - bk) {
      rem -= 5 + p - bk;
      ++bk;
    }
    const int bi = bk + rem;
    const T* xr = W + (16 * bi + (lane & 15)) * kLd + c0 + (lane >> 4);
    const T* yr = W + (16 * bk + (lane & 15)) * kLd + c0 + (lane >> 4);
    T* out = W + 16 * bi * kLd + 16 * bk + (lane & 15);
    T old[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) old[v] = out[Mfma<T>::row(lane, v) * kLd];
    typename Mfma<T>::acc_t acc = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 16; k += 4) acc = Mfma<T>::step(xr[k], yr[k], acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) out[Mfma<T>::row(lane, v) * kLd] = old[v] - acc[v];
  }
}

// Panel p (16 columns) of the diagonal block's factor on one wavefront.  The
// block is factored together with an identity appended below it: the factor
// of [[A, I], [I, .]] has L^-T in its lower-left block, so one elimination
// gives both L and its inverse (128 x 64 working matrix W).  Lane l holds
// row l mod 16 of the 16 x 16 diagonal block (ra: each 16-lane row of the
// wavefront a full copy) and one row of the panel below it (rb: lane row q
// takes row block q of the four that can be non-zero -- the A rows of the later
// blocks, the identity rows of the earlier panels and of this one; the
// identity rows of later panels are still zero in this column block).
// Column entries travel by the DPP row broadcast inside the multiply-adds
// (chol16), so the chain of 16 pivots takes no scalar registers and no barrier.
template <typename T>
__device__ __forceinline__ void diag_panel(T* W, int p, int& bad) {
  constexpr int kLd = staged_ld<T>();
  const int lane = threadIdx.x & 63, s = lane & 15, q = lane >> 4, c0 = 16 * p;
  const int bq = q < 3 - p ? p + 1 + q : 4 + (q - (3 - p));
  T* wa = W + (c0 + s) * kLd + c0;
  T* wb = W + (16 * bq + s) * kLd + c0;
  T ra[16], rb[16];
  get_row<T, 16>(wa, ra);
  get_row<T, 16>(wb, rb);
  chol16<T>(ra, rb, bad);
  // (the stores that depend on the lane come last: a branch here would sink
  // the rows' updates below it)
  put_row<T, 16>(wb, rb);
  if (q == 0) put_row<T, 16>(wa, ra);
}

// One launch of the factor: workgroups [0, n_task) are the level's tasks,
// the rest its updates (listed, or the pairs of rows of column impl).
// float32: two workgroups per CU (128 registers, 70 KB of LDS), for the
// updates; float64 holds one (139 KB).
template <typename T>
__global__ void __launch_bounds__(kLevelThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
sparse_level_kernel(T* A, T* Linv, T* v, const T* d0, SparsePlan P, const LevelTask* tasks, int n_task,
                    const UpdateTask* updates, int impl, int lev, int* status, unsigned int* min_bits) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  constexpr int ldM = staged_ld<T>(), kLd = ldM;
  T* sM = reinterpret_cast<T*>(dyn_lds);  // staged block of row I, then A_IK
  T* sK = sM + kBlk * staged_ld<T>();     // staged block of row K
  T* W = sK + kBlk * staged_ld<T>();      // 128 x 64
  T* sb = W + 2 * kBlk * kLd;             // 64: the column's right-hand side
  T* part = sb + kBlk;                    // 8 x 64 partial sums
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  typedef typename Mfma<T>::acc_t acc_t;
  const acc_t zero = {0, 0, 0, 0};
  if ((int)blockIdx.x >= n_task) {
    // ---- update of a block that is eliminated by a later launch
    const int u = blockIdx.x - n_task;
    int blk, ns, row;
    UpdateSrc one{0, 0, 0, 0};
    const UpdateSrc* src = nullptr;
    if (impl < 0) {
      const UpdateTask t = updates[u];
      blk = t.blk;
      ns = t.ns;
      row = t.row;
      src = P.srcs + t.s0;
      one = src[0];
    } else {  // pair a >= b of the column's rows
      int a = (int)((sqrtf(8.0f * (float)u + 1.0f) - 1.0f) * 0.5f);
      while (a * (a + 1) / 2 > u) --a;
      while ((a + 1) * (a + 2) / 2 <= u) ++a;
      const int b = u - a * (a + 1) / 2, c0 = P.colptr[impl] + 1;
      const int I = P.rowidx[c0 + a], J = P.rowidx[c0 + b];
      if (P.level[J] <= lev) return;  // a task of this launch
      int lo = P.colptr[J], hi = P.colptr[J + 1] - 1;  // block (I, J): I is one of column J's rows
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (P.rowidx[mid] < I) lo = mid + 1;
        else hi = mid;
      }
      blk = lo;
      ns = 1;
      row = a == b ? I : -1;
      one = UpdateSrc{c0 + a, c0 + b, impl, 0};
    }
    T* tgt = A + (size_t)blk * kBB;
    const int tr = w & 3, tc0 = 2 * (w >> 2);  // 16-row strip tr, column tiles tc0 and tc0 + 1
    const bool diag = row >= 0;                // only its lower 16 x 16 tiles, and one operand block
    const bool on0 = !diag || tc0 <= tr, on1 = !diag || tc0 + 1 <= tr;
    acc_t acc0 = zero, acc1 = zero;
    T bsum = (T)0;
    T old[8];  // the target's own entries
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const T* d = tgt + (16 * tr + Mfma<T>::row(lane, m)) * kBlk + (lane & 15);
      old[m] = on0 ? d[16 * tc0] : (T)0;
      old[4 + m] = on1 ? d[16 * (tc0 + 1)] : (T)0;
    }
    Stage<T> gx, gy;
    gx.load(A + (size_t)one.ij * kBB);
    if (!diag) gy.load(A + (size_t)one.jj * kBB);
    for (int x = 0; x < ns; ++x) {
      const int J = one.J;
      if (x) __syncthreads();  // the blocks before are still read
      gx.store(sM);
      if (!diag) gy.store(sK);
      __syncthreads();
      if (x + 1 < ns) {  // the next source's blocks load beside this one's products
        one = src[x + 1];
        gx.load(A + (size_t)one.ij * kBB);
        if (!diag) gy.load(A + (size_t)one.jj * kBB);
      }
      const T* Y = diag ? sM : sK;
      if (on0) acc0 = staged_mma<T>(sM, 16 * tr, Y, 16 * tc0, acc0);
      if (on1) acc1 = staged_mma<T>(sM, 16 * tr, Y, 16 * (tc0 + 1), acc1);
      if (diag) {  // row lane, columns 8 w ..
        const T* xr = sM + lane * ldM + 8 * w;
        const T* y = v + kBlk * J + 8 * w;
#pragma unroll
        for (int m = 0; m < 8; ++m) bsum += xr[m] * y[m];
      }
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      T* d = tgt + (16 * tr + Mfma<T>::row(lane, m)) * kBlk + (lane & 15);
      if (on0) d[16 * tc0] = old[m] - acc0[m];
      if (on1) d[16 * (tc0 + 1)] = old[4 + m] - acc1[m];
    }
    if (diag) {
      part[kBlk * w + lane] = bsum;
      __syncthreads();
      if (tid < kBlk) {
        T s = (T)0;
#pragma unroll
        for (int m = 0; m < 8; ++m) s += part[kBlk * m + tid];
        v[kBlk * row + tid] -= s;
      }
    }
    return;
  }

  // ---- task (I, K)
  const LevelTask t = tasks[blockIdx.x];
  const int K = t.K, size = t.size;
  const bool is_diag = t.blk == t.dblk;
  const int np = (size + 15) >> 4;  // panels with a used column (the rest of the block is identity)
  T* tgt = A + (size_t)t.blk * kBB;
  if (w == 0) __builtin_amdgcn_s_setprio(3);
  // everything that the task reads starts to load at once: the first child's
  // blocks, the diagonal block (its ten lower 16 x 16 tiles: one a wavefront,
  // a second on wavefronts 2 and 3) and A_IK (wavefronts 4..7: 16 rows each)
  Stage<T> gk, gi;
  bool has_i = !is_diag && t.nj > 0 && t.first.ij >= 0;
  if (t.nj > 0) gk.load(A + (size_t)t.first.kj * kBB);
  if (has_i) gi.load(A + (size_t)t.first.ij * kBB);
  const int r0m = 16 * (w & 3);
  const int nt = w == 2 || w == 3 ? 2 : 1;
  // tiles 0 .. 9 by rows: (0,0) (1,0) (1,1) (2,0) (2,1) (2,2) (3,0) .. (3,3)
  const int ti0 = w < 1 ? 0 : (w < 3 ? 1 : (w < 6 ? 2 : 3)), tj0 = w - ti0 * (ti0 + 1) / 2;
  auto ti = [&](int h) { return h ? 3 : ti0; };
  auto tj = [&](int h) { return h ? w : tj0; };
  T own[16], dk[8];
  {
    const T* DK = A + (size_t)t.dblk * kBB;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int m = 0; m < 4; ++m)
        dk[4 * h + m] = h < nt ? DK[(16 * ti(h) + Mfma<T>::row(lane, m)) * kBlk + 16 * tj(h) + (lane & 15)] : (T)0;
  }
  if (w >= 4 && !is_diag) {
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int m = 0; m < 4; ++m)
        own[4 * h + m] = tgt[(r0m + Mfma<T>::row(lane, m)) * kBlk + 16 * h + (lane & 15)];
  }
  {  // identity half of W
    const int r = tid >> 3, c0 = 8 * (tid & 7);
    T* wr = W + (kBlk + r) * kLd + c0;
#pragma unroll
    for (int c = 0; c < 8; ++c) wr[c] = (T)(c0 + c == r ? 1 : 0);
  }
  acc_t acc[4] = {zero, zero, zero, zero}, dacc[2] = {zero, zero};
  T bsum = (T)0;
  int J = t.first.J;
  // A_IK's (or, for the diagonal block's task, the right-hand side's) share of
  // the staged child, on wavefronts 4..7
  auto row_share = [&]() {
    if (!is_diag) {
      if (has_i) {
#pragma unroll
        for (int h = 0; h < 4; ++h) acc[h] = staged_mma<T>(sM, r0m, sK, 16 * h, acc[h]);
      }
    } else {
      const T* xr = sK + lane * ldM + r0m;
      const T* y = v + kBlk * J + r0m;
#pragma unroll
      for (int m = 0; m < 16; ++m) bsum += xr[m] * y[m];
    }
  };
  for (int j = 0; j < t.nj; ++j) {
    if (j) {  // rare: a column with several children of the level before
      if (w >= 4) row_share();
      const LevelChild ch = P.children[t.j0 + j];
      has_i = !is_diag && ch.ij >= 0;
      J = ch.J;
      gk.load(A + (size_t)ch.kj * kBB);
      if (has_i) gi.load(A + (size_t)ch.ij * kBB);
      __syncthreads();
    }
    gk.store(sK);
    if (has_i) gi.store(sM);
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (h < nt) dacc[h] = staged_mma<T>(sK, 16 * ti(h), sK, 16 * tj(h), dacc[h]);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if (h < nt) {
#pragma unroll
      for (int m = 0; m < 4; ++m)
        W[(16 * ti(h) + Mfma<T>::row(lane, m)) * kLd + 16 * tj(h) + (lane & 15)] = dk[4 * h + m] - dacc[h][m];
    }
  __syncthreads();
  int bad = 0;
  for (int p = 0; p < np; ++p) {
    if (w == 0) {
      diag_panel<T>(W, p, bad);
    } else if (w < 4) {
      // meanwhile wavefronts 1..3 finish panel p - 1: its update of the later column blocks
      if (p > 0) diag_update_blocks<T>(W, p - 1, p + 1, np - 1, w - 1, 3);
    } else if (p == 0) {
      // and wavefronts 4..7 finish A_IK less what the level before owes it (in
      // place of the rows of the staged block that only they read), or the
      // right-hand side's share
      if (t.nj > 0) row_share();
      if (!is_diag) {
#pragma unroll
        for (int h = 0; h < 4; ++h)
#pragma unroll
          for (int m = 0; m < 4; ++m)
            sM[(r0m + Mfma<T>::row(lane, m)) * ldM + 16 * h + (lane & 15)] = own[4 * h + m] - acc[h][m];
      } else {
        part[kBlk * (w - 4) + lane] = bsum;
      }
    }
    __syncthreads();
    // what the next panel needs first: column block p + 1 updated by this panel
    if (p + 1 < np) diag_update_blocks<T>(W, p, p + 1, p + 1, w, 8);
    __syncthreads();
  }
  if (!is_diag) {
    // L_IK = A_IK L_KK^-T: 16-row strip w mod 4, two column tiles with 20
    // product steps together (L_KK^-1 is lower triangular)
    const int r0 = 16 * (w & 3);
    const T* xr = sM + (r0 + (lane & 15)) * ldM + (lane >> 4);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int tj = w < 4 ? 3 * h : 1 + h;
      const T* yr = W + (kBlk + (lane >> 4)) * kLd + 16 * tj + (lane & 15);
      acc_t acc = zero;
#pragma unroll 4
      for (int s = 0; s < 4 * (tj + 1); ++s) acc = Mfma<T>::step(xr[4 * s], yr[4 * s * kLd], acc);
#pragma unroll
      for (int m = 0; m < 4; ++m) tgt[(r0 + Mfma<T>::row(lane, m)) * kBlk + 16 * tj + (lane & 15)] = acc[m];
    }
    return;
  }
  // the diagonal block's task keeps L_KK^-1 (entry (r, c) at W[64 + c][r]) and
  // y_K = L_KK^-1 (right-hand side)
  T* Lk = Linv + (size_t)K * kBB;
  for (int e = tid; e < kBB; e += kLevelThreads) {
    const int r = e >> 6, c = e & 63;
    Lk[e] = r >= c ? W[(kBlk + c) * kLd + r] : (T)0;
  }
  if (tid < kBlk)
    sb[tid] = v[kBlk * K + tid] - ((part[tid] + part[kBlk + tid]) + (part[2 * kBlk + tid] + part[3 * kBlk + tid]));
  __syncthreads();
  {
    T s = (T)0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int c = 8 * w + m;
      s += (lane >= c ? W[(kBlk + c) * kLd + lane] : (T)0) * sb[c];
    }
    part[kBlk * w + lane] = s;
  }
  __syncthreads();
  if (tid < kBlk) {
    T s = (T)0;
#pragma unroll
    for (int m = 0; m < 8; ++m) s += part[kBlk * m + tid];
    v[kBlk * K + tid] = s;
  }
  if (w == 0) {  // wavefront 0 met the pivots; L_ii^2 / S_ii of the used columns
    const T l = W[lane * kLd + lane];
    const float ratio = lane < size ? (float)(l * l / d0[kBlk * K + lane]) : 3.0e38f;
    unsigned int m = __float_as_uint(l > (T)0 && ratio == ratio ? fmaxf(ratio, 0.f) : 0.f);
    if (lane >= size) m = __float_as_uint(3.0e38f);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = min(m, (unsigned int)__shfl_xor((int)m, o));
    if (lane == 0) {
      if (bad) atomicOr(status, 1);
      atomicMin(min_bits, m);
    }
  }
}

// ------------------------------------------------------------ triangular solves

// The solved values travel with the call's epoch in 64-bit words (32 value
// bits low, the epoch high: one word per float32 value, two per float64
// value; separate arrays for the forward and the backward pass), stored and
// polled as single-copy-atomic agent-scope words, so a value is its own flag:
// no release of the producer's cache, no acquire on the consumer's, and the
// data arrives with the signal.  Every wait is bounded.
constexpr long long kSolveSpin = 1LL << 22;

template <typename T>
__device__ __forceinline__ void put_word(unsigned long long* xw, int row, T v, int epoch) {
  const unsigned long long tag = (unsigned long long)(unsigned)epoch << 32;
  if constexpr (sizeof(T) == 4) {
    __hip_atomic_store(xw + row, tag | (unsigned long long)__float_as_uint(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  } else {
    const unsigned long long bits = (unsigned long long)__double_as_longlong(v);
    __hip_atomic_store(xw + 2 * (size_t)row, tag | (bits & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(xw + 2 * (size_t)row + 1, tag | (bits >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// One word polled until it carries `epoch` (bounded); false on a timeout or
// another wait's failure (reported).
__device__ __forceinline__ bool poll_word(const unsigned long long* w, int epoch, int* err, int* host_err,
                                          unsigned long long* out) {
  unsigned long long word = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  long long spins = 0;
  while ((int)(word >> 32) != epoch) {
    __builtin_amdgcn_s_sleep(1);
    if (++spins > kSolveSpin ||
        (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & (kErrChain | kErrBarrier))) {
      report_device_error(err, host_err, kErrChain);
      return false;
    }
    word = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  *out = word;
  return true;
}

template <typename T>
__device__ __forceinline__ bool get_word(const unsigned long long* xw, int row, int epoch, int* err, int* host_err,
                                         T* v) {
  unsigned long long lo = 0, hi = 0;
  if constexpr (sizeof(T) == 4) {
    if (!poll_word(xw + row, epoch, err, host_err, &lo)) return false;
    *v = __uint_as_float((unsigned)(lo & 0xffffffffull));
  } else {
    if (!poll_word(xw + 2 * (size_t)row, epoch, err, host_err, &lo) ||
        !poll_word(xw + 2 * (size_t)row + 1, epoch, err, host_err, &hi))
      return false;
    *v = __longlong_as_double((long long)(((hi & 0xffffffffull) << 32) | (lo & 0xffffffffull)));
  }
  return true;
}

// Whether a refinement's residual (m[0]: the largest |r_i|, m[1]: |s_i|) is
// at or below tol; false without a residual, and for NaN.
__device__ __forceinline__ bool refine_done(const unsigned long long* m, double tol) {
  if (!m) return false;
  const double rmax = __longlong_as_double((long long)m[0]), smax = __longlong_as_double((long long)m[1]);
  return (smax > 0.0 ? rmax / smax : rmax) <= tol;
}

// Both triangular solves in one launch.  Block columns go to the workgroups
// by level (forward) and then by descending level (backward): workgroup g
// takes places g, g + G, ... of that order, so the first unfinished place is
// always some resident workgroup's next one and nobody waits for a place
// behind it.  A block's values are loaded before the wait for the vector they
// multiply; the products are summed per thread over all blocks and reduced
// once.  With stop given (the largest |r| and |s| of a refinement) the whole
// call is a no-op when the residual is small enough.
template <typename T>
__global__ void __launch_bounds__(256) sparse_solve_kernel(SparsePlan P, const T* A, const T* Linv, const T* b, T* y,
                                                           T* x, unsigned long long* words, int epoch, int* err,
                                                           int* host_err, int backward_only, const unsigned long long* stop,
                                                           double tol) {
  if (refine_done(stop, tol)) return;
  __shared__ T vk[2][kBlk];
  __shared__ T part[4][kBlk];
  __shared__ T sa[kBlk];
  __shared__ int fail_s;
  const int tid = threadIdx.x, nb = P.nb, G = gridDim.x;
  unsigned long long* xw = words;
  unsigned long long* yw = words + (size_t)nb * kBlk * (sizeof(T) / 4);
  if (tid == 0) fail_s = 0;
  __syncthreads();
  // forward: thread (r, q) takes row r, columns 16 q .. of each block of the row
  for (int g = backward_only ? nb : (int)blockIdx.x; g < nb; g += G) {
    const int K = P.by_level[g];
    const int r = tid >> 2, q = tid & 3;
    T li[16];  // row r of L_KK^-1
#pragma unroll
    for (int m = 0; m < 16; ++m) li[m] = Linv[(size_t)K * kBB + r * kBlk + 16 * q + m];
    T s = (T)0;
    for (int e = P.rptr[K]; e < P.rptr[K + 1]; ++e) {
      const int2 je = P.rlist[e];
      T l[16];
#pragma unroll
      for (int m = 0; m < 16; ++m) l[m] = A[(size_t)je.y * kBB + r * kBlk + 16 * q + m];
      T* vb = vk[e & 1];
      if (tid < kBlk && !get_word<T>(yw, kBlk * je.x + tid, epoch, err, host_err, &vb[tid])) fail_s = 1;
      __syncthreads();
      if (fail_s) return;
#pragma unroll
      for (int m = 0; m < 16; ++m) s += l[m] * vb[16 * q + m];
    }
    __syncthreads();
    part[q][r] = s;
    __syncthreads();
    if (tid < kBlk) sa[tid] = b[kBlk * K + tid] - ((part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]));
    __syncthreads();
    T z = (T)0;
#pragma unroll
    for (int m = 0; m < 16; ++m) z += li[m] * sa[16 * q + m];
    part[q][r] = z;
    __syncthreads();
    if (tid < kBlk) {
      const T o = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
      y[kBlk * K + tid] = o;
      put_word<T>(yw, kBlk * K + tid, o, epoch);
    }
    __syncthreads();
  }
  // backward: thread (c, q) takes column c, rows 16 q .. of each block of the
  // column, the last eliminated (first available) rows first.  y_K is this
  // workgroup's own value: its forward place and its backward place differ, so
  // it is read through the published words unless the factor left it.
  for (int g = blockIdx.x; g < nb; g += G) {
    const int K = P.by_level[nb - 1 - g];
    const int c = tid & 63, q = tid >> 6;
    T li[16];  // column c of L_KK^-1
#pragma unroll
    for (int m = 0; m < 16; ++m) li[m] = Linv[(size_t)K * kBB + (16 * q + m) * kBlk + c];
    T s = (T)0;
    const int e0 = P.colptr[K] + 1;
    for (int e = P.colptr[K + 1] - 1; e >= e0; --e) {
      const int I = P.rowidx[e];
      T l[16];
#pragma unroll
      for (int m = 0; m < 16; ++m) l[m] = A[(size_t)e * kBB + (16 * q + m) * kBlk + c];
      T* vb = vk[e & 1];
      if (tid < kBlk && !get_word<T>(xw, kBlk * I + tid, epoch, err, host_err, &vb[tid])) fail_s = 1;
      __syncthreads();
      if (fail_s) return;
#pragma unroll
      for (int m = 0; m < 16; ++m) s += l[m] * vb[16 * q + m];
    }
    __syncthreads();
    part[q][c] = s;
    T yv = (T)0;
    if (tid < kBlk) {
      if (backward_only) yv = y[kBlk * K + tid];
      else if (!get_word<T>(yw, kBlk * K + tid, epoch, err, host_err, &yv)) fail_s = 1;
    }
    __syncthreads();
    if (fail_s) return;
    if (tid < kBlk) sa[tid] = yv - ((part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]));
    __syncthreads();
    T z = (T)0;
#pragma unroll
    for (int m = 0; m < 16; ++m) z += li[m] * sa[16 * q + m];
    part[q][c] = z;
    __syncthreads();
    if (tid < kBlk) {
      const T o = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
      x[kBlk * K + tid] = o;
      put_word<T>(xw, kBlk * K + tid, o, epoch);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------ assembly and vectors

// One workgroup per block: its pose pairs summed from the tiles' shares in
// tile order (eight loads in flight) into LDS, then the whole block written
// as 16-byte vectors -- fill blocks as zeros, unused rows as identity -- so
// the storage needs no clearing pass.  Bound by the chain offset, source,
// value of each entry: a block near the diagonal has up to 100 pairs of 36
// entries, and few blocks are that full, so sixteen wavefronts take one
// with the loads of eight shares together: 26 us on 1000 keyframes (902 blocks),
// 19 us on 317 in float64 (227 blocks); with 256 threads, four loads together and
// the rest one by one 62 and 55 us.  A workgroup a block leaves most of the chip
// idle where blocks are few: at 100 keyframes (up to 55 of them) the gather phase
// takes 55 us, where a thread an entry of the dense system took 31.
constexpr int kGatherThreads = 1024;
template <typename TP, typename T>
__global__ void __launch_bounds__(kGatherThreads) sparse_gather_kernel(SparsePlan P, const TP* part_S, const int* off,
                                                            const int* src, T* A, const T* dB, T lambda, T lam_diag,
                                                            T* d0, T* rhs, float* A32, float* d032) {
  __shared__ __align__(16) T tile[kBB];
  const int id = blockIdx.x, tid = threadIdx.x;
  const int I = P.rowidx[id];
  const int p0 = P.pair_off[id], np = P.pair_off[id + 1] - p0;
  // the diagonal block comes first in its column, which is its row
  const bool diag = id == P.colptr[I];
  const int size = diag ? P.size[I] : kBlk;
  if (diag && tid >= size && tid < kBlk) rhs[kBlk * I + tid] = (T)0;  // rows that no pose uses
  for (int e = tid; e < kBB; e += kGatherThreads) tile[e] = (T)((e >> 6) == (e & 63) && (e >> 6) >= size ? 1 : 0);
  __syncthreads();
  for (int x = tid; x < np * 36; x += kGatherThreads) {
    const int2 pr = P.pairs[p0 + x / 36];
    const int e = x % 36, r = e / 6, c = e % 6;
    const bool dpair = (pr.y >> 17) & 1;
    if (dpair && r < c) continue;
    const int eo = (pr.y >> 16) & 1 ? r * 6 + c : c * 6 + r;  // the tiles store upper entries of their block pairs
    const int lo = off[pr.x], hi = off[pr.x + 1];
    T v = (T)0;
    for (int q = lo; q < hi; q += 8) {
      int at[8];
      TP t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) at[u] = src[min(q + u, hi - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = part_S[at[u] + eo];
#pragma unroll
      for (int u = 0; u < 8; ++u) v += q + u < hi ? (T)t[u] : (T)0;
    }
    const int row = (pr.y & 255) + r, col = ((pr.y >> 8) & 255) + c;
    if (dpair && r == c) {
      v += lam_diag * dB[kBlk * I + row] + lambda;
      d0[kBlk * I + row] = v;
      if (d032) d032[kBlk * I + row] = (float)v;
    }
    tile[row * kBlk + col] = v;
  }
  __syncthreads();
  typedef typename V16<T>::type vec_t;
  constexpr int V = 16 / (int)sizeof(T);
  vec_t* out = reinterpret_cast<vec_t*>(A + (size_t)id * kBB);
  for (int e = tid; e < kBB / V; e += kGatherThreads) out[e] = reinterpret_cast<const vec_t*>(tile)[e];
  if (A32)
    for (int e = tid; e < kBB; e += kGatherThreads) A32[(size_t)id * kBB + e] = (float)tile[e];
}

// Zero blocks (identity in unused rows) and right-hand side, 16 bytes a store;
// one more workgroup, the first, sums a pose graph's squared residuals beside them (cost
// null: none).
template <typename T>
__global__ void __launch_bounds__(256) sparse_clear_kernel(SparsePlan P, T* A, T* v, const double* r, int nr,
                                                           double* cost) {
  const int id = (int)blockIdx.x - (cost ? 1 : 0);
  if (id < 0) {
    sum_squares_256(r, nr, cost);
    return;
  }
  const int I = P.rowidx[id];
  const bool diag = id == P.colptr[I];
  const int size = diag ? P.size[I] : kBlk;
  typedef typename V16<T>::type vec_t;
  constexpr int V = 16 / (int)sizeof(T);
  vec_t* o = reinterpret_cast<vec_t*>(A + (size_t)id * kBB);
#pragma unroll
  for (int u = 0; u < kBB / V / 256; ++u) {
    const int e = V * (u * 256 + (int)threadIdx.x);
    vec_t x;
#pragma unroll
    for (int m = 0; m < V; ++m) x[m] = (T)(((e + m) >> 6) == ((e + m) & 63) && ((e + m) >> 6) >= size ? 1 : 0);
    o[e / V] = x;
  }
  if (diag && (int)threadIdx.x < kBlk) v[kBlk * I + threadIdx.x] = (T)0;
}

// One step of iterative refinement: x = x_in + c (x_in null: x = c; c left out
// when the solve that makes it was, as refine_done(stop, tol)), r = s - A x,
// and r rounded to float32 as the next solve's right-hand side.  One workgroup
// per block row over the original blocks of the symmetric matrix (the
// diagonal block's lower triangle counts for both); every row adds c to the x
// it reads, and its own part of x goes to x_out.  The largest |r_i| and |s_i|
// are kept as ordered bits of non-negative doubles (integer maxima, independent
// of the order of the atomics; cleared by sparse_refine_begin_kernel).  Bound
// by the latency of a row's blocks: four are read at a time, by 256 threads
// each (317 keyframes: 18.1 -> 15.8 us a step, without the five launches of
// 4.7 us around it).
__global__ void __launch_bounds__(1024) sparse_residual_kernel(SparsePlan P, const double* A, const double* s,
                                                               const double* x_in, const float* c,
                                                               const unsigned long long* stop, double tol,
                                                               double* x_out, float* rhs, unsigned long long* maxes) {
  __shared__ double part[16][kBlk];
  __shared__ double xs[4][kBlk];
  const int I = blockIdx.x, tid = threadIdx.x;
  const int grp = tid >> 8, a = tid & 63, q = (tid >> 6) & 3;
  const bool add = !refine_done(stop, tol);
  auto x_at = [&](int row) { return x_in ? (add ? x_in[row] + (double)c[row] : x_in[row]) : (double)c[row]; };
  double v = 0.0;
  const int e0 = P.nptr[I], e1 = P.nptr[I + 1];
  for (int eb = e0; eb < e1; eb += 4) {
    const int e = eb + grp;
    const bool on = e < e1;  // uniform in a group
    const int2 je = P.nlist[on ? e : e1 - 1];
    const double* B = A + (size_t)(je.y >> 1) * kBB;
    double b[16];
    if (je.x == I) {  // symmetric from the lower triangle
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        const int cc = 16 * q + m;
        b[m] = cc <= a ? B[a * kBlk + cc] : B[cc * kBlk + a];
      }
    } else if (je.y & 1) {
#pragma unroll
      for (int m = 0; m < 16; ++m) b[m] = B[(16 * q + m) * kBlk + a];
    } else {
#pragma unroll
      for (int m = 0; m < 16; ++m) b[m] = B[a * kBlk + 16 * q + m];
    }
    __syncthreads();
    if (q == 0) xs[grp][a] = on ? x_at(kBlk * je.x + a) : 0.0;
    __syncthreads();
    if (on) {
#pragma unroll
      for (int m = 0; m < 16; ++m) v += b[m] * xs[grp][16 * q + m];
    }
  }
  part[tid >> 6][a] = v;
  __syncthreads();
  if (tid < kBlk) {
    double ax = 0.0;
#pragma unroll
    for (int m = 0; m < 16; m += 4)
      ax += (part[m][tid] + part[m + 1][tid]) + (part[m + 2][tid] + part[m + 3][tid]);
    const double sv = s[kBlk * I + tid];
    const double rv = sv - ax;
    x_out[kBlk * I + tid] = x_at(kBlk * I + tid);
    rhs[kBlk * I + tid] = (float)rv;
    unsigned long long rm = (unsigned long long)__double_as_longlong(fabs(rv));
    unsigned long long sm = (unsigned long long)__double_as_longlong(fabs(sv));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const unsigned long long ro = __shfl_xor(rm, o), so = __shfl_xor(sm, o);
      rm = ro > rm ? ro : rm;
      sm = so > sm ? so : sm;
    }
    if (tid == 0) {
      atomicMax(maxes, rm);
      atomicMax(maxes + 1, sm);
    }
  }
}

// Start of a refined solve: the right-hand side in float32, and the cleared
// maxima of its n_res residuals.
__global__ void sparse_refine_begin_kernel(const double* s, float* y, int n, unsigned long long* maxes, int n_res) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = (float)s[i];
  if (i < 2 * n_res) maxes[i] = 0ull;
}

template <typename T>
__global__ void sparse_rows_kernel(SparsePlan P, const T* src, T* dst, const int* status, int out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P.bw * P.n_pose) return;
  const int f = i / P.bw, row = P.row0[f] + (i - f * P.bw);
  if (out) dst[i] = status && *status ? (T)0 : src[row];
  else dst[row] = src[i];
}

template <typename T>
__global__ void sparse_zero_kernel(T* x, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = (T)0;
}

// ------------------------------------------------------------ launchers

template <typename TP, typename T>
hipError_t launch_sparse_gather(const SparsePlan& p, const TP* part_S, const int* off, const int* src, T* A,
                                const T* dB, T lambda, T lam_diag, T* d0, T* rhs, float* A32, float* d032,
                                hipStream_t st) {
  if (p.nb == 0) return hipSuccess;
  hipLaunchKernelGGL((sparse_gather_kernel<TP, T>), dim3(p.n_blocks), dim3(kGatherThreads), 0, st, p, part_S, off, src, A, dB,
                     lambda, lam_diag, d0, rhs, A32, d032);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_sparse_clear(const SparsePlan& p, T* A, T* v, const double* r, int nr, double* cost, hipStream_t st) {
  if (p.nb == 0) return hipSuccess;
  hipLaunchKernelGGL((sparse_clear_kernel<T>), dim3(p.n_blocks + (cost ? 1 : 0)), dim3(256), 0, st, p, A, v, r, nr,
                     cost);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_sparse_factor(const SparsePlan& p, T* A, T* Linv, T* v, const T* d0, int* status,
                                unsigned int* min_bits, hipStream_t st) {
  const int lds = level_lds_elems<T>() * (int)sizeof(T);
  hipError_t e = opt_in_lds((const void*)sparse_level_kernel<T>, lds);
  if (e != hipSuccess) return e;
  for (int l = 0; l < p.n_level; ++l) {
    const int nt = p.task_off[l + 1] - p.task_off[l], impl = p.implicit_col[l];
    int nu = p.upd_off[l + 1] - p.upd_off[l];
    if (impl >= 0) {
      const int m = p.colptr_h[impl + 1] - p.colptr_h[impl] - 1;
      nu = m * (m + 1) / 2;
    }
    hipLaunchKernelGGL((sparse_level_kernel<T>), dim3(nt + nu), dim3(kLevelThreads), lds, st, A, Linv, v, d0, p,
                       p.tasks + p.task_off[l], nt, p.updates + p.upd_off[l], impl, l, status, min_bits);
  }
  return hipGetLastError();
}

template <typename T>
static int solve_grid(int nb) {
  int per_cu = 0, dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)sparse_solve_kernel<T>, 256, 0) != hipSuccess)
    return 0;
  return std::min(nb, per_cu * cus);
}

// The grid never exceeds the workgroups the device holds at once.
// cooperative = false (the default): an ordinary launch, relying on the
// device placing every workgroup while the others wait for their
// predecessors -- true when the device's other work finishes; every wait is
// bounded, so a violation is reported (kErrChain), never a hang.
// cooperative = true: the runtime guarantees co-residency, at the cost of a
// cooperative launch.
template <typename T>
hipError_t launch_sparse_solve(const SparsePlan& p, const T* A, const T* Linv, const T* b, T* y, T* x,
                               unsigned long long* words, int epoch, int* err, int* host_err, hipStream_t st,
                               bool backward_only, bool cooperative, const unsigned long long* stop, double tol) {
  if (p.nb == 0) return hipSuccess;
  const int grid = solve_grid<T>(p.nb);
  if (grid < 1) return hipErrorCooperativeLaunchTooLarge;
  int back = backward_only ? 1 : 0;
  if (!cooperative) {
    hipLaunchKernelGGL((sparse_solve_kernel<T>), dim3(grid), dim3(256), 0, st, p, A, Linv, b, y, x, words, epoch, err,
                       host_err, back, stop, tol);
    return hipGetLastError();
  }
  SparsePlan copy = p;
  void* args[] = {(void*)&copy, (void*)&A,     (void*)&Linv, (void*)&b,        (void*)&y,    (void*)&x,
                  (void*)&words, (void*)&epoch, (void*)&err,  (void*)&host_err, (void*)&back, (void*)&stop,
                  (void*)&tol};
  return hipLaunchCooperativeKernel((const void*)sparse_solve_kernel<T>, dim3(grid), dim3(256), args, 0, st);
}

hipError_t launch_sparse_residual(const SparsePlan& p, const double* A, const double* s, const double* x_in,
                                  const float* c, const unsigned long long* stop, double tol, double* x_out, float* rhs,
                                  unsigned long long* maxes, hipStream_t st) {
  if (p.nb == 0) return hipSuccess;
  hipLaunchKernelGGL(sparse_residual_kernel, dim3(p.nb), dim3(1024), 0, st, p, A, s, x_in, c, stop, tol, x_out, rhs,
                     maxes);
  return hipGetLastError();
}

hipError_t launch_sparse_refine_begin(const SparsePlan& p, const double* s, float* y, unsigned long long* maxes,
                                      int n_res, hipStream_t st) {
  if (p.nb == 0) return hipSuccess;
  hipLaunchKernelGGL(sparse_refine_begin_kernel, dim3((kBlk * p.nb + 255) / 256), dim3(256), 0, st, s, y, kBlk * p.nb,
                     maxes, n_res);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_sparse_rows_in(const SparsePlan& p, const T* src, T* dst, hipStream_t st) {
  const int n = p.bw * p.n_pose;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL((sparse_zero_kernel<T>), dim3((kBlk * p.nb + 255) / 256), dim3(256), 0, st, dst, kBlk * p.nb);
  hipLaunchKernelGGL((sparse_rows_kernel<T>), dim3((n + 255) / 256), dim3(256), 0, st, p, src, dst,
                     (const int*)nullptr, 0);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_sparse_rows_out(const SparsePlan& p, const T* src, T* dst, const int* status, hipStream_t st) {
  const int n = p.bw * p.n_pose;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL((sparse_rows_kernel<T>), dim3((n + 255) / 256), dim3(256), 0, st, p, src, dst, status, 1);
  return hipGetLastError();
}

template hipError_t launch_sparse_gather<float, float>(const SparsePlan&, const float*, const int*, const int*, float*,
                                                       const float*, float, float, float*, float*, float*,
                                                       float*, hipStream_t);
template hipError_t launch_sparse_gather<double, double>(const SparsePlan&, const double*, const int*, const int*,
                                                         double*, const double*, double, double, double*, double*,
                                                         float*, float*, hipStream_t);
template hipError_t launch_sparse_gather<float, double>(const SparsePlan&, const float*, const int*, const int*,
                                                        double*, const double*, double, double, double*, double*,
                                                        float*, float*, hipStream_t);
template hipError_t launch_sparse_clear<double>(const SparsePlan&, double*, double*, const double*, int, double*,
                                                hipStream_t);
#define DPVBA_SPARSE_INSTANTIATE(T)                                                                                  \
  template hipError_t launch_sparse_factor<T>(const SparsePlan&, T*, T*, T*, const T*, int*, unsigned int*,           \
                                              hipStream_t);                                                          \
  template hipError_t launch_sparse_solve<T>(const SparsePlan&, const T*, const T*, const T*, T*, T*,                 \
                                             unsigned long long*, int, int*, int*, hipStream_t, bool, bool,          \
                                             const unsigned long long*, double);                                     \
  template hipError_t launch_sparse_rows_in<T>(const SparsePlan&, const T*, T*, hipStream_t);                         \
  template hipError_t launch_sparse_rows_out<T>(const SparsePlan&, const T*, T*, const int*, hipStream_t);
DPVBA_SPARSE_INSTANTIATE(float)
DPVBA_SPARSE_INSTANTIATE(double)

}  // namespace dpvba
