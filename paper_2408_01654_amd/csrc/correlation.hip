// Patch correlation of DPV-SLAM eq. 4 (Sec. 3.1, "Patch correlation"):
//   C(u, v, a, b) = < g(u, v), f(P'(u, v) + Delta_ab) >
// for every edge (i, k, j): g the p x p patch features of patch k, f the
// feature map of the edge's target frame sampled bilinearly (zero outside)
// at the reprojected patch pixel shifted by the 7 x 7 grid of offsets
// Delta_ab = (a - 3, b - 3).
//
// All 49 samples of one patch pixel share the fractional position of the
// reprojected point, so their four-pixel footprints cover one 8 x 8 window of
// the map: the kernel takes 64 dot products (window pixel . g) and combines
// them bilinearly, instead of 196 four-pixel samples.  One wavefront per
// (edge, patch pixel): lanes split the feature dimension (D / 64 channels
// each), every window pixel arrives as one contiguous D-vector load per
// wavefront, each lane keeps 64 partial dots, and a halving butterfly (63
// shuffles) leaves window pixel l's total on lane l; lane 8 b + a then reads
// its three neighbours and writes C(u, v, a, b).  The four wavefronts of a
// workgroup take consecutive patch pixels of one edge, which share most of
// their windows in the caches.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.h"
#include "layout.h"
#include "mfma.h"

namespace dpvba {

constexpr int kCorrR = 3;               // offsets -3 .. 3
constexpr int kCorrGrid = 2 * kCorrR + 1;

template <int VPL>  // channels per lane (D = 64 VPL)
__global__ void __launch_bounds__(256) patch_corr_kernel(int n_items, int p2, const float* __restrict__ gmap,
                                                         int n_patches, const float* __restrict__ fmaps, int n_maps,
                                                         int H, int W, const int* __restrict__ kk,
                                                         const int* __restrict__ jj, const float* __restrict__ coords,
                                                         float* __restrict__ corr, int* dev_err, int* host_err) {
  constexpr int D = 64 * VPL;
  const int lane = threadIdx.x & 63;
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= n_items) return;  // whole wavefront
  const int e = item / p2, pix = item - (item / p2) * p2;
  const int k = kk[e], fj = jj[e];
  float* out = corr + (size_t)item * (kCorrGrid * kCorrGrid);
  if (k < 0 || k >= n_patches || fj < 0 || fj >= n_maps) {
    if (lane < kCorrGrid * kCorrGrid) out[lane] = 0.f;
    if (lane == 0) report_device_error(dev_err, host_err, kErrInput);
    return;
  }
  const float x = coords[2 * (size_t)item], y = coords[2 * (size_t)item + 1];
  const float xf = floorf(x), yf = floorf(y);
  const float fx = x - xf, fy = y - yf;
  // window of 8 x 8 map pixels starting at (floor(x) - 3, floor(y) - 3); points
  // far outside the map (or not finite) leave every window pixel outside
  const bool finite = fabsf(x) < 1e9f && fabsf(y) < 1e9f;
  const int wx0 = finite ? (int)xf - kCorrR : -(1 << 30), wy0 = finite ? (int)yf - kCorrR : -(1 << 30);
  float g[VPL];
  {
    const float* gp = gmap + ((size_t)k * p2 + pix) * D + lane * VPL;
#pragma unroll
    for (int m = 0; m < VPL; ++m) g[m] = gp[m];
  }
  const float* fm = fmaps + (size_t)fj * H * W * D + lane * VPL;
  float part[64];
#pragma unroll
  for (int w = 0; w < 64; ++w) {
    const int xx = wx0 + (w & 7), yy = wy0 + (w >> 3);
    float s = 0.f;
    if (xx >= 0 && xx < W && yy >= 0 && yy < H) {
      const float* fp = fm + ((size_t)yy * W + xx) * D;
#pragma unroll
      for (int m = 0; m < VPL; ++m) s += g[m] * fp[m];
    }
    part[w] = s;
  }
  // halving butterfly: after level s lane l holds the partial totals of the
  // window pixels whose top s index bits equal l's
#pragma unroll
  for (int h = 32; h >= 1; h >>= 1) {
    const bool hi = lane & h;
#pragma unroll
    for (int i = 0; i < h; ++i) {
      const float keep = hi ? part[h + i] : part[i];
      const float give = hi ? part[i] : part[h + i];
      part[i] = keep + __shfl_xor(give, h);
    }
  }
  const float d00 = part[0];
  const float d01 = __shfl(d00, (lane + 1) & 63);
  const float d10 = __shfl(d00, (lane + 8) & 63);
  const float d11 = __shfl(d00, (lane + 9) & 63);
  const int a = lane & 7, b = lane >> 3;  // window column (x offset), row (y offset)
  if (a < kCorrGrid && b < kCorrGrid) {
    const float c = (1.f - fx) * (1.f - fy) * d00 + fx * (1.f - fy) * d01 + (1.f - fx) * fy * d10 + fx * fy * d11;
    out[a * kCorrGrid + b] = c;
  }
}

// 3 x 3 patches (the odometry's) on the matrix cores.  The nine windows of one
// edge overlap almost entirely (their points lie about a pixel apart), so
// one wavefront per edge takes their union, clipped to the map, once: 16 map
// pixels at a time against the patch's nine feature vectors (rows 9 .. 15 of
// the 16 x 16 x 4 products are zero), every dot product accumulated in
// float32.  Lane l holds row l % 16 of the patch features and pixel l % 16 of
// the union at channels 16 s + 4 (l / 16) + c: both operands take the same
// order of the channels, so they arrive as 16-byte loads straight into the
// operand registers (two wavefronts per SIMD at least, four at up to 128
// channels: the products then stay in ordinary registers, without a move out of
// the accumulators).  The dots [9][union] go to LDS, and the 441 outputs of the edge
// are combined from them and written contiguously.  Patches whose union
// holds more than kCorrUnion pixels (scattered: seen at more than four times
// their size) take their nine windows one by one, and where there are few edges
// each has a workgroup of its own, whose four wavefronts share those windows.
// Against one wavefront per (edge, pixel) this reads 100 to 144 map pixels an
// edge instead of 576 and needs no reduction over lanes: 37,440 edges of 128
// channels took 1,564 us and take 229 us (the products alone 109 us at the float32
// matrix rate), 2.0 GB of map pixels read from the caches instead of 11 GB.

// Edges up to which each has a workgroup of its own: they all run at once either
// way (128 channels, points 6 pixels apart: 64 edges 44.0 -> 10.1 us, 512 edges
// 46.9 -> 20.8 us; compact patches the same or 5 % faster).  At 768 edges of 256
// channels compact patches take 25 us so, 21 us four to a workgroup.
constexpr int kCorrSpread = 512;
constexpr int kCorrUnion = 256;            // pixels of a union window
constexpr int kCorrLd = kCorrUnion + 4;    // row stride of the dots (the four row groups of a store on different banks)

// Sum of the products of N groups of 16 channels, as a binary tree.
template <int N>
__device__ __forceinline__ floatx4_t corr_tree(const float4* g, const float4* f) {
  if constexpr (N == 1) {
    const floatx4_t zero = {0.f, 0.f, 0.f, 0.f};
    return (Mfma<float>::step(g->x, f->x, zero) + Mfma<float>::step(g->y, f->y, zero)) +
           (Mfma<float>::step(g->z, f->z, zero) + Mfma<float>::step(g->w, f->w, zero));
  } else {
    return corr_tree<N / 2>(g, f) + corr_tree<N - N / 2>(g + N / 2, f + N / 2);
  }
}

// Sum of the products of N groups of 4 channels, as a binary tree.
template <int N>
__device__ __forceinline__ float dot_tree(const float4* g, const float4* f) {
  if constexpr (N == 1) return (g->x * f->x + g->y * f->y) + (g->z * f->z + g->w * f->w);
  else return dot_tree<N / 2>(g, f) + dot_tree<N - N / 2>(g + N / 2, f + N / 2);
}

// Sum over the 16 lanes of a row, on every lane of it (rotations within the row).
__device__ __forceinline__ float row_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xF, 0xF, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x124, 0xF, 0xF, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x122, 0xF, 0xF, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x121, 0xF, 0xF, true));
  return v;
}

template <int VPL>  // channels per lane quarter of 16 (D = 64 VPL)
__global__ void __launch_bounds__(256, VPL <= 2 ? 4 : 2) patch_corr3_kernel(int n_edges, int per_group,
                                                          const float* __restrict__ gmap, int n_patches,
                                                          const float* __restrict__ fmaps, int n_maps, int H, int W,
                                                          const int* __restrict__ kk, const int* __restrict__ jj,
                                                          const float* __restrict__ coords, float* __restrict__ corr,
                                                          int* dev_err, int* host_err) {
  constexpr int D = 64 * VPL, NS = D / 16, P2 = 9, G2 = kCorrGrid * kCorrGrid;
  __shared__ float dots_s[4][P2 * kCorrLd];
  __shared__ float4 pix_s[4][P2];  // window origin (x, y) as integers, fractional position
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e = per_group == 4 ? (int)blockIdx.x * 4 + wv : (int)blockIdx.x;
  const int g0 = per_group == 4 ? 0 : wv, dg = per_group == 4 ? 1 : 4;  // this wavefront's windows of a scattered patch
  if (e >= n_edges) return;  // whole wavefront; no workgroup barrier below
  const int k = kk[e], fj = jj[e];
  float* out = corr + (size_t)e * (P2 * G2);
  if (k < 0 || k >= n_patches || fj < 0 || fj >= n_maps) {
    if (g0 != 0) return;
    for (int o = lane; o < P2 * G2; o += 64) out[o] = 0.f;
    if (lane == 0) report_device_error(dev_err, host_err, kErrInput);
    return;
  }
  float* dots = dots_s[wv];
  float4* pixs = pix_s[wv];
  const int r = lane & 15, q = lane >> 4;
  const bool has = r < P2;
  float4 g[NS];
  {
    const float4* gp = reinterpret_cast<const float4*>(gmap + ((size_t)k * P2 + (has ? r : 0)) * D) + q;
#pragma unroll
    for (int s = 0; s < NS; ++s) g[s] = has ? gp[4 * s] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  // pixel r's window: 8 x 8 map pixels from (floor(x) - 3, floor(y) - 3);
  // points far outside or not finite leave it outside the map
  int xl = 1 << 30, xh = -(1 << 30), yl = 1 << 30, yh = -(1 << 30);
  if (has) {
    const float2 xy = reinterpret_cast<const float2*>(coords)[(size_t)e * P2 + r];
    const float xf = floorf(xy.x), yf = floorf(xy.y);
    const bool finite = fabsf(xy.x) < 1e9f && fabsf(xy.y) < 1e9f;
    const int wx0 = finite ? (int)xf - kCorrR : -(1 << 30), wy0 = finite ? (int)yf - kCorrR : -(1 << 30);
    if (lane < P2) pixs[r] = make_float4(__int_as_float(wx0), __int_as_float(wy0), xy.x - xf, xy.y - yf);
    const int a0 = max(wx0, 0), a1 = min(wx0 + kCorrGrid + 1, W), b0 = max(wy0, 0), b1 = min(wy0 + kCorrGrid + 1, H);
    if (a0 < a1 && b0 < b1) {
      xl = a0;
      xh = a1;
      yl = b0;
      yh = b1;
    }
  }
  int ux0 = xl, ux1 = xh, uy0 = yl, uy1 = yh;
#pragma unroll
  for (int h = 1; h < 16; h <<= 1) {
    ux0 = min(ux0, __shfl_xor(ux0, h));
    ux1 = max(ux1, __shfl_xor(ux1, h));
    uy0 = min(uy0, __shfl_xor(uy0, h));
    uy1 = max(uy1, __shfl_xor(uy1, h));
  }
  const float* fm = fmaps + (size_t)fj * H * W * D + 4 * q;
  // an empty union (every window outside) has no pixels, and dots stays unread
  const bool one = ux1 <= ux0 || (long long)(ux1 - ux0) * (uy1 - uy0) <= kCorrUnion;
  // outputs o0 .. o1 - 1 from the dots of the window (x0, y0), w pixels wide
  auto combine = [&](int o0, int o1, int x0, int y0, int w) {
    // the wavefront's own LDS writes, in order: only the compiler must not
    // move the reads above them
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int o = o0 + lane; o < o1; o += 64) {
      const int px = o / G2, ab = o - px * G2, a = ab / kCorrGrid, b = ab - a * kCorrGrid;
      const float4 pp = pixs[px];
      const int xx = __float_as_int(pp.x) + a, yy = __float_as_int(pp.y) + b;
      const bool in0 = xx >= 0 && xx < W, in1 = xx + 1 >= 0 && xx + 1 < W;
      const bool jn0 = yy >= 0 && yy < H, jn1 = yy + 1 >= 0 && yy + 1 < H;
      const float* d = dots + px * kCorrLd + (yy - y0) * w + (xx - x0);
      const float d00 = in0 && jn0 ? d[0] : 0.f, d01 = in1 && jn0 ? d[1] : 0.f;
      const float d10 = in0 && jn1 ? d[w] : 0.f, d11 = in1 && jn1 ? d[w + 1] : 0.f;
      const float fx = pp.z, fy = pp.w;
      out[o] = (1.f - fx) * (1.f - fy) * d00 + fx * (1.f - fy) * d01 + (1.f - fx) * fy * d10 + fx * fy * d11;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if (one) {
    if (g0 != 0) return;
    const int x0 = __builtin_amdgcn_readfirstlane(ux0), x1 = __builtin_amdgcn_readfirstlane(ux1);
    const int y0 = __builtin_amdgcn_readfirstlane(uy0), y1 = __builtin_amdgcn_readfirstlane(uy1);
    const int w = x1 - x0, n = x1 > x0 ? w * (y1 - y0) : 0;
    const float rw = 1.f / (float)max(w, 1);
    // pixel t of the union (row-major): t < 256, so the quotient is exact
    auto pixel = [&](int t) {
      const int tc = min(t, n - 1);
      const int y = (int)(((float)tc + 0.5f) * rw), x = tc - y * w;
      return reinterpret_cast<const float4*>(fm + ((size_t)(y0 + y) * W + (x0 + x)) * D);
    };
    if (n > 0) {
      float4 f[NS];
      const float4* fp = pixel(r);
#pragma unroll
      for (int s = 0; s < NS; ++s) f[s] = fp[4 * s];
      for (int t0 = 0; t0 < n; t0 += 16) {
        // the next 16 pixels load while this tile's products run (the last
        // tile reloads its own last pixel)
        float4 nf[NS];
        const float4* np = pixel(t0 + 16 + r);
#pragma unroll
        for (int s = 0; s < NS; ++s) nf[s] = np[4 * s];
        // every product step starts from zero and the steps are summed as a
        // binary tree over the channels, like the sum over lanes that this
        // replaces (one chain of 32 steps had 1.7 times its error)
        // (the loads all go out before the products; at up to 128 channels that
        // keeps to the registers of four wavefronts a SIMD, 241 -> 232 us)
        if constexpr (VPL <= 2) __builtin_amdgcn_sched_barrier(0);
        const floatx4_t acc = corr_tree<NS>(g, f);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = Mfma<float>::row(lane, v);
          if (row < P2) dots[row * kCorrLd + t0 + r] = acc[v];
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) f[s] = nf[s];
      }
    }
    combine(0, P2 * G2, x0, y0, w);
    return;
  }
  const float* fw = fmaps + (size_t)fj * H * W * D;
  for (int gi = g0; gi < P2; gi += dg) {
    // uniform over the wavefront
    const int x0 = __builtin_amdgcn_readfirstlane(__shfl(xl, gi)), x1 = __builtin_amdgcn_readfirstlane(__shfl(xh, gi));
    const int y0 = __builtin_amdgcn_readfirstlane(__shfl(yl, gi)), y1 = __builtin_amdgcn_readfirstlane(__shfl(yh, gi));
    const int w = x1 - x0, n = x1 > x0 ? w * (y1 - y0) : 0;
    const float rw = 1.f / (float)max(w, 1);
    // one row of products would leave 15 of 16 matrix rows idle: four pixels at
    // a time on the vector units, 16 lanes a pixel, so that a load covers 256
    // contiguous bytes of each; 16 pixels in flight.  Bound by those loads (128
    // channels, points 6 pixels apart: 1,000 edges 49 -> 40 us, 12,000 edges 470 -> 474;
    // one wavefront per point of every edge takes 57 and 584; at 256 channels 12,000
    // edges take 924 us so and 820 by points, which read neighbouring windows together).
    if (n > 0) {
      float4 h[VPL], f[4][VPL];
      const float4* hp = reinterpret_cast<const float4*>(gmap + ((size_t)k * P2 + gi) * D) + r;
      auto load = [&](int t0, float4(*o)[VPL]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = min(t0 + 4 * u + q, n - 1), y = (int)(((float)t + 0.5f) * rw), x = t - y * w;
          const float4* fp = reinterpret_cast<const float4*>(fw + ((size_t)(y0 + y) * W + (x0 + x)) * D) + r;
#pragma unroll
          for (int j = 0; j < VPL; ++j) o[u][j] = fp[16 * j];
        }
      };
#pragma unroll
      for (int j = 0; j < VPL; ++j) h[j] = hp[16 * j];
      load(0, f);
      for (int t0 = 0; t0 < n; t0 += 16) {
        float4 nf[4][VPL];
        load(t0 + 16, nf);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float d = row_sum(dot_tree<VPL>(h, f[u]));
          if (r == 0) dots[gi * kCorrLd + t0 + 4 * u + q] = d;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int j = 0; j < VPL; ++j) f[u][j] = nf[u][j];
      }
    }
    combine(gi * G2, (gi + 1) * G2, x0, y0, w);
  }
}

hipError_t launch_patch_correlation(int n_edges, int p, int dim, const float* gmap, int n_patches, const float* fmaps,
                                    int n_maps, int H, int W, const int* kk, const int* jj, const float* coords,
                                    float* corr, int* dev_err, int* host_err, hipStream_t st) {
  const int p2 = p * p;
  const long long items = (long long)n_edges * p2;
  if (items == 0) return hipSuccess;
  // 3 x 3 patches whose features and maps can be read as 16-byte vectors (the
  // rows are: dim is a multiple of 64).  Other patch sizes would leave more of
  // the 16 rows empty (1 x 1) or need several row tiles, and keep one
  // wavefront per patch pixel.
  const bool aligned = (((uintptr_t)gmap | (uintptr_t)fmaps) & 15) == 0 && ((uintptr_t)coords & 7) == 0;
  // Nor do a few edges of 256 channels, which are over when one wavefront has
  // loaded its first pixels (64 edges: 14.3 us by points, 17.5 by edges; 128
  // edges: 23.0 and 17.6; 192 channels: 14.6 and 14.4 at 64 edges).
  const int few = dim == 256 ? 96 : 0;
  if (p == 3 && aligned && n_edges > few) {
    const int per_group = n_edges <= kCorrSpread ? 1 : 4;
    const int grid3 = (n_edges + per_group - 1) / per_group;
    switch (dim / 64) {
#define DPVBA_CORR3_CASE(V)                                                                                        \
  case V:                                                                                                          \
    hipLaunchKernelGGL(patch_corr3_kernel<V>, dim3(grid3), dim3(256), 0, st, n_edges, per_group, gmap, n_patches,  \
                       fmaps, n_maps, H, W, kk, jj, coords, corr, dev_err, host_err);                                     \
    break;
      DPVBA_CORR3_CASE(1)
      DPVBA_CORR3_CASE(2)
      DPVBA_CORR3_CASE(3)
      DPVBA_CORR3_CASE(4)
#undef DPVBA_CORR3_CASE
      default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  const int grid = (int)((items + 3) / 4);
  switch (dim / 64) {
#define DPVBA_CORR_CASE(V)                                                                                         \
  case V:                                                                                                          \
    hipLaunchKernelGGL(patch_corr_kernel<V>, dim3(grid), dim3(256), 0, st, (int)items, p2, gmap, n_patches, fmaps, \
                       n_maps, H, W, kk, jj, coords, corr, dev_err, host_err);                                     \
    break;
    DPVBA_CORR_CASE(1)
    DPVBA_CORR_CASE(2)
    DPVBA_CORR_CASE(3)
    DPVBA_CORR_CASE(4)
#undef DPVBA_CORR_CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace dpvba
