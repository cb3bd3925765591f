// Map growth: expansion by the opacity mask (Sec. III-C.2, Eq. 8) and sky Gaussians
// initialised from nearest-neighbour distances (Sec. III-C.1).
//
// Expansion: one lane per candidate point projects it into the keyframe view, finds the
// pixel it falls on and keeps it when the pixel's opacity O = 1 - T_final is below tau.
// The kept points are compacted in input order (exclusive scan of the flags) and become
// Gaussians by the point initialisation rule. The pixel is an integer decision taken in
// FP32 with a fixed operation order and no contraction:
//   x_c = ((R00 x + R01 y) + R02 z) + t0 (same for y_c, z_c), u = f_x (x_c / z_c) + c_x,
//   inside = z_c > near and 0 <= u < W and 0 <= v < H, pixel = (floor u, floor v).
#include "gs_common.h"
#include "kernels.h"

namespace gs {

__global__ void __launch_bounds__(256)
k_expand_flags(const float* __restrict__ xyz, int64_t n, ViewDev V, const float* __restrict__ T, float tau,
               float near_z, uint32_t* __restrict__ flags) {
#pragma clang fp contract(off)
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const float x = xyz[3 * j], y = xyz[3 * j + 1], z = xyz[3 * j + 2];
  const float xc = ((V.R[0] * x + V.R[1] * y) + V.R[2] * z) + V.t[0];
  const float yc = ((V.R[3] * x + V.R[4] * y) + V.R[5] * z) + V.t[1];
  const float zc = ((V.R[6] * x + V.R[7] * y) + V.R[8] * z) + V.t[2];
  uint32_t keep = 0;
  if (zc > near_z) {
    const float u = V.fx * __fdiv_rn(xc, zc) + V.cx;
    const float v = V.fy * __fdiv_rn(yc, zc) + V.cy;
    if (u >= 0.0f && u < (float)V.W && v >= 0.0f && v < (float)V.H) {
      const int px = min((int)floorf(u), V.W - 1), py = min((int)floorf(v), V.H - 1);
      const float O = 1.0f - T[(int64_t)py * V.W + px];
      keep = O < tau ? 1u : 0u;
    }
  }
  flags[j] = keep;
}

// Sec. III-C.1 row initialisation shared by every point source: mean, isotropic
// log-scale, identity rotation, opacity logit, SH DC from a colour (colour = Y00 dc + 0.5),
// higher SH zero; gradients and Adam moments zero; not visible.
__device__ __forceinline__ void init_row(float* __restrict__ buf, int64_t cap, int32_t F, int32_t K, int64_t i,
                                         float x, float y, float z, float ls, float logit0, float r, float g,
                                         float b, uint8_t* __restrict__ vis) {
  float* P = buf;
  P[i] = x;
  P[cap + i] = y;
  P[2 * cap + i] = z;
  P[3 * cap + i] = ls;
  P[4 * cap + i] = ls;
  P[5 * cap + i] = ls;
  P[6 * cap + i] = 1.0f;
  P[7 * cap + i] = 0.0f;
  P[8 * cap + i] = 0.0f;
  P[9 * cap + i] = 0.0f;
  P[10 * cap + i] = logit0;
  P[11 * cap + i] = (r - 0.5f) / kSH0;
  P[12 * cap + i] = (g - 0.5f) / kSH0;
  P[13 * cap + i] = (b - 0.5f) / kSH0;
  for (int f = 14; f < 11 + 3 * K; ++f) P[f * cap + i] = 0.0f;
  for (int f = 0; f < F; ++f) {
    buf[(int64_t)(F + f) * cap + i] = 0.0f;
    buf[(int64_t)(2 * F + f) * cap + i] = 0.0f;
    buf[(int64_t)(3 * F + f) * cap + i] = 0.0f;
  }
  vis[i] = 0;
}

// Kept points (flags[j] = 1) go to row n0 + offsets[j]; scale d / f_x with d the point's
// camera-frame depth clamped below at near.
__global__ void __launch_bounds__(256)
k_init_selected(float* __restrict__ buf, int64_t cap, int32_t F, int32_t K, int64_t n0, int64_t n,
                const float* __restrict__ xyz, const float* __restrict__ rgb, const uint32_t* __restrict__ flags,
                const uint32_t* __restrict__ offsets, ViewDev V, float near_z, float logit0,
                uint8_t* __restrict__ vis) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n || !flags[j]) return;
  const float x = xyz[3 * j], y = xyz[3 * j + 1], z = xyz[3 * j + 2];
  const float d = V.R[6] * x + V.R[7] * y + V.R[8] * z + V.t[2];
  init_row(buf, cap, F, K, n0 + offsets[j], x, y, z, logf(fmaxf(d, near_z) / V.fx), logit0, rgb[3 * j],
           rgb[3 * j + 1], rgb[3 * j + 2], vis);
}

// Squared distance from each point to its closest other point: every lane owns kNnPer points
// and sweeps its block's segment of all points through LDS in tiles of 256; part[s n + j] is
// point j's least over segment s. Bound by VALU work (seven instructions per pair, of which
// none but the minimum's order may change: a pair's distance rounds as it always did). With
// one block per 256 points and no segments a sky of 20k ran on 79 of 256 CUs, 1389 us; with
// enough segments for kNnBlocks blocks 97.
constexpr int kNnThreads = 256, kNnPer = 2, kNnBlocks = 2048;
__global__ void __launch_bounds__(kNnThreads)
k_nn_dist2(const float* __restrict__ xyz, int64_t n, float* __restrict__ part) {
  __shared__ float4 s_p[kNnThreads];
  const int64_t j0 = (int64_t)blockIdx.x * (kNnThreads * kNnPer);
  float x[kNnPer], y[kNnPer], z[kNnPer], best[kNnPer];
#pragma unroll
  for (int u = 0; u < kNnPer; ++u) {
    const int64_t j = j0 + u * kNnThreads + threadIdx.x;
    x[u] = y[u] = z[u] = 0.f;
    best[u] = __builtin_huge_valf();
    if (j < n) {
      x[u] = xyz[3 * j];
      y[u] = xyz[3 * j + 1];
      z[u] = xyz[3 * j + 2];
    }
  }
  const int64_t tiles = (n + kNnThreads - 1) / kNnThreads;
  const int64_t b0 = (int64_t)blockIdx.y * tiles / gridDim.y, b1 = (int64_t)(blockIdx.y + 1) * tiles / gridDim.y;
  for (int64_t b = b0; b < b1; ++b) {
    const int64_t base = b * kNnThreads, k = base + threadIdx.x;
    __syncthreads();
    // (past the end: infinitely far)
    const float inf = __builtin_huge_valf();
    s_p[threadIdx.x] = k < n ? make_float4(xyz[3 * k], xyz[3 * k + 1], xyz[3 * k + 2], 0.f) : make_float4(inf, inf, inf, 0.f);
    __syncthreads();
    const int64_t own = base - j0;
    const bool meets = own >= 0 && own < kNnThreads * kNnPer;  // the tile holds points of this block
#pragma unroll 8
    for (int t = 0; t < kNnThreads; ++t) {
      const float4 p = s_p[t];
#pragma unroll
      for (int u = 0; u < kNnPer; ++u) {
        const float dx = p.x - x[u], dy = p.y - y[u], dz = p.z - z[u];
        const float e = __fmaf_rn(dz, dz, __fmaf_rn(dx, dx, __fmul_rn(dy, dy)));
        if (!meets || (int)own + t != u * kNnThreads + (int)threadIdx.x) best[u] = fminf(best[u], e);
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kNnPer; ++u) {
    const int64_t j = j0 + u * kNnThreads + threadIdx.x;
    if (j < n) part[blockIdx.y * n + j] = best[u];
  }
}
static int64_t nn_blocks(int64_t n) { return (n + kNnThreads * kNnPer - 1) / (kNnThreads * kNnPer); }
int nn_segments(int64_t n) {
  const int64_t tiles = (n + kNnThreads - 1) / kNnThreads;
  return (int)std::max<int64_t>(1, std::min(tiles, kNnBlocks / nn_blocks(n)));
}

// Sky rows: white DC, opacity logit0, isotropic scale = nearest-neighbour distance.
__global__ void __launch_bounds__(256)
k_init_sky(float* __restrict__ buf, int64_t cap, int32_t F, int32_t K, int64_t n0, int64_t n,
           const float* __restrict__ xyz, const float* __restrict__ part, int segments, float logit0,
           uint8_t* __restrict__ vis) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  float d2 = part[j];
#pragma unroll 8
  for (int g = 1; g < segments; ++g) d2 = fminf(d2, part[g * n + j]);
  init_row(buf, cap, F, K, n0 + j, xyz[3 * j], xyz[3 * j + 1], xyz[3 * j + 2], 0.5f * logf(d2), logit0, 1.0f,
           1.0f, 1.0f, vis);
}

static unsigned blocks(int64_t n) { return (unsigned)((n + 255) / 256); }

hipError_t expand_flags(const float* xyz, int64_t n, const ViewDev& V, const float* T, float tau, float near_z,
                        uint32_t* flags, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_expand_flags, dim3(blocks(n)), dim3(256), 0, s, xyz, n, V, T, tau, near_z, flags);
  return hipGetLastError();
}

hipError_t init_selected(float* buf, int64_t cap, int32_t F, int32_t K, int64_t n0, int64_t n, const float* xyz,
                         const float* rgb, const uint32_t* flags, const uint32_t* offsets, const ViewDev& V,
                         float near_z, float logit0, uint8_t* vis, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_init_selected, dim3(blocks(n)), dim3(256), 0, s, buf, cap, F, K, n0, n, xyz, rgb, flags,
                     offsets, V, near_z, logit0, vis);
  return hipGetLastError();
}

hipError_t init_sky(float* buf, int64_t cap, int32_t F, int32_t K, int64_t n0, int64_t n, const float* xyz,
                    float* d2, float logit0, uint8_t* vis, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int segments = nn_segments(n);
  hipLaunchKernelGGL(k_nn_dist2, dim3((unsigned)nn_blocks(n), (unsigned)segments), dim3(kNnThreads), 0, s, xyz, n, d2);
  hipLaunchKernelGGL(k_init_sky, dim3(blocks(n)), dim3(256), 0, s, buf, cap, F, K, n0, n, xyz, d2, segments, logit0, vis);
  return hipGetLastError();
}

}  // namespace gs
