// dmr_device.h -- device helpers shared by the forward kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace dmr {

// Base-level per-entity arithmetic, shared by the streaming kernel, the
// several-step kernel and the patch tiles of the combined step (which
// recompute coarse E on the patch boundary lines), so all round identically.
__device__ __forceinline__ float base_kap(float kn, float n0, float n1) { return kn * (0.5f * (n0 + n1)); }
__device__ __forceinline__ float base_hz(float hz, float S, float ey1, float ey, float exu, float ex) {
  return hz - S * ((ey1 - ey) - (exu - ex));
}
// new E from the old one, the curl term and J~; rc = 1 / (1 + kap)
__device__ __forceinline__ float base_ex(float e, float kap, float S, float h, float hp, float c1, float j, float rc) {
  return ((1.f - kap) * e + S * (h - hp) - c1 * j) * rc;
}
__device__ __forceinline__ float base_ey(float e, float kap, float curl, float c1, float j, float rc) {
  return ((1.f - kap) * e + curl - c1 * j) * rc;
}
__device__ __forceinline__ float base_rcp(float kap) { return __builtin_amdgcn_rcpf(1.f + kap); }
__device__ __forceinline__ float base_ex(float e, float kap, float S, float h, float hp, float c1, float j) {
  return base_ex(e, kap, S, h, hp, c1, j, base_rcp(kap));
}
__device__ __forceinline__ float base_ey(float e, float kap, float curl, float c1, float j) {
  return base_ey(e, kap, curl, c1, j, base_rcp(kap));
}

// Window accumulator of a node after a step: plus the mean square of its
// x-edges (left, right) and that of its y-edges (below, above).  A node on
// the outer boundary has one edge along that axis: the other value is 0 and
// the axis' factor f is 2 instead of 1.
__device__ __forceinline__ float base_win(float acc, float xl, float xr, float yd, float yu,
                                          float fx = 1.f, float fy = 1.f) {
  float sx = xl * xl;
  sx += xr * xr;
  float sy = yd * yd;
  sy += yu * yu;
  const float e2 = fx * sx + fy * sy;
  return acc + 0.5f * e2;
}

// Workgroups are dispatched to the 8 XCDs round-robin by linear id, and each
// XCD has its own L2.  Hand XCD x a contiguous band of the row-major
// (column block, segment) grid so that neighbouring blocks, which read the
// same cache lines at their common columns and rows, share an L2.
__device__ __forceinline__ int xcd_band(int L, int N) {
  const int x = L & 7, k = L >> 3, q = N >> 3, r = N & 7;
  return x * q + min(x, r) + k;
}

}  // namespace dmr
