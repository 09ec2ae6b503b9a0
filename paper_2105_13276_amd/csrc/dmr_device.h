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

// the same for a node of row 0, which has one y-edge (above, yu)
__device__ __forceinline__ float base_win0(float acc, float xl, float xr, float yu, float fx) {
  float sx = xl * xl;
  sx += xr * xr;
  const float mx = 0.5f * fx * sx;
  return acc + __builtin_fmaf(yu, yu, mx);
}

// ---------------------------------------------------------------------------
// Per-entity arithmetic of the patch substep, shared by the one-substep and
// the two-substep kernels so that all round identically.
// ---------------------------------------------------------------------------
// 5-point Laplacian; neighbours outside the patch already replaced by c
__device__ __forceinline__ float lap5(float c, float l, float r, float d, float u) {
  return l + r + d + u - 4.f * c;
}
// E filter of the patch interior: E - gamma L(L(E))
__device__ __forceinline__ float filter_e(float e, float gamma, float l2) { return e - gamma * l2; }
// Faraday, Eq. (2), scaled: H~ - S [(Ey_{i+1}-Ey_i) - (Ex_{j+1}-Ex_j)]
__device__ __forceinline__ float faraday(float ho, float S, float dey, float dex) {
  return ho - S * (dey - dex);
}
// Ampere + Drude, Eqs. (1), (3): new E from the old E, the curl term and J~
// (times the hardware reciprocal of 1 + kap, as the base level: two
// instructions where a correctly rounded division takes eleven)
__device__ __forceinline__ float ampere(float e, float kap, float curl, float c1, float jo) {
  return ((1.f - kap) * e + curl - c1 * jo) * __builtin_amdgcn_rcpf(1.f + kap);
}
// new J~ = a J~ + 2k (E + E+)
__device__ __forceinline__ float drude(float a, float jo, float kap, float e, float en) {
  return a * jo + 2.f * kap * (e + en);
}
// Eq. (5b): space weights w0, w1 on two coarse edges, time fraction frac
__device__ __forceinline__ float cfb(float w0, float w1, float o0, float o1, float n0, float n1,
                            float frac) {
  const float vo = w0 * o0 + w1 * o1;
  const float vn = w0 * n0 + w1 * n1;
  return (1.f - frac) * vo + frac * vn;
}
// window increment of a node from its existing edges (mean per axis)
__device__ __forceinline__ float win_e2(float sx, int cx, float sy, int cy) {
  return (cx == 2 ? 0.5f * sx : sx) + (cy == 2 ? 0.5f * sy : sy);
}

// value of the lane one column to the right / left (0 beyond the wave)
__device__ __forceinline__ float lane_right(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
      0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));  // wave_shl:1
}
__device__ __forceinline__ float lane_left(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
      0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));  // wave_shr:1
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
