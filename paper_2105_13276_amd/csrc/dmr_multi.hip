// dmr_multi.hip -- several base-level EM steps (Eqs. (1)-(3), Mur/PEC, TF/SF,
// E^2 window) in one launch, where nothing outside the level enters between
// them (no patch, or far enough from it).
//
// One step per launch moves 52 bytes per cell-update: every plane of the
// state is read and written once a step, and on small grids every step pays a
// launch and a memory round trip.  Here a block holds a region of 64 columns
// x NW R rows in registers (a lane one column, a wave R rows) and takes t
// steps of it; the region it can trust shrinks by one cell on each side per
// step, so it owns the 64 - 2t columns and NW R - 2t rows in the middle and
// recomputes the rest, which its neighbours own.  x-neighbours come from the
// next lane (DPP, no LDS), y-neighbours from the next register; only the rows
// at the border of two waves go through LDS, once a step (the wave below its
// first row recomputes that Hz row itself, so one barrier a step suffices).
// Every entity is computed by the operations of k_em_stream, so the results
// are identical to t launches of it.
#include "dmr_device.h"
#include "dmr_kernels.h"

namespace dmr {

namespace {

// The region is stepped by the interior update everywhere, also where it
// reaches beyond the grid.  Of E that does not exist, x-edges beside columns 0 and
// NX and y-edges of row NY reach an entity of the grid (the window of its boundary
// nodes) and are left out there, whatever they hold; all others end in entities
// that do not exist either, or in walls, which are set by themselves.  With PEC
// walls (P) E on them and beyond is set to +0 by bit masks.  XE: the region holds
// column 0 or NX or a source column; YE: the wave holds row 0 or NY.  A factor 0
// in place of 1 / (1 + kap) was cheaper, but left -0 and, beside an infinite value,
// NaN.  us a step of a uniform run, factor / masks in all forms / these: 256x128
// 1.91 / 1.97 / 1.89, 1024x512 3.27 / 3.33 / 3.30, 2048x1024 8.18 / 8.35 / 8.20,
// 8192x4096 103.4 / 105.0 / 102.9.
template <int R, bool XE, bool YE, bool P>
__device__ __forceinline__ void multi_tile(const MultiArgs& M, int t, const float2* in, float* hzp,
                                           int x0, int y0, int own_x, int own_lo, int own_hi,
                                           float (*sE)[3][64]) {
  const EMArgs& A = M.em;
  const int NX = A.R, NY = A.T;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nw = (int)(blockDim.x >> 6);
  const int i = x0 + lane, jt = y0 + w * R;  // column, first row of the wave
  const float S = A.S, c1 = A.c1, a = A.a, kn = A.kn, cm = A.cmur;

  // rows jt .. jt + R - 1 of every plane, row jt - 1 of Hz, row jt + R of n,
  // all requested before any is used
  float ex[R], ey[R], hz[R], jx[R], jy[R], ac[R], n[R + 1], hm;
  {
    const unsigned o = (unsigned)(XE ? min(max(i, 0), NX) : i) << 2;
    auto row = [&](const float* p, int j) {
      return *(const float*)((const char*)(p + (size_t)min(max(j, 0), NY) * A.pitch) + o);
    };
#pragma unroll
    for (int r = 0; r < R; r++) {
      n[r] = row(A.n, jt + r);
      ey[r] = row(A.ey0, jt + r);
      ex[r] = row(A.ex0, jt + r);
      hz[r] = row(A.hz0, jt + r);
      jx[r] = row(A.jx0, jt + r);
      jy[r] = row(A.jy0, jt + r);
      ac[r] = row(A.acc, jt + r);
    }
    n[R] = row(A.n, jt + R);
    hm = row(A.hz0, jt - 1);
  }
  const int rb = -jt, rt = NY - jt;  // rows 0 and NY of the grid in the wave
  const bool mur_x = !P || A.bc_x == kBcMur, mur_y = !P || A.bc_y == kBcMur;
  const bool c0 = i == 0, cN = i == NX;
  const bool mur0 = mur_x && x0 <= 0, murN = mur_x && x0 + 63 >= NX;
  const bool src = A.is > 0 && A.is >= x0 && A.is - 1 <= x0 + 63;
  const float fx = XE && (c0 || cN) ? 2.f : 1.f;

  // edges that exist (PEC walls left out): by column, and by row as bits r
  // (x-edges) and 16 + r (y-edges)
  const bool colx = !XE | ((i >= 0) & (i < NX));
  const bool coly = !XE | ((i >= 0) & (i <= NX) & (mur_x | !(c0 | cN)));
  int rows = 0;
  if (YE && P) {
#pragma unroll
    for (int r = 0; r < R; r++) {
      const int j = jt + r;
      rows |= ((j >= 0) & (j <= NY) & (mur_y | ((j != 0) & (j != NY)))) << r;
      rows |= ((j >= 0) & (j < NY)) << (16 + r);
    }
  }
  rows = __builtin_amdgcn_readfirstlane(rows);
  float kx[R], ky[R], rx[R], ry[R];
#pragma unroll
  for (int r = 0; r < R; r++) {
    kx[r] = base_kap(kn, n[r], lane_right(n[r]));
    ky[r] = base_kap(kn, n[r], n[r + 1]);
    rx[r] = base_rcp(kx[r]);
    ry[r] = base_rcp(ky[r]);
  }

  // window of the wave's node row r, Ey of the row below it
  auto window = [&](int r, float yd) {
    const float fy = YE && (r == rb || r == rt) ? 2.f : 1.f;
    const float yu = YE && !P && r == rt ? 0.f : ey[r];
    const float exl = lane_left(ex[r]);
    const float v = base_win(ac[r], exl, ex[r], yd, yu, fx, fy);
    const float v0 = base_win0(ac[r], exl, ex[r], ey[r], fx);
    return YE && r == rb ? v0 : v;
  };
  // the wave's border rows to its neighbours
  auto publish = [&](int b) {
    float (*e)[64] = sE[b * nw + w];
    e[0][lane] = ex[0];
    e[1][lane] = ex[R - 1];
    e[2][lane] = ey[R - 1];
  };

  // whether this launch writes the entities at (i, j)
  const bool in_sx = i >= M.sL && i < M.sR;
  auto mine = [&](int j) {
    if (M.near)
      return M.near[(size_t)(min(j, NY - 1) >> M.nbs) * M.nnx + (min(i, NX - 1) >> M.nbs)] == 0;
    return !(in_sx && j >= M.sB && j < M.sT);
  };

  for (int s = 0; s < t; s++) {
    const int b = (s & 1) * nw;
    // (a mask of its own for every row, kept over the steps, spilled)
    int rw = 0;
    if (YE && P) asm volatile("s_mov_b32 %0, %1" : "=s"(rw) : "s"(rows));
    auto keep = [&](float v, bool col, int bit) {
      int q = __builtin_bit_cast(int, v);
      if (YE && P) q &= (rw << (31 - bit)) >> 31;
      return XE && !col ? 0.f : __builtin_bit_cast(float, q);
    };
    publish(s & 1);
    __syncthreads();
    if (s == t - 1 && hzp) {  // Hz entering the last step
#pragma unroll
      for (int r = 0; r < R; r++) {
        const int j = jt + r;
        if (j >= own_lo && j < own_hi && j < NY && i >= own_x && lane < 64 - t && i < NX && mine(j))
          hzp[(size_t)j * A.pitch + i] = hz[r];
      }
    }
    const float exu = sE[b + (w + 1 < nw ? w + 1 : w)][0][lane];  // Ex of row jt + R
    const int wb = b + (w > 0 ? w - 1 : 0);
    const float exm = sE[wb][1][lane], eym = sE[wb][2][lane];  // row jt - 1
    // the window of the wave's first node row waits for Ey of the row below
    // (before the first step the accumulator stays)
    const float a0 = window(0, YE && rb == 0 ? 0.f : eym);
    ac[0] = s > 0 ? a0 : ac[0];

    // Faraday, Eq. (2)
    hm = base_hz(hm, S, lane_right(eym), eym, ex[0], exm);
#pragma unroll
    for (int r = 0; r < R; r++)
      hz[r] = base_hz(hz[r], S, lane_right(ey[r]), ey[r], r + 1 < R ? ex[r + 1 < R ? r + 1 : r] : exu,
                      ex[r]);
    // source terms; -0 (which changes no value) off the source columns
    float add_e = -0.f;
    if (XE && src) {
      const float add_h = i == A.is - 1 ? S * in[s].x : -0.f;
      add_e = i == A.is ? S * in[s].y : -0.f;
      hm += add_h;
#pragma unroll
      for (int r = 0; r < R; r++) hz[r] += add_h;
    }

    // Ampere + Drude, Eqs. (1), (3)
    float en[R];
#pragma unroll
    for (int r = 0; r < R; r++)
      en[r] = keep(base_ex(ex[r], kx[r], S, hz[r], r > 0 ? hz[r > 0 ? r - 1 : 0] : hm, c1, jx[r], rx[r]),
                   colx, r);
    if (YE && (!P || mur_y)) {
#pragma unroll
      for (int r = 0; r + 1 < R; r++) {
        const float eb = ex[r + 1] + cm * (en[r + 1] - ex[r]);
        const float et = ex[r] + cm * (en[r] - ex[r + 1]);
        if (r == rb) en[r] = colx ? eb : 0.f;
        if (r + 1 == rt) en[r + 1] = colx ? et : 0.f;
      }
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
      jx[r] = a * jx[r] + 2.f * kx[r] * (ex[r] + en[r]);
      ex[r] = en[r];
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
      float curl = -S * (hz[r] - lane_left(hz[r]));
      if (XE && src) curl += add_e;
      const float eyo = ey[r];
      en[r] = base_ey(eyo, ky[r], curl, c1, jy[r], ry[r]);
      if (P) en[r] = keep(en[r], coly, 16 + r);
      if (XE && mur0) {
        const float m = lane_right(eyo) + cm * (lane_right(en[r]) - eyo);
        en[r] = c0 ? m : en[r];
      }
      if (XE && murN) {
        const float m = lane_left(eyo) + cm * (lane_left(en[r]) - eyo);
        en[r] = cN ? m : en[r];
      }
      if (P && XE && YE && (jt + r < 0 || jt + r >= NY)) en[r] = 0.f;
      jy[r] = a * jy[r] + 2.f * ky[r] * (eyo + en[r]);
      ey[r] = en[r];
    }
#pragma unroll
    for (int r = 1; r < R; r++) ac[r] = window(r, ey[r - 1]);
  }
  publish(t & 1);
  __syncthreads();
  {
    const float eym = sE[(t & 1) * nw + (w > 0 ? w - 1 : 0)][2][lane];
    ac[0] = window(0, YE && rb == 0 ? 0.f : eym);
  }

  if (!(i >= own_x && lane < 64 - t) || i > NX) return;
  const unsigned o = (unsigned)i << 2;
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int j = jt + r;
    if (j < own_lo || j >= own_hi || !mine(j)) continue;
    const size_t ro = (size_t)j * A.pitch;
    auto put = [&](float* p, float v) { *(float*)((char*)(p + ro) + o) = v; };
    if (!XE || i < NX) {
      if (j < NY) put(A.hz1, hz[r]);
      put(A.ex1, ex[r]);
      put(A.jx1, jx[r]);
    }
    if (j < NY) {
      put(A.ey1, ey[r]);
      put(A.jy1, jy[r]);
    }
    put(A.acc1, ac[r]);
  }
}

// Block (bx, by) of the t-step launch; in: the incident values of the steps,
// hzp: where Hz entering the last one goes (nullable)
template <int R>
__device__ __forceinline__ void multi_block(const MultiArgs& M, int t, const float2* in, float* hzp,
                                            int bx, int by, float (*sE)[3][64]) {
  const EMArgs& A = M.em;
  const int rows = (int)(blockDim.x >> 6) * R;
  const int NX = A.R, NY = A.T;
  const int own_x = bx * (64 - 2 * t);
  const int own_lo = by * (rows - 2 * t);
  const int own_hi = min(own_lo + rows - 2 * t, NY + 1);
  // Mur entities depend on the new value one cell further in: a region that
  // owns none but the last column (row) takes one more beside it
  const int x0 = own_x - t - (own_x == NX ? 1 : 0);
  // Ex(i, 0) is formed with Ex(i, 1) and Ex(i, NY) with Ex(i, NY-1), which
  // have to be rows of one wave: shift the region by a row where they are not
  // (towards the inside of the grid, where the boundary leaves rows to spare)
  int y0 = own_lo - t - (own_lo == NY ? 1 : 0);
  if (y0 <= 0 && NY - y0 < rows) y0 = NY % R == 0 ? -1 : 0;
  else if (y0 <= 0 && -y0 % R == R - 1) y0++;
  else if (y0 > 0 && NY - y0 < rows && (NY - y0) % R == 0) y0--;
  // nothing of it is this launch's to write
  if (own_x >= M.sL && min(own_x + 64 - 2 * t, NX + 1) <= M.sR && own_lo >= M.sB && own_hi <= M.sT)
    return;
  const bool xe = x0 < 1 || x0 + 63 > NX - 1 || (A.is > 0 && A.is >= x0 && A.is - 1 <= x0 + 63);
  // (chosen per wave; every form passes the same barriers)
  const int jt = y0 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * R;
  const bool ye = jt < 1 || jt + R > NY;
  const bool pec = A.bc_x != kBcMur || A.bc_y != kBcMur;
#define TILE(X, Y, P) multi_tile<R, X, Y, P>(M, t, in, hzp, x0, y0, own_x, own_lo, own_hi, sE)
  if (!xe && !ye) TILE(false, false, false);
  else if (pec) {
    if (xe && ye) TILE(true, true, true);
    else if (xe) TILE(true, false, true);
    else TILE(false, true, true);
  } else {
    if (xe && ye) TILE(true, true, false);
    else if (xe) TILE(true, false, false);
    else TILE(false, true, false);
  }
#undef TILE
}

// R rows a wave, at most NW waves a block, EU waves per SIMD
template <int R, int NW, int EU>
__global__ __launch_bounds__(64 * NW, EU) void k_em_multi(MultiArgs M) {
  __shared__ float sE[2 * NW][3][64];
  const int b = xcd_band(blockIdx.x, M.ntx * M.nty);
  multi_block<R>(M, M.t, M.src, M.hzp, b % M.ntx, b / M.ntx, sE);
}

// over the blocks of many instances, blk[b] = (instance, block within it);
// step k of the interval is the first, its incident values src[instance *
// kSrcSteps + k]
template <int R, int NW, int EU>
__global__ __launch_bounds__(64 * NW, EU) void k_em_multi_batch(const MultiArgs* __restrict__ args,
                                                                const int2* __restrict__ blk,
                                                                const float2* __restrict__ src,
                                                                int k, int t, int last) {
  __shared__ float sE[2 * NW][3][64];
  const int2 bi = blk[blockIdx.x];
  const MultiArgs& M = args[bi.x];
  multi_block<R>(M, t, src + (size_t)bi.x * kSrcSteps + k, last ? M.hzp : nullptr, bi.y % M.ntx,
                 bi.y / M.ntx, sE);
}

}  // namespace

bool multi_grid(MultiArgs* M, int waves) {
  const int t = M->t, h = 4 * waves - 2 * t;
  if (t < 1 || t > kMultiSteps || waves < 1 || waves > 16 || h < 2) return false;
  M->ntx = (M->em.R + 1 + 63 - 2 * t) / (64 - 2 * t);
  M->nty = (M->em.T + 1 + h - 1) / h;
  return true;
}

hipError_t launch_em_multi_batch(const MultiArgs* args, const int2* blk, int nblk,
                                 const float2* src, int k, int t, int last, int waves,
                                 hipStream_t st) {
  if (nblk <= 0) return hipSuccess;
  if (waves > 12) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_em_multi_batch<4, 12, 6>), dim3(nblk), dim3(64 * waves), 0, st, args, blk,
                     src, k, t, last);
  return hipGetLastError();
}

hipError_t launch_em_multi(MultiArgs& M, int waves, hipStream_t st) {
  if (!multi_grid(&M, waves)) return hipErrorInvalidValue;
  const dim3 g(M.ntx * M.nty), bl(64 * waves);
  if (waves <= 8) hipLaunchKernelGGL((k_em_multi<4, 8, 5>), g, bl, 0, st, M);
  else if (waves <= 12) hipLaunchKernelGGL((k_em_multi<4, 12, 6>), g, bl, 0, st, M);
  else hipLaunchKernelGGL((k_em_multi<4, 16, 4>), g, bl, 0, st, M);
  return hipGetLastError();
}

}  // namespace dmr
