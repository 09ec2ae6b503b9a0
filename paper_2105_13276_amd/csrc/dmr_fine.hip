// dmr_fine.hip -- both r = 2 substeps of a coarse step on the rectangular patch
// (Eqs. (1)-(3), E filter, Eq. (5b), fine -> coarse transfer) in registers.
//
// The one-substep tiles move the patch state once a substep, and the LDS tiles
// that take both substeps spend their time in LDS phases (a 13-point filter
// read from LDS twice).  Here a block holds a region of 64 columns x NW R rows
// in registers (a lane one column, a wave R rows): x-neighbours come from the
// next lane (DPP), y-neighbours from the next register, and only the rows at
// the border of two waves go through LDS (two of raw E for the filter, one of
// filtered E for Faraday).  A substep reaches 3 cells, and the window one more
// to the left and below: of the region the block owns the columns and rows
// from 8 on and up to 6 before its end, whole 2 x 2 coarse cells.  Every entity is
// computed by the operations of the other patch kernels (dmr_device.h), so the
// results are identical.
#include "dmr_device.h"
#include "dmr_kernels.h"

namespace dmr {

namespace {

constexpr int kLo = 8, kHi = 6;  // halo below / left, above / right

// XE: the region reaches column L or R of the patch, YE: the wave reaches row
// B or T (one beyond counts).  sR: raw E rows of every wave (0, 1 and R-2, R-1
// of Ex and Ey), sF: filtered Ex rows 0, R-1 and Ey row R-1.
template <int R, bool XE, bool YE>
__device__ __forceinline__ void fine_reg_tile(const EMArgs& A, int x0, int y0, int own_x, int own_y,
                                              int end_y, float (*sR)[8][64], float (*sF)[3][64]) {
  const int L = A.L, RR = A.R, B = A.B, T = A.T, pitch = A.pitch;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int nw = (int)(blockDim.x >> 6);
  const int i = x0 + lane, jt = y0 + w * R;
  const bool filt = A.gamma > 0.f;

  // every load before any use, from addresses clamped into the patch
  float ex[R], ey[R], hz[R], jx[R], jy[R], ac[R], n[R + 1], hm;
  {
    const unsigned oc = (unsigned)(XE ? min(max(i, L), RR - 1) : i) << 2;  // cells, x-edges
    const unsigned on = (unsigned)(XE ? min(max(i, L), RR) : i) << 2;      // y-edges, nodes
    auto row = [&](const float* p, int j, unsigned o) {
      return *(const float*)((const char*)(p + (size_t)j * pitch) + o);
    };
    auto jc = [&](int j) { return min(max(j, B), T - 1); };
    auto jn = [&](int j) { return min(max(j, B), T); };
#pragma unroll
    for (int r = 0; r < R; r++) {
      const int j = jt + r;
      ex[r] = row(A.ex0, jn(j), oc);
      ey[r] = row(A.ey0, jc(j), on);
      n[r] = row(A.n, jn(j), on);
      hz[r] = row(A.hz0, jc(j), oc);
      jx[r] = row(A.jx0, jn(j), oc);
      jy[r] = row(A.jy0, jc(j), on);
      ac[r] = 0.f;
      if (j >= own_y && j < end_y) ac[r] = row(A.acc, j, on);
    }
    n[R] = row(A.n, jn(jt + R), on);
    hm = row(A.hz0, jc(jt - 1), oc);
  }
  // Eq. (5b): on rows B and T from the two coarse x-edges of the line beside
  // this column, on columns L and R from the two coarse y-edges beside each
  // row, before (o) and after (a) the coarse step
  const int rb = B - jt, rt = T - jt;  // rows B and T in the wave
  const bool cL = i == L, cR = i == RR;
  const bool odd = ((i - L) & 1) != 0;
  float bo[2] = {0.f, 0.f}, ba[2] = {0.f, 0.f};        // rows B, T
  float co[XE ? R : 1], ca[XE ? R : 1];                // columns
  if (YE) {
    const int ii = min(max(i, L), RR - 1);
    const int k = (ii & 1) ? ii >> 1 : (ii >> 1) - 1;
    const float w0 = (ii & 1) ? 0.75f : 0.25f, w1 = (ii & 1) ? 0.25f : 0.75f;
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const size_t o = (size_t)((q ? T : B) >> 1) * A.cpitch + k;
      bo[q] = w0 * A.cex0[o] + w1 * A.cex0[o + 1];
      ba[q] = w0 * A.cex1[o] + w1 * A.cex1[o + 1];
    }
  }
  if (XE) {
    const int I = (cR ? RR : L) >> 1;
#pragma unroll
    for (int r = 0; r < R; r++) {
      const int j = min(max(jt + r, B), T - 1);
      const int k = (j & 1) ? j >> 1 : (j >> 1) - 1;
      const float w0 = (j & 1) ? 0.75f : 0.25f, w1 = (j & 1) ? 0.25f : 0.75f;
      const size_t o = (size_t)k * A.cpitch + I, o1 = o + A.cpitch;
      co[r] = w0 * A.cey0[o] + w1 * A.cey0[o1];
      ca[r] = w0 * A.cey1[o] + w1 * A.cey1[o1];
    }
  }
  float kx[R], ky[R];
#pragma unroll
  for (int r = 0; r < R; r++) {
    const float nex = 0.5f * (n[r] + lane_right(n[r]));
    const float ney = 0.5f * (n[r] + n[r + 1]);
    kx[r] = A.kn * nex;
    ky[r] = A.kn * ney;
  }

  // 5-point Laplacian at a row: c and the rows below and above; x the column
  // extent of the component (left end lo, right end hi of the patch): a
  // neighbour outside is replaced by c
  auto lap = [&](float c, float d, float u, bool lo, bool hi) {
    float l = lane_left(c), r = lane_right(c);
    if (XE) {
      l = lo ? c : l;
      r = hi ? c : r;
    }
    return lap5(c, l, r, d, u);
  };
  const bool xl = cL, xr = i == RR - 1, yl = cL, yr = cR;  // ends of Ex, of Ey

  auto window = [&](int r, float xw, float ys) {  // Ex of the left edge, Ey of the one below
    float a = xw, b = ex[r], d = ys, u = ey[r];
    int cx = 2, cy = 2;
    if (XE) {
      a = cL ? 0.f : a;
      b = cR ? 0.f : b;
      cx = (cL | cR) ? 1 : 2;
    }
    if (YE) {
      d = r == rb ? 0.f : d;
      u = r == rt ? 0.f : u;
      cy = r == rb || r == rt ? 1 : 2;
    }
    float sx = 0.f, sy = 0.f;
    sx += a * a;
    sx += b * b;
    sy += d * d;
    sy += u * u;
    return ac[r] + win_e2(sx, cx, sy, cy);
  };

  float h1[R];  // Hz after substep 1
  const int wd = w > 0 ? w - 1 : 0, wu = w + 1 < nw ? w + 1 : w;
#pragma unroll 1
  for (int m = 0; m < 2; m++) {
    // raw E of the rows next to the wave's borders
    {
      float (*p)[64] = sR[w];
      p[0][lane] = ex[0]; p[1][lane] = ex[1];
      p[2][lane] = ex[R - 2]; p[3][lane] = ex[R - 1];
      p[4][lane] = ey[0]; p[5][lane] = ey[1];
      p[6][lane] = ey[R - 2]; p[7][lane] = ey[R - 1];
    }
    __syncthreads();
    const float exd1 = sR[wd][3][lane], exd2 = sR[wd][2][lane];  // rows jt-1, jt-2
    const float eyd1 = sR[wd][7][lane], eyd2 = sR[wd][6][lane];
    const float exu1 = sR[wu][0][lane], exu2 = sR[wu][1][lane];  // rows jt+R, jt+R+1
    const float eyu1 = sR[wu][4][lane], eyu2 = sR[wu][5][lane];
    // the window of the first node row after substep 1 waited for Ey below
    const float a0 = window(0, lane_left(ex[0]), eyd1);
    ac[0] = m > 0 ? a0 : ac[0];
    if (filt) {
      // L(E) on rows jt-1 .. jt+R, then E - gamma L(L(E)) of the interior edges
      float qx[R + 2], qy[R + 2];
#pragma unroll
      for (int r = -1; r <= R; r++) {
        const float cx = r < 0 ? exd1 : r >= R ? exu1 : ex[r < 0 ? 0 : r >= R ? 0 : r];
        float dx = r < 0 ? exd2 : r == 0 ? exd1 : ex[r <= 0 ? 0 : r - 1];
        float ux = r >= R ? exu2 : r == R - 1 ? exu1 : ex[r >= R - 1 ? 0 : r + 1];
        const float cy = r < 0 ? eyd1 : r >= R ? eyu1 : ey[r < 0 ? 0 : r >= R ? 0 : r];
        float dy = r < 0 ? eyd2 : r == 0 ? eyd1 : ey[r <= 0 ? 0 : r - 1];
        float uy = r >= R ? eyu2 : r == R - 1 ? eyu1 : ey[r >= R - 1 ? 0 : r + 1];
        if (YE) {
          dx = r == rb ? cx : dx;
          ux = r == rt ? cx : ux;
          dy = r == rb ? cy : dy;
          uy = r == rt - 1 ? cy : uy;
        }
        qx[r + 1] = lap(cx, dx, ux, xl, xr);
        qy[r + 1] = lap(cy, dy, uy, yl, yr);
      }
#pragma unroll
      for (int r = 0; r < R; r++) {
        float dx = qx[r], ux = qx[r + 2], dy = qy[r], uy = qy[r + 2];
        if (YE) {
          dx = r == rb ? qx[r + 1] : dx;
          ux = r == rt ? qx[r + 1] : ux;
          dy = r == rb ? qy[r + 1] : dy;
          uy = r == rt - 1 ? qy[r + 1] : uy;
        }
        const float fx = filter_e(ex[r], A.gamma, lap(qx[r + 1], dx, ux, xl, xr));
        const float fy = filter_e(ey[r], A.gamma, lap(qy[r + 1], dy, uy, yl, yr));
        ex[r] = YE && (r == rb || r == rt) ? ex[r] : fx;
        ey[r] = (XE && (cL | cR)) ? ey[r] : fy;
      }
    }
    sF[w][0][lane] = ex[0];
    sF[w][1][lane] = ex[R - 1];
    sF[w][2][lane] = ey[R - 1];
    __syncthreads();
    const float fxu = sF[wu][0][lane], fxd = sF[wd][1][lane], fyd = sF[wd][2][lane];
    // Faraday, Eq. (2) (row jt-1 here too, for Ampere of the first row)
    {
      const float dey = lane_right(fyd) - fyd;
      const float dex = ex[0] - fxd;
      hm = faraday(hm, A.S, dey, dex);
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
      const float dey = lane_right(ey[r]) - ey[r];
      const float dex = (r + 1 < R ? ex[r + 1 < R ? r + 1 : r] : fxu) - ex[r];
      hz[r] = faraday(hz[r], A.S, dey, dex);
      if (m == 0) h1[r] = hz[r];
    }
    // Ampere + Drude, Eqs. (1), (3); the boundary edges take Eq. (5b)
    const float frac = m ? 1.f : A.frac;
#pragma unroll
    for (int r = 0; r < R; r++) {
      const float dhx = hz[r] - (r > 0 ? hz[r > 0 ? r - 1 : 0] : hm);
      float en = ampere(ex[r], kx[r], A.S * dhx, A.c1, jx[r]);
      if (YE) {
        const float v0 = (1.f - frac) * bo[0] + frac * ba[0];
        const float v1 = (1.f - frac) * bo[1] + frac * ba[1];
        en = r == rb ? v0 : r == rt ? v1 : en;
      }
      jx[r] = drude(A.a, jx[r], kx[r], ex[r], en);
      ex[r] = en;
      const float dhy = hz[r] - lane_left(hz[r]);
      en = ampere(ey[r], ky[r], -A.S * dhy, A.c1, jy[r]);
      if (XE) {
        const float v = (1.f - frac) * co[r] + frac * ca[r];
        en = (cL | cR) ? v : en;
      }
      jy[r] = drude(A.a, jy[r], ky[r], ey[r], en);
      ey[r] = en;
    }
#pragma unroll
    for (int r = 1; r < R; r++) ac[r] = window(r, lane_left(ex[r]), ey[r - 1]);
  }
  sR[w][7][lane] = ey[R - 1];  // (sF may still be read)
  __syncthreads();
  ac[0] = window(0, lane_left(ex[0]), sR[wd][7][lane]);

  // results: own columns and rows of the patch
  const bool own = i >= own_x && lane < 64 - kHi && i <= RR;
  const unsigned o = (unsigned)i << 2;
#pragma unroll
  for (int r = 0; r < R; r++) {
    const int j = jt + r;
    if (j < own_y || j >= end_y || !own) continue;
    const size_t ro = (size_t)j * pitch;
    auto put = [&](float* p, float v) { *(float*)((char*)(p + ro) + o) = v; };
    if (!XE || i < RR) {
      if (j < T) put(A.hz1, hz[r]);
      put(A.ex1, ex[r]);
      put(A.jx1, jx[r]);
    }
    if (j < T) {
      put(A.ey1, ey[r]);
      put(A.jy1, jy[r]);
    }
    put(A.acc, ac[r]);
  }
  // fine -> coarse transfer: rows come in pairs of the same wave, columns by
  // the lane to the right
#pragma unroll
  for (int r = 0; r < R; r += 2) {
    const int j = jt + r;
    const float a0 = h1[r] + hz[r], a1 = h1[r + 1] + hz[r + 1];
    const float b0 = lane_right(a0), b1 = lane_right(a1);
    const float ex1 = lane_right(ex[r]), jx1 = lane_right(jx[r]);
    if (j < own_y || j >= end_y || !own || odd || i >= RR || j >= T) continue;
    const size_t c = (size_t)(j >> 1) * A.cpitch + (i >> 1);
    float s = 0.f;
    s += 0.5f * a0;
    s += 0.5f * a1;
    s += 0.5f * b0;
    s += 0.5f * b1;
    A.chz[c] = 0.25f * s;
    if (!YE || (j > B)) {
      A.cex[c] = 0.5f * (ex[r] + ex1);
      A.cjx[c] = jx[r] + jx1;  // J~ scales with dt
    }
    if (!XE || i > L) {
      A.cey[c] = 0.5f * (ey[r] + ey[r + 1]);
      A.cjy[c] = jy[r] + jy[r + 1];
    }
  }
}

template <int R>
__device__ __forceinline__ void fine_reg_block(const EMArgs& A, int bx, int by, float (*sR)[8][64],
                                               float (*sF)[3][64]) {
  const int rows = (int)(blockDim.x >> 6) * R;
  const int own_x = A.L + bx * (64 - kLo - kHi), own_y = A.B + by * (rows - kLo - kHi);
  const int end_y = min(own_y + rows - kLo - kHi, A.T + 1);
  const int x0 = own_x - kLo, y0 = own_y - kLo;
  const bool xe = (x0 <= A.L) | (x0 + 63 >= A.R - 1);
  // (per wave; every form passes the same barriers)
  const int jt = y0 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * R;
  const bool ye = (jt - 1 <= A.B) | (jt + R + 1 >= A.T);
  if (xe && ye) fine_reg_tile<R, true, true>(A, x0, y0, own_x, own_y, end_y, sR, sF);
  else if (xe) fine_reg_tile<R, true, false>(A, x0, y0, own_x, own_y, end_y, sR, sF);
  else if (ye) fine_reg_tile<R, false, true>(A, x0, y0, own_x, own_y, end_y, sR, sF);
  else fine_reg_tile<R, false, false>(A, x0, y0, own_x, own_y, end_y, sR, sF);
}

template <int R, int NW, int EU>
__global__ __launch_bounds__(64 * NW, EU) void k_fine_reg(EMArgs A) {
  __shared__ float sR[NW][8][64], sF[NW][3][64];
  const int nbx = (A.R - A.L + 1 + 63 - kLo - kHi) / (64 - kLo - kHi);
  const int b = xcd_band(blockIdx.x, gridDim.x);
  fine_reg_block<R>(A, b % nbx, b / nbx, sR, sF);
}

// blk[b] = (instance, block within its patch)
template <int R, int NW, int EU>
__global__ __launch_bounds__(64 * NW, EU) void k_fine_reg_batch(const EMArgs* __restrict__ args,
                                                                const int2* __restrict__ blk) {
  __shared__ float sR[NW][8][64], sF[NW][3][64];
  const int2 bi = blk[blockIdx.x];
  const EMArgs& A = args[bi.x];
  const int nbx = (A.R - A.L + 1 + 63 - kLo - kHi) / (64 - kLo - kHi);
  fine_reg_block<R>(A, bi.y % nbx, bi.y / nbx, sR, sF);
}

}  // namespace

// waves per block for patches of `count` x (w, h) cells in all: the region of
// a block is 4 rows a wave, and a compute unit holds one block of 12 or 16
// waves or two of 8
int fine_reg_waves(const int* w, const int* h, int count) {
  const int ws[] = {16, 12, 8}, held[] = {1, 1, 2};
  int best = 16;
  double least = 1e30;
  for (int k = 0; k < 3; k++) {
    long n = 0;
    for (int q = 0; q < count; q++) n += (long)fine_reg_blocks(w[q], h[q], ws[k]);
    const double cost = (double)((n + 256 * held[k] - 1) / (256 * held[k])) * (6.0 + 0.45 * ws[k]);
    if (cost < least) { least = cost; best = ws[k]; }
  }
  return best;
}

int fine_reg_blocks(int w, int h, int waves) {
  const int own = 64 - kLo - kHi, rows = 4 * waves - kLo - kHi;
  return ((w + 1 + own - 1) / own) * ((h + 1 + rows - 1) / rows);
}

hipError_t launch_fine_reg(const EMArgs& A, int waves, hipStream_t st) {
  if (A.rf == 4 || A.act || A.stn || !A.restrict_on) return hipErrorInvalidValue;
  const int w = A.R - A.L, h = A.T - A.B;
  if (waves <= 0) waves = fine_reg_waves(&w, &h, 1);
  const dim3 g(fine_reg_blocks(w, h, waves)), bl(64 * waves);
  if (waves == 16) hipLaunchKernelGGL((k_fine_reg<4, 16, 4>), g, bl, 0, st, A);
  else if (waves == 12) hipLaunchKernelGGL((k_fine_reg<4, 12, 5>), g, bl, 0, st, A);
  else if (waves == 8) hipLaunchKernelGGL((k_fine_reg<4, 8, 5>), g, bl, 0, st, A);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_fine_reg_batch(const EMArgs* args, const int2* blk, int nblk, int waves,
                                 hipStream_t st) {
  if (nblk <= 0) return hipSuccess;
  const dim3 g(nblk), bl(64 * waves);
  if (waves == 16) hipLaunchKernelGGL((k_fine_reg_batch<4, 16, 4>), g, bl, 0, st, args, blk);
  else if (waves == 12) hipLaunchKernelGGL((k_fine_reg_batch<4, 12, 5>), g, bl, 0, st, args, blk);
  else if (waves == 8) hipLaunchKernelGGL((k_fine_reg_batch<4, 8, 5>), g, bl, 0, st, args, blk);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace dmr
