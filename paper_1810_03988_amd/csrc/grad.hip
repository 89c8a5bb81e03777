// Differentiable forms of the stitching path on float frames, in FP64 throughout:
//   * the whole path of a plan, R_0 = F(frames, maps) (Alg. 4 steps 1 and 6 before
//     quantisation), and its vector-Jacobian product;
//   * the loss of a stitched pair,
//       l = 1/(6|Omega|) sum_{p in Omega, c} (P_c - A_c)^2 + (P_c - B_c)^2
//     (P: blended R_0, A/B: the warped frames G_0, Omega: canvas pixels where both frames have
//     all four taps inside and z > 0), with bilinear cells and Omega frozen by
//     stitch_grad_freeze, and its adjoint.
// They refine the transformation the paper obtains from feature matching (Alg. 3, Alg. 4 step
// 5) on the stitched output of Alg. 4 step 6 itself.
//
// Both run the same kernels (the pair with FROZEN cells).  The passes are bound by memory
// traffic and launches, so nothing of level-0 size is stored that a later kernel can form
// again: G_0 is warped twice (once under REDUCE in LDS, once at the collapse), the seam weights
// are read as bytes, and dL_k and EXPAND's inputs are products taken where they are read.
// Every array of a camera covers only its region of a level (the rectangles the blend needs,
// as the planned uint8 path), and up to kGroup cameras share a launch (blockIdx.z).  A
// 1280x720 pair on a 2304x720 canvas, 3 levels, forward and backward: 1.79 ms when each
// operator was a pass over the whole canvas with FP64 planes at level 0, 0.36 ms now.
//
// The transposes of REDUCE / EXPAND are gathers over the fine-domain reflect-101 fold, the
// frame transpose a gather over canvas pixels, and the map sums block partials in a fixed
// order: no atomics on values, every result repeats bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "stitch.h"
#include "stitch_internal.h"

using namespace stitch;

namespace {

constexpr int kT = 256;
constexpr int kGroup = 8;      // cameras per launch (their descriptors are kernel arguments)

struct Map9 { float h[9]; };
struct Inv9 { double h[9]; };
struct Box { int x, y, w, h; };

// single reflect-101 fold (overshoot below the side), or -1 when outside that range
__device__ __forceinline__ int fold1(int i, int n) {
  if (i < 0) i = -i;
  if (i > n - 1) i = 2 * (n - 1) - i;
  return (i >= 0 && i < n) ? i : -1;
}

__device__ __forceinline__ void gcoords(const float* h, int X, int Y, float& x, float& y, bool& zpos) {
#pragma clang fp contract(off)
  const float Xf = (float)X, Yf = (float)Y;
  const float u = (h[0] * Xf + h[1] * Yf) + h[2];
  const float v = (h[3] * Xf + h[4] * Yf) + h[5];
  const float z = (h[6] * Xf + h[7] * Yf) + h[8];
  zpos = z > 0.0f;
  x = u / z;
  y = v / z;
}

// One camera: its map, its float CHW frame, frozen cells (whole canvas; NULL: the map's own)
// and the seam weights on their support box (row y of it is row wrow[y] of wrows, or row y
// when wrow is NULL).
struct VCam {
  Map9 m;
  int fw, fh;
  const float* src;
  int64_t srow, splane;
  const int* x0a;
  const int* y0a;
  const uint8_t* wrows;
  const uint32_t* wrow;
  Box wbox;
};

// Three planes, FP32 or FP64 (elements).
struct Img3 {
  const void* p;
  int64_t row, plane;
  int f64;
};
__device__ __forceinline__ void ld3(const Img3& a, int x, int y, double v[3]) {
  const int64_t i = (int64_t)y * a.row + x;
  if (a.f64) {
    const double* p = (const double*)a.p + i;
    v[0] = p[0]; v[1] = p[a.plane]; v[2] = p[2 * a.plane];
  } else {
    const float* p = (const float*)a.p + i;
    const float u0 = p[0], u1 = p[a.plane], u2 = p[2 * a.plane];
    v[0] = (double)u0; v[1] = (double)u1; v[2] = (double)u2;
  }
}

__device__ __forceinline__ uint32_t seam_at(const VCam& c, int X, int Y) {
  const int x = X - c.wbox.x, y = Y - c.wbox.y;
  if (x < 0 || x >= c.wbox.w || y < 0 || y >= c.wbox.h) return 0;
  const uint32_t r = c.wrow ? c.wrow[y] : (uint32_t)y;
  return c.wrows[(int64_t)r * c.wbox.w + x];
}

// Cell, fraction and source coordinates of canvas pixel (X, Y), and whether the sample is
// defined.  The map's own cell: floor of the FP32 coordinates, the fraction taken in FP32 as
// the uint8 path takes it.  A frozen cell: the stored one, the fraction in FP64.
template <bool FROZEN>
__device__ __forceinline__ bool vcell(const VCam& c, int W, int X, int Y, int& x0, int& y0, double& fx, double& fy,
                                      double& xd, double& yd) {
  float x, y;
  bool zpos;
  gcoords(c.m.h, X, Y, x, y, zpos);
  xd = (double)x;
  yd = (double)y;
  if (FROZEN) {
    if (!zpos) return false;
    const int64_t p = (int64_t)Y * W + X;
    x0 = c.x0a[p];
    y0 = c.y0a[p];
    fx = xd - x0;
    fy = yd - y0;
    return true;
  }
  if (!(zpos && fabsf(x) < 1.0e7f && fabsf(y) < 1.0e7f)) return false;
  const float xf = floorf(x), yf = floorf(y);
  x0 = (int)xf;
  y0 = (int)yf;
  fx = (double)(x - xf);
  fy = (double)(y - yf);
  return true;
}

// The cell's four taps of every channel (0 outside the frame).  All twelve reads are issued,
// without a branch, from the tap's position clamped into the frame: a read under a condition
// is waited for where the paths join.
__device__ __forceinline__ void taps12(const VCam& c, int x0, int y0, double t[3][4]) {
  const bool xa = x0 >= 0 && x0 < c.fw, xb = x0 >= -1 && x0 < c.fw - 1;
  const bool ya = y0 >= 0 && y0 < c.fh, yb = y0 >= -1 && y0 < c.fh - 1;
  const int xc0 = min(max(x0, 0), c.fw - 1), xc1 = min(max(x0, -1) + 1, c.fw - 1);
  const int64_t r0 = (int64_t)min(max(y0, 0), c.fh - 1) * c.srow, r1 = (int64_t)min(max(y0, -1) + 1, c.fh - 1) * c.srow;
  float f[3][4];
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) {
    const float* s = c.src + ch * c.splane;
    f[ch][0] = s[r0 + xc0];
    f[ch][1] = s[r0 + xc1];
    f[ch][2] = s[r1 + xc0];
    f[ch][3] = s[r1 + xc1];
  }
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) {
    t[ch][0] = (double)(xa && ya ? f[ch][0] : 0.0f);
    t[ch][1] = (double)(xb && ya ? f[ch][1] : 0.0f);
    t[ch][2] = (double)(xa && yb ? f[ch][2] : 0.0f);
    t[ch][3] = (double)(xb && yb ? f[ch][3] : 0.0f);
  }
}

template <bool FROZEN>
__device__ __forceinline__ void warp3(const VCam& c, int W, int X, int Y, double g[3]) {
  int x0, y0;
  double fx, fy, xd, yd;
  g[0] = g[1] = g[2] = 0.0;
  if (!vcell<FROZEN>(c, W, X, Y, x0, y0, fx, fy, xd, yd)) return;
  if (!FROZEN && !(x0 >= -1 && x0 < c.fw && y0 >= -1 && y0 < c.fh)) return;   // no tap inside
  double t[3][4];
  taps12(c, x0, y0, t);
#pragma unroll
  for (int ch = 0; ch < 3; ++ch)
    g[ch] = (1.0 - fy) * ((1.0 - fx) * t[ch][0] + fx * t[ch][1]) + fy * ((1.0 - fx) * t[ch][2] + fx * t[ch][3]);
}

// ---------------------------------------------------------------------------- pyramids
// EXPAND along one axis at fine index i of n: three coarse indices and weights (odd samples
// have two taps: the first then stands twice, at half its weight each time, which changes no bit
// of the sum; a third tap of weight 0 would make NaN of an infinity).
struct Tap3 {
  int j[3];
  double w[3];
};
__device__ __forceinline__ Tap3 expand_taps(int i, int n) {
  Tap3 t;
  if (i & 1) {
    t.j[0] = t.j[1] = i >> 1;
    t.j[2] = fold1(i + 1, n) >> 1;
    t.w[0] = t.w[1] = 0.25;
    t.w[2] = 0.5;
  } else {
    t.j[0] = fold1(i - 2, n) >> 1;
    t.j[1] = i >> 1;
    t.j[2] = fold1(i + 2, n) >> 1;
    t.w[0] = t.w[2] = 0.125;
    t.w[1] = 0.75;
  }
  return t;
}

// Separable 3 x 3 sum over NP planes stored on box b: rows jy with weights wy, columns jx with
// weights wx; positions outside the box count 0 (read from the nearest position inside, so that
// no read is under a condition, and then replaced, in the few waves that have any).
template <int NP>
__device__ __forceinline__ void stencil3(const double* __restrict__ g, const Box& b, const int jx[3],
                                         const double wx[3], const int jy[3], const double wy[3], double e[NP]) {
  const int64_t plane = (int64_t)b.w * b.h;
  int ox[3];
  int64_t oy[3];
  bool xin[3], yin[3], all = true;
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    const int i = jx[v] - b.x, k = jy[v] - b.y;
    ox[v] = min(max(i, 0), b.w - 1);
    xin[v] = i == ox[v];
    const int kc = min(max(k, 0), b.h - 1);
    oy[v] = (int64_t)kc * b.w;
    yin[v] = k == kc;
    all &= xin[v] & yin[v];
  }
  double q[NP][3][3];
#pragma unroll
  for (int c = 0; c < NP; ++c)
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
      for (int v = 0; v < 3; ++v) q[c][u][v] = g[c * plane + oy[u] + ox[v]];
  if (!all) {
#pragma unroll
    for (int c = 0; c < NP; ++c)
#pragma unroll
      for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int v = 0; v < 3; ++v) q[c][u][v] = xin[v] && yin[u] ? q[c][u][v] : 0.0;
  }
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    e[c] = 0.0;
#pragma unroll
    for (int u = 0; u < 3; ++u) e[c] += wy[u] * ((wx[0] * q[c][u][0] + wx[1] * q[c][u][1]) + wx[2] * q[c][u][2]);
  }
}

// EXPAND of NP planes stored on box b (0 outside it) of a coarse level, at fine sample
// (x, y) of an nw x nh level.
template <int NP>
__device__ __forceinline__ void expand_at(const double* __restrict__ g, const Box& b, int x, int y, int nw, int nh,
                                          double e[NP]) {
  const Tap3 tx = expand_taps(x, nw), ty = expand_taps(y, nh);
  stencil3<NP>(g, b, tx.j, tx.w, ty.j, ty.w, e);
}

// EXPAND's coefficient of coarse sample j in fine sample i (n fine samples) along one axis.
__device__ __forceinline__ double etap(int d) { return d == 0 ? 0.75 : (d == 1 || d == -1) ? 0.5 : (d == 2 || d == -2) ? 0.125 : 0.0; }
__device__ __forceinline__ double expand_coef(int i, int j, int n) {
  double w = etap(i - 2 * j);
  if (j > 0) w += etap(i + 2 * j);
  if (2 * j != n - 1) w += etap(i - 2 * (n - 1) + 2 * j);
  return w;
}
// REDUCE's coefficient of fine sample i (of n) in coarse sample j along one axis.
__device__ __forceinline__ double rtap(int d) { return d == 0 ? 0.375 : (d == 1 || d == -1) ? 0.25 : (d == 2 || d == -2) ? 0.0625 : 0.0; }
__device__ __forceinline__ double reduce_coef(int i, int j, int n) {
  double w = rtap(i - 2 * j);
  if (i > 0) w += rtap(-i - 2 * j);
  if (i != n - 1) w += rtap(2 * (n - 1) - i - 2 * j);
  return w;
}

// The coarse samples that fine sample i has a share in and its coefficients there: j0 = (i - 1) >> 1
// and the two after it where i is even, the one after it where i is odd (j0 then stands twice, as
// in expand_taps).  Away from the borders the coefficients depend on the parity alone.
__device__ __forceinline__ void reduce_taps(int i, int n, int j[3], double w[3]) {
  const int j0 = (i - 1) >> 1;                         // coarse ceil((i - 2) / 2)
  const bool odd = (i & 1) != 0;
  j[0] = j0;
  j[1] = odd ? j0 : j0 + 1;
  j[2] = odd ? j0 + 1 : j0 + 2;
  w[0] = odd ? 0.125 : 0.0625;
  w[1] = odd ? 0.125 : 0.375;
  w[2] = odd ? 0.25 : 0.0625;
  if (i < 3 || i > n - 4) {
    for (int v = 0; v < 3; ++v) w[v] = reduce_coef(i, j[v], n);
    if (odd) {
      w[0] *= 0.5;
      w[1] *= 0.5;
    }
  }
}

// REDUCE^T of three planes on box b (0 outside) of a coarse level, at fine sample (x, y).
__device__ __forceinline__ void reduceT_at(const double* __restrict__ d, const Box& b, int x, int y, int nw, int nh,
                                           double e[3]) {
  int jx[3], jy[3];
  double wx[3], wy[3];
  reduce_taps(x, nw, jx, wx);
  reduce_taps(y, nh, jy, wy);
  stencil3<3>(d, b, jx, wx, jy, wy, e);
}

// Level 0 -> 1 of up to kGroup cameras: G_1 = REDUCE of the warped frame (IMG) and Gm_1 of the
// seam weights on each camera's level-1 region.  A 32x8 coarse tile's 67x19 window is warped
// once into LDS (a sample feeds 6.25 outputs) and reduced along rows, then columns.  The
// weights stay integers (exact in FP32) until one division by 255 * 256.
struct Reduce0Cam {
  VCam c;
  Box roi;
  double* g;
  double* gm;
};
struct Reduce0Args {
  Reduce0Cam cam[kGroup];
  int W, H;
};
constexpr int kRX = 32, kRY = 8, kRW = 2 * kRX + 3, kRH = 2 * kRY + 3;

template <bool FROZEN, bool IMG>
__global__ void __launch_bounds__(kT) k_vreduce0(const Reduce0Args a) {
  const Reduce0Cam& q = a.cam[blockIdx.z];
  const int tx0 = (int)blockIdx.x * kRX, ty0 = (int)blockIdx.y * kRY;
  if (tx0 >= q.roi.w || ty0 >= q.roi.h) return;
  constexpr int NP = IMG ? 3 : 1;
  __shared__ double sG[NP][IMG ? kRH : 1][kRW + 1];
  __shared__ double sR[NP][IMG ? kRH : 1][kRX];
  __shared__ float sM[kRH][kRW + 1], sMR[kRH][kRX];
  const int tid = threadIdx.x;
  const int X0 = 2 * (q.roi.x + tx0) - 2, Y0 = 2 * (q.roi.y + ty0) - 2;
  constexpr int NE = kRH * kRW, NQ = (NE + kT - 1) / kT;
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    const int e = tid + k * kT;
    if (e >= NE) break;
    const int r = e / kRW, c = e - r * kRW;
    const int X = fold1(X0 + c, a.W), Y = fold1(Y0 + r, a.H);
    const bool in = X >= 0 && Y >= 0;
    if (IMG) {
      double g[3] = {0.0, 0.0, 0.0};
      if (in) warp3<FROZEN>(q.c, a.W, X, Y, g);
#pragma unroll
      for (int ch = 0; ch < NP; ++ch) sG[ch][r][c] = g[ch];
    }
    sM[r][c] = in ? (float)seam_at(q.c, X, Y) : 0.0f;
  }
  __syncthreads();
  for (int e = tid; e < kRH * kRX; e += kT) {
    const int r = e / kRX, c = e - r * kRX;
    if (IMG) {
#pragma unroll
      for (int ch = 0; ch < NP; ++ch) {
        const double* s = &sG[ch][r][2 * c];
        sR[ch][r][c] = 0.0625 * (s[0] + s[4]) + 0.25 * (s[1] + s[3]) + 0.375 * s[2];
      }
    }
    const float* s = &sM[r][2 * c];
    sMR[r][c] = (s[0] + s[4]) + 4.0f * (s[1] + s[3]) + 6.0f * s[2];
  }
  __syncthreads();
  const int c = tid % kRX, r = tid / kRX;
  if (tx0 + c >= q.roi.w || ty0 + r >= q.roi.h) return;
  const int64_t at = (int64_t)(ty0 + r) * q.roi.w + tx0 + c, plane = (int64_t)q.roi.w * q.roi.h;
  if (IMG) {
#pragma unroll
    for (int ch = 0; ch < NP; ++ch)
      q.g[ch * plane + at] = 0.0625 * (sR[ch][2 * r][c] + sR[ch][2 * r + 4][c]) +
                             0.25 * (sR[ch][2 * r + 1][c] + sR[ch][2 * r + 3][c]) + 0.375 * sR[ch][2 * r + 2][c];
  }
  if (q.gm)
    q.gm[at] = (double)((sMR[2 * r][c] + sMR[2 * r + 4][c]) + 4.0f * (sMR[2 * r + 1][c] + sMR[2 * r + 3][c]) +
                        6.0f * sMR[2 * r + 2][c]) / (255.0 * 256.0);
}

// Level k -> k+1 (k >= 1): REDUCE of each camera's planes (three image planes, one weight
// plane; either may be absent), which are 0 outside their region.
struct ReduceCam {
  const double* g;
  const double* gm;
  Box in;
  double* og;
  double* ogm;
  Box out;
};
struct ReduceArgs {
  ReduceCam cam[kGroup];
  int nw, nh;
};
__global__ void __launch_bounds__(kT) k_vreduce(const ReduceArgs a) {
  const ReduceCam& q = a.cam[blockIdx.z];
  const int lx = (int)blockIdx.x * 64 + (threadIdx.x & 63), ly = (int)blockIdx.y * 4 + (threadIdx.x >> 6);
  if (lx >= q.out.w || ly >= q.out.h) return;
  const int x = q.out.x + lx, y = q.out.y + ly;
  const double wt[5] = {0.0625, 0.25, 0.375, 0.25, 0.0625};
  int ox[5];
  bool in[5];             // (outside, the value counts 0, not its weight: a sample read there may be infinite)
#pragma unroll
  for (int b = 0; b < 5; ++b) {
    const int i = fold1(2 * x + b - 2, a.nw) - q.in.x;
    in[b] = i >= 0 && i < q.in.w;
    ox[b] = in[b] ? i : 0;
  }
  const int64_t plane = (int64_t)q.in.w * q.in.h, oplane = (int64_t)q.out.w * q.out.h;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < 5; ++u) {
    const int i = fold1(2 * y + u - 2, a.nh) - q.in.y;
    if (i < 0 || i >= q.in.h) continue;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double* s = c < 3 ? q.g : q.gm;
      if (!s) continue;
      s += (c < 3 ? c * plane : 0) + (int64_t)i * q.in.w;
      double v[5];
#pragma unroll
      for (int b = 0; b < 5; ++b) v[b] = s[ox[b]];
#pragma unroll
      for (int b = 0; b < 5; ++b) v[b] = in[b] ? v[b] : 0.0;
      acc[c] += wt[u] * ((wt[0] * v[0] + wt[4] * v[4]) + (wt[1] * v[1] + wt[3] * v[3]) + wt[2] * v[2]);
    }
  }
  const int64_t at = (int64_t)ly * q.out.w + lx;
  if (q.g)
    for (int c = 0; c < 3; ++c) q.og[c * oplane + at] = acc[c];
  if (q.gm) q.ogm[at] = acc[3];
}

// ---------------------------------------------------------------------------- synthesis
// out = [acc +] sum over the group's cameras of Gm_k L_k on their bands [+ EXPAND(R_{k+1})],
// L_k = G_k - EXPAND(G_{k+1}) (G_k at the top), k >= 1, on the whole level canvas.
struct BlendCamV {
  const double* g;
  const double* gm;
  Box roi, band;
  const double* cg;       // G_{k+1} on croi, NULL at the top
  Box croi;
};
struct BlendArgsV {
  BlendCamV cam[kGroup];
  int n, w, h;
  const double* acc;      // NULL: 0 (may be out)
  const double* rc;       // R_{k+1}, NULL: none
  int cw, ch;
  double* out;
};
__global__ void __launch_bounds__(kT) k_vblend(const BlendArgsV a) {
  const int x = (int)blockIdx.x * 64 + (threadIdx.x & 63), y = (int)blockIdx.y * 4 + (threadIdx.x >> 6);
  if (x >= a.w || y >= a.h) return;
  const int64_t np = (int64_t)a.w * a.h, at = (int64_t)y * a.w + x;
  double v[3] = {0.0, 0.0, 0.0};
  if (a.acc)
    for (int c = 0; c < 3; ++c) v[c] = a.acc[c * np + at];
  for (int i = 0; i < a.n; ++i) {
    const BlendCamV& q = a.cam[i];
    if (x < q.band.x || x >= q.band.x + q.band.w || y < q.band.y || y >= q.band.y + q.band.h) continue;
    const int64_t p = (int64_t)(y - q.roi.y) * q.roi.w + (x - q.roi.x), plane = (int64_t)q.roi.w * q.roi.h;
    const double m = q.gm[p];
    double e[3] = {0.0, 0.0, 0.0};
    if (q.cg) expand_at<3>(q.cg, q.croi, x, y, a.w, a.h, e);
    for (int c = 0; c < 3; ++c) v[c] += m * (q.g[c * plane + p] - e[c]);
  }
  if (a.rc) {
    double e[3];
    expand_at<3>(a.rc, Box{0, 0, a.cw, a.ch}, x, y, a.w, a.h, e);
    for (int c = 0; c < 3; ++c) v[c] += e[c];
  }
  for (int c = 0; c < 3; ++c) a.out[c * np + at] = v[c];
}

// Level 0: the same with G_0 warped on the spot and byte weights; the result goes to an FP32
// image (out32) or, between camera groups, to FP64 planes.
struct PanoCam {
  VCam c;
  Box band;
  const double* cg;       // G_1 on croi, NULL for a single level
  Box croi;
};
struct PanoArgs {
  PanoCam cam[kGroup];
  int n, W, H;
  const double* acc;
  const double* rc;       // R_1
  int cw, ch;
  double* out64;
  float* out32;
  int64_t orow, oplane;
};
__global__ void __launch_bounds__(kT) k_vpano(const PanoArgs a) {
  const int X = (int)blockIdx.x * 64 + (threadIdx.x & 63), Y = (int)blockIdx.y * 4 + (threadIdx.x >> 6);
  if (X >= a.W || Y >= a.H) return;
  const int64_t np = (int64_t)a.W * a.H, at = (int64_t)Y * a.W + X;
  double v[3] = {0.0, 0.0, 0.0};
  if (a.acc)
    for (int c = 0; c < 3; ++c) v[c] = a.acc[c * np + at];
  for (int i = 0; i < a.n; ++i) {
    const PanoCam& q = a.cam[i];
    if (X < q.band.x || X >= q.band.x + q.band.w || Y < q.band.y || Y >= q.band.y + q.band.h) continue;
    const double m = (double)seam_at(q.c, X, Y) / 255.0;
    double g[3], e[3] = {0.0, 0.0, 0.0};
    warp3<false>(q.c, a.W, X, Y, g);
    if (q.cg) expand_at<3>(q.cg, q.croi, X, Y, a.W, a.H, e);
    for (int c = 0; c < 3; ++c) v[c] += m * (g[c] - e[c]);
  }
  if (a.rc) {
    double e[3];
    expand_at<3>(a.rc, Box{0, 0, a.cw, a.ch}, X, Y, a.W, a.H, e);
    for (int c = 0; c < 3; ++c) v[c] += e[c];
  }
  for (int c = 0; c < 3; ++c) {
    if (a.out32) a.out32[c * a.oplane + (int64_t)Y * a.orow + X] = (float)v[c];
    else a.out64[c * np + at] = v[c];
  }
}

// ---------------------------------------------------------------------------- the transposes
// dR_{k+1} = EXPAND^T dR_k (three planes, whole level canvases).
__global__ void __launch_bounds__(kT) k_vexpandT(Img3 d, int nw, int nh, double* __restrict__ out, int mw, int mh) {
  const int x = (int)blockIdx.x * 64 + (threadIdx.x & 63), y = (int)blockIdx.y * 4 + (threadIdx.x >> 6);
  if (x >= mw || y >= mh) return;
  double acc[3] = {0.0, 0.0, 0.0};
  double wx[5];
  int ox[5];
  bool in[5];             // (outside, the value counts 0, as in k_vreduce)
#pragma unroll
  for (int b = 0; b < 5; ++b) {
    const int i = 2 * x + b - 2;
    in[b] = i >= 0 && i < nw;
    ox[b] = in[b] ? i : 0;
    wx[b] = expand_coef(i, x, nw);
  }
#pragma unroll
  for (int u = 0; u < 5; ++u) {
    const int i = 2 * y + u - 2;
    if (i < 0 || i >= nh) continue;
    const double wy = expand_coef(i, y, nh);
    double t[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < 5; ++b) {
      double v[3];
      ld3(d, ox[b], i, v);
      for (int c = 0; c < 3; ++c) t[c] += wx[b] * (in[b] ? v[c] : 0.0);
    }
    for (int c = 0; c < 3; ++c) acc[c] += wy * t[c];
  }
  const int64_t np = (int64_t)mw * mh, at = (int64_t)y * mw + x;
  for (int c = 0; c < 3; ++c) out[c * np + at] = acc[c];
}

// dG_k = Gm_k dR_k - EXPAND^T(Gm_{k-1} dR_{k-1}) + REDUCE^T dG_{k+1} on each camera's level-k
// region, k >= 2 (k = 1: k_vtileT); the products live on the bands.
struct DgCam {
  const double* gm;       // Gm_k on roi
  Box roi, band;
  const double* fgm;      // Gm_{k-1} on froi (level 0: the bytes of c)
  Box froi, fband;
  VCam c;
  const double* dgc;      // dG_{k+1} on croi, NULL at the top
  Box croi;
  double* out;
};
struct DgArgs {
  DgCam cam[kGroup];
  const double* dr;       // dR_k
  int w, h;
  Img3 fdr;               // dR_{k-1}
  int nw, nh;
};
__global__ void __launch_bounds__(kT) k_vdg(const DgArgs a) {
  const DgCam& q = a.cam[blockIdx.z];
  const int lx = (int)blockIdx.x * 64 + (threadIdx.x & 63), ly = (int)blockIdx.y * 4 + (threadIdx.x >> 6);
  if (lx >= q.roi.w || ly >= q.roi.h) return;
  const int x = q.roi.x + lx, y = q.roi.y + ly;
  const int64_t at = (int64_t)ly * q.roi.w + lx, plane = (int64_t)q.roi.w * q.roi.h;
  double v[3] = {0.0, 0.0, 0.0};
  if (x >= q.band.x && x < q.band.x + q.band.w && y >= q.band.y && y < q.band.y + q.band.h) {
    const double m = q.gm[at];
    const int64_t np = (int64_t)a.w * a.h, p = (int64_t)y * a.w + x;
    for (int c = 0; c < 3; ++c) v[c] = m * a.dr[c * np + p];
  }
  double t[3] = {0.0, 0.0, 0.0};
  if (q.fband.w > 0 && 2 * x + 2 >= q.fband.x && 2 * x - 2 < q.fband.x + q.fband.w) {
    double wx[5];
    int ix[5];
    bool in[5];           // (outside, the product counts 0, as in k_vreduce)
#pragma unroll
    for (int b = 0; b < 5; ++b) {
      const int i = 2 * x + b - 2;
      ix[b] = min(max(i, q.fband.x), q.fband.x + q.fband.w - 1);
      in[b] = i == ix[b];
      wx[b] = expand_coef(i, x, a.nw);
    }
#pragma unroll
    for (int u = 0; u < 5; ++u) {
      const int i = 2 * y + u - 2;
      if (i < q.fband.y || i >= q.fband.y + q.fband.h) continue;     // uniform over a row of threads
      const double wy = expand_coef(i, y, a.nh);
      double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int b = 0; b < 5; ++b) {
        const double m = wx[b] * q.fgm[(int64_t)(i - q.froi.y) * q.froi.w + (ix[b] - q.froi.x)];
        double d[3];
        ld3(a.fdr, ix[b], i, d);
#pragma unroll
        for (int c = 0; c < 3; ++c) s[c] += m * (in[b] ? d[c] : 0.0);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) t[c] += wy * s[c];
    }
  }
  if (q.dgc) {
    double e[3];
    reduceT_at(q.dgc, q.croi, x, y, a.w, a.h, e);
    for (int c = 0; c < 3; ++c) v[c] += e[c];
  }
  for (int c = 0; c < 3; ++c) q.out[c * plane + at] = v[c] - t[c];
}

// Level 0 -> 1 of the transposed EXPANDs, the same results as k_vexpandT and k_vdg there:
// slices z < ncam hold dG_1 of a camera (its fine operand: seam byte times dR_0 on band 0,
// divided by 255 at the end), slice ncam (whole) dR_1.  At level 0 a 5 x 5 gather per coarse
// sample reads 100 values; here a 32x8 coarse tile's 67x19 window is formed once in LDS and
// summed along rows, then columns (28 + 68 us -> 17 + 31 us for a 1280x720 pair).
struct TileTArgs {
  DgArgs dg;
  int ncam;
  double* dr1;            // NULL: cameras only
};
__global__ void __launch_bounds__(kT) k_vtileT(const TileTArgs a) {
  const int z = (int)blockIdx.z;
  const bool whole = z == a.ncam;
  const DgCam& q = a.dg.cam[whole ? 0 : z];
  const Box roi = whole ? Box{0, 0, a.dg.w, a.dg.h} : q.roi;
  const int tx0 = (int)blockIdx.x * kRX, ty0 = (int)blockIdx.y * kRY;
  if (tx0 >= roi.w || ty0 >= roi.h) return;
  __shared__ double sG[3][kRH][kRW + 1], sR[3][kRH][kRX];
  const int tid = threadIdx.x;
  const Box fb = whole ? Box{0, 0, a.dg.nw, a.dg.nh} : q.fband;
  const int X0 = 2 * (roi.x + tx0) - 2, Y0 = 2 * (roi.y + ty0) - 2;
  const bool some = fb.w > 0 && X0 + kRW > fb.x && X0 < fb.x + fb.w && Y0 + kRH > fb.y && Y0 < fb.y + fb.h;
  const int c = tid % kRX, r = tid / kRX;
  const int x = roi.x + tx0 + c, y = roi.y + ty0 + r;
  double t[3] = {0.0, 0.0, 0.0};
  if (some) {                                          // uniform over the block
    constexpr int NE = kRH * kRW, NQ = (NE + kT - 1) / kT;
    double d[NQ][3];
    double m[NQ];
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const int e = min(tid + k * kT, NE - 1), rr = e / kRW, X = X0 + e - rr * kRW, Y = Y0 + rr;
      const int Xc = min(max(X, fb.x), fb.x + fb.w - 1), Yc = min(max(Y, fb.y), fb.y + fb.h - 1);
      ld3(a.dg.fdr, Xc, Yc, d[k]);
      m[k] = whole ? 1.0 : (double)seam_at(q.c, Xc, Yc);
      if (X != Xc || Y != Yc) m[k] = d[k][0] = d[k][1] = d[k][2] = 0.0;
    }
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const int e = tid + k * kT;
      if (e >= NE) break;
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) sG[ch][e / kRW][e % kRW] = m[k] * d[k][ch];
    }
    __syncthreads();
    double w[5];
#pragma unroll
    for (int b = 0; b < 5; ++b) w[b] = expand_coef(2 * x + b - 2, x, a.dg.nw);
    for (int e = tid; e < kRH * kRX; e += kT) {        // the thread's column is the same each time
      const int rr = e / kRX;
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        const double* s = &sG[ch][rr][2 * c];
        sR[ch][rr][c] = (w[0] * s[0] + w[4] * s[4]) + (w[1] * s[1] + w[3] * s[3]) + w[2] * s[2];
      }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 5; ++b) w[b] = expand_coef(2 * y + b - 2, y, a.dg.nh);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch)
      t[ch] = (w[0] * sR[ch][2 * r][c] + w[4] * sR[ch][2 * r + 4][c]) +
              (w[1] * sR[ch][2 * r + 1][c] + w[3] * sR[ch][2 * r + 3][c]) + w[2] * sR[ch][2 * r + 2][c];
  }
  if (tx0 + c >= roi.w || ty0 + r >= roi.h) return;
  const int64_t at = (int64_t)(ty0 + r) * roi.w + tx0 + c, plane = (int64_t)roi.w * roi.h;
  if (whole) {
    for (int ch = 0; ch < 3; ++ch) a.dr1[ch * plane + at] = t[ch];
    return;
  }
  double v[3] = {0.0, 0.0, 0.0};
  if (x >= q.band.x && x < q.band.x + q.band.w && y >= q.band.y && y < q.band.y + q.band.h) {
    const double m = q.gm[at];
    const int64_t np = (int64_t)a.dg.w * a.dg.h, p = (int64_t)y * a.dg.w + x;
    for (int ch = 0; ch < 3; ++ch) v[ch] = m * a.dg.dr[ch * np + p];
  }
  if (q.dgc) {
    double e[3];
    reduceT_at(q.dgc, q.croi, x, y, a.dg.w, a.dg.h, e);
    for (int ch = 0; ch < 3; ++ch) v[ch] += e[ch];
  }
  for (int ch = 0; ch < 3; ++ch) q.out[ch * plane + at] = v[ch] - t[ch] / 255.0;
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  for (int i = 0; i < kT / 64; ++i) t += sh[i];
  __syncthreads();
  return t;
}

// dG_0 = m dR_0 + REDUCE^T dG_1 [+ the direct term] on each camera's domain, and the map's
// nine sums there.  A block walks 64 columns x kDgRows rows, so the sums cost one block
// reduction per 1024 samples.  Samples with no tap in the frame have no share in either result and are
// left out (nothing reads their dG_0).
struct Dg0Cam {
  VCam c;
  Box band, dom;
  const double* dg1;      // dG_1 on croi, NULL for a single level
  Box croi;
  Img3 direct;            // p NULL: none
  double* out;
  double* part;           // nine sums per block of the domain
};
struct Dg0Args {
  Dg0Cam cam[kGroup];
  Img3 dr0;
  int W, H;
};
constexpr int kDgRows = 16;
template <bool FROZEN>
__global__ void __launch_bounds__(kT) k_vdg0(const Dg0Args a) {
  const Dg0Cam& q = a.cam[blockIdx.z];
  if ((int)blockIdx.x * 64 >= q.dom.w || (int)blockIdx.y * kDgRows >= q.dom.h) return;
  __shared__ double sh[kT / 64][9];
  const int lx = (int)blockIdx.x * 64 + (threadIdx.x & 63);
  const int64_t plane = (int64_t)q.dom.w * q.dom.h;
  double t9[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int k = 0; k < kDgRows / 4; ++k) {
    const int ly = (int)blockIdx.y * kDgRows + 4 * k + (threadIdx.x >> 6);
    if (lx >= q.dom.w || ly >= q.dom.h) continue;
    const int X = q.dom.x + lx, Y = q.dom.y + ly;
    int x0, y0;
    double fx, fy, xd, yd;
    if (!vcell<FROZEN>(q.c, a.W, X, Y, x0, y0, fx, fy, xd, yd)) continue;
    if (!(x0 >= -1 && x0 < q.c.fw && y0 >= -1 && y0 < q.c.fh)) continue;
    double t[3][4];
    taps12(q.c, x0, y0, t);
    double v[3] = {0.0, 0.0, 0.0};
    if (X >= q.band.x && X < q.band.x + q.band.w && Y >= q.band.y && Y < q.band.y + q.band.h) {
      const double m = (double)seam_at(q.c, X, Y) / 255.0;
      ld3(a.dr0, X, Y, v);
      for (int c = 0; c < 3; ++c) v[c] *= m;
    }
    if (q.dg1) {
      double e[3];
      reduceT_at(q.dg1, q.croi, X, Y, a.W, a.H, e);
      for (int c = 0; c < 3; ++c) v[c] += e[c];
    }
    if (q.direct.p) {
      double e[3];
      ld3(q.direct, X, Y, e);
      for (int c = 0; c < 3; ++c) v[c] += e[c];
    }
    double gx = 0.0, gy = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      q.out[c * plane + (int64_t)ly * q.dom.w + lx] = v[c];
      gx += v[c] * ((1 - fy) * (t[c][1] - t[c][0]) + fy * (t[c][3] - t[c][2]));
      gy += v[c] * ((1 - fx) * (t[c][2] - t[c][0]) + fx * (t[c][3] - t[c][1]));
    }
    if (gx != 0.0 || gy != 0.0) {   // (also keeps 0 * inf out where the coordinates overflow)
      const float* h = q.c.m.h;
      const double z = ((double)h[6] * (double)X + (double)h[7] * (double)Y) + (double)h[8];
      const double iz = 1.0 / z, s = -(gx * xd + gy * yd) * iz;
      gx *= iz;
      gy *= iz;
      t9[0] += gx * X; t9[1] += gx * Y; t9[2] += gx;
      t9[3] += gy * X; t9[4] += gy * Y; t9[5] += gy;
      t9[6] += s * X; t9[7] += s * Y; t9[8] += s;
    }
  }
  const int nbx = (q.dom.w + 63) / 64;
  const int64_t b = (int64_t)blockIdx.y * nbx + blockIdx.x;
#pragma unroll
  for (int k = 0; k < 9; ++k)
    for (int o = 32; o > 0; o >>= 1) t9[k] += __shfl_xor(t9[k], o);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < 9; ++k) sh[threadIdx.x >> 6][k] = t9[k];
  __syncthreads();
  if (threadIdx.x < 9) {
    const int k = threadIdx.x;
    q.part[b * 9 + k] = (sh[0][k] + sh[1][k]) + (sh[2][k] + sh[3][k]);
  }
}

// out[i * 9 + k] = sum of the nine-entry partials of camera i (grid: 9 x cameras).
struct SumArgs {
  const double* part[kGroup];
  int n[kGroup];
  double* out;
};
__global__ void __launch_bounds__(kT) k_vsum9(const SumArgs a) {
  __shared__ double sh[kT / 64];
  const double* p = a.part[blockIdx.y];
  double v = 0.0;
  for (int i = threadIdx.x; i < a.n[blockIdx.y]; i += kT) v += p[(int64_t)i * 9 + blockIdx.x];
  const double t = block_sum(v, sh);
  if (threadIdx.x == 0) a.out[blockIdx.y * 9 + blockIdx.x] = t;
}

// Adjoint of the warp with respect to the frames, as a gather (deterministic, no atomics):
// source pixel (x, y) sums w dG_0 over the canvas pixels whose cell holds it as a tap.  Those
// lie in the image under hf (the FP64 inverse of the map the cells belong to) of the source
// square [x-1, x+1) x [y-1, y+1).  The cells come from FP32 coordinates, off by at most
// `delta` source samples (bounded on the host): the image of the square widened by delta
// holds every candidate.  Where the projective depth varies by less than 2 over the square's
// corners, the map's slopes inside vary by less than 4.5, so widening the image's bounding
// box by 4.5 delta of its own span covers that; elsewhere, and for a delta above 1/64, it is
// one canvas pixel.  (One pixel always: 25 candidates a pixel at scale 1 instead of 4 to 9.)
// A box over 48 pixels a side (a map magnifying about 20 times) or a square reaching the
// map's horizon sets *flag.
struct SrcCam {
  VCam c;
  Inv9 hf;
  double delta;
  const double* dg;       // dG_0 on dom
  Box dom;
  float* out;
  int64_t orow, oplane;
};
struct SrcArgs {
  SrcCam cam[kGroup];
  int W, H;
};
template <bool FROZEN>
__global__ void __launch_bounds__(kT) k_vsrcT(const SrcArgs a, int* __restrict__ flag) {
  const SrcCam& q = a.cam[blockIdx.z];
  const int x = (int)blockIdx.x * 64 + (threadIdx.x & 63), y = (int)blockIdx.y * 4 + (threadIdx.x >> 6);
  if (x >= q.c.fw || y >= q.c.fh) return;
  double bx0 = 1e300, bx1 = -1e300, by0 = 1e300, by1 = -1e300, wmin = 1e300, wmax = -1e300;
  bool bounded = true;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double sx = (double)(x - 1 + 2 * (k & 1)), sy = (double)(y - 1 + (k & 2));
    const double w = (q.hf.h[6] * sx + q.hf.h[7] * sy) + q.hf.h[8];
    bounded = bounded && w > 0.0;
    const double iw = 1.0 / w;
    const double X = ((q.hf.h[0] * sx + q.hf.h[1] * sy) + q.hf.h[2]) * iw;
    const double Y = ((q.hf.h[3] * sx + q.hf.h[4] * sy) + q.hf.h[5]) * iw;
    bx0 = fmin(bx0, X); bx1 = fmax(bx1, X); by0 = fmin(by0, Y); by1 = fmax(by1, Y);
    wmin = fmin(wmin, w); wmax = fmax(wmax, w);
  }
  double acc[3] = {0.0, 0.0, 0.0};
  if (bounded && bx1 >= -2.0 && by1 >= -2.0 && bx0 <= a.W + 1.0 && by0 <= a.H + 1.0) {
    if (bx1 - bx0 > 46.0 || by1 - by0 > 46.0) {
      atomicOr(flag, 1);
    } else {
      const bool tight = q.delta <= 0x1p-6 && wmin >= 0.5 * wmax;
      const double mx = tight ? 4.5 * q.delta * (bx1 - bx0) + 1e-6 : 1.0;
      const double my = tight ? 4.5 * q.delta * (by1 - by0) + 1e-6 : 1.0;
      const int X0 = max(q.dom.x, (int)ceil(bx0 - mx)), X1 = min(q.dom.x + q.dom.w - 1, (int)floor(bx1 + mx));
      const int Y0 = max(q.dom.y, (int)ceil(by0 - my)), Y1 = min(q.dom.y + q.dom.h - 1, (int)floor(by1 + my));
      const int64_t plane = (int64_t)q.dom.w * q.dom.h;
      for (int Y = Y0; Y <= Y1; ++Y)
        for (int X = X0; X <= X1; ++X) {
          int x0, y0;
          double fx, fy, xd, yd;
          if (!vcell<FROZEN>(q.c, a.W, X, Y, x0, y0, fx, fy, xd, yd)) continue;
          const int i = x - x0, j = y - y0;
          if (i < 0 || i > 1 || j < 0 || j > 1) continue;
          const double wt = (i ? fx : 1.0 - fx) * (j ? fy : 1.0 - fy);
          const double* d = q.dg + (int64_t)(Y - q.dom.y) * q.dom.w + (X - q.dom.x);
#pragma unroll
          for (int ch = 0; ch < 3; ++ch) acc[ch] += wt * d[ch * plane];
        }
    }
  } else if (!bounded) {
    atomicOr(flag, 2);
  }
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) q.out[ch * q.oplane + (int64_t)y * q.orow + x] = (float)acc[ch];
}

// ---------------------------------------------------------------------------- the pair loss
// Frozen cells of both cameras, Omega, and |Omega| by block partial counts.
__global__ void __launch_bounds__(kT) k_gcells(Map9 m0, Map9 m1, int w0, int h0, int w1, int h1, int W, int H,
                                               int* __restrict__ x0a, int* __restrict__ y0a,
                                               uint8_t* __restrict__ omega, double* __restrict__ part) {
  __shared__ double sh[kT / 64];
  const int X = (int)blockIdx.x * 64 + (threadIdx.x & 63);
  const int64_t np = (int64_t)W * H;
  double count = 0.0;
  for (int k = 0; k < kDgRows / 4; ++k) {
    const int Y = (int)blockIdx.y * kDgRows + 4 * k + (threadIdx.x >> 6);
    if (X >= W || Y >= H) continue;
    const int64_t p = (int64_t)Y * W + X;
    bool all = true;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const float* hm = c ? m1.h : m0.h;
      const int w = c ? w1 : w0, h = c ? h1 : h0;
      float x, y;
      bool zpos;
      gcoords(hm, X, Y, x, y, zpos);
      const bool fin = zpos && fabsf(x) < 1.0e7f && fabsf(y) < 1.0e7f;
      const int cx = fin ? (int)floorf(x) : -10, cy = fin ? (int)floorf(y) : -10;
      x0a[c * np + p] = cx;
      y0a[c * np + p] = cy;
      all = all && fin && cx >= 0 && cx + 1 <= w - 1 && cy >= 0 && cy + 1 <= h - 1;
    }
    omega[p] = all ? 1 : 0;
    count += all ? 1.0 : 0.0;
  }
  const double t = block_sum(count, sh);
  if (threadIdx.x == 0) part[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
}

// The loss's terms and the gradients it sends into A and B (that into P is minus their sum).
// P is collapsed at the pixel itself, and only on Omega.
struct LossArgs {
  PanoCam cam[2];
  int W, H;
  const double* rc;
  int cw, ch;
  const uint8_t* omega;
  double scale;
  double* ga;
  double* gb;
  double* part;
};
__global__ void __launch_bounds__(kT) k_gloss(const LossArgs a) {
  __shared__ double sh[kT / 64];
  const int X = (int)blockIdx.x * 64 + (threadIdx.x & 63);
  const int64_t np = (int64_t)a.W * a.H;
  double term = 0.0;
  for (int k = 0; k < kDgRows / 4; ++k) {
    const int Y = (int)blockIdx.y * kDgRows + 4 * k + (threadIdx.x >> 6);
    if (X >= a.W || Y >= a.H) continue;
    const int64_t p = (int64_t)Y * a.W + X;
    double da[3] = {0.0, 0.0, 0.0}, db[3] = {0.0, 0.0, 0.0};
    if (a.omega[p]) {
      double P[3] = {0.0, 0.0, 0.0}, g[2][3];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const PanoCam& q = a.cam[i];
        warp3<true>(q.c, a.W, X, Y, g[i]);
        if (X < q.band.x || X >= q.band.x + q.band.w || Y < q.band.y || Y >= q.band.y + q.band.h) continue;
        const double m = (double)seam_at(q.c, X, Y) / 255.0;
        double e[3] = {0.0, 0.0, 0.0};
        if (q.cg) expand_at<3>(q.cg, q.croi, X, Y, a.W, a.H, e);
        for (int c = 0; c < 3; ++c) P[c] += m * (g[i][c] - e[c]);
      }
      if (a.rc) {
        double e[3];
        expand_at<3>(a.rc, Box{0, 0, a.cw, a.ch}, X, Y, a.W, a.H, e);
        for (int c = 0; c < 3; ++c) P[c] += e[c];
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        da[c] = P[c] - g[0][c];
        db[c] = P[c] - g[1][c];
        term += da[c] * da[c] + db[c] * db[c];
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      a.ga[c * np + p] = -2.0 * a.scale * da[c];
      a.gb[c * np + p] = -2.0 * a.scale * db[c];
    }
  }
  const double t = block_sum(term, sh);
  if (threadIdx.x == 0) a.part[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
}

// One block: *out = sum of n partials.
__global__ void __launch_bounds__(kT) k_gsum(const double* __restrict__ part, int n, double* __restrict__ out) {
  __shared__ double sh[kT / 64];
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += kT) v += part[i];
  const double t = block_sum(v, sh);
  if (threadIdx.x == 0) *out = t;
}

// dl/dP = -(gA + gB): as FP64 planes (out), or all three as FP32 images.
__global__ void __launch_bounds__(kT) k_gpano(const double* __restrict__ ga, const double* __restrict__ gb, int64_t n,
                                              double* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (p < n) out[p] = -(ga[p] + gb[p]);
}
struct Out3 {
  float* p;
  int64_t row, plane;
};
__global__ void __launch_bounds__(kT) k_gupstream(const double* __restrict__ ga, const double* __restrict__ gb, int W,
                                                  int H, Out3 dp, Out3 da, Out3 db) {
  const int X = (int)blockIdx.x * 64 + (threadIdx.x & 63), Y = (int)blockIdx.y * 4 + (threadIdx.x >> 6);
  if (X >= W || Y >= H) return;
  const int64_t np = (int64_t)W * H, p = (int64_t)Y * W + X;
  for (int c = 0; c < 3; ++c) {
    const double u = ga[c * np + p], v = gb[c * np + p];
    dp.p[c * dp.plane + (int64_t)Y * dp.row + X] = (float)-(u + v);
    da.p[c * da.plane + (int64_t)Y * da.row + X] = (float)u;
    db.p[c * db.plane + (int64_t)Y * db.row + X] = (float)v;
  }
}

__global__ void k_gzero(double* __restrict__ out) { *out = 0.0; }

// ==================================================================================== host
int blocks(int64_t n) { return (int)((n + kT - 1) / kT); }
int cdiv(int a, int b) { return (a + b - 1) / b; }

size_t take(size_t& top, size_t bytes) {
  const size_t off = top;
  top = (top + bytes + 255) / 256 * 256;
  return off;
}

stitch_status dev_ok(hipError_t e, const char* what) { return e == hipSuccess ? STITCH_OK : hip_fail(e, what); }

// Sizes of one camera's partial sums over a domain.
int64_t dg0_blocks(const Box& d) { return (int64_t)cdiv(d.w, 64) * cdiv(d.h, kDgRows); }

// What the passes need of one camera: descriptor, level regions and bands, and its arrays.
struct CamWork {
  VCam c;
  Box roi[kMaxLevels], band[kMaxLevels];
  double* g[kMaxLevels] = {};     // k >= 1
  double* gm[kMaxLevels] = {};    // k >= 1
  double* dg[kMaxLevels] = {};    // k >= 0; dg[0] on dom
  Box dom{0, 0, 0, 0};
  double* part = nullptr;
  Img3 direct{nullptr, 0, 0, 0};
  Inv9 hf;
  double delta = 0.0;
};

struct Dims {
  int W = 0, H = 0, L = 0, dw[kMaxLevels] = {}, dh[kMaxLevels] = {};
  void set(int w, int h, int levels) {
    W = w; H = h; L = levels;
    dw[0] = w; dh[0] = h;
    for (int k = 1; k < levels; ++k) { dw[k] = (dw[k - 1] + 1) / 2; dh[k] = (dh[k - 1] + 1) / 2; }
  }
};

int64_t area(const Box& b) { return (int64_t)b.w * b.h; }

// Weight (and image) pyramids of the cameras, levels 1 .. L-1.
template <bool FROZEN>
void launch_pyramids(const Dims& d, const std::vector<CamWork>& cw, bool img, bool wgt, hipStream_t s) {
  if (d.L < 2) return;
  const int n = (int)cw.size();
  Reduce0Args a;
  std::memset(&a, 0, sizeof a);
  a.W = d.W; a.H = d.H;
  int mw = 0, mh = 0;
  for (int i = 0; i < n; ++i) {
    a.cam[i].c = cw[i].c;
    a.cam[i].roi = cw[i].roi[1];
    a.cam[i].g = cw[i].g[1];
    a.cam[i].gm = wgt ? cw[i].gm[1] : nullptr;
    mw = std::max(mw, cw[i].roi[1].w);
    mh = std::max(mh, cw[i].roi[1].h);
  }
  if (mw <= 0 || mh <= 0) return;
  const dim3 g0(cdiv(mw, kRX), cdiv(mh, kRY), n);
  if (img) hipLaunchKernelGGL((k_vreduce0<FROZEN, true>), g0, dim3(kT), 0, s, a);
  else hipLaunchKernelGGL((k_vreduce0<FROZEN, false>), g0, dim3(kT), 0, s, a);
  for (int k = 1; k + 1 < d.L; ++k) {
    ReduceArgs r;
    std::memset(&r, 0, sizeof r);
    r.nw = d.dw[k]; r.nh = d.dh[k];
    mw = mh = 0;
    for (int i = 0; i < n; ++i) {
      ReduceCam& q = r.cam[i];
      q.g = img ? cw[i].g[k] : nullptr;
      q.gm = wgt ? cw[i].gm[k] : nullptr;
      q.in = cw[i].roi[k];
      q.og = cw[i].g[k + 1];
      q.ogm = cw[i].gm[k + 1];
      q.out = cw[i].roi[k + 1];
      mw = std::max(mw, q.out.w);
      mh = std::max(mh, q.out.h);
    }
    hipLaunchKernelGGL(k_vreduce, dim3(cdiv(mw, 64), cdiv(mh, 4), n), dim3(kT), 0, s, r);
  }
}

// One synthesis level k >= 1 of the cameras (see k_vblend).
void launch_blend_level(const Dims& d, int k, const std::vector<CamWork>& cw, const double* acc, const double* rc,
                        double* out, hipStream_t s) {
  BlendArgsV a;
  std::memset(&a, 0, sizeof a);
  a.n = (int)cw.size();
  a.w = d.dw[k]; a.h = d.dh[k];
  for (int i = 0; i < a.n; ++i) {
    BlendCamV& q = a.cam[i];
    q.g = cw[i].g[k];
    q.gm = cw[i].gm[k];
    q.roi = cw[i].roi[k];
    q.band = cw[i].band[k];
    if (k + 1 < d.L) {
      q.cg = cw[i].g[k + 1];
      q.croi = cw[i].roi[k + 1];
    }
  }
  a.acc = acc;
  a.rc = rc;
  if (k + 1 < d.L) { a.cw = d.dw[k + 1]; a.ch = d.dh[k + 1]; }
  a.out = out;
  hipLaunchKernelGGL(k_vblend, dim3(cdiv(a.w, 64), cdiv(a.h, 4)), dim3(kT), 0, s, a);
}

PanoCam pano_cam(const Dims& d, const CamWork& w) {
  PanoCam q;
  std::memset(&q, 0, sizeof q);
  q.c = w.c;
  q.band = w.band[0];
  if (d.L > 1) {
    q.cg = w.g[1];
    q.croi = w.roi[1];
  }
  return q;
}

// Arguments of one level of the cameras' dG recursion, k >= 1; false when every region is empty.
bool dg_args(const Dims& d, int k, const std::vector<CamWork>& cw, const Img3& dr0, double* const* dr, DgArgs& a,
             int& mw, int& mh) {
  std::memset(&a, 0, sizeof a);
  a.dr = dr[k];
  a.w = d.dw[k]; a.h = d.dh[k];
  a.fdr = k == 1 ? dr0 : Img3{dr[k - 1], d.dw[k - 1], (int64_t)d.dw[k - 1] * d.dh[k - 1], 1};
  a.nw = d.dw[k - 1]; a.nh = d.dh[k - 1];
  mw = mh = 0;
  for (size_t i = 0; i < cw.size(); ++i) {
    DgCam& q = a.cam[i];
    q.gm = cw[i].gm[k];
    q.roi = cw[i].roi[k]; q.band = cw[i].band[k];
    q.fgm = k == 1 ? nullptr : cw[i].gm[k - 1];
    q.froi = cw[i].roi[k - 1]; q.fband = cw[i].band[k - 1];
    q.c = cw[i].c;
    if (k + 1 < d.L) {
      q.dgc = cw[i].dg[k + 1];
      q.croi = cw[i].roi[k + 1];
    }
    q.out = cw[i].dg[k];
    mw = std::max(mw, q.roi.w);
    mh = std::max(mh, q.roi.h);
  }
  return mw > 0 && mh > 0;
}

// dR_{k+1} = EXPAND^T dR_k down to the top level; dr[k] for k >= 1.
void launch_dr(const Dims& d, const Img3& dr0, double* const* dr, hipStream_t s) {
  for (int k = 0; k + 1 < d.L; ++k) {
    if (k == 0) {
      TileTArgs a;
      std::memset(&a, 0, sizeof a);
      a.dg.w = d.dw[1]; a.dg.h = d.dh[1];
      a.dg.nw = d.W; a.dg.nh = d.H;
      a.dg.fdr = dr0;
      a.dr1 = dr[1];
      hipLaunchKernelGGL(k_vtileT, dim3(cdiv(d.dw[1], kRX), cdiv(d.dh[1], kRY)), dim3(kT), 0, s, a);
      continue;
    }
    hipLaunchKernelGGL(k_vexpandT, dim3(cdiv(d.dw[k + 1], 64), cdiv(d.dh[k + 1], 4)), dim3(kT), 0, s,
                       Img3{dr[k], d.dw[k], (int64_t)d.dw[k] * d.dh[k], 1}, d.dw[k], d.dh[k], dr[k + 1], d.dw[k + 1],
                       d.dh[k + 1]);
  }
}

// The cameras' dG recursion down to level 0, the map sums into sums[9 i ..] and the frame
// gradients; flag collects the gathers' refusals.
template <bool FROZEN>
void launch_adjoint(const Dims& d, const std::vector<CamWork>& cw, const Img3& dr0, double* const* dr,
                    const stitch_image* d_frames, double* sums, int* flag, hipStream_t s) {
  const int n = (int)cw.size(), L = d.L;
  int mw = 0, mh = 0;
  for (int k = L - 1; k >= 1; --k) {
    TileTArgs a;
    std::memset(&a, 0, sizeof a);
    if (!dg_args(d, k, cw, dr0, dr, a.dg, mw, mh)) continue;
    a.ncam = n;
    if (k == 1) hipLaunchKernelGGL(k_vtileT, dim3(cdiv(mw, kRX), cdiv(mh, kRY), n), dim3(kT), 0, s, a);
    else hipLaunchKernelGGL(k_vdg, dim3(cdiv(mw, 64), cdiv(mh, 4), n), dim3(kT), 0, s, a.dg);
  }
  Dg0Args a;
  std::memset(&a, 0, sizeof a);
  a.dr0 = dr0;
  a.W = d.W; a.H = d.H;
  SrcArgs t;
  std::memset(&t, 0, sizeof t);
  t.W = d.W; t.H = d.H;
  SumArgs u;
  std::memset(&u, 0, sizeof u);
  u.out = sums;
  int fw = 0, fh = 0;
  mw = mh = 0;
  for (int i = 0; i < n; ++i) {
    const CamWork& w = cw[i];
    Dg0Cam& q = a.cam[i];
    q.c = w.c;
    q.band = w.band[0];
    q.dom = w.dom;
    if (L > 1 && area(w.roi[1]) > 0) {
      q.dg1 = w.dg[1];
      q.croi = w.roi[1];
    }
    q.direct = w.direct;
    q.out = w.dg[0];
    q.part = w.part;
    mw = std::max(mw, w.dom.w);
    mh = std::max(mh, w.dom.h);
    u.part[i] = w.part;
    u.n[i] = (int)dg0_blocks(w.dom);
    SrcCam& g = t.cam[i];
    g.c = w.c;
    g.hf = w.hf;
    g.delta = w.delta;
    g.dg = w.dg[0];
    g.dom = w.dom;
    g.out = (float*)d_frames[i].data;
    g.orow = d_frames[i].row_pitch / 4;
    g.oplane = d_frames[i].plane_pitch / 4;
    fw = std::max(fw, w.c.fw);
    fh = std::max(fh, w.c.fh);
  }
  if (mw > 0 && mh > 0)
    hipLaunchKernelGGL((k_vdg0<FROZEN>), dim3(cdiv(mw, 64), cdiv(mh, kDgRows), n), dim3(kT), 0, s, a);
  hipLaunchKernelGGL(k_vsum9, dim3(9, n), dim3(kT), 0, s, u);
  hipLaunchKernelGGL((k_vsrcT<FROZEN>), dim3(cdiv(fw, 64), cdiv(fh, 4), n), dim3(kT), 0, s, t, flag);
}

// DLT: the homography (h33 = 1) taking the frame corners to q; false if singular.
bool dlt(const double q[8], int w, int h, double A[64], double hv[8]) {
  const double cx[4] = {0.0, (double)w - 1, (double)w - 1, 0.0}, cy[4] = {0.0, 0.0, (double)h - 1, (double)h - 1};
  double M[8][9];
  for (int k = 0; k < 4; ++k) {
    const double x = cx[k], y = cy[k], X = q[2 * k], Y = q[2 * k + 1];
    const double r0[9] = {x, y, 1, 0, 0, 0, -X * x, -X * y, X};
    const double r1[9] = {0, 0, 0, x, y, 1, -Y * x, -Y * y, Y};
    for (int j = 0; j < 9; ++j) { M[2 * k][j] = r0[j]; M[2 * k + 1][j] = r1[j]; }
  }
  for (int i = 0; i < 8; ++i)
    for (int j = 0; j < 8; ++j) A[i * 8 + j] = M[i][j];
  // Gaussian elimination with partial pivoting on the augmented system
  for (int c = 0; c < 8; ++c) {
    int piv = c;
    for (int r = c + 1; r < 8; ++r)
      if (std::fabs(M[r][c]) > std::fabs(M[piv][c])) piv = r;
    if (std::fabs(M[piv][c]) < 1e-300) return false;
    if (piv != c)
      for (int j = 0; j < 9; ++j) std::swap(M[c][j], M[piv][j]);
    for (int r = 0; r < 8; ++r) {
      if (r == c) continue;
      const double f = M[r][c] / M[c][c];
      for (int j = c; j < 9; ++j) M[r][j] -= f * M[c][j];
    }
  }
  for (int i = 0; i < 8; ++i) hv[i] = M[i][8] / M[i][i];
  return true;
}

// Solve A x = b (8x8) by elimination; false if singular.
bool solve8(const double A_in[64], const double b_in[8], double x[8]) {
  double M[8][9];
  for (int i = 0; i < 8; ++i) {
    for (int j = 0; j < 8; ++j) M[i][j] = A_in[i * 8 + j];
    M[i][8] = b_in[i];
  }
  for (int c = 0; c < 8; ++c) {
    int piv = c;
    for (int r = c + 1; r < 8; ++r)
      if (std::fabs(M[r][c]) > std::fabs(M[piv][c])) piv = r;
    if (std::fabs(M[piv][c]) < 1e-300) return false;
    if (piv != c)
      for (int j = 0; j < 9; ++j) std::swap(M[c][j], M[piv][j]);
    for (int r = 0; r < 8; ++r) {
      if (r == c) continue;
      const double f = M[r][c] / M[c][c];
      for (int j = c; j < 9; ++j) M[r][j] -= f * M[c][j];
    }
  }
  for (int i = 0; i < 8; ++i) x[i] = M[i][8] / M[i][i];
  return true;
}

bool inv3(const double* a, double* o) {
  const double c00 = a[4] * a[8] - a[5] * a[7], c01 = a[5] * a[6] - a[3] * a[8], c02 = a[3] * a[7] - a[4] * a[6];
  const double det = a[0] * c00 + a[1] * c01 + a[2] * c02;
  if (det == 0.0 || !std::isfinite(det)) return false;
  o[0] = c00 / det; o[1] = (a[2] * a[7] - a[1] * a[8]) / det; o[2] = (a[1] * a[5] - a[2] * a[4]) / det;
  o[3] = c01 / det; o[4] = (a[0] * a[8] - a[2] * a[6]) / det; o[5] = (a[2] * a[3] - a[0] * a[5]) / det;
  o[6] = c02 / det; o[7] = (a[1] * a[6] - a[0] * a[7]) / det; o[8] = (a[0] * a[4] - a[1] * a[3]) / det;
  return true;
}


// Bound, in source samples, of the FP32 coordinate sequence's error at any canvas pixel whose
// FP32 source position lies in [-1, fw] x [-1, fh]; hf is the FP64 inverse of m.  With
// e = 2^-24 each of u, v, z is within 3.1 e of its own sum of magnitudes; hf's last row
// applied to (u, v, z) is 1, which bounds z from below by 0.5 over the largest depth of the
// frame (as long as the errors' share of that 1 stays under a half), and a quotient is off by
// the numerator's and denominator's errors over z plus its own rounding.  1 (the caller then
// widens by a whole pixel) when the premises fail.
double coord_delta(const Map9& m, const Inv9& hf, int W, int H, int fw, int fh) {
  const double e = 3.1 * 0x1p-24;
  double d[3];
  for (int i = 0; i < 3; ++i)
    d[i] = e * (std::fabs((double)m.h[3 * i]) * W + std::fabs((double)m.h[3 * i + 1]) * H + std::fabs((double)m.h[3 * i + 2]));
  double share = 0.0, wmax = 0.0;
  for (int i = 0; i < 3; ++i) share += std::fabs(hf.h[6 + i]) * d[i];
  for (int k = 0; k < 4; ++k) {
    const double x = (k & 1) ? fw + 1.0 : -2.0, y = (k & 2) ? fh + 1.0 : -2.0;
    wmax = std::max(wmax, hf.h[6] * x + hf.h[7] * y + hf.h[8]);
  }
  if (!(share < 0.5) || !(wmax > 0.0)) return 1.0;
  const double zlo = 0.5 / wmax, side = std::max(fw, fh) + 2.0;
  if (!(d[2] < 0.5 * zlo)) return 1.0;
  const double r = (std::max(d[0], d[1]) + side * d[2]) / (zlo - d[2]) + side * 0x1p-24;
  return r < 1.0 ? r : 1.0;
}

// Level regions and bands of a camera whose seam weights have the support box sup: the band is
// the weights' support at each level, the region what the blend needs below it (as the
// planner's, without the footprint).
void regions_of(const Dims& d, const Box& sup, Box roi[], Box band[]) {
  const int L = d.L;
  int lo0[2] = {1, 1}, hi0[2] = {0, 0};
  int blo[2][kMaxLevels], bhi[2][kMaxLevels];
  for (int ax = 0; ax < 2; ++ax) {
    int a = ax ? sup.y : sup.x, b = (ax ? sup.y + sup.h : sup.x + sup.w) - 1;
    for (int k = 0; k < L; ++k) {
      if (k > 0) { a = (a - 1) >> 1; b = (b + 2) >> 1; }
      blo[ax][k] = std::max(0, a);
      bhi[ax][k] = std::min((ax ? d.dh[k] : d.dw[k]) - 1, b);
    }
    int lo = blo[ax][L - 1], hi = bhi[ax][L - 1], mlo = lo, mhi = hi;
    for (int k = L - 2; k >= 0; --k) {
      lo = std::min(lo, (blo[ax][k] - 1) >> 1);     // EXPAND's support of band k
      hi = std::max(hi, (bhi[ax][k] + 2) >> 1);
      lo = std::min(blo[ax][k], 2 * lo - 2);
      hi = std::max(bhi[ax][k], 2 * hi + 2);
      mlo = std::min(blo[ax][k], 2 * mlo - 2);
      mhi = std::max(bhi[ax][k], 2 * mhi + 2);
    }
    lo0[ax] = std::min(lo, mlo);
    hi0[ax] = std::max(hi, mhi);
  }
  const int A = 1 << (L - 1);
  int x0 = std::max(0, lo0[0]) / A * A, y0 = std::max(0, lo0[1]) / A * A;
  int x1 = std::min(d.W, cdiv(std::max(hi0[0] + 1, 0), A) * A), y1 = std::min(d.H, cdiv(std::max(hi0[1] + 1, 0), A) * A);
  const bool none = sup.w <= 0 || sup.h <= 0 || x0 >= x1 || y0 >= y1;
  for (int k = 0; k < L; ++k) {
    roi[k] = band[k] = Box{0, 0, 0, 0};
    if (none) continue;
    const int xa = x0 >> k, ya = y0 >> k;
    const int xb = std::min(d.dw[k], (x1 + (1 << k) - 1) >> k), yb = std::min(d.dh[k], (y1 + (1 << k) - 1) >> k);
    roi[k] = Box{xa, ya, xb - xa, yb - ya};
    band[k] = Box{blo[0][k], blo[1][k], bhi[0][k] - blo[0][k] + 1, bhi[1][k] - blo[1][k] + 1};
  }
}

}  // namespace

struct stitch_grad {
  Dims d;
  int fw[2] = {}, fh[2] = {};
  std::vector<uint8_t> masks;        // 2 * W * H
  uint8_t* ws = nullptr;
  size_t bytes = 0;
  Box roi[2][kMaxLevels], band[2][kMaxLevels];
  // offsets
  size_t o_mask, o_gm[2][kMaxLevels], o_x0, o_y0, o_om, o_g[2][kMaxLevels], o_r[kMaxLevels];
  size_t o_ga, o_gb, o_gp, o_dr[kMaxLevels], o_dg[2][kMaxLevels], o_part9[2];
  size_t o_part, o_res, o_flag;
  int nbx = 0, nby = 0;              // 64 x kDgRows blocks of the canvas
  bool frozen = false;
  Inv9 freeze_inv[2];   // FP64 inverses of the maps the cells were frozen at
  double freeze_delta[2] = {};
  double omega_n = 0.0;
  Map9 maps[2];
  const float* fsrc[2] = {};
  int64_t frow[2] = {}, fplane[2] = {};
  bool have_forward = false;
  double* dptr(size_t o) const { return (double*)(ws + o); }
};

namespace {

stitch_status maps_from(const double* H, Map9 out[2]) {
  for (int c = 0; c < 2; ++c) {
    const char* why = nullptr;
    if (!hinv_spec(H + 9 * c, out[c].h, nullptr, &why)) return fail(STITCH_E_HOMOGRAPHY, "camera %d: %s", c, why);
  }
  return STITCH_OK;
}

// Both cameras of the pair with their arrays; frames and maps as of the last forward.
std::vector<CamWork> pair_work(const stitch_grad* g) {
  std::vector<CamWork> cw(2);
  const int64_t np = (int64_t)g->d.W * g->d.H;
  for (int c = 0; c < 2; ++c) {
    CamWork& w = cw[c];
    std::memset(&w.c, 0, sizeof w.c);
    w.c.m = g->maps[c];
    w.c.fw = g->fw[c];
    w.c.fh = g->fh[c];
    w.c.src = g->fsrc[c];
    w.c.srow = g->frow[c];
    w.c.splane = g->fplane[c];
    w.c.x0a = (const int*)(g->ws + g->o_x0) + c * np;
    w.c.y0a = (const int*)(g->ws + g->o_y0) + c * np;
    w.c.wrows = g->ws + g->o_mask + c * np;
    w.c.wbox = Box{0, 0, g->d.W, g->d.H};
    for (int k = 0; k < g->d.L; ++k) {
      w.roi[k] = g->roi[c][k];
      w.band[k] = g->band[c][k];
      if (k >= 1) {
        w.g[k] = g->dptr(g->o_g[c][k]);
        w.gm[k] = g->dptr(g->o_gm[c][k]);
      }
      w.dg[k] = g->dptr(g->o_dg[c][k]);
    }
    w.dom = Box{0, 0, g->d.W, g->d.H};
    w.part = g->dptr(g->o_part9[c]);
    w.hf = g->freeze_inv[c];
    w.delta = g->freeze_delta[c];
  }
  return cw;
}

}  // namespace

extern "C" {

stitch_status stitch_grad_create(const int32_t frame_w[2], const int32_t frame_h[2], const uint8_t* const* masks,
                                 int32_t canvas_w, int32_t canvas_h, int32_t levels, stitch_grad** out) {
  if (!out) return fail(STITCH_E_NULL, "out is NULL");
  *out = nullptr;
  if (!frame_w || !frame_h || !masks || !masks[0] || !masks[1]) return fail(STITCH_E_NULL, "sizes or masks NULL");
  if (levels < 1 || levels > kMaxLevels) return fail(STITCH_E_LEVELS, "levels %d outside 1..%d", levels, kMaxLevels);
  if (canvas_w <= 0 || canvas_h <= 0 || (int64_t)canvas_w * canvas_h > (1 << 26))
    return fail(STITCH_E_SHAPE, "canvas %dx%d outside the gradient form's range", canvas_w, canvas_h);
  stitch_grad* g = new (std::nothrow) stitch_grad();
  if (!g) return fail(STITCH_E_UNSUPPORTED, "out of host memory");
  struct Guard { stitch_grad*& g; ~Guard() { delete g; } } guard{g};
  g->d.set(canvas_w, canvas_h, levels);
  for (int k = 0; k < levels; ++k)
    if (g->d.dw[k] < 3 || g->d.dh[k] < 3) return fail(STITCH_E_LEVELS, "level %d side below 3", k);
  for (int c = 0; c < 2; ++c) {
    if (frame_w[c] <= 0 || frame_h[c] <= 0 || (int64_t)frame_w[c] * frame_h[c] > (1 << 26))
      return fail(STITCH_E_SHAPE, "frame %d size %dx%d", c, frame_w[c], frame_h[c]);
    g->fw[c] = frame_w[c]; g->fh[c] = frame_h[c];
  }
  const size_t np = (size_t)canvas_w * canvas_h;
  int off = 0;
  for (size_t i = 0; i < np; ++i) off |= ((int)masks[0][i] + (int)masks[1][i]) ^ 255;
  if (off) return fail(STITCH_E_MASK, "seam weights do not sum to 255");
  for (int c = 0; c < 2; ++c) g->masks.insert(g->masks.end(), masks[c], masks[c] + np);
  for (int c = 0; c < 2; ++c) {
    int box[4] = {0, 0, 0, 0};
    weight_box(masks[c], canvas_w, canvas_h, box);
    regions_of(g->d, Box{box[0], box[1], box[2], box[3]}, g->roi[c], g->band[c]);
  }
  size_t top = 0;
  const Box all{0, 0, canvas_w, canvas_h};
  g->o_mask = take(top, 2 * np);
  for (int c = 0; c < 2; ++c)
    for (int k = 1; k < levels; ++k) {
      g->o_gm[c][k] = take(top, area(g->roi[c][k]) * 8);
      g->o_g[c][k] = take(top, 3 * area(g->roi[c][k]) * 8);
    }
  g->o_x0 = take(top, 2 * np * 4);
  g->o_y0 = take(top, 2 * np * 4);
  g->o_om = take(top, np);
  for (int k = 1; k < levels; ++k) {
    g->o_r[k] = take(top, 3 * (size_t)g->d.dw[k] * g->d.dh[k] * 8);
    g->o_dr[k] = take(top, 3 * (size_t)g->d.dw[k] * g->d.dh[k] * 8);
  }
  g->o_gp = take(top, 3 * np * 8);
  g->o_ga = take(top, 3 * np * 8);
  g->o_gb = take(top, 3 * np * 8);
  g->nbx = cdiv(canvas_w, 64);
  g->nby = cdiv(canvas_h, kDgRows);
  for (int c = 0; c < 2; ++c) {
    for (int k = 0; k < levels; ++k) g->o_dg[c][k] = take(top, 3 * area(k ? g->roi[c][k] : all) * 8);
    g->o_part9[c] = take(top, (size_t)dg0_blocks(all) * 9 * 8);
  }
  g->o_part = take(top, (size_t)g->nbx * g->nby * 8);
  g->o_res = take(top, 32 * 8);
  g->o_flag = g->o_res + 18 * 8;
  g->bytes = top;
  *out = g;
  g = nullptr;
  return STITCH_OK;
}

size_t stitch_grad_workspace_bytes(const stitch_grad* g) { return g ? g->bytes : 0; }

stitch_status stitch_grad_bind(stitch_grad* g, void* workspace, size_t bytes, void* stream) {
  return guarded([&]() -> stitch_status {
    if (!g) return fail(STITCH_E_NULL, "grad is NULL");
    if (!workspace || ((uintptr_t)workspace & 255) || bytes < g->bytes)
      return fail(STITCH_E_WORKSPACE, "workspace missing, misaligned or smaller than %zu bytes", g->bytes);
    const hipStream_t s = (hipStream_t)stream;
    g->ws = (uint8_t*)workspace;
    g->frozen = false;
    g->have_forward = false;
    stitch_status st = dev_ok(hipMemcpyAsync(g->ws + g->o_mask, g->masks.data(), g->masks.size(), hipMemcpyHostToDevice, s),
                              "mask upload");
    if (!st) {
      launch_pyramids<true>(g->d, pair_work(g), false, true, s);
      st = dev_ok(hipGetLastError(), "weight pyramid launch");
    }
    if (!st) st = dev_ok(hipStreamSynchronize(s), "bind synchronise");
    if (st) g->ws = nullptr;
    return st;
  });
}

stitch_status stitch_grad_freeze(stitch_grad* g, const double H[18], int64_t* omega_count, void* stream) {
  if (!g || !H) return fail(STITCH_E_NULL, "grad or H is NULL");
  if (!g->ws) return fail(STITCH_E_STATE, "no workspace bound");
  Map9 m[2];
  stitch_status st = maps_from(H, m);
  if (st) return st;
  Inv9 inv[2];
  for (int c = 0; c < 2; ++c) {
    double M[9];
    for (int j = 0; j < 9; ++j) M[j] = (double)m[c].h[j];
    if (!inv3(M, inv[c].h)) return fail(STITCH_E_HOMOGRAPHY, "camera %d: its map is singular", c);
  }
  const hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_gcells, dim3(g->nbx, g->nby), dim3(kT), 0, s, m[0], m[1], g->fw[0], g->fh[0], g->fw[1], g->fh[1],
                     g->d.W, g->d.H, (int*)(g->ws + g->o_x0), (int*)(g->ws + g->o_y0), g->ws + g->o_om,
                     g->dptr(g->o_part));
  hipLaunchKernelGGL(k_gsum, dim3(1), dim3(kT), 0, s, g->dptr(g->o_part), g->nbx * g->nby, g->dptr(g->o_res));
  st = dev_ok(hipGetLastError(), "freeze launch");
  double n = 0.0;
  if (!st) st = dev_ok(hipMemcpyAsync(&n, g->dptr(g->o_res), 8, hipMemcpyDeviceToHost, s), "count copy");
  if (!st) st = dev_ok(hipStreamSynchronize(s), "freeze synchronise");
  if (st) return st;
  if (n < 1.0) return fail(STITCH_E_SHAPE, "the frames do not overlap at these maps (|Omega| = 0)");
  g->omega_n = n;
  for (int c = 0; c < 2; ++c) {
    g->freeze_inv[c] = inv[c];
    g->freeze_delta[c] = coord_delta(m[c], inv[c], g->d.W, g->d.H, g->fw[c], g->fh[c]);
  }
  g->frozen = true;
  g->have_forward = false;
  if (omega_count) *omega_count = (int64_t)n;
  return STITCH_OK;
}

stitch_status stitch_grad_forward(stitch_grad* g, const stitch_image* frames, const double H[18], double* loss,
                                  void* stream) {
  return guarded([&]() -> stitch_status {
    if (!g || !frames || !H || !loss) return fail(STITCH_E_NULL, "grad, frames, H or loss is NULL");
    if (!g->ws) return fail(STITCH_E_STATE, "no workspace bound");
    if (!g->frozen) return fail(STITCH_E_STATE, "call stitch_grad_freeze first");
    for (int c = 0; c < 2; ++c) {
      stitch_status st = check_image(&frames[c], c ? "frames[1]" : "frames[0]", STITCH_F32, STITCH_CHW, 3);
      if (st) return st;
      if (frames[c].width != g->fw[c] || frames[c].height != g->fh[c])
        return fail(STITCH_E_SHAPE, "frames[%d] does not match the planned size", c);
    }
    Map9 m[2];
    stitch_status st = maps_from(H, m);
    if (st) return st;
    const hipStream_t s = (hipStream_t)stream;
    const Dims& d = g->d;
    for (int c = 0; c < 2; ++c) {
      g->maps[c] = m[c];
      g->fsrc[c] = (const float*)frames[c].data;
      g->frow[c] = frames[c].row_pitch / 4;
      g->fplane[c] = frames[c].plane_pitch / 4;
    }
    const std::vector<CamWork> cw = pair_work(g);
    launch_pyramids<true>(d, cw, true, false, s);
    for (int k = d.L - 1; k >= 1; --k)
      launch_blend_level(d, k, cw, nullptr, k + 1 < d.L ? g->dptr(g->o_r[k + 1]) : nullptr, g->dptr(g->o_r[k]), s);
    LossArgs a;
    std::memset(&a, 0, sizeof a);
    for (int c = 0; c < 2; ++c) a.cam[c] = pano_cam(d, cw[c]);
    a.W = d.W; a.H = d.H;
    if (d.L > 1) { a.rc = g->dptr(g->o_r[1]); a.cw = d.dw[1]; a.ch = d.dh[1]; }
    a.omega = g->ws + g->o_om;
    a.scale = 1.0 / (6.0 * g->omega_n);
    a.ga = g->dptr(g->o_ga);
    a.gb = g->dptr(g->o_gb);
    a.part = g->dptr(g->o_part);
    hipLaunchKernelGGL(k_gloss, dim3(g->nbx, g->nby), dim3(kT), 0, s, a);
    hipLaunchKernelGGL(k_gsum, dim3(1), dim3(kT), 0, s, g->dptr(g->o_part), g->nbx * g->nby, g->dptr(g->o_res));
    st = dev_ok(hipGetLastError(), "forward launch");
    double sum = 0.0;
    if (!st) st = dev_ok(hipMemcpyAsync(&sum, g->dptr(g->o_res), 8, hipMemcpyDeviceToHost, s), "loss copy");
    if (!st) st = dev_ok(hipStreamSynchronize(s), "forward synchronise");
    if (st) return st;
    *loss = sum / (6.0 * g->omega_n);
    g->have_forward = true;
    return STITCH_OK;
  });
}

stitch_status stitch_grad_backward(stitch_grad* g, stitch_image* d_frames, double d_map[18], void* stream) {
  return guarded([&]() -> stitch_status {
    if (!g || !d_frames || !d_map) return fail(STITCH_E_NULL, "grad, d_frames or d_map is NULL");
    if (!g->have_forward) return fail(STITCH_E_STATE, "call stitch_grad_forward first");
    for (int c = 0; c < 2; ++c) {
      stitch_status st = check_image(&d_frames[c], c ? "d_frames[1]" : "d_frames[0]", STITCH_F32, STITCH_CHW, 3);
      if (st) return st;
      if (d_frames[c].width != g->fw[c] || d_frames[c].height != g->fh[c])
        return fail(STITCH_E_SHAPE, "d_frames[%d] does not match the planned size", c);
    }
    const hipStream_t s = (hipStream_t)stream;
    const Dims& d = g->d;
    const int64_t np = (int64_t)d.W * d.H;
    double* dr[kMaxLevels] = {};
    for (int k = 1; k < d.L; ++k) dr[k] = g->dptr(g->o_dr[k]);
    const Img3 dr0{g->dptr(g->o_gp), d.W, np, 1};
    hipLaunchKernelGGL(k_gzero, dim3(1), dim3(1), 0, s, g->dptr(g->o_flag));
    hipLaunchKernelGGL(k_gpano, dim3(blocks(3 * np)), dim3(kT), 0, s, g->dptr(g->o_ga), g->dptr(g->o_gb), 3 * np,
                       g->dptr(g->o_gp));
    launch_dr(d, dr0, dr, s);
    std::vector<CamWork> cw = pair_work(g);
    cw[0].direct = Img3{g->dptr(g->o_ga), d.W, np, 1};
    cw[1].direct = Img3{g->dptr(g->o_gb), d.W, np, 1};
    launch_adjoint<true>(d, cw, dr0, dr, d_frames, g->dptr(g->o_res), (int*)(g->ws + g->o_flag), s);
    stitch_status st = dev_ok(hipGetLastError(), "backward launch");
    double res[19];
    if (!st) st = dev_ok(hipMemcpyAsync(res, g->dptr(g->o_res), sizeof res, hipMemcpyDeviceToHost, s), "grad copy");
    if (!st) st = dev_ok(hipStreamSynchronize(s), "backward synchronise");
    if (st) return st;
    int flag = 0;
    std::memcpy(&flag, &res[18], sizeof flag);
    if (flag)
      return fail(STITCH_E_UNSUPPORTED, "a frozen map %s",
                  (flag & 2) ? "reaches its horizon over the frame" : "magnifies a source pixel over about 20 times");
    for (int i = 0; i < 18; ++i) d_map[i] = res[i];
    return STITCH_OK;
  });
}

stitch_status stitch_grad_upstream(stitch_grad* g, stitch_image* d_pano, stitch_image* d_warped, void* stream) {
  if (!g || !d_pano || !d_warped) return fail(STITCH_E_NULL, "grad, d_pano or d_warped is NULL");
  if (!g->have_forward) return fail(STITCH_E_STATE, "call stitch_grad_forward first");
  stitch_image* outs[3] = {d_pano, &d_warped[0], &d_warped[1]};
  const char* names[3] = {"d_pano", "d_warped[0]", "d_warped[1]"};
  Out3 o[3];
  for (int i = 0; i < 3; ++i) {
    const stitch_status st = check_image(outs[i], names[i], STITCH_F32, STITCH_CHW, 3);
    if (st) return st;
    if (outs[i]->width != g->d.W || outs[i]->height != g->d.H) return fail(STITCH_E_SHAPE, "%s is not canvas-sized", names[i]);
    o[i] = Out3{(float*)outs[i]->data, outs[i]->row_pitch / 4, outs[i]->plane_pitch / 4};
  }
  hipLaunchKernelGGL(k_gupstream, dim3(cdiv(g->d.W, 64), cdiv(g->d.H, 4)), dim3(kT), 0, (hipStream_t)stream,
                     g->dptr(g->o_ga), g->dptr(g->o_gb), g->d.W, g->d.H, o[0], o[1], o[2]);
  return dev_ok(hipGetLastError(), "upstream launch");
}

void stitch_grad_destroy(stitch_grad* g) { delete g; }

}  // extern "C"

// ------------------------------------------------------------------------------------ VJP host
namespace {

// Workspace of the float-frame forward and its VJP for one plan.  The size is that of the
// whole-canvas form (per level a weight plane and four 3-plane arrays: room for any camera's
// regions).  R_k or dR_k (k >= 1) and the sums come first, then, with several camera groups,
// the FP64 level-0 accumulator; the rest holds the regions of one group of cameras at a time.
struct VjpLayout {
  Dims d;
  int n = 0;
  size_t o_r[kMaxLevels] = {}, o_acc = 0, o_res = 0, o_flag = 0, o_group = 0, o_group_acc = 0, bytes = 0;
};

stitch_status vjp_layout(const stitch_plan* p, VjpLayout& v) {
  if (!p) return fail(STITCH_E_NULL, "plan is NULL");
  int fw[kMaxCameras], fh[kMaxCameras], W, H;
  bool bound = false;
  plan_geometry(p, &v.n, fw, fh, &W, &H, &bound);
  if ((int64_t)W * H > (1 << 26))
    return fail(STITCH_E_SHAPE, "canvas %dx%d above the differentiable form's 2^26 pixels", W, H);
  v.d.set(W, H, plan_levels(p));
  size_t whole = 0;
  for (int k = 0; k < v.d.L; ++k) {
    const size_t nk = (size_t)v.d.dw[k] * v.d.dh[k] * 8;
    take(whole, nk);
    for (int j = 0; j < 4; ++j) take(whole, 3 * nk);
  }
  take(whole, (size_t)blocks((int64_t)W * H) * 9 * 8);
  size_t top = 0;
  v.o_res = take(top, (size_t)(9 * v.n + 1) * 8);
  v.o_flag = v.o_res + (size_t)9 * v.n * 8;
  for (int k = 1; k < v.d.L; ++k) v.o_r[k] = take(top, 3 * (size_t)v.d.dw[k] * v.d.dh[k] * 8);
  v.o_group = top;
  v.o_acc = take(top, 3 * (size_t)W * H * 8);
  v.o_group_acc = top;
  // one camera on whole-canvas regions always fits behind the accumulator
  for (int k = 1; k < v.d.L; ++k) {
    take(top, (size_t)v.d.dw[k] * v.d.dh[k] * 8);
    take(top, 3 * (size_t)v.d.dw[k] * v.d.dh[k] * 8);
  }
  take(top, 3 * (size_t)W * H * 8);
  take(top, (size_t)dg0_blocks(Box{0, 0, W, H}) * 9 * 8);
  take(top, (size_t)W * H + (size_t)H * 4);
  v.bytes = std::max(whole, top);
  return STITCH_OK;
}

stitch_status vjp_check_frames(const stitch_plan* p, int n, const stitch_image* frames, const char* what) {
  for (int i = 0; i < n; ++i) {
    PlanCamera pc;
    plan_camera(p, i, &pc);
    char name[48];
    snprintf(name, sizeof name, "%s[%d]", what, i);
    const stitch_status st = check_image(&frames[i], name, STITCH_F32, STITCH_CHW, 3);
    if (st) return st;
    if (frames[i].width != pc.fw || frames[i].height != pc.fh)
      return fail(STITCH_E_SHAPE, "%s is %dx%d, planned %dx%d", name, frames[i].width, frames[i].height, pc.fw, pc.fh);
  }
  return STITCH_OK;
}

// Camera i of the plan; false (HOMOGRAPHY) when its map has no inverse.
bool vjp_camera(const stitch_plan* p, const VjpLayout& v, int i, const stitch_image& frame, CamWork& w, PlanCamera& pc) {
  plan_camera(p, i, &pc);
  std::memset(&w.c, 0, sizeof w.c);
  std::memcpy(w.c.m.h, pc.hinv, sizeof pc.hinv);
  double M[9];
  for (int j = 0; j < 9; ++j) M[j] = (double)pc.hinv[j];
  if (!inv3(M, w.hf.h)) return false;
  w.c.fw = pc.fw;
  w.c.fh = pc.fh;
  w.c.src = (const float*)frame.data;
  w.c.srow = frame.row_pitch / 4;
  w.c.splane = frame.plane_pitch / 4;
  w.delta = coord_delta(w.c.m, w.hf, v.d.W, v.d.H, pc.fw, pc.fh);
  for (int k = 0; k < v.d.L; ++k) {
    w.roi[k] = Box{pc.roi[k][0], pc.roi[k][1], pc.roi[k][2], pc.roi[k][3]};
    w.band[k] = Box{pc.band[k][0], pc.band[k][1], pc.band[k][2], pc.band[k][3]};
  }
  return true;
}

// Place camera w's arrays at `top` of the workspace (nothing is written yet).
void vjp_place(const VjpLayout& v, uint8_t* ws, bool backward, const PlanCamera& pc, CamWork& w, size_t& top) {
  const size_t wd = take(top, pc.wdict_bytes);
  w.c.wbox = Box{pc.wx, pc.wy, pc.wdict_bytes ? pc.ww : 0, pc.wdict_bytes ? pc.wh : 0};
  w.c.wrow = (const uint32_t*)(ws + wd);
  w.c.wrows = ws + wd + (size_t)pc.wh * 4;
  for (int k = 1; k < v.d.L; ++k) {
    const size_t a = (size_t)area(w.roi[k]) * 8;
    w.gm[k] = (double*)(ws + take(top, a));
    (backward ? w.dg[k] : w.g[k]) = (double*)(ws + take(top, 3 * a));
  }
  if (backward) {
    w.dg[0] = (double*)(ws + take(top, 3 * (size_t)area(w.dom) * 8));
    w.part = (double*)(ws + take(top, (size_t)dg0_blocks(w.dom) * 9 * 8));
  }
}

// The plan's cameras as groups that fit behind `base` of the workspace, at most kGroup each.
struct VjpGroup {
  int first = 0;
  std::vector<CamWork> cw;
  std::vector<PlanCamera> pc;
};
std::vector<VjpGroup> vjp_groups(const VjpLayout& v, uint8_t* ws, size_t base, bool backward,
                                 const std::vector<CamWork>& cams, const std::vector<PlanCamera>& pcs) {
  std::vector<VjpGroup> out;
  size_t top = base;
  for (int i = 0; i < v.n; ++i) {
    CamWork w = cams[i];
    size_t t = top;
    vjp_place(v, ws, backward, pcs[i], w, t);
    if (out.empty() || (int)out.back().cw.size() == kGroup || t > v.bytes) {
      out.emplace_back();
      out.back().first = i;
      t = base;
      vjp_place(v, ws, backward, pcs[i], w, t);
    }
    top = t;
    out.back().cw.push_back(w);
    out.back().pc.push_back(pcs[i]);
  }
  return out;
}

// Upload the group's seam weights (the copies of pageable memory have left it on return).
stitch_status vjp_upload(const VjpGroup& g, hipStream_t s) {
  for (size_t i = 0; i < g.cw.size(); ++i) {
    if (!g.pc[i].wdict_bytes) continue;
    const hipError_t e = hipMemcpyAsync((void*)g.cw[i].c.wrow, g.pc[i].wdict, g.pc[i].wdict_bytes, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "weight upload");
  }
  return STITCH_OK;
}

stitch_status vjp_check_ws(const VjpLayout& v, void* ws, size_t bytes) {
  if (!ws || ((uintptr_t)ws & 255) || bytes < v.bytes)
    return fail(STITCH_E_WORKSPACE, "workspace missing, misaligned or smaller than %zu bytes", v.bytes);
  return STITCH_OK;
}

}  // namespace

extern "C" {

size_t stitch_frame_backward_workspace_bytes(const stitch_plan* plan) {
  VjpLayout v;
  return vjp_layout(plan, v) ? 0 : v.bytes;
}

stitch_status stitch_frame_forward_f32(stitch_plan* plan, const stitch_image* frames, stitch_image* r0,
                                       void* workspace, size_t bytes, void* stream) {
  return guarded([&]() -> stitch_status {
    if (!plan || !frames || !r0) return fail(STITCH_E_NULL, "plan, frames or r0 is NULL");
    VjpLayout v;
    stitch_status st = vjp_layout(plan, v);
    if (st) return st;
    if ((st = vjp_check_ws(v, workspace, bytes))) return st;
    if ((st = vjp_check_frames(plan, v.n, frames, "frames"))) return st;
    std::vector<CamWork> cams(v.n);
    std::vector<PlanCamera> pcs(v.n);
    for (int i = 0; i < v.n; ++i)
      if (!vjp_camera(plan, v, i, frames[i], cams[i], pcs[i]))
        return fail(STITCH_E_HOMOGRAPHY, "camera %d: its map is singular", i);
    if ((st = check_image(r0, "r0", STITCH_F32, STITCH_CHW, 3))) return st;
    if (r0->width != v.d.W || r0->height != v.d.H) return fail(STITCH_E_SHAPE, "r0 is not canvas-sized");
    const hipStream_t s = (hipStream_t)stream;
    uint8_t* ws = (uint8_t*)workspace;
    auto D = [&](size_t o) { return (double*)(ws + o); };
    const int L = v.d.L;
    std::vector<VjpGroup> groups = vjp_groups(v, ws, v.o_group, false, cams, pcs);
    if (groups.size() > 1) groups = vjp_groups(v, ws, v.o_group_acc, false, cams, pcs);
    for (size_t q = 0; q < groups.size() && !st; ++q) {
      const VjpGroup& g = groups[q];
      const bool first = q == 0, last = q + 1 == groups.size();
      if ((st = vjp_upload(g, s))) break;
      launch_pyramids<false>(v.d, g.cw, true, true, s);
      // B_k accumulates over the groups in R_k's place; the last one collapses
      for (int k = L - 1; k >= 1; --k)
        launch_blend_level(v.d, k, g.cw, first ? nullptr : D(v.o_r[k]), last && k + 1 < L ? D(v.o_r[k + 1]) : nullptr,
                           D(v.o_r[k]), s);
      PanoArgs a;
      std::memset(&a, 0, sizeof a);
      a.n = (int)g.cw.size();
      for (int i = 0; i < a.n; ++i) a.cam[i] = pano_cam(v.d, g.cw[i]);
      a.W = v.d.W; a.H = v.d.H;
      a.acc = first ? nullptr : D(v.o_acc);
      if (last && L > 1) { a.rc = D(v.o_r[1]); a.cw = v.d.dw[1]; a.ch = v.d.dh[1]; }
      if (last) {
        a.out32 = (float*)r0->data;
        a.orow = r0->row_pitch / 4;
        a.oplane = r0->plane_pitch / 4;
      } else {
        a.out64 = D(v.o_acc);
      }
      hipLaunchKernelGGL(k_vpano, dim3(cdiv(a.W, 64), cdiv(a.H, 4)), dim3(kT), 0, s, a);
      st = dev_ok(hipGetLastError(), "forward launch");
    }
    return st;
  });
}

stitch_status stitch_frame_backward(stitch_plan* plan, const stitch_image* frames, const stitch_image* d_pano,
                                    const stitch_image* d_warped, stitch_image* d_frames, double* d_hinv,
                                    void* workspace, size_t bytes, void* stream) {
  return guarded([&]() -> stitch_status {
    if (!plan || !frames || !d_pano || !d_frames || !d_hinv)
      return fail(STITCH_E_NULL, "plan, frames, d_pano, d_frames or d_hinv is NULL");
    VjpLayout v;
    stitch_status st = vjp_layout(plan, v);
    if (st) return st;
    if ((st = vjp_check_ws(v, workspace, bytes))) return st;
    if ((st = vjp_check_frames(plan, v.n, frames, "frames"))) return st;
    std::vector<CamWork> cams(v.n);
    std::vector<PlanCamera> pcs(v.n);
    for (int i = 0; i < v.n; ++i)
      if (!vjp_camera(plan, v, i, frames[i], cams[i], pcs[i]))
        return fail(STITCH_E_HOMOGRAPHY, "camera %d: its map is singular", i);
    if ((st = vjp_check_frames(plan, v.n, d_frames, "d_frames"))) return st;
    if ((st = check_image(d_pano, "d_pano", STITCH_F32, STITCH_CHW, 3))) return st;
    if (d_pano->width != v.d.W || d_pano->height != v.d.H) return fail(STITCH_E_SHAPE, "d_pano is not canvas-sized");
    for (int i = 0; i < v.n; ++i) {
      // dG_0 is needed where the weights reach; with a direct term, everywhere
      cams[i].dom = cams[i].roi[0];
      if (!d_warped || !d_warped[i].data) continue;
      char name[40];
      snprintf(name, sizeof name, "d_warped[%d]", i);
      if ((st = check_image(&d_warped[i], name, STITCH_F32, STITCH_CHW, 3))) return st;
      if (d_warped[i].width != v.d.W || d_warped[i].height != v.d.H)
        return fail(STITCH_E_SHAPE, "%s is not canvas-sized", name);
      cams[i].direct = Img3{d_warped[i].data, d_warped[i].row_pitch / 4, d_warped[i].plane_pitch / 4, 0};
      cams[i].dom = Box{0, 0, v.d.W, v.d.H};
    }
    const hipStream_t s = (hipStream_t)stream;
    uint8_t* ws = (uint8_t*)workspace;
    auto D = [&](size_t o) { return (double*)(ws + o); };
    double* dr[kMaxLevels] = {};
    for (int k = 1; k < v.d.L; ++k) dr[k] = D(v.o_r[k]);
    const Img3 dr0{d_pano->data, d_pano->row_pitch / 4, d_pano->plane_pitch / 4, 0};
    hipLaunchKernelGGL(k_gzero, dim3(1), dim3(1), 0, s, D(v.o_flag));
    launch_dr(v.d, dr0, dr, s);
    st = dev_ok(hipGetLastError(), "backward launch");
    for (const VjpGroup& g : vjp_groups(v, ws, v.o_group, true, cams, pcs)) {
      if (st || (st = vjp_upload(g, s))) break;
      launch_pyramids<false>(v.d, g.cw, false, true, s);
      launch_adjoint<false>(v.d, g.cw, dr0, dr, d_frames + g.first, D(v.o_res) + 9 * g.first, (int*)(ws + v.o_flag), s);
      st = dev_ok(hipGetLastError(), "backward launch");
    }
    std::vector<double> res(9 * (size_t)v.n + 1, 0.0);
    if (!st) st = dev_ok(hipMemcpyAsync(res.data(), D(v.o_res), res.size() * 8, hipMemcpyDeviceToHost, s), "gradient copy");
    if (!st) st = dev_ok(hipStreamSynchronize(s), "backward synchronise");
    if (st) return st;
    int flag = 0;
    std::memcpy(&flag, &res[9 * (size_t)v.n], sizeof flag);
    if (flag)
      return fail(STITCH_E_UNSUPPORTED, "a map magnifies a source pixel beyond the gather's reach or crosses its "
                  "horizon inside a frame (flags %d); d_frames is incomplete", flag);
    for (size_t j = 0; j + 1 < res.size(); ++j) d_hinv[j] = res[j];
    return STITCH_OK;
  });
}

stitch_status stitch_corners_to_h(const double q[8], int32_t w, int32_t h, double H[9]) {
  if (!q || !H) return fail(STITCH_E_NULL, "q or H is NULL");
  if (w < 2 || h < 2) return fail(STITCH_E_SHAPE, "frame %dx%d", w, h);
  double A[64], hv[8];
  if (!dlt(q, w, h, A, hv)) return fail(STITCH_E_HOMOGRAPHY, "corners are degenerate");
  for (int i = 0; i < 8; ++i) H[i] = hv[i];
  H[8] = 1.0;
  return STITCH_OK;
}

stitch_status stitch_map_grad_to_corners(const double q[8], int32_t w, int32_t h, const double d_map[9],
                                         double d_q[8]) {
  if (!q || !d_map || !d_q) return fail(STITCH_E_NULL, "q, d_map or d_q is NULL");
  double A[64], hv[8];
  if (!dlt(q, w, h, A, hv)) return fail(STITCH_E_HOMOGRAPHY, "corners are degenerate");
  const double Hm[9] = {hv[0], hv[1], hv[2], hv[3], hv[4], hv[5], hv[6], hv[7], 1.0};
  double N[9];
  if (!inv3(Hm, N)) return fail(STITCH_E_HOMOGRAPHY, "H(q) is singular");
  // dl/dH_j = sum_m dl/dM_m dM_m/dH_j with M = N / N22, dN = -N dH N
  double dH[9];
  for (int j = 0; j < 9; ++j) {
    const int r = j / 3, c = j % 3;
    double dN[9];
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) dN[a * 3 + b] = -N[a * 3 + r] * N[c * 3 + b];
    double acc = 0.0;
    for (int m = 0; m < 9; ++m) acc += d_map[m] * (dN[m] / N[8] - N[m] * dN[8] / (N[8] * N[8]));
    dH[j] = acc;
  }
  // dh/dq_k = A^-1 (db/dq_k - dA/dq_k h) with h33 fixed to 1
  const double cx[4] = {0.0, (double)w - 1, (double)w - 1, 0.0}, cy[4] = {0.0, 0.0, (double)h - 1, (double)h - 1};
  for (int k = 0; k < 8; ++k) {
    const int corner = k / 2, row = k;   // q_k is X (k even) or Y (k odd) of corner k/2: equation row k
    double rhs[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    rhs[row] = 1.0 + cx[corner] * hv[6] + cy[corner] * hv[7];
    double dh[8];
    if (!solve8(A, rhs, dh)) return fail(STITCH_E_HOMOGRAPHY, "corner system is singular");
    double acc = 0.0;
    for (int i = 0; i < 8; ++i) acc += dH[i] * dh[i];
    d_q[k] = acc;
  }
  return STITCH_OK;
}

}  // extern "C"

