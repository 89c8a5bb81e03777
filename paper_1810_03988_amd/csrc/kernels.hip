// gfx950 kernels of the per-frame stitching path (wave64, LDS-tiled, no MFMA: nothing
// here is a dense contraction).  The warp pass is bound by vector arithmetic, the large blends and
// single stages by HBM traffic, small levels by latency; each kernel says which.
//
//   k_pyr    fused pyramid pass from level k to k+1 for many cameras at once.  A
//            64-column level-k tile is walked in 16-row sub-steps; each is staged in LDS
//            with a (4,3)-sample halo -- at level 0 it is produced by the homography warp
//            itself (Alg. 4, step 1), so G_0 never reaches HBM -- then REDUCE gives the
//            level-(k+1) tile with a one-sample halo,
//            EXPAND of that tile is subtracted from G_k to give L_k (multi-band fusion,
//            Sec. 1), and the seam-weight pyramid is reduced in the same pass.
//   k_blend  one level of the synthesis side (Alg. 4, step 6): B_k = sum_i Gm_i L_i and
//            R_k = B_k + EXPAND(R_{k+1}); level 0 writes the uint8 panorama.
//   k_tail, k_blend_tail: the small levels of either in one launch.
//   k_warp, k_warp_coords, k_expand_sub, k_level0: single-stage kernels behind the
//            stitch_warp / stitch_pyramid entry points (its REDUCEs run in k_tail).
//
// Borders: reflect-101 folded in the fine domain.  Staging the fine tile through the
// periodic reflect-101 extension makes the locally reduced coarse tile equal to the
// fine-domain-folded zero-inserted coarse signal, so EXPAND inside a tile needs no
// border cases at all.
#include <hip/hip_runtime.h>

#include <cstring>
#include <type_traits>

#include "kernarg.h"
#include "stitch_internal.h"

namespace stitch {
namespace {

constexpr float kW0 = 1.0f / 16.0f, kW1 = 4.0f / 16.0f, kW2 = 6.0f / 16.0f;
constexpr float kInv255 = 1.0f / 255.0f;

#define GLB __attribute__((address_space(1)))
#define CST __attribute__((address_space(4)))

// Descriptor tables are written by the host before a launch and never during it: read them
// through the constant address space, so uniform reads become scalar loads.
template <typename T>
__device__ __forceinline__ const CST T* cst(const T* p) { return (const CST T*)p; }
// A whole descriptor by value (dword copies, merged into wide scalar loads).
template <typename T>
__device__ __forceinline__ T ld_cst(const CST T* p) {
  static_assert(sizeof(T) % 4 == 0, "descriptors are dword multiples");
  T v;
  uint32_t* d = reinterpret_cast<uint32_t*>(&v);
  const CST uint32_t* s = reinterpret_cast<const CST uint32_t*>(p);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) d[i] = s[i];
  return v;
}

// Views of descriptor-held pointers as global memory, so accesses compile to global (not
// flat) instructions.
template <typename T>
__device__ __forceinline__ const GLB T* cg(const void* p) { return (const GLB T*)p; }
template <typename T>
__device__ __forceinline__ GLB T* mg(void* p) { return (GLB T*)p; }
__device__ __forceinline__ float ldg(const GLB float* p, int64_t i) { return p[i]; }
__device__ __forceinline__ float ldg(const GLB _Float16* p, int64_t i) { return (float)p[i]; }
__device__ __forceinline__ void stg(GLB float* p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void stg(GLB _Float16* p, int64_t i, float v) { p[i] = (_Float16)v; }

// Raw bits of a stored sample (zero-extended), converted separately: loads can then all be
// issued before the first conversion.
template <typename T> struct RawOf;
template <> struct RawOf<float> { using type = uint32_t; };
template <> struct RawOf<_Float16> { using type = uint16_t; };
template <typename T>
__device__ __forceinline__ typename RawOf<T>::type ld_raw(const GLB T* p, int64_t i) {
  return *(const GLB typename RawOf<T>::type*)(p + i);
}
__device__ __forceinline__ float from_raw(uint32_t b) { return __builtin_bit_cast(float, b); }
__device__ __forceinline__ float from_raw(uint16_t b) { return (float)__builtin_bit_cast(_Float16, b); }
typedef float vf4 __attribute__((ext_vector_type(4)));
typedef _Float16 vh4 __attribute__((ext_vector_type(4)));

// Streaming stores for the pyramid levels (written once, read by a later kernel long after
// the lines would have left L2); the four-sample forms need 4-sample alignment (checked by
// the caller).
__device__ __forceinline__ void stgnt(GLB float* p, int64_t i, float v) { __builtin_nontemporal_store(v, p + i); }
__device__ __forceinline__ void stgnt(GLB _Float16* p, int64_t i, float v) {
  __builtin_nontemporal_store((_Float16)v, p + i);
}
__device__ __forceinline__ void stg4nt(GLB float* p, const float v[4]) {
  __builtin_nontemporal_store(vf4{v[0], v[1], v[2], v[3]}, reinterpret_cast<GLB vf4*>(p));
}
__device__ __forceinline__ void stg4nt(GLB _Float16* p, const float v[4]) {
  __builtin_nontemporal_store(vh4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]},
                              reinterpret_cast<GLB vh4*>(p));
}

// Eight FP16 samples as one 16-byte streaming store: four dwords of packed halves (low
// half = lower column).
__device__ __forceinline__ uint32_t pack_h2(float a, float b) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)a) | ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)b) << 16);
}
__device__ __forceinline__ void stg8nt(GLB _Float16* p, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  typedef uint32_t vu4s __attribute__((ext_vector_type(4)));
  __builtin_nontemporal_store(vu4s{a, b, c, d}, reinterpret_cast<GLB vu4s*>(p));
}

// Periodic reflect-101 extension: index -> [0, n), n >= 2 (period 2(n-1)).
__device__ __forceinline__ int fold(int i, int n) {
  if (i >= 0 && i < n) return i;
  const int p = 2 * (n - 1);
  i %= p;
  if (i < 0) i += p;
  return i < n ? i : p - i;
}

// EXPAND at even samples, 1/8 (a + c) + 3/4 b with s = a + c: along rows first (exp_h), then down
// the columns (exp_v).  Every kernel that expands uses these two, whose roundings differ, so
// that all of them give the same bits.  (At odd samples 1/2 (a + b) has one rounding however
// it is formed; so do REDUCE's 1/16 and 1/4 terms.)
__device__ __forceinline__ float exp_h(float s, float b) { return __builtin_fmaf(0.75f, b, 0.125f * s); }
__device__ __forceinline__ float exp_v(float s, float b) { return __builtin_fmaf(0.125f, s, 0.75f * b); }

// REDUCE along one axis from its outer pair's sum, its inner pair's and the middle: one rounding each
// for the first two products together and for the third (k_pyr's rows take the same
// steps on 16 times the value).
__device__ __forceinline__ float reduce5(float outer, float inner, float mid) {
  return __builtin_fmaf(kW2, mid, __builtin_fmaf(kW1, inner, kW0 * outer));
}

// FP16 storage rounds a float to half; where that float is itself a multiply-add the compiler may
// round the exact sum to half at once (v_fma_mixlo_f16) or to float first, and the two differ
// about once in 10^7 samples.  Which of the two is part of a result that several kernels share,
// so it is written down: fma_half rounds once, settled(v) keeps v the float it is.
__device__ __forceinline__ float fma_half(float a, float b, float c) {
  _Float16 r;
  asm("v_fma_mixlo_f16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return (float)r;
}
__device__ __forceinline__ float settled(float v) {
  asm("" : "+v"(v));
  return v;
}
// Column `col` (0 .. 3 of an aligned four) of a band's odd row: g - s/2, s the sum of the two
// rows it lies between.
__device__ __forceinline__ float band_odd(float g, float s, int, float) { return __builtin_fmaf(-0.5f, s, g); }
__device__ __forceinline__ float band_odd(float g, float s, int col, _Float16) {
  return col < 2 ? fma_half(-0.5f, s, g) : settled(__builtin_fmaf(-0.5f, s, g));
}

// Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a contiguous
// run of logical tiles so neighbouring tiles (which share halos) share an L2.
__device__ __forceinline__ int xcd_remap(int b, int g) {
  const int q = g >> 3, r = g & 7, x = b & 7, i = b >> 3;
  return x * q + (x < r ? x : r) + i;
}

// FP32 canvas -> source coordinates: (h0*X + h1*Y) + h2 etc., every operation rounded
// on its own (no contraction into FMA), IEEE divide.
__device__ __forceinline__ void warp_coords(const float* __restrict__ h, int X, int Y, float& x, float& y,
                                            bool& zpos) {
#pragma clang fp contract(off)
  const float Xf = (float)X, Yf = (float)Y;
  const float u = (h[0] * Xf + h[1] * Yf) + h[2];
  const float v = (h[3] * Xf + h[4] * Yf) + h[5];
  const float z = (h[6] * Xf + h[7] * Yf) + h[8];
  zpos = z > 0.0f;
  x = u / z;
  y = v / z;
}

// The same sequence from canvas coordinates already held as (exact) floats.
__device__ __forceinline__ void warp_coords_f(const float* __restrict__ h, float Xf, float Yf, float& x, float& y,
                                              bool& zpos) {
#pragma clang fp contract(off)
  const float u = (h[0] * Xf + h[1] * Yf) + h[2];
  const float v = (h[3] * Xf + h[4] * Yf) + h[5];
  const float z = (h[6] * Xf + h[7] * Yf) + h[8];
  zpos = z > 0.0f;
  x = u / z;
  y = v / z;
}

// The same sequence, also returning z.
__device__ __forceinline__ void warp_coords_z(const float* __restrict__ h, float Xf, float Yf, float& x, float& y,
                                              float& z) {
#pragma clang fp contract(off)
  const float u = (h[0] * Xf + h[1] * Yf) + h[2];
  const float v = (h[3] * Xf + h[4] * Yf) + h[5];
  z = (h[6] * Xf + h[7] * Yf) + h[8];
  x = u / z;
  y = v / z;
}

// x = u/z and y = v/z, correctly rounded, for operands in the range where the hardware
// division sequence scales nothing and fixes nothing up: z in [2^-10, 2^20] and |u|, |v|
// in [2^-12, 2^44] (exponent gaps far below 96, no denormal reciprocal, numerator or
// quotient).  In that range the IEEE divide of the
// compiler is exactly: r = rcp(z) refined by one Newton step, q = u r, two residual
// corrections; the refined reciprocal is shared by both quotients.
__device__ __forceinline__ void div2_in_range(float u, float v, float z, float& x, float& y) {
  float r = __builtin_amdgcn_rcpf(z);
  r = __builtin_fmaf(__builtin_fmaf(-z, r, 1.0f), r, r);
  float qx = u * r, qy = v * r;
  qx = __builtin_fmaf(__builtin_fmaf(-z, qx, u), r, qx);
  qy = __builtin_fmaf(__builtin_fmaf(-z, qy, v), r, qy);
  x = __builtin_fmaf(__builtin_fmaf(-z, qx, u), r, qx);
  y = __builtin_fmaf(__builtin_fmaf(-z, qy, v), r, qy);
}

// Eight bytes at any byte address (global memory accepts unaligned dword accesses).
typedef unsigned long long __attribute__((aligned(1))) u64_unaligned;
__device__ __forceinline__ unsigned long long ld8(const GLB uint8_t* p) { return *(const GLB u64_unaligned*)p; }

// Bilinear sample of a uint8 HWC RGB frame at the preimage of canvas pixel (X, Y);
// taps outside the frame contribute 0.  Values in [0, 1].
__device__ __forceinline__ void warp_px(const uint8_t* __restrict__ src, int64_t row, int w, int h,
                                        const float* __restrict__ hv, int X, int Y, float out[3]) {
  float x, y;
  bool zpos;
  warp_coords(hv, X, Y, x, y, zpos);
  out[0] = out[1] = out[2] = 0.0f;
  if (!(zpos && x >= -1.0f && x < (float)w && y >= -1.0f && y < (float)h)) return;
  const float x0f = floorf(x), y0f = floorf(y);
  const float fx = x - x0f, fy = y - y0f;
  const int x0 = (int)x0f, y0 = (int)y0f;
  const bool xa = x0 >= 0, xb = x0 + 1 < w, ya = y0 >= 0, yb = y0 + 1 < h;
  const int xc0 = xa ? x0 : 0, xc1 = xb ? x0 + 1 : w - 1;
  const int yc0 = ya ? y0 : 0, yc1 = yb ? y0 + 1 : h - 1;
  const uint8_t* r0 = src + (int64_t)yc0 * row;
  const uint8_t* r1 = src + (int64_t)yc1 * row;
  const float gx = 1.0f - fx, gy = 1.0f - fy;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float p00 = (ya && xa) ? (float)r0[xc0 * 3 + c] : 0.0f;
    const float p01 = (ya && xb) ? (float)r0[xc1 * 3 + c] : 0.0f;
    const float p10 = (yb && xa) ? (float)r1[xc0 * 3 + c] : 0.0f;
    const float p11 = (yb && xb) ? (float)r1[xc1 * 3 + c] : 0.0f;
    out[c] = (gy * (gx * p00 + fx * p01) + fy * (gx * p10 + fx * p11)) * kInv255;
  }
}

__device__ __forceinline__ int find_item(const PyrItem* __restrict__ items, int nitems, int t) {
  int lo = 0, hi = nitems - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cst(items)[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// ------------------------------------------------------------------------------------
// Fused pyramid pass from level k to k+1 (256 threads, four waves per workgroup).
//
// A tile is 64 level-k columns by 16 * sub rows; the workgroup walks down it in sub-steps
// of 16 rows.  Persistent, XCD-aware schedule: the tiles are split into eight contiguous
// ranges, one per XCD (workgroup b runs on XCD b % 8), and the workgroups of an XCD stride
// through its range, so neighbouring tiles -- which share halos -- share that XCD's L2.
//
// Stages of one sub-step:
//   A  (whole workgroup, then a barrier) stage the 71-column window of the sub-step's 23
//      rows (its 16 rows plus 4 above and 3 below) of every channel in LDS: three image
//      channels (the bilinear warp of the source frame at level 0, the stored G_k above)
//      and the seam weight.  LDS rows form a ring of 23: the 7 rows a sub-step shares with
//      the previous one stay where they are, so only its 16 new rows are staged (all 23 on
//      a tile's first sub-step).  At level 0 the source rectangle under a source-interior
//      window is first read into LDS as aligned 16-byte chunks (one more barrier) and the
//      bilinear taps come from there;
//   B..E  (wave w alone on channel slot w, no workgroup barrier)
//      B+C  REDUCE -> extended 34x10 coarse tile (horizontal then vertical in registers,
//           then into the wave's LDS rows); its interior, G_{k+1} / Gm_{k+1}, is stored
//           from LDS with one 16-byte store per lane;
//      D+E  horizontal and vertical EXPAND of the coarse tile and L_k = G_k - EXPAND(G_{k+1}),
//           stored on the band window (image channels only).
struct PyrTile {
  int item, X0, Y0, nsub;
};

__device__ __forceinline__ PyrTile decode_tile(const PyrItem* __restrict__ items, int nitems, int t) {
  PyrTile d;
  d.item = find_item(items, nitems, t);
  const CST PyrItem& it = cst(items)[d.item];
  const int lt = t - it.tile_begin;
  const int tyi = lt / it.tiles_x, txi = lt - tyi * it.tiles_x;
  d.X0 = it.tile_x0 + txi * kPyrTX;
  d.Y0 = it.tile_y0 + tyi * (kPyrTY * it.sub);
  d.nsub = min(it.sub, it.rows16 - tyi * it.sub);
  return d;
}

template <int N>
struct Rows {
  static constexpr int value = N;
};

template <typename T, bool WARP>
__global__ void __launch_bounds__(kThreads, 4) k_pyr(const PyrItem* __restrict__ items, int nitems, int ntiles,
                                                     FrameArgs fa) {
  constexpr int TX = kPyrTX, TY = kPyrTY;
  constexpr int EW = TX + 7, EH = TY + 7;            // staged window: 4 before, 3 after
  constexpr int SW = 72;                             // LDS row strides are 16-byte multiples
  constexpr int CW = TX / 2 + 2, CH = TY / 2 + 2;    // coarse tile + one-sample halo
  // coarse tile of every channel: coarse column j at index j + 3, so the interior columns
  // 1 .. 32 start on a 16-byte boundary
  constexpr int HS = 40, CO = 3;
  __shared__ __attribute__((aligned(16))) float sIn[4][EH][SW];   // rows: ring
  __shared__ __attribute__((aligned(16))) float sC[4][CH][HS];
  // warp only: the rounded products h0 X, h3 X, h6 X of every staged column and h1 Y,
  // h4 Y, h7 Y of every window row, shared by the workgroup's samples
  constexpr int NCT = WARP ? EW : 1, NRT = WARP ? EH : 1;
  __shared__ __attribute__((aligned(16))) float sColT[NCT][4];
  __shared__ __attribute__((aligned(16))) float sRowT[NRT][4];
  // warp only: the class of every sub-step's 16-row window, classified together at the
  // tile's first sub-step (slot kMaxSub: the 7 rows that sub-step also stages)
  constexpr int kMaxSub = 8;
  __shared__ int sCls[kMaxSub + 1];
  // warp only: the source rectangle under a source-interior 16-row window, one 256-byte
  // LDS row per source row (read as aligned 16-byte chunks), and its origin
  constexpr int FH = 24, FWB = 256;
  static_assert(FWB == 256, "an LDS row of the source rectangle is 1 << 8 bytes");
  __shared__ __attribute__((aligned(16))) uint32_t sSrc[WARP ? FH : 1][FWB / 4];
  __shared__ int sBox[kMaxSub][4];   // per sub-step: bx0, by0, rows, 16-byte chunks per row
  constexpr uint32_t kPlaneRing = EH * SW * 4;       // bytes of one channel's ring of rows

  const int tid = threadIdx.x;
  // ---- schedule ----
  const int G = gridDim.x, b = blockIdx.x;
  int t, t_end, stride;
  if (G >= 8) {
    const int xcd = b & 7, rank = b >> 3;
    const int q = ntiles >> 3, r = ntiles & 7;
    const int t0 = xcd * q + min(xcd, r);
    t = t0 + rank;
    t_end = t0 + q + (xcd < r ? 1 : 0);
    stride = (G - xcd + 7) >> 3;
  } else {
    t = b;
    t_end = ntiles;
    stride = G;
  }

  for (; t < t_end; t += stride) {
    const PyrTile d = decode_tile(items, nitems, t);
    const CST PyrItem& it = cst(items)[d.item];
    const int X0 = d.X0;
    const int fw = it.fine_w, fh = it.fine_h;
    const int rx = it.roi_x, ry = it.roi_y, rw = it.roi_w, rh = it.roi_h;

    for (int s = 0; s < d.nsub; ++s) {
      const int Y0 = d.Y0 + s * TY;
      const int off = (s * TY) % EH;   // logical row r of the window lives in ring row (r + off) mod EH
      const uint32_t off4 = (uint32_t)off * (SW * 4);
      const bool interior = X0 >= 4 && X0 + TX + 3 <= fw && Y0 >= 4 && Y0 + TY + 3 <= fh;
      // stored levels of an interior window can be staged as aligned 16-byte chunks (above
      // level 0; see stage A)
      constexpr int kChunk = 16 / (int)sizeof(T);
      const bool chunked = !WARP && interior && rw > 0 && rh > 0 && ((X0 - rx) % kChunk) == 0 &&
                           ((uintptr_t)it.img & 15) == 0 && (it.img_row % kChunk) == 0 &&
                           (it.img_plane % kChunk) == 0 && ((uintptr_t)it.msk & 15) == 0 && (it.msk_row % kChunk) == 0;
      if (WARP) {
        // the coordinate tables (the columns once per tile, the rows per sub-step); their
        // last readers (the previous sub-step's stage A) finished before its closing barrier
        if (tid < EW) {
          if (s == 0) {
            const float Xf = (float)(X0 - 4 + tid);
            const float4 c = {it.hinv[0] * Xf, it.hinv[3] * Xf, it.hinv[6] * Xf, 0.0f};
            *reinterpret_cast<float4*>(sColT[tid]) = c;
          }
        } else if (tid >= 128 && tid < 128 + EH) {
          const float Yf = (float)(Y0 - 4 + (tid - 128));
          const float4 r = {it.hinv[1] * Yf, it.hinv[4] * Yf, it.hinv[7] * Yf, 0.0f};
          *reinterpret_cast<float4*>(sRowT[tid - 128]) = r;
        } else if (tid >= 192 && s == 0) {
          // Window classes of every sub-step of the tile, once per tile (wave 3; lanes
          // 8 u .. 8 u + 3: the corners of sub-step u's 16 new rows, lanes 4-7: of the 7
          // rows the first sub-step also stages).
          // Source-interior (bit 0): z > 0 at the four corners (so on all of the window: z
          // is affine) and their source positions inside [1, w-3) x [1, h-2).  The map is
          // projective there, so every staged sample lies in the convex hull of the corner
          // images (up to FP32 rounding, far below the one-sample margin): its four taps
          // are in the frame and the pair of taps of a row is one 8-byte read that ends
          // inside the row.  Source-exterior (bit 1): z > 0 at the corners and all four
          // corner images at least one sample beyond the same side of the frame (x <= -2,
          // x >= w + 1, y <= -2 or y >= h + 1): every staged sample's taps are outside,
          // its G_0 is 0.  Either also needs the window inside the canvas (checked by the
          // stage).
          const int lane = tid - 192, u = lane >> 3, j = lane & 7;
          const int nsc = min(d.nsub, kMaxSub);
          bool bad = false, zok = false, lft = false, rgt = false, top = false, bot = false;
          float xc = 0.0f, yc = 0.0f;
          const int w = it.frame_w, h = it.frame_h;
          if (u < nsc && (j < 4 || u == 0)) {
            float hv[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) hv[i] = it.hinv[i];
            const int r0 = j < 4 ? EH - TY : 0, r1 = j < 4 ? EH - 1 : EH - TY - 1;
            float zc;
            warp_coords_z(hv, (float)(X0 - 4 + ((j & 1) ? EW - 1 : 0)),
                          (float)(d.Y0 + u * TY - 4 + ((j & 2) ? r1 : r0)), xc, yc, zc);
            zok = zc >= 0x1p-10f && zc <= 0x1p20f;
            bad = !(zok && xc >= 1.0f && xc < (float)(w - 3) && yc >= 1.0f && yc < (float)(h - 2));
            lft = xc <= -2.0f;
            rgt = xc >= (float)(w + 1);
            top = yc <= -2.0f;
            bot = yc >= (float)(h + 1);
          }
          const uint64_t mb = __ballot(bad), mz = __ballot(zok), ml = __ballot(lft), mr = __ballot(rgt),
                         mt = __ballot(top), mo = __ballot(bot);
          // bounding box of each group of four corner images
          float mnx = xc, mxx = xc, mny = yc, mxy = yc;
#pragma unroll
          for (int dd = 1; dd < 4; dd <<= 1) {
            mnx = fminf(mnx, __shfl_xor(mnx, dd));
            mxx = fmaxf(mxx, __shfl_xor(mxx, dd));
            mny = fminf(mny, __shfl_xor(mny, dd));
            mxy = fmaxf(mxy, __shfl_xor(mxy, dd));
          }
          if (u < nsc && (j == 0 || (j == 4 && u == 0))) {
            const int sh = lane;
            auto all4 = [sh](uint64_t m) { return ((m >> sh) & 15ull) == 15ull; };
            const bool fast = ((mb >> sh) & 15ull) == 0ull;
            const bool outside = all4(mz) && (all4(ml) || all4(mr) || all4(mt) || all4(mo));
            // Staged (bit 2, 16-row windows only): every tap lies in the box [bx0, bx1] x
            // [by0, by1] (the corner images' bounding box, one sample wider on each side
            // for rounding), which fits the LDS rows, and the 16-byte chunks covering a
            // box row (from its start rounded down to 16 bytes, at most 15 + 3 nbx + 15
            // bytes) stay inside the frame row: bx0 >= 5 and bx1 <= w - 11.  The row
            // pitch is a multiple of 16 bytes, so every box row starts at the same offset
            // in its LDS row.
            bool staged = false;
            const int64_t srow = fa.n ? fa.row[it.frame_slot] : it.img_row;
            if (j == 0 && fast && (srow & 15) == 0) {
              const int bx0 = (int)floorf(mnx) - 1, bx1 = (int)floorf(mxx) + 2;
              const int by0 = (int)floorf(mny) - 1, by1 = (int)floorf(mxy) + 2;
              const int nbx = bx1 - bx0 + 1, nby = by1 - by0 + 1;
              staged = bx0 >= 5 && bx1 <= w - 11 && by0 >= 0 && by1 <= h - 1 && 15 + 3 * nbx <= FWB && nby <= FH;
              if (staged) {
                sBox[u][0] = bx0;
                sBox[u][1] = by0;
                sBox[u][2] = nby;
                sBox[u][3] = (15 + 3 * nbx + 15) / 16;
              }
            }
            sCls[j == 0 ? u : kMaxSub] = (fast ? 1 : 0) | (outside ? 2 : 0) | (staged ? 4 : 0);
          }
        }
      }
      __syncthreads();   // the previous sub-step's readers of LDS are done

      // ---- A: stage logical rows R0 .. R0+NR-1 ----
      auto stage_a = [&](auto rows_c, auto r0_c) __attribute__((always_inline)) {
        constexpr int NR = decltype(rows_c)::value;
        constexpr int R0 = decltype(r0_c)::value;
        // Slots.  Level 0: a lane keeps one of the window's first 64 columns and its wave takes
        // every fourth row, so rows, their ring offsets and their tabled products are the wave's
        // own; the remaining 7 columns of every row are one last round.  (One numbering of
        // all samples cost divisions and per-lane row addresses: the pass of 8 jobs at 640 to 3840
        // columns, FP16, took 174 million instructions and 409 us; with B's shorter rows 144
        // million and 385 us; 379 since no sample asks whether its source is there.)  Above
        // it, samples are numbered through.
        constexpr int NE = NR * EW;
        constexpr int NM = (NR + 3) / 4;
        constexpr int NQ = WARP ? NM + 1 : (NE + kThreads - 1) / kThreads;
        // recomputed per sub-step (cheap) rather than held in registers across the loop
        int tid_l = tid;
        asm volatile("" : "+v"(tid_l));
        const int wvu = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
        int rr[NQ], cc[NQ];                       // logical row (-1: idle slot) and column
        uint32_t row4[NQ], col4[NQ];              // byte offsets of the slot in a channel's rows, unrotated
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          if (WARP && q < NM) {
            rr[q] = R0 + wvu + 4 * q;
            cc[q] = tid_l & 63;
          } else {
            const int e = WARP ? tid_l : tid_l + q * kThreads;
            constexpr int W = WARP ? EW - 64 : EW;
            rr[q] = e < NR * W ? R0 + e / W : -1;
            cc[q] = e < NR * W ? EW - W + e % W : 0;
          }
          // idle slots write the padding column EW (read by stage B's last float4 but never
          // used), so stores need no branch and loads are never sunk into one
          row4[q] = (uint32_t)((rr[q] < 0 ? R0 : rr[q]) * SW) * 4u;
          col4[q] = (uint32_t)(rr[q] < 0 ? EW : cc[q]) * 4u;
        }
        // A round that is idle for whole waves (the 16-row stage's last one: the waves of threads
        // 128 .. 255) is skipped by them.
        auto live = [&](int q) {
          if (WARP) return q < NM ? NR % 4 == 0 || wvu + 4 * q < NR : wvu * 64 < NR * (EW - 64);
          return q < NQ - 1 || NE % kThreads == 0 || wvu * 64 + (NQ - 1) * kThreads < NE;
        };
        // the slot's cell in channel plane ch, rotated into the ring
        auto cell = [&](int ch, int q) -> float& {
          const uint32_t a = row4[q] + off4;
          return *reinterpret_cast<float*>(reinterpret_cast<char*>(&sIn[ch][0][0]) + (min(a, a - kPlaneRing) + col4[q]));
        };
        // canvas position of a slot (idle slots take the window's first sample)
        auto canvas = [&](int q, int& X, int& Y) {
          X = X0 - 4 + cc[q];
          Y = Y0 - 4 + (rr[q] < 0 ? R0 : rr[q]);
          if (!interior) {
            X = fold(X, fw);
            Y = fold(Y, fh);
          }
        };
        if (WARP) {
          const GLB uint8_t* src = cg<uint8_t>(fa.n ? (const void*)fa.ptr[it.frame_slot] : it.img);
          const int64_t srow = fa.n ? fa.row[it.frame_slot] : it.img_row;
          const int w = it.frame_w, h = it.frame_h;
          float hv[9];
#pragma unroll
          for (int i = 0; i < 9; ++i) hv[i] = it.hinv[i];
          const uint32_t srow32 = (uint32_t)srow;
          // seam weights (uint8 on the ROI, 0 outside): read first, used last
          const GLB uint8_t* msk = cg<uint8_t>(it.msk);
          uint32_t mv[NQ];
          const bool inside = interior && X0 - 4 >= rx && X0 + TX + 3 <= rx + rw && Y0 - 4 + R0 >= ry &&
                              Y0 - 4 + R0 + NR <= ry + rh;
          if (inside) {
            const GLB uint8_t* m0 = msk + (int64_t)(Y0 - 4 + R0 - ry) * it.msk_row + (X0 - 4 - rx);
            const uint32_t mrow = (uint32_t)it.msk_row;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
              if (live(q)) mv[q] = m0[__umul24((uint32_t)(rr[q] < 0 ? 0 : rr[q] - R0), mrow) + (uint32_t)cc[q]];
          } else {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              if (!live(q)) continue;
              int X, Y;
              canvas(q, X, Y);
              const int my = Y - ry, mx = X - rx;
              const bool in = my >= 0 && my < rh && mx >= 0 && mx < rw;
              const uint32_t m = msk[in ? (int64_t)my * it.msk_row + mx : 0];
              mv[q] = in ? m : 0u;
            }
          }
          const float fwf = (float)w, fhf = (float)h, fwm1 = (float)(w - 1), fhm1 = (float)(h - 1);
          // the window's class, computed before the sub-step's barrier
          const int cls = !interior ? 0 : R0 == 0 ? sCls[kMaxSub] : s < kMaxSub ? sCls[s] : 0;
          const bool fast = (cls & 1) != 0, outside = (cls & 2) != 0;
          if (outside) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              if (!live(q)) continue;
              cell(0, q) = 0.0f;
              cell(1, q) = 0.0f;
              cell(2, q) = 0.0f;
              cell(3, q) = (float)mv[q] * kInv255;
            }
          } else if (fast && (cls & 4) != 0) {
            // Source rectangle staged in LDS: its rows are read as aligned 16-byte chunks
            // (the reads of the whole workgroup cover it once), each sample's coordinates
            // are computed meanwhile, and its two 8-byte tap pairs come from LDS.
            const int bx0 = sBox[s][0], by0 = sBox[s][1], nby = sBox[s][2], nck = sBox[s][3];
            constexpr int NCK = (FH * (FWB / 16) + kThreads - 1) / kThreads;
            typedef uint32_t vu4 __attribute__((ext_vector_type(4)));
            vu4 ck[NCK];
#pragma unroll
            for (int k = 0; k < NCK; ++k) {
              // spare lanes repeat a chunk of the box (the same bytes to the same place)
              const int e = tid + k * kThreads, r = min(e / (FWB / 16), nby - 1), c = min(e % (FWB / 16), nck - 1);
              const uintptr_t a = ((uintptr_t)src + __umul24((uint32_t)(by0 + r), srow32) + 3u * (uint32_t)bx0) & ~(uintptr_t)15;
              ck[k] = *reinterpret_cast<const GLB vu4*>(a + 16u * (uint32_t)c);
            }
            // every box row starts in its LDS row at byte (frame address of the box row) mod 16
            const uint32_t s1 = ((uint32_t)(uintptr_t)src + 3u * (uint32_t)bx0) & 15u;
            float fxq[NQ], fyq[NQ];
            uint32_t o1[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              if (!live(q)) continue;
              // the coordinate sequence from the tabled products (the same roundings as
              // the direct one; the in-range division is the IEEE one)
              const float4 ct = *reinterpret_cast<const float4*>(sColT[cc[q]]);
              const float4 rt = *reinterpret_cast<const float4*>(sRowT[rr[q] < 0 ? R0 : rr[q]]);
              float u, v, z, x, y;
              {
#pragma clang fp contract(off)
                u = (ct.x + rt.x) + hv[2];
                v = (ct.y + rt.y) + hv[5];
                z = (ct.z + rt.z) + hv[8];
              }
              div2_in_range(u, v, z, x, y);
              fxq[q] = __builtin_amdgcn_fractf(x);
              fyq[q] = __builtin_amdgcn_fractf(y);
              const uint32_t xi = (uint32_t)(int)x, yi = (uint32_t)(int)y;
              // 24-bit multiplies (full rate): the box is under 256 samples wide and 24 rows
              const uint32_t r = yi - (uint32_t)by0, dx = __umul24(xi - (uint32_t)bx0, 3u);
              o1[q] = (r << 8) + s1 + dx;
            }
#pragma unroll
            for (int k = 0; k < NCK; ++k) {
              const int e = tid + k * kThreads, r = min(e / (FWB / 16), nby - 1), c = min(e % (FWB / 16), nck - 1);
              *reinterpret_cast<vu4*>(&sSrc[r][4 * c]) = ck[k];
            }
            __syncthreads();
            const uint8_t* sb = reinterpret_cast<const uint8_t*>(&sSrc[0][0]);
            auto ld8s = [&](uint32_t o) -> unsigned long long {
              const uint32_t* d = reinterpret_cast<const uint32_t*>(sb + (o & ~3u));
              const uint32_t w0 = d[0], w1 = d[1], w2 = d[2];
              const uint32_t lo = __builtin_amdgcn_alignbyte(w1, w0, o & 3u);
              const uint32_t hi = __builtin_amdgcn_alignbyte(w2, w1, o & 3u);
              return (unsigned long long)lo | ((unsigned long long)hi << 32);
            };
            // every sample's tap reads first, then the bilinear combination
            unsigned long long ras[NQ], rbs[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              if (!live(q)) continue;
              ras[q] = ld8s(o1[q]);
              rbs[q] = ld8s(o1[q] + FWB);
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              if (!live(q)) continue;
              const unsigned long long ra = ras[q], rb = rbs[q];
              const float fx = fxq[q], fy = fyq[q], gx = 1.0f - fx, gy = 1.0f - fy;
              const float gyi = gy * kInv255, fyi = fy * kInv255;
              const float w00 = gyi * gx, w01 = gyi * fx, w10 = fyi * gx, w11 = fyi * fx;
              const uint32_t a0 = (uint32_t)ra, a1 = (uint32_t)(ra >> 32);
              const uint32_t b0 = (uint32_t)rb, b1 = (uint32_t)(rb >> 32);
              const float p00[3] = {(float)(a0 & 255u), (float)((a0 >> 8) & 255u), (float)((a0 >> 16) & 255u)};
              const float p01[3] = {(float)(a0 >> 24), (float)(a1 & 255u), (float)((a1 >> 8) & 255u)};
              const float p10[3] = {(float)(b0 & 255u), (float)((b0 >> 8) & 255u), (float)((b0 >> 16) & 255u)};
              const float p11[3] = {(float)(b0 >> 24), (float)(b1 & 255u), (float)((b1 >> 8) & 255u)};
#pragma unroll
              for (int ch = 0; ch < 3; ++ch)
                cell(ch, q) = w00 * p00[ch] + w01 * p01[ch] + w10 * p10[ch] + w11 * p11[ch];
              cell(3, q) = (float)mv[q] * kInv255;
            }
          } else if (fast) {
            // every sample: coordinates and both row reads issued first, so a wave keeps
            // 2 * NQ reads in flight; then the bilinear combination
            unsigned long long ra[NQ], rb[NQ];
            float fxq[NQ], fyq[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              if (!live(q)) continue;
              // z lies between its corner values and x, y in [1, w) x [1, h): the in-range
              // division is the IEEE one, x - floor(x) is exact and truncation is floor
              // the coordinate sequence from the tabled products (the same roundings)
              const float4 ct = *reinterpret_cast<const float4*>(sColT[cc[q]]);
              const float4 rt = *reinterpret_cast<const float4*>(sRowT[rr[q] < 0 ? R0 : rr[q]]);
              float u, v, z, x, y;
              {
#pragma clang fp contract(off)
                u = (ct.x + rt.x) + hv[2];
                v = (ct.y + rt.y) + hv[5];
                z = (ct.z + rt.z) + hv[8];
              }
              div2_in_range(u, v, z, x, y);
              fxq[q] = __builtin_amdgcn_fractf(x);
              fyq[q] = __builtin_amdgcn_fractf(y);
              const uint32_t o = __umul24((uint32_t)(int)y, srow32) + __umul24((uint32_t)(int)x, 3u);
              ra[q] = ld8(src + o);
              rb[q] = ld8(src + (o + srow32));
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              if (!live(q)) continue;
              const float fx = fxq[q], fy = fyq[q], gx = 1.0f - fx, gy = 1.0f - fy;
              const float gyi = gy * kInv255, fyi = fy * kInv255;
              const float w00 = gyi * gx, w01 = gyi * fx, w10 = fyi * gx, w11 = fyi * fx;
              const uint32_t a0 = (uint32_t)ra[q], a1 = (uint32_t)(ra[q] >> 32);
              const uint32_t b0 = (uint32_t)rb[q], b1 = (uint32_t)(rb[q] >> 32);
              const float p00[3] = {(float)(a0 & 255u), (float)((a0 >> 8) & 255u), (float)((a0 >> 16) & 255u)};
              const float p01[3] = {(float)(a0 >> 24), (float)(a1 & 255u), (float)((a1 >> 8) & 255u)};
              const float p10[3] = {(float)(b0 & 255u), (float)((b0 >> 8) & 255u), (float)((b0 >> 16) & 255u)};
              const float p11[3] = {(float)(b0 >> 24), (float)(b1 & 255u), (float)((b1 >> 8) & 255u)};
#pragma unroll
              for (int ch = 0; ch < 3; ++ch)
                cell(ch, q) = w00 * p00[ch] + w01 * p01[ch] + w10 * p10[ch] + w11 * p11[ch];
              cell(3, q) = (float)mv[q] * kInv255;
            }
          } else {
            // General window (frame borders, canvas edges): taps outside the frame weigh
            // 0.  Each row pair is still one 8-byte read, from a start clamped into
            // [0, 3w - 8] of a row clamped into the frame (w >= 3), so no read leaves its
            // row; the pair is shifted into place afterwards.
            unsigned long long ra[NQ], rb[NQ];
            float fxq[NQ], fyq[NQ];
            uint32_t tapq[NQ];                   // bits: 00 01 10 11 inside, << 4: byte shift + 3
            const uint32_t lastc = 3u * (uint32_t)w - 8u;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              if (!live(q)) continue;
              int Xc, Yc;
              canvas(q, Xc, Yc);
              float x, y;
              bool zpos;
              warp_coords_f(hv, (float)Xc, (float)Yc, x, y, zpos);
              const bool ok = zpos && x >= -1.0f && x < fwf && y >= -1.0f && y < fhf;
              const float xs = ok ? x : 0.0f, ys = ok ? y : 0.0f;
              const float x0f = floorf(xs), y0f = floorf(ys);
              fxq[q] = xs - x0f;
              fyq[q] = ys - y0f;
              const bool xa = ok && x0f >= 0.0f, xb = ok && x0f < fwm1, ya = y0f >= 0.0f, yb = y0f < fhm1;
              const int x0 = (int)x0f, y0 = (int)y0f;              // x0 >= -1, y0 >= -1
              const int c3 = 3 * x0;
              const uint32_t start = (uint32_t)min(max(c3, 0), (int)lastc);
              const uint32_t r0 = (uint32_t)max(y0, 0), r1 = (uint32_t)min(y0 + 1, h - 1);
              tapq[q] = (uint32_t)(ya && xa) | ((uint32_t)(ya && xb) << 1) | ((uint32_t)(yb && xa) << 2) |
                        ((uint32_t)(yb && xb) << 3) | ((uint32_t)(c3 - (int)start + 3) << 4);
              ra[q] = ld8(src + (__umul24(r0, srow32) + start));
              rb[q] = ld8(src + (__umul24(r1, srow32) + start));
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              if (!live(q)) continue;
              const int sh = (int)(tapq[q] >> 4) - 3;              // byte offset of tap 0: -3 .. 5
              const unsigned long long a = sh >= 0 ? ra[q] >> (8 * sh) : ra[q] << 24;
              const unsigned long long bq = sh >= 0 ? rb[q] >> (8 * sh) : rb[q] << 24;
              const float fx = fxq[q], fy = fyq[q], gx = 1.0f - fx, gy = 1.0f - fy;
              const float gyi = gy * kInv255, fyi = fy * kInv255;
              const uint32_t tp = tapq[q];
              const float w00 = (tp & 1u) ? gyi * gx : 0.0f, w01 = (tp & 2u) ? gyi * fx : 0.0f;
              const float w10 = (tp & 4u) ? fyi * gx : 0.0f, w11 = (tp & 8u) ? fyi * fx : 0.0f;
              const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
              const uint32_t b0 = (uint32_t)bq, b1 = (uint32_t)(bq >> 32);
              const float p00[3] = {(float)(a0 & 255u), (float)((a0 >> 8) & 255u), (float)((a0 >> 16) & 255u)};
              const float p01[3] = {(float)(a0 >> 24), (float)(a1 & 255u), (float)((a1 >> 8) & 255u)};
              const float p10[3] = {(float)(b0 & 255u), (float)((b0 >> 8) & 255u), (float)((b0 >> 16) & 255u)};
              const float p11[3] = {(float)(b0 >> 24), (float)(b1 & 255u), (float)((b1 >> 8) & 255u)};
#pragma unroll
              for (int ch = 0; ch < 3; ++ch)
                cell(ch, q) = w00 * p00[ch] + w01 * p01[ch] + w10 * p10[ch] + w11 * p11[ch];
              cell(3, q) = (float)mv[q] * kInv255;
            }
          }
        } else if (chunked) {
          // Stored G_k planes and Gm_k on the ROI (0 outside) as aligned 16-byte chunks of C
          // samples: window row r of channel slot c is chunks k = 0 .. NCH-1 of plane row
          // Y0 - 4 + R0 + r - ry from plane column X0 - C - rx + C k (the tile's X0 - rx, the
          // row pitches and plane strides are multiples of C, the planes start on 16-byte
          // boundaries, and a row's pitch covers its width rounded up to C).  Every read is
          // issued, without a branch, from a chunk clamped into the plane (its row into
          // [0, rh), its column into the rounded width); samples outside the ROI, the
          // channel set or the window are dropped afterwards.
          constexpr int C = 16 / (int)sizeof(T);
          constexpr int NCH = 64 / C + 2;
          constexpr int NT = NR * 4 * NCH;
          constexpr int NQC = (NT + kThreads - 1) / kThreads;
          typedef uint32_t vu4c __attribute__((ext_vector_type(4)));
          const int rwc = (rw + C - 1) / C;
          const int k0 = (X0 - C - rx) / C;   // plane chunk of k = 0
          // the descriptor's fields once, as scalars (a per-lane choice between two fields
          // would read them per lane and wait for each)
          const GLB T* const gimg = cg<T>(it.img);
          const GLB T* const gmsk = cg<T>(it.msk);
          const uint32_t iplane = (uint32_t)it.img_plane, irow = (uint32_t)it.img_row, mrow = (uint32_t)it.msk_row;
          uint32_t raw[NQC][4];   // plain dwords: an array of 4-vectors lost its upper elements at NQC = 5
#pragma unroll
          for (int q = 0; q < NQC; ++q) {
            const int e = min(tid_l + q * kThreads, NT - 1);
            const int k = e % NCH, rest = e / NCH, slot = rest & 3, r = rest >> 2;
            const GLB T* base = slot < 3 ? gimg + (uint32_t)slot * iplane : gmsk;
            const uint32_t pitch = slot < 3 ? irow : mrow;
            const int prow = min(max(Y0 - 4 + R0 + r - ry, 0), rh - 1);
            const int pck = min(max(k0 + k, 0), rwc - 1);
            const vu4c t = *reinterpret_cast<const GLB vu4c*>(base + (__umul24((uint32_t)prow, pitch) + (uint32_t)(C * pck)));
            raw[q][0] = t.x;
            raw[q][1] = t.y;
            raw[q][2] = t.z;
            raw[q][3] = t.w;
          }
#pragma unroll
          for (int q = 0; q < NQC; ++q) {
            const int e = tid_l + q * kThreads;
            if (e >= NT) continue;
            const int k = e % NCH, rest = e / NCH, slot = rest & 3, r = rest >> 2;
            const int prow = Y0 - 4 + R0 + r - ry, c0 = C * (k0 + k);
            const bool ok = prow >= 0 && prow < rh;
            const int keep = ok ? min(max(rw - c0, 0), (c0 < 0 ? 0 : C)) : 0;   // leading samples kept
            float v[C];
#pragma unroll
            for (int i = 0; i < C; ++i) {
              const float smp = sizeof(T) == 4 ? __builtin_bit_cast(float, raw[q][i & 3])
                                               : from_raw((uint16_t)(raw[q][i >> 1] >> (16 * (i & 1))));
              v[i] = i < keep ? smp : 0.0f;
            }
            // window column of v[0], a multiple of 4; only columns 0 .. SW-1 exist
            const int wc = C * k - C + 4;
            const uint32_t a0 = (uint32_t)((R0 + r) * SW) * 4u + off4;
            char* rowb = reinterpret_cast<char*>(&sIn[slot][0][0]) + min(a0, a0 - kPlaneRing);
#pragma unroll
            for (int h = 0; h < C / 4; ++h) {
              const int col = wc + 4 * h;
              if (col >= 0 && col < SW)
                *reinterpret_cast<float4*>(rowb + 4 * col) = float4{v[4 * h], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3]};
            }
          }
        } else {
          // stored G_k planes and Gm_k on the ROI (0 outside): every read is issued first, as
          // raw bits from an address inside the planes (offset 0 outside the ROI); conversion and
          // zeroing come afterwards
          const GLB T* g = cg<T>(it.img);
          const GLB T* m = cg<T>(it.msk);
          const uint32_t grow = (uint32_t)it.img_row, gplane = (uint32_t)it.img_plane, mrow = (uint32_t)it.msk_row;
          typename RawOf<T>::type raw[NQ][4];
          bool inq[NQ];
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            if (!live(q)) continue;
            int X, Y;
            canvas(q, X, Y);
            Y -= ry;
            X -= rx;
            inq[q] = X >= 0 && X < rw && Y >= 0 && Y < rh;
            const uint32_t og = inq[q] ? __umul24((uint32_t)Y, grow) + (uint32_t)X : 0u;
            const uint32_t om = inq[q] ? __umul24((uint32_t)Y, mrow) + (uint32_t)X : 0u;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) raw[q][ch] = ld_raw(g, (uint32_t)ch * gplane + og);
            raw[q][3] = ld_raw(m, om);
          }
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            if (!live(q)) continue;
#pragma unroll
            for (int ch = 0; ch < 4; ++ch) cell(ch, q) = inq[q] ? from_raw(raw[q][ch]) : 0.0f;
          }
        }
      };
      // a tile's first sub-step also stages the 7 rows the ring would otherwise carry over
      if (s == 0) stage_a(Rows<EH - TY>(), Rows<0>());
      stage_a(Rows<TY>(), Rows<EH - TY>());
      __syncthreads();

      // ---- B..E: wave w works on channel slot w alone, and exchanges data only through
      //      its own LDS rows (sC[ch]), so the next workgroup barrier is the next sub-step's ----
      const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
      const int lane = tid & 63;
      // The mask (whose wave has no D+E) goes to wave s & 1: a
      // workgroup's waves run on the compute unit's four SIMDs one each, and waves 0 and 1
      // also took stage A's last, partial round of samples, so every SIMD gets about the
      // same arithmetic per two sub-steps.
      const int mw = s & 1;
      const int ch = wv == mw ? 3 : wv - (wv > mw ? 1 : 0);
      // logical row r of the channel's ring (byte offsets keep the arithmetic 32-bit)
      const char* plane = reinterpret_cast<const char*>(&sIn[ch][0][0]);
      auto rowp = [&](int r) -> const float* {
        const uint32_t a = (uint32_t)r * (SW * 4) + off4;
        return reinterpret_cast<const float*>(plane + min(a, a - kPlaneRing));
      };
      // B+C: REDUCE -> extended coarse tile (CH x CW with a one-sample halo) in sC[ch].
      // Lane (g, jp), g < 3: coarse columns 2jp, 2jp+1 of NG coarse rows from F + 3g on, from the
      // 2 NG + 3 fine rows they need, each reduced horizontally from two b128 reads.  A tile's
      // first sub-step makes rows 0 .. 9 (NG = 4; rows 3 and 6 are written by the group that
      // starts there); the others keep the last two of the sub-step before as rows 0 and 1 and
      // make the remaining eight (NG = 3; the last group's third is past them).  Rows are
      // reduced to 16 times their value -- the same roundings, one product less -- and the
      // columns' weights take the 16 back.
      auto reduce = [&](auto ng_c, auto first_c) __attribute__((always_inline)) {
        constexpr int NG = decltype(ng_c)::value, F = decltype(first_c)::value;
        if (lane < 3 * (CW / 2)) {
          const int g = lane / (CW / 2), jp = lane - (CW / 2) * g, rs = F + 3 * g;
          float2 hr[2 * NG + 3];
#pragma unroll
          for (int u = 0; u < 2 * NG + 3; ++u) {
            // (the last group's last rows are past the window: any row will do)
            const float* row = rowp(2 * (F + 6) + u < EH ? 2 * rs + u : min(2 * rs + u, EH - 1)) + 4 * jp;
            const float4 a = *reinterpret_cast<const float4*>(row);
            const float4 bq = *reinterpret_cast<const float4*>(row + 4);
            hr[u].x = __builtin_fmaf(6.0f, a.z, __builtin_fmaf(4.0f, a.y + a.w, a.x + bq.x));
            hr[u].y = __builtin_fmaf(6.0f, bq.x, __builtin_fmaf(4.0f, a.w + bq.y, a.z + bq.z));
          }
          constexpr float V0 = kW0 / 16.0f, V1 = kW1 / 16.0f, V2 = kW2 / 16.0f;
#pragma unroll
          for (int m = 0; m < NG; ++m) {
            if (NG == 4 ? m == 0 && g > 0 : m == 2 && g == 2) continue;
            float* c = &sC[ch][rs + m][CO + 2 * jp];
            c[0] = __builtin_fmaf(V2, hr[2 * m + 2].x, __builtin_fmaf(V1, hr[2 * m + 1].x + hr[2 * m + 3].x,
                                                                      V0 * (hr[2 * m].x + hr[2 * m + 4].x)));
            c[1] = __builtin_fmaf(V2, hr[2 * m + 2].y, __builtin_fmaf(V1, hr[2 * m + 1].y + hr[2 * m + 3].y,
                                                                      V0 * (hr[2 * m].y + hr[2 * m + 4].y)));
          }
        }
      };
      if (s == 0) {
        reduce(Rows<4>(), Rows<0>());
      } else {
        if (lane < CW) {
          const float c0 = sC[ch][CH - 2][CO + lane], c1 = sC[ch][CH - 1][CO + lane];
          sC[ch][0][CO + lane] = c0;
          sC[ch][1][CO + lane] = c1;
        }
        reduce(Rows<3>(), Rows<2>());
      }
      // the wave's own sC[ch] rows: LDS accesses of one wave complete in order
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // the interior (8 x 32) is G_{k+1} / Gm_{k+1}: lane (i, m) stores coarse row 1 + i,
      // columns 1 + 4m .. 4 + 4m, one 16-byte store where the four are inside the coarse ROI
      {
        const int i = 1 + (lane >> 3), j = 1 + 4 * (lane & 7);
        const float4 v4 = *reinterpret_cast<const float4*>(&sC[ch][i][CO + j]);
        const float v[4] = {v4.x, v4.y, v4.z, v4.w};
        const int cy = Y0 / 2 - 1 + i - it.croi_y, cx = X0 / 2 - 1 + j - it.croi_x;
        // FP16: lanes 2m and 2m+1 hold eight adjacent samples; the even lane stores all
        // eight as one 16-byte vector (the partner's four halves come by a lane swap)
        uint32_t h01 = 0, h23 = 0, p01 = 0, p23 = 0;
        if (sizeof(T) == 2) {
          h01 = pack_h2(v[0], v[1]);
          h23 = pack_h2(v[2], v[3]);
          p01 = __shfl_xor(h01, 1);
          p23 = __shfl_xor(h23, 1);
        }
        if (cy >= 0 && cy < it.croi_h) {
          GLB T* out = ch < 3 ? mg<T>(it.g_out) : mg<T>(it.gm_out);
          // 32-bit element offsets (the host keeps every level's planes under 2^31
          // elements and its rows under 2^23)
          const uint32_t orow = (uint32_t)(ch < 3 ? it.g_row : it.gm_row);
          const uint32_t obase = ch < 3 ? (uint32_t)ch * (uint32_t)it.g_plane : 0u;
          const int ob = (int)(obase + __umul24((uint32_t)cy, orow)) + cx;
          const bool odd = (lane & 1) != 0;
          const int cxe = cx - (odd ? 4 : 0), obe = ob - (odd ? 4 : 0);
          if (sizeof(T) == 2 && cxe >= 0 && cxe + 7 < it.croi_w && ((uintptr_t)(out + obe) & 15) == 0) {
            if (!odd) stg8nt(reinterpret_cast<GLB _Float16*>(out + obe), h01, h23, p01, p23);
          } else if (cx >= 0 && cx + 3 < it.croi_w && ((uintptr_t)(out + ob) & (4 * sizeof(T) - 1)) == 0) {
            stg4nt(out + ob, v);
          } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (cx + u >= 0 && cx + u < it.croi_w) stgnt(out, ob + u, v[u]);
          }
        }
      }
      if (ch == 3) continue;
      const bool lap_tile = it.lw_w > 0 && X0 < it.lw_x + it.lw_w && X0 + TX > it.lw_x &&
                            Y0 < it.lw_y + it.lw_h && Y0 + TY > it.lw_y;
      if (!lap_tile) continue;

      // D+E: lane (rq, mm): fine columns 4mm .. 4mm+3 of fine rows 4rq .. 4rq+3.  Horizontal
      // EXPAND of coarse rows 2rq .. 2rq+3, then vertical EXPAND and the band
      // L_k = G_k - EXPAND(G_{k+1}), stored on the band window.
      {
        const int mm = lane & 15, rq = lane >> 4, x = 4 * mm;
        float4 eh[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float* c = &sC[ch][2 * rq + k][CO + 2 * mm];
          const float2 lo = {c[0], c[1]}, hi = {c[2], c[3]};
          eh[k].x = exp_h(lo.x + hi.x, lo.y);
          eh[k].y = 0.5f * (lo.y + hi.x);
          eh[k].z = exp_h(lo.y + hi.y, hi.x);
          eh[k].w = 0.5f * (hi.x + hi.y);
        }
        const int X = X0 + x - it.lw_x;
        GLB T* lout = mg<T>(it.l_out);
        float l[4][4];
#pragma unroll
        for (int yy = 0; yy < 4; ++yy) {
          const int y = 4 * rq + yy, k = yy >> 1;
          const float4 gv = *reinterpret_cast<const float4*>(rowp(y + 4) + x + 4);
          if (yy & 1) {
            l[yy][0] = band_odd(gv.x, eh[k + 1].x + eh[k + 2].x, 0, T());
            l[yy][1] = band_odd(gv.y, eh[k + 1].y + eh[k + 2].y, 1, T());
            l[yy][2] = band_odd(gv.z, eh[k + 1].z + eh[k + 2].z, 2, T());
            l[yy][3] = band_odd(gv.w, eh[k + 1].w + eh[k + 2].w, 3, T());
          } else {
            l[yy][0] = gv.x - exp_v(eh[k].x + eh[k + 2].x, eh[k + 1].x);
            l[yy][1] = gv.y - exp_v(eh[k].y + eh[k + 2].y, eh[k + 1].y);
            l[yy][2] = gv.z - exp_v(eh[k].z + eh[k + 2].z, eh[k + 1].z);
            l[yy][3] = gv.w - exp_v(eh[k].w + eh[k + 2].w, eh[k + 1].w);
          }
        }
        // FP16: lanes 2m and 2m+1 hold eight adjacent columns of the same four rows; the
        // even lane stores rows 0-1 and the odd lane rows 2-3 as 16-byte vectors, each
        // taking the partner's halves of those rows by a lane swap
        const bool odd = (mm & 1) != 0;
        const int Xe = X - (odd ? 4 : 0);
        bool pair = false;
        uint32_t own[2][2] = {}, oth[2][2] = {};
        if (sizeof(T) == 2) {
          uint32_t hp[4][2];
#pragma unroll
          for (int yy = 0; yy < 4; ++yy) {
            hp[yy][0] = pack_h2(l[yy][0], l[yy][1]);
            hp[yy][1] = pack_h2(l[yy][2], l[yy][3]);
          }
#pragma unroll
          for (int r2 = 0; r2 < 2; ++r2)
#pragma unroll
            for (int w2 = 0; w2 < 2; ++w2) {
              // send the rows the partner stores, keep the ones this lane stores
              own[r2][w2] = odd ? hp[2 + r2][w2] : hp[r2][w2];
              oth[r2][w2] = __shfl_xor(odd ? hp[r2][w2] : hp[2 + r2][w2], 1);
            }
          pair = Xe >= 0 && Xe + 7 < it.lw_w && ((uintptr_t)(lout + Xe) & 15) == 0 &&
                 ((it.l_row | it.l_plane) & 7) == 0;
        }
#pragma unroll
        for (int yy = 0; yy < 4; ++yy) {
          const int y = 4 * rq + yy;
          const int Y = Y0 + y - it.lw_y;
          const bool rowin = Y >= 0 && Y < it.lw_h;
          if (sizeof(T) == 2 && pair) {
            // this lane's two rows (the even lane's 0-1, the odd lane's 2-3)
            if (yy < 2) {
              const int Ys = Y + (odd ? 2 : 0);
              if (Ys >= 0 && Ys < it.lw_h) {
                const int base = ch * (int)it.l_plane + __mul24(Ys, (int)it.l_row) + Xe;
                GLB _Float16* q = reinterpret_cast<GLB _Float16*>(lout + base);
                if (odd) stg8nt(q, oth[yy][0], oth[yy][1], own[yy][0], own[yy][1]);
                else stg8nt(q, own[yy][0], own[yy][1], oth[yy][0], oth[yy][1]);
              }
            }
            continue;
          }
          const bool full = rowin && X >= 0 && X + 3 < it.lw_w;
          const int base = ch * (int)it.l_plane + __mul24(Y, (int)it.l_row) + X;
          if (full && ((uintptr_t)(lout + base) & (4 * sizeof(T) - 1)) == 0) {
            stg4nt(lout + base, l[yy]);
          } else if (full) {
#pragma unroll
            for (int u = 0; u < 4; ++u) stgnt(lout, base + u, l[yy][u]);
          } else if (rowin) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (X + u >= 0 && X + u < it.lw_w) stgnt(lout, base + u, l[yy][u]);
          }
        }
      }
    }
  }
}

// Four adjacent samples as read, from or to any sample address (global memory takes vectors at
// any byte).
typedef uint32_t __attribute__((aligned(1))) u32_unaligned;
template <typename T>
struct Quad;
template <>
struct Quad<float> {
  uint32_t d[4];
  // (load_dwords: dword by dword, `step` bytes apart -- four bytes' worth at step 0 -- so that the
  // choice between byte and sample weights is not a branch)
  __device__ __forceinline__ void load(const GLB float* p) {
    typedef uint32_t vu __attribute__((ext_vector_type(4), aligned(4)));
    const vu t = *reinterpret_cast<const GLB vu*>(p);
    d[0] = t.x; d[1] = t.y; d[2] = t.z; d[3] = t.w;
  }
  __device__ __forceinline__ void load_dwords(const GLB uint8_t* p, int step) {
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = *(const GLB u32_unaligned*)(p + i * step);
  }
  __device__ __forceinline__ void clear() { d[0] = d[1] = d[2] = d[3] = 0; }
  __device__ __forceinline__ void put(int u, uint32_t raw) { d[u] = raw; }
  __device__ __forceinline__ float at(int u) const { return __builtin_bit_cast(float, d[u]); }
};
template <>
struct Quad<_Float16> {
  uint32_t d[2];
  __device__ __forceinline__ void load(const GLB _Float16* p) {
    typedef uint32_t vu __attribute__((ext_vector_type(2), aligned(2)));
    const vu t = *reinterpret_cast<const GLB vu*>(p);
    d[0] = t.x; d[1] = t.y;
  }
  __device__ __forceinline__ void load_dwords(const GLB uint8_t* p, int step) {
#pragma unroll
    for (int i = 0; i < 2; ++i) d[i] = *(const GLB u32_unaligned*)(p + i * step);
  }
  __device__ __forceinline__ void clear() { d[0] = d[1] = 0; }
  __device__ __forceinline__ void put(int u, uint32_t raw) { d[u >> 1] |= raw << (16 * (u & 1)); }
  __device__ __forceinline__ float at(int u) const { return from_raw((uint16_t)(d[u >> 1] >> (16 * (u & 1)))); }
};
__device__ __forceinline__ void store4_any(GLB float* p, const float v[4]) {
  typedef float vf __attribute__((ext_vector_type(4), aligned(4)));
  *reinterpret_cast<GLB vf*>(p) = vf{v[0], v[1], v[2], v[3]};
}
__device__ __forceinline__ void store4_any(GLB _Float16* p, const float v[4]) {
  typedef _Float16 vh __attribute__((ext_vector_type(4), aligned(2)));
  *reinterpret_cast<GLB vh*>(p) = vh{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
}

__device__ __forceinline__ int find_blend_item(const BlendItem* __restrict__ items, int nitems, int t) {
  int lo = 0, hi = nitems - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cst(items)[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Quantise one tile row (64 lanes, column X0 + x) of the panorama.  A full tile row in an
// aligned panorama goes out as whole dwords: each group of four lanes (four adjacent pixels,
// 12 bytes) packs its bytes into three dwords in its first lane; otherwise byte by byte.
__device__ __forceinline__ void put_row(uint8_t* pano_ptr, int64_t pano_row, int X0, int x, int Y, int W, int H,
                                        const float r[3]) {
  const int X = X0 + x;
  const bool words = X0 + kBlendTX <= W && (pano_row & 3) == 0 && ((uintptr_t)pano_ptr & 3) == 0;
  // rint(255 R_0) clamped to [0, 255] by the byte conversion, packed byte by byte
  uint32_t v = __builtin_amdgcn_cvt_pk_u8_f32(255.0f * r[0], 0u, 0u);
  v = __builtin_amdgcn_cvt_pk_u8_f32(255.0f * r[1], 1u, v);
  v = __builtin_amdgcn_cvt_pk_u8_f32(255.0f * r[2], 2u, v);
  GLB uint8_t* prow = mg<uint8_t>(pano_ptr) + (int64_t)Y * pano_row + (int64_t)X * 3;
  if (words) {
    const uint32_t v1 = __shfl_down(v, 1), v2 = __shfl_down(v, 2), v3 = __shfl_down(v, 3);
    if ((x & 3) == 0 && Y < H) {
      typedef uint32_t vu3 __attribute__((ext_vector_type(3)));
      *reinterpret_cast<GLB vu3*>(prow) = vu3{v | (v1 << 24), (v1 >> 8) | (v2 << 16), (v2 >> 16) | (v3 << 8)};
    }
  } else if (X < W && Y < H) {
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) prow[ch] = (uint8_t)(v >> (8 * ch));
  }
}

// ------------------------------------------------------------------------------------
// One synthesis level: B_k over cameras + EXPAND(R_{k+1}) -> R_k (and the panorama at k = 0), 64x16
// tiles, four adjacent pixels of a row a thread.
template <typename T, bool FINAL, bool KARG>
__global__ void __launch_bounds__(kThreads) k_blend(const BlendItem* __restrict__ items, int nitems, BlendItem one,
                                                    PanoArg po) {
  constexpr int TX = kBlendTX, TY = kBlendTY;
  constexpr int CW = TX / 2 + 2, CH = TY / 2 + 2;
  // coarse column j at index j + CO, so that columns 1 .. 32 start on a 16-byte boundary
  constexpr int HS = 40, CO = 3, ES = TX + 4;
  __shared__ __attribute__((aligned(16))) float sC[3][CH][HS];
  __shared__ __attribute__((aligned(16))) float sE[3][CH][ES];

  const int tid = threadIdx.x;
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  const BlendItem a = KARG ? one : ld_cst(cst(items) + find_blend_item(items, nitems, t));
  const int lt = t - a.tile_begin;
  const int tyi = lt / a.tiles_x, txi = lt - tyi * a.tiles_x;
  const int X0 = txi * TX, Y0 = tyi * TY;
  const bool has_coarse = a.has_coarse != 0;

  // every wave builds the tile's camera set itself (lane i tests camera i): no LDS, no barrier
  uint64_t cams;
  {
    const int i = tid & 63;
    bool hit = false;
    if (i < a.ncam) {
      const CST BlendCam& c = cst(a.cams)[i];
      const int x0 = max(c.lx, c.wx), x1 = min(c.lx + c.lw, c.wx + c.ww);
      const int y0 = max(c.ly, c.wy), y1 = min(c.ly + c.lh, c.wy + c.wh);
      hit = x0 < x1 && y0 < y1 && x0 < X0 + TX && x1 > X0 && y0 < Y0 + TY && y1 > Y0;
    }
    cams = __ballot(hit);
  }

  // A thread has four adjacent pixels of one row (a wave rows of one parity, so its EXPAND takes
  // one form): bands, weights, R and panorama bytes go as vectors.  Bound by memory; by the vector
  // arithmetic when a thread had one column of four rows, sample by sample (8 jobs at 640 to 3840
  // columns, FP16, level 0, 47.7 million pixels: 109 instructions a pixel, 154 us); now 135 us
  // at 4.1 TB/s, four fifths of a copy's rate.
  const int m = tid & 15, wvi = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int odd = wvi & 1, y = 8 * (wvi >> 1) + odd + 2 * ((tid >> 4) & 3);
  const int X = X0 + 4 * m, Y = Y0 + y;
  // One camera's band and weight samples of the four pixels, as read; used after the coarse
  // stage.  Its descriptor is read once (scalar loads issued together), offsets are 32-bit (the
  // host keeps every band and weight plane under 2^31 elements and its rows under 2^23); an FP32
  // weight's place in bytes is not (2^30 samples are 2^32 bytes).
  struct CamSamples {
    Quad<T> l[3], w;        // (byte weights: w.d[0])
    bool in, u8;
  };
  auto fetch = [&](int ci, CamSamples& cs) __attribute__((always_inline)) {
    const BlendCam c = ld_cst(cst(a.cams) + ci);
    const int lx = X - c.lx, wx = X - c.wx, ly = Y - c.ly, wy = Y - c.wy;
    const bool yin = (ly >= 0) & (ly < c.lh) & (wy >= 0) & (wy < c.wh);
    const int u0 = max(max(-lx, -wx), 0), u1 = min(min(c.lw - lx, c.ww - wx), 4);   // pixels u0 .. u1-1 are inside
    cs.in = yin & (u0 < u1);
    cs.u8 = c.wgt_u8 != 0;
    const uint32_t loff = __umul24((uint32_t)ly, (uint32_t)c.lap_row) + (uint32_t)lx;
    const uint32_t woff = __umul24((uint32_t)wy, (uint32_t)c.wgt_row) + (uint32_t)wx;
    const GLB T* l = cg<T>(c.lap);
    using Bytes = std::conditional_t<sizeof(T) == 4, uint64_t, uint32_t>;
    const Bytes wes = cs.u8 ? 1 : sizeof(T);
    if (cs.in & (u0 == 0) & (u1 == 4)) {
      cs.w.load_dwords(cg<uint8_t>(c.wgt) + woff * wes, cs.u8 ? 0 : 4);
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) cs.l[ch].load(l + ((uint32_t)ch * (uint32_t)c.lap_plane + loff));
    } else if (cs.in) {
      // the few quads across a window's edge, pixel by pixel: pixels outside repeat one inside,
      // every read in flight, and then count 0 (weight and sample: the one inside may be infinite)
      typename RawOf<T>::type lv[3][4];
      uint32_t wv[4][sizeof(T)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int v = min(max(u, u0), u1 - 1);
        const GLB uint8_t* wp = cg<uint8_t>(c.wgt) + (woff + v) * wes;
#pragma unroll
        for (int b = 0; b < (int)sizeof(T); ++b) wv[u][b] = wp[cs.u8 ? 0 : b];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) lv[ch][u] = ld_raw(l, (uint32_t)ch * (uint32_t)c.lap_plane + loff + v);
      }
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) cs.l[ch].clear();
      cs.w.clear();
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool ok = (u >= u0) & (u < u1);
        uint32_t w = 0;                              // the sample's bytes
#pragma unroll
        for (int b = 0; b < (int)sizeof(T); ++b) w |= wv[u][b] << (8 * b);
        if (cs.u8) cs.w.d[0] |= ok ? wv[u][0] << (8 * u) : 0u;
        else cs.w.put(u, ok ? w : 0u);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) cs.l[ch].put(u, ok ? lv[ch][u] : 0);
      }
    }
  };
  float acc[3][4];
#pragma unroll
  for (int ch = 0; ch < 3; ++ch)
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[ch][u] = 0.0f;
  auto accumulate = [&](const CamSamples& cs) __attribute__((always_inline)) {
    if (!cs.in) return;
    float w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) w[u] = cs.u8 ? (float)((cs.w.d[0] >> (8 * u)) & 255u) * kInv255 : cs.w.at(u);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch)
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[ch][u] = __builtin_fmaf(w[u], cs.l[ch].at(u), acc[ch][u]);
  };
  // the first camera's reads fly together with the coarse level's
  const int first = cams ? (int)__builtin_ctzll(cams) : -1;
  CamSamples cs0;
  if (first >= 0) fetch(first, cs0);

  if (has_coarse) {
    const GLB T* r = cg<T>(a.r_in);
    const int cx0 = X0 / 2 - 1, cy0 = Y0 / 2 - 1;
    // A tile whose coarse samples all have their fine position inside the level needs no
    // folding: eight quads of every row and channel, and the two columns beside them.
    const bool inner = cx0 >= 0 && 2 * (cx0 + CW - 1) < a.W && cy0 >= 0 && 2 * (cy0 + CH - 1) < a.H;
    if (inner) {
      const int rowq = min(tid >> 3, 3 * CH - 1), cq = rowq / CH, iq = rowq - cq * CH, k = tid & 7;
      const int rowe = min(tid >> 1, 3 * CH - 1), ce = rowe / CH, ie = rowe - ce * CH;
      Quad<T> v;
      v.load(r + (cq * a.rin_plane + (int64_t)(cy0 + iq) * a.rin_row + (X0 / 2 + 4 * k)));
      float e = 0.0f;
      if (tid < 2 * 3 * CH)
        e = from_raw(ld_raw(r, ce * a.rin_plane + (int64_t)(cy0 + ie) * a.rin_row + cx0 + (tid & 1) * (CW - 1)));
      // (threads past the last row repeat it: the same values to the same place)
      *reinterpret_cast<float4*>(&sC[cq][iq][CO + 1 + 4 * k]) = float4{v.at(0), v.at(1), v.at(2), v.at(3)};
      if (tid < 2 * 3 * CH) sC[ce][ie][CO + (tid & 1) * (CW - 1)] = e;
    } else {
      constexpr int NC = 3 * CH * CW, NIT = (NC + kThreads - 1) / kThreads;
#pragma unroll 1
      for (int q = 0; q < NIT; ++q) {
        const int e = min(tid + q * kThreads, NC - 1), row = e / CW, j = e - row * CW, c = row / CH, i = row - c * CH;
        const int cy = min(fold(2 * (cy0 + i), a.H) >> 1, a.cH - 1);
        const int cx = min(fold(2 * (cx0 + j), a.W) >> 1, a.cW - 1);
        sC[c][i][CO + j] = from_raw(ld_raw(r, c * a.rin_plane + (int64_t)cy * a.rin_row + cx));
      }
    }
    __syncthreads();
    // horizontal EXPAND: item e = tid + k kThreads is (channel, row, quad m) of the
    // 3 x CH x 16 quads
    constexpr int PER = CH * (TX / 4);
    static_assert(TX / 4 == 16 && kThreads < 2 * PER && 3 * PER <= 2 * kThreads, "two rounds, one carry");
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int e = tid + k * kThreads;
      if (e < 3 * PER) {
        const int ch = (e >= PER ? 1 : 0) + (e >= 2 * PER ? 1 : 0), rem = e - ch * PER;
        const int i = rem >> 4, q = rem & 15;
        const float* c = &sC[ch][i][CO + 2 * q];
        const float2 lo = {c[0], c[1]}, hi = {c[2], c[3]};
        float4 o;
        o.x = exp_h(lo.x + hi.x, lo.y);
        o.y = 0.5f * (lo.y + hi.x);
        o.z = exp_h(lo.y + hi.y, hi.x);
        o.w = 0.5f * (hi.x + hi.y);
        *reinterpret_cast<float4*>(&sE[ch][i][4 * q]) = o;
      }
    }
    __syncthreads();
  }
  // cameras in ascending index order
  if (first >= 0) {
    accumulate(cs0);
    for (uint64_t rest = cams & (cams - 1); rest; rest &= rest - 1) {
      CamSamples cs;
      fetch((int)__builtin_ctzll(rest), cs);
      accumulate(cs);
    }
  }
  if (has_coarse) {
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      const float* e = &sE[ch][y >> 1][4 * m];       // rows e, e + ES, e + 2 ES
      const float4 e1 = *reinterpret_cast<const float4*>(e + ES), e2 = *reinterpret_cast<const float4*>(e + 2 * ES);
      if (odd) {
        acc[ch][0] = __builtin_fmaf(0.5f, e1.x + e2.x, acc[ch][0]);
        acc[ch][1] = __builtin_fmaf(0.5f, e1.y + e2.y, acc[ch][1]);
        acc[ch][2] = __builtin_fmaf(0.5f, e1.z + e2.z, acc[ch][2]);
        acc[ch][3] = __builtin_fmaf(0.5f, e1.w + e2.w, acc[ch][3]);
      } else {
        const float4 e0 = *reinterpret_cast<const float4*>(e);
        acc[ch][0] = acc[ch][0] + exp_v(e0.x + e2.x, e1.x);
        acc[ch][1] = acc[ch][1] + exp_v(e0.y + e2.y, e1.y);
        acc[ch][2] = acc[ch][2] + exp_v(e0.z + e2.z, e1.z);
        acc[ch][3] = acc[ch][3] + exp_v(e0.w + e2.w, e1.w);
      }
    }
  }
  if (X >= a.W || Y >= a.H) return;
  const bool whole = X + 3 < a.W;
  if (a.r_out != nullptr) {
    GLB T* ro = mg<T>(a.r_out) + (int64_t)Y * a.rout_row + X;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = settled(acc[ch][u]);
      GLB T* p = ro + ch * a.rout_plane;
      if (whole) {
        store4_any(p, v);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (X + u < a.W) stg(p, u, v[u]);
      }
    }
  }
  if (FINAL) {
    // rint(255 R_0) clamped to [0, 255] by the byte conversion, packed byte by byte; four pixels
    // are three dwords, stored as such at any byte (byte by byte, as a
    // panorama of odd pitch would need at dword alignment, the 8 jobs took 181 us)
    uint8_t* const pano_ptr = po.ptr ? po.ptr : a.pano;
    const int64_t pano_row = po.ptr ? po.row : a.pano_row;
    GLB uint8_t* prow = mg<uint8_t>(pano_ptr) + (int64_t)Y * pano_row + (int64_t)X * 3;
    uint32_t d[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < 12; ++k)
      d[k >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(255.0f * acc[k % 3][k / 3], (uint32_t)(k & 3), d[k >> 2]);
    if (whole) {
      typedef uint32_t vu3 __attribute__((ext_vector_type(3), aligned(1)));
      *reinterpret_cast<GLB vu3*>(prow) = vu3{d[0], d[1], d[2]};
    } else {
#pragma unroll
      for (int k = 0; k < 12; ++k)
        if (X + k / 3 < a.W) prow[k] = (uint8_t)(d[k >> 2] >> (8 * (k & 3)));
    }
  }
}

// ------------------------------------------------------------------------------------
// The tail of a pyramid: up to three consecutive REDUCEs (and the bands between them) of small
// levels in one launch.  A level pass of a few hundred workgroups takes 7-10 us however small
// it is -- launch, descriptor, window and store latencies one after another, with the chip
// nearly empty -- so three levels cost 25-30 us.  Here a workgroup takes one channel of a
// 64x32 tile with the halo all three levels need (104x69 samples: 3.5 times the tile's own,
// which is why only levels below the host's size limit are done this way), and the coarser
// levels never leave LDS between their uses.  VGA pair, levels 1 .. 4: 23.5 -> 12.3 us;
// four 1080p cameras, levels 2 .. 5: 27.7 -> 23 us.
//
// stitch_pyramid's chains run here as well (an item by value; no bands, whose EXPAND there takes
// the stored coarse level): a VGA image's three levels 25 -> 12-15 us, a 2240x1080 byte map's
// four, conversion included, 50 -> 24 us.
//
// The values are those of the level passes bit for bit: the same expressions, a level's
// samples rounded to the storage type before they are reduced again, 0 outside its region,
// reflect-101 at its canvas edges (each level's own for REDUCE; the reduced reflected fine
// samples, as they come, for EXPAND).
//
// Windows in LDS, (0, 0) the tile's first sample of a level: level 0 columns -24 .. 79, rows
// -22 .. 46; level 1 columns -12 .. 39, rows -10 .. 22; level 2 columns -8 .. 19, rows
// -4 .. 10; level 3 columns -1 .. 10, rows -1 .. 4.
constexpr int kT0S = 104, kT0R = 69;                      // the finest window (f below, d = 0)
constexpr int kT1S = 52, kT1R = 33, kT2S = 28, kT2R = 15, kT3S = 12, kT3R = 6;

__device__ __forceinline__ float as_stored(float v, float) { return v; }
__device__ __forceinline__ float as_stored(float v, _Float16) { return (float)(_Float16)v; }
__device__ __forceinline__ float byte_as_stored(uint32_t v, float) { return (float)v * kInv255; }
__device__ __forceinline__ float byte_as_stored(uint32_t v, _Float16) { return fma_half((float)v, kInv255, 0.0f); }

// Periodic reflect-101 by repeated reflection (a short loop; one turn where the overshoot is
// below the side).
__device__ __forceinline__ int fold_loop(int i, int n) {
  for (;;) {
    i = i < 0 ? -i : i;
    if (i < n) return i;
    i = 2 * (n - 1) - i;
  }
}

// Read one dword of every 64-byte line of a descriptor at once, so that its fields, wanted one
// level after another, come from the scalar cache (each line's first read is a trip to memory
// otherwise: 4 x 1000 cycles of a tail's 20000).
template <typename D>
__device__ __forceinline__ void touch(const CST D* p) {
  const CST int* w = (const CST int*)p;
  int any = 0;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(D) / 4); i += 16) any |= w[i];
  asm volatile("" ::"s"(any));
}

// Four adjacent samples from an address aligned to all of them.
__device__ __forceinline__ void load4(const GLB float* p, float v[4]) {
  typedef float vf __attribute__((ext_vector_type(4)));
  const vf t = *reinterpret_cast<const GLB vf*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
__device__ __forceinline__ void load4(const GLB _Float16* p, float v[4]) {
  typedef _Float16 vh __attribute__((ext_vector_type(4)));
  const vh t = *reinterpret_cast<const GLB vh*>(p);
  v[0] = (float)t.x; v[1] = (float)t.y; v[2] = (float)t.z; v[3] = (float)t.w;
}

// Four adjacent samples, columns X .. X+3 of a window w wide, to row pointer p (elements).
template <typename T>
__device__ __forceinline__ void store4(GLB T* p, int X, int w, const float v[4]) {
  if (X >= 0 && X + 3 < w && ((uintptr_t)(p + X) & (4 * sizeof(T) - 1)) == 0) {
    stg4nt(p + X, v);
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (X + u >= 0 && X + u < w) stgnt(p, X + u, v[u]);
  }
}

template <typename S>
struct SampleKind {
  using sample = S;
};
// Adjacent samples read at once from any sample address: 16 bytes, eight of a byte image.
template <typename S>
struct Chunk {
  uint32_t w0, w1, w2, w3;
  __device__ __forceinline__ void load(const GLB S* p) {
    typedef uint32_t vu4a __attribute__((ext_vector_type(4), aligned(2)));
    const vu4a v = *reinterpret_cast<const GLB vu4a*>(p);
    w0 = v.x; w1 = v.y; w2 = v.z; w3 = v.w;
  }
  template <typename T>
  __device__ __forceinline__ float at(int i, T) const {
    const int d = i * (int)sizeof(S) / 4;
    const uint32_t w = d == 0 ? w0 : d == 1 ? w1 : d == 2 ? w2 : w3;
    return sizeof(S) == 4 ? __builtin_bit_cast(float, w) : from_raw((uint16_t)(w >> (16 * (i & 1))));
  }
};
template <>
struct Chunk<uint8_t> {
  unsigned long long w;
  __device__ __forceinline__ void load(const GLB uint8_t* p) { w = ld8(p); }
  template <typename T>
  __device__ __forceinline__ float at(int i, T) const {
    return byte_as_stored((uint32_t)(w >> (8 * i)) & 255u, T());
  }
};

// One sample as the tail holds it.
template <typename S, typename T>
__device__ __forceinline__ float one_sample(const GLB S* p, int64_t i, T) {
  return from_raw(ld_raw(p, i));
}
template <typename T>
__device__ __forceinline__ float one_sample(const GLB uint8_t* p, int64_t i, T) {
  return byte_as_stored(p[i], T());
}

template <typename T, bool KARG>
__global__ void __launch_bounds__(kThreads) k_tail(const TailItem one, const TailItem* __restrict__ items, int nitems,
                                                   int nslot) {
  // sm: the finest window, then levels 1 and 2 as the next REDUCE reads them; sc: levels 1 .. 3
  // as reduced
  __shared__ __attribute__((aligned(16))) float sm[kT0R * kT0S + kT1R * kT1S + kT2R * kT2S];
  __shared__ __attribute__((aligned(16))) float sc[kT1R * kT1S + kT2R * kT2S + kT3R * kT3S];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t = (int)blockIdx.x / nslot, slot = (int)blockIdx.x - t * nslot;
  const CST TailItem* itp;
  if (KARG) {
    itp = first_arg<TailItem>();
  } else {
    int lo = 0, hi = nitems - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (cst(items)[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
    }
    itp = cst(items) + lo;
  }
  const CST TailItem& it = *itp;
  touch(itp);
  const int lt = t - it.tile_begin, tyi = lt / it.tiles_x, txi = lt - tyi * it.tiles_x;
  const int X0 = it.tile_x0 + txi * kTailTX, Y0 = it.tile_y0 + tyi * kTailTY;
  const int nch = it.nch;
  const bool img = slot < nch;

  // ---- the finest level's window ----
  {
    const TailLevel l0 = ld_cst(it.lev);
    const int wx0 = X0 - 24, wy0 = Y0 - 22;
    // the rows that this depth reads (a shallower tail repeats the outermost ones: cheaper than
    // other windows for it)
    const int rlo = KARG ? (it.depth == 1 ? 18 : it.depth == 2 ? 12 : 0) : 0;
    const int rhi = KARG ? (it.depth == 1 ? 56 : it.depth == 2 ? 60 : kT0R - 1) : kT0R - 1;
    const int rx = l0.roi_x, ry = l0.roi_y, rw = l0.roi_w, rh = l0.roi_h, lw = l0.w, lh = l0.h;
    const int64_t row = img ? it.img_row : it.msk_row;
    const bool u8 = KARG && img && it.src_u8 != 0;
    const GLB T* src = img ? cg<T>(it.img) + slot * it.img_plane : cg<T>(it.msk);
    // A lane takes C adjacent samples of a row, a wave RPW rows at a time, every read issued
    // before any is used.  A read that would begin or end outside its row is moved inside; its
    // samples are then written where they belong, after zeros where the row has none (a row of
    // fewer than C samples is read one by one).
    auto stage = [&](auto kind) __attribute__((always_inline)) {
      using S = typename decltype(kind)::sample;
      constexpr int C = sizeof(S) == 4 ? 4 : 8, NCK = kT0S / C, RPW = 64 / NCK, NQ = (kT0R + 4 * RPW - 1) / (4 * RPW);
      static_assert(RPW * NQ <= 64, "a lane per row of the wave");
      const GLB S* base = sizeof(S) == 1 ? (const GLB S*)cg<uint8_t>(it.img) : (const GLB S*)src;
      // lane i: plane row of the wave's window row i
      const int wr = (lane / RPW * 4 + wv) * RPW + lane % RPW;
      const int yi = fold_loop(wy0 + min(max(wr, rlo), rhi), lh) - ry;
      const int rs = lane / NCK, k = lane - rs * NCK, c0 = wx0 - rx + C * k;
      const int col = min(max(c0, 0), rw - C);
      const bool own = c0 == col, part = !own & (c0 > -C) & (c0 < rw);
      float* out = sm + (wv * RPW + rs) * kT0S + C * k;
      if (rw >= C) {
        Chunk<S> raw[NQ];
        bool in[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const int y = __shfl(yi, q * RPW + min(rs, RPW - 1));
          in[q] = (y >= 0) & (y < rh);
          raw[q].load(base + (min(max(y, 0), rh - 1) * row + col));
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          if ((rs >= RPW) | ((q * 4 + wv) * RPW + rs >= kT0R)) continue;
          float v[C];
#pragma unroll
          for (int i = 0; i < C; ++i) v[i] = raw[q].at(i, T());
          float* o = out + q * 4 * RPW * kT0S;
#pragma unroll
          for (int h = 0; h < C / 4; ++h) {
            const bool ok = own & in[q];
            *reinterpret_cast<float4*>(o + 4 * h) = float4{ok ? v[4 * h] : 0.0f, ok ? v[4 * h + 1] : 0.0f,
                                                           ok ? v[4 * h + 2] : 0.0f, ok ? v[4 * h + 3] : 0.0f};
          }
          if (part & in[q]) {
            const int at = C * k + col - c0;
#pragma unroll
            for (int i = 0; i < C; ++i)
              if ((at + i >= 0) & (at + i < kT0S)) o[col - c0 + i] = v[i];
          }
        }
      } else {
#pragma unroll 1
        for (int q = 0; q < NQ; ++q) {
          const int y = __shfl(yi, q * RPW + min(rs, RPW - 1));
          if ((rs >= RPW) | ((q * 4 + wv) * RPW + rs >= kT0R)) continue;
#pragma unroll 1
          for (int i = 0; i < C; ++i) {
            const bool in1 = (y >= 0) & (y < rh) & (c0 + i >= 0) & (c0 + i < rw);
            float v = 0.0f;
            if (in1) v = one_sample(base, y * row + c0 + i, T());
            out[q * 4 * RPW * kT0S + i] = v;
          }
        }
      }
    };
    if (!u8) stage(SampleKind<T>());
    else if (KARG) stage(SampleKind<uint8_t>());
    if (wx0 < 0 || wx0 + kT0S > lw) {
      // columns outside the canvas, from their reflections (one beyond the window feeds nothing
      // that is kept: any column will do)
      __syncthreads();
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = lane + 64 * h, x = wx0 + c;
        if ((c >= kT0S) | ((x >= 0) & (x < lw))) continue;
        const int from = min(max(fold_loop(x, lw) - wx0, 0), kT0S - 1);
#pragma unroll 6
        for (int r = wv; r < kT0R; r += 4) sm[r * kT0S + c] = sm[r * kT0S + from];
      }
    }
  }
  __syncthreads();
  if (KARG && it.copy_out && img) {
    // the finest level itself, on its region
    const CST TailLevel& l0 = it.lev[0];
    GLB T* out = mg<T>(it.copy_out) + slot * it.copy_plane;
#pragma unroll 1
    for (int e = tid; e < (kTailTX / 4) * kTailTY; e += kThreads) {
      const int r = e / (kTailTX / 4), m = e - r * (kTailTX / 4), y = Y0 + r - l0.roi_y;
      if (y < 0 || y >= l0.roi_h) continue;
      const float4 v4 = *reinterpret_cast<const float4*>(&sm[(22 + r) * kT0S + 24 + 4 * m]);
      const float v[4] = {v4.x, v4.y, v4.z, v4.w};
      store4(out + y * it.copy_row, X0 + 4 * m - l0.roi_x, l0.roi_w, v);
    }
  }

  // ---- level by level: f the fine window, c the coarse one as reduced, g as the next level
  //      reads it (one body for all three: the code is fetched once, and fetching it is much
  //      of what a launch this small waits for; above the finest level a stage's few items
  //      are spread over the waves, since every stage is then one thread's latency) ----
  int fs = kT0S, fr = kT0R, fx = 24, fy = 22;       // stride, rows, column and row of (0, 0)
  float* f = sm;
  float* c = sc;
  const int depth = it.depth;
#pragma unroll 1
  for (int d = 0; d < depth; ++d) {
    const TailLevel lv = ld_cst(it.lev + d);    // every field at once, none behind a test
    const int cs = d == 0 ? kT1S : d == 1 ? kT2S : kT3S, cr = d == 0 ? kT1R : d == 1 ? kT2R : kT3R;
    const int cx = d == 0 ? 12 : d == 1 ? 8 : 1, cy = d == 0 ? 10 : d == 1 ? 4 : 1;
    float* g = f + fr * fs;
    // REDUCE: pair p of coarse columns reads fine columns fo + 4p .. fo + 4p + 7, coarse row i
    // fine rows 2i .. 2i + 4; a thread takes a pair and four rows (one above the finest level)
    {
      const int np = d == 0 ? 25 : d == 1 ? 12 : 5, fo = d == 2 ? 4 : 0, co = d == 0 ? 1 : d == 1 ? 3 : 0;
      const int i = (tid * (d == 0 ? 2622 : d == 1 ? 5462 : 13108)) >> 16, p = tid - i * np;   // tid / np
      const int step = d == 0 ? 4 : 1, i0 = step * i, i1 = min(i0 + step, cr);
      auto hrow = [&](int r) -> float2 {
        const float* rowp = f + r * fs + fo + 4 * p;
        const float4 u = *reinterpret_cast<const float4*>(rowp);
        const float4 v = *reinterpret_cast<const float4*>(rowp + 4);
        return float2{reduce5(u.x + v.x, u.y + u.w, u.z), reduce5(u.z + v.z, u.w + v.y, v.x)};
      };
      if (i0 < cr) {
        float2 h0 = hrow(2 * i0), h1 = hrow(2 * i0 + 1), h2 = hrow(2 * i0 + 2);
#pragma unroll 1
        for (int m = i0; m < i1; ++m) {
          const float2 h3 = hrow(2 * m + 3), h4 = hrow(2 * m + 4);
          float* o = c + m * cs + co + 2 * p;
          o[0] = reduce5(h0.x + h4.x, h1.x + h3.x, h2.x);
          o[1] = reduce5(h0.y + h4.y, h1.y + h3.y, h2.y);
          h0 = h2; h1 = h3; h2 = h4;
        }
      }
    }
    __syncthreads();
    // L = G - EXPAND(coarse), four columns and two rows a thread
    const int rq = tid >> (4 - d), mm = tid & ((16 >> d) - 1);
    if (img & (lv.lw_w > 0) & (rq < (16 >> d))) {
      float4 eh[3];
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        const float* r = c + (cy - 1 + rq + u) * cs + cx - 1 + 2 * mm;
        const float2 lo = {r[0], r[1]}, hi = {r[2], r[3]};
        eh[u].x = exp_h(lo.x + hi.x, lo.y);
        eh[u].y = 0.5f * (lo.y + hi.x);
        eh[u].z = exp_h(lo.y + hi.y, hi.x);
        eh[u].w = 0.5f * (hi.x + hi.y);
      }
#pragma unroll 1
      for (int yy = 0; yy < 2; ++yy) {
        const int y = (Y0 >> d) + 2 * rq + yy - lv.lw_y;
        if ((y < 0) | (y >= lv.lw_h)) continue;
        const float4 gv = *reinterpret_cast<const float4*>(f + (fy + 2 * rq + yy) * fs + fx + 4 * mm);
        float l[4];
        l[0] = yy ? band_odd(gv.x, eh[1].x + eh[2].x, 0, T()) : gv.x - exp_v(eh[0].x + eh[2].x, eh[1].x);
        l[1] = yy ? band_odd(gv.y, eh[1].y + eh[2].y, 1, T()) : gv.y - exp_v(eh[0].y + eh[2].y, eh[1].y);
        l[2] = yy ? band_odd(gv.z, eh[1].z + eh[2].z, 2, T()) : gv.z - exp_v(eh[0].z + eh[2].z, eh[1].z);
        l[3] = yy ? band_odd(gv.w, eh[1].w + eh[2].w, 3, T()) : gv.w - exp_v(eh[0].w + eh[2].w, eh[1].w);
        store4(mg<T>(lv.l_out) + slot * lv.l_plane + y * lv.l_row, (X0 >> d) + 4 * mm - lv.lw_x, lv.lw_w, l);
      }
    }
    // the tile's own coarse samples, four columns a thread (waves 0 and 1; above the finest
    // level, where wave 0 has the band, wave 1)
    {
      const int e = d == 0 ? tid : tid - 64;
      const int i = e >> (3 - d), m = e & ((8 >> d) - 1), y = (Y0 >> (d + 1)) + i - lv.croi_y;
      if ((e >= 0) & (i < (16 >> d)) & (y >= 0) & (y < lv.croi_h)) {
        const float* q = c + (cy + i) * cs + cx + 4 * m;
        const float v[4] = {q[0], q[1], q[2], q[3]};
        GLB T* out = img ? mg<T>(lv.g_out) + slot * lv.g_plane + y * lv.g_row : mg<T>(lv.gm_out) + y * lv.gm_row;
        store4(out, (X0 >> (d + 1)) + 4 * m - lv.croi_x, lv.croi_w, v);
      }
    }
    if (d + 1 == depth) break;
    // the next REDUCE's input: samples as stored, 0 outside the level's region, reflect-101
    // outside its canvas (a reflected position beyond the window feeds nothing that is kept:
    // clamped into it); a wave's rows are all read before any is written
    {
      const TailLevel nx = ld_cst(it.lev + d + 1);
      const int x0 = (X0 >> (d + 1)) - cx, y0 = (Y0 >> (d + 1)) - cy;
      const int x = fold_loop(x0 + min(lane, cs - 1), nx.w), xc = min(max(x - x0, 0), cs - 1);
      const bool xin = x >= nx.roi_x && x < nx.roi_x + nx.roi_w;
      constexpr int NR = 5;
#pragma unroll 1
      for (int r0 = wv; r0 < cr; r0 += 4 * NR) {
        float v[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
          const int y = fold_loop(y0 + min(r0 + 4 * i, cr - 1), nx.h);
          v[i] = c[min(max(y - y0, 0), cr - 1) * cs + xc];
          v[i] = xin & (y >= nx.roi_y) & (y < nx.roi_y + nx.roi_h) ? as_stored(v[i], T()) : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < NR; ++i)
          if ((lane < cs) & (r0 + 4 * i < cr)) g[(r0 + 4 * i) * cs + lane] = v[i];
      }
    }
    __syncthreads();
    f = g;
    c += cr * cs;
    fs = cs; fr = cr; fx = cx; fy = cy;
  }
}

// ------------------------------------------------------------------------------------
// stitch_pyramid's level 0 where no level is reduced from it in the same launch: four adjacent samples
// of one row and channel a thread, converted as k_tail converts them.  Bound by memory: three
// channels of 4000x3000, FP16, 25.5 us (38 with a sample a thread, 68 as a k_tail of no steps, which
// stages the halo of three); FP32 47 (67 and 78); 8192x4096 bytes to FP16 19.7 (53 and 72).
template <typename T, bool U8>
__global__ void __launch_bounds__(kThreads) k_level0(const void* __restrict__ s, int64_t srow, int64_t splane,
                                                     T* __restrict__ d, int64_t drow, int64_t dplane, int w, int h) {
  const int x = 4 * ((int)blockIdx.x * 64 + ((int)threadIdx.x & 63));
  const int y = (int)blockIdx.y * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (x >= w || y >= h) return;
  const int64_t from = (int64_t)blockIdx.z * splane + (int64_t)y * srow + x;
  GLB T* to = mg<T>(d) + (int64_t)blockIdx.z * dplane + (int64_t)y * drow + x;
  if (x + 3 < w) {
    float v[4];
    if (U8) {
      const uint32_t b = *reinterpret_cast<const GLB u32_unaligned*>(cg<uint8_t>(s) + from);
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = byte_as_stored((b >> (8 * u)) & 255u, T());
    } else {
      Quad<T> q;
      q.load(cg<T>(s) + from);
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = q.at(u);
    }
    store4_any(to, v);
  } else {
    for (int u = 0; x + u < w; ++u)
      stg(to, u, U8 ? one_sample(cg<uint8_t>(s), from + u, T()) : one_sample(cg<T>(s), from + u, T()));
  }
}

// ------------------------------------------------------------------------------------
// The small levels' collapse in one launch, bit for bit k_blend's level by level: a workgroup
// of 512 takes a 64x16 tile of the finest level and, beside it, the windows of the coarser
// levels its EXPANDs reach (34x10, 19x7, 11x5).  Every level's B is independent of the others',
// so all are read at once -- chunks of 64 samples of a coarse level per wave -- and only the
// collapse, in LDS, goes level by level.  Four launches of 5-7 us each (VGA pair, levels 4 .. 1)
// become one of 10.4 us; four 1080p cameras' panorama, levels 5 .. 2: 24.7 -> 14.4 us.
constexpr int kBtThreads = 512;
constexpr int kBw[4] = {64, 34, 19, 11}, kBh[4] = {16, 10, 7, 5}, kBs[4] = {0, 35, 20, 12};

constexpr int kB1 = 3 * kBh[1] * kBs[1], kB2 = 3 * kBh[2] * kBs[2], kB3 = 3 * kBh[3] * kBs[3];

// Coarse sample (of m) that coarse position i stands for in EXPAND to n fine samples: 2i folded
// by reflect-101, halved -- for the positions a window reaches, -1 .. m (beyond m nothing is
// used).
__device__ __forceinline__ int coarse_at(int i, int n, int m) { return i < 0 ? 1 : i >= m ? m - 1 - (n & 1) : i; }

// Value at (x, y) of EXPAND of one channel's window r (stride st; its entry (0, 0) is coarse
// position (bx, by), nx x ny entries), rows first combined horizontally, as k_blend does.
__device__ __forceinline__ float expand_from(const float* r, int st, int nx, int ny, int bx, int by, int x, int y) {
  const int q = (x >> 1) - bx, p = (y >> 1) - by;
  const int c0 = min(max(q - 1, 0), nx - 1), c1 = min(max(q, 0), nx - 1), c2 = min(max(q + 1, 0), nx - 1);
  const int cl = (x & 1) ? c1 : c0;
  float m[3], n[3], o[3], e[3];
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const float* row = r + min(max(p - 1 + u, 0), ny - 1) * st;
    o[u] = row[cl];
    m[u] = row[c1];
    n[u] = row[c2];
  }
#pragma unroll
  for (int u = 0; u < 3; ++u) e[u] = (x & 1) ? 0.5f * (o[u] + n[u]) : exp_h(o[u] + n[u], m[u]);
  const float s = ((y & 1) ? e[1] : e[0]) + e[2];
  return (y & 1) ? 0.5f * s : exp_v(s, e[1]);
}

template <typename T, bool FINAL, bool KARG>
__global__ void __launch_bounds__(kBtThreads) k_blend_tail(const BlendTailItem one,
                                                           const BlendTailItem* __restrict__ items, int nitems,
                                                           PanoArg po) {
  __shared__ float sB[kB1 + kB2 + kB3];       // levels 1, 2, 3: [channel][row][column]
  const int tid = threadIdx.x;
  const int t = (int)blockIdx.x;
  const CST BlendTailItem* itp;
  if (KARG) {
    itp = first_arg<BlendTailItem>();
  } else {
    int lo = 0, hi = nitems - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (cst(items)[mid].tile_begin <= t) lo = mid; else hi = mid - 1;
    }
    itp = cst(items) + lo;
  }
  const CST BlendTailItem& it = *itp;
  touch(itp);
  const int lt = t - it.tile_begin, tyi = lt / it.tiles_x, txi = lt - tyi * it.tiles_x;
  const int X0 = txi * kBlendTX, Y0 = tyi * kBlendTY;
  const int depth = it.depth;
  const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);

  // B at canvas position (x, y) of a level, one camera: raw samples from an address valid for
  // any (x, y), used later
  using RawT = typename RawOf<T>::type;
  struct Smp {
    RawT l[3];
    uint32_t w;
    bool in, u8;
  };
  auto fetch = [&](const BlendCam& c, int x, int y, Smp& s) __attribute__((always_inline)) {
    const GLB T* l = cg<T>(c.lap);
    const int lx = x - c.lx, wx = x - c.wx, ly = y - c.ly, wy = y - c.wy;
    s.in = (x >= c.vx0) & (x < c.vx1) & (y >= c.vy0) & (y < c.vy1);
    const uint32_t loff = s.in ? __umul24((uint32_t)ly, (uint32_t)c.lap_row) + (uint32_t)lx : 0u;
    const uint32_t woff = s.in ? __umul24((uint32_t)wy, (uint32_t)c.wgt_row) + (uint32_t)wx : 0u;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) s.l[ch] = ld_raw(l, (uint32_t)ch * (uint32_t)c.lap_plane + loff);
    s.u8 = c.wgt_u8 != 0;
    s.w = s.u8 ? (uint32_t)cg<uint8_t>(c.wgt)[woff] : (uint32_t)ld_raw(cg<T>(c.wgt), woff);
  };
  auto add = [&](const Smp& s, float acc[3]) __attribute__((always_inline)) {
    const float w = !s.in ? 0.0f : s.u8 ? (float)s.w * kInv255 : from_raw((RawT)s.w);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) acc[ch] = __builtin_fmaf(w, s.in ? from_raw(s.l[ch]) : 0.0f, acc[ch]);
  };

  // ---- B of every level ----
  // The cameras of every level whose band and weights meet the tile (lane i tests camera i),
  // all levels' rectangles read together.
  auto hits = [&](auto lc) __attribute__((always_inline)) -> uint64_t {
    constexpr int l = decltype(lc)::value;
    const CST BlendItem& a = it.lev[min(l, depth)];
    const int x0 = (X0 >> l) - (l ? 2 : 0), y0 = (Y0 >> l) - (l ? 2 : 0);
    const CST BlendCam& c = cst(a.cams)[min(lane, max(a.ncam - 1, 0))];
    const bool h = (lane < a.ncam) & (c.vx0 < x0 + kBw[l] + 2) & (c.vx1 > x0) & (c.vy0 < y0 + kBh[l] + 2) & (c.vy1 > y0);
    return __ballot(h);
  };
  const uint64_t hit0 = hits(Rows<0>()), hit1 = hits(Rows<1>()), hit2 = hits(Rows<2>()), hit3 = hits(Rows<3>());
  // Coarse windows: entry (i, j) of level l stands for coarse position (X0 >> l) - 1 + j, row
  // (Y0 >> l) - 1 + i, folded through the finer level's reflect-101 into the level.  A wave
  // takes chunks wv and wv + 8 of 64 entries; with its rows of the finest level that is three
  // positions a lane, whose first cameras' samples are all in flight together.
  constexpr int N1 = (kBw[1] * kBh[1] + 63) / 64, N2 = (kBw[2] * kBh[2] + 63) / 64, N3 = (kBw[3] * kBh[3] + 63) / 64;
  const int nchunk = N1 + (depth > 1 ? N2 : 0) + (depth > 2 ? N3 : 0);
  static_assert(N1 + N2 + N3 <= 2 * (kBtThreads / 64), "two chunks a wave");
  struct Job {
    int l, x, y;          // level, position in it
    float* out;           // its LDS entry, channel stride `step`
    int step;
    uint64_t cams;
  };
  auto job = [&](int chunk) __attribute__((always_inline)) {
    Job j;
    j.l = chunk < N1 ? 1 : chunk < N1 + N2 ? 2 : 3;
    const int w = j.l == 1 ? kBw[1] : j.l == 2 ? kBw[2] : kBw[3], h = j.l == 1 ? kBh[1] : j.l == 2 ? kBh[2] : kBh[3];
    const int st = j.l == 1 ? kBs[1] : j.l == 2 ? kBs[2] : kBs[3];
    const int first = chunk - (j.l == 1 ? 0 : j.l == 2 ? N1 : N1 + N2);
    float* sb = sB + (j.l == 1 ? 0 : j.l == 2 ? kB1 : kB1 + kB2);
    j.cams = j.l == 1 ? hit1 : j.l == 2 ? hit2 : hit3;
    const CST BlendItem& a = it.lev[j.l];
    const CST BlendItem& f = it.lev[j.l - 1];
    const int e = min(first * 64 + lane, w * h - 1);
    const int r = j.l == 1 ? e / kBw[1] : j.l == 2 ? e / kBw[2] : e / kBw[3], c = e - r * w;
    j.x = coarse_at((X0 >> j.l) - 1 + c, f.W, a.W);
    j.y = coarse_at((Y0 >> j.l) - 1 + r, f.H, a.H);
    j.out = sb + r * st + c;
    j.step = h * st;
    return j;
  };
  const CST BlendItem& a0 = it.lev[0];
  const int X = X0 + lane, Yw = Y0 + 2 * wv;       // this thread: column X, rows Yw, Yw + 1
  const Job ja = job(min(wv, nchunk - 1)), jb = job(min(wv + kBtThreads / 64, nchunk - 1));
  const bool has_b = wv + kBtThreads / 64 < nchunk;      // uniform over the wave
  float va[3] = {0.0f, 0.0f, 0.0f}, vb[3] = {0.0f, 0.0f, 0.0f}, acc[2][3] = {};
  {
    // each turn: the next camera of each position, every sample read before any is used
    uint64_t ra = ja.cams, rb = has_b ? jb.cams : 0, rm = hit0;
#pragma unroll 1
    while (ra | rb | rm) {
      Smp sa, sb, s0, s1;
      const bool ca = ra != 0, cb = rb != 0, cm = rm != 0;
      if (ca) fetch(ld_cst(cst(it.lev[ja.l].cams) + (int)__builtin_ctzll(ra)), ja.x, ja.y, sa);
      if (cm) {
        const BlendCam c = ld_cst(cst(a0.cams) + (int)__builtin_ctzll(rm));
        fetch(c, X, Yw, s0);
        fetch(c, X, Yw + 1, s1);
      }
      if (cb) fetch(ld_cst(cst(it.lev[jb.l].cams) + (int)__builtin_ctzll(rb)), jb.x, jb.y, sb);
      if (ca) add(sa, va);
      if (cm) {
        add(s0, acc[0]);
        add(s1, acc[1]);
      }
      if (cb) add(sb, vb);
      ra &= ra - 1;
      rb &= rb - 1;
      rm &= rm - 1;
    }
  }
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) {
    ja.out[ch * ja.step] = va[ch];
    if (has_b) jb.out[ch * jb.step] = vb[ch];
  }
  __syncthreads();

  // ---- collapse, from the top (one body for all levels; a thread takes one channel of an
  //      entry, two at level 1) ----
#pragma unroll 1
  for (int l = depth; l >= 1; --l) {
    const BlendItem a = ld_cst(it.lev + l);     // every field at once, none behind a test
    const int fW = it.lev[l - 1].W, fH = it.lev[l - 1].H;
    const int w = l == 1 ? kBw[1] : l == 2 ? kBw[2] : kBw[3], h = l == 1 ? kBh[1] : l == 2 ? kBh[2] : kBh[3];
    const int st = l == 1 ? kBs[1] : l == 2 ? kBs[2] : kBs[3];
    const int nw = l == 1 ? kBw[2] : kBw[3], nh = l == 1 ? kBh[2] : kBh[3], ns = l == 1 ? kBs[2] : kBs[3];
    float* sb = sB + (l == 1 ? 0 : l == 2 ? kB1 : kB1 + kB2);
    const int iw = l == 1 ? 1928 : l == 2 ? 3450 : 5958;          // ceil(65536 / w)
#pragma unroll 1
    for (int e = tid; e < 3 * w * h; e += kBtThreads) {
      const int q = (e * iw) >> 16, c = e - q * w;                // q = e / w: channel and row
      const int ch = (q >= h ? 1 : 0) + (q >= 2 * h ? 1 : 0), r = q - ch * h;
      const int ox = (X0 >> l) - 1 + c, oy = (Y0 >> l) - 1 + r;
      float* p = sb + q * st + c;
      float v = *p;
      if (l < depth) {
        const int x = coarse_at(ox, fW, a.W), y = coarse_at(oy, fH, a.H);
        v = settled(v + expand_from(sb + 3 * h * st + ch * nh * ns, ns, nw, nh, (X0 >> (l + 1)) - 1,
                                    (Y0 >> (l + 1)) - 1, x, y));
      }
      if ((c >= 1) & (c <= (kBlendTX >> l)) & (r >= 1) & (r <= (kBlendTY >> l)) & (ox < a.W) & (oy < a.H) &
          (a.r_out != nullptr))
        stg(mg<T>(a.r_out), ch * a.rout_plane + (int64_t)oy * a.rout_row + ox, v);
      *p = as_stored(v, T());
    }
    __syncthreads();
  }

  // the finest level: this thread's two rows share their three coarse rows' horizontal EXPAND
  GLB T* ro = mg<T>(a0.r_out);
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) {
    float e[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      // coarse rows wv - 1 .. wv + 1 and columns x / 2 - 1 .. x / 2 + 1 of the tile
      const float* row = sB + (ch * kBh[1] + wv + u) * kBs[1] + (lane >> 1);
      const float m = row[1], sum = row[lane & 1] + row[2];
      e[u] = (lane & 1) ? 0.5f * sum : exp_h(sum, m);
    }
    acc[0][ch] = settled(acc[0][ch] + exp_v(e[0] + e[2], e[1]));
    acc[1][ch] = settled(acc[1][ch] + 0.5f * (e[1] + e[2]));
  }
  if (ro != nullptr) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int Y = Yw + j;
      if (X < a0.W && Y < a0.H) {
        const int64_t off = (int64_t)Y * a0.rout_row + X;
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) stg(ro, ch * a0.rout_plane + off, acc[j][ch]);
      }
    }
  }
  if (FINAL) {
    uint8_t* const pano_ptr = po.ptr ? po.ptr : a0.pano;
    const int64_t pano_row = po.ptr ? po.row : a0.pano_row;
#pragma unroll
    for (int j = 0; j < 2; ++j) put_row(pano_ptr, pano_row, X0, lane, Yw + j, a0.W, a0.H, acc[j]);
  }
}

// ------------------------------------------------------------------------------------
// The warp on its own: 64 x 16 samples a workgroup, a thread four rows of one column, every
// sample's two row reads (eight bytes, the pair of taps in them) issued before any is used.
// Bound by the FP32 arithmetic and the stores; one sample a thread with twelve byte reads took
// 21 us for 2240x1080 FP16, this takes 13.
constexpr int kWarpRows = 4;
template <typename T>
__global__ void __launch_bounds__(kThreads) k_warp(const uint8_t* __restrict__ src, int64_t srow, int w, int h,
                                                   Hinv9 hi, int rx, int ry, T* __restrict__ dst, int64_t drow,
                                                   int64_t dplane, int dw, int dh) {
  const int x = blockIdx.x * 64 + (threadIdx.x & 63);
  const int yb = (blockIdx.y * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)) * kWarpRows;
  if (x >= dw || yb >= dh) return;
  const GLB uint8_t* fr = cg<uint8_t>(src);
  GLB T* const out = mg<T>(dst);
  const int64_t lastc = 3 * (int64_t)w - 8;      // below 0: a row of fewer than eight bytes
  if (lastc < 0) {
    for (int y = yb; y < min(yb + kWarpRows, dh); ++y) {
      float v[3];
      warp_px(src, srow, w, h, hi.h, rx + x, ry + y, v);
#pragma unroll
      for (int c = 0; c < 3; ++c) stg(out, c * dplane + (int64_t)y * drow + x, v[c]);
    }
    return;
  }
  unsigned long long ra[kWarpRows], rb[kWarpRows];
  float fxq[kWarpRows], fyq[kWarpRows];
  uint32_t tapq[kWarpRows];                      // as in k_pyr's general window
  const float Xf = (float)(rx + x);
#pragma unroll
  for (int q = 0; q < kWarpRows; ++q) {
    float px, py;
    bool zpos;
    warp_coords_f(hi.h, Xf, (float)(ry + yb + q), px, py, zpos);
    const bool ok = zpos && px >= -1.0f && px < (float)w && py >= -1.0f && py < (float)h;
    const float xs = ok ? px : 0.0f, ys = ok ? py : 0.0f;
    const float x0f = floorf(xs), y0f = floorf(ys);
    fxq[q] = xs - x0f;
    fyq[q] = ys - y0f;
    const int x0 = (int)x0f, y0 = (int)y0f;
    const bool xa = ok && x0 >= 0, xb = ok && x0 + 1 < w, ya = y0 >= 0, yc = y0 + 1 < h;
    const int64_t c3 = 3 * (int64_t)x0, start = min(max(c3, (int64_t)0), lastc);
    tapq[q] = (uint32_t)(ya && xa) | ((uint32_t)(ya && xb) << 1) | ((uint32_t)(yc && xa) << 2) |
              ((uint32_t)(yc && xb) << 3) | ((uint32_t)((int)(c3 - start) + 3) << 4);
    ra[q] = ld8(fr + (max(y0, 0) * srow + start));
    rb[q] = ld8(fr + (min(y0 + 1, h - 1) * srow + start));
  }
#pragma unroll
  for (int q = 0; q < kWarpRows; ++q) {
    const int sh = (int)(tapq[q] >> 4) - 3;      // byte offset of tap 0: -3 .. 5
    const unsigned long long a = sh >= 0 ? ra[q] >> (8 * sh) : ra[q] << 24;
    const unsigned long long b = sh >= 0 ? rb[q] >> (8 * sh) : rb[q] << 24;
    const float fx = fxq[q], fy = fyq[q], gx = 1.0f - fx, gy = 1.0f - fy;
    const uint32_t tp = tapq[q];
    if (yb + q >= dh) break;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float p00 = (tp & 1u) ? (float)((uint32_t)(a >> (8 * c)) & 255u) : 0.0f;
      const float p01 = (tp & 2u) ? (float)((uint32_t)(a >> (8 * c + 24)) & 255u) : 0.0f;
      const float p10 = (tp & 4u) ? (float)((uint32_t)(b >> (8 * c)) & 255u) : 0.0f;
      const float p11 = (tp & 8u) ? (float)((uint32_t)(b >> (8 * c + 24)) & 255u) : 0.0f;
      stg(out, c * dplane + (int64_t)(yb + q) * drow + x,
          settled((gy * (gx * p00 + fx * p01) + fy * (gx * p10 + fx * p11)) * kInv255));
    }
  }
}

__global__ void __launch_bounds__(kThreads) k_warp_coords(Hinv9 hi, int rx, int ry, float* __restrict__ dst,
                                                          int64_t drow, int64_t dplane, int dw, int dh) {
  const int x = blockIdx.x * 64 + (threadIdx.x & 63);
  const int y = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (x >= dw || y >= dh) return;
  // the warp pass's arithmetic: the shared-reciprocal division where its range holds
  // (z in [2^-10, 2^20], |u|, |v| in [2^-12, 2^44]), the compiler's IEEE divide elsewhere
  const float* h = hi.h;
  const float Xf = (float)(rx + x), Yf = (float)(ry + y);
  float u, v, z;
  {
#pragma clang fp contract(off)
    u = (h[0] * Xf + h[1] * Yf) + h[2];
    v = (h[3] * Xf + h[4] * Yf) + h[5];
    z = (h[6] * Xf + h[7] * Yf) + h[8];
  }
  const bool zpos = z > 0.0f;
  const float au = fabsf(u), av = fabsf(v);
  float sx, sy;
  if (z >= 0x1p-10f && z <= 0x1p20f && au >= 0x1p-12f && au <= 0x1p44f && av >= 0x1p-12f && av <= 0x1p44f) {
    div2_in_range(u, v, z, sx, sy);
  } else {
    sx = u / z;
    sy = v / z;
  }
  const int64_t off = (int64_t)y * drow + x;
  dst[off] = zpos ? sx : __builtin_nanf("");
  dst[dplane + off] = zpos ? sy : __builtin_nanf("");
}

// d = f - EXPAND(coarse) on the fine rectangle (d may be f); both levels are zero outside their
// rectangles; fine-domain reflect-101 on the level-k canvas (W x H).  A thread takes four columns
// (aligned in the canvas, so EXPAND's phases are fixed) by two rows of one channel: three rows of
// four coarse samples, read once.  EXPAND here goes tap by tap in ascending order, rows first, as
// ep3 and a rounded 1/2 (a + b) do.  Bound by memory; one sample a thread with up to nine folded
// taps took 78 us for 2240x1080x3 FP16, this takes 10.6.
__device__ __forceinline__ float ep3(float a, float b, float c) {
  return __builtin_fmaf(0.125f, c, __builtin_fmaf(0.75f, b, 0.125f * a));
}
template <typename T>
__global__ void __launch_bounds__(kThreads) k_expand_sub(const T* f, int64_t frow, int64_t fplane, T* d, int64_t drow,
                                                         int64_t dplane, int fx0, int fy0, int fwid, int fhei,
                                                         const T* __restrict__ g, int64_t grow, int64_t gplane,
                                                         int gx0, int gy0, int gwid, int ghei, int W, int H) {
  const int X = (fx0 & ~3) + 4 * (blockIdx.x * 64 + (threadIdx.x & 63));
  const int Y = (fy0 & ~1) + 2 * (blockIdx.y * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6));
  if (X >= fx0 + fwid || Y >= fy0 + fhei) return;
  const int ch = blockIdx.z;
  const GLB T* gc = cg<T>(g) + ch * gplane;
  int cx[4];
  bool xin[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    cx[u] = (fold(X - 2 + 2 * u, W) >> 1) - gx0;
    xin[u] = cx[u] >= 0 && cx[u] < gwid;
    cx[u] = xin[u] ? cx[u] : 0;
  }
  using RawT = typename RawOf<T>::type;
  RawT raw[3][4];
  bool yin[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const int cy = (fold(Y - 2 + 2 * r, H) >> 1) - gy0;
    yin[r] = cy >= 0 && cy < ghei;
    const GLB T* row = gc + (yin[r] ? cy : 0) * grow;
#pragma unroll
    for (int u = 0; u < 4; ++u) raw[r][u] = ld_raw(row, cx[u]);
  }
  // the fine samples, all in the rectangle and aligned as a vector or one by one
  const int x = X - fx0;
  const bool full = x >= 0 && x + 3 < fwid;
  float fv[2][4];
#pragma unroll
  for (int yy = 0; yy < 2; ++yy) {
    const int y = Y + yy - fy0;
    if (y < 0 || y >= fhei) continue;
    const GLB T* p = cg<T>(f) + ch * fplane + y * frow;
    if (full && ((uintptr_t)(p + x) & (4 * sizeof(T) - 1)) == 0) {
      load4(p + x, fv[yy]);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) fv[yy][u] = from_raw(ld_raw(p, min(max(x + u, 0), fwid - 1)));
    }
  }
  float h[3][4];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    float c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) c[u] = yin[r] && xin[u] ? from_raw(raw[r][u]) : 0.0f;
    h[r][0] = ep3(c[0], c[1], c[2]);
    h[r][1] = 0.5f * (c[1] + c[2]);
    h[r][2] = ep3(c[1], c[2], c[3]);
    h[r][3] = 0.5f * (c[2] + c[3]);
  }
#pragma unroll
  for (int yy = 0; yy < 2; ++yy) {
    const int y = Y + yy - fy0;
    if (y < 0 || y >= fhei) continue;
    float l[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      l[u] = settled(fv[yy][u] - settled(yy ? 0.5f * (h[1][u] + h[2][u]) : ep3(h[0][u], h[1][u], h[2][u])));
    store4(mg<T>(d) + ch * dplane + y * drow, x, fwid, l);
  }
}

// Workgroups of a persistent launch: at most wg_per_cu per compute unit (0: as many as
// fit; negative: one per tile), never more than there are tiles.  The occupancy query
// runs once per kernel.
int persistent_grid(const void* kernel, int tiles, int wg_per_cu) {
  static thread_local const void* cached_k[16] = {};
  static thread_local int cached_cus[16] = {}, cached_per[16] = {};
  int slot = -1;
  for (int i = 0; i < 16; ++i)
    if (cached_k[i] == kernel || cached_k[i] == nullptr) { slot = i; break; }
  if (slot < 0) slot = 0;
  if (cached_k[slot] != kernel) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) !=
        hipSuccess || hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, kThreads, 0) != hipSuccess ||
        cus <= 0 || per <= 0) {
      cus = 256;
      per = 2;
    }
    cached_k[slot] = kernel;
    cached_cus[slot] = cus;
    cached_per[slot] = per;
  }
  if (wg_per_cu < 0) return tiles;
  const int per = wg_per_cu > 0 && wg_per_cu < cached_per[slot] ? wg_per_cu : cached_per[slot];
  const int n = cached_cus[slot] * per;
  return tiles < n ? tiles : n;
}

}  // namespace

// ------------------------------------------------------------------------------------ launchers
hipError_t launch_pyr(bool f16, bool warp, const PyrItem* items_dev, int nitems, int total_tiles,
                      const FrameArgs& fa, hipStream_t s, int wg_per_cu) {
  if (total_tiles <= 0) return hipSuccess;
  const dim3 grid(total_tiles), block(kThreads);
#define STITCH_PYR(TT)                                                                                          \
  do {                                                                                                          \
    if (warp) {                                                                                                 \
      const dim3 g(persistent_grid((const void*)k_pyr<TT, true>, total_tiles, wg_per_cu));                             \
      hipLaunchKernelGGL((k_pyr<TT, true>), g, block, 0, s, items_dev, nitems, total_tiles, fa);               \
    } else {                                                                                                    \
      const dim3 g(persistent_grid((const void*)k_pyr<TT, false>, total_tiles, wg_per_cu));                            \
      hipLaunchKernelGGL((k_pyr<TT, false>), g, block, 0, s, items_dev, nitems, total_tiles, fa);              \
    }                                                                                                           \
  } while (0)
  if (f16) STITCH_PYR(_Float16);
  else STITCH_PYR(float);
#undef STITCH_PYR
  return hipGetLastError();
}

void prepare_launches() {
  // fill the occupancy cache outside any stream capture
  persistent_grid((const void*)k_pyr<float, true>, 1, 0);
  persistent_grid((const void*)k_pyr<float, false>, 1, 0);
  persistent_grid((const void*)k_pyr<_Float16, true>, 1, 0);
  persistent_grid((const void*)k_pyr<_Float16, false>, 1, 0);
}

hipError_t launch_blend(bool f16, bool final_level, const BlendItem* items_dev, int nitems, int total_tiles,
                        const PanoArg& po, hipStream_t s, const BlendItem* one) {
  if (total_tiles <= 0) return hipSuccess;
  const dim3 grid(total_tiles), block(kThreads);
  BlendItem k1;
  if (one) k1 = *one;
  else std::memset(&k1, 0, sizeof k1);
#define STITCH_BLEND(TT, FIN)                                                                                    \
  do {                                                                                                           \
    if (one) hipLaunchKernelGGL((k_blend<TT, FIN, true>), grid, block, 0, s, items_dev, nitems, k1, po);          \
    else hipLaunchKernelGGL((k_blend<TT, FIN, false>), grid, block, 0, s, items_dev, nitems, k1, po);             \
  } while (0)
  if (f16) {
    if (final_level) STITCH_BLEND(_Float16, true);
    else STITCH_BLEND(_Float16, false);
  } else {
    if (final_level) STITCH_BLEND(float, true);
    else STITCH_BLEND(float, false);
  }
#undef STITCH_BLEND
  return hipGetLastError();
}

hipError_t launch_tail(bool f16, const TailItem* items_dev, int nitems, int total_tiles, int nslot, hipStream_t s,
                       const TailItem* one) {
  if (total_tiles <= 0 || nslot <= 0) return hipSuccess;
  const dim3 grid(total_tiles * nslot), block(kThreads);
  TailItem k1;
  if (one) k1 = *one;
  else std::memset(&k1, 0, sizeof k1);
#define STITCH_TAIL(TT)                                                                                  \
  do {                                                                                                   \
    if (one) hipLaunchKernelGGL((k_tail<TT, true>), grid, block, 0, s, k1, items_dev, nitems, nslot);    \
    else hipLaunchKernelGGL((k_tail<TT, false>), grid, block, 0, s, k1, items_dev, nitems, nslot);       \
  } while (0)
  if (f16) STITCH_TAIL(_Float16);
  else STITCH_TAIL(float);
#undef STITCH_TAIL
  return hipGetLastError();
}

hipError_t launch_blend_tail(bool f16, bool final_level, const BlendTailItem* items_dev, int nitems, int total_tiles,
                             const PanoArg& po, hipStream_t s, const BlendTailItem* one) {
  if (total_tiles <= 0) return hipSuccess;
  const dim3 grid(total_tiles), block(kBtThreads);
  BlendTailItem k1;
  if (one) k1 = *one;
  else std::memset(&k1, 0, sizeof k1);
#define STITCH_BTAIL(TT, FIN, KA) \
  hipLaunchKernelGGL((k_blend_tail<TT, FIN, KA>), grid, block, 0, s, k1, items_dev, nitems, po)
  if (!one) {                        // a batch's middle levels
    if (f16) STITCH_BTAIL(_Float16, false, false);
    else STITCH_BTAIL(float, false, false);
  } else if (f16) {
    if (final_level) STITCH_BTAIL(_Float16, true, true);
    else STITCH_BTAIL(_Float16, false, true);
  } else {
    if (final_level) STITCH_BTAIL(float, true, true);
    else STITCH_BTAIL(float, false, true);
  }
#undef STITCH_BTAIL
  return hipGetLastError();
}

hipError_t launch_warp(bool f16, const uint8_t* src, int64_t src_row, int w, int h, const float* hinv9, int roi_x,
                       int roi_y, void* dst, int64_t dst_row, int64_t dst_plane, int dw, int dh, hipStream_t s) {
  if (dw <= 0 || dh <= 0) return hipSuccess;
  Hinv9 hi;
  for (int i = 0; i < 9; ++i) hi.h[i] = hinv9[i];
  const dim3 grid((dw + 63) / 64, (dh + 4 * kWarpRows - 1) / (4 * kWarpRows)), block(kThreads);
  if (f16)
    hipLaunchKernelGGL((k_warp<_Float16>), grid, block, 0, s, src, src_row, w, h, hi, roi_x, roi_y, (_Float16*)dst,
                       dst_row, dst_plane, dw, dh);
  else
    hipLaunchKernelGGL((k_warp<float>), grid, block, 0, s, src, src_row, w, h, hi, roi_x, roi_y, (float*)dst,
                       dst_row, dst_plane, dw, dh);
  return hipGetLastError();
}

hipError_t launch_warp_coords(const float* hinv9, int roi_x, int roi_y, float* dst, int64_t row, int64_t plane,
                              int dw, int dh, hipStream_t s) {
  if (dw <= 0 || dh <= 0) return hipSuccess;
  Hinv9 hi;
  for (int i = 0; i < 9; ++i) hi.h[i] = hinv9[i];
  const dim3 grid((dw + 63) / 64, (dh + 3) / 4), block(kThreads);
  hipLaunchKernelGGL(k_warp_coords, grid, block, 0, s, hi, roi_x, roi_y, dst, row, plane, dw, dh);
  return hipGetLastError();
}

hipError_t launch_level0(bool f16, bool u8, int nch, const Planes& src, const Planes& out, int w, int h, hipStream_t s) {
  const dim3 grid((w + 255) / 256, (h + 3) / 4, nch), block(kThreads);
#define STITCH_LEVEL0(TT, U)                                                                                         \
  hipLaunchKernelGGL((k_level0<TT, U>), grid, block, 0, s, src.data, src.row, src.plane, (TT*)out.data, out.row, out.plane, w, h)
  if (f16) {
    if (u8) STITCH_LEVEL0(_Float16, true);
    else STITCH_LEVEL0(_Float16, false);
  } else {
    if (u8) STITCH_LEVEL0(float, true);
    else STITCH_LEVEL0(float, false);
  }
#undef STITCH_LEVEL0
  return hipGetLastError();
}

hipError_t launch_expand_sub(bool f16, int nch, const Planes& fine, const Planes& out, int fx, int fy, int fw, int fh,
                             const Planes& coarse, int cx, int cy, int cw, int ch, int canvas_w, int canvas_h,
                             hipStream_t s) {
  if (fw <= 0 || fh <= 0) return hipSuccess;
  const int gw = (fw + (fx & 3) + 3) / 4, gh = (fh + (fy & 1) + 1) / 2;       // threads
  const dim3 grid((gw + 63) / 64, (gh + 3) / 4, nch), block(kThreads);
#define STITCH_EXPAND(TT)                                                                                             \
  hipLaunchKernelGGL((k_expand_sub<TT>), grid, block, 0, s, (const TT*)fine.data, fine.row, fine.plane, (TT*)out.data, \
                     out.row, out.plane, fx, fy, fw, fh, (const TT*)coarse.data, coarse.row, coarse.plane, cx, cy, cw, \
                     ch, canvas_w, canvas_h)
  if (f16) STITCH_EXPAND(_Float16);
  else STITCH_EXPAND(float);
#undef STITCH_EXPAND
  return hipGetLastError();
}

}  // namespace stitch
