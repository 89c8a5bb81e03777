// Internal descriptors shared by the host runtime (stitch_api.cpp) and the gfx950
// kernels (kernels.hip).  Plain structs: they are copied to device memory or passed
// as kernel arguments.
#pragma once
#include <stdint.h>
#include <hip/hip_runtime.h>

#include <new>

#include "stitch.h"

namespace stitch {

constexpr int kMaxLevels = 16;
constexpr int kMaxCameras = 64;

// Tile shape of the fused pyramid pass and of the blend pass (level-k pixels).
constexpr int kPyrTX = 64, kPyrTY = 16;
constexpr int kBlendTX = 64, kBlendTY = 16;
constexpr int kThreads = 256;

struct Hinv9 { float h[9]; };

// One camera's tile range in a fused REDUCE (+ EXPAND/subtract) pass from level k
// to level k+1.  Level-k input covers roi (zero outside it, reflect-101 at canvas
// edges) except for a warp source, which is evaluated wherever it is needed.
struct PyrItem {
  int32_t tile_begin, tiles_x, tiles_y;
  int32_t tile_x0, tile_y0;               // level-k origin of tile (0,0); both even
  int32_t fine_w, fine_h;                 // level-k canvas sides
  int32_t roi_x, roi_y, roi_w, roi_h;     // level-k input rectangle
  // image source: three planes, or at level 0 the warped frame
  const void* img;                        // planes (storage type) or u8 HWC frame
  int64_t img_row, img_plane;             // elements (planes) / bytes (frame row)
  int32_t frame_w, frame_h, frame_slot, pad0;
  float hinv[9];
  // weight (mask) source, one channel
  const void* msk;                        // u8 plane (level 0) or storage-type plane on roi
  int64_t msk_row;                        // elements
  // outputs at level k+1 on croi
  int32_t croi_x, croi_y, croi_w, croi_h;
  void* g_out;  int64_t g_row, g_plane;   // nch planes
  void* gm_out; int64_t gm_row;           // 1 plane
  // Laplacian band at level k on the window lw (w == 0: not written)
  int32_t lw_x, lw_y, lw_w, lw_h;
  void* l_out;  int64_t l_row, l_plane;
  // a tile is kPyrTX columns by sub * kPyrTY rows; rows16 = 16-row blocks of the item
  int32_t sub, rows16;
};

// Per-call frame pointers of the fused level-0 pass (kernel argument).
struct FrameArgs {
  int32_t n, pad;
  const uint8_t* ptr[kMaxCameras];
  int64_t row[kMaxCameras];               // bytes
};

// One camera's contribution to a blend level.
struct BlendCam {
  const void* lap; int64_t lap_row, lap_plane;   // storage type, 3 planes
  int32_t lx, ly, lw, lh;                         // band rectangle (level-k canvas)
  const void* wgt; int64_t wgt_row;               // weights: storage type or u8
  int32_t wgt_u8, pad;
  int32_t wx, wy, ww, wh;                         // weight rectangle
  int32_t vx0, vy0, vx1, vy1;                     // where both are (half open; the blend tail's tests)
};

// One canvas level of one stitch job in a blend launch; a launch covers the tiles of
// several items (jobs), tile_begin being each item's first tile.
struct BlendItem {
  int32_t tile_begin, tiles_x, tiles_y;
  int32_t W, H;                     // level-k canvas sides
  int32_t cW, cH;                   // level-(k+1) canvas sides (used when has_coarse)
  int32_t ncam, has_coarse, pad;
  const BlendCam* cams;             // device array of ncam cameras
  const void* r_in; int64_t rin_row, rin_plane;    // R_{k+1} (storage type)
  void* r_out; int64_t rout_row, rout_plane;       // R_k (storage type) or nullptr
  uint8_t* pano; int64_t pano_row;                 // U8 HWC (level 0) or nullptr
};

// Several consecutive small levels in one launch (the tail of a pyramid): level k of a tail
// is REDUCEd to k+1 and its band stored, from samples the workgroup holds itself.
constexpr int kTailTX = 64, kTailTY = 32;   // tile of the tail's finest level
constexpr int kTailDepth = 3;               // levels a tail reduces at most
struct TailLevel {
  int32_t w, h;                           // level-k canvas sides
  int32_t roi_x, roi_y, roi_w, roi_h;     // level-k samples outside count 0
  int32_t croi_x, croi_y, croi_w, croi_h; // stored rectangle of level k+1
  void* g_out; int64_t g_row, g_plane;    // image planes (elements)
  void* gm_out; int64_t gm_row;           // weight plane
  int32_t lw_x, lw_y, lw_w, lw_h;         // band window of level k (w == 0: not stored)
  void* l_out; int64_t l_row, l_plane;
};
struct TailItem {
  int32_t tile_begin, tiles_x, depth, nch;
  int32_t tile_x0, tile_y0;               // finest-level origin of tile (0,0), multiples of 2^depth
  int32_t src_u8;                         // the image source is bytes (read as u8/255)
  int32_t pad;
  const void* img; int64_t img_row, img_plane;   // finest-level image planes on lev[0].roi
  const void* msk; int64_t msk_row;              // finest-level weight plane (slot nch)
  void* copy_out; int64_t copy_row, copy_plane;  // NULL, or where the finest level is copied
  TailLevel lev[kTailDepth];
};
// Collapse of the levels lev[depth] (the top) .. lev[0] of one panorama in one launch.
struct BlendTailItem {
  int32_t tile_begin, tiles_x, depth, pad;
  BlendItem lev[kTailDepth + 1];
};

// Launchers (kernels.hip).  f16 selects half-precision storage.
// warp: level-0 pass whose image source is the homography warp.
// wg_per_cu: persistent workgroups per compute unit (0: as many as fit, < 0: one per tile).
hipError_t launch_pyr(bool f16, bool warp, const PyrItem* items_dev, int nitems, int total_tiles,
                      const FrameArgs& frames, hipStream_t s, int wg_per_cu = 0);
// Runs the occupancy queries the launchers cache, so later launches (e.g. inside a stream
// capture) make no device queries.
void prepare_launches();
// Table sizes the kernels accept.
constexpr int kMaxBlendCams = kMaxCameras;
// Per-call panorama of a single-item level-0 launch (kernel argument; ptr == nullptr:
// every item's own pano field is used).
struct PanoArg {
  uint8_t* ptr;
  int64_t row;
};

// final_level: level 0, which writes the uint8 panorama of every item.
// one != nullptr: a single item passed by value (items_dev unused).
hipError_t launch_blend(bool f16, bool final_level, const BlendItem* items_dev, int nitems, int total_tiles,
                        const PanoArg& po, hipStream_t s, const BlendItem* one = nullptr);
// Tails: nslot planes per tile (image channels, then the weight plane); one != nullptr: a
// single item passed by value.  final_level as for launch_blend (lev[0] is level 0).
hipError_t launch_tail(bool f16, const TailItem* items_dev, int nitems, int total_tiles, int nslot, hipStream_t s,
                       const TailItem* one = nullptr);
// (a table of several blend tails: middle levels only)
hipError_t launch_blend_tail(bool f16, bool final_level, const BlendTailItem* items_dev, int nitems, int total_tiles,
                             const PanoArg& po, hipStream_t s, const BlendTailItem* one = nullptr);
hipError_t launch_warp(bool f16, const uint8_t* src, int64_t src_row, int w, int h, const float* hinv9,
                       int roi_x, int roi_y, void* dst, int64_t dst_row, int64_t dst_plane, int dw, int dh,
                       hipStream_t s);
hipError_t launch_warp_coords(const float* hinv9, int roi_x, int roi_y, float* dst, int64_t row,
                              int64_t plane, int dw, int dh, hipStream_t s);
// Planes of one image in the storage type: data, row and plane strides in elements.
struct Planes {
  void* data;
  int64_t row, plane;
};
// out = src, converted where src holds bytes (strides of src in its own elements).
hipError_t launch_level0(bool f16, bool u8, int nch, const Planes& src, const Planes& out, int w, int h, hipStream_t s);
// out = fine - EXPAND(coarse), out's rectangle being fine's (out may be fine).
hipError_t launch_expand_sub(bool f16, int nch, const Planes& fine, const Planes& out, int fx, int fy, int fw, int fh,
                             const Planes& coarse, int cx, int cy, int cw, int ch, int canvas_w, int canvas_h,
                             hipStream_t s);

// Geometry of a plan for the other host files: cameras, their frame sizes (arrays of at
// least kMaxCameras), the canvas, and whether a workspace is bound.
void plan_geometry(const stitch_plan* p, int* n, int* frame_w, int* frame_h, int* canvas_w, int* canvas_h,
                   bool* bound);

// One camera of a plan for the float-frame forward and its vector-Jacobian product: frame
// size, the FP32 canvas -> source map, the seam weights on their support box (wdict: wh
// uint32 row numbers, then rows of ww bytes; empty when the camera has no weight anywhere),
// and per level the region its pyramid needs and the band the blend reads ({x, y, w, h}).
struct PlanCamera {
  int fw, fh;
  float hinv[9];
  int wx, wy, ww, wh;
  const uint8_t* wdict;
  size_t wdict_bytes;
  int roi[kMaxLevels][4], band[kMaxLevels][4];
};
int plan_levels(const stitch_plan* p);
void plan_camera(const stitch_plan* p, int i, PlanCamera* out);

// Host helpers shared by the API files (stitch_api.cpp).
stitch_status fail(stitch_status s, const char* fmt, ...);
stitch_status hip_fail(hipError_t e, const char* what);
// The body of an entry point that takes host memory: running out of it is a status, not an exception
// that leaves through C.  (A message short enough to need no memory itself.)
template <typename F>
stitch_status guarded(F&& body) {
  try {
    return body();
  } catch (const std::bad_alloc&) {
    return fail(STITCH_E_UNSUPPORTED, "no host memory");
  }
}
stitch_status check_image(const stitch_image* im, const char* name, int dtype, int layout, int channels);
bool hinv_spec(const double* H, float out[9], double* sign_out, const char** why);
// Bounding box {x, y, w, h} of the non-zero bytes of a w x h map; false when there is none.
bool weight_box(const uint8_t* m, int w, int h, int box[4]);

}  // namespace stitch
