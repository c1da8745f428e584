// mer_internal.h -- launchers shared between the C-ABI layer and the kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "mer_device.h"

namespace mer {
constexpr int kBinBlock = 256;  // threads per workgroup of the binning passes (one triangle each)

constexpr int kLongList = 4096;  // entries of a coarse tile that one workgroup takes: sixteen rounds, about 40 us
constexpr int kItemBytes = 32;
// Plans of at most so many coarse tiles, with so many triangles for each, keep
// each tile's counters on a cache line of their own: the adds of triangles in
// no order, one for each, went to one line for 16 tiles.  300,000 triangles of 4
// px over 256 tiles 151 us, 59 padded, 1,500,000 over 4096 tiles 250 and 216.
// Clearing and reading padded ones takes 3 us longer for 10,752 tiles, and 1 us
// for 1024 (of 160 triangles).
constexpr int kPaddedTiles = 4096, kPaddedTris = 192;

// The coarse tiles of a plan (small_px > 0) and their regions of the
// workspace, after the last one mer_plan names: mer_plan lies in the caller's
// memory, so its size belongs to the ABI and these are worked out where they
// are used.
struct CoarsePlan {
  int ctl;                       // log2 of the tiles' side
  int64_t n;                     // tiles
  int64_t off_count, off_tile;   // int2 and CTile per tile
  int count_shift;               // log2 of the int2's distance, in int2
  int64_t item, n_items, off_item;  // long lists: entries per part, parts at most, CItem per part
  int64_t end;
};
inline int64_t align256(int64_t x) { return (x + 255) & ~(int64_t)255; }
inline CoarsePlan coarse_plan(const mer_plan* P) {
  CoarsePlan c;
  c.ctl = (int)(P->big_tiles & 255);
  c.n = P->big_tiles >> 8;
  c.off_count = align256(P->off_bigflat + P->total_tris * 4);
  c.count_shift = c.n <= kPaddedTiles && P->total_tris >= kPaddedTris * c.n ? 4 : 0;
  c.off_tile = align256(c.off_count + (c.n * 8 << c.count_shift));
  c.off_item = align256(c.off_tile + c.n * 16);
  // Lists longer than kLongList and than two parts are split (mer_coarse.h).
  // A part is 1024 entries, or as many as make 4096 parts of two entries a
  // triangle; no list of a plan with fewer triangles is as long.  1.8 M
  // triangles over 64 / 200 px of a 2048 x 2048 view, parts of 512, 1024 and
  // 2048 entries: 102 / 167, 102 / 167 and 110 / 159 us.
  c.item = P->total_tris > 2048 * 1024 ? (P->total_tris / 2048 + 255) & ~(int64_t)255 : 1024;
  c.n_items = P->total_tris > kLongList ? (2 * P->total_tris / c.item + 7) & ~(int64_t)7 : 0;
  c.end = align256(c.off_item + c.n_items * kItemBytes);
  return c;
}

// attr/out (nullable): interpolate in the resolve, as launch_interpolate
// would; tail as in ResolveOut
int launch_rasterize(const mer_plan* P, const mer_view* views, const float* v, const int32_t* tri, int32_t* tri_id,
                     float* depth, float* bary, const float* attr, int C_a, int tail, float* out, void* ws,
                     hipStream_t st);
int launch_interpolate(const mer_plan* P, const mer_view* views, const float* attr, int C_a, const float* v,
                       const int32_t* tri, const int32_t* tri_id, const float* bary, int append_z, float* out,
                       hipStream_t st);
int launch_transform(const mer_plan* P, const mer_view* views, const mer_camera* cams, const float* v_world,
                     float* v_screen, void* ws, hipStream_t st);
int launch_transform_bwd(const mer_plan* P, const mer_view* views, const mer_camera* cams, const float* v_world,
                         const float* g_screen, float* g_world, void* ws, hipStream_t st);
int launch_backface(const mer_plan* P, const mer_view* views, const float* v, const int32_t* tri,
                    const int32_t* tri_id, float* out, hipStream_t st);
// g: dL/d(img) rows of ld_g floats, or NULL with target != NULL for the fused
// L2 loss (dL/d(img) = 2 w (img - target), loss += w sum (img - target)^2).
// Scratch: tab, 2 (n_views + 1) int64 (the 16x16 tile prefix per view, written
// here; not for one view); loss_part, total_btiles floats (per-tile loss
// partials, written here; only read when loss != NULL).
int launch_backward(const mer_plan* P, const mer_view* views, const float* v, const int32_t* tri,
                    const int32_t* tri_id, const float* attr, int C_a, int append_z, const float* img,
                    const float* g, const float* target, float w_l2, float* loss, int C_e, int ld_g, int flags,
                    float* g_attr, float* g_v, long long* tab, float* loss_part, hipStream_t st);
// forward-mode image tangent (flags: MER_NO_INTERSECT, MER_SKIP_EDGE, MER_SKIP_INTERP)
int launch_jvp(const mer_plan* P, const mer_view* views, const float* v, const int32_t* tri, const int32_t* tri_id,
               const float* attr, const float* dattr, int C_a, int append_z, const float* img, int C_e,
               const float* dv, int flags, float* dimg, void* ws, hipStream_t st);
// bilinear clamp-to-edge texture sampling and its adjoint
int launch_texture(const mer_plan* P, const mer_view* views, const int32_t* tri_id, const float* uv, int ld_uv,
                   const float* tex, int th, int tw, int C, float* out, hipStream_t st);
int launch_texture_bwd(const mer_plan* P, const mer_view* views, const int32_t* tri_id, const float* uv, int ld_uv,
                       const float* tex, int th, int tw, int C, const float* g_out, float* g_tex, float* g_uv,
                       void* ws, hipStream_t st);
// per-view prefix tables (triangles, tiles of 2^tw_log2 x 2^th_log2) and status reset
__global__ void __launch_bounds__(1024) k_prep(const mer_view* __restrict__ views, int n_views, int tw_log2, int th_log2,
                       long long* __restrict__ tri_base, long long* __restrict__ tile_base,
                       long long* __restrict__ status);
}  // namespace mer
