// mer_coarse.h -- the rasterizer: triangles binned into lists of coarse
// screen tiles (32 x 32, 16 x 16 or 8 x 8 pixels), each tile rasterized by one
// workgroup that sorts its triangles into 8 x 8 pixel tiles in LDS
// (supplement, "Rasterization module" and "Barycentrics module").
//
//   k_cinit    per-view prefix tables, tile counters and status cleared
//   k_ccount   one thread per (view, triangle): snap, cull, box of pixel
//              centres; every coarse tile it may touch is counted, and the
//              count gives the triangle its rank in the tile's list
//   k_clarge   the same for triangles over many tiles, a workgroup each
//   k_calloc   one thread per coarse tile: its range of the bin pool
//   k_cfill    the ranked entries copied to their lists (no tests, no atomics)
//   k_craster  one workgroup per coarse tile, or several where its list is long
//
// What this replaced listed every triangle in 8 x 8 tiles (count, scan, fill)
// and rasterized triangles of at most 16 centres with global atomics: fifteen
// launches, and on rough meshes most of the time went into the lists.  A
// triangle of the rough 2M-triangle meshes touches 4.6 tiles of 8 x 8 pixels
// but 1.9 of 32 x 32, so the lists hold less than half the entries, and a
// triangle is snapped and prepared once per coarse tile.  Measured, rasterize
// and interpolate, before and after (us): 16 views of the 2M-triangle pair
// 11,700 and 5,950 (k_craster 4,600: vector issue 71 % of it, the rest LDS
// latency and barriers; count 740, fill 400); 256 scenes 2,750 and 1,980
// (1,700 + 180 + 95); 64 head views 1,470 and 680 (570 + 70 + 24; its writes
// alone take 440 at the rate of a large copy); one 64 x 64 view 41 and 12.
// The visible triangle is the largest (1/z, ~id) key at every pixel, in any
// order of candidates, so the result does not depend on any of this.
#pragma once
#include "mer_internal.h"
#include "mer_resolve.h"

namespace mer {

constexpr int kSegStride = 8 * kBinBlock;  // ranked entries of one workgroup of the count pass: 8 a triangle
constexpr int kRankBits = 24;              // an entry's rank in its tile's list, beside the 8-bit triangle number
constexpr unsigned kRankMax = (1u << kRankBits) - 1u;

// Coarse tile: its list bins[base, base + n), n < 0 when the list does not
// fit (every triangle of the view is scanned instead); view and tile position.
struct __align__(16) CTile {
  int base, n, view;
  unsigned xy;  // column | row << 16, and the bits below
};
constexpr unsigned kPart = 1u << 31;   // a part of a long list (CItem)
constexpr unsigned kGone = 1u << 15;   // nothing to do: the list is split, or no part

// One part of a long list, as a tile with that part of the entries.  A tile's
// parts lie one after another, each a workgroup of its own; they meet in the
// key image (64-bit maxima in memory), and the one that finishes last writes
// the tile's pixels.  done counts them, in the first.
struct CItem {
  CTile t;
  int part, parts, done, pad;
};
// Per tile: entries counted by rank (x), and by walking (y).
struct Counts {
  int2* p;
  int shift;  // log2 of their distance, in counters
  __device__ __forceinline__ int2& operator[](long long tile) const { return p[tile << shift]; }
};

static_assert(sizeof(CItem) == kItemBytes, "the plan's region of them");

__global__ void __launch_bounds__(1024) k_cinit(const mer_view* __restrict__ views, int n_views, int ctl,
                                                long long* __restrict__ tri_base, long long* __restrict__ tile_base,
                                                long long* __restrict__ status, const Counts count,
                                                long long n_tiles, CItem* __restrict__ items, int n_items) {
  if (blockIdx.x > 0) {  // the first workgroup has the prefixes
    const int step = (int)(gridDim.x - 1) * 1024, t = (int)(blockIdx.x - 1) * 1024 + (int)threadIdx.x;
    for (int i = t; i < n_items; i += step) items[i].t.xy = kGone;
    for (long long i = t; i < n_tiles; i += step) count[i] = make_int2(0, 0);
    return;
  }
  view_prefix(views, n_views, ctl, ctl, tri_base, tile_base, status);
}

// ---------------------------------------------------------------- geometry
struct PixBox {
  int x0, y0, x1, y1;  // inclusive range of pixels whose centres may be covered; x0 > x1 when none
};

// Box of pixel centres of a snapped triangle inside the view: centres
// 256 p + 128 within [min, max] are p in [ceil((min - 128) / 256),
// floor((max - 128) / 256)].
__device__ __forceinline__ PixBox pixel_box(const Snap& s, const mer_view& vw) {
  const int xmin = min(s.X[0], min(s.X[1], s.X[2])), xmax = max(s.X[0], max(s.X[1], s.X[2]));
  const int ymin = min(s.Y[0], min(s.Y[1], s.Y[2])), ymax = max(s.Y[0], max(s.Y[1], s.Y[2]));
  PixBox b;
  b.x0 = max(-((-(xmin - 128)) >> 8), 0);
  b.x1 = min((xmax - 128) >> 8, vw.W - 1);
  b.y0 = max(-((-(ymin - 128)) >> 8), 0);
  b.y1 = min((ymax - 128) >> 8, vw.H - 1);
  if (b.y0 > b.y1) b.x0 = 1, b.x1 = 0;
  return b;
}

// One large triangle's coarse tiles over a workgroup's lanes, or over a wave's
// where there are more triangles than workgroups; f(triangle, tile) for the
// tiles it may cover.  The listed triangles go to the grid's workgroups
// `first`, first + 1, ..., or to their waves, in turn (200,000 triangles over
// about 20 tiles each: k_clarge 86 us by workgroups, 37 by waves).
template <typename F>
__device__ __forceinline__ void walk_large(const mer_view* __restrict__ views, int n_views,
                                           const long long* __restrict__ tri_base,
                                           const long long* __restrict__ tile_base, const float* __restrict__ v,
                                           const int32_t* __restrict__ tri, int ctl, const int* __restrict__ large,
                                           int n_large, int first, F f) {
  const int b0 = (int)blockIdx.x - first, nb = (int)gridDim.x - first;
  const bool waves = n_large > nb;
  const int lanes = waves ? 64 : kBinBlock, lane = threadIdx.x & (lanes - 1);
  const int step = waves ? nb * (kBinBlock / 64) : nb;
  for (int i = waves ? b0 * (kBinBlock / 64) + (threadIdx.x >> 6) : b0; i < n_large; i += step) {
    const int g = __builtin_amdgcn_readfirstlane(large[i]);
    const int vi = __builtin_amdgcn_readfirstlane(find_bucket(tri_base, n_views, g));
    const mer_view vw = views[vi];
    const Snap s = snap_visible(v, vw, tri_row(tri, vw, (int)(g - tri_base[vi])));
    const PixBox b = pixel_box(s, vw);
    const Rec R = make_rec(s);
    const int tx0 = b.x0 >> ctl, ty0 = b.y0 >> ctl, ntx = (b.x1 >> ctl) - tx0 + 1, nty = (b.y1 >> ctl) - ty0 + 1;
    const int tiles_x = (vw.W + (1 << ctl) - 1) >> ctl;
    for (int k = lane; k < ntx * nty; k += lanes) {
      const int dy = (int)((unsigned)k / (unsigned)ntx), tx = tx0 + k - dy * ntx, ty = ty0 + dy;
      if (box_may_cover(R, max(tx << ctl, b.x0), max(ty << ctl, b.y0), min(((tx + 1) << ctl) - 1, b.x1),
                        min(((ty + 1) << ctl) - 1, b.y1)))
        f(g, (int)(tile_base[vi] + (long long)ty * tiles_x + tx));
    }
  }
}

// ------------------------------------------------------------------- count
// Workgroup table of tile counters: neighbouring triangles share tiles, so
// the workgroup counts in LDS and adds each tile's total to memory once; that
// add returns where the workgroup's run starts in the tile's list, and with it
// every entry's rank.
constexpr int kCSlotsLog2 = 9, kCSlots = 1 << kCSlotsLog2, kCProbe = 8;

__device__ __forceinline__ int ctile_slot(int* s_key, int key) {
  const unsigned h = ((unsigned)key * 2654435761u) >> (32 - kCSlotsLog2);
#pragma unroll 1
  for (int probe = 0; probe < kCProbe; ++probe) {
    const int sl = (int)((h + probe) & (kCSlots - 1));
    int cur = s_key[sl];
    if (cur == -1) cur = atomicCAS(&s_key[sl], -1, key);
    if (cur == -1 || cur == key) return sl;
  }
  return -1;
}

constexpr int kMidTiles = 16;  // a triangle over 5 to this many tiles: 16 lanes test them
constexpr int kMidTris = 128;  // such triangles of one workgroup

struct MidTri {
  int X[3], Y[3];
  int first, tiles_x;  // the box's first tile and the view's tiles per row
  PixBox b;
  int tid;
};

// Exact test of MidTri's part in the tile whose first pixel is (tx0, ty0):
// each edge at the corner centre its inward normal points to.
__device__ __forceinline__ bool mid_may_cover(const MidTri& m, int tx0, int ty0, int side) {
  const int x0 = max(tx0, m.b.x0), x1 = min(tx0 + side - 1, m.b.x1), y0 = max(ty0, m.b.y0), y1 = min(ty0 + side - 1, m.b.y1);
  const long long D = (long long)(m.X[1] - m.X[0]) * (long long)(m.Y[2] - m.Y[0]) -
                      (long long)(m.X[2] - m.X[0]) * (long long)(m.Y[1] - m.Y[0]);
  bool in = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int a = (k + 1) % 3, b = (k + 2) % 3;
    const int dy = m.Y[a] - m.Y[b], dx = m.X[b] - m.X[a];
    const int A = D < 0 ? -dy : dy, B = D < 0 ? -dx : dx;
    const int px = (A > 0 ? x1 : x0) * 256 + 128 - m.X[a], py = (B > 0 ? y1 : y0) * 256 + 128 - m.Y[a];
    const long long E = (long long)A * px + (long long)B * py;
    in &= E > 0 || (E == 0 && (A > 0 || (A == 0 && B > 0)));
  }
  return in;
}

// One thread per (view, triangle).  Every tile a triangle may cover gets an
// entry {tile, rank << 8 | triangle} in the workgroup's part of seg, which
// holds 8 entries per triangle: one over at most four tiles is tested by its
// thread, one over 5 to 16 by 16 lanes (while the workgroup has room for
// them).  The rest are listed in large (their number in status[4]): k_clarge
// and the fill pass give each a workgroup of its own, and the tile's second
// counter counts them.
__global__ void __launch_bounds__(kBinBlock) k_ccount(const mer_view* __restrict__ views, int n_views,
                                                      const float* __restrict__ v, const int32_t* __restrict__ tri,
                                                      const long long* __restrict__ tri_base,
                                                      const long long* __restrict__ tile_base, int total_tris, int ctl,
                                                      const Counts count, uint2* __restrict__ seg,
                                                      int* __restrict__ seg_n, int* __restrict__ large,
                                                      long long* __restrict__ status) {
  __shared__ int s_key[kCSlots], s_cnt[kCSlots];
  __shared__ unsigned s_ent[kSegStride];  // slot << 17 | rank in the workgroup << 8 | triangle; or kEntDone
  __shared__ MidTri s_mid[kMidTris];
  __shared__ int s_big[kBinBlock];
  __shared__ int s_nbig, s_bigat, s_nmid, s_room, s_n;
  constexpr unsigned kEntDone = 0xffffffffu;
  for (int i = threadIdx.x; i < kCSlots; i += kBinBlock) {
    s_key[i] = -1;
    s_cnt[i] = 0;
  }
  const long long g0 = (long long)blockIdx.x * kBinBlock;
  if (threadIdx.x == 0) {
    s_nbig = s_nmid = s_n = 0;
    s_room = 4 * (int)min((long long)kBinBlock, total_tris - g0);  // 8 entries a triangle, 4 of them its own
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint2* out = seg + (long long)blockIdx.x * kSegStride;
  // entry `at` of the workgroup: triangle `who` in tile `ct`.  A tile the
  // table does not take gets its rank from memory at once.
  auto enter = [&](int at, int ct, int who) {
    const int sl = ctile_slot(s_key, ct);
    if (sl >= 0) {
      s_ent[at] = (unsigned)sl << 17 | (unsigned)atomicAdd(&s_cnt[sl], 1) << 8 | (unsigned)who;
    } else {
      const unsigned r = (unsigned)atomicAdd(&count[ct].x, 1);
      out[at] = make_uint2((unsigned)ct, min(r, kRankMax) << 8 | (unsigned)who);
      s_ent[at] = kEntDone;
    }
  };
  const long long g = g0 + threadIdx.x;
  bool culled = false;
  int tile[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) tile[j] = -1;
  if (g < total_tris) {
    const int vi = wave_bucket(tri_base, n_views, g);
    const mer_view vw = views[vi];
    const Snap s = snap_triangle<false>(v, vw, tri_row(tri, vw, (int)(g - tri_base[vi])));
    culled = !s.ok;
    PixBox b = pixel_box(s, vw);
    // Where many triangles are smaller than a pixel most cover no centre:
    // boxes of at most 2 x 2 centres are tested here (32-bit edge values: the
    // triangle spans less than 128 px, the centres lie in its box).
    const int bw = b.x1 - b.x0, bh = b.y1 - b.y0;
    const int ex = max(s.X[0], max(s.X[1], s.X[2])) - min(s.X[0], min(s.X[1], s.X[2]));
    const int ey = max(s.Y[0], max(s.Y[1], s.Y[2])) - min(s.Y[0], min(s.Y[1], s.Y[2]));
    const bool tiny = s.ok & (b.x0 <= b.x1) & (bw <= 1) & (bh <= 1) & (max(ex, ey) < (1 << 15));
    if (__popcll(__builtin_amdgcn_ballot_w64(tiny)) >= 16 && tiny) {
      int f00 = 0, f10 = 0, f01 = 0, f11 = 0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int a = (k + 1) % 3;
        int A, B;
        const int tl = inward_tl(s, k, A, B);
        const int F = mul_i24(A, b.x0 * 256 + 128 - s.X[a]) + mul_i24(B, b.y0 * 256 + 128 - s.Y[a]) + tl - 1;
        const int dx = A * 256 * bw, dy = B * 256 * bh;
        f00 |= F;
        f10 |= F + dx;
        f01 |= F + dy;
        f11 |= F + dx + dy;
      }
      if ((f00 & f10 & f01 & f11) < 0) b.x1 = b.x0 - 1;  // no centre has all three edge values in
    }
    if (s.ok && b.x0 <= b.x1) {
      const int tx0 = b.x0 >> ctl, ty0 = b.y0 >> ctl, ntx = (b.x1 >> ctl) - tx0 + 1, nty = (b.y1 >> ctl) - ty0 + 1;
      const int nt = ntx * nty;  // at most 2048^2
      const int tiles_x = (vw.W + (1 << ctl) - 1) >> ctl;
      const int first = (int)(tile_base[vi] + (long long)ty0 * tiles_x + tx0);
      if (nt > 4) {
        int i = kMidTris;
        if (nt <= kMidTiles && atomicSub(&s_room, nt) >= nt) i = atomicAdd(&s_nmid, 1);
        if (i < kMidTris) {
          MidTri m;
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            m.X[k] = s.X[k];
            m.Y[k] = s.Y[k];
          }
          m.first = first;
          m.tiles_x = tiles_x;
          m.b = b;
          m.tid = (int)threadIdx.x;
          s_mid[i] = m;
        } else {
          s_big[atomicAdd(&s_nbig, 1)] = (int)threadIdx.x;
        }
      } else if (nt < 4 || ntx != 2) {
        // a row or column of tiles: the box is tight, so each is met
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (j < nt) tile[j] = first + (ntx == 1 ? j * tiles_x : j);
      } else {
        MidTri m;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          m.X[k] = s.X[k];
          m.Y[k] = s.Y[k];
        }
        m.b = b;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (mid_may_cover(m, (tx0 + (j & 1)) << ctl, (ty0 + (j >> 1)) << ctl, 1 << ctl))
            tile[j] = first + (j >> 1) * tiles_x + (j & 1);
      }
    }
  }
  const int n = (tile[0] >= 0) + (tile[1] >= 0) + (tile[2] >= 0) + (tile[3] >= 0);
  const int inc = wave_scan_i32(n);
  int at = 0;
  if (lane == 63 && inc > 0) at = atomicAdd(&s_n, inc);
  at = __builtin_amdgcn_readlane(at, 63) + inc - n;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (tile[j] >= 0) enter(at++, tile[j], (int)threadIdx.x);
  __syncthreads();  // the lists of larger triangles are complete
  const int nbig = s_nbig, nmid = min(s_nmid, kMidTris);
  for (int i0 = 0; i0 < nmid; i0 += 16) {
    const int i = i0 + (threadIdx.x >> 4), k = threadIdx.x & 15;
    int ct = -1, who = 0;
    if (i < nmid) {
      const MidTri& m = s_mid[i];
      const int tx0 = m.b.x0 >> ctl, ty0 = m.b.y0 >> ctl, ntx = (m.b.x1 >> ctl) - tx0 + 1, nty = (m.b.y1 >> ctl) - ty0 + 1;
      who = m.tid;
      if (k < ntx * nty) {
        const int dy = k / ntx, dx = k - dy * ntx;
        if (mid_may_cover(m, (tx0 + dx) << ctl, (ty0 + dy) << ctl, 1 << ctl)) ct = m.first + dy * m.tiles_x + dx;
      }
    }
    const unsigned long long m = __ballot(ct >= 0);
    int base = 0;
    if (lane == 0 && m) base = atomicAdd(&s_n, (int)__popcll(m));
    base = __builtin_amdgcn_readfirstlane(base);
    if (ct >= 0) enter(base + (int)__popcll(m & ((1ull << lane) - 1ull)), ct, who);
  }
  if (threadIdx.x == 0 && nbig)
    s_bigat = (int)atomicAdd((unsigned long long*)status + 4, (unsigned long long)nbig);
  __syncthreads();
  for (int i = threadIdx.x; i < kCSlots; i += kBinBlock)
    if (s_key[i] >= 0) s_cnt[i] = atomicAdd(&count[s_key[i]].x, s_cnt[i]);
  __syncthreads();
  const int total = s_n;
  for (int i = threadIdx.x; i < total; i += kBinBlock) {
    const unsigned e = s_ent[i];
    if (e == kEntDone) continue;
    const int sl = (int)(e >> 17);
    const unsigned r = (unsigned)s_cnt[sl] + ((e >> 8) & 511u);
    out[i] = make_uint2((unsigned)s_key[sl], min(r, kRankMax) << 8 | (e & 255u));
  }
  if (threadIdx.x == 0) seg_n[blockIdx.x] = total;
  if ((int)threadIdx.x < nbig) large[s_bigat + threadIdx.x] = (int)g0 + s_big[threadIdx.x];
  const unsigned long long m = __ballot(culled);
  if (m && lane == 0) atomicAdd((unsigned long long*)status + 1, (unsigned long long)__popcll(m));
}

// Workgroups for the large triangles, whether there are any or not.  us in
// k_clarge and in the fill with 256, 1024 and 2048: 16 views of few large
// triangles 8.7 + 9.4, 4.9 + 5.4, 4.9 + 5.5; 200,000 of up to 60 px in one of
// 1024 x 1024 89 + 111, 37 + 56, 32 + 41; none 1.6 + 2.6, 1.8 + 2.7, 1.9 + 2.7.
constexpr int kLargeGrid = 1024;

__global__ void __launch_bounds__(kBinBlock) k_clarge(const mer_view* __restrict__ views, int n_views,
                                                      const float* __restrict__ v, const int32_t* __restrict__ tri,
                                                      const long long* __restrict__ tri_base,
                                                      const long long* __restrict__ tile_base, int ctl,
                                                      const int* __restrict__ large, const long long* __restrict__ status,
                                                      const Counts count) {
  walk_large(views, n_views, tri_base, tile_base, v, tri, ctl, large, (int)status[4], 0,
             [&](int, int ct) { atomicAdd(&count[ct].y, 1); });
}

// ---------------------------------------------------------- ranges and fill
// Ranges need no order, so a workgroup of tiles takes its part of the pool
// with one add.  Ranked entries come first in a tile's list, walked ones
// after them.  A list longer than two parts is split while there is room for
// its parts (their number in status[3]), and its tile's keys are cleared.
__global__ void __launch_bounds__(256) k_calloc(const mer_view* __restrict__ views, int n_views, int ctl,
                                                const long long* __restrict__ tile_base, long long n_tiles,
                                                const Counts count, long long bin_cap,
                                                CTile* __restrict__ tiles, int item, int n_items,
                                                CItem* __restrict__ items, unsigned long long* __restrict__ key,
                                                long long* __restrict__ status) {
  __shared__ long long s_wave[4], s_base;
  __shared__ CTile s_split[256];
  __shared__ int s_nsplit;
  if (threadIdx.x == 0) s_nsplit = 0;
  const long long g = (long long)blockIdx.x * 256 + threadIdx.x;
  const int2 c = g < n_tiles ? count[g] : make_int2(0, 0);
  const long long n = (long long)c.x + c.y;
  long long inc = wave_incl_scan(n);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 63) s_wave[wv] = inc;
  __syncthreads();
  if (threadIdx.x == 0) {
    const long long total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    s_base = total ? (long long)atomicAdd((unsigned long long*)status + 2, (unsigned long long)total) : 0;
  }
  __syncthreads();
  long long base = s_base + inc - n;
  for (int i = 0; i < wv; ++i) base += s_wave[i];
  const bool over = base + n > bin_cap || (unsigned)c.x >= kRankMax;
  const unsigned long long m = __ballot(over && g < n_tiles && n > 0);
  if (m && lane == 0) atomicAdd((unsigned long long*)status, (unsigned long long)__popcll(m));
  if (g < n_tiles) {
    const int vi = wave_bucket(tile_base, n_views, g);
    int tx, ty;
    grid_xy(g - tile_base[vi], (views[vi].W + (1 << ctl) - 1) >> ctl, tx, ty);
    CTile t;
    t.base = over ? 0 : (int)base;
    t.n = n == 0 ? 0 : over ? -1 : (int)n;
    t.view = vi;
    t.xy = (unsigned)tx | (unsigned)ty << 16;
    if (n_items > 0 && t.n > max(kLongList, 2 * item)) {
      const int want = (t.n + item - 1) / item;
      const long long at = (long long)atomicAdd((unsigned long long*)status + 3, (unsigned long long)want);
      const int got = (int)max(min((long long)want, n_items - at), 0ll);
      if (got > 1) {
        s_split[atomicAdd(&s_nsplit, 1)] = t;
        const int size = ((t.n + got - 1) / got + 255) & ~255;
        for (int i = 0; i < got; ++i) {
          const int lo = (int)min((long long)i * size, (long long)t.n);
          items[at + i] = {{t.base + lo, min(size, t.n - lo), vi, t.xy | kPart}, i, got, 0, 0};
        }
        t.xy |= kGone;
      }
    }
    tiles[g] = t;
    if (c.y > 0) count[g].x = over ? -1 : t.base + c.x;  // where the walked ones go
  }
  __syncthreads();
  for (int i = 0; i < s_nsplit; ++i) {
    const mer_view vw = views[s_split[i].view];
    const int x0 = (int)(s_split[i].xy & 0xffffu) << ctl, y0 = (int)(s_split[i].xy >> 16) << ctl;
    for (int k = threadIdx.x; k < 1 << 2 * ctl; k += 256) {
      const int x = x0 + (k & ((1 << ctl) - 1)), y = y0 + (k >> ctl);
      if (x < vw.W && y < vw.H) key[vw.px_off + (long long)y * vw.W + x] = 0ull;
    }
  }
}

// The first n_groups workgroups copy the count pass's entries, the others
// take the large triangles.
__global__ void __launch_bounds__(kBinBlock) k_cfill(const mer_view* __restrict__ views, int n_views,
                                                     const float* __restrict__ v, const int32_t* __restrict__ tri,
                                                     const long long* __restrict__ tri_base,
                                                     const long long* __restrict__ tile_base, int ctl, int n_groups,
                                                     const Counts count, const uint2* __restrict__ seg,
                                                     const int* __restrict__ seg_n, const int* __restrict__ large,
                                                     const long long* __restrict__ status,
                                                     const CTile* __restrict__ tiles, int* __restrict__ bins) {
  if ((int)blockIdx.x >= n_groups) {
    walk_large(views, n_views, tri_base, tile_base, v, tri, ctl, large, (int)status[4], n_groups, [&](int g, int ct) {
      // both counters in one access: the place is the first one's value (-1:
      // no room) plus the second's, which goes down.  Read by loads of their
      // own beside the atomics, 100,000 triangles' 650,000 entries in 1024
      // tiles took 199 us, and take 40.
      const unsigned long long c = atomicAdd(reinterpret_cast<unsigned long long*>(&count[ct]), ~0ull << 32);
      const int at = (int)(unsigned)c;
      if (at >= 0) bins[at + (int)(c >> 32) - 1] = g;
    });
    return;
  }
  const int n = seg_n[blockIdx.x];
  const int g0 = (int)blockIdx.x * kBinBlock;
  const uint2* in = seg + (long long)blockIdx.x * kSegStride;
  for (int i = threadIdx.x; i < n; i += kBinBlock) {
    const uint2 e = in[i];
    const int2 t = *reinterpret_cast<const int2*>(&tiles[e.x]);
    if (t.y >= 0) bins[t.x + (int)(e.y >> 8)] = g0 + (int)(e.y & 255u);
  }
}

// ------------------------------------------------------------------ raster
typedef short short2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int dot2(int a, int b, int c) {
  return __builtin_amdgcn_sdot2(__builtin_bit_cast(short2v, a), __builtin_bit_cast(short2v, b), c, false);
}
__device__ __forceinline__ int pack2(int x, int y) { return (x & 0xffff) | (int)((unsigned)y << 16); }

// The wave's LDS accesses before this are done before those after it; lanes of
// one wave only.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Candidate record, 64 bytes.  "Tight" triangles span less than 128 px
// along each axis (|A|, |B| < 2^15) and their vertex 1/z lie in [2^-64, 2^64].
// At a centre inside the triangle's box an edge value is twice the area of a
// triangle within the box, below 2^30 (as |D| is), and 31 pixels away in x and
// y, the farthest a centre of a tile the box meets can lie, it has changed by
// less than 2^29: every value fits 32 bits and is one 16-bit dot product,
//   F_k = F0_k + A_k (256 dx) + B_k (256 dy) = E'_k - 1,
// with (dx, dy) the pixel in the tile and E'_k the value biased by the
// top-left rule: covered iff no F_k is negative, and e_k = F_k + 1 - tl_k.
//   tight:   F0[3], 1 / d | (A, B)[3] as pairs, d | q[3], ~t | (1 - tl)[3], depth bound
//   general: C[3] (64-bit, at the tile's first centre), ~t, B1 | q[3], B2 | A[3], B0
typedef int int4v __attribute__((ext_vector_type(4)));
struct __align__(16) CRec {
  int4v r[4];
};
struct CandRec {
  int4v a, b, c, d;
};

constexpr int kSmallPx = 40;  // a box of at most this many centres can be rasterized by the candidate's own lane
constexpr int kStageC = 16;  // channels of a row staged in the records' memory: 64 a wave
constexpr int kMaskSlot = 20;  // from this bit on: the record's place
constexpr int kMaskGen = 16;  // bit of the candidate's tile mask: general record; the three above it: tl

// One workgroup (four waves) per coarse tile of 2^CTL x 2^CTL pixels, keys in
// LDS.  The tile's candidates are taken 256 at a time, one per lane: snap,
// clip the box to the tile, and either rasterize the few centres right there
// with LDS maxima (when enough of the wave's triangles are that small), or
// write a record and a mask of the 8 x 8 tiles it may cover.  The records are
// put in order of their nearest possible depth (64 buckets), then each wave
// takes its 8 x 8 tiles, one lane per pixel, and walks the mask bits: a
// candidate is skipped once no pixel's surface is as far as its bound.
// direct: no lists; the plan's one view has few triangles and every tile
// scans them all.  n_split workgroups of the grid, from split0 on, take the
// parts of long lists, as many as there are, the others a tile each.  One workgroup for a
// list whatever its length made 1.8 M triangles over 64 px of a 2048 x 2048
// view take 483 us (104 in parts), and over 200 px 1088 (168).
// STAGED: the resolve writes its image rows by way of LDS (below).
template <int CTL, int NT, bool STAGED>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(5))) k_craster(const mer_view* __restrict__ views, const CTile* __restrict__ tiles,
                                                 const Counts count, const int* __restrict__ bins,
                                                 const long long* __restrict__ tri_base, int direct, ResolveOut R,
                                                 int split0, int n_split, int n_tiles, CItem* __restrict__ items,
                                                 unsigned long long* __restrict__ key,
                                                 long long* __restrict__ status) {
  constexpr int CT = 1 << CTL, NPX = CT * CT, NF = NPX / 64, FX = CT / 8, NW = NT / 64;
  constexpr int kChunk = NT;  // candidates taken at a time
  __shared__ unsigned long long s_key[NPX];
  __shared__ CRec s_rec[kChunk];
  static_assert(sizeof(CRec) * kChunk >= sizeof(float) * 64 * kStageC * NW, "a wave's staged rows fit the records");
  __shared__ unsigned s_mask[kChunk];
  __shared__ float s_qb[kChunk];
  __shared__ int s_hist[64];
  __shared__ float s_mm[2 * NW];
  __shared__ int s_culled, s_next;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int sb = (int)blockIdx.x - split0;
  const bool split = (unsigned)sb < (unsigned)n_split;
  const long long g = xcd_tile((int)blockIdx.x - (sb < 0 ? 0 : n_split), n_tiles);
  CTile T;
  if (direct) {
    const int tiles_x = (views[0].W + CT - 1) >> CTL;
    const unsigned q = (unsigned)g / (unsigned)tiles_x;
    T.base = 0;
    T.n = -1;
    T.view = 0;
    T.xy = ((unsigned)g - q * tiles_x) | q << 16;
  } else {
    T = *(split ? &items[sb].t : tiles + g);
    // integrity: the fill pass takes every walked count back to 0; every
    // 256th tile's workgroup looks at as many
    if (!split && (g & (NT - 1)) == 0 && g + tid < n_tiles && count[g + tid].y != 0)
      atomicAdd((unsigned long long*)status + 6, 1ull);
    if (T.xy & kGone) return;
  }
  const mer_view vw = views[T.view];
  const int x0 = (int)(T.xy & 0x7fffu) << CTL, y0 = (int)(T.xy >> 16 & 0x7fffu) << CTL;
  const int tb = direct ? 0 : (int)tri_base[T.view];
  int n_items = T.n < 0 ? vw.n_t : T.n;
  // keys are swizzled by row so that the rows of an 8 x 8 tile fall on
  // different banks
  auto key_at = [&](int x, int y) -> int { return (y << CTL) + (x ^ ((y & (CT / 8 - 1)) << 3)); };
  if (n_items > 0) {
    for (int i = tid; i < NPX; i += NT) s_key[i] = 0ull;
    if (tid < 64) s_hist[tid] = 0;
    if (tid == 0) s_culled = 0;
  }
  // candidate c0 + tid of the tile, -1 when there is none
  auto candidate = [&](int c0) -> int {
    if (c0 + tid >= n_items) return -1;
    if (T.n < 0) return c0 + tid;
    const int t = bins[T.base + c0 + tid] - tb;
    // integrity: an entry names a triangle of this tile's view; any other
    // value is counted (mer_status fails on it) and not read
    if ((unsigned)t < (unsigned)vw.n_t) return t;
    atomicAdd((unsigned long long*)status + 5, 1ull);
    return -1;
  };
  int row[3] = {0, 0, 0};
  auto load_row = [&](int t) {
    if (t < 0) return;
    const int32_t* r = tri_row(R.tri, vw, t);
#pragma unroll
    for (int k = 0; k < 3; ++k) row[k] = r[k];
  };
  int t_next = candidate(0);
  load_row(t_next);
  for (int c0 = 0; c0 < n_items; c0 += kChunk) {
    __syncthreads();  // the keys are set, the last chunk's records are read
    // ---- one candidate per lane; the next chunk's is loaded ahead
    const int t = t_next;
    Snap s;
    s.ok = false;
    if (t >= 0) s = T.n >= 0 ? snap_visible(R.v, vw, row) : snap_triangle(R.v, vw, row);
    t_next = candidate(c0 + kChunk);
    if (direct && t >= 0 && !s.ok && blockIdx.x == 0) atomicAdd(&s_culled, 1);
    PixBox b = {1, 1, 0, 0};
    if (s.ok) {
      b = pixel_box(s, vw);
      b.x0 = max(b.x0 - x0, 0);
      b.y0 = max(b.y0 - y0, 0);
      b.x1 = min(b.x1 - x0, CT - 1);
      b.y1 = min(b.y1 - y0, CT - 1);
    }
    bool live = s.ok && b.x0 <= b.x1 && b.y0 <= b.y1;
    unsigned mask = 0u;
    float qb = 0.f;
    bool tight = false;
    int F[3] = {0, 0, 0}, A[3], B[3], bias[3];
    float d = 1.f, rd = 1.f;
    if (live) {
      const float qlo = fminf(s.q[0], fminf(s.q[1], s.q[2])), qhi = fmaxf(s.q[0], fmaxf(s.q[1], s.q[2]));
      const int ex = max(s.X[0], max(s.X[1], s.X[2])) - min(s.X[0], min(s.X[1], s.X[2]));
      const int ey = max(s.Y[0], max(s.Y[1], s.Y[2])) - min(s.Y[0], min(s.Y[1], s.Y[2]));
      tight = max(ex, ey) < (1 << 15) && qlo >= 0x1p-64f && qhi <= 0x1p64f;
      // no key of the triangle exceeds this bound: the key is a convex
      // combination of the vertices' 1/z up to a few roundings (< 2^-20)
      qb = fmaxf(qhi * (1.0f + 0x1p-20f), 0x1p-126f);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int tl = inward_tl(s, k, A[k], B[k]);
        bias[k] = 1 - tl;
      }
    }
    if (live && tight) {
      // vertices relative to the tile's first centre: below 2^16 in magnitude;
      // the sums are exact modulo 2^32 and their values fit
      int rx[3], ry[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        rx[k] = s.X[k] - (x0 * 256 + 128);
        ry[k] = s.Y[k] - (y0 * 256 + 128);
      }
      int Dabs = 0;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        // orient(a, b, origin) with sign(D): the edge's inward normal dotted with (origin - vertex a)
        const int e = -(mul_i24(A[k], rx[(k + 1) % 3]) + mul_i24(B[k], ry[(k + 1) % 3]));
        Dabs += e;
        F[k] = e - bias[k];
      }
      d = (float)Dabs;
      rd = rcp_rn(d);
    }
    // ---- small triangles, by their own lanes
    // The wave takes as many steps as its largest such triangle has centres,
    // about 40 instructions each; a triangle costs about 25 the other way.
    const int bw = b.x1 - b.x0 + 1, area = live && tight ? bw * (b.y1 - b.y0 + 1) : 0x7fffffff;
    int small_px = 0;
#pragma unroll
    for (int K = 8; K <= kSmallPx; K += 8)
      if (5 * __popcll(__builtin_amdgcn_ballot_w64(area <= K)) >= 8 * K) small_px = K;
    if (small_px > 0) {
      const bool small = area <= small_px;
      if (small) {
        const unsigned tn = ~(unsigned)t;
        int f[3], dx256[3], wrap[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          dx256[k] = A[k] * 256;
          f[k] = F[k] + A[k] * (b.x0 * 256) + B[k] * (b.y0 * 256);
          wrap[k] = B[k] * 256 - A[k] * (bw - 1) * 256;  // from a row's last centre to the next row's first
        }
        int x = b.x0, y = b.y0;
#pragma unroll 1
        for (int i = 0; i < area; ++i) {
          if ((f[0] | f[1] | f[2]) >= 0) {
            const float a0 = (float)(f[0] + bias[0]) * s.q[0];
            const float a1 = (float)(f[1] + bias[1]) * s.q[1];
            const float a2 = (float)(f[2] + bias[2]) * s.q[2];
            float nq = a0 + a1;
            nq = nq + a2;
            atomicMax(&s_key[key_at(x, y)], ((unsigned long long)__float_as_uint(div_rn(nq, d, rd)) << 32) | tn);
          }
          const bool last = x == b.x1;
#pragma unroll
          for (int k = 0; k < 3; ++k) f[k] += last ? wrap[k] : dx256[k];
          x = last ? b.x0 : x + 1;
          y += last ? 1 : 0;
        }
        live = false;
      }
    }
    // ---- the others: record and mask of the 8 x 8 tiles
    if (live) {
      const int fx0 = b.x0 >> 3, fx1 = b.x1 >> 3, fy0 = b.y0 >> 3, fy1 = b.y1 >> 3;
      const unsigned cols = ((2u << fx1) - (1u << fx0)) * (FX == 4 ? 0x1111u : FX == 2 ? 5u : 1u);
      mask = cols & ((1u << ((fy1 + 1) * FX)) - (1u << (fy0 * FX)));  // the box's tiles
      if (tight) {
        // each edge's largest value over the 8 x 8 centres of tile (0, 0) and
        // its steps to the next column and row of tiles; the sign bits of the
        // tiles, last tile first, shifted into one word
        int top[3], sx[3], sy[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          sx[k] = A[k] * 2048;
          sy[k] = B[k] * 2048;
          top[k] = F[k] + max(A[k], 0) * 1792 + max(B[k], 0) * 1792 + sx[k] * (FX - 1) + sy[k] * (FX - 1);
        }
        unsigned out_m = 0u;
#pragma unroll
        for (int j = FX - 1; j >= 0; --j) {
#pragma unroll
          for (int i = FX - 1; i >= 0; --i) {
            out_m = __builtin_amdgcn_alignbit(out_m, (unsigned)(top[0] | top[1] | top[2]), 31);
#pragma unroll
            for (int k = 0; k < 3; ++k) top[k] -= i > 0 ? sx[k] : sy[k] - sx[k] * (FX - 1);
          }
        }
        mask &= ~out_m;
        s_rec[tid].r[0] = int4v{F[0], F[1], F[2], __float_as_int(rd)};
        s_rec[tid].r[1] = int4v{pack2(A[0], B[0]), pack2(A[1], B[1]), pack2(A[2], B[2]), __float_as_int(d)};
        s_rec[tid].r[2] = int4v{__float_as_int(s.q[0]), __float_as_int(s.q[1]), __float_as_int(s.q[2]), ~t};
        s_rec[tid].r[3] = int4v{bias[0], bias[1], bias[2], __float_as_int(qb)};
      } else {
        // biased edge values at the tile's first centre
        long long C[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const int a = (k + 1) % 3;
          C[k] = (long long)A[k] * (x0 * 256 + 128 - s.X[a]) + (long long)B[k] * (y0 * 256 + 128 - s.Y[a]) + (1 - bias[k]);
        }
        mask |= (1u | (unsigned)(7 ^ (bias[0] | bias[1] << 1 | bias[2] << 2)) << 1) << kMaskGen;
        s_rec[tid].r[0] = int4v{(int)C[0], (int)(C[0] >> 32), (int)C[1], (int)(C[1] >> 32)};
        s_rec[tid].r[1] = int4v{(int)C[2], (int)(C[2] >> 32), ~t, B[1]};
        s_rec[tid].r[2] = int4v{__float_as_int(s.q[0]), __float_as_int(s.q[1]), __float_as_int(s.q[2]), B[2]};
        s_rec[tid].r[3] = int4v{A[0], A[1], A[2], B[0]};
      }
    }
    // ---- nearest first: 64 buckets of the depth bound (positive floats order like their bits)
    const unsigned long long live_m = __ballot(mask != 0u);
    unsigned lo_b = 0x7f800000u, hi_b = 0u;
    if (live_m) {
      lo_b = wave_min_u32(mask ? __float_as_uint(qb) : 0x7f800000u);
      hi_b = wave_max_u32(mask ? __float_as_uint(qb) : 0u);
    }
    if (tid == 0) s_next = 0;
    if (lane == 0) {
      s_mm[wv] = __uint_as_float(lo_b);
      s_mm[NW + wv] = __uint_as_float(hi_b);
    }
    __syncthreads();
    float lo = s_mm[0], hi = s_mm[NW];
#pragma unroll
    for (int i = 1; i < NW; ++i) {
      lo = fminf(lo, s_mm[i]);
      hi = fmaxf(hi, s_mm[NW + i]);
    }
    int n_rec = 0;
    if (hi > 0.f) {  // uniform: some candidate has a record
      const float scale = hi > lo ? 63.0f / (hi - lo) : 0.f;
      const int bk = max(0, min(63, (int)((hi - qb) * scale)));
      int at = 0;
      if (mask) at = atomicAdd(&s_hist[bk], 1);
      __syncthreads();
      const int h = s_hist[lane], inc = wave_scan_i32(h);
      n_rec = __builtin_amdgcn_readlane(inc, 63);
      at += __shfl(inc - h, bk, 64);
      if (mask) {
        s_mask[at] = mask | (unsigned)tid << kMaskSlot;
        s_qb[at] = qb;
      }
      __syncthreads();
      if (tid < 64) s_hist[tid] = 0;
    }
    load_row(t_next);
    // ---- 8 x 8 tiles, one lane per pixel
    if (n_rec > 0) {
      // this lane's candidate of each group of 64
      unsigned mk[NW];
      float bound[NW];
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const bool have = 64 * i + lane < n_rec;
        mk[i] = have ? s_mask[64 * i + lane] : 0u;
        bound[i] = have ? s_qb[64 * i + lane] : 0.f;
      }
#pragma unroll 1
      for (int i = 0; i < NF; ++i) {
        int f = wv;
        if (NF <= NW && (i > 0 || f >= NF)) break;
        if (NF > NW) {  // whichever tile is next: their candidates differ in number
          if (lane == 0) f = atomicAdd(&s_next, 1);
          f = __builtin_amdgcn_readfirstlane(f);
          if (f >= NF) break;
        }
        const int fx = (f % FX) * 8, fy = (f / FX) * 8;
        if (x0 + fx >= vw.W || y0 + fy >= vw.H) continue;
        const int lx = fx + (lane & 7), ly = fy + (lane >> 3);
        const bool inside = x0 + lx < vw.W && y0 + ly < vw.H;
        const unsigned long long inside_m = __builtin_amdgcn_ballot_w64(inside);
        const int dxy = pack2(lx * 256, ly * 256);
        unsigned long long best = s_key[key_at(lx, ly)];
        const unsigned long long best0 = best;
        // the larger key on the lanes of cov_m
        auto take = [&](float q, unsigned tn, unsigned long long cov_m) {
          const unsigned long long k = ((unsigned long long)__float_as_uint(q) << 32) | tn;
          const bool win = __builtin_amdgcn_inverse_ballot_w64(__builtin_amdgcn_ballot_w64(k > best) & cov_m);
          best = win ? k : best;
        };
#pragma unroll 1
        for (int k0 = 0; k0 < n_rec; k0 += 64) {
          unsigned mg = mk[0];
          float bd = bound[0];
#pragma unroll
          for (int i2 = 1; i2 < NW; ++i2)
            if (k0 == 64 * i2) {
              mg = mk[i2];
              bd = bound[i2];
            }
          unsigned long long m = __builtin_amdgcn_ballot_w64((int)(mg << (31 - f)) < 0);
          if (!m) continue;
          // candidates that no pixel's surface is as far as drop out
          if (!(__builtin_amdgcn_ballot_w64(best == 0ull) & inside_m)) {
            const float far = __uint_as_float(wave_min_u32(inside ? (unsigned)(best >> 32) : 0x7f800000u));
            m &= __builtin_amdgcn_ballot_w64(bd >= far);
          }
          unsigned long long gen = __builtin_amdgcn_ballot_w64((mg >> kMaskGen & 1u) != 0u) & m;
          m &= ~gen;
          // one at a time, the next one's record on its way
          auto fetch = [&](CandRec& c) {  // the first candidate of m (some record when m is empty)
            const int slot = __builtin_amdgcn_readlane((int)mg, __builtin_ctzll(m | 1ull << 63)) >> kMaskSlot;
            const CRec& r = s_rec[slot];
            c = {r.r[0], r.r[1], r.r[2], r.r[3]};
          };
          auto test = [&](CandRec& c) {
            // whole-record loads, waited for here
            asm volatile("" : "+v"(c.a), "+v"(c.b), "+v"(c.c), "+v"(c.d));
            const int F0 = dot2(c.b.x, dxy, c.a.x), F1 = dot2(c.b.y, dxy, c.a.y), F2 = dot2(c.b.z, dxy, c.a.z);
            const unsigned long long cov_m = __builtin_amdgcn_ballot_w64((F0 | F1 | F2) >= 0) &
                                             __builtin_amdgcn_ballot_w64(__int_as_float(c.d.w) >= key_q(best)) & inside_m;
            if (!cov_m) return;
            const float p0 = (float)(F0 + c.d.x) * __int_as_float(c.c.x);
            const float p1 = (float)(F1 + c.d.y) * __int_as_float(c.c.y);
            const float p2 = (float)(F2 + c.d.z) * __int_as_float(c.c.z);
            float nq = p0 + p1;
            nq = nq + p2;
            take(div_rn(nq, __int_as_float(c.b.w), __int_as_float(c.a.w)), (unsigned)c.c.w, cov_m);
          };
          if (m) {
            CandRec A, B;
            fetch(A);
            do {
              m &= m - 1ull;
              fetch(B);
              test(A);
              if (!m) break;
              m &= m - 1ull;
              fetch(A);
              test(B);
            } while (m);
          }
          for (; gen; gen &= gen - 1ull) {
            const int w = __builtin_amdgcn_readlane((int)mg, __builtin_ctzll(gen));
            const int j = w >> kMaskSlot, tl = w >> (kMaskGen + 1);
            const int4v r0 = s_rec[j].r[0], r1 = s_rec[j].r[1], r2 = s_rec[j].r[2], r3 = s_rec[j].r[3];
            auto l64 = [](int l, int h) { return (long long)(((unsigned long long)(unsigned)h << 32) | (unsigned)l); };
            const long long X = lx * 256, Y = ly * 256;
            const long long E0 = l64(r0.x, r0.y) + (long long)r3.x * X + (long long)r3.w * Y;
            const long long E1 = l64(r0.z, r0.w) + (long long)r3.y * X + (long long)r1.w * Y;
            const long long E2 = l64(r1.x, r1.y) + (long long)r3.z * X + (long long)r2.w * Y;
            const unsigned long long cov_m = __builtin_amdgcn_ballot_w64(E0 > 0) & __builtin_amdgcn_ballot_w64(E1 > 0) &
                                             __builtin_amdgcn_ballot_w64(E2 > 0) & inside_m;
            if (!cov_m) continue;
            const long long u0 = E0 - (tl & 1), u1 = E1 - ((tl >> 1) & 1), u2 = E2 - ((tl >> 2) & 1);
            const float p0 = (float)u0 * __int_as_float(r2.x);
            const float p1 = (float)u1 * __int_as_float(r2.y);
            const float p2 = (float)u2 * __int_as_float(r2.z);
            float nq = p0 + p1;
            nq = nq + p2;
            take(nq / (float)(u0 + u1 + u2), (unsigned)r1.z, cov_m);
          }
        }
        if (best != best0) s_key[key_at(lx, ly)] = best;
      }
    }
  }
  __syncthreads();
  if (__builtin_expect((T.xy & kPart) != 0u, 0)) {
    int b = (int)blockIdx.x - split0;
    asm volatile("" : "+s"(b));  // read again: not kept through the loops
    const int part = items[b].part, parts = items[b].parts;
    // Every access here is an atomic that returns its old value, so it has
    // taken place in memory, whichever L2 a workgroup sits behind, before the
    // wave goes on.  Fences instead write the L2 back: 120 and 286 us for the
    // two meshes above.
    unsigned long long* kv = key + vw.px_off;
    unsigned long long seen = 0;
    if (n_items > 0) {
#pragma unroll 1
      for (int i = tid; i < NPX; i += NT) {
        const int x = i & (CT - 1), y = i >> CTL;
        const unsigned long long k = x0 + x < vw.W && y0 + y < vw.H ? s_key[key_at(x, y)] : 0ull;
        if (k) seen |= atomicMax(kv + (long long)(y0 + y) * vw.W + x0 + x, k);
      }
    }
    asm volatile("" ::"v"(seen));
    __syncthreads();  // the part's maxima are in memory
    if (tid == 0) s_next = atomicAdd(&items[b - part].done, 1);
    __syncthreads();
    if (s_next != parts - 1) return;
#pragma unroll 1
    for (int i = tid; i < NPX; i += NT) {
      const int x = i & (CT - 1), y = i >> CTL;
      if (x0 + x < vw.W && y0 + y < vw.H)
        s_key[key_at(x, y)] = atomicMax(kv + (long long)(y0 + y) * vw.W + x0 + x, 0ull);
    }
    n_items = 1;  // the tile's keys are in LDS
    __syncthreads();
  }
  if (direct && blockIdx.x == 0 && tid < 8) status[tid] = tid == 1 ? (long long)(n_items > 0 ? s_culled : 0) : 0;
  // ---- resolve, a row of the tile at a time.  STAGED: the image rows go
  // through the wave's part of the records' memory, and the wave writes them as
  // spans of consecutive floats.
  const int C = out_channels(R);
  float* stage = reinterpret_cast<float*>(s_rec) + wv * 64 * kStageC;
#pragma unroll 1
  for (int i = tid; i < NPX; i += NT) {
    const int x = i & (CT - 1), y = i >> CTL;
    const int px = x0 + x, py = y0 + y;
    const bool inside = px < vw.W && py < vw.H;
    if constexpr (!STAGED)
      if (!inside) continue;
    if (!STAGED || inside) {
      const unsigned long long best = n_items > 0 ? s_key[key_at(x, y)] : 0ull;
      const int t = key_tri(best);
      const long long p = vw.px_off + (long long)py * vw.W + px;
      R.tri_id[p] = t;
      if (R.depth) R.depth[p] = t >= 0 ? rcp_rn(key_q(best)) : 0.0f;
      if (R.bary || R.out) {
        float b0 = 0.f, b1 = 0.f;
        int idx[3] = {0, 0, 0};
        if (t >= 0) {
          const int32_t* r = tri_row(R.tri, vw, t);
#pragma unroll
          for (int k = 0; k < 3; ++k) idx[k] = r[k];
          float wa, wb, wn;
          resolve_products(snap_visible(R.v, vw, idx), px, py, wa, wb, wn);
          const float rr = __builtin_amdgcn_rcpf(wn);
          b0 = wa * rr;
          b1 = wb * rr;
        }
        if (R.bary) {
          R.bary[2 * p] = b0;
          R.bary[2 * p + 1] = b1;
        }
        if constexpr (STAGED) resolve_attr(R, vw, stage + lane * C, 0, t, b0, b1, idx);
        else if (R.out) resolve_attr(R, vw, R.out + p * C, row_vec(C, R.out), t, b0, b1, idx);
      }
    }
    if constexpr (STAGED) {
      // the wave's 64 pixels are 64 / CT rows of the tile; each row's pixels
      // inside the view are one span of the image
      wave_lds_fence();
      constexpr int PW = CT < 64 ? CT : 64;
      const int n = min(CT, vw.W - x0) * C, yb = y0 + ((i - lane) >> CTL);
#pragma unroll 1
      for (int k = 0; k < 64 / PW; ++k) {
        if (yb + k >= vw.H) break;
        float* o = R.out + (vw.px_off + (long long)(yb + k) * vw.W + x0) * C;
        const float* sp = stage + k * PW * C;
        for (int e = lane; e < n; e += 64) o[e] = sp[e];
      }
      wave_lds_fence();
    }
  }
}

// ------------------------------------------------------------------ launch
// A small view of few triangles needs no lists: where each tile has at most
// kDirectPerTile chunks of candidates to look at, and all together at most
// kDirectChunks, every tile scans every triangle, in one launch instead of
// six.  A chunk takes a tile's workgroup 2 to 3 us, the lists 15 to 20: without
// / with lists, us, 16 tiles of 4 chunks 21 / 27, 7 27 / 26, 10 33 / 25, 16
// 45 / 26; 64 tiles of 8 chunks 26 / 29; 4 tiles of 125 240 / 25.  The total's
// line is not where the two meet: 242 tiles of 2 chunks 11 / 38 on this side of
// it, 484 12 / 37 and 3249 32 / 45 on the other.
constexpr int kDirectChunks = 512, kDirectPerTile = 8;

static bool direct_tiles(const mer_plan* P, long long n_tiles) {
  const long long chunks = (P->total_tris + 255) / 256;
  return P->n_views == 1 && chunks <= kDirectPerTile && n_tiles * chunks <= kDirectChunks;
}

// Image rows that no vector store takes whole (other than 3, 4, 8, ... floats)
// are written a float a lane, C lines a store; from some width on it is faster
// to pass them through LDS.  k_craster, us, own rows / through LDS: 16 head
// views of 1024 x 667 (32 x 32 tiles) 2 channels 97 / 108, 5 147 / 137, 7 206 /
// 150, 11 435 / 198, 14 671 / 234; 4 views of 731 x 413 (16 x 16 tiles, half as
// long spans) 5 57 / 61, 7 60 / 60, 9 68 / 60, 14 98 / 64; one 300 x 300 view
// (8 x 8 tiles, an eighth of the chip) 9 36 / 37, 14 38 / 39.
static bool staged_rows(const ResolveOut& R, int ctl) {
  if (!R.out) return false;
  const int C = out_channels(R);
  return row_vec(C, R.out) == 0 && C <= kStageC && (ctl == 5 ? C >= 5 : ctl == 4 && C >= 9);
}

static int launch_coarse(const mer_plan* P, const mer_view* views, const ResolveOut& R, void* ws, hipStream_t st) {
  char* w = (char*)ws;
  long long* tri_base = (long long*)(w + P->off_viewtab);
  long long* tile_base = tri_base + (P->n_views + 1);
  long long* status = (long long*)(w + P->off_status);
  const CoarsePlan cp = coarse_plan(P);
  const Counts count = {(int2*)(w + cp.off_count), cp.count_shift};
  CTile* tiles = (CTile*)(w + cp.off_tile);
  uint2* seg = (uint2*)(w + P->off_rec);
  int* bins = (int*)(w + P->off_bins);
  int* seg_n = (int*)(w + P->off_bign);
  int* large = (int*)(w + P->off_bigflat);
  CItem* items = (CItem*)(w + cp.off_item);
  unsigned long long* key = (unsigned long long*)(w + P->off_key) - P->px_begin;  // by pixel
  const int ctl = cp.ctl;
  const long long nt = cp.n;
  const int direct = direct_tiles(P, nt);
  if (!direct) {
    hipLaunchKernelGGL(k_cinit, dim3(1 + (unsigned)min((nt + 1023) / 1024, 512ll)), dim3(1024), 0, st, views, P->n_views,
                       ctl, tri_base, tile_base, status, count, nt, items, (int)cp.n_items);
    if (P->total_tris > 0) {
      hipLaunchKernelGGL(k_ccount, dim3((unsigned)P->n_bingroups), dim3(kBinBlock), 0, st, views, P->n_views, R.v, R.tri,
                         tri_base, tile_base, (int)P->total_tris, ctl, count, seg, seg_n, large, status);
      hipLaunchKernelGGL(k_clarge, dim3(kLargeGrid), dim3(kBinBlock), 0, st, views, P->n_views, R.v, R.tri, tri_base,
                         tile_base, ctl, large, status, count);
    }
    hipLaunchKernelGGL(k_calloc, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, st, views, P->n_views, ctl, tile_base,
                       nt, count, P->bin_cap, tiles, (int)cp.item, (int)cp.n_items, items, key, status);
    if (P->total_tris > 0)
      hipLaunchKernelGGL(k_cfill, dim3((unsigned)P->n_bingroups + kLargeGrid), dim3(kBinBlock), 0, st, views, P->n_views,
                         R.v, R.tri, tri_base, tile_base, ctl, (int)P->n_bingroups, count, seg, seg_n, large, status,
                         tiles, bins);
  }
  // Parts go first in the grid, so as not to be its tail (1.8 M triangles over
  // 64 px: 104 us, 109 when last), but last where there is room for few, since
  // in front they delay the tiles when there are none: 1936 of them by 3 us.
  const int n_split = direct ? 0 : (int)cp.n_items, split0 = n_split >= 2048 ? 0 : (int)nt;
#define MER_CRASTER(CTL, ST)                                                                                          \
  hipLaunchKernelGGL((k_craster<CTL, 256, ST>), dim3((unsigned)(nt + n_split)), dim3(256), 0, st, views, tiles,       \
                     count, bins, tri_base, direct, R, split0, n_split, (int)nt, items, key, status)
  const bool staged = staged_rows(R, ctl);
  if (ctl == 5 && staged) MER_CRASTER(5, true);
  else if (ctl == 5) MER_CRASTER(5, false);
  else if (ctl == 4 && staged) MER_CRASTER(4, true);
  else if (ctl == 4) MER_CRASTER(4, false);
  else MER_CRASTER(3, false);
#undef MER_CRASTER
  return hipGetLastError() == hipSuccess ? MER_OK : MER_ELAUNCH;
}

}  // namespace mer
