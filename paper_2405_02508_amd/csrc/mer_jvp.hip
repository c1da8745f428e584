// mer_jvp.hip -- forward mode: the per-pixel image tangent for a tangent of
// the screen vertices (and attributes), i.e. the derivative of every pixel
// with respect to one scene parameter (Sec. 5, "Forward gradients").  It is
// the transpose of the backward sweep: the same micro-edge pairs and
// classification (Sec. 4.2-4.4), with the edge position's tangent in place of
// dL/dp, plus the forward derivative of the interpolation (Sec. 3, the smooth
// term).  One thread per pixel gathers the pairs it belongs to, so every
// output element is written once, with no atomics.
#include "mer_internal.h"

namespace mer {

// Screen barycentrics e_k / |D| at pixel (px, py) of snapped triangle s.
__device__ __forceinline__ void screen_beta(const Snap& s, int px, int py, float beta[3]) {
  const Rel32 r = rel32(s, px, py);
  if (r.ok) {  // the same values from 32-bit edge values (|D| = their sum)
    int E[3];
    edge32(s, r, E);
    const float id = __builtin_amdgcn_rcpf((float)(E[0] + E[1] + E[2]));
#pragma unroll
    for (int k = 0; k < 3; ++k) beta[k] = (float)E[k] * id;
    return;
  }
  long long E[3];
  edge_at(s, px, py, E);
  const long long Dabs = s.D < 0 ? -s.D : s.D;
  const float id = __builtin_amdgcn_rcpf((float)Dabs);
#pragma unroll
  for (int k = 0; k < 3; ++k) beta[k] = (float)E[k] * id;
}

// The three vertices' tangent rows (dx, dy, dz) of snapped triangle s, from
// the view's rows dvb.
struct TriTangent {
  float r[9];
};
__device__ __forceinline__ TriTangent tri_tangent(const float* __restrict__ dvb, const Snap& s) {
  TriTangent g;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float* q = dvb + (size_t)(unsigned)s.idx[k] * 3u;
    g.r[3 * k] = q[0];
    g.r[3 * k + 1] = q[1];
    g.r[3 * k + 2] = q[2];
  }
  return g;
}

// Tangent (x, y, 1/z) of the fragment at pixel (px, py) of snapped triangle
// s: the point with that centre's screen barycentrics moves with its
// vertices, and 1/z_k moves by -(1/z_k)^2 dz_k.
__device__ __forceinline__ void frag_tangent(const TriTangent& g, const Snap& s, int px, int py, float dr[3]) {
  float beta[3];
  screen_beta(s, px, py, beta);
  dr[0] = dr[1] = dr[2] = 0.f;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    dr[0] += beta[k] * g.r[3 * k];
    dr[1] += beta[k] * g.r[3 * k + 1];
    dr[2] += beta[k] * ((-(s.q[k] * s.q[k])) * g.r[3 * k + 2]);
  }
}

// One workgroup per TS x TS tile of one view, one thread per pixel, as in the
// backward sweep: each lane snaps its pixel's triangle once and publishes its
// id and which neighbours' centres it holds; the first 4 TS lanes do so for
// the pixels around the tile.  A pair is classified from one bit of each side,
// and the side that is on top (both at an intersection) publishes its
// fragment's tangent, once for all its pairs; then every pixel takes the edge
// tangents dp of its four pairs (d4) from there, and per channel
//   dimg = interior tangent (c < C_out) + 1/2 sum_dir (I_A - I_B) d_dir
// with A the left/upper pixel of each pair.  Only intersections snap the
// neighbour's triangle, for its plane's slope.
//
// Bound by vector issue: building a table of the tile's distinct triangles in
// LDS first (a hash, then one snap each) and evaluating a pair's tangent on
// both its sides took 795 instructions per wave and 1.28 ms on 128 scenes (54
// M px, 3 channels); this takes 546 and 1.02.
template <int TS>  // side of the tile: 8 or 16
__global__ void __launch_bounds__(TS * TS) __attribute__((amdgpu_waves_per_eu(6))) k_jvp(
    const mer_view* __restrict__ views, int n_views, const long long* __restrict__ btile_base,
    const float* __restrict__ v, const int32_t* __restrict__ tri, const int32_t* __restrict__ tri_id,
    const float* __restrict__ attr, const float* __restrict__ dattr, int C_a, int append_z,
    const float* __restrict__ img, int C_e, const float* __restrict__ dv, int flags, float* __restrict__ dimg) {
  constexpr int NP = TS * TS, kJq = NP + 4 * TS;  // tile pixels, then TS around it per side: left, right, up, down
  __shared__ int s_t[kJq];             // triangle, -1 background, outside the view or one that does not snap
  __shared__ unsigned char s_cm[kJq];  // bit d: that triangle holds the centre of neighbour d (0 left, 1 right, 2 up, 3 down)
  __shared__ float s_dr[3][kJq];       // fragment tangents (x, y, 1/z) of the pixels that are on top of some pair
  // 16 x 16 tiles; of 8 x 8 ones, four workgroups share one
  constexpr int SUB = TS == 8 ? 2 : 0;
  const long long part = xcd_tile(blockIdx.x, gridDim.x);
  long long local_tile;
  const int vi = tile_view(btile_base, n_views, part >> SUB, local_tile);
  const mer_view vw = views[vi];
  int x0, y0;
  grid_xy(local_tile, (vw.W + 15) >> 4, x0, y0);
  x0 = x0 * 16 + (SUB ? ((int)part & 1) * 8 : 0);
  y0 = y0 * 16 + (SUB ? ((int)part >> 1 & 1) * 8 : 0);
  if (SUB && (x0 >= vw.W || y0 >= vw.H)) return;
  const float* dvb = dv ? dv + vw.v_off * 3 : nullptr;
  const int lt = threadIdx.x, lx = lt % TS, ly = lt / TS;
  const int px = x0 + lx, py = y0 + ly;
  const bool inside = px < vw.W && py < vw.H;
  const long long p = vw.px_off + (long long)py * vw.W + px;
  const bool want_edge = dv && !(flags & MER_SKIP_EDGE);
  const bool no_isect = (flags & MER_NO_INTERSECT) != 0;

  // a pixel around the tile (lanes of the first wave): its place, and the
  // tile pixel next to it
  const int side = lt / TS & 3, ri = lt % TS;
  const int ix = side == 0 ? 0 : side == 1 ? TS - 1 : ri, iy = side == 2 ? 0 : side == 3 ? TS - 1 : ri;
  const int qx = x0 + (side == 0 ? -1 : side == 1 ? TS : ri), qy = y0 + (side == 2 ? -1 : side == 3 ? TS : ri);
  if (want_edge && lt < 4 * TS) {
    int rt = -1;
    if (qx >= 0 && qy >= 0 && qx < vw.W && qy < vw.H) rt = tri_id[vw.px_off + (long long)qy * vw.W + qx];
    if (rt >= vw.n_t) rt = -1;
    unsigned rc = 0;
    if (rt >= 0) {
      const Snap R = snap_triangle<false>(v, vw, tri_row(tri, vw, rt));
      if (!R.ok) rt = -1;
      else if (contains(R, x0 + ix, y0 + iy)) rc = 1u << (side ^ 1);
    }
    s_t[NP + lt] = rt;
    s_cm[NP + lt] = (unsigned char)rc;
  }
  int t = inside ? tri_id[p] : -1;
  if (t >= vw.n_t || t < 0) t = -1;
  Snap S;
  S.ok = false;
  if (t >= 0) S = snap_triangle<false>(v, vw, tri_row(tri, vw, t));
  if (!S.ok) t = -1;
  TriTangent gt;
#pragma unroll
  for (int i = 0; i < 9; ++i) gt.r[i] = 0.f;
  if (dv && t >= 0) gt = tri_tangent(dvb, S);

  // ---- micro-edge term: tangent of the edge position of each differing pair
  float d4[4] = {0.f, 0.f, 0.f, 0.f};  // left, right, up, down
  if (want_edge) {
    const unsigned cm = t >= 0 ? cover_mask(S, px, py) : 0u;
    s_t[lt] = t;
    s_cm[lt] = (unsigned char)cm;
    __syncthreads();
    // the place of neighbour d
    auto nq = [&](int d) -> int {
      if (d == 0) return lx > 0 ? lt - 1 : NP + ly;
      if (d == 1) return lx < TS - 1 ? lt + 1 : NP + TS + ly;
      if (d == 2) return ly > 0 ? lt - TS : NP + 2 * TS + lx;
      return ly < TS - 1 ? lt + TS : NP + 3 * TS + lx;
    };
    // One side background: the other is on top.  Both covered: the side whose
    // centre the other triangle holds too, both sides at an intersection;
    // triangles that merely touch have no term.
    auto on_top = [&](int ta, int tb, bool a_holds, bool b_holds) -> bool {  // a of the pair (a, b)
      return (ta >= 0) & (ta != tb) & ((tb < 0) | (b_holds & !(a_holds & no_isect)));
    };
    unsigned self = 0u, other = 0u;  // bit d: this pixel, its neighbour d is on top of their pair
    const bool in_view[4] = {px > 0, px + 1 < vw.W, py > 0, py + 1 < vw.H};
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int q = nq(d), tn = s_t[q];
      const bool mine = (cm >> d) & 1u, theirs = (s_cm[q] >> (d ^ 1)) & 1u, in = inside & in_view[d];
      self |= in & on_top(t, tn, mine, theirs) ? 1u << d : 0u;
      other |= in & on_top(tn, t, theirs, mine) ? 1u << d : 0u;
    }
    if (self) {
      float dr[3];
      frag_tangent(gt, S, px, py, dr);
#pragma unroll
      for (int k = 0; k < 3; ++k) s_dr[k][lt] = dr[k];
    }
    if (lt < 4 * TS) {
      const int rt = s_t[NP + lt], it = iy * TS + ix, ti = s_t[it];
      const bool r_holds = (s_cm[NP + lt] >> (side ^ 1)) & 1u, i_holds = (s_cm[it] >> side) & 1u;
      if (x0 + ix < vw.W && y0 + iy < vw.H && on_top(rt, ti, r_holds, i_holds)) {
        const Snap R = snap_triangle<false>(v, vw, tri_row(tri, vw, rt));
        float dr[3];
        frag_tangent(tri_tangent(dvb, R), R, qx, qy, dr);
#pragma unroll
        for (int k = 0; k < 3; ++k) s_dr[k][NP + lt] = dr[k];
      }
    }
    __syncthreads();  // the tangents are published
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int axis = d >> 1;
      const unsigned both = (self & other) >> d & 1u;
      if (!both && ((self | other) >> d & 1u)) d4[d] = s_dr[axis][(self >> d & 1u) ? lt : nq(d)];
    }
    unsigned isect = self & other;
#pragma unroll 1
    while (isect) {
      const int d = __builtin_ctz(isect);
      isect &= isect - 1;
      const int q = nq(d), axis = d >> 1;
      const bool selfA = d & 1;  // this pixel has the smaller coordinate
      // dp = (-sA drA_axis + drA_q + sB drB_axis - drB_q) / (sB - sA), A the left/upper pixel
      const Snap Sn = snap_triangle<false>(v, vw, tri_row(tri, vw, s_t[q]));
      Snap So = S;
      asm volatile("" : "+v"(So.z[0]), "+v"(So.z[1]), "+v"(So.z[2]), "+v"(So.X[0]), "+v"(So.X[1]), "+v"(So.X[2]),
                   "+v"(So.Y[0]), "+v"(So.Y[1]), "+v"(So.Y[2]), "+v"(So.D));  // the slope stays in this rare branch
      const float s_self = plane_slope(So, axis), s_n = plane_slope(Sn, axis);
      const float sA = selfA ? s_self : s_n, sB = selfA ? s_n : s_self;
      const float dlt = sB - sA;
      if (!(dlt > 0.f) || !isfinite(dlt)) continue;
      const int qA = selfA ? lt : q, qB = selfA ? q : lt;
      const float num = ((-sA) * s_dr[axis][qA] + s_dr[2][qA]) + (sB * s_dr[axis][qB] - s_dr[2][qB]);
      const float dp = num / dlt;
      if (d == 0) d4[0] = dp;
      else if (d == 1) d4[1] = dp;
      else if (d == 2) d4[2] = dp;
      else d4[3] = dp;
    }
  }
  if (!inside) return;

  // ---- interior: forward derivative of sum_k b_k a_kc at the fixed index
  float db[3] = {0.f, 0.f, 0.f}, b[3] = {0.f, 0.f, 0.f};
  float zt = 0.f;  // tangent of the interpolated z
  const bool interior = t >= 0 && !(flags & MER_SKIP_INTERP);
  if (interior) {
    const PixBary pb = pixel_bary(S, px, py);
#pragma unroll
    for (int k = 0; k < 3; ++k) b[k] = pb.b[k];
    if (dv) {
      // the material point at this centre moves by delta = sum_j beta_j dv_j,
      // so beta_i changes by -grad_P beta_i . delta
      float ex = 0.f, ey = 0.f;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        ex += pb.beta[j] * gt.r[3 * j];
        ey += pb.beta[j] * gt.r[3 * j + 1];
      }
      const float invD = 256.0f * __builtin_amdgcn_rcpf(S.D < 0 ? -pb.d : pb.d);  // (float)D, already converted
      float dw[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const int a = (i + 1) % 3, c = (i + 2) % 3;
        const float gxi = (float)(-(S.Y[c] - S.Y[a])) * invD;
        const float gyi = (float)(S.X[c] - S.X[a]) * invD;
        const float dbeta = -(gxi * ex + gyi * ey);
        dw[i] = dbeta * S.q[i] + pb.beta[i] * ((-(S.q[i] * S.q[i])) * gt.r[3 * i + 2]);
      }
      const float dW = (dw[0] + dw[1]) + dw[2];
      const float iW = __builtin_amdgcn_rcpf(pb.Wq);
#pragma unroll
      for (int k = 0; k < 3; ++k) db[k] = (dw[k] - b[k] * dW) * iW;
      if (append_z) {
        zt = (db[0] * S.z[0] + db[1] * S.z[1]) + db[2] * S.z[2];
        zt += (b[0] * gt.r[2] + b[1] * gt.r[5]) + b[2] * gt.r[8];
      }
    }
  }
  const int C_out = (flags & MER_SKIP_INTERP) ? 0 : C_a + append_z;

  // ---- per channel
  const bool has_edge = (d4[0] != 0.f) | (d4[1] != 0.f) | (d4[2] != 0.f) | (d4[3] != 0.f);
  const long long W = vw.W;
  const float* i0 = img ? img + p * C_e : nullptr;
  long long arow[3] = {0, 0, 0};
  if (interior) {
#pragma unroll
    for (int k = 0; k < 3; ++k) arow[k] = (vw.a_off + S.idx[k]) * C_a;
  }
  // four channels at a time, rows as vector loads where the channel counts
  // allow (image rows of C_e floats, attribute and tangent rows of C_a);
  // each channel's arithmetic is the same, in the same order, as one at a time
  const int vimg = img ? row_vec(C_e, img) : 0;
  const bool a_al = ((vw.a_off * C_a) & 3) == 0;
  const int va = row_vec(C_a, attr) == 3 ? 3 : row_vec(C_a, attr) == 4 && a_al ? 4 : 0;
  const int vda = !dattr ? 0 : row_vec(C_a, dattr) == 3 ? 3 : row_vec(C_a, dattr) == 4 && a_al ? 4 : 0;
  const int vout = row_vec(C_e, dimg);
  float* out = dimg + p * C_e;
  for (int c0 = 0; c0 < C_e; c0 += 4) {
    const int n = min(4, C_e - c0);
    float xs[4] = {0.f, 0.f, 0.f, 0.f};
    if (interior && c0 < C_out) {
      if (c0 < C_a) {
        const int na = min(4, C_a - c0);
        const float4 a0 = row4(attr + arow[0] + c0, va, na), a1 = row4(attr + arow[1] + c0, va, na),
                     a2 = row4(attr + arow[2] + c0, va, na);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (j < na) xs[j] = (db[0] * f4(a0, j) + db[1] * f4(a1, j)) + db[2] * f4(a2, j);
        if (dattr) {
          const float4 e0 = row4(dattr + arow[0] + c0, vda, na), e1 = row4(dattr + arow[1] + c0, vda, na),
                       e2 = row4(dattr + arow[2] + c0, vda, na);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (j < na) xs[j] += (b[0] * f4(e0, j) + b[1] * f4(e1, j)) + b[2] * f4(e2, j);
        }
      }
      if (C_out > C_a && C_a >= c0 && C_a < c0 + n) {  // the z channel
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (c0 + j == C_a) xs[j] = zt;
      }
    }
    if (has_edge) {
      const float4 s0 = row4(i0 + c0, vimg, n);
      float e[4] = {0.f, 0.f, 0.f, 0.f};
      if (d4[0] != 0.f) {
        const float4 q = row4(i0 - C_e + c0, vimg, n);
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] += (f4(q, j) - f4(s0, j)) * d4[0];
      }
      if (d4[1] != 0.f) {
        const float4 q = row4(i0 + C_e + c0, vimg, n);
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] += (f4(s0, j) - f4(q, j)) * d4[1];
      }
      if (d4[2] != 0.f) {
        const float4 q = row4(i0 - W * C_e + c0, vimg, n);
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] += (f4(q, j) - f4(s0, j)) * d4[2];
      }
      if (d4[3] != 0.f) {
        const float4 q = row4(i0 + W * C_e + c0, vimg, n);
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] += (f4(s0, j) - f4(q, j)) * d4[3];
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) xs[j] += 0.5f * e[j];
    }
    if (vout == 4) {
      *reinterpret_cast<float4*>(out + c0) = make_float4(xs[0], xs[1], xs[2], xs[3]);
    } else if (vout == 3) {
      *reinterpret_cast<float3*>(out + c0) = make_float3(xs[0], xs[1], xs[2]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < n) out[c0 + j] = xs[j];
    }
  }
}

// Rows that no vector store takes are read and written a float at a time, and
// the wave of a tile that has most of that to do holds its three neighbours'
// place: 8 x 8 tiles, one wave each, finish on their own, though their border
// is half their pixels.  us, 16 x 16 / 8 x 8 tiles (and before either), views of
// 600 x 600 and 1000 x 1000: rows of 2 floats 28 / 28 (2 small views); of 7 52
// / 44 (51), 16 large views 644 / 621 (720); of 11 75 / 60 (65), 8 large 498 /
// 489, 16 978 / 960; of 17 117 / 94 (98), 2 large 222 / 198 (203), 4 483 / 500,
// 16 1823 / 1912 (2004).
static bool small_jvp_tiles(long long tiles16, int C_e, const float* dimg) {
  return row_vec(C_e, dimg) == 0 && C_e >= 5 && (C_e <= 11 || tiles16 <= 8192);
}

int launch_jvp(const mer_plan* P, const mer_view* views, const float* v, const int32_t* tri, const int32_t* tri_id,
               const float* attr, const float* dattr, int C_a, int append_z, const float* img, int C_e,
               const float* dv, int flags, float* dimg, void* ws, hipStream_t st) {
  // 16x16 tile prefix per view (one view needs none); the rasterizer's status
  // words are left alone
  long long* tab = (long long*)((char*)ws + P->off_bviewtab);
  const long long* base = P->n_views > 1 ? tab + (P->n_views + 1) : nullptr;
  if (base)
    hipLaunchKernelGGL(k_prep, dim3(1), dim3(1024), 0, st, views, P->n_views, 4, 4, tab, tab + (P->n_views + 1),
                       (long long*)nullptr);
#define MER_JVP(TS)                                                                                                    \
  hipLaunchKernelGGL(k_jvp<TS>, dim3((unsigned)(P->total_btiles * (256 / (TS * TS)))), dim3(TS * TS), 0, st, views,    \
                     P->n_views, base, v, tri, tri_id, attr, dattr, C_a, append_z, img, C_e, dv, flags, dimg)
  if (P->total_btiles <= 0) return MER_OK;
  if (small_jvp_tiles(P->total_btiles, C_e, dimg)) MER_JVP(8);
  else MER_JVP(16);
#undef MER_JVP
  return hipGetLastError() == hipSuccess ? MER_OK : MER_ELAUNCH;
}

}  // namespace mer
