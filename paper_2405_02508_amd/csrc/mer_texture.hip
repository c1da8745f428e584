// mer_texture.hip -- deferred texturing: a texture sampled at per-pixel uv
// coordinates (which the interpolator produces from per-vertex uv), and its
// adjoint to the texture and to uv (supplement, "Implementation detail":
// uv interpolated per pixel, then a neural texture sampled in a deferred
// shading step; Sec. 3 lists the texture sampler among the parts the smooth
// term differentiates through).
//
// Bilinear filtering, clamp-to-edge addressing.  Texel (x, y) of a th x tw
// texture is centred at ((x + 1/2) / tw, (y + 1/2) / th); s = u tw - 1/2 and
// t = v th - 1/2 are clamped to [-1, tw] and [-1, th], x0 = floor(s),
// fx = s - x0 (likewise y0, fy), and texels (x0 + i, y0 + j) are read with
// each index clamped into the texture.
#include "mer_internal.h"

namespace mer {

struct TexCell {
  int x[2], y[2];  // clamped texel indices
  float fx, fy;
  bool ok;         // sampled (covered pixel, finite uv)
};

// want == false gives an unsampled cell (indices 0).  The texel coordinate
// is formed in binary64: u * tw for tw ~ 1000 would otherwise lose the
// fraction's low bits (binary32 spacing 2^-14 at 1000).
__device__ __forceinline__ TexCell tex_cell(bool want, float u, float v, int th, int tw) {
  TexCell c;
  c.ok = want && isfinite(u) && isfinite(v);
  double s = c.ok ? (double)u * (double)tw - 0.5 : 0.0;
  double t = c.ok ? (double)v * (double)th - 0.5 : 0.0;
  s = fmin(fmax(s, -1.0), (double)tw);
  t = fmin(fmax(t, -1.0), (double)th);
  const double x0 = floor(s), y0 = floor(t);
  c.fx = (float)(s - x0);
  c.fy = (float)(t - y0);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    c.x[i] = c.ok ? min(max((int)x0 + i, 0), tw - 1) : 0;
    c.y[i] = c.ok ? min(max((int)y0 + i, 0), th - 1) : 0;
  }
  return c;
}

// Pixel p's view (searched once per wave, then per lane only across a view
// end) and whether p lies inside it (not in a gap between views).
__device__ __forceinline__ bool pixel_in_view(const mer_view* views, int n_views, long long p, int wvi) {
  int vi = wvi;
  if (vi + 1 < n_views && p >= views[vi + 1].px_off) vi = find_view_px(views, n_views, p);
  const mer_view& vw = views[vi];
  const long long local = p - vw.px_off;
  return local >= 0 && local < (long long)vw.H * vw.W;
}

// ---------------------------------------------------------------- forward
// One thread per pixel: out[p, :] = bilinear sample, or 0.  V4: C is a
// multiple of 4 and tex, out are 16-byte aligned, so texel rows and output
// rows move as float4.
template <bool V4>
__global__ void __launch_bounds__(256) k_texture(const mer_view* __restrict__ views, int n_views,
                                                 const int32_t* __restrict__ tri_id, const float* __restrict__ uv,
                                                 int ld_uv, const float* __restrict__ tex, int th, int tw, int C,
                                                 float* __restrict__ out, long long px_begin, long long total_px) {
  const long long p = px_begin + (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int wvi = wave_view(views, n_views, p - (threadIdx.x & 63));
  // the wave's view through scalar loads; lanes past its end (a wave across
  // two views) look theirs up
  const long long off0 = views[wvi].px_off, n0 = (long long)views[wvi].H * views[wvi].W;
  bool in = p < total_px && p - off0 < n0;
  if (__builtin_amdgcn_ballot_w64(p < total_px && p - off0 >= n0))
    in = p < total_px && pixel_in_view(views, n_views, p, wvi);
  if (!in) return;
  float* o = out + p * C;
  // the uv row (every pixel has one) and the index in flight together
  const float u = uv[p * ld_uv], v = uv[p * ld_uv + 1];
  const int tid = tri_id ? tri_id[p] : 0;
  const bool want = tid >= 0;
  const TexCell cell = tex_cell(want, u, v, th, tw);
  if (!cell.ok) {
    if constexpr (V4) {
      for (int c = 0; c < C; c += 4) *reinterpret_cast<float4*>(o + c) = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
      for (int c = 0; c < C; ++c) o[c] = 0.f;
    }
    return;
  }
  const float w00 = (1.0f - cell.fx) * (1.0f - cell.fy), w10 = cell.fx * (1.0f - cell.fy);
  const float w01 = (1.0f - cell.fx) * cell.fy, w11 = cell.fx * cell.fy;
  const float* t00 = tex + ((long long)cell.y[0] * tw + cell.x[0]) * C;
  const float* t10 = tex + ((long long)cell.y[0] * tw + cell.x[1]) * C;
  const float* t01 = tex + ((long long)cell.y[1] * tw + cell.x[0]) * C;
  const float* t11 = tex + ((long long)cell.y[1] * tw + cell.x[1]) * C;
  if constexpr (V4) {
    auto mix = [&](float4 a, float4 b, float4 d, float4 e) {
      float4 r;
      r.x = (w00 * a.x + w10 * b.x) + (w01 * d.x + w11 * e.x);
      r.y = (w00 * a.y + w10 * b.y) + (w01 * d.y + w11 * e.y);
      r.z = (w00 * a.z + w10 * b.z) + (w01 * d.z + w11 * e.z);
      r.w = (w00 * a.w + w10 * b.w) + (w01 * d.w + w11 * e.w);
      return r;
    };
    auto ld = [](const float* q) { return *reinterpret_cast<const float4*>(q); };
    int c = 0;
    for (; c + 8 <= C; c += 8) {  // eight channels: all eight texel loads before the arithmetic
      const float4 a0 = ld(t00 + c), b0 = ld(t10 + c), d0 = ld(t01 + c), e0 = ld(t11 + c);
      const float4 a1 = ld(t00 + c + 4), b1 = ld(t10 + c + 4), d1 = ld(t01 + c + 4), e1 = ld(t11 + c + 4);
      *reinterpret_cast<float4*>(o + c) = mix(a0, b0, d0, e0);
      *reinterpret_cast<float4*>(o + c + 4) = mix(a1, b1, d1, e1);
    }
    if (c < C) *reinterpret_cast<float4*>(o + c) = mix(ld(t00 + c), ld(t10 + c), ld(t01 + c), ld(t11 + c));
  } else {
    for (int c = 0; c < C; ++c) o[c] = (w00 * t00[c] + w10 * t10[c]) + (w01 * t01[c] + w11 * t11[c]);
  }
}

// --------------------------------------------------------------- backward
// One workgroup per 16x16 pixel tile of one view.  g_uv is written per
// pixel.  The texture gradient is summed in LDS over the box of texels the
// tile touches when that box holds at most kTexWin values (then one global
// atomic per touched texel channel), else added straight to memory.
//
// The LDS sums are 64-bit fixed point: LDS float atomics cost about one
// cycle per active lane on this chip, integer ones a few cycles per
// instruction.  With M the tile's largest |dL/d(out)| (every contribution
// w g has |w g| <= M, and a texel takes at most 4 x 256 of them) and
// M < 2^e, contributions are scaled by 2^(51 - e) and rounded to integers:
// the sums stay below 2^61, each contribution is rounded by at most
// 2^(e - 52) <= 2^-51 M, and the sum is exact and independent of order.  A
// tile with a non-finite dL/d(out) adds straight to memory instead.
//
// Bound now by the L2's float atomics: a 16 x 16 tile at one texel per pixel
// flushes about 160 requests of 16 floats, 15.5 M on 96 scenes (35.8 M px),
// 0.8 ms at the 19.2 G/s that a plain kernel of atomic adds reaches; the
// kernel takes 0.94 ms, 1.28 when it formed each contribution in five
// operations, reduced the tile's box through LDS and divided in the flush.
constexpr int kTexWin = 3072;

// round(w g) to the nearest integer (ties to even) for |w g| < 2^51, as the
// bits of a 64-bit integer: w g + 1.5 2^52 lies in [2^52, 2^53), where the
// binary64 spacing is 1, so the one rounding of the fused multiply-add (the
// product is exact in it) is the rounding to an integer, and the integer is
// the difference of the sum's bits and the constant's, whose low word is 0.
// w is the weight times the tile's scale, g the gradient, both in binary64:
// two operations per contribution where forming w g in binary32, converting
// and subtracting 64 bits took five.
__device__ __forceinline__ unsigned long long fixed_round(double w, double g) {
  const double magic = 6755399441055744.0;  // 1.5 * 2^52
  const unsigned long long bits = (unsigned long long)__double_as_longlong(fma(w, g, magic));
  return (unsigned long long)((unsigned)(bits >> 32) - 0x43380000u) << 32 | (unsigned)bits;
}

// floor(i / d) for i < 2^16, 2 <= d < 2^16 by a high product with
// m = ceil(2^32 / d): i (m d - 2^32) < 2^32.  d = 1 has m = 0.
__device__ __forceinline__ unsigned div_magic(unsigned d) { return d > 1 ? 0xffffffffu / d + 1u : 0u; }
__device__ __forceinline__ unsigned div_by(unsigned i, unsigned m) { return m ? __umulhi(i, m) : i; }

template <bool V4>
__global__ void __launch_bounds__(256) k_texture_bwd(const mer_view* __restrict__ views, int n_views,
                                                     const long long* __restrict__ btile_base,
                                                     const int32_t* __restrict__ tri_id,
                                                     const float* __restrict__ uv, int ld_uv,
                                                     const float* __restrict__ tex, int th, int tw, int C,
                                                     const float* __restrict__ g_out, float* __restrict__ g_tex,
                                                     float* __restrict__ g_uv) {
  __shared__ __align__(16) unsigned long long s_acc[kTexWin];
  __shared__ int4 s_box[4];        // per wave: x min, y min, x max, y max
  __shared__ unsigned s_gmax[4];   // per wave: bits of max |g|
  const long long tile = xcd_tile(blockIdx.x, gridDim.x);
  long long local_tile;
  const int vi = tile_view(btile_base, n_views, tile, local_tile);
  const mer_view vw = views[vi];
  const int tiles_x = (vw.W + 15) >> 4;
  int px, py;
  grid_xy(local_tile, tiles_x, px, py);
  px = px * 16 + (threadIdx.x & 15);
  py = py * 16 + (threadIdx.x >> 4);
  const bool inside = px < vw.W && py < vw.H;
  const long long p = vw.px_off + (long long)py * vw.W + px;

  const long long pc = inside ? p : vw.px_off;
  const int tid = inside && tri_id ? tri_id[p] : 0;
  const bool want = inside && tid >= 0;
  const TexCell cell = tex_cell(want, uv[pc * ld_uv], uv[pc * ld_uv + 1], th, tw);
  const float* g = g_out + (cell.ok ? p : 0) * C;
  const float w00 = (1.0f - cell.fx) * (1.0f - cell.fy), w10 = cell.fx * (1.0f - cell.fy);
  const float w01 = (1.0f - cell.fx) * cell.fy, w11 = cell.fx * cell.fy;
  const long long r00 = ((long long)cell.y[0] * tw + cell.x[0]) * C, r10 = ((long long)cell.y[0] * tw + cell.x[1]) * C;
  const long long r01 = ((long long)cell.y[1] * tw + cell.x[0]) * C, r11 = ((long long)cell.y[1] * tw + cell.x[1]) * C;

  // dL/duv and the largest |dL/d(out)| in one pass over the channels (an
  // infinity or NaN sorts above every finite value by its bits)
  unsigned gmax = 0u;
  float du = 0.f, dv = 0.f;
  if (cell.ok) {
    if constexpr (V4) {
      for (int c = 0; c < C; c += 4) {
        const float4 gg = *reinterpret_cast<const float4*>(g + c);
        const float gs[4] = {gg.x, gg.y, gg.z, gg.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) gmax = max(gmax, __float_as_uint(gs[k]) & 0x7fffffffu);
        if (g_uv) {
          const float4 a = *reinterpret_cast<const float4*>(tex + r00 + c);
          const float4 b = *reinterpret_cast<const float4*>(tex + r10 + c);
          const float4 d = *reinterpret_cast<const float4*>(tex + r01 + c);
          const float4 f = *reinterpret_cast<const float4*>(tex + r11 + c);
          const float t00[4] = {a.x, a.y, a.z, a.w}, t10[4] = {b.x, b.y, b.z, b.w};
          const float t01[4] = {d.x, d.y, d.z, d.w}, t11[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            du += gs[k] * ((1.0f - cell.fy) * (t10[k] - t00[k]) + cell.fy * (t11[k] - t01[k]));
            dv += gs[k] * ((1.0f - cell.fx) * (t01[k] - t00[k]) + cell.fx * (t11[k] - t10[k]));
          }
        }
      }
    } else {
      for (int c = 0; c < C; ++c) {
        gmax = max(gmax, __float_as_uint(g[c]) & 0x7fffffffu);
        if (g_uv) {
          const float t00 = tex[r00 + c], t10 = tex[r10 + c], t01 = tex[r01 + c], t11 = tex[r11 + c];
          du += g[c] * ((1.0f - cell.fy) * (t10 - t00) + cell.fy * (t11 - t01));
          dv += g[c] * ((1.0f - cell.fx) * (t01 - t00) + cell.fx * (t11 - t10));
        }
      }
    }
  }
  if (g_uv && inside) {
    g_uv[2 * p] = du * (float)tw;
    g_uv[2 * p + 1] = dv * (float)th;
  }
  if (!g_tex) return;  // uniform: every thread leaves before the barriers

  // the tile's box of texels and largest |dL/d(out)|: a reduction per wave in
  // registers, then the four waves' values (texel indices are below 2^31)
  const unsigned far = 0x7fffffffu;
  const unsigned bx = wave_min_u32(cell.ok ? (unsigned)cell.x[0] : far), by = wave_min_u32(cell.ok ? (unsigned)cell.y[0] : far);
  const unsigned ex = wave_max_u32(cell.ok ? (unsigned)cell.x[1] : 0u), ey = wave_max_u32(cell.ok ? (unsigned)cell.y[1] : 0u);
  const unsigned gm = wave_max_u32(gmax);
  if ((threadIdx.x & 63) == 0) {
    s_box[threadIdx.x >> 6] = make_int4((int)bx, (int)by, (int)ex, (int)ey);
    s_gmax[threadIdx.x >> 6] = gm;
  }
  __syncthreads();
  int4 box = s_box[0];
  unsigned Mb = s_gmax[0];
#pragma unroll
  for (int i = 1; i < 4; ++i) {
    const int4 o = s_box[i];
    box = make_int4(min(box.x, o.x), min(box.y, o.y), max(box.z, o.z), max(box.w, o.w));
    Mb = max(Mb, s_gmax[i]);
  }
  const int bx0 = box.x, by0 = box.y;
  const bool any = bx0 != 0x7fffffff;
  if (!any || Mb == 0u) return;  // nothing to add (uniform)
  const long long bw = (long long)box.z - bx0 + 1, bh = (long long)box.w - by0 + 1;
  const long long nwin = bw * bh * C;
  if (nwin > kTexWin || Mb >= 0x7f800000u) {
    // Straight to memory (uniform: the whole workgroup is here).  Each wave
    // stages its pixels' four (texel row, weight) pairs in the window's LDS,
    // then adds them channel-fastest: lanes l and l + 1 take channels c and
    // c + 1 of one pair, so an instruction falls on the few cache lines of
    // 64 / C texel rows (one L2 atomic request per line) instead of on one
    // line per lane.
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    long long* s_row = reinterpret_cast<long long*>(s_acc) + wv * 320;  // 256 texel rows (-1: none), 64 g rows
    float* s_w = reinterpret_cast<float*>(s_acc + 4 * 320) + wv * 256;  // 256 weights
    const long long rr[4] = {r00, r10, r01, r11};
    const float ww[4] = {w00, w10, w01, w11};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      s_row[4 * ln + k] = cell.ok ? rr[k] : -1;
      s_w[4 * ln + k] = ww[k];
    }
    s_row[256 + ln] = cell.ok ? p * C : 0;
    __syncthreads();
    const int dq = 64 / C, dr = 64 % C;  // (pair, channel) steps per 64 values
    int pr = ln / C, c = ln % C;
    for (int i = ln; i < 256 * C; i += 64) {
      const long long r = s_row[pr];
      if (r >= 0) {
        const float gc = g_out[s_row[256 + (pr >> 2)] + c];
        if (gc != 0.f) atomicAdd(g_tex + r + c, s_w[pr] * gc);
      }
      pr += dq;
      c += dr;
      if (c >= C) {
        c -= C;
        ++pr;
      }
    }
    return;
  }
  int e;
  frexpf(__uint_as_float(Mb), &e);  // M < 2^e
  const int sh = 51 - e;
  const double scale = ldexp(1.0, sh);
  for (int i = threadIdx.x; i < ((int)nwin + 1) / 2; i += blockDim.x) reinterpret_cast<int4*>(s_acc)[i] = make_int4(0, 0, 0, 0);
  __syncthreads();
  // channel-major window (value c of texel i at c * ncell + i): the lanes of
  // a wave touch neighbouring texels, which then sit 8 bytes apart in LDS
  // rather than C * 8 bytes (with C = 8, four banks for the whole wave)
  const int ncell = (int)(bw * bh), bwi = (int)bw;
  if (cell.ok) {
    const int l00 = (cell.y[0] - by0) * bwi + (cell.x[0] - bx0), l10 = l00 + (cell.x[1] - cell.x[0]);
    const int down = (cell.y[1] - cell.y[0]) * bwi, l01 = l00 + down, l11 = l10 + down;
    // |w g 2^sh| < 2^51: the product is exact in the multiply-add, rounded to
    // the nearest integer by it
    const double d00 = (double)w00 * scale, d10 = (double)w10 * scale, d01 = (double)w01 * scale, d11 = (double)w11 * scale;
    auto add = [&](int c, float gc) {
      unsigned long long* a = s_acc + c * ncell;
      const double gd = (double)gc;
      atomicAdd(a + l00, fixed_round(d00, gd));
      atomicAdd(a + l10, fixed_round(d10, gd));
      atomicAdd(a + l01, fixed_round(d01, gd));
      atomicAdd(a + l11, fixed_round(d11, gd));
    };
    if constexpr (V4) {
      // the row four channels a load, every load issued before the adds
      for (int c0 = 0; c0 < C; c0 += 8) {
        const float4 ga = *reinterpret_cast<const float4*>(g + c0);
        const float4 gb = c0 + 4 < C ? *reinterpret_cast<const float4*>(g + c0 + 4) : make_float4(0.f, 0.f, 0.f, 0.f);
        add(c0, ga.x);
        add(c0 + 1, ga.y);
        add(c0 + 2, ga.z);
        add(c0 + 3, ga.w);
        if (c0 + 4 < C) {
          add(c0 + 4, gb.x);
          add(c0 + 5, gb.y);
          add(c0 + 6, gb.z);
          add(c0 + 7, gb.w);
        }
      }
    } else {
      for (int c = 0; c < C; ++c) add(c, g[c]);
    }
  }
  __syncthreads();
  // the flush walks texel-major, so a wave's global atomics stay contiguous;
  // 32-bit divisions by the channel count and the box width as products
  const unsigned mC = div_magic((unsigned)C), mW = div_magic((unsigned)bwi);
  float* gt = g_tex + ((long long)by0 * tw + bx0) * C;
  for (unsigned i = threadIdx.x; i < (unsigned)nwin; i += blockDim.x) {
    const unsigned ci = div_by(i, mC), c = i - ci * (unsigned)C;
    const long long q = (long long)s_acc[c * (unsigned)ncell + ci];
    if (q == 0) continue;
    const unsigned y = div_by(ci, mW), x = ci - y * (unsigned)bwi;
    atomicAdd(gt + ((long long)y * tw + x) * C + c, (float)ldexp((double)q, -sh));
  }
}

int launch_texture(const mer_plan* P, const mer_view* views, const int32_t* tri_id, const float* uv, int ld_uv,
                   const float* tex, int th, int tw, int C, float* out, hipStream_t st) {
  const long long n = P->total_px - P->px_begin;
  const bool v4 = C % 4 == 0 && ((uintptr_t)tex % 16) == 0 && ((uintptr_t)out % 16) == 0;
  if (n > 0) {
    if (v4)
      hipLaunchKernelGGL(k_texture<true>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, views, P->n_views,
                         tri_id, uv, ld_uv, tex, th, tw, C, out, P->px_begin, P->total_px);
    else
      hipLaunchKernelGGL(k_texture<false>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, views, P->n_views,
                         tri_id, uv, ld_uv, tex, th, tw, C, out, P->px_begin, P->total_px);
  }
  return hipGetLastError() == hipSuccess ? MER_OK : MER_ELAUNCH;
}

int launch_texture_bwd(const mer_plan* P, const mer_view* views, const int32_t* tri_id, const float* uv, int ld_uv,
                       const float* tex, int th, int tw, int C, const float* g_out, float* g_tex, float* g_uv,
                       void* ws, hipStream_t st) {
  long long* tab = (long long*)((char*)ws + P->off_bviewtab);
  const long long* base = P->n_views > 1 ? tab + (P->n_views + 1) : nullptr;
  if (base)
    hipLaunchKernelGGL(k_prep, dim3(1), dim3(1024), 0, st, views, P->n_views, 4, 4, tab, tab + (P->n_views + 1),
                       (long long*)nullptr);
  const bool v4 = C % 4 == 0 && ((uintptr_t)tex % 16) == 0 && ((uintptr_t)g_out % 16) == 0;
  if (P->total_btiles > 0) {
    if (v4)
      hipLaunchKernelGGL(k_texture_bwd<true>, dim3((unsigned)P->total_btiles), dim3(256), 0, st, views, P->n_views,
                         base, tri_id, uv, ld_uv, tex, th, tw, C, g_out, g_tex, g_uv);
    else
      hipLaunchKernelGGL(k_texture_bwd<false>, dim3((unsigned)P->total_btiles), dim3(256), 0, st, views, P->n_views,
                         base, tri_id, uv, ld_uv, tex, th, tw, C, g_out, g_tex, g_uv);
  }
  return hipGetLastError() == hipSuccess ? MER_OK : MER_ELAUNCH;
}

}  // namespace mer
