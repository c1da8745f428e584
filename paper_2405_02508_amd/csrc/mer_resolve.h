// mer_resolve.h -- what the rasterizers write for a pixel once its visible
// triangle is known: index, depth, barycentrics and interpolated attributes.
#pragma once
#include "mer_device.h"

namespace mer {

// Outputs of a rasterizer's resolve; depth, bary and out may be NULL, attr
// belongs to out.  tail: the channels after the C_a attributes, bit 0 the
// interpolated z, bit 1 the coverage mask (1 where a triangle is visible).
// Written with its row the mask costs nothing; a copy of the image beside it
// and two passes over the index image took 16 us on 512 x 512 of 8 channels.
struct ResolveOut {
  const float* __restrict__ v;
  const int32_t* __restrict__ tri;
  int32_t* __restrict__ tri_id;
  float* __restrict__ depth;
  float* __restrict__ bary;
  const float* __restrict__ attr;
  int C_a, tail;
  float* __restrict__ out;
};

__host__ __device__ __forceinline__ int out_channels(const ResolveOut& R) { return R.C_a + (R.tail & 1) + (R.tail >> 1); }

// Interpolated row of a pixel (triangle t with index row idx, -1 background)
// with perspective barycentrics b0, b1: the arithmetic of the interpolation kernel, four
// channels a load and a store where the channel counts allow.  o: where the
// row goes, vout: the vector width of a store there.
__device__ __forceinline__ void resolve_attr(const ResolveOut& R, const mer_view& vw, float* o, int vout, int t,
                                             float b0, float b1, const int32_t* idx) {
  const int C_a = R.C_a, C = out_channels(R);
  const float* attr = R.attr;
  const bool a_al = ((vw.a_off * C_a) & 3) == 0;
  const int va = row_vec(C_a, attr) == 3 ? 3 : row_vec(C_a, attr) == 4 && a_al ? 4 : 0;
  float b2 = 0.f, zv = 0.f;
  const float *a0 = attr, *a1 = attr, *a2 = attr;
  if (t >= 0) {
    b2 = (1.0f - b0) - b1;
    const int i0 = idx[0], i1 = idx[1], i2 = idx[2];
    a0 = attr + (vw.a_off + i0) * C_a;
    a1 = attr + (vw.a_off + i1) * C_a;
    a2 = attr + (vw.a_off + i2) * C_a;
    if (R.tail & 1) {
      const float* vb = R.v + vw.v_off * 3;
      const float z0 = vb[(size_t)i0 * 3 + 2], z1 = vb[(size_t)i1 * 3 + 2], z2 = vb[(size_t)i2 * 3 + 2];
      zv = (b0 * z0 + b1 * z1) + b2 * z2;
    }
  }
  for (int c0 = 0; c0 < C; c0 += 4) {
    const int n = min(4, C - c0);
    float xs[4] = {0.f, 0.f, 0.f, 0.f};
    if (t >= 0) {
      if (c0 < C_a) {
        const int na = min(4, C_a - c0);
        const float4 x0 = row4(a0 + c0, va, na), x1 = row4(a1 + c0, va, na), x2 = row4(a2 + c0, va, na);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (j < na) xs[j] = (b0 * f4(x0, j) + b1 * f4(x1, j)) + b2 * f4(x2, j);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (c0 + j >= C_a) xs[j] = c0 + j == C_a && (R.tail & 1) ? zv : 1.0f;
    }
    if (vout == 4) {
      *reinterpret_cast<float4*>(o + c0) = make_float4(xs[0], xs[1], xs[2], xs[3]);
    } else if (vout == 3) {
      *reinterpret_cast<float3*>(o + c0) = make_float3(xs[0], xs[1], xs[2]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < n) o[c0 + j] = xs[j];
    }
  }
}

}  // namespace mer
