// Trilinear gather of one grid level for one lane (Sec. 3.1; coefficient
// vector and Jacobian of the supplementary "Second-order Grid Sampler").
#pragma once
#include "device.h"

namespace gs {

// per-lane gather state of one level
struct LevelSample {
  float f[3];
  long long row;   // corner 000
  int sy, sz;      // row strides of +y, +z corners
  int cell3[3];    // cell indices
  float inv_v;
};

// Sizes of the grid level one lane works on.  The by-value grid description
// lives in the kernel-argument segment; indexing its per-level arrays with a
// per-lane level makes the compiler read them from memory at every use, and
// such a read waits for all earlier memory operations of the wave (the
// scatter's atomics included, which share the vector-memory counter).  So each
// entry is read once as a wave-uniform scalar and the lane's value selected in
// registers.
struct LevelConst {
  int n[3];
  float voxel, inv_v;   // inv_v: 1 / voxel, correctly rounded
  long long off;
};

__device__ __forceinline__ int uniform_i(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int pick_level(const int (&a)[4], int q) {
  const int v0 = uniform_i(a[0]), v1 = uniform_i(a[1]), v2 = uniform_i(a[2]), v3 = uniform_i(a[3]);
  return q == 0 ? v0 : q == 1 ? v1 : q == 2 ? v2 : v3;
}

__device__ __forceinline__ LevelConst level_const(const Grid& g, int q) {
  LevelConst c;
  c.n[0] = pick_level(g.nx, q);
  c.n[1] = pick_level(g.ny, q);
  c.n[2] = pick_level(g.nz, q);
  const int vb[4] = {__float_as_int(g.voxel[0]), __float_as_int(g.voxel[1]), __float_as_int(g.voxel[2]),
                     __float_as_int(g.voxel[3])};
  c.voxel = __int_as_float(pick_level(vb, q));
  c.inv_v = 1.f / c.voxel;
  const int lo[4] = {(int)g.off[0], (int)g.off[1], (int)g.off[2], (int)g.off[3]};
  const int hi[4] = {(int)(g.off[0] >> 32), (int)(g.off[1] >> 32), (int)(g.off[2] >> 32), (int)(g.off[3] >> 32)};
  c.off = (long long)(((unsigned long long)(unsigned)pick_level(hi, q) << 32) | (unsigned)pick_level(lo, q));
  return c;
}

// x / v, correctly rounded, for v with y = 1 / v correctly rounded: two
// residual corrections of x * y (Markstein's method: the first leaves the
// quotient within an ulp, the second rounds it correctly).  The cell a point
// falls in hangs on this rounding.  5 instructions where the compiler's general
// division takes about 11, three of them per level and point.
__device__ __forceinline__ float div_voxel(float x, float v, float y) {
  float q = x * y;
  q = fmaf(fmaf(-q, v, x), y, q);
  return fmaf(fmaf(-q, v, x), y, q);
}

__device__ __forceinline__ void locate(const Grid& g, const LevelConst& lc, float x, float y, float z,
                                       LevelSample& ls) {
  const float xyz[3] = {x, y, z};
  const float v = lc.voxel;
  int i0[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float u = div_voxel(xyz[a] - g.p0[a], v, lc.inv_v);
    int c = (int)floorf(u);
    c = c < 0 ? 0 : (c > lc.n[a] - 2 ? lc.n[a] - 2 : c);
    i0[a] = c;
    ls.f[a] = u - (float)c;
  }
  ls.sy = lc.n[0];
  ls.sz = lc.n[0] * lc.n[1];
  ls.row = lc.off + ((long long)i0[2] * lc.n[1] + i0[1]) * lc.n[0] + i0[0];
#pragma unroll
  for (int a = 0; a < 3; ++a) ls.cell3[a] = i0[a];
  ls.inv_v = lc.inv_v;
}

__device__ __forceinline__ float comp(const float4& v, int k) {
  return k == 0 ? v.x : (k == 1 ? v.y : (k == 2 ? v.z : v.w));
}

// Off-diagonal second derivatives d^2 z_k / dx_a dx_b of one level (the
// supplementary's h12, h13, h23; the diagonal is zero), in world units.
struct LevelHess {
  float h[4][3];   // [feature][h12, h13, h23]
};

// trilinear value (z) and, optionally, dz/dx (G[k][axis]) and the second
// derivatives (H) of one level.  Value and first derivatives are weighted sums
// over the corners: decoder units near 0 hang on the value's last bit, and
// differences interpolated along the axes, 36 instructions fewer for the
// derivatives, moved single gradient entries of small batches by 1e-3.  The
// second derivatives share their differences (18 instructions a feature, 24
// apart).
template <bool NEED_G, bool BF, bool NEED_H = false>
__device__ __forceinline__ void interp(const float* __restrict__ grid, const uint16_t* __restrict__ grid_bf,
                                       const LevelSample& ls, bool valid, float z[4], float G[4][3],
                                       LevelHess* H = nullptr) {
#pragma unroll
  for (int k = 0; k < 4; ++k) { z[k] = 0.f; G[k][0] = G[k][1] = G[k][2] = 0.f; }
  if constexpr (NEED_H) {
#pragma unroll
    for (int k = 0; k < 4; ++k) H->h[k][0] = H->h[k][1] = H->h[k][2] = 0.f;
  }
  if (!valid) return;
  const float fx = ls.f[0], fy = ls.f[1], fz = ls.f[2];
  float4 th[8];   // corner c = 4 bx + 2 by + bz
#pragma unroll
  for (int e = 0; e < 4; ++e) {   // the edge along x at (by, bz), e = 2 by + bz: two neighbouring rows
    const long long row = ls.row + (long long)(e >> 1) * ls.sy + (long long)(e & 1) * ls.sz;
#pragma unroll
    for (int bx = 0; bx < 2; ++bx) {
      if constexpr (BF) {
        const uint2 u = reinterpret_cast<const uint2*>(grid_bf + row * 4)[bx];
        th[4 * bx + e] = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
                                     __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
      } else {
        th[4 * bx + e] = reinterpret_cast<const float4*>(grid + row * 4)[bx];
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const float wx = c & 4 ? fx : 1.f - fx, wy = c & 2 ? fy : 1.f - fy, wz = c & 1 ? fz : 1.f - fz;
    const float w = wx * wy * wz;
#pragma unroll
    for (int k = 0; k < 4; ++k) z[k] = fmaf(w, comp(th[c], k), z[k]);
    if constexpr (NEED_G) {
      const float jx = (c & 4 ? 1.f : -1.f) * wy * wz, jy = (c & 2 ? 1.f : -1.f) * wx * wz,
                  jz = (c & 1 ? 1.f : -1.f) * wx * wy;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        G[k][0] = fmaf(jx, comp(th[c], k), G[k][0]);
        G[k][1] = fmaf(jy, comp(th[c], k), G[k][1]);
        G[k][2] = fmaf(jz, comp(th[c], k), G[k][2]);
      }
    }
  }
  if constexpr (NEED_G) {
#pragma unroll
    for (int k = 0; k < 4; ++k) { G[k][0] *= ls.inv_v; G[k][1] *= ls.inv_v; G[k][2] *= ls.inv_v; }
  }
  if constexpr (NEED_H) {
    const float iv2 = ls.inv_v * ls.inv_v;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float dz[4];   // difference along z, per 2 bx + by
#pragma unroll
      for (int p = 0; p < 4; ++p) dz[p] = comp(th[2 * p + 1], k) - comp(th[2 * p], k);
      const float dxy = (comp(th[6], k) - comp(th[2], k)) - (comp(th[4], k) - comp(th[0], k));
      const float g0 = dz[1] - dz[0], g1 = dz[3] - dz[2], dxz = dz[2] - dz[0], dxyz = g1 - g0;
      H->h[k][0] = fmaf(fz, dxyz, dxy) * iv2;
      H->h[k][1] = fmaf(fy, dxyz, dxz) * iv2;
      H->h[k][2] = fmaf(fx, dxyz, g0) * iv2;
    }
  }
}

}  // namespace gs
