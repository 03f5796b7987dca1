// Ray batch and smoothness-point sampling on the device.
//
// Philox picks a ray's pixel of any frame, the pixel is back-projected through
// the pinhole, and its samples are the stratified list over the span merged in
// order with the stratified list around the observed depth.  A wave builds one
// ray or a few.  Smoothness pairs are built one per thread.
#include "args.h"

namespace gs {

struct PixelRay {
  float o[3], r[3];
};

// (which product is rounded is written out: the compiler's choice differs
// between kernels, and the rays of a batch do not hang on its kernel)
template <bool POINT>
__device__ __forceinline__ PixelRay pixel_ray(const SampleArgs& A, unsigned long long pix) {
  // (pixel numbers below 2^32 take the 32-bit division, about a fifth of the
  // 64-bit one's instructions)
  const unsigned long long hw = (unsigned long long)A.H * A.W;
  const int f = (pix | hw) >> 32 ? (int)(pix / hw) : (int)((uint32_t)pix / (uint32_t)hw);
  const int rem = (int)(pix - (unsigned long long)f * hw);
  const int v = rem / A.W, u = rem - v * A.W;
  const float* M = A.c2w + 16 * (size_t)f;
  const float dx = ((float)u + 0.5f - A.cx) / A.fx;
  const float dy = ((float)v + 0.5f - A.cy) / A.fy;
  PixelRay pr;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float mx = M[4 * a], my = M[4 * a + 1];
    pr.r[a] = (POINT ? fmaf(mx, dx, my * dy) : fmaf(my, dy, mx * dx)) + M[4 * a + 2];
    pr.o[a] = M[4 * a + 3];
  }
  return pr;
}

__device__ __forceinline__ unsigned long long pick_pixel(uint32_t x, unsigned long long thw) {
  return ((unsigned long long)x * thw) >> 32;
}

// What a ray's samples are drawn from: list a (stratified stream) has ns
// samples, the first ds wide cell starting at a0; list b (near-depth stream) nn,
// likewise.  a: the span, or a confident ray's interval; b: around the observed
// depth, or a confident ray's free space [t_lo, near] before its interval.
struct RayLists {
  float a0, ds, b0, dn;
  int ns, nn;
  int first;   // of its samples among the wave's
  int unit;    // of its units among the wave's
  int base;    // of its samples in the batch
};

__device__ __forceinline__ RayLists ray_lists(const SampleArgs& A, int m, const float o[3], const float r[3],
                                              float D) {
  float tn, tf;
  ray_span(A.g, o, r, A.span_mode, A.near_t, A.far_t, tn, tf);
  const int n_tot = A.n_strat + A.n_near;
  const bool proposed = A.prop3 != nullptr && A.prop3[3 * m + 2] >= A.conf_thr;
  const bool two = !proposed && D > 0.f && A.n_near > 0;
  RayLists l;
  l.ns = proposed ? A.n_prop : (two ? A.n_strat : n_tot);
  l.nn = proposed ? A.n_free : (two ? A.n_near : 0);
  l.b0 = D - A.trunc;
  l.dn = (2.f * A.trunc) / (float)(l.nn > 0 ? l.nn : 1);
  if (proposed) {
    const float pn = A.prop3[3 * m], pf = A.prop3[3 * m + 1];
    l.b0 = tn;
    l.dn = (pn - tn) / (float)(l.nn > 0 ? l.nn : 1);
    tn = pn;
    tf = pf;
  }
  l.a0 = tn;
  l.ds = (tf - tn) / (float)l.ns;
  l.first = l.unit = 0;
  l.base = A.prop3 != nullptr ? A.seg[m] : (int)((size_t)m * n_tot);
  return l;
}

// Ray m of the batch: its pixel, ray, colour and depth.
__device__ __forceinline__ void pick_ray(const SampleArgs& A, int m, float o[3], float r[3], float& D) {
  const unsigned long long thw = (unsigned long long)A.T * A.H * A.W;
  const U4 w0 = philox((uint32_t)m, A.step, 0u, 0u, A.k0, A.k1);
  const unsigned long long pix = pick_pixel(w0.x, thw);
  D = A.depth[pix];
  const PixelRay pr = pixel_ray<false>(A, pix);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    o[a] = pr.o[a];
    r[a] = pr.r[a];
    A.o[3 * m + a] = pr.o[a];
    A.r[3 * m + a] = pr.r[a];
    A.rgb_out[3 * m + a] = (float)A.rgb[3 * pix + a] / 255.f;
  }
  A.depth_out[m] = D;
  if (A.pixel) A.pixel[m] = (long long)pix;
}

__device__ __forceinline__ void sample_point(const SampleArgs& A, int p);

// Rays of a wave.  A wave's time is mostly the latency of its chain (pixel,
// pose, span, draw, rank), so batches that fill the chip otherwise share it
// between up to 8 rays.  On MI355X 65536 rays of about 27 samples take 18.5 us
// with 8 (30 us with one Philox block per sample and two rays a wave).  Whole
// sampling calls with one ray a wave below 16384 rays and with two from 4096 on:
// 12133 proposal rays 40.8 and 39.0 us, 16000 importance rays 120 and 114 us; from
// 1024 to 6144 rays they differ by less than 1 us.
constexpr int kRaysPerWave = 8;

inline int rays_per_wave(int M) {
  const int n = M / 2048;
  return n < 1 ? 1 : (n > kRaysPerWave ? kRaysPerWave : n);
}

// A wave builds the samples of R neighbouring rays: one lane per ray for what
// the ray's samples are drawn from (RAY: it also picks the pixel and writes the
// ray), then one lane per sample of all of them.  Every sample value is
// computed by one lane; its place in the merged order is its index in its own
// list plus the number of values of the other list that precede it (stratified
// first on ties), counted on the same float32 values, so the ranks form a
// permutation.  With a proposal, confident rays get n_prop stratified samples
// in [near, far] and their first sample comes from the precomputed seg.
// 6144 rays of 96 samples: 9.4 us with 16384 points, 26.5 us when arrays indexed
// by lane made the compiler place them in LDS (its addressing reads the launch
// packet from host memory, 8 us in each wave) and the points had their launch.
// cap: LDS floats of a wave, R times the most samples a ray can have.
// RAY: the blocks from ray_blocks on build the smoothness points.
template <bool RAY>
__global__ __launch_bounds__(256) void sample_rays_kernel(SampleArgs A, int R, int cap, int ray_blocks) {
  if constexpr (RAY) {
    if ((int)blockIdx.x >= ray_blocks) {
      sample_point(A, ((int)blockIdx.x - ray_blocks) * 256 + threadIdx.x);
      return;
    }
  }
  extern __shared__ float lists[];
  __shared__ RayLists rays[4][kRaysPerWave];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int m0 = (blockIdx.x * 4 + wv) * R;
  if (m0 >= A.M) return;
  const int nr = min(R, A.M - m0);
  float* list = lists + wv * cap;   // the stratified list of a ray followed by its near-depth one
  RayLists* L = rays[wv];
  if (lane < nr) {
    const int m = m0 + lane;
    float o[3], r[3], D;
    if constexpr (RAY) {
      pick_ray(A, m, o, r, D);
    } else {
#pragma unroll
      for (int a = 0; a < 3; ++a) { o[a] = A.o[3 * m + a]; r[a] = A.r[3 * m + a]; }
      D = A.depth_out[m];
    }
    RayLists l = ray_lists(A, m, o, r, D);
    const int n = l.ns + l.nn, nu = ((l.ns + 3) >> 2) + ((l.nn + 3) >> 2);
    int end = n, uend = nu;   // inclusive sums over the wave's rays
#pragma unroll
    for (int d = 1; d < kRaysPerWave; d <<= 1) {
      const int up = __shfl_up(end, d), uup = __shfl_up(uend, d);
      if (lane >= d) { end += up; uend += uup; }
    }
    l.first = end - n;
    l.unit = uend - nu;
    L[lane] = l;
    if (RAY) {
      A.seg[m] = l.base;
      if (m == A.M - 1) A.seg[A.M] = l.base + n;
    }
  }
  wave_lds_fence();
  const RayLists last = L[nr - 1];
  const int total = last.first + last.ns + last.nn;
  const int units = last.unit + ((last.ns + 3) >> 2) + ((last.nn + 3) >> 2);
  int j = 0;
#pragma unroll 1
  for (int k = lane; k < units; k += 64) {
    while (j + 1 < nr && k >= L[j + 1].unit) ++j;
    const RayLists l = L[j];
    int q = k - l.unit;
    const int qa = (l.ns + 3) >> 2;
    const bool b = q >= qa;
    q = b ? q - qa : q;
    const U4 w = philox((uint32_t)(m0 + j), A.step, b ? 2u : 1u, (uint32_t)q, A.k0, A.k1);
    const uint32_t x[4] = {w.x, w.y, w.z, w.w};
    const int n = b ? l.nn : l.ns;
    float* to = list + l.first + (b ? l.ns : 0);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = 4 * q + c;
      if (i < n) to[i] = (b ? l.b0 : l.a0) + ((float)i + u01(x[c])) * (b ? l.dn : l.ds);
    }
  }
  // ranks: stratified value a_i precedes near value b_j iff a_i <= b_j.  Both
  // lists are non-decreasing in float32 (each value is a monotone rounding of
  // an increasing exact value), so a binary search over the other list in LDS
  // gives the same counts as comparing with every value.
  wave_lds_fence();
  j = 0;
#pragma unroll 1
  for (int k = lane; k < total; k += 64) {
    while (j + 1 < nr && k >= L[j + 1].first) ++j;
    const int first = L[j].first, base = L[j].base, ns = L[j].ns, s = k - first;
    const bool b = s >= ns;
    const float v = list[k];
    const float* other = list + first + (b ? 0 : ns);
    int lo = 0, hi = b ? ns : L[j].nn;   // near values strictly below a_i; stratified values at or below b_j
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      const float u = other[mid];
      if (u < v || (b && u == v)) lo = mid + 1;
      else hi = mid;
    }
    A.t[base + (b ? s - ns : s) + lo] = v;
    A.ray_of[base + s] = m0 + j;
  }
}

// Rays and smoothness points only (proposal mode, before the proposal runs):
// one thread per ray, exactly as the kernel above picks them, and the blocks
// from ray_blocks on for the points.
__global__ __launch_bounds__(256) void sample_pixels_kernel(SampleArgs A, int ray_blocks) {
  if ((int)blockIdx.x >= ray_blocks) {
    sample_point(A, ((int)blockIdx.x - ray_blocks) * 256 + threadIdx.x);
    return;
  }
  const int m = blockIdx.x * 256 + threadIdx.x;
  if (m >= A.M) return;
  float o[3], r[3], D;
  pick_ray(A, m, o, r, D);
}

// One thread per smoothness pair.
__device__ __forceinline__ void sample_point(const SampleArgs& A, int p) {
  if (p >= A.S) return;
  const unsigned long long thw = (unsigned long long)A.T * A.H * A.W;
  int found = -1;
  U4 wf{};
  unsigned long long pix = 0;
  for (int att = 0; att < 8; ++att) {
    const U4 w = philox((uint32_t)p, A.step, 3u, (uint32_t)att, A.k0, A.k1);
    const unsigned long long c = pick_pixel(w.x, thw);
    if (A.depth[c] > 0.f) { found = att; wf = w; pix = c; break; }
  }
  if (found < 0) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      A.xs[3 * p + a] = 0.5f * (A.g.p0[a] + A.g.p1[a]);
      A.eps[3 * p + a] = 0.f;
    }
    return;
  }
  const PixelRay pr = pixel_ray<true>(A, pix);
  const float d = A.depth[pix] + (2.f * u01(wf.y) - 1.f) * A.trunc;
  const float zc = 1.f - 2.f * u01(wf.z);
  const float ph = 6.283185307179586f * u01(wf.w);
  const float rr = sqrtf(fmaxf(0.f, 1.f - zc * zc));
  float sn, cs;
  sincosf(ph, &sn, &cs);
  const float e[3] = {rr * cs, rr * sn, zc};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    A.xs[3 * p + a] = pr.o[a] + d * pr.r[a];
    A.eps[3 * p + a] = A.delta_s * e[a];
  }
}

// Both launches: the smoothness points in blocks after the rays', which spares
// a launch of about 5 us.
static hipError_t launch_rays(const SampleArgs& a, bool pick, hipStream_t st) {
  const int R = rays_per_wave(a.M);
  const int plain = a.n_strat + a.n_near, prop = a.prop3 ? a.n_prop + a.n_free : 0;
  const int cap = R * (plain > prop ? plain : prop);
  const int rays = (a.M + 4 * R - 1) / (4 * R);
  const size_t lds = 4 * (size_t)cap * sizeof(float);
  if (pick) {
    const int points = (a.S + 255) / 256;
    hipLaunchKernelGGL(sample_rays_kernel<true>, dim3(rays + points), dim3(256), lds, st, a, R, cap, rays);
  } else {
    hipLaunchKernelGGL(sample_rays_kernel<false>, dim3(rays), dim3(256), lds, st, a, R, cap, rays);
  }
  return hipGetLastError();
}

hipError_t launch_sample(const SampleArgs& a, hipStream_t st) { return launch_rays(a, true, st); }

// proposal mode: rays first, then (after inference and the seg scan) samples
hipError_t launch_sample_rays_only(const SampleArgs& a, hipStream_t st) {
  const int rays = (a.M + 255) / 256;
  hipLaunchKernelGGL(sample_pixels_kernel, dim3(rays + (a.S + 255) / 256), dim3(256), 0, st, a, rays);
  return hipGetLastError();
}

hipError_t launch_sample_gen_only(const SampleArgs& a, hipStream_t st) { return launch_rays(a, false, st); }

}  // namespace gs
