// Grid scatter of the backward: dL/dtheta_c,k = w_c dz_k + a_k (J_c . gv) / v
// summed over all records (supplementary "Second-order Grid Sampler", the
// first-order block and the J^T block).
//
// What bounds it: float atomics in memory run at about 20 G requests of 64
// bytes per second, and a record spans about 20 such requests (8 corners of 4
// levels), so adding each record to memory costs several times what computing
// it does.  Records are therefore grouped by bin (8^3 cells of the finest
// level) and summed in a window in LDS that holds every vertex the bin uses;
// a window's sums go to memory once per bin and wave.
#include "args.h"
#include "gather.h"

namespace gs {

// ---------------------------------------------------------------- plan
// Window of each level for bins of 2^shift cells of the finest level: a bin
// edge covers `ratio` cells of level l.  Where the edges of cells and bins
// coincide (ratio or its inverse whole, as in grids whose voxels divide each
// other) it uses ratio + 1 vertices (at least 2), otherwise one cell more.
// The largest shift up to 3 whose windows fit the LDS and, along z, the columns
// of a flush is taken; at shift 2 they always do (5^3 vertices of the finest
// level, at most 6^3 of each coarser one).
void plan_bins(const Grid& g, Bins& B) {
  B.level = 0;
  for (int l = 1; l < 4; ++l)
    if (g.voxel[l] < g.voxel[B.level]) B.level = l;
  const int f = B.level;
  const int n[3] = {g.nx[f], g.ny[f], g.nz[f]};
  for (B.shift = 3;; --B.shift) {
    int verts = 0, edge = 0;
    for (int l = 0; l < 4; ++l) {
      const float r = (float)(1 << B.shift) * (g.voxel[f] / g.voxel[l]);
      const float up = floorf(r + 0.5f), inv = floorf(1.f / r + 0.5f);
      int w;
      if (r >= 0.75f && fabsf(r - up) < 1e-3f) w = (int)up + 1;
      else if (r < 0.75f && fabsf(1.f / r - inv) < 1e-3f * inv) w = 2;
      else w = (int)ceilf(r) + 2;
      const int dim[3] = {g.nx[l], g.ny[l], g.nz[l]};
      B.ratio[l] = r;
      B.wbase[l] = verts;
      int c = 1;
      for (int a = 0; a < 3; ++a) {
        B.wd[l][a] = w < dim[a] ? w : dim[a];
        c *= B.wd[l][a];
      }
      verts += c;
      if (B.wd[l][2] > edge) edge = B.wd[l][2];
    }
    if ((verts <= kWinVerts && edge <= kWinEdge) || B.shift == 0) break;
  }
  for (int a = 0; a < 3; ++a) {
    B.nb[a] = ((n[a] - 2) >> B.shift) + 1;
    B.last[a] = n[a] - 2;
    B.p0[a] = g.p0[a];
  }
  B.inv_v = 1.f / g.voxel[f];
}

// Grids so small that many samples share every vertex.
static bool few_bins(long long bins) { return bins <= 256; }

// The points (samples and pair points) from which a batch is scattered through
// records.  Without them the field kernel adds to memory itself, about 8 requests
// per sample overlapped with its decoders; with them it writes records of up to
// 160 bytes, and the scatter's time comes on top, with a share for every bin that
// is touched.  `far`: levels the field kernel would not accumulate in LDS;
// `ragged`: most rays have their samples about the surface (a proposal drew them).
// Measured (MI355X, backward call, us, direct / records), 96 samples per ray and
// 16384 pairs unless stated:
//   room at 3 cm, 16128 bins: 0.59 M samples 352 / 388, 1.57 M 820 / 803,
//     2.1 M 1077 / 1023, 3.1 M 1579 / 1460, 6.3 M 3050 / 2701; no pairs: 1.25 M
//     631 / 662, 1.57 M 786 / 789, 1.82 M 912 / 891
//   at 2 cm, 54432 bins: no pairs 0.79 M 423 / 600, 1.57 M 807 / 908; 2^18 pairs
//     2.1 M 1512 / 1287, 4.2 M 2517 / 2169
//   at 1 cm, 435456 bins, no pairs: 3.1 M 1638 / 2800, 6.3 M 3231 / 4456
//   two levels kept in LDS (6 cm mapping grid): 3.1 M 1122 / 1278, 6.3 M 2241 / 2425
// On a small grid the direct adds queue at few addresses:
//   64 bins, no pairs: 33 k 53 / 68, 66 k 72 / 80, 77 k 82 / 85, 96 k 98 / 90,
//     131 k 123 / 100; 4096 pairs: 74 k 91 / 85, 91 k 103 / 91
//   125 bins: 64 k 74 / 87, 128 k 118 / 103, 192 k 166 / 122
//   64 bins, rays of 24 samples about the surface, whose runs merge before they are
//     added: 104 k 82 / 93, 177 k 114 / 128, 323 k 178 / 171
// The lines lie where the two meet in FP32, a little above it at 3 cm, where they
// run side by side from 1.5 to 2 M.  BF16 decoders take less time to cover the
// direct adds with, and the two meet earlier:
//   3 cm, no pairs: 0.39 M 235 / 238, 0.59 M 328 / 296, 1.57 M 801 / 587; rays of
//     24 or 96 samples: 0.36 M 209 / 216, 0.60 M 300 / 283, 2.4 M 954 / 775
//   2 cm, no pairs: 0.79 M 429 / 502, 1.57 M 822 / 716; 1 cm: 6.3 M 3395 / 3576
// On small grids the two precisions share a line, and two levels in LDS keep BF16
// direct too, where the sides meet at 1.3 M.
long long records_from(const Bins& B, int far, bool bf16, bool ragged) {
  const long long bins = (long long)B.nb[0] * B.nb[1] * B.nb[2];
  if (few_bins(bins)) return (ragged ? 4 : 1) * (50000 + 256 * bins);
  if (far < 3) return 1LL << 62;
  const long long per_bin = (bf16 ? 24 : 48) * bins, least = bf16 ? 1LL << 19 : 1LL << 21;
  return per_bin > least ? per_bin : least;
}

// Slots of the counting table (about 2^14 for grids of fewer bins, see
// bin_slot), the small levels (coarsest first, while their vertices add up to
// at most kSmallVerts), and the arrays in `tables`: queues, counts, copies of
// the small levels, all of which start at zero.  Returns their floats.
long long plan_tables(const Grid& g, ScatterRecords& R, float* tables) {
  const long long n = (long long)R.bins.nb[0] * R.bins.nb[1] * R.bins.nb[2];
  R.spread = 0;
  while ((n << (R.spread + 1)) <= (1 << 14) && R.spread < 8) ++R.spread;
  R.slots = n < kMaxBins ? (int)n << R.spread : kMaxBins;
  R.small_mask = 0;
  R.small_verts = 0;
  for (int l = 0; l < 4; ++l) {
    const long long nv = (long long)g.nx[l] * g.ny[l] * g.nz[l];
    R.small_off[l] = R.small_verts;
    if (R.small_verts + nv > kSmallVerts) continue;
    R.small_mask |= 1 << l;
    R.small_verts += (int)nv;
  }
  const long long counts = (R.slots + 2 + 15) / 16 * 16;
  R.queue = reinterpret_cast<unsigned*>(tables);
  R.count = R.queue + 16 * kQueues;
  R.small = tables + 16 * kQueues + counts;
  return 16 * kQueues + counts + 4LL * kSmallCopies * R.small_verts;
}
long long max_tables() { return 16 * kQueues + kMaxBins + 32 + 4LL * kSmallCopies * kSmallVerts; }

// ---------------------------------------------------------------- first records of the slots
// Block b sums its 1024 slots and takes its records' ranges from two running
// totals: slots of at least kDense records from the front of the records,
// sparse ones from their end.  The order of the blocks' ranges does not matter.
// A batch whose count decides against records has counted none: this kernel and
// the scatter then find no work, without a look at the choice (whose arguments
// would add a round trip of about 1 us at their start).
__global__ __launch_bounds__(256) void bin_first_kernel(ScatterRecords R) {
  __shared__ unsigned wsum[2][4], base[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int s0 = blockIdx.x * 1024 + tid * 4;
  unsigned c[4], sum[2] = {0u, 0u};
  bool sparse[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    c[u] = s0 + u < R.slots ? R.count[s0 + u] : 0u;
    sparse[u] = (c[u] << R.spread) < kDense;   // (a slot holds its share of the bin)
    sum[sparse[u]] += c[u];
  }
  unsigned inc[2] = {sum[0], sum[1]};
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned u0 = __shfl_up(inc[0], d, 64), u1 = __shfl_up(inc[1], d, 64);
    if (lane >= d) { inc[0] += u0; inc[1] += u1; }
  }
  if (lane == 63) { wsum[0][wave] = inc[0]; wsum[1][wave] = inc[1]; }
  __syncthreads();
  if (tid < 2) base[tid] = atomicAdd(R.count + R.slots + tid, wsum[tid][0] + wsum[tid][1] + wsum[tid][2] + wsum[tid][3]);
  __syncthreads();
  unsigned at[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    at[k] = base[k] + inc[k] - sum[k];
    for (int w = 0; w < wave; ++w) at[k] += wsum[k][w];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const unsigned front = at[0], back = (unsigned)R.cap - at[1] - c[u];
    if (s0 + u < R.slots) R.first[s0 + u] = sparse[u] ? back : front;
    at[sparse[u]] += c[u];
  }
}

// ---------------------------------------------------------------- scatter
// Keeps the compiler from moving LDS accesses across; the hardware serves a
// wave's LDS accesses in order.
__device__ __forceinline__ void wave_lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// First vertex of bin coordinate c's window along one axis of a level.
__device__ __forceinline__ int window_origin(int c, float ratio, int n, int wd) {
  return min((int)((float)c * ratio + 1e-3f), n - wd);
}

// base[offset bytes] += v in the lanes whose v is not 0 (base is the same in
// every lane).  Written out, as the compiler puts a branch around a memory
// operation under a lane mask: with one in each of a window's 68 columns a flush
// took 13000 cycles.  A memory instruction must not read a scalar register within
// five wait states of a vector instruction that wrote it (base may come from a
// readlane or a register spilled to a lane), and the compiler does not look into
// the block: it keeps that distance from its own start.
__device__ __forceinline__ void add_nonzero(float* base, unsigned offset, float v) {
  unsigned long long saved;
  asm volatile(
      "v_cmp_neq_f32_e32 vcc, 0, %1\n\t"
      "s_and_saveexec_b64 %0, vcc\n\t"
      "s_nop 2\n\t"
      "global_atomic_add_f32 %2, %1, %3\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved)
      : "v"(v), "v"(offset), "s"(base)
      : "vcc", "scc", "memory");
}

// Level constants of the lane's level q = lane / 16 (staging lanes).
struct WindowLevel {
  int wx, wy, wz, wb;   // window: vertices per axis, first vertex
  int n[3];             // grid: vertices per axis
  float ratio;
  unsigned base_lo, base_hi;   // where the level's sums go: the gradient's first row of it, or a copy's
};

// Adds the window of bin `bin` to the gradient and clears it.  Each level is
// walked in columns along z: the lanes cover (x, y, feature) of a slab with
// features innermost, so that a 64-byte chunk of the gradient is one request,
// and read their column before they write any of it.
__device__ __forceinline__ void flush_window(const WindowLevel& L, float* win, int verts, int bin, int nbx,
                                             int nby, int lane) {
  const int bx = bin % nbx, by = (bin / nbx) % nby, bz = bin / (nbx * nby);
  wave_lds_fence();
#pragma unroll 1
  for (int l = 0; l < 4; ++l) {
    const int k = 16 * l;   // a lane that holds level l
    const int wx = __builtin_amdgcn_readlane(L.wx, k), wy = __builtin_amdgcn_readlane(L.wy, k),
              wz = __builtin_amdgcn_readlane(L.wz, k);
    const int nx = __builtin_amdgcn_readlane(L.n[0], k), ny = __builtin_amdgcn_readlane(L.n[1], k),
              nz = __builtin_amdgcn_readlane(L.n[2], k);
    const float ratio = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(L.ratio), k));
    const int x0 = window_origin(bx, ratio, nx, wx), y0 = window_origin(by, ratio, ny, wy),
              z0 = window_origin(bz, ratio, nz, wz);
    const int n = 4 * wx * wy;   // floats of a slab
    const float inv_wx = 1.f / (float)wx;
    // the same in every lane
    const unsigned long long base = (unsigned)__builtin_amdgcn_readlane((int)L.base_lo, k) |
                                    ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)L.base_hi, k) << 32);
    const int row = __builtin_amdgcn_readfirstlane((z0 * ny + y0) * nx + x0);
    float* g0 = reinterpret_cast<float*>(base) + 4 * (long long)row;
    const long long zstep = 4LL * nx * ny;
    float* w0 = win + 4 * __builtin_amdgcn_readlane(L.wb, k);
#pragma unroll 1
    for (int e = lane; e < n; e += 64) {
      const int v = e >> 2;
      const int y = (int)(((float)v + 0.5f) * inv_wx), x = v - y * wx;
      const unsigned at = 4u * (unsigned)(y * nx + x) + (unsigned)(e & 3);
      float* w = w0 + e;
      float s[kWinEdge];
#pragma unroll
      for (int z = 0; z < kWinEdge; ++z) s[z] = z < wz ? w[z * n] : 0.f;
      float* g = g0;
#pragma unroll
      for (int z = 0; z < kWinEdge; ++z) {
        add_nonzero(g, 4u * at, s[z]);
        g += zstep;
      }
    }
  }
  // (the window is contiguous: cleared in whole vertices)
  wave_lds_fence();
  for (int e = lane; e < verts; e += 64) reinterpret_cast<float4*>(win)[e] = make_float4(0.f, 0.f, 0.f, 0.f);
  wave_lds_fence();
}

// Adds each lane's vertex (row of its level, four features v) without a window
// (a quad's lanes are corners of one level): the four lanes of a quad take their vertices in turn, a feature each,
// so that a vertex is one request instead of four.
template <int I>
__device__ __forceinline__ void direct_turn(float* grad, const float4& v, int row, int k) {
  constexpr int kFrom = 0x55 * I;   // quad_perm: every lane reads lane I of its quad
  const int r = dpp_i<kFrom>(row);
  const float v0 = dpp_f<kFrom>(v.x), v1 = dpp_f<kFrom>(v.y), v2 = dpp_f<kFrom>(v.z), v3 = dpp_f<kFrom>(v.w);
  const float s = k == 0 ? v0 : (k == 1 ? v1 : (k == 2 ? v2 : v3));
  if (r >= 0) atomic_add_global(grad + 4 * (long long)r + k, s);
}
__device__ __forceinline__ void add_direct(float* grad, const float4& v, int row, int lane) {
  direct_turn<0>(grad, v, row, lane & 3);
  direct_turn<1>(grad, v, row, lane & 3);
  direct_turn<2>(grad, v, row, lane & 3);
  direct_turn<3>(grad, v, row, lane & 3);
}

__device__ __forceinline__ void add4(float4* w, const float4& v) {
  float4 x = *w;
  x.x += v.x; x.y += v.y; x.z += v.z; x.w += v.w;
  *w = x;
}

// Tiles of a chunk: a wave takes one chunk of its share of the tiles, or several
// of 32 tiles, which even out the bins' differences; small batches use fewer
// waves, so that a window collects 4 tiles before it goes to memory.
__host__ __device__ inline unsigned scatter_chunk(unsigned tiles, unsigned waves) {
  const unsigned c = (tiles + waves - 1) / (4 * waves);
  return c < 4u ? 4u : (c > 32u ? 32u : c);
}

// One wave per block: the windows are private to a wave, so nothing waits at
// a barrier.  A wave takes chunks of consecutive tiles (16 records).
//
// Lane (q, j) first stages level q of record j in LDS: cell fractions and
// place in the window, dL/dz, and the second-order terms.  Then the wave adds
// two records at a time, 32 lanes each: a lane is one corner of one level.  A
// record's 32 vertices differ, so the window is updated by plain reads and
// writes of whole vertices, one half wave after the other; the wave's in-order
// LDS accesses keep them apart.  (LDS float atomics are served about one lane
// per clock: 85 us of a room batch and 2 ms of 8.4 M samples, against none for
// reads and writes.)
__global__ __launch_bounds__(64) void scatter_kernel(ScatterArgs A, int waves) {
  __shared__ float4 win[kWinVerts];
  __shared__ float4 st_f[64], st_dz[64], st_a[64], st_g[16];   // [record][level]
  __shared__ int st_row[64];
  const int lane = threadIdx.x, q = lane >> 4, j = lane & 15;
  const ScatterRecords& R = A.rec;
  // dense records [0, n_front), sparse ones [n_back0, cap); their tiles follow
  // each other
  const unsigned cap = (unsigned)R.cap;
  const unsigned n_front = min(R.count[R.slots], cap), n_back0 = cap - min(R.count[R.slots + 1], cap);
  const unsigned front_tiles = (n_front + 15) / 16, tiles = front_tiles + (cap - n_back0 + 15) / 16;
  const unsigned chunk = scatter_chunk(tiles, waves);
  if (blockIdx.x * chunk >= tiles) return;

  // staging lane: its level's sizes
  const LevelConst lc = level_const(A.g, q);
  const int wdx[4] = {R.bins.wd[0][0], R.bins.wd[1][0], R.bins.wd[2][0], R.bins.wd[3][0]};
  const int wdy[4] = {R.bins.wd[0][1], R.bins.wd[1][1], R.bins.wd[2][1], R.bins.wd[3][1]};
  const int wdz[4] = {R.bins.wd[0][2], R.bins.wd[1][2], R.bins.wd[2][2], R.bins.wd[3][2]};
  const int wx = pick_level(wdx, q), wy = pick_level(wdy, q), wz = pick_level(wdz, q), wb = pick_level(R.bins.wbase, q);
  const int rb[4] = {__float_as_int(R.bins.ratio[0]), __float_as_int(R.bins.ratio[1]), __float_as_int(R.bins.ratio[2]),
                     __float_as_int(R.bins.ratio[3])};
  const float ratio = __int_as_float(pick_level(rb, q));
  float* level_base = A.grad_grid + 4 * lc.off;
  if ((R.small_mask >> q) & 1)
    level_base = R.small + 4 * ((long long)(blockIdx.x % kSmallCopies) * R.small_verts + pick_level(R.small_off, q));
  const unsigned long long lb = reinterpret_cast<unsigned long long>(level_base);
  const WindowLevel wl{wx, wy, wz, wb, {lc.n[0], lc.n[1], lc.n[2]}, ratio, (unsigned)lb, (unsigned)(lb >> 32)};
  const int nbx = R.bins.nb[0], nby = R.bins.nb[1];
  const int verts = R.bins.wbase[3] + R.bins.wd[3][0] * R.bins.wd[3][1] * R.bins.wd[3][2];
  // adding lane: half h, level l, corner (cx, cy, cz); its weights are
  // f-linear, w_x = mx + px f_x, with px also the sign of dw_x/dx
  const int h = lane >> 5, l = (lane >> 3) & 3;
  const int cx = (lane >> 2) & 1, cy = (lane >> 1) & 1, cz = lane & 1;
  const float px = cx ? 1.f : -1.f, py = cy ? 1.f : -1.f, pz = cz ? 1.f : -1.f;
  const float mx = cx ? 0.f : 1.f, my = cy ? 0.f : 1.f, mz = cz ? 0.f : 1.f;
  const int lwx = pick_level(wdx, l), lwy = pick_level(wdy, l);
  const int corner = cx + cy * lwx + cz * lwx * lwy;
  const int lnx = pick_level(A.g.nx, l), lny = pick_level(A.g.ny, l);
  const unsigned al = (unsigned)__shfl((int)wl.base_lo, 16 * l, 64), ah = (unsigned)__shfl((int)wl.base_hi, 16 * l, 64);
  float* add_base = reinterpret_cast<float*>(al | ((unsigned long long)ah << 32));   // of its level
  const int vb[4] = {__float_as_int(A.g.voxel[0]), __float_as_int(A.g.voxel[1]), __float_as_int(A.g.voxel[2]),
                     __float_as_int(A.g.voxel[3])};
  const float inv_v = 1.f / __int_as_float(pick_level(vb, l));
  const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int e = lane; e < kWinVerts; e += 64) win[e] = zero4;

  // The wave's tiles in order: the chunk of its own number, then chunks drawn
  // from one of kQueues counters (queue k hands out the chunks k, k + kQueues,
  // ... past the waves' own), each drawn a chunk ahead.  Past the last tile the
  // sequence stays at `tiles`.
  const unsigned queue = blockIdx.x % kQueues;
  unsigned long long seq = (unsigned long long)blockIdx.x * chunk, seq_end = seq + chunk;
  unsigned drawn = 0u;
  auto draw = [&] {
    if (lane == 0) drawn = __hip_atomic_fetch_add(R.queue + 16 * queue, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto next_tile = [&]() -> unsigned {
    const unsigned t = seq < tiles ? (unsigned)seq : tiles;
    if (++seq == seq_end) {
      const unsigned d = (unsigned)__builtin_amdgcn_readfirstlane((int)drawn);
      seq = (gridDim.x + (unsigned long long)d * kQueues + queue) * chunk;
      seq_end = seq + chunk;
      if (seq < tiles) draw();
    }
    return t;
  };
  draw();

  const float4 *r_pos = R.pos, *r_dz = R.dz, *r_a = R.a, *r_gv = R.gv;
  const Bins bins = R.bins;
  // the position and tag of a record are loaded two tiles ahead, what the tag
  // says it has one tile ahead
  constexpr int kNone = kTagBin | kTagNoFirst;   // tag of a lane without a record
  auto load_pos = [&](unsigned t) {
    const bool front = t < front_tiles;
    const unsigned i = front ? t * 16 + j : n_back0 + (t - front_tiles) * 16 + j;
    return i < (front ? n_front : (t < tiles ? cap : 0u)) ? r_pos[i] : make_float4(0.f, 0.f, 0.f, __int_as_float(kNone));
  };
  float4 dz_n, a_n, gv_n;
  auto load_terms = [&](unsigned t, const float4& p) {
    const size_t i = t < front_tiles ? t * 16 + j : n_back0 + (t - front_tiles) * 16 + j;
    const int tag = __float_as_int(p.w);
    dz_n = a_n = gv_n = zero4;
    if (!(tag & kTagNoFirst)) dz_n = r_dz[4 * i + q];
    if (tag & kTagSecond) {
      a_n = r_a[4 * i + q];
      gv_n = r_gv[i];
    }
  };
  int cur = -1;
  unsigned t = next_tile(), tn = next_tile();
  float4 pos = load_pos(t), pos_n = load_pos(tn);
  load_terms(t, pos);
#pragma unroll 1
  while (t < tiles) {
    const bool sparse = t >= front_tiles;
    const float4 p = pos;
    const int tag = __float_as_int(p.w);
    // stage this tile
    bool in;
    {
      LevelSample ls;
      locate(A.g, lc, p.x, p.y, p.z, ls);
      int bc[3];
      bin_coords(bins, p.x, p.y, p.z, bc);
      const int x = ls.cell3[0] - window_origin(bc[0], ratio, lc.n[0], wx);
      const int y = ls.cell3[1] - window_origin(bc[1], ratio, lc.n[1], wy);
      const int z = ls.cell3[2] - window_origin(bc[2], ratio, lc.n[2], wz);
      in = x >= 0 && x < wx - 1 && y >= 0 && y < wy - 1 && z >= 0 && z < wz - 1;
      // -1: a cell outside its window (a bin edge that rounds the other way)
      const int at = in ? wb + (z * wy + y) * wx + x : -1;
      st_row[4 * j + q] = (int)(ls.row - lc.off);
      st_f[4 * j + q] = make_float4(ls.f[0], ls.f[1], ls.f[2], __int_as_float(at));
      st_dz[4 * j + q] = dz_n;
    }
    const bool second = __ballot((tag & kTagSecond) != 0) != 0ull;
    if (second) {
      st_a[4 * j + q] = a_n;
      if (q == 0) st_g[j] = gv_n;
    }
    wave_lds_order();
    t = tn;
    pos = pos_n;
    load_terms(t, pos);
    tn = next_tile();
    pos_n = load_pos(tn);
    const int bin = tag & kTagBin;

    // every record in the open window: no decisions between the updates
    const bool plain = !sparse && __ballot(bin != cur || !in) == 0ull;
#pragma unroll 1
    for (int s0 = 0; s0 < 8; s0 += 4) {
      float4 v[4], f[4];
      int at[4];
      // the staged values of four steps are read before any is used
#pragma unroll
      for (int s = 0; s < 4; ++s) f[s] = st_f[4 * (2 * (s0 + s) + h) + l];
#pragma unroll
      for (int s = 0; s < 4; ++s) v[s] = st_dz[4 * (2 * (s0 + s) + h) + l];
      if (second) {
        float4 a[4], g[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          a[s] = st_a[4 * (2 * (s0 + s) + h) + l];
          g[s] = st_g[2 * (s0 + s) + h];
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const float ux = fmaf(px, f[s].x, mx), uy = fmaf(py, f[s].y, my), uz = fmaf(pz, f[s].z, mz);
          const float w = ux * uy * uz;
          const float jg = (px * g[s].x * (uy * uz) + py * g[s].y * (ux * uz) + pz * g[s].z * (ux * uy)) * inv_v;
          v[s] = make_float4(fmaf(a[s].x, jg, w * v[s].x), fmaf(a[s].y, jg, w * v[s].y), fmaf(a[s].z, jg, w * v[s].z),
                             fmaf(a[s].w, jg, w * v[s].w));
        }
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const float w = fmaf(px, f[s].x, mx) * fmaf(py, f[s].y, my) * fmaf(pz, f[s].z, mz);
          v[s] = make_float4(w * v[s].x, w * v[s].y, w * v[s].z, w * v[s].w);
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) at[s] = __float_as_int(f[s].w);
      if (plain) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          float4* w = win + at[s] + corner;
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            if (h == half) add4(w, v[s]);
            wave_lds_order();
          }
        }
        continue;
      }
#pragma unroll 1
      for (int u = 0; u < 8; ++u) {
        const int s = u >> 1, half = u & 1;
        const int b = __builtin_amdgcn_readlane(bin, 2 * s0 + u);
        if (b == kTagBin) continue;
        bool window = b == cur;
        // a bin of few records does not pay for a window
        if (!window && !sparse) {
          if (cur >= 0) flush_window(wl, reinterpret_cast<float*>(win), verts, cur, nbx, nby, lane);
          cur = b;
          window = true;
        }
        const float4 x = s == 0 ? v[0] : (s == 1 ? v[1] : (s == 2 ? v[2] : v[3]));
        const int to = s == 0 ? at[0] : (s == 1 ? at[1] : (s == 2 ? at[2] : at[3]));
        if (h == half && window && to >= 0) add4(win + to + corner, x);
        wave_lds_order();
        const bool out = h == half && (!window || to < 0);
        if (__ballot(out) != 0ull) {
          const int row = st_row[4 * (2 * s0 + u) + l] + cx + (cy + cz * lny) * lnx;
          add_direct(add_base, x, out ? row : -1, lane);
        }
      }
    }
  }
  if (cur >= 0) flush_window(wl, reinterpret_cast<float*>(win), verts, cur, nbx, nby, lane);
}

// The small levels' copies as rows for the sums that end the pass.
static_assert(kSmallCopies == kSumRows, "the copies are the rows of the sums");
LevelSums small_sums(const Grid& g, const ScatterRecords& r) {
  LevelSums m;
  m.floats = 4 * r.small_verts;
  m.mask = r.small_mask;
  for (int l = 0; l < 4; ++l) {
    m.off[l] = 4 * r.small_off[l];
    m.cnt[l] = (r.small_mask >> l) & 1 ? 4 * g.nx[l] * g.ny[l] * g.nz[l] : 0;
    m.first[l] = g.off[l];
  }
  return m;
}

hipError_t launch_bin_first(const ScatterRecords& r, hipStream_t st) {
  hipLaunchKernelGGL(bin_first_kernel, dim3((r.slots + 1023) / 1024), dim3(256), 0, st, r);
  return hipGetLastError();
}

// At most one resident round of waves: 9 windows with their staging fit the
// 160 KB of a CU (the occupancy query's answer too; sized for 8, ragged BF16 rays
// take 2.5 % longer).  The kernel takes its chunks from the records there are, which
// may be fewer than the arrays hold: four a wave, or two (as for half the waves) on
// small grids, whose bins are alike and whose windows queue at the same addresses
// (64 bins, 1 M samples: 435 us with four, 399 with two; 1.2 M in BF16 at 3 cm: 475
// and 529).
hipError_t launch_scatter(const ScatterArgs& a, hipStream_t st) {
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const long long tiles = (a.rec.cap + 15) / 16, waves = (9LL * cus + kQueues - 1) / kQueues * kQueues;
  const Bins& b = a.rec.bins;
  const long long share = few_bins((long long)b.nb[0] * b.nb[1] * b.nb[2]) ? waves / 2 : waves;
  const long long chunk = scatter_chunk((unsigned)tiles, (unsigned)share);
  long long blocks = (tiles + chunk - 1) / chunk;
  if (blocks > waves) blocks = waves;   // a multiple of kQueues, as drawing needs
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(scatter_kernel, dim3((unsigned)blocks), dim3(64), 0, st, a, (int)share);
  return hipGetLastError();
}

}  // namespace gs
