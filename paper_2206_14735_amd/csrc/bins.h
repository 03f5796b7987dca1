// Spatial bins of the grid scatter.
//
// A bin is a block of 2^shift cells per axis of the finest level.  The
// backward groups its scatter records by bin, so that the records of one bin
// can be summed in a small LDS window that holds, for every level, the
// vertices the bin's cells use; only the window's sums go to memory.
#pragma once
#include "device.h"

namespace gs {

constexpr int kMaxBins = 1 << 20;        // entries of the counting tables
constexpr int kWinVerts = 912;           // vertices of a window (all levels): 14.25 KB of float4
constexpr int kWinEdge = 9;              // vertices of a window along z: a flush holds a column in registers
constexpr int kQueues = 64;              // work counters of the scatter, 64 bytes apart
constexpr unsigned kDense = 16;          // records for which a bin gets the window
constexpr int kSmallVerts = 1024;        // vertices of the small levels together, at most
constexpr int kSmallCopies = 64;
constexpr int kTagSecond = 1 << 31;      // record tag: has second-order terms (rec_a, rec_gv)
constexpr int kTagNoFirst = 1 << 30;     // record tag: has no first-order term (rec_dz)
constexpr int kTagBin = kTagNoFirst - 1;

struct Bins {
  int level, shift;
  int nb[3];            // bins per axis
  int last[3];          // last cell of the level per axis
  float p0[3], inv_v;   // cell = (x - p0) * inv_v (grouping only: its rounding changes no result)
  // window of each level: vertices per axis, first vertex in the window, bin
  // edge in the level's cells
  int wd[4][3], wbase[4];
  float ratio[4];
};

// Bin coordinates of a point.
__device__ __forceinline__ void bin_coords(const Bins& B, float x, float y, float z, int c[3]) {
  const float p[3] = {x, y, z};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    int i = (int)floorf((p[a] - B.p0[a]) * B.inv_v);
    i = i < 0 ? 0 : (i > B.last[a] ? B.last[a] : i);
    c[a] = i >> B.shift;
  }
}
__device__ __forceinline__ int bin_of(const Bins& B, float x, float y, float z) {
  int c[3];
  bin_coords(B, x, y, z, c);
  return (c[2] * B.nb[1] + c[1]) * B.nb[0] + c[0];
}
// Table slot of a bin's record: a bin has 2^spread neighbouring slots, and the
// records of different rays take different ones, so that few bins do not queue
// at few counters.  Grids of more than kMaxBins bins share slots: records of
// bins that share one are grouped together, which costs window changes but no
// correctness.
__device__ __forceinline__ int bin_slot(int bin, int spread, int ray) {
  return ((bin << spread) | (ray & ((1 << spread) - 1))) & (kMaxBins - 1);
}

}  // namespace gs
