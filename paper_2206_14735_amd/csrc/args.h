// Kernel argument blocks (passed by value to the kernels).
#pragma once
#include "bins.h"
#include "device.h"

namespace gs {

constexpr int kChunks = GOSURF_MAX_SAMPLES_PER_RAY / 64;

// Depth-edge test of the proposal's segment pass: the frames' depth images
// [T][H][W], each ray's pixel, the threshold (metres; 0 = off).
struct EdgeCheck {
  const float* depth;
  int H, W;
  const long long* pixel;
  float edge;
};

// Whether a backward pass scatters through records.  The host decides by the
// number of samples where it knows it.  Of a batch drawn with a proposal it knows
// the capacity, up to three times the samples there are; where that leaves it
// open, the kernels of both ways are launched, and each decides by the count on
// the device (all read the same) whether it runs or ends at once.
struct RecordChoice {
  const int* seg_end;   // sample count on the device, or nullptr: the host's word holds
  int records;
  int total;            // capacity
  int from;             // records from this many samples on
  __device__ __forceinline__ bool operator()() const { return records && (!seg_end || min(*seg_end, total) >= from); }
};

// Scatter records of the backward, grouped by bin.  An item is a ray sample
// (0 .. total - 1) or a point of smoothness pair p (total + 2 p, total + 2 p + 1).
struct ScatterRecords {
  RecordChoice choice;
  Bins bins;
  int2* place;            // [total + 2 S]: table slot and rank inside it; slot < 0: no record
  unsigned* queue;        // [kQueues][16]: work counters of the scatter
  unsigned* count;        // [slots + 2], behind the queues: records per slot, then of all dense and all sparse slots
  unsigned* first;        // [slots]: first record of a slot
  int slots, spread;
  long long cap;          // records the arrays hold
  // Levels of few vertices are summed in kSmallCopies copies (behind the
  // counts) and folded into the gradient afterwards: windows all over the grid
  // add to the same few of their vertices.
  int small_mask;         // bit l: level l is small
  int small_off[4];       // its first vertex in a copy
  int small_verts;        // vertices of a copy
  float* small;           // [kSmallCopies][small_verts][4]
  float4* pos;            // [cap]: position, tag (bin and kTag flags, as an int)
  float4* dz;             // [cap][4 levels]: dL/dz
  float4* a;              // [cap][4 levels]: d(phi)/dz (second-order terms)
  float4* gv;             // [cap]: dL/d(grad phi)
};

struct ScatterArgs {
  Grid g;
  ScatterRecords rec;
  float* grad_grid;       // [V][4]
};

struct FieldArgs {
  Grid g;
  const float* grid;
  const uint16_t* grid_bf16;   // non-null: BF16 decoders and gathers from this mirror
  const float* mlp;
  // ray samples
  const float* o;
  const float* r;
  const float* t;
  const int* ray_of;
  int total;
  // smoothness pairs
  const float* xs;
  const float* eps;
  int S;
  // forward outputs
  float* out4;            // [total][4] phi, c
  float* eik;             // [total] (1 - |grad phi|)^2
  float* smooth_partial;  // [gridDim.x]
  float* grad_phi;        // [total + 2 S][3] d(phi)/dx (forward, optional; total = the capacity)
  float* pair_terms;      // [S] per-pair smoothness value (forward, optional)
  // backward
  const float* seed4;     // [total][4] dL/dphi, dL/dc (scaled)
  const float* posw;      // [total][4]: sample position (as the forward computed it), Eikonal
                          // weight (scaled, 0 outside S_fs)
  float smooth_coef;      // 2 * lambda_smooth * loss_scale / S
  float* mlp_partial;     // [gridDim.x][kMlpNumel]
  int need_gx;            // ray mode: compute grad phi for the Eikonal term
  const float* depth;     // forward, optional: [M] observed depth per ray; with it, wave-tiles
                          // with no sample in S_fs = {D - t > trunc} skip grad phi
  float trunc;
  float* grad_x;          // backward, optional: [total][4] dL/dx of each sample (x, y, z, 0)
  int colour;             // ray mode: 1 = colour from the geometry decoder's features; 0 = no colour
                          // here (the paper's colour path runs in its own kernel)
  const int* seg_end;     // ray mode: device copy of the sample count (seg[M]); total is then a capacity
  // backward: one kernel writes scatter records, at the place the binning gave
  // each item, and the scatter kernel adds them to the gradient; the other adds
  // to grad_grid itself (rec.choice says which of them runs).  Then the levels in
  // priv_mask are accumulated in LDS per block, each at its float offset of the
  // block's LDS area
  ScatterRecords rec;
  float* grad_grid;       // [V][4]
  int priv_mask;
  int priv_off[4];
  int priv_floats;        // floats of the LDS area
  float* priv_partial;    // [gridDim.x][priv_floats] block partials
};

// the paper's colour path (colour grid at the finest level + view direction)
struct ColourArgs {
  Grid g;
  const float* cgrid;     // [V_finest][8]: 6 features, 2 unused
  const float* cmlp;      // packed V1 e1 V2 e2 V3 e3
  const float* o;
  const float* r;
  const float* t;
  const int* ray_of;
  int total;
  const int* seg_end;     // device copy of the sample count (seg[M]); total is then a capacity
  float* out4;            // forward: colour into components 1..3 of [total][4]
  const float* seed4;     // backward: [total][4] seeds (components 1..3: dL/dc, scaled)
  const float* posw;      // backward: [total][4] sample positions
  float* grad_cgrid;      // backward: [V_finest][8]
  float* partial;         // backward: [gridDim.x][colour decoder size] block partials
};

struct RenderArgs {
  Grid g;
  const float* o;
  const float* r;
  const float* rgb;
  const float* depth;
  const float* t;
  const int* seg;
  int M;
  int total;            // sample capacity of the batch
  const float* mlp;
  const float* out4;    // [total][4]
  const float* eik;     // [total] or null
  float trunc, alpha_fs;
  float lam[6];
  int depth_mid;        // d_hat attributes w_i to (t_i + t_i+1) / 2 instead of t_i
  // forward outputs
  float* rgb_hat;
  float* depth_hat;
  float* wsum;
  float* weights;       // or null
  float* ray_partial;   // [M][8]
  // backward
  const float* n_depth_rays;  // device scalar (losses[7])
  float loss_scale;
  float* seed4;         // [total][4]
  float* posw;          // [total][4]: sample position, Eikonal weight
  float* ray_dv;        // [M]
  ScatterRecords rec;
  const float* xs;      // smoothness pairs, binned by the same launch
  const float* eps;
  int S;
};

// proposal network over a set of rays
struct PropArgs {
  Grid g;
  const float* grid;
  const float* prop;     // packed proposal parameters
  const float* o;
  const float* r;
  int M;
  int span_mode;
  float near_t, far_t;
  float* out3;           // [M][3] near, far, confidence (or null)
  const float* tgt;      // [M][3] training targets
  float beta;            // smooth-L1 transition
  float cover_tol;       // confidence label: interval covers the target within this
  float* grad_partial;   // [gridDim.x][numel + 1] (last entry: loss)
};

// training targets from logged per-sample weights
struct TargetArgs {
  Grid g;
  const float* t;
  const float* w;
  const int* seg;
  const float* o;
  const float* r;
  int M;
  int span_mode;
  float near_t, far_t;
  float widen, q_lo, q_hi, conf_min;
  float* tgt;            // [M][3]
};

// Levels whose gradient is summed in kSumRows rows of `floats` floats before it
// joins the grid's: level l of the mask takes cnt[l] floats from off[l] on and starts at
// row first[l] of the grid.
constexpr int kSumRows = 64;
struct LevelSums {
  int floats;
  int mask;
  int off[4], cnt[4];
  long long first[4];
};

// The sums that end a backward pass.
struct GradReduceArgs {
  RecordChoice choice;
  const float* mlp_part;   // [rows][kMlpNumel] block partials, of rec_rows rows with records
  int rows, rec_rows;
  float* mlp_tmp;          // [kSumRows][kMlpNumel]
  const float* ray_dv;     // [M]
  int M;
  float* ray_part;         // [64][8]
  float* grad_mlp;
  LevelSums lev;           // without records (floats = 0: none)
  const float* lev_part;   // [rows][lev.floats] block partials
  float* lev_tmp;          // [kSumRows][lev.floats]
  LevelSums rec_lev;       // with records (floats = 0: none)
  const float* rec_tmp;    // [kSumRows][rec_lev.floats], written by the scatter
  float* grad_grid;
};

struct SampleArgs {
  Grid g;
  const uint8_t* rgb;
  const float* depth;
  const float* c2w;
  int T, H, W;
  float fx, fy, cx, cy;
  int M, n_strat, n_near, span_mode;
  float near_t, far_t, trunc;
  int S;
  float delta_s;
  uint32_t k0, k1, step;
  float* o;
  float* r;
  float* rgb_out;
  float* depth_out;
  float* t;
  int* seg;
  int* ray_of;
  float* xs;
  float* eps;
  long long* pixel;
  // proposal-driven sampling: per-ray (near, far, confidence); rays with
  // confidence >= conf_thr get n_free samples on [t_lo, near] and n_prop in
  // [near, far], the others the plain n_strat + n_near; seg is then filled
  // beforehand by the scan
  const float* prop3;
  float conf_thr;
  int n_prop;
  int n_free;
};


// Hierarchical importance sampling: one step (new depths from the current
// samples of every ray, all rays with n samples) and the merge of the new
// depths into the sorted lists.
constexpr int kImpMaxAdd = 64;   // samples added per ray and step
struct ImpArgs {
  Grid g;
  const float* o;
  const float* r;
  const float* t;        // [M][n] sorted
  const float* phi;      // SDF of the samples
  const float* mlp;      // sharpness s = exp(10 v)
  int M, n, n_add;
  float eps;             // added to every interval weight
  uint32_t k0, k1, iteration, stream;   // Philox key and counter words
  float* t_new;          // [M][n_add]
  int* ray_of_new;       // [M][n_add] or null
};
struct ImpMergeArgs {
  const float* ta;       // [M][na] sorted
  const float* pa;       // value carried with ta
  int na;
  const float* tb;       // [M][nb]
  const float* pb;
  int nb;
  int M;
  float* t_out;          // [M][na + nb]
  float* p_out;          // or null
  int* ray_of_out;       // or null
  int* seg_out;          // [M + 1] or null
};

// SDF alone, of ray samples (t, ray_of) or, without them, of lattice points
// p0 + h (i, j, k), x fastest, z layers from k0 on.
struct PhiArgs {
  Grid g;
  const float* grid;
  const uint16_t* grid_bf16;
  const float* mlp;
  const float* o;
  const float* r;
  const float* t;
  const int* ray_of;
  int total;
  float* phi;               // [total]
  float p0[3];
  float h;
  int nx, ny, k0;
};
// Marching tetrahedra over the SDF lattice.
struct MtArgs {
  const float* phi;         // [nz][ny][nx]
  float p0[3];
  float h;
  int nx, ny, nz;
  float* tris;              // [max_tris][3][3]
  long long max_tris;
  unsigned* count;          // triangles found (may exceed max_tris)
};

}  // namespace gs
