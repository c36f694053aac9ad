// Internal declarations shared by the HIP kernels and the host runtime.
//
// Every kernel takes a table of work items in device memory.  An item is one
// field-sized piece of work (one squaring of one direction, one composition,
// one session pair, ...) on its own grid, so a single launch can cover every
// interval, pair and subject of a batch with uneven grids.  Items in a table
// are sorted by tile0, the first global tile index of the item; a block finds
// its item by binary search.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace muster {

// Deterministic accumulation (a job's params.deterministic): every scatter
// that would add into a float field with global atomics adds 64-bit fixed
// point instead, at a scale shared by all blocks of the job in that launch:
// 2^(61 - e) with 2^e >= blocks * m, m the largest summed magnitude any of
// the job's blocks spreads (found by a pass of the same kernel that only
// reduces it), so no cell can overflow and integer adds make the sum
// independent of their order.  A fold then adds the fixed-point field into
// the float one.  One slot per such launch of an iteration.
constexpr int DET_SLOTS = 96;

// Blocks that add into one double follow each other at about 13 ns, so the
// regularisers' sums are spread over slots on lines of their own.
constexpr int LOSS_SLOTS = 16, LOSS_STRIDE = 16;
inline __host__ __device__ double slot_sum(const double* s) {
  double v = 0.0;
  for (int k = 0; k < LOSS_SLOTS; ++k) v += s[k * LOSS_STRIDE];
  return v;
}

// Per-job device state: optimiser step counter and schedule, loss
// accumulators and the loss history.  Lives in device memory so that a
// captured iteration can be replayed without host involvement.
struct JobState {
  int t;            // completed Adam steps at the current level
  int T;            // steps at this level
  int W;            // warm-up steps
  int nonfinite;    // set once the loss is not finite
  float lr0, b1, b2, eps;
  double loss_sim;  // accumulated over the current iteration
  double loss_reg[LOSS_SLOTS * LOSS_STRIDE];  // weighted regularisers, in slots
  double* history;  // loss per step (device), length hist_len
  int hist_len;
  int* flags;       // per Exp-backward step: its fixed-point field was added to (deterministic
  int n_flags;      // mode); cleared per iteration
  int hist_base;    // index of this level's first step in history
  unsigned int det_max[DET_SLOTS];  // deterministic mode: largest block magnitude (float bits)
};

struct GridDims {
  int D, H, W;
};

// u_{s+1} = u + u o (Omega + u) with u = a * src.
struct ExpFwdItem {
  int tile0;
  int D, H, W;
  const float* src;
  float* dst;
  float a;
  int zc;            // planes per march tile
};

// out = prev + C o (Omega + prev).
struct ComposeItem {
  int tile0;
  int D, H, W;
  const float* prev;
  const float* C;
  float* out;
};

// One backward squaring: gout = oscale * dL/du_s from gin = dL/du_{s+1}, with
// u_s = a * src, over march tiles of zc planes; then, over point tiles, what
// the voxels that sample a voxel or more away spread.
struct ExpBwdItem {
  int tile0;
  int D, H, W;
  int zc;            // planes per march tile
  float a;
  float oscale;
  const float* src;
  const float* gin;
  float* gout;       // written whole by k_exp_bwd, added to by k_exp_far
  int* far;          // per point tile: holds voxels for k_exp_far; 0 between steps
  // Deterministic accumulation: k_exp_far adds into gout64 ([3][V] 64-bit
  // fixed point) instead, at the scale of the job's slot det_slot over
  // det_blocks blocks (see DET_SLOTS); null otherwise.
  JobState* js;
  long long* gout64;
  int* flag64;       // set where gout64 is added to
  int det_slot;
  int det_blocks;
};

// Backward of one composition out = prev + C o (Omega + prev): given
// g = dL/dout, add (I + J_C^T) g to gprev (atomically if prev_atomic) and
// scatter g into gc.
struct ComposeBwdItem {
  int tile0;
  int D, H, W;
  const float* g;
  const float* prev;
  const float* C;
  float* gprev;
  float* gc;
  int prev_atomic;
  int pad;
  // Deterministic accumulation: the scatter into gc goes to gc64 ([3][V]
  // 64-bit fixed point) at the scale of the job's slot (see DET_SLOTS), and
  // gprev, whose only float writer in the launch is then this item, is
  // updated with plain stores; null otherwise.
  long long* gc64;
  JobState* js;
  int det_slot;
  int det_blocks;
};

// Fold of a 64-bit fixed-point field into its float field: f += q / scale,
// q = 0, over n = 3V elements, for the scale of the job's slot; skipped when
// flag is set and *flag is 0 (no block of the launch added into q).
struct DetFoldItem {
  int tile0;
  int n;
  float* f;
  long long* q;
  const JobState* js;
  const int* flag;
  int det_slot;
  int det_blocks;
};

// One session pair (target F = I_i, source I_j, field U = U[j->i]).
// Rigid adjustment of one session (Sec. 2.5): parameters (angles about z, y,
// x; translation), their Adam moments, the displacement the similarity
// kernels add, d(p) = A p + off with A = R - I and off = c + t - R c, and the
// gradient sums of the current iteration.
struct RigidState {
  float theta[3], t[3];
  float m[6], v[6];
  float A[9], off[3];
  double gsum[3];   // sum_p G(p)
  double gmom[9];   // sum_p G(p) (p - c)^T, row-major
};

// R = Rz Ry Rx in (z, y, x) components (Rz turns y towards x, Ry turns x
// towards z, Rx turns z towards y), or its derivative with respect to one
// angle (deriv = 0, 1, 2).
__host__ __device__ inline void rigid_rotation(const float th[3], int deriv, float R[9]) {
  float f[3][9];
  const int ax[3][2] = {{1, 2}, {2, 0}, {0, 1}};
  for (int k = 0; k < 3; ++k) {
    float c = cosf(th[k]), s = sinf(th[k]);
    const bool d = deriv == k;
    for (int e = 0; e < 9; ++e) f[k][e] = 0.f;
    if (d) {
      const float cc = -s;
      s = c;
      c = cc;
    } else {
      for (int e = 0; e < 3; ++e) f[k][4 * e] = 1.f;
    }
    const int a = ax[k][0], b = ax[k][1];
    f[k][3 * a + a] = c;
    f[k][3 * b + b] = c;
    f[k][3 * a + b] = -s;
    f[k][3 * b + a] = s;
  }
  float t[9];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      float acc = 0.f;
      for (int l = 0; l < 3; ++l) acc += f[0][3 * i + l] * f[1][3 * l + j];
      t[3 * i + j] = acc;
    }
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      float acc = 0.f;
      for (int l = 0; l < 3; ++l) acc += t[3 * i + l] * f[2][3 * l + j];
      R[3 * i + j] = acc;
    }
}

struct SimItem {
  int tile0;
  int D, H, W;
  int zc;        // z-chunk length of the tiling: the statistics' sums are formed per chunk
  int zs;        // windows along z that a block of the statistics walks: zc, or less, then a
                 // multiple of the window
  int zg;        // planes that a block of the gradient walks
  const float* F;
  const float* I;
  const float* U;
  float* M;      // [V]: I warped by U (and the rigid adjustment), written by k_warp and read
                 // by k_sim_stats; may be the first plane of gU, which k_sim_grad overwrites
  float* coef;   // [V][3]: alpha, beta, gamma per window centre (may be null in sim_stats)
  float* gU;     // [3][V]: dSim/dU, written by sim_grad
  double inv_nr; // 1 / number of windows
  JobState* js;  // loss accumulator (may be null)
  double* sim_out;  // optional per-pair accumulator
  const RigidState* rigid;  // rigid adjustment of the source session, or null
};

// Gradient sums of a rigid adjustment from one pair's dSim/dU on the image grid.
struct RigidGradItem {
  int tile0;
  int D, H, W;
  const float* G;
  RigidState* rg;
};

// Adam step of one session's rigid parameters.
struct RigidStepItem {
  RigidState* rg;
  const JobState* js;
  float c[3];       // centre of the image grid
  float rot_lr;     // step scale of the angles (1 / largest half-extent)
};

// Mode 0: Adam step on phi with the gradient gsrc.  Mode 1: gout = gscale *
// gsrc.
struct AdamItem {
  int tile0;
  int n;          // voxels
  float* phi;
  const float* gsrc;
  float* m;
  float* v;
  float* gout;
  float gscale;
  int mode;
  JobState* js;
};

// The gradient of an SVF: out = gmul * (gf + gb + the regularisers'
// gradients), gf and gb the (scaled, signed) G_0 of its two directions, each
// of them and out NULL where not wanted; the regularisers' values are added
// to loss (NULL: not wanted).
struct CombineItem {
  int tile0;
  int D, H, W;
  const float* gf;
  const float* gb;
  float* out;
  const float* flow;   // the flow the regularisers act on
  double* loss;        // LOSS_SLOTS slots
  double loss_w[3];    // weights of the L_ss value's squares along z, y, x, the counts divided out
  float gmul;
  float reg_w;         // weight of the L_ss gradient
  // L_L2 and L_ts: the gradient gains w_self f_i + w_prev f_{i-1} + w_next
  // f_{i+1} (flows of the neighbouring intervals, NULL where absent), and the
  // loss l2_loss_w |f_i|^2 + ts_loss_w |f_{i-1} inv_dprev - f_i inv_dself|^2
  // per voxel.
  int ext;
  float w_self, w_prev, w_next;
  float l2_loss_w, ts_loss_w, inv_dprev, inv_dself;
  const float* flow_prev;
  const float* flow_next;
  void set_loss_weight(double w) {
    loss_w[0] = w / ((double)(D - 1) * H * W);
    loss_w[1] = w / ((double)D * (H - 1) * W);
    loss_w[2] = w / ((double)D * H * (W - 1));
  }
};

// One separable pass of the periodic Gaussian smoothing along one axis, for
// one field of three components.  A tile holds whole lines of one component
// in LDS: `lines` adjacent x columns of lines along z or y, or `lines`
// consecutive rows along x.  Taps w[SMOOTH_WPAD + k] for k = 0..2*radius are
// the filter's weights at offsets k - radius along the periodic line (the
// host derives them from the Fourier-domain transfer function); every other
// entry is zero.
constexpr int MAX_SMOOTH_RADIUS = 128;
constexpr float MAX_SMOOTH_SIGMA = 22.0f;      // radius 5.66 sigma fits 128
constexpr int SMOOTH_S = 8;                    // outputs per thread along a line
constexpr int SMOOTH_WPAD = SMOOTH_S;
constexpr int SMOOTH_XR = 2;                   // chunks per thread of a tile of rows (x)
constexpr int SMOOTH_WLEN = 2 * MAX_SMOOTH_RADIUS + 1 + 2 * SMOOTH_WPAD;
constexpr int SMOOTH_LDS = 16384;              // floats of LDS per block, at most
// Preferred, for occupancy: of a tile of columns (z, y) and of rows (x).  15
// million voxels at sigma 3: columns 160 / 139 us at 8192 / 4096, rows 118 / 133.
constexpr int SMOOTH_LDS_COLS = 4096, SMOOTH_LDS_ROWS = 8192;
constexpr int SMOOTH_MAX_DIM = 4096;           // a row has at most SMOOTH_XR * 256 chunks

struct SmoothItem {
  int tile0;
  int D, H, W;
  int axis;        // 0 = z, 1 = y, 2 = x
  int radius;
  int lines;       // lines per tile, a power of two in 1..64
  int lshift;      // log2(lines)
  int tiles_comp;  // tiles per component
  int pad[3];
  const float* src;
  float* dst;
  float w[SMOOTH_WLEN];
};

struct PoolItem {
  int tile0;
  int D, H, W;  // source dims
  const float* src;
  float* dst;
};

struct UpItem {
  int tile0;
  int D, H, W;  // coarse dims
  const float* src;
  float* dst;   // [3][2D][2H][2W]
};

// Tiles of the upsampling: UF_TZ x UF_TY x UF_TX fine voxels (D, H, W
// coarse).
constexpr int UF_TZ = 8, UF_TY = 8, UF_TX = 32;
inline int up_tiles(int D, int H, int W) {
  return ((2 * D + UF_TZ - 1) / UF_TZ) * ((2 * H + UF_TY - 1) / UF_TY) *
         ((2 * W + UF_TX - 1) / UF_TX);
}

// Tiles of the upsampling adjoint: UA_TZ x UA_TY x UA_TX coarse voxels.
constexpr int UA_TZ = 4, UA_TY = 8, UA_TX = 16;
inline int up_adj_tiles(int D, int H, int W) {
  return ((D + UA_TZ - 1) / UA_TZ) * ((H + UA_TY - 1) / UA_TY) * ((W + UA_TX - 1) / UA_TX);
}

// Tiles of the gather/scatter kernels.
constexpr int PT_Z = 8, PT_Y = 8, PT_X = 16;   // 1024 voxels, 256 threads
constexpr int PT_VOX = PT_Z * PT_Y * PT_X;
constexpr int BLOCK = 256;
constexpr int SCATTER_CELLS = 2048;          // LDS bins per component
// Columns of a marching block (y, x).
constexpr int MT_Y = 8, MT_X = 32;
// Blocks of the marching kernels that run at once: five and eight per CU (94
// and 56 registers).
constexpr int EXP_BWD_SLOTS = 1280, EXP_FWD_SLOTS = 2048;
// Tiles of the combination of the SVF gradients.
constexpr int CT_Z = 4, CT_Y = 8, CT_X = 32;
// Tiles of the windowed-statistics kernels: TY x TX columns, z chunks.
// Tile shapes (centres in y x x) of the window-statistics kernels; the block
// has one thread per centre.
constexpr int SIM_SHAPES = 3;
constexpr int SIM_SHAPE_Y[SIM_SHAPES] = {8, 16, 8};
constexpr int SIM_SHAPE_X[SIM_SHAPES] = {32, 32, 64};
// Blocks of each shape of the statistics and of the gradient that run at once
// (by their registers: 74 to 102 and 93 to 97 at w 7).
constexpr int STAT_SLOTS[SIM_SHAPES] = {1024, 768, 512};
constexpr int GRAD_SLOTS[SIM_SHAPES] = {1024, 512, 512};
constexpr int ELEM_PER_BLOCK = 1024;           // elementwise kernels

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline int point_tiles(int D, int H, int W) {
  return ceil_div(D, PT_Z) * ceil_div(H, PT_Y) * ceil_div(W, PT_X);
}
inline int march_tiles(int D, int H, int W, int zc) {
  return ceil_div(D, zc) * ceil_div(H, MT_Y) * ceil_div(W, MT_X);
}
inline int combine_tiles(int D, int H, int W) {
  return ceil_div(D, CT_Z) * ceil_div(H, CT_Y) * ceil_div(W, CT_X);
}
inline int sim_cols(int H, int W, int shape) {
  return ceil_div(H, SIM_SHAPE_Y[shape]) * ceil_div(W, SIM_SHAPE_X[shape]);
}
inline int stat_tiles(int D, int H, int W, int zc, int zs, int shape) {
  return ceil_div(D, zc) * ceil_div(zc, zs) * sim_cols(H, W, shape);
}
inline int grad_tiles(int D, int H, int W, int zg, int shape) {
  return ceil_div(D, zg) * sim_cols(H, W, shape);
}

// Launchers (kernels.hip).  All return hipError_t of the launch.  Those of a
// table of items in device memory have a twin for one item, which travels with
// the launch's arguments.
// Start and stop events for every following launch on this thread (null:
// untimed).  Each plan stage is one launch.
void set_launch_events(hipEvent_t start, hipEvent_t stop);
hipError_t launch_exp_fwd(const ExpFwdItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_exp_fwd(const ExpFwdItem& one, int n_tiles, hipStream_t s);
hipError_t launch_compose_fwd(const ComposeItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_compose_fwd(const ComposeItem& one, int n_tiles, hipStream_t s);
hipError_t launch_exp_bwd(const ExpBwdItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_exp_bwd(const ExpBwdItem& one, int n_tiles, hipStream_t s);
hipError_t launch_exp_far(const ExpBwdItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_exp_far(const ExpBwdItem& one, int n_tiles, hipStream_t s);
hipError_t launch_combine(const CombineItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_combine(const CombineItem& one, int n_tiles, hipStream_t s);
hipError_t launch_compose_bwd(const ComposeBwdItem* items, int n_items, int n_tiles,
                              hipStream_t s);
hipError_t launch_compose_bwd(const ComposeBwdItem& one, int n_tiles, hipStream_t s);
// Deterministic mode: the passes of the composition and Exp adjoints that
// only reduce each job's largest block magnitude into its slot (no other
// writes), the fold of the fixed-point fields, and the clearing of the slots.
hipError_t launch_compose_bwd_detmax(const ComposeBwdItem* items, int n_items, int n_tiles,
                                     hipStream_t s);
hipError_t launch_exp_far_detmax(const ExpBwdItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_det_fold(const DetFoldItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_det_clear(JobState* const* states, int n_jobs, hipStream_t s);
// M = I o (Omega + U) of each item, over point tiles of its grid.
hipError_t launch_warp(const SimItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_warp(const SimItem& one, int n_tiles, hipStream_t s);
hipError_t launch_sim_stats(const SimItem* items, int n_items, int n_tiles, int window, int metric,
                            int shape, hipStream_t s);
hipError_t launch_sim_stats(const SimItem& one, int n_tiles, int window, int metric, int shape,
                            hipStream_t s);
hipError_t launch_sim_grad(const SimItem* items, int n_items, int n_tiles, int window, int shape,
                           hipStream_t s);
hipError_t launch_sim_grad(const SimItem& one, int n_tiles, int window, int shape, hipStream_t s);
hipError_t launch_adam(const AdamItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_smooth(const SmoothItem* items, int n_items, int n_tiles, int lds_floats,
                         hipStream_t s);
// Fills the geometry and taps of a smoothing item; returns its tile count and
// raises *lds_floats to the LDS the item needs.
int smooth_item_setup(SmoothItem& it, const int dims[3], int axis, float sigma, int* lds_floats);
// Radius of the smoothing taps on a periodic line of n samples.
int smooth_radius(int n, float sigma);
hipError_t launch_finish(JobState* const* states, int n_jobs, hipStream_t s);
hipError_t launch_pool2(const PoolItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_pool2(const PoolItem& one, int n_tiles, hipStream_t s);
hipError_t launch_upsample2(const UpItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_upsample2(const UpItem& one, int n_tiles, hipStream_t s);
// adjoint: src [3][2D][2H][2W] (fine), dst [3][D][H][W] (coarse), tiles over the coarse grid
hipError_t launch_upsample2_adj(const UpItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_upsample2_adj(const UpItem& one, int n_tiles, hipStream_t s);
hipError_t launch_adam_flat(int64_t n, float* x, const float* g, float* m, float* v, int t,
                            float lr, float b1, float b2, float eps, hipStream_t s);
hipError_t launch_fill(float* p, int64_t n, float v, hipStream_t s);

// Scratch of the allocation-free similarity entry point: a file-scope device
// array (each GPU holds its own copy until the process ends) with the pair's
// sum in its first 256 bytes, then the warped source image and the window
// coefficients, for grids of up to NOALLOC_MAX_VOXELS voxels.
constexpr size_t NOALLOC_MAX_VOXELS = (size_t)6 << 20;
constexpr size_t NOALLOC_SCRATCH_BYTES = 256 + 16 * NOALLOC_MAX_VOXELS;
// Device address of the scratch array on `device`, which must be current:
// looked up once per device with hipGetSymbolAddress and kept (the array's
// name is a host-side stand-in, not a device address).
hipError_t noalloc_scratch_address(int device, void** ptr);
hipError_t launch_jacobian_det(GridDims d, const float* U, float* out, hipStream_t s);
hipError_t launch_rigid_grad(const RigidGradItem* items, int n_items, int n_tiles, hipStream_t s);
hipError_t launch_rigid_step(const RigidStepItem* items, int n_items, hipStream_t s);
// field [3][D][H][W] += the displacement of a rigid state
hipError_t launch_add_rigid(GridDims d, float* field, const RigidState* rg, hipStream_t s);
// 27 sums over the voxels with roi[p] != 0 (all if roi is NULL), added to out
hipError_t launch_field_stats(int V, const float* a, const float* b, const unsigned char* roi,
                              double* out, hipStream_t s);
// p[c][z][y][x] = off + amp * (a smooth periodic pattern); scratch data for
// the autotuner.
hipError_t launch_pattern(float* p, int64_t n, const int dims[3], float off, float amp,
                          float phase, hipStream_t s);

}  // namespace muster
