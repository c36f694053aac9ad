// HIP kernels (gfx950) of the MUSTER iteration.
//
// Data layout: a volume is float32 [D][H][W] (x fastest); a vector field is
// three such planes (components z, y, x).  Fields hold displacements in
// voxels.  Every kernel walks a table of work items (see muster_internal.h),
// so one launch covers all intervals, pairs and subjects of a stage.
//
// Sampling (paper Sec. 2.2, "trilinear interpolation"): the sample position
// q = p + u is clamped to the grid; the cell index is p + floor(u) and the
// fraction u - floor(u), which keeps the fraction exact for large p; an axis
// whose coordinate was clamped contributes no derivative.  Interpolation is
// the nested linear form a + t (b - a), so a constant field is reproduced
// exactly.
//
// The gather/scatter kernels use 8x8x16-voxel tiles and an XCD-aware
// block-to-tile map: blocks are dealt round-robin over the 8 XCDs, and the
// map hands each XCD a contiguous run of tiles so the neighbouring rows that
// the gathers touch stay in that XCD's L2.
#include <map>
#include <mutex>
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <algorithm>
#include <climits>
#include <cmath>

#include "muster_internal.h"

namespace muster {

namespace {

// Field pointers are used through the global address space so that loads,
// stores and atomics compile to global (not flat) memory instructions.
#define GLOBAL __attribute__((address_space(1)))
typedef GLOBAL float gfloat;
typedef GLOBAL const float cgfloat;
typedef float float2a __attribute__((ext_vector_type(2), aligned(4)));

__device__ __forceinline__ const cgfloat* gp(const float* p) { return (const cgfloat*)p; }
__device__ __forceinline__ gfloat* gp(float* p) { return (gfloat*)p; }
__device__ __forceinline__ void gadd(gfloat* p, float v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr float EPS_LNCC = 1e-10f;
constexpr float EPS_SILNCC = 1e-6f;

__device__ __forceinline__ int xcd_remap(int b, int n) {
  const int q = n >> 3, r = n & 7;
  const int x = b & 7, j = b >> 3;
  return x * q + min(x, r) + j;
}

template <class Item>
__device__ __forceinline__ int find_item(const Item* __restrict__ items, int n, int tile) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (items[mid].tile0 <= tile) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Where a kernel finds its item: a table in device memory, or, for calls of one
// item, the launch's own arguments, which spares the upload and, in every
// block, a dependent load.
template <class Item>
struct Table {
  const Item* __restrict__ items;
  int n;
  __device__ __forceinline__ const Item& at(int tile) const { return items[find_item(items, n, tile)]; }
};

template <class Item>
struct One {
  Item it;
  __device__ __forceinline__ const Item& at(int) const { return it; }
};

struct Ax {
  int i0;
  float t;
  float live;  // 1 inside the grid, 0 where the coordinate was clamped
};

// Axis of a displaced position p + u on n grid points.
__device__ __forceinline__ Ax axis_disp(int p, float u, int n) {
  u = fminf(fmaxf(u, -1.0e6f), 1.0e6f);
  const float fl = floorf(u);
  const int i = p + (int)fl;
  const float t = u - fl;
  Ax a;
  if (i < 0) {
    a.i0 = 0; a.t = 0.f; a.live = 0.f;
  } else if (i >= n - 1) {
    a.i0 = n - 2; a.t = 1.f; a.live = (i == n - 1 && t == 0.f) ? 1.f : 0.f;
  } else {
    a.i0 = i; a.t = t; a.live = 1.f;
  }
  return a;
}

// Axis of an absolute position q on n grid points.
__device__ __forceinline__ Ax axis_pos(float q, int n) {
  q = fminf(fmaxf(q, -1.0e6f), 1.0e6f);
  const float fl = floorf(q);
  const int i = (int)fl;
  const float t = q - fl;
  Ax a;
  if (i < 0) {
    a.i0 = 0; a.t = 0.f; a.live = 0.f;
  } else if (i >= n - 1) {
    a.i0 = n - 2; a.t = 1.f; a.live = (i == n - 1 && t == 0.f) ? 1.f : 0.f;
  } else {
    a.i0 = i; a.t = t; a.live = 1.f;
  }
  return a;
}

__device__ __forceinline__ float lerp_(float a, float b, float t) { return fmaf(t, b - a, a); }

// Loads at element i of a plane whose base is uniform across the wave: the
// byte offset is formed in 32 bits (i < 2^30 for any volume the library
// accepts), so the load takes the scalar base plus a 32-bit vector offset
// instead of a 64-bit vector address.  ld2o takes two consecutive floats in one
// 8-byte load (dword alignment suffices for multi-dword global loads).
__device__ __forceinline__ float2a ld2o(const cgfloat* plane, uint32_t i) {
  return *(const GLOBAL float2a*)((const GLOBAL char*)plane + (i << 2));
}

__device__ __forceinline__ float ldo(const cgfloat* plane, uint32_t i) {
  return *(const GLOBAL float*)((const GLOBAL char*)plane + (i << 2));
}
// One float per lane from global memory straight into LDS: lane l of the
// wave writes lds_wave[l], where lds_wave is the same for the whole wave (the
// first element of its run).  No register holds the value, and the barrier
// that follows waits for the load like for any other.  The callers walk
// element i = threadIdx.x + k * (block size), with block sizes multiples of
// 64, so a wave's run starts at i & ~63; lanes past the end stay inactive
// and write nothing.
__device__ __forceinline__ void ld_to_lds(const cgfloat* src, float* lds_wave) {
  __builtin_amdgcn_global_load_lds((const GLOBAL void*)src,
                                   (__attribute__((address_space(3))) void*)lds_wave, 4, 0, 0);
}

__device__ __forceinline__ void sto(gfloat* plane, uint32_t i, float v) {
  *(GLOBAL float*)((GLOBAL char*)plane + (i << 2)) = v;
}

// The window statistics' coefficients alpha, beta, gamma of one voxel, at voxel
// i of a plane whose base is uniform across the wave: one 12-byte access at a
// 32-bit offset (a plane has fewer than 2^28 voxels, the grid at least three
// planes).
struct Coef {
  float a, b, c;
};
__device__ __forceinline__ Coef ldo_coef(const GLOBAL Coef* plane, uint32_t i) {
  const cgfloat* p = (const cgfloat*)((const GLOBAL char*)plane + i * (uint32_t)sizeof(Coef));
  return {p[0], p[1], p[2]};
}
__device__ __forceinline__ void sto_coef(GLOBAL Coef* plane, uint32_t i, Coef v) {
  gfloat* p = (gfloat*)((GLOBAL char*)plane + i * (uint32_t)sizeof(Coef));
  p[0] = v.a;
  p[1] = v.b;
  p[2] = v.c;
}

// The 8 corners of a cell.  Corner order: bit 0 = x+1, bit 1 = y+1,
// bit 2 = z+1; the x pairs are adjacent in memory and come in one load.
__device__ __forceinline__ void load8(const cgfloat* __restrict__ f, int base, int sy, int sz,
                                      float (&v)[8]) {
  const uint32_t b0 = (uint32_t)base;
  const float2a a = ld2o(f, b0);
  const float2a b = ld2o(f, b0 + (uint32_t)sy);
  const float2a c = ld2o(f, b0 + (uint32_t)sz);
  const float2a d = ld2o(f, b0 + (uint32_t)(sz + sy));
  v[0] = a.x; v[1] = a.y;
  v[2] = b.x; v[3] = b.y;
  v[4] = c.x; v[5] = c.y;
  v[6] = d.x; v[7] = d.y;
}

__device__ __forceinline__ float tri_val(const float (&v)[8], float tz, float ty, float tx) {
  const float c00 = lerp_(v[0], v[1], tx);
  const float c01 = lerp_(v[2], v[3], tx);
  const float c10 = lerp_(v[4], v[5], tx);
  const float c11 = lerp_(v[6], v[7], tx);
  const float c0 = lerp_(c00, c01, ty);
  const float c1 = lerp_(c10, c11, ty);
  return lerp_(c0, c1, tz);
}

// Value and the three partial derivatives of the trilinear interpolant.
__device__ __forceinline__ float tri_grad(const float (&v)[8], float tz, float ty, float tx,
                                          float& dz, float& dy, float& dx) {
  const float c00 = lerp_(v[0], v[1], tx);
  const float c01 = lerp_(v[2], v[3], tx);
  const float c10 = lerp_(v[4], v[5], tx);
  const float c11 = lerp_(v[6], v[7], tx);
  const float c0 = lerp_(c00, c01, ty);
  const float c1 = lerp_(c10, c11, ty);
  dz = c1 - c0;
  dy = lerp_(c01 - c00, c11 - c10, tz);
  const float e0 = lerp_(v[1] - v[0], v[3] - v[2], ty);
  const float e1 = lerp_(v[5] - v[4], v[7] - v[6], ty);
  dx = lerp_(e0, e1, tz);
  return lerp_(c0, c1, tz);
}

struct PTile {
  int z0, y0, x0;
};

__device__ __forceinline__ PTile point_tile(int local, int H, int W) {
  const int ntx = (W + PT_X - 1) / PT_X;
  const int nty = (H + PT_Y - 1) / PT_Y;
  PTile t;
  t.x0 = (local % ntx) * PT_X;
  const int r = local / ntx;
  t.y0 = (r % nty) * PT_Y;
  t.z0 = (r / nty) * PT_Z;
  return t;
}

// Sum over a block of NT threads; the result is valid in thread 0.
template <int NT = BLOCK>
__device__ __forceinline__ double block_sum(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < NT / 64; ++i) s += red[i];
  return s;
}

// Minimum / maximum over a wave: four DPP steps leave each row of 16 lanes
// holding its row's result (swap neighbours, swap pairs, mirror the half
// rows, mirror the rows), and the four row results are read from lanes 15,
// 31, 47 and 63.  The result is wave-uniform.  Every lane must be active.
__device__ __forceinline__ int dpp_min(int v) {
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xF, 0xF, false));
  return min(min(__builtin_amdgcn_readlane(v, 15), __builtin_amdgcn_readlane(v, 31)),
             min(__builtin_amdgcn_readlane(v, 47), __builtin_amdgcn_readlane(v, 63)));
}
__device__ __forceinline__ int dpp_max(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xF, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xF, 0xF, false));
  return max(max(__builtin_amdgcn_readlane(v, 15), __builtin_amdgcn_readlane(v, 31)),
             max(__builtin_amdgcn_readlane(v, 47), __builtin_amdgcn_readlane(v, 63)));
}

// Sum over a wave by the same four DPP steps: after them every lane of a row
// holds its row's sum, in the same order in every lane, so the result is
// wave-uniform and does not depend on the lane a value came from.
__device__ __forceinline__ float dpp_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0xB1, 0xF, 0xF, false));
  v += __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x4E, 0xF, 0xF, false));
  v += __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x141, 0xF, 0xF, false));
  v += __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x140, 0xF, 0xF, false));
  const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 15));
  const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 31));
  const float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 47));
  const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
  return (a + b) + (c + d);
}

// Bounding box of the cells a tile touches.
struct BBox {
  int lz, ly, lx, ez, ey, ex, cells;
};

// ---------------------------------------------------------------------------
// Point tiles.  A thread owns VPT voxels of an 8x8x16 tile.  Their loads are
// issued together, component by component across the voxels, so each round
// trip to memory carries VPT gathers per thread: the gather kernels are bound
// by memory latency, not by bandwidth or address throughput, so memory-level
// parallelism is what sets their speed.  Voxels beyond the grid are clamped
// onto it (their loads stay in bounds) and their results are discarded.
// ---------------------------------------------------------------------------
constexpr int VPT = PT_VOX / BLOCK;

struct VoxSet {
  int p[VPT];           // linear index of the (clamped) voxel
  int z[VPT], y[VPT], x[VPT];
  bool ok[VPT];
};

__device__ __forceinline__ void vox_set(const PTile& tc, int D, int H, int W, VoxSet& vs) {
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const int k = threadIdx.x + j * BLOCK;
    const int x = tc.x0 + (k % PT_X), y = tc.y0 + (k / PT_X) % PT_Y, z = tc.z0 + k / (PT_X * PT_Y);
    vs.ok[j] = x < W && y < H && z < D;
    vs.x[j] = min(x, W - 1);
    vs.y[j] = min(y, H - 1);
    vs.z[j] = min(z, D - 1);
    vs.p[j] = (vs.z[j] * H + vs.y[j]) * W + vs.x[j];
  }
}

struct CellSet {
  int base[VPT];
  Ax az[VPT], ay[VPT], ax[VPT];
};

// Displacements (scaled by a) of the owned voxels and the cells they sample.
__device__ __forceinline__ void load_cells(const cgfloat* __restrict__ u, float a, int D, int H,
                                           int W, const VoxSet& vs, float (&uu)[VPT][3],
                                           CellSet& cs) {
  const int V = D * H * W;
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    uu[j][0] = a * ldo(u, vs.p[j]);
    uu[j][1] = a * ldo(u + V, vs.p[j]);
    uu[j][2] = a * ldo(u + 2 * V, vs.p[j]);
  }
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    cs.az[j] = axis_disp(vs.z[j], uu[j][0], D);
    cs.ay[j] = axis_disp(vs.y[j], uu[j][1], H);
    cs.ax[j] = axis_disp(vs.x[j], uu[j][2], W);
    cs.base[j] = (cs.az[j].i0 * H + cs.ay[j].i0) * W + cs.ax[j].i0;
  }
}

// Trilinear values of the three components of f at the cells.
__device__ __forceinline__ void sample_cells(const cgfloat* __restrict__ f, int V, int H, int W,
                                             const CellSet& cs, float (&out)[VPT][3]) {
  const int HW = H * W;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    float v[VPT][8];
#pragma unroll
    for (int j = 0; j < VPT; ++j) load8(f + c * V, cs.base[j], W, HW, v[j]);
#pragma unroll
    for (int j = 0; j < VPT; ++j) out[j][c] = tri_val(v[j], cs.az[j].t, cs.ay[j].t, cs.ax[j].t);
  }
}

// Scatter of per-voxel cell contributions into a field through LDS bins.
// Each thread holds up to VPT voxels: cell origin (cz, cy, cx), fractions,
// the 3-vector to spread with the trilinear weights, and optionally an own
// term to add at its own position (oz, oy, ox).
//
// The bins are 32-bit fixed point: every contribution is scaled by
// min(2^23 / m, 2^30 / S), where m is the largest magnitude the block
// spreads and S the sum over its voxels of their largest magnitudes,
// truncated, and added with an integer LDS atomic; integer LDS atomics run
// several times faster than float ones on this hardware and make the in-block
// sum independent of the order of the adds.  A bin holds at most the weighted
// values of the block's voxels, so its magnitude stays below 2^30 however
// strongly the sampling positions crowd into one cell: no bin can overflow.
// The error per contribution is below one quantum, 2^-23 m for spread-out
// boxes and 2^-30 S where many voxels share cells.  Each non-zero bin is then
// added to the field with one hardware float atomic.
constexpr float FIX_SCALE = 8388608.0f;   // 2^23
constexpr float FIX_TOTAL = 1073741824.0f; // 2^30
static_assert(SCATTER_CELLS % 4 == 0, "bin planes are cleared as int4");

struct ScatterVox {
  int cz, cy, cx;      // cell origin; cz < 0 marks an empty slot
  float tz, ty, tx;
  float g[3];          // value spread over the 8 corners
};

// Bounding box (lo/hi per axis), largest magnitude and sum of magnitudes over
// the block in one reduction: wave DPP steps, one LDS exchange, one barrier.
struct ScatterBox {
  BBox bb;
  float bmax;
  float bsum;
};

template <int NT>
__device__ __forceinline__ ScatterBox scatter_box(int (&lo)[3], int (&hi)[3], float mx, float sm,
                                                  int* sred) {
  // mx >= 0 (fmaxf drops NaN operands), so its bits order like its values
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lo[d] = dpp_min(lo[d]);
    hi[d] = dpp_max(hi[d]);
  }
  const int mxb = dpp_max(__float_as_int(mx));
  const float smw = dpp_sum(sm);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      sred[w * 8 + d] = lo[d];
      sred[w * 8 + 3 + d] = hi[d];
    }
    sred[w * 8 + 6] = mxb;
    sred[w * 8 + 7] = __float_as_int(smw);
  }
  __syncthreads();
  int l[3] = {INT_MAX, INT_MAX, INT_MAX}, h[3] = {INT_MIN, INT_MIN, INT_MIN};
  int mb = 0;
  float sb_sum = 0.f;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      l[d] = min(l[d], sred[i * 8 + d]);
      h[d] = max(h[d], sred[i * 8 + 3 + d]);
    }
    mb = max(mb, sred[i * 8 + 6]);
    sb_sum += __int_as_float(sred[i * 8 + 7]);
  }
  ScatterBox sb;
  sb.bmax = __int_as_float(mb);
  sb.bsum = sb_sum;
  sb.bb.lz = l[0]; sb.bb.ly = l[1]; sb.bb.lx = l[2];
  if (h[0] < l[0]) {
    sb.bb.ez = sb.bb.ey = sb.bb.ex = 0;
    sb.bb.cells = 0;
    return sb;
  }
  sb.bb.ez = h[0] - l[0] + 1;
  sb.bb.ey = h[1] - l[1] + 1;
  sb.bb.ex = h[2] - l[2] + 1;
  const long long c = (long long)sb.bb.ez * sb.bb.ey * sb.bb.ex;
  sb.bb.cells = c > (long long)INT_MAX ? INT_MAX : (int)c;
  return sb;
}

// ---------------------------------------------------------------------------
// Gathers from a box staged in LDS.  The block reduces the bounding box of
// the cells its voxels sample (the reduction of the scatters), loads that box
// of the three component planes straight into LDS (coalesced loads that do
// not pass through registers), and reads the 8 corners of each cell there.  A
// few wide row loads per cell then replace the scattered corner loads of every
// voxel, which otherwise keep the L1 and texture path saturated.  The values
// and the arithmetic are those of sample_cells, so the result is
// bit-identical; a box larger than GATHER_CELLS falls back to sample_cells.
// box: LDS of 3 * GATHER_CELLS floats.  Every thread of the block must call
// this.
//
// 2560 cells (30 KB of LDS) let five blocks share a CU, and the kernels that
// stage a box are held to five waves per SIMD (at most 102 VGPRs, no spill):
// 3-7 % faster than 3072 cells at four waves.  2048 cells at six waves per
// SIMD (80 VGPRs, a few bytes of spill) ran no faster.
// ---------------------------------------------------------------------------
constexpr int GATHER_CELLS = 2560;
// The adjoints read their corners from a box in the scatter bins' LDS.
constexpr int ADJ_BOX_CELLS = GATHER_CELLS < SCATTER_CELLS ? GATHER_CELLS : SCATTER_CELLS;
#define GATHER_WAVES __attribute__((amdgpu_waves_per_eu(5)))

__device__ __forceinline__ void sample_cells_lds(const cgfloat* __restrict__ f, int V, int H, int W,
                                                 const VoxSet& vs, const CellSet& cs,
                                                 float* __restrict__ box, int* sred,
                                                 float (&out)[VPT][3]) {
  int lo[3] = {INT_MAX, INT_MAX, INT_MAX};
  int hi[3] = {INT_MIN, INT_MIN, INT_MIN};
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    if (!vs.ok[j]) continue;
    lo[0] = min(lo[0], cs.az[j].i0); hi[0] = max(hi[0], cs.az[j].i0 + 1);
    lo[1] = min(lo[1], cs.ay[j].i0); hi[1] = max(hi[1], cs.ay[j].i0 + 1);
    lo[2] = min(lo[2], cs.ax[j].i0); hi[2] = max(hi[2], cs.ax[j].i0 + 1);
  }
  const BBox bb = scatter_box<BLOCK>(lo, hi, 0.f, 0.f, sred).bb;
  if (bb.cells == 0 || bb.cells > GATHER_CELLS) {  // block-uniform
    sample_cells(f, V, H, W, cs, out);
    return;
  }
  const int cells = bb.cells;
  // cell i -> (lz, ly, lx) by float reciprocals: exact here since i < 2^22
  const float inv_ex = 1.f / (float)bb.ex, inv_ey = 1.f / (float)bb.ey;
  for (int i = threadIdx.x; i < cells; i += BLOCK) {
    const int r = (int)(((float)i + 0.5f) * inv_ex);
    const int lx = i - r * bb.ex;
    const int lz = (int)(((float)r + 0.5f) * inv_ey);
    const int ly = r - lz * bb.ey;
    const int g = ((bb.lz + lz) * H + (bb.ly + ly)) * W + (bb.lx + lx);
    const int w0 = i & ~63;  // the wave's first cell: i = threadIdx.x + k * block
    ld_to_lds(f + g, box + w0);
    ld_to_lds(f + V + g, box + cells + w0);
    ld_to_lds(f + 2 * V + g, box + 2 * cells + w0);
  }
  __syncthreads();
  const int sy = bb.ex, sz = bb.ex * bb.ey;
  int l[VPT];
#pragma unroll
  for (int j = 0; j < VPT; ++j)
    l[j] = vs.ok[j] ? ((cs.az[j].i0 - bb.lz) * bb.ey + (cs.ay[j].i0 - bb.ly)) * bb.ex +
                          (cs.ax[j].i0 - bb.lx)
                    : 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float* __restrict__ b = box + c * cells;
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      const float* q = b + l[j];
      const float v[8] = {q[0], q[1], q[sy], q[sy + 1], q[sz], q[sz + 1], q[sz + sy], q[sz + sy + 1]};
      out[j][c] = tri_val(v, cs.az[j].t, cs.ay[j].t, cs.ax[j].t);
    }
  }
}

// ---------------------------------------------------------------------------
// Composition forward: out = prev + C o (Omega + prev)   (Eq. cum_deformation)
// ---------------------------------------------------------------------------
template <class Items>
__global__ __launch_bounds__(BLOCK) GATHER_WAVES void k_compose_fwd(const Items items, int n_tiles) {
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const ComposeItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W, V = D * H * W;
  const PTile tc = point_tile(tile - it.tile0, H, W);
  const cgfloat* __restrict__ pr = gp(it.prev);
  const cgfloat* __restrict__ C = gp(it.C);
  gfloat* __restrict__ o = gp(it.out);
  __shared__ float box[3 * GATHER_CELLS];
  __shared__ int sred[8 * (BLOCK / 64)];
  VoxSet vs;
  vox_set(tc, D, H, W, vs);
  float uu[VPT][3];
  CellSet cs;
  load_cells(pr, 1.f, D, H, W, vs, uu, cs);
  float sm[VPT][3];
  sample_cells_lds(C, V, H, W, vs, cs, box, sred, sm);
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    if (!vs.ok[j]) continue;
    sto(o, vs.p[j], uu[j][0] + sm[j][0]);
    sto(o + V, vs.p[j], uu[j][1] + sm[j][1]);
    sto(o + 2 * V, vs.p[j], uu[j][2] + sm[j][2]);
  }
}

// Deterministic accumulation: a block that would add into the float field
// with global atomics adds round(value * scale) into out64 instead (64-bit
// integer atomics, whose sum does not depend on their order).
struct DetOut {
  long long* out64 = nullptr;
  double scale = 0.0;
};

__device__ __forceinline__ void det_add(long long* p, float v, double scale) {
  const long long q = __double2ll_rn((double)v * scale);
  if (q != 0) atomicAdd(reinterpret_cast<unsigned long long*>(p), (unsigned long long)q);
}

// Scale of a job's deterministic slot over `blocks` blocks: 2^(61 - e) with
// 2^e >= blocks * m (m the slot's largest summed block magnitude), so that
// no cell of the 64-bit field can exceed 2^61; 0 when nothing finite was
// recorded.
__device__ __forceinline__ double det_scale(const JobState* js, int slot, int blocks) {
  const float m = __int_as_float((int)js->det_max[slot]);
  if (!(m > 0.f) || !(m < 3.0e38f)) return 0.0;
  int e;
  frexp((double)m * (double)blocks, &e);
  return ldexp(1.0, 61 - e);
}

// Bounding box, largest magnitude and summed magnitudes of a block's
// scatter (every thread must call it).
template <int NT>
__device__ __forceinline__ ScatterBox scatter_bound(const ScatterVox (&sv)[PT_VOX / NT], int* sred) {
  constexpr int VP = PT_VOX / NT;
  int lo[3] = {INT_MAX, INT_MAX, INT_MAX};
  int hi[3] = {INT_MIN, INT_MIN, INT_MIN};
  float mx = 0.f, sm = 0.f;
#pragma unroll
  for (int j = 0; j < VP; ++j) {
    if (sv[j].cz < 0) continue;
    lo[0] = min(lo[0], sv[j].cz); hi[0] = max(hi[0], sv[j].cz + 1);
    lo[1] = min(lo[1], sv[j].cy); hi[1] = max(hi[1], sv[j].cy + 1);
    lo[2] = min(lo[2], sv[j].cx); hi[2] = max(hi[2], sv[j].cx + 1);
    const float gm = fmaxf(fabsf(sv[j].g[0]), fmaxf(fabsf(sv[j].g[1]), fabsf(sv[j].g[2])));
    mx = fmaxf(mx, gm);
    sm += gm;
  }
  return scatter_box<NT>(lo, hi, mx, sm, sred);
}

// Largest magnitude and summed magnitudes of a block's scatter whose
// bounding box is already known; the same per-thread order and reductions as
// scatter_bound, so the scale is the same (every thread must call it).
template <int NT>
__device__ __forceinline__ ScatterBox scatter_mag(const ScatterVox (&sv)[PT_VOX / NT], int* sred,
                                                  const BBox& bb) {
  constexpr int VP = PT_VOX / NT;
  float mx = 0.f, sm = 0.f;
#pragma unroll
  for (int j = 0; j < VP; ++j) {
    if (sv[j].cz < 0) continue;
    const float gm = fmaxf(fabsf(sv[j].g[0]), fmaxf(fabsf(sv[j].g[1]), fabsf(sv[j].g[2])));
    mx = fmaxf(mx, gm);
    sm += gm;
  }
  const int mxb = dpp_max(__float_as_int(mx));
  const float smw = dpp_sum(sm);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sred[w * 8 + 6] = mxb;
    sred[w * 8 + 7] = __float_as_int(smw);
  }
  __syncthreads();
  int mb = 0;
  float sb_sum = 0.f;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    mb = max(mb, sred[i * 8 + 6]);
    sb_sum += __int_as_float(sred[i * 8 + 7]);
  }
  ScatterBox sb;
  sb.bb = bb;
  sb.bmax = __int_as_float(mb);
  sb.bsum = sb_sum;
  return sb;
}

// Deterministic mode, reduce-only pass: a block that will add into the flat
// field raises the job's slot to its summed magnitude.
template <int NT>
__device__ __forceinline__ void det_bound(const ScatterVox (&sv)[PT_VOX / NT], int* sred,
                                          JobState* js, int slot) {
  const ScatterBox sb = scatter_bound<NT>(sv, sred);
  if (sb.bb.cells == 0 || !(sb.bmax > 0.f)) return;
  if (threadIdx.x == 0) atomicMax(&js->det_max[slot], (unsigned int)__float_as_int(sb.bsum));
}

// RN: contributions rounded to nearest instead of truncated, two instructions
// where truncation takes one.
template <int NT, bool RN>
__device__ __forceinline__ void scatter_tile(const ScatterVox (&sv)[PT_VOX / NT], gfloat* __restrict__ out,
                                             int D, int H, int W, int* acc, int* sred,
                                             const DetOut& det = DetOut{},
                                             const BBox* known = nullptr) {
  constexpr int VP = PT_VOX / NT;
  const int HW = H * W, V = D * HW;
  const ScatterBox sb = known ? scatter_mag<NT>(sv, sred, *known) : scatter_bound<NT>(sv, sred);
  const BBox& bb = sb.bb;
  const float bmax = sb.bmax;
  // the bins take finite values only; bsum bounds every bin's magnitude
  const bool finite = bmax > 0.f && bmax < 3.0e38f && sb.bsum < 3.0e38f;
  if (bb.cells == 0) return;
  if (bb.cells <= SCATTER_CELLS && finite) {
    const float scale = fminf(FIX_SCALE / bmax, FIX_TOTAL / sb.bsum);
    const float inv = 1.f / scale;
    const int cells = bb.cells;
    // one plane of SCATTER_CELLS bins per component: the plane offsets are
    // constants, which the LDS instructions take as immediate offsets
    {
      int4* a4 = reinterpret_cast<int4*>(acc);
      const int n4 = (cells + 3) >> 2;
#pragma unroll
      for (int c = 0; c < 3; ++c)
        for (int i = threadIdx.x; i < n4; i += NT) a4[c * (SCATTER_CELLS / 4) + i] = make_int4(0, 0, 0, 0);
    }
    __syncthreads();
    const int sy = bb.ex, sz = bb.ex * bb.ey;
#pragma unroll
    for (int j = 0; j < VP; ++j) {
      if (sv[j].cz < 0) continue;
      const int l = ((sv[j].cz - bb.lz) * bb.ey + (sv[j].cy - bb.ly)) * bb.ex + (sv[j].cx - bb.lx);
      const float tz = sv[j].tz, ty = sv[j].ty, tx = sv[j].tx;
      const float w0z = 1.f - tz, w0y = 1.f - ty, w0x = 1.f - tx;
      const float w[8] = {w0z * w0y * w0x, w0z * w0y * tx, w0z * ty * w0x, w0z * ty * tx,
                          tz * w0y * w0x,  tz * w0y * tx,  tz * ty * w0x,  tz * ty * tx};
      const int off[8] = {0, 1, sy, sy + 1, sz, sz + 1, sz + sy, sz + sy + 1};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float g = sv[j].g[c] * scale;
        int* a = acc + c * SCATTER_CELLS + l;
#pragma unroll
        for (int q = 0; q < 8; ++q) atomicAdd(a + off[q], RN ? (int)rintf(w[q] * g) : (int)(w[q] * g));
      }
    }
    __syncthreads();
    // i -> (lz, ly, lx) by float reciprocals: exact here since i < 2^22
    const float inv_ex = 1.f / (float)bb.ex, inv_ey = 1.f / (float)bb.ey;
    for (int i = threadIdx.x; i < cells; i += NT) {
      const int r = (int)(((float)i + 0.5f) * inv_ex);
      const int lx = i - r * bb.ex;
      const int lz = (int)(((float)r + 0.5f) * inv_ey);
      const int ly = r - lz * bb.ey;
      const int gpos = ((bb.lz + lz) * H + (bb.ly + ly)) * W + (bb.lx + lx);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const int v = acc[c * SCATTER_CELLS + i];
        if (v == 0) continue;
        if (det.out64)
          det_add(det.out64 + c * V + gpos, (float)v * inv, det.scale);
        else
          gadd(out + c * V + gpos, (float)v * inv);
      }
    }
  } else {
    // The footprint does not fit the bins (or the values are not finite):
    // global float atomics.
#pragma unroll
    for (int j = 0; j < VP; ++j) {
      if (sv[j].cz < 0) continue;
      const int base = (sv[j].cz * H + sv[j].cy) * W + sv[j].cx;
      const float tz = sv[j].tz, ty = sv[j].ty, tx = sv[j].tx;
      const float w0z = 1.f - tz, w0y = 1.f - ty, w0x = 1.f - tx;
      const float w[8] = {w0z * w0y * w0x, w0z * w0y * tx, w0z * ty * w0x, w0z * ty * tx,
                          tz * w0y * w0x,  tz * w0y * tx,  tz * ty * w0x,  tz * ty * tx};
      const int off[8] = {0, 1, W, W + 1, HW, HW + 1, HW + W, HW + W + 1};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float g = sv[j].g[c];
        if (g == 0.f) continue;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          if (det.out64)
            det_add(det.out64 + c * V + base + off[q], w[q] * g, det.scale);
          else
            gadd(out + c * V + base + off[q], w[q] * g);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Marching blocks.  A block owns MT_Y x MT_X columns of the grid and walks a
// chunk of z, one plane per pass, with the columns' one-voxel halo: for
// fields whose displacement stays below one voxel, everything a voxel reads
// or receives lies in the 3 x 3 x 3 voxels around it, so the planes it needs
// are in LDS, and no box has to be found, loaded by cell index or exchanged.
//
// The patch of a block is its columns and the ring around them: PY x PX
// columns; thread t holds its own column and, for t < RING, one of the ring.
// ---------------------------------------------------------------------------
constexpr int MT_NT = MT_Y * MT_X, MT_PY = MT_Y + 2, MT_PX = MT_X + 2, MT_P1 = MT_PY * MT_PX,
              MT_RING = MT_P1 - MT_NT;
static_assert(MT_RING <= MT_NT, "one ring column per thread at most");

struct MTile {
  int z0, z1, y0, x0;
};

__device__ __forceinline__ MTile march_tile(int local, int D, int H, int W, int zc) {
  const int ntx = (W + MT_X - 1) / MT_X;
  const int nty = (H + MT_Y - 1) / MT_Y;
  MTile t;
  t.x0 = (local % ntx) * MT_X;
  const int r = local / ntx;
  t.y0 = (r % nty) * MT_Y;
  t.z0 = (r / nty) * zc;
  t.z1 = min(t.z0 + zc, D);
  return t;
}

// Patch coordinates of ring column r: top row, bottom row, then the sides.
__device__ __forceinline__ void ring_site(int r, int& row, int& col) {
  if (r < 2 * MT_PX) {
    row = r < MT_PX ? 0 : MT_PY - 1;
    col = r < MT_PX ? r : r - MT_PX;
  } else {
    const int q = r - 2 * MT_PX;
    row = 1 + (q >> 1);
    col = (q & 1) ? MT_PX - 1 : 0;
  }
}

// The three component planes of a field, their addresses held in scalar
// registers (the compiler otherwise adds the plane offset to each lane's
// 64-bit address).
template <class T>
struct Planes {
  T* c[3];
  __device__ __forceinline__ Planes(T* f, int V) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      c[k] = f + k * V;
      asm("" : "+s"(c[k]));
    }
  }
};

// One column of the patch: its offset in a plane (clamped onto the grid) and
// the bounds of an in-plane displacement that keep the sample on the grid.
struct MCol {
  uint32_t off;
  int place;     // row * MT_PX + column in the patch
  float ylo, yhi, xlo, xhi;
  bool in;
};

__device__ __forceinline__ MCol march_col(const MTile& tc, int row, int col, int H, int W) {
  MCol m;
  const int yy = tc.y0 - 1 + row, xx = tc.x0 - 1 + col;
  m.in = yy >= 0 && yy < H && xx >= 0 && xx < W;
  const int y = min(max(yy, 0), H - 1), x = min(max(xx, 0), W - 1);
  m.off = (uint32_t)(y * W + x);
  m.place = row * MT_PX + col;
  m.ylo = (float)-y; m.yhi = (float)(H - 1 - y);
  m.xlo = (float)-x; m.xhi = (float)(W - 1 - x);
  return m;
}

// Displacements held to the grid; a NaN goes to the lower bound, as the
// clamp of axis_disp takes it.
__device__ __forceinline__ void hold(const float (&u)[3], int z, int D, const MCol& m,
                                     float (&e)[3]) {
  e[0] = __builtin_amdgcn_fmed3f(u[0], (float)-z, (float)(D - 1 - z));
  e[1] = __builtin_amdgcn_fmed3f(u[1], m.ylo, m.yhi);
  e[2] = __builtin_amdgcn_fmed3f(u[2], m.xlo, m.xhi);
}

// max(0, v) of a v below 1, in one instruction (fmaxf quiets its operand first).
__device__ __forceinline__ float unit(float v) { return __builtin_amdgcn_fmed3f(v, 0.f, 1.f); }

// A voxel whose sample lies less than one voxel away along every axis.
__device__ __forceinline__ bool is_near(const float (&e)[3]) {
  return fmaxf(fabsf(e[0]), fmaxf(fabsf(e[1]), fabsf(e[2]))) < 1.f;
}

// The same of a voxel whose gradient the adjoint may gather: 0 * g is 0 for a
// finite g and NaN for any other, which compares as false.  Gathered, a value
// that is not finite would reach all 27 voxels around (a weight of 0 does not
// take it out), so its voxel goes to k_exp_far, which takes it to the cell's 8 corners.
__device__ __forceinline__ bool is_near(const float (&e)[3], const float (&g)[3]) {
  const float m = fmaxf(fabsf(e[0]), fmaxf(fabsf(e[1]), fabsf(e[2])));
  return fmaf(0.f, g[0], fmaf(0.f, g[1], fmaf(0.f, g[2], m))) < 1.f;
}

// ---------------------------------------------------------------------------
// Exp forward: one squaring u' = u + u o (Omega + u)   (Alg. 1)
//
// The corners of a near voxel's cell come from a ring of the last planes of u
// in LDS; a voxel that samples a voxel or more away reads its corners from
// memory.  Values and arithmetic are the same either way.
//
// Bound by memory: 24 bytes per voxel at 4 TB/s, the planes' halo coming from
// cache.  Against a box of sampled cells found and loaded per 8 x 8 x 16 tile
// (187 vector instructions per voxel, about 100 here): one 160x192x160 field
// 34.0 -> 28.3 us, six of them at once 38.7 -> 29.8 us per field.
//
// Far voxels lack the reuse that the box gave.  A whole integration of that
// field at K 7, before and now: 248 -> 207 us at 2.5 voxels, 239 -> 221 at 8, but
// 247 -> 261 at 16 and 293 -> 354 at 40, where most squarings are far.  A box for
// blocks of far voxels inside this kernel wins less than half of that back and
// costs near fields 2 %.
// ---------------------------------------------------------------------------
template <class Items>
__global__ __launch_bounds__(MT_NT) void k_exp_fwd(const Items items, int n_tiles) {
  constexpr int PX = MT_PX, ROW = 3 * PX, PLANE = MT_PY * ROW;
  __shared__ float up[4 * PLANE];  // a * src of the last planes, [plane & 3][row][component][column]
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const ExpFwdItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W, HW = H * W, V = D * HW;
  const MTile tc = march_tile(tile - it.tile0, D, H, W, it.zc);
  const float a = it.a;
  const Planes<const cgfloat> sp(gp(it.src), V);
  const Planes<gfloat> dp(gp(it.dst), V);
  const int ly = threadIdx.x / MT_X, lx = threadIdx.x % MT_X;
  const int y = tc.y0 + ly, x = tc.x0 + lx;
  const MCol own = march_col(tc, ly + 1, lx + 1, H, W);
  const bool ring = threadIdx.x < MT_RING;
  int rrow = 0, rcol = 0;
  if (ring) ring_site(threadIdx.x, rrow, rcol);
  const MCol rim = march_col(tc, rrow, rcol, H, W);
  float* const own_up = up + (ly + 1) * ROW + lx + 1;
  float* const rim_up = up + rrow * ROW + rcol;
  auto load = [&](int z, const MCol& m, float (&u)[3]) {
    const uint32_t p = (uint32_t)(min(max(z, 0), D - 1) * HW) + m.off;
#pragma unroll
    for (int c = 0; c < 3; ++c) u[c] = ldo(sp.c[c], p);
  };
  float nu[3], ru[3], pu[3] = {0.f, 0.f, 0.f}, res[3];
  load(tc.z0 - 1, own, nu);
  if (ring) load(tc.z0 - 1, rim, ru);
  for (int zp = tc.z0 - 1;; ++zp) {
    // plane zp into the ring: its slot was last read two passes ago
    float cu[3];
    const int slot = (zp & 3) * PLANE;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      cu[c] = a * nu[c];
      own_up[slot + c * PX] = cu[c];
    }
    if (ring) {
#pragma unroll
      for (int c = 0; c < 3; ++c) rim_up[slot + c * PX] = a * ru[c];
    }
    __syncthreads();
    // the last pass's results before the next plane's loads (see k_exp_bwd)
    if (zp - 2 >= tc.z0 && own.in) {
      const uint32_t p = (uint32_t)((zp - 2) * HW) + own.off;
#pragma unroll
      for (int c = 0; c < 3; ++c) sto(dp.c[c], p, res[c]);
    }
    if (zp > tc.z1) break;
    if (zp < tc.z1) {
      load(zp + 1, own, nu);
      if (ring) load(zp + 1, rim, ru);
    }
    const int zo = zp - 1;
    if (zo >= tc.z0 && own.in) {
      float e[3];
      hold(pu, zo, D, own, e);
      if (is_near(e)) {
        const bool bz = e[0] < 0.f || zo == D - 1, by = e[1] < 0.f || y == H - 1,
                   bx = e[2] < 0.f || x == W - 1;
        const int q = (ly + 1 - (by ? 1 : 0)) * ROW + lx + 1 - (bx ? 1 : 0);
        const float* q0 = up + ((bz ? zo - 1 : zo) & 3) * PLANE + q;
        const float* q1 = up + ((bz ? zo : zo + 1) & 3) * PLANE + q;
        const float tz = e[0] + (bz ? 1.f : 0.f), ty = e[1] + (by ? 1.f : 0.f),
                    tx = e[2] + (bx ? 1.f : 0.f);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const int o = c * PX;
          const float v[8] = {q0[o], q0[o + 1], q0[o + ROW], q0[o + ROW + 1],
                              q1[o], q1[o + 1], q1[o + ROW], q1[o + ROW + 1]};
          res[c] = pu[c] + tri_val(v, tz, ty, tx);
        }
      } else {
        const Ax az = axis_disp(zo, pu[0], D), ay = axis_disp(y, pu[1], H),
                 ax = axis_disp(x, pu[2], W);
        const int base = (az.i0 * H + ay.i0) * W + ax.i0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          float v[8];
          load8(sp.c[c], base, W, HW, v);
          res[c] = pu[c] + a * tri_val(v, az.t, ay.t, ax.t);
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) pu[c] = cu[c];
  }
}

// ---------------------------------------------------------------------------
// Exp backward: one squaring, dL/du_s from dL/du_{s+1}
//   G_s(p) = G(p) + J_u(q)^T G(p) + sum_{p': corners of q(p') contain p} w G(p')
// scaled by the item's oscale.
//
// The sum is formed as a gather.  A near voxel p' (held displacement e below
// one voxel on every axis) reaches p only from the 27 voxels around p, with
// the weight hat(e_z + dz) hat(e_y + dy) hat(e_x + dx), where p' = p + d and
// hat(v) = max(0, 1 - |v|); for |e| < 1 the three hats of an axis are
// max(0, e), 1 - |e| and max(0, -e): one instruction each.  Walking z, plane
// zp adds to the sums of planes zp - 1, zp and zp + 1, which each thread
// keeps in registers, so a plane's G and displacements are read from LDS
// once per output column (9 records).  The corners of J_u come from a ring of
// the last planes of u.  Voxels that are not near, or whose G is not finite,
// take no part here: the block marks their point tile in `far`, and k_exp_far
// adds what they spread.
//
// Plain sums in a fixed order: no atomics, no fixed point, and the result
// does not depend on the tiling or on what shares the launch.  Held to 96
// registers: five blocks per CU (98 would leave four).
//
// Bound by vector issue: about 330 instructions per voxel, where the exchange
// of scatter boxes in LDS that this replaced took 512 and moved 60 bytes per
// voxel against 43 (the columns' halo included).  160x192x160, K 7, the whole
// adjoint with its forward steps: 975 -> 672 us (584 with those marching as
// well), and the error against 64 bits 1.2e-5 -> 1.2e-7.  8 x 32 columns: whole 128-byte lines per row and no bank
// conflicts between a wave's rows; six 160x192x160 fields at once take 284 us,
// with 16 x 16 columns 361, with 16 x 32 300, with 8 x 16 403, with 4 x 64 324.
// ---------------------------------------------------------------------------
template <class Items>
__global__ __launch_bounds__(MT_NT) GATHER_WAVES void k_exp_bwd(const Items items, int n_tiles) {
  constexpr int PX = MT_PX, ROW = 3 * PX, PLANE = MT_PY * ROW;
  __shared__ float4 ra[2][MT_P1];  // e_z, e_y, e_x, G_z of a plane
  __shared__ float2 rb[2][MT_P1];  // G_y, G_x
  __shared__ float up[4 * PLANE];  // u of the last planes, [plane & 3][row][component][column]
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const ExpBwdItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W, HW = H * W, V = D * HW;
  const MTile tc = march_tile(tile - it.tile0, D, H, W, it.zc);
  const float a = it.a;
  const cgfloat* __restrict__ s = gp(it.src);
  const Planes<const cgfloat> sp(s, V), gi(gp(it.gin), V);
  const Planes<gfloat> go(gp(it.gout), V);
  const int ly = threadIdx.x / MT_X, lx = threadIdx.x % MT_X;
  const int y = tc.y0 + ly, x = tc.x0 + lx;
  const MCol own = march_col(tc, ly + 1, lx + 1, H, W);
  const bool ring = threadIdx.x < MT_RING;
  int rrow = 0, rcol = 0;
  if (ring) ring_site(threadIdx.x, rrow, rcol);
  const MCol rim = march_col(tc, rrow, rcol, H, W);
  auto load = [&](int z, const MCol& m, float (&u)[3], float (&g)[3]) {
    const uint32_t p = (uint32_t)(min(max(z, 0), D - 1) * HW) + m.off;
#pragma unroll
    for (int c = 0; c < 3; ++c) u[c] = ldo(sp.c[c], p);
#pragma unroll
    for (int c = 0; c < 3; ++c) g[c] = ldo(gi.c[c], p);
  };
  // a column's record of plane z, u scaled by a; whether its voxel is gathered
  auto record = [&](int z, const MCol& m, const float (&u)[3], const float (&g)[3]) {
    float e[3];
    hold(u, z, D, m, e);
    const bool take = m.in && is_near(e, g);
    ra[z & 1][m.place] = make_float4(e[0], e[1], e[2], take ? g[0] : 0.f);
    rb[z & 1][m.place] = make_float2(take ? g[1] : 0.f, take ? g[2] : 0.f);
    float* q = up + (z & 3) * PLANE + (m.place / PX) * ROW + m.place % PX;
#pragma unroll
    for (int c = 0; c < 3; ++c) q[c * PX] = u[c];
    return take;
  };
  float nu[3], ng[3], ru[3], rg[3];  // plane zp of the own and the ring column, loaded ahead
  load(tc.z0 - 1, own, nu, ng);
  if (ring) load(tc.z0 - 1, rim, ru, rg);
  float s0[3] = {0.f, 0.f, 0.f}, s1[3] = {0.f, 0.f, 0.f}, s2[3] = {0.f, 0.f, 0.f};
  float pu[3] = {0.f, 0.f, 0.f}, pg[3] = {0.f, 0.f, 0.f};  // own column at plane zp - 1
  bool near = false;  // the own voxel of plane zp - 1 is gathered
  float res[3];
  for (int zp = tc.z0 - 1;; ++zp) {
    float cu[3], cg[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      cu[c] = a * nu[c];
      cg[c] = ng[c];
    }
    // records of plane zp.  The buffers written here were last read two
    // (records) and three (ring of u) planes ago, before the last barrier.
    const bool in_z = zp >= 0 && zp < D && zp <= tc.z1;
    bool next = false;
    if (in_z) {
      next = record(zp, own, cu, cg);
      if (ring) {
        const float v[3] = {a * ru[0], a * ru[1], a * ru[2]};
        record(zp, rim, v, rg);
      }
    }
    __syncthreads();
    // the last pass's results go out before the next plane's loads, so that
    // the wait for those does not also wait for stores issued after them
    if (zp - 2 >= tc.z0 && own.in) {
      const uint32_t p = (uint32_t)((zp - 2) * HW) + own.off;
#pragma unroll
      for (int c = 0; c < 3; ++c) sto(go.c[c], p, res[c]);
    }
    if (zp > tc.z1) break;
    if (zp < tc.z1) {
      load(zp + 1, own, nu, ng);
      if (ring) load(zp + 1, rim, ru, rg);
    }
    if (in_z) {
      // first column of the 3 x 3 around the own one, so that every offset
      // is an immediate one
      const float4* qa = ra[zp & 1] + (own.place - PX - 1);
      const float2* qb = rb[zp & 1] + (own.place - PX - 1);
      // what goes to plane zp - 1, to zp + 1, and to all three: the hats of
      // an axis sum to one
      float dn[3] = {0.f, 0.f, 0.f}, all[3] = {0.f, 0.f, 0.f};
#pragma unroll
      for (int dy = 0; dy <= 2; ++dy)
#pragma unroll
        for (int dx = 0; dx <= 2; ++dx) {
          const float4 A = qa[dy * PX + dx];
          const float2 B = qb[dy * PX + dx];
          const float hy = dy == 1 ? 1.f - fabsf(A.y) : unit(dy < 1 ? A.y : -A.y);
          const float hx = dx == 1 ? 1.f - fabsf(A.z) : unit(dx < 1 ? A.z : -A.z);
          const float w = hy * hx, wd = w * unit(-A.x), wu = w * unit(A.x);
          const float g[3] = {A.w, B.x, B.y};
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            all[c] = fmaf(w, g[c], all[c]);
            dn[c] = fmaf(wd, g[c], dn[c]);
            s2[c] = fmaf(wu, g[c], s2[c]);
          }
        }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        s0[c] += dn[c];
        s1[c] += all[c] - dn[c] - s2[c];
      }
    }
    const int zo = zp - 1;
    if (zo >= tc.z0 && own.in) {
      // (J^T g) of the Jacobian J of u at q is the gradient of the
      // interpolant of sum_c g_c u_c: combine the corners first, then one
      // gradient; clamped axes contribute nothing
      float e[3], jz, jy, jx, v[8], lz, ly_, lx_;
      hold(pu, zo, D, own, e);
      if (near) {
        const bool bz = e[0] < 0.f || zo == D - 1, by = e[1] < 0.f || y == H - 1,
                   bx = e[2] < 0.f || x == W - 1;
        const int row = ly + 1 - (by ? 1 : 0), col = lx + 1 - (bx ? 1 : 0);
        const int q = row * ROW + col;
        const float* q0 = up + ((bz ? zo - 1 : zo) & 3) * PLANE + q;
        const float* q1 = up + ((bz ? zo : zo + 1) & 3) * PLANE + q;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int o = (k >> 1) * ROW + (k & 1);
          v[k] = fmaf(pg[2], q0[o + 2 * PX], fmaf(pg[1], q0[o + PX], pg[0] * q0[o]));
          v[4 + k] = fmaf(pg[2], q1[o + 2 * PX], fmaf(pg[1], q1[o + PX], pg[0] * q1[o]));
        }
        tri_grad(v, e[0] + (bz ? 1.f : 0.f), e[1] + (by ? 1.f : 0.f), e[2] + (bx ? 1.f : 0.f), jz,
                 jy, jx);
        lz = e[0] == pu[0] ? jz : 0.f;
        ly_ = e[1] == pu[1] ? jy : 0.f;
        lx_ = e[2] == pu[2] ? jx : 0.f;
      } else {
        const Ax az = axis_disp(zo, pu[0], D), ay = axis_disp(y, pu[1], H),
                 ax = axis_disp(x, pu[2], W);
        const int base = (az.i0 * H + ay.i0) * W + ax.i0;
        float t[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          load8(s + c * V, base, W, HW, t);
#pragma unroll
          for (int k = 0; k < 8; ++k) v[k] = fmaf(a * pg[c], t[k], v[k]);
        }
        tri_grad(v, az.t, ay.t, ax.t, jz, jy, jx);
        lz = az.live * jz;
        ly_ = ay.live * jy;
        lx_ = ax.live * jx;
        const int ntx = (W + PT_X - 1) / PT_X, nty = (H + PT_Y - 1) / PT_Y;
        ((GLOBAL int*)it.far)[((zo / PT_Z) * nty + y / PT_Y) * ntx + x / PT_X] = 1;
      }
      const float o = it.oscale;
      res[0] = o * (s0[0] + (pg[0] + lz));
      res[1] = o * (s0[1] + (pg[1] + ly_));
      res[2] = o * (s0[2] + (pg[2] + lx_));
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      s0[c] = s1[c];
      s1[c] = s2[c];
      s2[c] = 0.f;
      pu[c] = cu[c];
      pg[c] = cg[c];
    }
    near = next;
  }
}

// v spread over the 8 corners of a cell of one plane by float atomics.
__device__ __forceinline__ void spread(gfloat* __restrict__ out, int base, int W, int HW,
                                       const ScatterVox& s, float v) {
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const float wz = k & 4 ? s.tz : 1.f - s.tz, wy = k & 2 ? s.ty : 1.f - s.ty,
                wx = k & 1 ? s.tx : 1.f - s.tx;
    gadd(out + base + (k & 4 ? HW : 0) + (k & 2 ? W : 0) + (k & 1), wz * wy * wx * v);
  }
}

// What the voxels that k_exp_bwd left out spread, added into the field that it
// has written, over the point tiles it marked.  A block looks at
// `group` marks, a grid apart, with one load and ends there when none is set,
// which is the usual case: displacements reach a voxel only in the last
// squarings of a large deformation, and then in neighbouring tiles, which so
// fall to different blocks.  The marks are cleared once read.  DETMAX: the
// deterministic mode's reduce-only pass (no writes but the job's slot).
template <bool DETMAX, class Items>
__global__ __launch_bounds__(BLOCK) void k_exp_far(const Items items, int n_tiles, int group) {
  __shared__ __align__(16) int acc[DETMAX ? 4 : 3 * SCATTER_CELLS];
  __shared__ int sred[8 * (BLOCK / 64)];
  const int lane = threadIdx.x & 63;
  const int mine = blockIdx.x + lane * gridDim.x;
  int mark = 0;
  if (lane < group && mine < n_tiles) {
    const ExpBwdItem& m = items.at(mine);
    mark = m.far[mine - m.tile0];
  }
  uint64_t todo = __ballot(mark != 0);  // the same in every wave of the block
  if (!todo) return;
  __syncthreads();  // every wave has read the marks
  while (todo) {
    const int tile = blockIdx.x + __builtin_ctzll(todo) * gridDim.x;
    todo &= todo - 1;
    const ExpBwdItem it = items.at(tile);
    const int D = it.D, H = it.H, W = it.W, V = D * H * W;
    const PTile tc = point_tile(tile - it.tile0, H, W);
    const cgfloat* __restrict__ s = gp(it.src);
    const cgfloat* __restrict__ gin = gp(it.gin);
    if (!DETMAX && threadIdx.x == 0) it.far[tile - it.tile0] = 0;
    VoxSet vs;
    vox_set(tc, D, H, W, vs);
    float uu[VPT][3];
    CellSet cs;
    load_cells(s, it.a, D, H, W, vs, uu, cs);
    ScatterVox sv[VPT];
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      MCol m;
      m.ylo = (float)-vs.y[j]; m.yhi = (float)(H - 1 - vs.y[j]);
      m.xlo = (float)-vs.x[j]; m.xhi = (float)(W - 1 - vs.x[j]);
      float e[3];
      hold(uu[j], vs.z[j], D, m, e);
      sv[j].cz = -1;
      float g[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) g[c] = ldo(gin + c * V, vs.p[j]);
      if (!vs.ok[j] || is_near(e, g)) continue;
      sv[j].cz = cs.az[j].i0; sv[j].cy = cs.ay[j].i0; sv[j].cx = cs.ax[j].i0;
      sv[j].tz = cs.az[j].t; sv[j].ty = cs.ay[j].t; sv[j].tx = cs.ax[j].t;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        float v = it.oscale * g[c];
        if (!(fabsf(v) < INFINITY)) {
          // no sum of the bins: straight to the corners, in any order
          if (!DETMAX) spread(gp(it.gout) + c * V, cs.base[j], W, H * W, sv[j], v);
          v = 0.f;
        }
        sv[j].g[c] = v;
      }
    }
    if (DETMAX) {
      det_bound<BLOCK>(sv, sred, it.js, it.det_slot);
    } else {
      DetOut det;
      if (it.gout64) {
        det.out64 = it.gout64;
        det.scale = det_scale(it.js, it.det_slot, it.det_blocks);
        if (threadIdx.x == 0) *it.flag64 = 1;
      }
      scatter_tile<BLOCK, true>(sv, gp(it.gout), D, H, W, acc, sred, det);
    }
    __syncthreads();  // acc and sred are free for the next tile
  }
}

// ---------------------------------------------------------------------------
// The gradient of each SVF from the G_0 of its forward and backward
// directions, and the regularisers (Eq. reg_sum): out = gmul (gf + gb +
// the regularisers' gradients), and their weighted values added to loss.
// Blocks of CT_Y x CT_X columns walk CT_Z planes; the neighbours along z stay
// in registers and those in the plane come from cache, so the field is read
// from memory once and the kernel moves 12 bytes per field named in the item.
// Bound by latency: few planes per thread, many blocks, and the values' sums in
// slots (LOSS_SLOTS).  Three fields of 160x192x160: the values alone 103 -> 74
// us, with the gradient of two directions 170 -> 154 us.
// ---------------------------------------------------------------------------
template <class Items>
__global__ __launch_bounds__(CT_Y * CT_X) void k_combine(const Items items, int n_tiles) {
  __shared__ double red[CT_Y * CT_X / 64];
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const CombineItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W, HW = H * W, V = D * HW;
  const int local = tile - it.tile0;
  const int ntx = (W + CT_X - 1) / CT_X, nty = (H + CT_Y - 1) / CT_Y;
  const int x = (local % ntx) * CT_X + threadIdx.x % CT_X;
  const int r = local / ntx;
  const int y = (r % nty) * CT_Y + threadIdx.x / CT_X;
  const int z0 = (r / nty) * CT_Z, z1 = min(z0 + CT_Z, D);
  const cgfloat* __restrict__ gf = gp(it.gf);
  const cgfloat* __restrict__ gb = gp(it.gb);
  const cgfloat* __restrict__ f = gp(it.flow);
  gfloat* __restrict__ out = gp(it.out);
  const bool reg = it.reg_w != 0.f || it.loss_w[0] != 0.0;  // uniform
  const bool grad = it.out != nullptr;  // the value alone takes forward differences only
  const float inv_mz = 1.f / (float)((D - 1) * H * W), inv_my = 1.f / (float)(D * (H - 1) * W),
              inv_mx = 1.f / (float)(D * H * (W - 1));
  double sz = 0.0, sy = 0.0, sx = 0.0, ext = 0.0;
  if (y < H && x < W) {
    float fm[3] = {0.f, 0.f, 0.f}, fc[3] = {0.f, 0.f, 0.f};
    uint32_t p = (uint32_t)((z0 * H + y) * W + x);
    if (reg) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        fc[c] = ldo(f + c * V, p);
        if (grad && z0 > 0) fm[c] = ldo(f + c * V, p - HW);
      }
    }
    for (int z = z0; z < z1; ++z, p += HW) {
      float g[3] = {0.f, 0.f, 0.f}, fp[3];
      if (it.gf) {
#pragma unroll
        for (int c = 0; c < 3; ++c) g[c] = ldo(gf + c * V, p);
      }
      if (it.gb) {
#pragma unroll
        for (int c = 0; c < 3; ++c) g[c] += ldo(gb + c * V, p);
      }
      if (reg) {
        float ym[3], yp[3], xm[3], xp[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const cgfloat* __restrict__ q = f + c * V;
          fp[c] = z + 1 < D ? ldo(q, p + HW) : 0.f;
          ym[c] = grad && y > 0 ? ldo(q, p - W) : 0.f;
          yp[c] = y + 1 < H ? ldo(q, p + W) : 0.f;
          xm[c] = grad && x > 0 ? ldo(q, p - 1) : 0.f;
          xp[c] = x + 1 < W ? ldo(q, p + 1) : 0.f;
        }
        // the differences are floats, their squares and sums doubles
        auto square = [](double& v, float d) { v = fma((double)d, (double)d, v); };
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          float rg = 0.f;
          if (z + 1 < D) { const float d = fp[c] - fc[c]; rg -= 2.f * d * inv_mz; square(sz, d); }
          if (z > 0)     { const float d = fc[c] - fm[c]; rg += 2.f * d * inv_mz; }
          if (y + 1 < H) { const float d = yp[c] - fc[c]; rg -= 2.f * d * inv_my; square(sy, d); }
          if (y > 0)     { const float d = fc[c] - ym[c]; rg += 2.f * d * inv_my; }
          if (x + 1 < W) { const float d = xp[c] - fc[c]; rg -= 2.f * d * inv_mx; square(sx, d); }
          if (x > 0)     { const float d = fc[c] - xm[c]; rg += 2.f * d * inv_mx; }
          g[c] = fmaf(it.reg_w, rg, g[c]);
          fm[c] = fc[c];
          fc[c] = fp[c];
        }
      }
      if (it.ext) {
        // L_L2 and L_ts (Sec. 2.4): linear in the flows of this interval and its neighbours
        double a2 = 0.0, t2 = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float v = ldo(f + c * V, p);
          g[c] = fmaf(it.w_self, v, g[c]);
          a2 += (double)v * v;
          if (it.flow_prev) {
            const float vp = ldo(gp(it.flow_prev) + c * V, p);
            g[c] = fmaf(it.w_prev, vp, g[c]);
            const double d = (double)vp * it.inv_dprev - (double)v * it.inv_dself;
            t2 += d * d;
          }
          if (it.flow_next) g[c] = fmaf(it.w_next, ldo(gp(it.flow_next) + c * V, p), g[c]);
        }
        ext += (double)it.l2_loss_w * a2 + (double)it.ts_loss_w * t2;
      }
      if (it.out) {
#pragma unroll
        for (int c = 0; c < 3; ++c) sto(out + c * V, p, it.gmul * g[c]);
      }
    }
  }
  if (it.loss && (reg || it.ext)) {
    const double tot = block_sum<CT_Y * CT_X>(it.loss_w[0] * sz + it.loss_w[1] * sy + it.loss_w[2] * sx + ext, red);
    if (threadIdx.x == 0)
      unsafeAtomicAdd(it.loss + (blockIdx.x % LOSS_SLOTS) * LOSS_STRIDE, tot);
  }
}

// ---------------------------------------------------------------------------
// Composition backward
// ---------------------------------------------------------------------------
// The composition adjoint runs 512 threads per point tile (two voxels each):
// with its extra streams (G, U_prev, G_prev) it gains more from the higher
// occupancy than it loses in loads in flight per thread (measured: 11 %).
constexpr int CB_NT = 2 * BLOCK, CB_VP = PT_VOX / CB_NT;
static_assert(BLOCK % 64 == 0 && CB_NT % 64 == 0, "blocks of whole waves (ld_to_lds)");

template <bool DETMAX, class Items>
__global__ __launch_bounds__(CB_NT) void k_compose_bwd(const Items items, int n_tiles) {
  __shared__ __align__(16) int acc[3 * SCATTER_CELLS];
  __shared__ int sred[16 * (CB_NT / 64)];
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const ComposeBwdItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W, HW = H * W, V = D * HW;
  const PTile tc = point_tile(tile - it.tile0, H, W);
  const cgfloat* __restrict__ C = gp(it.C);
  const cgfloat* __restrict__ pr = gp(it.prev);
  const cgfloat* __restrict__ G = gp(it.g);
  gfloat* __restrict__ gpv = gp(it.gprev);
  // the owned voxels, the cells they sample and G there
  int vp[CB_VP], vz[CB_VP], vy[CB_VP], vx[CB_VP];
  bool vok[CB_VP];
  Ax cz[CB_VP], cy[CB_VP], cx[CB_VP];
  float gv[CB_VP][3];
#pragma unroll
  for (int j = 0; j < CB_VP; ++j) {
    const int k = threadIdx.x + j * CB_NT;
    vx[j] = tc.x0 + (k % PT_X);
    vy[j] = tc.y0 + (k / PT_X) % PT_Y;
    vz[j] = tc.z0 + k / (PT_X * PT_Y);
    vok[j] = vx[j] < W && vy[j] < H && vz[j] < D;
    vp[j] = vok[j] ? (vz[j] * H + vy[j]) * W + vx[j] : 0;
    const float uz = ldo(pr, vp[j]), uy = ldo(pr + V, vp[j]), ux = ldo(pr + 2 * V, vp[j]);
    cz[j] = axis_disp(vz[j], uz, D);
    cy[j] = axis_disp(vy[j], uy, H);
    cx[j] = axis_disp(vx[j], ux, W);
    gv[j][0] = ldo(G, vp[j]);
    gv[j][1] = ldo(G + V, vp[j]);
    gv[j][2] = ldo(G + 2 * V, vp[j]);
  }
  // the corners come from a box of C staged in acc (the bounding box of the
  // cells, which is also the scatter's box; the values are those of the
  // direct loads), or directly when the box is larger than ADJ_BOX_CELLS; the
  // reduce-only pass needs no corners
  BBox gb{};
  bool lds_box = false;
  if (!DETMAX) {
    int lo[3] = {INT_MAX, INT_MAX, INT_MAX};
    int hi[3] = {INT_MIN, INT_MIN, INT_MIN};
#pragma unroll
    for (int j = 0; j < CB_VP; ++j) {
      if (!vok[j]) continue;
      lo[0] = min(lo[0], cz[j].i0); hi[0] = max(hi[0], cz[j].i0 + 1);
      lo[1] = min(lo[1], cy[j].i0); hi[1] = max(hi[1], cy[j].i0 + 1);
      lo[2] = min(lo[2], cx[j].i0); hi[2] = max(hi[2], cx[j].i0 + 1);
    }
    // the second half of sred: the scatter's own reduction uses the first
    gb = scatter_box<CB_NT>(lo, hi, 0.f, 0.f, sred + 8 * (CB_NT / 64)).bb;
    lds_box = gb.cells > 0 && gb.cells <= ADJ_BOX_CELLS;  // block-uniform
    if (lds_box) {
      float* box = reinterpret_cast<float*>(acc);
      const int cells = gb.cells;
      // cell i -> (lz, ly, lx) by float reciprocals: exact here since i < 2^22
      const float inv_ex = 1.f / (float)gb.ex, inv_ey = 1.f / (float)gb.ey;
      for (int i = threadIdx.x; i < cells; i += CB_NT) {
        const int r = (int)(((float)i + 0.5f) * inv_ex);
        const int lx = i - r * gb.ex;
        const int lz = (int)(((float)r + 0.5f) * inv_ey);
        const int ly = r - lz * gb.ey;
        const int g = ((gb.lz + lz) * H + (gb.ly + ly)) * W + (gb.lx + lx);
        const int w0 = i & ~63;  // the wave's first cell: i = threadIdx.x + k * block
        ld_to_lds(C + g, box + w0);
        ld_to_lds(C + V + g, box + cells + w0);
        ld_to_lds(C + 2 * V + g, box + 2 * cells + w0);
      }
      __syncthreads();
    }
  }
  ScatterVox sv[CB_VP];
#pragma unroll
  for (int j = 0; j < CB_VP; ++j) {
    sv[j].cz = -1;
    if (!vok[j]) continue;
    const int p = vp[j];
    const Ax az = cz[j], ay = cy[j], ax = cx[j];
    const float g0 = gv[j][0], g1 = gv[j][1], g2 = gv[j][2];
    float v0[8], v1[8], v2[8], dz, dy, dx;
    if (lds_box) {
      const float* box = reinterpret_cast<const float*>(acc);
      const int cells = gb.cells, sy = gb.ex, sz = gb.ex * gb.ey;
      const int l = ((az.i0 - gb.lz) * gb.ey + (ay.i0 - gb.ly)) * gb.ex + (ax.i0 - gb.lx);
      const int off[8] = {0, 1, sy, sy + 1, sz, sz + 1, sz + sy, sz + sy + 1};
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        v0[k] = box[l + off[k]];
        v1[k] = box[cells + l + off[k]];
        v2[k] = box[2 * cells + l + off[k]];
      }
    } else if (!DETMAX) {
      const int base = (az.i0 * H + ay.i0) * W + ax.i0;
      load8(C, base, W, HW, v0);
      load8(C + V, base, W, HW, v1);
      load8(C + 2 * V, base, W, HW, v2);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) v0[k] = v1[k] = v2[k] = 0.f;
    }
    tri_grad(v0, az.t, ay.t, ax.t, dz, dy, dx);
    float jz = dz * g0, jy = dy * g0, jx = dx * g0;
    tri_grad(v1, az.t, ay.t, ax.t, dz, dy, dx);
    jz = fmaf(dz, g1, jz); jy = fmaf(dy, g1, jy); jx = fmaf(dx, g1, jx);
    tri_grad(v2, az.t, ay.t, ax.t, dz, dy, dx);
    jz = fmaf(dz, g2, jz); jy = fmaf(dy, g2, jy); jx = fmaf(dx, g2, jx);
    const float o0 = fmaf(az.live, jz, g0);
    const float o1 = fmaf(ay.live, jy, g1);
    const float o2 = fmaf(ax.live, jx, g2);
    if (DETMAX) {
      // reduce-only pass: no writes
    } else if (it.prev_atomic && !it.gc64) {
      gadd(gpv + p, o0);
      gadd(gpv + V + p, o1);
      gadd(gpv + 2 * V + p, o2);
    } else {
      gpv[p] += o0;
      gpv[V + p] += o1;
      gpv[2 * V + p] += o2;
    }
    sv[j].cz = az.i0; sv[j].cy = ay.i0; sv[j].cx = ax.i0;
    sv[j].tz = az.t; sv[j].ty = ay.t; sv[j].tx = ax.t;
    sv[j].g[0] = g0; sv[j].g[1] = g1; sv[j].g[2] = g2;
  }
  if (DETMAX) {
    det_bound<CB_NT>(sv, sred, it.js, it.det_slot);
    return;
  }
  DetOut det;
  if (it.gc64) {
    det.out64 = it.gc64;
    det.scale = det_scale(it.js, it.det_slot, it.det_blocks);
  }
  // with the box known, the scatter reduces only the magnitudes; the gathers
  // from acc end before its barrier, after which the bins are cleared
  scatter_tile<CB_NT, false>(sv, gp(it.gc), D, H, W, acc, sred, det, &gb);
}

// ---------------------------------------------------------------------------
// Deterministic mode: fold of a 64-bit fixed-point field into its float
// field (one pass over the elements, in no particular order: each element
// is independent), and the clearing of the jobs' slots.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_det_fold(const DetFoldItem* __restrict__ items,
                                                    int n_items, int n_tiles) {
  const int tile = blockIdx.x;
  const DetFoldItem it = items[find_item(items, n_items, tile)];
  if (it.flag && *it.flag == 0) return;
  const double sc = det_scale(it.js, it.det_slot, it.det_blocks);
  const double inv = sc > 0.0 ? 1.0 / sc : 0.0;
  const int e0 = (tile - it.tile0) * ELEM_PER_BLOCK;
  for (int k = threadIdx.x; k < ELEM_PER_BLOCK; k += BLOCK) {
    const int e = e0 + k;
    if (e >= it.n) break;
    const long long q = it.q[e];
    if (q == 0) continue;
    it.f[e] += (float)((double)q * inv);
    it.q[e] = 0;
  }
}

__global__ void k_det_clear(JobState* const* __restrict__ states, int n_jobs) {
  const int j = blockIdx.x;
  if (j >= n_jobs) return;
  for (int k = threadIdx.x; k < DET_SLOTS; k += blockDim.x) states[j]->det_max[k] = 0u;
}

// ---------------------------------------------------------------------------
// Window sums of the coefficients.  A block of TY x TX threads owns as many
// columns of the grid and walks a chunk of z.  For every input slice, the
// (TY + 2r) x (TX + 2r) patch around the columns goes to LDS, is summed over x
// there in segments of 8 outputs (a sliding sum from 8 + 2r values read once),
// and each thread then sums 2r + 1 of the x-sums along y for its own column.
// The sums over z need no subtraction and no moving ring: slices are taken in
// groups of w = 2r + 1, and a window that ends inside a group is the sum of
// that group so far plus a suffix sum of the group before, so a column keeps w
// values per quantity at fixed registers (the loop is unrolled over a group).
//
// The stages work on several slices at once (loading n + 3, storing n + 2,
// summing n + 1 over x, and n over y and z) in two buffers, with one barrier per
// slice.  Bound by memory (coefficients with their halo, field, images,
// gradient): 12 pairs of 160x192x160 at w 7 took 1040 us with z-sums of every
// patch column in a moving ring first, at three barriers per slice, and 660 like
// this.  The coefficients of a voxel lie together, so that a patch row of 38
// voxels touches five 128-byte lines where three planes made it nine: 582 us.
// ---------------------------------------------------------------------------
struct STile {
  int z0, z1, y0, x0;
};

template <int TY, int TX>
__device__ __forceinline__ STile stat_tile(int local, int D, int H, int W, int zc) {
  const int ntx = (W + TX - 1) / TX;
  const int nty = (H + TY - 1) / TY;
  STile t;
  t.x0 = (local % ntx) * TX;
  const int r = local / ntx;
  t.y0 = (r % nty) * TY;
  t.z0 = (r / nty) * zc;
  t.z1 = min(t.z0 + zc, D);
  return t;
}

template <int R, int TY, int TX>
struct Win {
  static constexpr int NT = TY * TX, WN = 2 * R + 1;
  static constexpr int PY = TY + 2 * R, PX = TX + 2 * R;
  static constexpr int PXS = PX | 1;              // odd: the rows a wave reads fall in distinct banks
  static constexpr int SITES = PY * PXS;          // patch slots, the odd padding included
  static constexpr int NS = (SITES + NT - 1) / NT;
  static constexpr int SLICE = NS * NT;           // floats of one loaded slice in LDS
  static constexpr int SEG = 8, NSEG = TX / SEG, XT = PY * NSEG;  // x-sum tasks of one quantity
  static constexpr int TXS = TX + 1, XQ = PY * TXS;
  static_assert(TX % SEG == 0, "tile not a multiple of the segments");
};

// Sliding sums of WN consecutive values of v, 8 of them, to d at a stride.
template <int WN, int STRIDE>
__device__ __forceinline__ void slide8(const float (&v)[7 + WN], float* __restrict__ d) {
  float acc = v[0];
#pragma unroll
  for (int k = 1; k < WN; ++k) acc += v[k];
  d[0] = acc;
#pragma unroll
  for (int i = 1; i < 8; ++i) {
    acc += v[i + WN - 1] - v[i - 1];
    d[i * STRIDE] = acc;
  }
}

// Sum over the last WN values of a column, v being value j of its group: ring
// holds, at j and above, the suffix sums of the group before, and below j the
// group's own values; pre is the group's sum so far.
template <int WN>
__device__ __forceinline__ float window_sum(float (&ring)[WN], float& pre, int j, float v) {
  pre = j == 0 ? v : pre + v;
  const float s = j + 1 < WN ? pre + ring[j + 1 < WN ? j + 1 : 0] : pre;
  ring[j] = v;
  if (j == WN - 1) {
#pragma unroll
    for (int k = WN - 2; k >= 0; --k) ring[k] += ring[k + 1];
  }
  return s;
}

// Warp of the source image by the pair field (Sec. 2.1): M(p) = I(p + U(p)),
// with the rigid adjustment of the source session added to U (Sec. 2.5).
template <class Items>
__global__ __launch_bounds__(BLOCK) void k_warp(const Items items, int n_tiles) {
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const SimItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W, HW = H * W, V = D * HW;
  const PTile tc = point_tile(tile - it.tile0, H, W);
  const cgfloat* __restrict__ I = gp(it.I);
  const cgfloat* __restrict__ U = gp(it.U);
  gfloat* __restrict__ M = gp(it.M);
  VoxSet vs;
  vox_set(tc, D, H, W, vs);
  float u[VPT][3];
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    u[j][0] = ldo(U, vs.p[j]);
    u[j][1] = ldo(U + V, vs.p[j]);
    u[j][2] = ldo(U + 2 * V, vs.p[j]);
  }
  if (it.rigid) {
    float rA[9], rO[3];
#pragma unroll
    for (int k = 0; k < 9; ++k) rA[k] = it.rigid->A[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) rO[k] = it.rigid->off[k];
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      const float fz = (float)vs.z[j], fy = (float)vs.y[j], fx = (float)vs.x[j];
#pragma unroll
      for (int c = 0; c < 3; ++c)
        u[j][c] += fmaf(rA[3 * c], fz, fmaf(rA[3 * c + 1], fy, fmaf(rA[3 * c + 2], fx, rO[c])));
    }
  }
  float v[VPT][8];
  Ax az[VPT], ay[VPT], ax[VPT];
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    az[j] = axis_disp(vs.z[j], u[j][0], D);
    ay[j] = axis_disp(vs.y[j], u[j][1], H);
    ax[j] = axis_disp(vs.x[j], u[j][2], W);
    load8(I, (az[j].i0 * H + ay[j].i0) * W + ax[j].i0, W, HW, v[j]);
  }
#pragma unroll
  for (int j = 0; j < VPT; ++j)
    if (vs.ok[j]) sto(M, vs.p[j], tri_val(v[j], az[j].t, ay[j].t, ax[j].t));
}

// Statistics of the windows (Sec. 2.6): LNCC / SiLNCC per window, the loss, and
// the adjoint's coefficients alpha, beta, gamma per window centre (0 where the
// window leaves the volume).  The images are shifted by one value per chunk of
// z before the products, which keeps the variance differences well conditioned.
//
// Where the images are flat those differences keep few digits, so the order of
// every sum is part of the result.  It is: per patch column, running sums over
// z of f, m, f^2, m^2 and f m, formed anew from the last w slices at the first
// window of a chunk and every w-th after; then sums over x and over y in
// segments of 8 that slide from the segment's start.  A block may take a part
// of a chunk: parts are multiples of w windows, so each starts where the sums
// are formed anew and the same values come out however the chunk is cut.
//
// Bound by vector issue and by the four barriers of a slice (z-sums written,
// x-sums written, finished sums written, finished sums read: sharing the z-sums'
// LDS costs the last).  The places of a thread's segments are worked out once, waves without a second patch column
// skip it, and the finished sums take the z-sums' LDS: three blocks of 16 x 32
// columns share a CU.  12 pairs of 160x192x160 at w 7: 600 -> 417 us.
template <int R, int TY, int TX>
struct Box {
  static constexpr int NT = TY * TX, WN = 2 * R + 1;
  static constexpr int PY = TY + 2 * R, PX = TX + 2 * R, P1 = PY * PX;
  static constexpr int NS = (P1 + NT - 1) / NT;   // patch columns per thread
  static constexpr int PXS = PX | 1, TXS = TX + 1;  // odd: a wave's rows fall in distinct banks
  static constexpr int SEG = 8, NXS = TX / SEG, NYS = TY / SEG;
  static constexpr int ZQ = PY * PXS, XQ = PY * TXS, YQ = TY * TX;
  static constexpr int XT = 5 * PY * NXS, XI = (XT + NT - 1) / NT;  // x tasks, and rounds of them
  static constexpr int YT = 5 * TX * NYS;
  static_assert(TX % SEG == 0 && TY % SEG == 0 && YT <= NT, "tile not a multiple of the segments");
};

template <int R, int TY, int TX, class Items>
__global__ __launch_bounds__(TY * TX) void k_sim_stats(const Items items, int n_tiles, int metric) {
  using B = Box<R, TY, TX>;
  constexpr int WN = B::WN, PX = B::PX, P1 = B::P1, NS = B::NS, NT = B::NT;
  __shared__ float zs[5 * (B::ZQ > B::YQ ? B::ZQ : B::YQ)];  // z-sums; then the finished sums
  __shared__ float xs[5 * B::XQ];
  __shared__ double red[NT / 64];
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const SimItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W, HW = H * W;
  // the block's columns, its chunk [c0, c1) and its part [z0, z1) of it
  const STile tc = stat_tile<TY, TX>(tile - it.tile0, D, H, W, 1);
  const int parts = (it.zc + it.zs - 1) / it.zs;
  const int chunk = tc.z0 / parts;
  const int c0 = chunk * it.zc, c1 = min(c0 + it.zc, D);
  const int z0 = c0 + (tc.z0 - chunk * parts) * it.zs, z1 = min(z0 + it.zs, c1);
  if (z0 >= z1) return;
  const cgfloat* __restrict__ F = gp(it.F);
  const cgfloat* __restrict__ M = gp(it.M);
  GLOBAL Coef* const cf = (GLOBAL Coef*)it.coef;
  const bool coef = it.coef != nullptr;
  const int pm = (min((c0 + c1) / 2, D - 1) * H + min(tc.y0 + TY / 2, H - 1)) * W +
                 min(tc.x0 + TX / 2, W - 1);
  const float sF = F[pm], sM = M[pm];
  const float inv_n = 1.f / (float)(WN * WN * WN);
  const int tid = threadIdx.x, ty = tid / TX, tx = tid % TX;
  const int y = tc.y0 + ty, x = tc.x0 + tx;
  const bool yx_in = (y < H) && (x < W);
  const bool yx_valid = yx_in && y >= R && y <= H - 1 - R && x >= R && x <= W - 1 - R;
  // owned patch columns: offset in a slice and place in the z-sum rows.  A
  // wave none of whose threads has a k-th column skips it.
  uint32_t cofs[NS];
  int zofs[NS];
  bool cval[NS], cin[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    const int col = tid + k * NT;
    const int row = col / PX, cx = col % PX;
    const int yy = tc.y0 - R + row, xx = tc.x0 - R + cx;
    cval[k] = col < P1;
    cin[k] = cval[k] && yy >= 0 && yy < H && xx >= 0 && xx < W;
    cofs[k] = cin[k] ? (uint32_t)(yy * W + xx) : 0u;
    zofs[k] = row * B::PXS + cx;
  }
  // values of slice z at the owned columns
  float fn[NS], mn[NS];
  auto load = [&](int z) {
    const uint32_t base = (uint32_t)(min(max(z, 0), D - 1) * HW);
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      if (!cval[k]) continue;
      fn[k] = ldo(F, base + cofs[k]);
      mn[k] = ldo(M, base + cofs[k]);
    }
  };
  // this thread's segments of the x and y sums
  int xsrc[B::XI], xdst[B::XI];
  bool xon[B::XI];
#pragma unroll
  for (int i = 0; i < B::XI; ++i) {
    const int e = tid + i * NT;
    const int q = e / (B::PY * B::NXS), r = e - q * (B::PY * B::NXS);
    const int row = r / B::NXS, seg = r - row * B::NXS;
    xon[i] = e < B::XT;
    xsrc[i] = q * B::ZQ + row * B::PXS + seg * B::SEG;
    xdst[i] = q * B::XQ + row * B::TXS + seg * B::SEG;
  }
  const bool yon = tid < B::YT;
  int ysrc, ydst;
  {
    const int q = tid / (TX * B::NYS), r = tid - q * (TX * B::NYS);
    const int seg = r / TX, sx = r - seg * TX;
    ysrc = q * B::XQ + seg * B::SEG * B::TXS + sx;
    ydst = q * B::YQ + seg * B::SEG * TX + sx;
  }
  float rf[NS][WN], rm[NS][WN], S[NS][5];
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    fn[k] = mn[k] = 0.f;
#pragma unroll
    for (int j = 0; j < WN; ++j) rf[k][j] = rm[k][j] = 0.f;
#pragma unroll
    for (int q = 0; q < 5; ++q) S[k][q] = 0.f;
  }
  load(z0 - R);
  int phase = 0;
  double lsum = 0.0;
  for (int zi = z0 - R; zi < z1 + R; ++zi) {
    const bool exact = ++phase == WN;
    if (exact) phase = 0;
    const bool zin = zi >= 0 && zi < D;
    float fv[NS], mv[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const bool in = zin && cin[k];
      fv[k] = in ? fn[k] - sF : 0.f;
      mv[k] = in ? mn[k] - sM : 0.f;
    }
    load(zi + 1);
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      if (!cval[k]) continue;
      const float fo = rf[k][0], mo = rm[k][0];
#pragma unroll
      for (int j = 0; j + 1 < WN; ++j) {
        rf[k][j] = rf[k][j + 1];
        rm[k][j] = rm[k][j + 1];
      }
      const float f = fv[k], m = mv[k];
      rf[k][WN - 1] = f;
      rm[k][WN - 1] = m;
      if (exact) {
        float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f, s4 = 0.f;
#pragma unroll
        for (int j = 0; j < WN; ++j) {
          s0 += rf[k][j];
          s1 += rm[k][j];
          s2 = fmaf(rf[k][j], rf[k][j], s2);
          s3 = fmaf(rm[k][j], rm[k][j], s3);
          s4 = fmaf(rf[k][j], rm[k][j], s4);
        }
        S[k][0] = s0; S[k][1] = s1; S[k][2] = s2; S[k][3] = s3; S[k][4] = s4;
      } else {
        S[k][0] += f - fo;
        S[k][1] += m - mo;
        S[k][2] += fmaf(f, f, -fo * fo);
        S[k][3] += fmaf(m, m, -mo * mo);
        S[k][4] += fmaf(f, m, -fo * mo);
      }
    }
    const int zcen = zi - R;
    if (zcen < z0) continue;
    const bool zvalid = zcen >= R && zcen <= D - 1 - R;
    if (zvalid) {
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (!cval[k]) continue;
#pragma unroll
        for (int q = 0; q < 5; ++q) zs[q * B::ZQ + zofs[k]] = S[k][q];
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < B::XI; ++i) {
        if (!xon[i]) continue;
        float v[7 + WN];
#pragma unroll
        for (int k = 0; k < 7 + WN; ++k) v[k] = zs[xsrc[i] + k];
        slide8<WN, 1>(v, xs + xdst[i]);
      }
      __syncthreads();
      if (yon) {
        float v[7 + WN];
#pragma unroll
        for (int k = 0; k < 7 + WN; ++k) v[k] = xs[ysrc + k * B::TXS];
        slide8<WN, TX>(v, zs + ydst);
      }
      __syncthreads();
    }
    if (yx_in) {
      float al = 0.f, be = 0.f, ga = 0.f;
      if (zvalid && yx_valid) {
        float Sw[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) Sw[q] = zs[q * B::YQ + tid];
        const float mF = Sw[0] * inv_n, mM = Sw[1] * inv_n;
        const float vFr = Sw[2] * inv_n - mF * mF;
        const float vMr = Sw[3] * inv_n - mM * mM;
        const float c = Sw[4] * inv_n - mF * mM;
        const float vF = fmaxf(vFr, 0.f), vM = fmaxf(vMr, 0.f);
        float l, av, ac;
        if (metric == 0) {
          const float den = vF * vM;
          if (den > EPS_LNCC) {
            const float sd = sqrtf(den);
            l = 1.f - c / sd;
            ac = -1.f / sd;
            av = c / (2.f * vM * sd);
          } else {
            const float sd = sqrtf(EPS_LNCC);
            l = 1.f - c / sd;
            ac = -1.f / sd;
            av = 0.f;
          }
        } else {
          const float dd = fmaxf(vF, EPS_SILNCC);
          l = vM - c * c / dd;
          ac = -2.f * c / dd;
          av = 1.f;
        }
        if (!(vMr > 0.f)) av = 0.f;
        lsum += (double)l;
        const float mFt = mF + sF, mMt = mM + sM;
        al = -(2.f * mMt * av + mFt * ac) * inv_n;
        be = av * inv_n;
        ga = ac * inv_n;
      }
      if (coef) {
        sto_coef(cf + (size_t)zcen * HW, (uint32_t)(y * W + x), Coef{al, be, ga});
      }
    }
    if (zvalid) __syncthreads();  // zs is written again next
  }
  const double tot = block_sum<NT>(lsum, red);
  if (tid == 0) {
    const double v = tot * it.inv_nr;
    if (it.js) unsafeAtomicAdd(&it.js->loss_sim, v);
    if (it.sim_out) unsafeAtomicAdd(it.sim_out, v);
  }
}

// Gradient of Sim with respect to the pair field:
//   dSim/dM(y) = (Box alpha + 2 M Box beta + F Box gamma)(y) / N_R,
//   dSim/dU(y) = dSim/dM(y) * grad I_j(y + U(y)).
// The window sums of the coefficients are formed like those of k_sim_stats.
// The field at an output voxel is loaded two slices ahead of its use, the
// corners of the cell it samples one slice ahead.
template <int R, int TY, int TX, class Items>
__global__ __launch_bounds__(TY * TX) void k_sim_grad(const Items items, int n_tiles) {
  using B = Win<R, TY, TX>;
  constexpr int NT = B::NT, NS = B::NS, WN = B::WN, XT = B::XT, XQ = B::XQ;
  static_assert(3 * XT <= NT, "one x-sum task per thread");
  __shared__ float raw[2][3][B::SLICE];
  __shared__ float xs[2][3 * XQ];
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const SimItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W, HW = H * W, V = D * HW;
  const STile tc = stat_tile<TY, TX>(tile - it.tile0, D, H, W, it.zg);
  const cgfloat* __restrict__ F = gp(it.F);
  const cgfloat* __restrict__ I = gp(it.I);
  const Planes<const cgfloat> Up(gp(it.U), V);
  const GLOBAL Coef* const cf = (const GLOBAL Coef*)it.coef;
  const Planes<gfloat> gU(gp(it.gU), V);
  const float inv_nr = (float)it.inv_nr;
  const int tid = threadIdx.x, ty = tid / TX, tx = tid % TX;
  const int y = min(tc.y0 + ty, H - 1), x = min(tc.x0 + tx, W - 1);
  const bool yx_in = tc.y0 + ty < H && tc.x0 + tx < W;
  const uint32_t off = (uint32_t)(y * W + x);
  uint32_t soff[NS];
  bool sin[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    const int i = tid + k * NT, row = i / B::PXS, col = i - row * B::PXS;
    const int yy = tc.y0 - R + row, xx = tc.x0 - R + col;
    sin[k] = yy >= 0 && yy < H && xx >= 0 && xx < W;
    soff[k] = sin[k] ? (uint32_t)(yy * W + xx) : 0u;
  }
  float cv[3][NS];  // coefficients off the grid are 0
#pragma unroll
  for (int k = 0; k < NS; ++k) cv[0][k] = cv[1][k] = cv[2][k] = 0.f;
  auto load = [&](int z) {
    const GLOBAL Coef* const plane = cf + (size_t)min(max(z, 0), D - 1) * HW;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      if (!sin[k]) continue;
      const Coef v = ldo_coef(plane, soff[k]);
      cv[0][k] = v.a;
      cv[1][k] = v.b;
      cv[2][k] = v.c;
    }
  };
  auto put = [&](int b) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int k = 0; k < NS; ++k) raw[b][q][tid + k * NT] = cv[q][k];
  };
  const bool xt = tid < 3 * XT;
  const int xq = xt ? tid / XT : 0, xr = xt ? tid - xq * XT : 0;
  const int xrow = xr / B::NSEG, xseg = (xr - xrow * B::NSEG) * B::SEG;
  const int xsrc = xq * B::SLICE + xrow * B::PXS + xseg,
            xdst = xq * XQ + xrow * B::TXS + xseg;
  auto sum_x = [&](int b) {
    if (!xt) return;
    const float* s = &raw[b][0][0] + xsrc;
    float v[7 + WN];
#pragma unroll
    for (int k = 0; k < 7 + WN; ++k) v[k] = s[k];
    slide8<WN, 1>(v, xs[b] + xdst);
  };
  float rA[9], rO[3];
  const bool rigid = it.rigid != nullptr;
  if (rigid) {
#pragma unroll
    for (int k = 0; k < 9; ++k) rA[k] = it.rigid->A[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) rO[k] = it.rigid->off[k];
  }
  float u[3];  // U at the own column, of the output after next's preparation
  auto load_u = [&](int z) {
    const uint32_t p = (uint32_t)(min(z, D - 1) * HW) + off;
#pragma unroll
    for (int c = 0; c < 3; ++c) u[c] = ldo(Up.c[c], p);
  };
  const int zb = tc.z0 - R, total = tc.z1 - tc.z0 + 2 * R;
  load(zb);
  put(0);
  load(zb + 1);
  load_u(tc.z0);
  __syncthreads();
  sum_x(0);
  put(1);
  load(zb + 2);
  __syncthreads();
  float ring[3][WN], pre[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    pre[q] = 0.f;
#pragma unroll
    for (int k = 0; k < WN; ++k) ring[q][k] = 0.f;
  }
  float vI[8], fo = 0.f;   // corners of I and F of the next output
  Ax az{}, ay{}, ax{};
#pragma unroll
  for (int k = 0; k < 8; ++k) vI[k] = 0.f;
  bool more = true;
  for (int n0 = 0; more; n0 += WN) {
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const int n = n0 + j;
      if (n >= total) {
        more = false;
        break;
      }
      const int zi = zb + n, zo = zi - R;
      const bool zin = zi >= 0 && zi < D;  // slices off the grid hold zeros
      put(n & 1);
      load(zi + 3);
      float S[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const float* s = xs[n & 1] + q * XQ + ty * B::TXS + tx;
        float v = s[0];
#pragma unroll
        for (int k = 1; k < WN; ++k) v += s[k * B::TXS];
        S[q] = window_sum<WN>(ring[q], pre[q], j, zin ? v : 0.f);
      }
      if (zo >= tc.z0 && yx_in) {
        float dz, dy, dx;
        const float M = tri_grad(vI, az.t, ay.t, ax.t, dz, dy, dx);
        const float dM = (S[0] + 2.f * M * S[1] + fo * S[2]) * inv_nr;
        const uint32_t p = (uint32_t)(zo * HW) + off;
        sto(gU.c[0], p, dM * dz * az.live);
        sto(gU.c[1], p, dM * dy * ay.live);
        sto(gU.c[2], p, dM * dx * ax.live);
      }
      if (zo + 1 >= tc.z0 && zo + 1 < tc.z1) {
        const int zn = zo + 1;
        if (rigid) {
          const float fz = (float)zn, fy = (float)y, fx = (float)x;
#pragma unroll
          for (int c = 0; c < 3; ++c)
            u[c] += fmaf(rA[3 * c], fz, fmaf(rA[3 * c + 1], fy, fmaf(rA[3 * c + 2], fx, rO[c])));
        }
        az = axis_disp(zn, u[0], D);
        ay = axis_disp(y, u[1], H);
        ax = axis_disp(x, u[2], W);
        load8(I, (az.i0 * H + ay.i0) * W + ax.i0, W, HW, vI);
        fo = ldo(F, (uint32_t)(zn * HW) + off);
        load_u(zn + 1);
      }
      sum_x((n + 1) & 1);
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// Adam (PyTorch semantics) with the warm-up + cosine schedule (Sec. 2.7),
// or the scaled gradient (mode 1).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double schedule_lr(const JobState* js, int step) {
  const int T = js->T, Wu = js->W;
  if (step <= Wu) return (double)js->lr0 * step / (double)Wu;
  if (T == Wu) return (double)js->lr0;
  return (double)js->lr0 * 0.5 * (1.0 + cos(M_PI * (double)(step - Wu) / (double)(T - Wu)));
}

__global__ __launch_bounds__(BLOCK) void k_adam(const AdamItem* __restrict__ items, int n_items,
                                                int n_tiles) {
  const int tile = blockIdx.x;
  const AdamItem it = items[find_item(items, n_items, tile)];
  const int n = it.n;
  const int q0 = (tile - it.tile0) * ELEM_PER_BLOCK;
  const cgfloat* __restrict__ gs = gp(it.gsrc);
  if (it.mode != 0) {
    gfloat* __restrict__ go = gp(it.gout);
    for (int k = threadIdx.x; k < ELEM_PER_BLOCK; k += BLOCK) {
      const int q = q0 + k;
      if (q >= n) break;
#pragma unroll
      for (int c = 0; c < 3; ++c) go[c * n + q] = gs[c * n + q] * it.gscale;
    }
    return;
  }
  const JobState* js = it.js;
  const int step = js->t + 1;
  const double lr = schedule_lr(js, step);
  const double bc1 = 1.0 - pow((double)js->b1, (double)step);
  const double bc2 = 1.0 - pow((double)js->b2, (double)step);
  const float step_size = (float)(lr / bc1);
  const float bc2s = (float)sqrt(bc2);
  const float b1 = js->b1, b2 = js->b2, eps = js->eps;
  gfloat* __restrict__ phi = gp(it.phi);
  gfloat* __restrict__ mm = gp(it.m);
  gfloat* __restrict__ vv = gp(it.v);
  for (int k = threadIdx.x; k < ELEM_PER_BLOCK; k += BLOCK) {
    const int q = q0 + k;
    if (q >= n) break;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const int i = c * n + q;
      const float g = gs[i];
      float m = mm[i], v = vv[i];
      m = fmaf(1.f - b1, g - m, m);
      v = fmaf(1.f - b2, g * g, v * b2);
      const float den = sqrtf(v) / bc2s + eps;
      phi[i] -= step_size * (m / den);
      mm[i] = m;
      vv[i] = v;
    }
  }
}

// ---------------------------------------------------------------------------
// Gaussian smoothing of the flow (Sec. 2.4, Appendix A): one separable pass of
// the periodic filter along one axis, on the three components.  Appendix A
// applies the Gaussian transfer function in the Fourier domain; its spatial
// form on a periodic line is a circular convolution whose taps the host
// computes from that transfer function (out to where they vanish below float
// rounding, or over the whole line), so one pass per axis applies the whole
// 3-D filter.  The taps are symmetric, so the same pass is its own adjoint.
// ---------------------------------------------------------------------------
// SMOOTH_S consecutive outputs of the convolution of a line held in LDS with
// the taps w: line is the first sample the first output reaches, ls the
// samples' stride, m the samples that the eight reach.  Every sample feeds each
// output (taps outside 0..2r are zero), so an output sums its taps in the order
// k = 0..2r.  The samples are read in groups of SMOOTH_S and the rest one by one:
// one beyond the m would make the outputs NaN if it is not finite.
__device__ __forceinline__ void smooth_chunk(const float* line, int ls, int m,
                                             const float* __restrict__ w,
                                             float (&acc)[SMOOTH_S]) {
#pragma unroll
  for (int o = 0; o < SMOOTH_S; ++o) acc[o] = 0.f;
  int j = 0;
  for (; j + SMOOTH_S <= m; j += SMOOTH_S) {
    float v[SMOOTH_S];
#pragma unroll
    for (int k = 0; k < SMOOTH_S; ++k) v[k] = line[(j + k) * ls];
    const float* t = w + SMOOTH_WPAD + j;
#pragma unroll
    for (int k = 0; k < SMOOTH_S; ++k)
#pragma unroll
      for (int o = 0; o < SMOOTH_S; ++o) acc[o] = fmaf(t[k - o], v[k], acc[o]);
  }
  for (; j < m; ++j) {
    const float v = line[j * ls];
#pragma unroll
    for (int o = 0; o < SMOOTH_S; ++o) acc[o] = fmaf(w[SMOOTH_WPAD + j - o], v, acc[o]);
  }
}

// Position of staged sample e on a periodic line of n, r samples being staged
// ahead of it.
__device__ __forceinline__ int smooth_wrap(int e, int r, int n) {
  int p = e - r;
  while (p < 0) p += n;
  while (p >= n) p -= n;
  return p;
}

// One pass of the separable periodic Gaussian with the item's taps.  A block
// stages whole lines of one component in LDS, with the samples that the ends
// reach round the period, so every sample is read from HBM once and written
// once and the sums run over consecutive samples.  Bound by vector issue: 8
// fused multiply-adds per sample read from LDS, taps in scalar registers; the
// staging costs few instructions (direct loads, positions that step), where
// working out every sample's position took more than the sums.  15 million
// voxels at sigma 3: z and y 200 -> 139 us, x 161 -> 118 us (24 bytes per voxel
// at 2.6 and 3.0 TB/s).
__global__ __launch_bounds__(BLOCK) void k_smooth(const SmoothItem* __restrict__ items, int n_items,
                                                  int n_tiles) {
  extern __shared__ float lds[];
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const SmoothItem& it = items[find_item(items, n_items, tile)];
  const int D = it.D, H = it.H, W = it.W;
  const int V = D * H * W;
  const int local = tile - it.tile0;
  const int comp = local / it.tiles_comp;
  const int t = local - comp * it.tiles_comp;
  const cgfloat* __restrict__ src = gp(it.src) + comp * V;
  gfloat* __restrict__ dst = gp(it.dst) + comp * V;
  const int r = it.radius, L = it.lines, ls = it.lshift;
  const int m = 2 * r + SMOOTH_S;  // samples of a chunk
  if (it.axis < 2) {
    // lines along z (axis 0) or y (axis 1); the tile is L adjacent x columns
    const int n = it.axis == 0 ? D : H;
    const int stride = it.axis == 0 ? H * W : W;
    const int nxc = (W + L - 1) >> ls;
    const int outer = t / nxc;
    const int x0 = (t - outer * nxc) << ls;
    const int width = min(L, W - x0);
    const int base = (it.axis == 0 ? outer * W : outer * H * W) + x0;
    const int chunks = (n + SMOOTH_S - 1) / SMOOTH_S;
    // straight into LDS; a thread's column stays, its position steps along the
    // line and round the period
    const int total = (chunks * SMOOTH_S - SMOOTH_S + m) << ls;
    {
      const int c = threadIdx.x & (L - 1);
      int step = BLOCK >> ls;
      while (step >= n) step -= n;
      int p = smooth_wrap(threadIdx.x >> ls, r, n);
      uint32_t off = (uint32_t)(base + p * stride + c);
      const uint32_t dstep = (uint32_t)(step * stride), dline = (uint32_t)(n * stride);
      for (int e = threadIdx.x; e < total; e += BLOCK) {
        if (c < width) ld_to_lds(src + off, lds + (e & ~63));
        p += step;
        off += dstep;
        if (p >= n) {
          p -= n;
          off -= dline;
        }
      }
    }
    __syncthreads();
    const int c = threadIdx.x & (L - 1);
    if (c < width) {
      for (int q = threadIdx.x >> ls; q < chunks; q += BLOCK >> ls) {
        const int p0 = q * SMOOTH_S;
        float acc[SMOOTH_S];
        smooth_chunk(lds + (p0 << ls) + c, L, m, it.w, acc);
#pragma unroll
        for (int o = 0; o < SMOOTH_S; ++o)
          if (p0 + o < n) dst[base + (p0 + o) * stride + c] = acc[o];
      }
    }
  } else {
    // lines along x: the tile is L consecutive rows, staged with an odd row
    // pitch so lanes on different rows hit different banks; the outputs go out
    // through LDS in whole rows
    const int Wp = W | 1;
    const int chunks = (W + SMOOTH_S - 1) / SMOOTH_S;
    const int Ws = chunks * SMOOTH_S - SMOOTH_S + m, Wsp = Ws | 1;
    const int row0 = t << ls;
    const int rows = min(L, D * H - row0);
    const cgfloat* __restrict__ tsrc = src + row0 * W;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int col = lane; col < Ws; col += 64) {
      uint32_t off = (uint32_t)(wave * W + smooth_wrap(col, r, W));
      float* to = lds + wave * Wsp + (col & ~63);
      for (int row = wave; row < rows; row += BLOCK / 64) {
        ld_to_lds(tsrc + off, to);
        off += (BLOCK / 64) * W;
        to += (BLOCK / 64) * Wsp;
      }
    }
    __syncthreads();
    // at most SMOOTH_XR chunks per thread (smooth_item_setup); their outputs
    // take the samples' place in LDS
    const int rr = threadIdx.x & (L - 1);
    float acc[SMOOTH_XR][SMOOTH_S];
#pragma unroll
    for (int i = 0; i < SMOOTH_XR; ++i) {
      const int q = (threadIdx.x + i * BLOCK) >> ls;
      if (rr < rows && q < chunks) smooth_chunk(lds + rr * Wsp + q * SMOOTH_S, 1, m, it.w, acc[i]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SMOOTH_XR; ++i) {
      const int p0 = ((threadIdx.x + i * BLOCK) >> ls) * SMOOTH_S;
      if (rr >= rows) continue;
#pragma unroll
      for (int o = 0; o < SMOOTH_S; ++o)
        if (p0 + o < W) lds[rr * Wp + p0 + o] = acc[i][o];
    }
    __syncthreads();
    gfloat* __restrict__ tdst = dst + row0 * W;
    for (int row = wave; row < rows; row += BLOCK / 64)
      for (int col = lane; col < W; col += 64) sto(tdst, (uint32_t)(row * W + col), lds[row * Wp + col]);
  }
}

__global__ void k_finish(JobState* const* __restrict__ states, int n_jobs) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_jobs) return;
  JobState* js = states[i];
  const double L = js->loss_sim + slot_sum(js->loss_reg);
  const int h = js->hist_base + js->t;
  if (js->history && h >= 0 && h < js->hist_len) js->history[h] = L;
  if (!isfinite(L)) js->nonfinite = 1;
  js->loss_sim = 0.0;
  for (int k = 0; k < LOSS_SLOTS; ++k) js->loss_reg[k * LOSS_STRIDE] = 0.0;
  for (int k = 0; k < js->n_flags; ++k) js->flags[k] = 0;
  js->t += 1;
}

// ---------------------------------------------------------------------------
// Pyramid (Sec. 2.7)
// ---------------------------------------------------------------------------
template <class Items>
__global__ __launch_bounds__(BLOCK) void k_pool2(const Items items, int n_tiles) {
  const int tile = blockIdx.x;
  const PoolItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W;
  const int D2 = D / 2, H2 = H / 2, W2 = W / 2;
  const int n = D2 * H2 * W2;
  const int q0 = (tile - it.tile0) * ELEM_PER_BLOCK;
  for (int k = threadIdx.x; k < ELEM_PER_BLOCK; k += BLOCK) {
    const int q = q0 + k;
    if (q >= n) break;
    const int X = q % W2, Y = (q / W2) % H2, Z = q / (W2 * H2);
    const float* s = it.src + ((2 * Z) * H + 2 * Y) * W + 2 * X;
    const int HW = H * W;
    const float a = (s[0] + s[1]) + (s[W] + s[W + 1]);
    const float b = (s[HW] + s[HW + 1]) + (s[HW + W] + s[HW + W + 1]);
    it.dst[q] = (a + b) * 0.125f;
  }
}

// A block stages the coarse cells behind a tile of UF_TZ x UF_TY x UF_TX fine
// voxels (t/2 + 2 per axis, three components, coordinates clamped to the
// grid) in LDS; every fine voxel then reads its 8 corners from there.
template <class Items>
__global__ __launch_bounds__(BLOCK) void k_upsample2(const Items items, int n_tiles) {
  constexpr int CZ = UF_TZ / 2 + 2, CY = UF_TY / 2 + 2, CX = UF_TX / 2 + 2, CN = CZ * CY * CX;
  constexpr int PER = UF_TZ * UF_TY * UF_TX / BLOCK;
  static_assert(UF_TY * UF_TX == BLOCK, "one fine slice of the tile per thread pass");
  __shared__ float cs[3 * CN];
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const UpItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W, HW = H * W, V = D * HW;
  const int D2 = 2 * D, H2 = 2 * H, W2 = 2 * W;
  const int n = D2 * H2 * W2;
  const int local = tile - it.tile0;
  const int ntx = (W2 + UF_TX - 1) / UF_TX, nty = (H2 + UF_TY - 1) / UF_TY;
  const int fx0 = (local % ntx) * UF_TX, fy0 = ((local / ntx) % nty) * UF_TY,
            fz0 = (local / ntx / nty) * UF_TZ;
  // first staged coarse cell per axis: the floor cell of the tile's first
  // fine sample, (f0 - 0.5) / 2 = f0 / 2 - 0.25
  const int cz0 = fz0 / 2 - 1, cy0 = fy0 / 2 - 1, cx0 = fx0 / 2 - 1;
  const cgfloat* __restrict__ src = gp(it.src);
  for (int i = threadIdx.x; i < 3 * CN; i += BLOCK) {
    const int c = i / CN, r = i - c * CN;
    const int lz = r / (CY * CX), r2 = r - lz * (CY * CX), ly = r2 / CX, lx = r2 - ly * CX;
    const int z = min(max(cz0 + lz, 0), D - 1), y = min(max(cy0 + ly, 0), H - 1),
              x = min(max(cx0 + lx, 0), W - 1);
    cs[i] = src[c * V + (z * H + y) * W + x];
  }
  __syncthreads();
  const int fy = fy0 + threadIdx.x / UF_TX, fx = fx0 + threadIdx.x % UF_TX;
  const Ax ay = axis_pos(((float)fy - 0.5f) * 0.5f, H), ax = axis_pos(((float)fx - 0.5f) * 0.5f, W);
  gfloat* __restrict__ dst = gp(it.dst);
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int fz = fz0 + j;
    if (fz >= D2 || fy >= H2 || fx >= W2) continue;
    const Ax az = axis_pos(((float)fz - 0.5f) * 0.5f, D);
    const int base = ((az.i0 - cz0) * CY + (ay.i0 - cy0)) * CX + (ax.i0 - cx0);
    const int q = (fz * H2 + fy) * W2 + fx;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float* p = cs + c * CN + base;
      const float v[8] = {p[0], p[1], p[CX], p[CX + 1],
                          p[CY * CX], p[CY * CX + 1], p[CY * CX + CX], p[CY * CX + CX + 1]};
      dst[c * n + q] = 2.f * tri_val(v, az.t, ay.t, ax.t);
    }
  }
}

// Adjoint of k_upsample2 (flow grid -> image grid, values doubled): each
// coarse voxel gathers, with weight 2 w, the fine voxels whose sample cell has
// it as a corner.  Along an axis those are the fine indices 2c-1 .. 2c+2; the
// weight is evaluated with the forward's own clamp and cell rules, so borders
// match it exactly.  A gather, so no atomics and a fixed summation order.
__device__ __forceinline__ float up_weight(int f, int c, int n) {
  const Ax a = axis_pos(((float)f - 0.5f) * 0.5f, n);
  return c == a.i0 ? 1.f - a.t : (c == a.i0 + 1 ? a.t : 0.f);
}

// The weights are separable, so a block stages the fine region behind a tile
// of UA_TZ x UA_TY x UA_TX coarse voxels (2t + 2 fine samples per axis) in
// LDS, one component at a time, and sums along x, then y, then z, with the
// 4 weights per coarse index of each axis computed once per block: every fine
// sample is read from HBM once and the 64-tap gather becomes 3 x 4 taps.  A
// thread stages whole columns of the region (one offset each, where every
// sample's position was worked out from its index): 96x128x112 coarse voxels
// 76 -> 60 us, against 149 MB moved.
template <class Items>
__global__ __launch_bounds__(BLOCK) void k_upsample2_adj(const Items items, int n_tiles) {
  constexpr int FZ = 2 * UA_TZ + 2, FY = 2 * UA_TY + 2, FX = 2 * UA_TX + 2;
  constexpr int FN = FZ * FY * FX;           // fine region; later the y sums
  constexpr int S1 = FZ * FY * UA_TX;        // x sums
  constexpr int S2 = FZ * UA_TY * UA_TX;     // y sums
  constexpr int TN = UA_TZ * UA_TY * UA_TX;  // outputs
  static_assert(S2 <= FN, "the y sums reuse the fine region");
  __shared__ float fine[FN];
  __shared__ float s1[S1];
  __shared__ float wz[UA_TZ][4], wy[UA_TY][4], wx[UA_TX][4];
  const int tile = xcd_remap(blockIdx.x, n_tiles);
  const UpItem it = items.at(tile);
  const int D = it.D, H = it.H, W = it.W, V = D * H * W;
  const int D2 = 2 * D, H2 = 2 * H, W2 = 2 * W, n2 = 8 * V;
  const int local = tile - it.tile0;
  const int ntx = (W + UA_TX - 1) / UA_TX, nty = (H + UA_TY - 1) / UA_TY;
  const int cx0 = (local % ntx) * UA_TX, cy0 = ((local / ntx) % nty) * UA_TY,
            cz0 = (local / ntx / nty) * UA_TZ;
  // fine index of the first staged sample along each axis: 2 c0 - 1
  const int fz0 = 2 * cz0 - 1, fy0 = 2 * cy0 - 1, fx0 = 2 * cx0 - 1;
  // w[o][k]: weight of fine 2(c0 + o) - 1 + k for coarse c0 + o (0 off the grid)
  auto weight = [](int f, int c, int n) { return (f >= 0 && f < 2 * n) ? up_weight(f, c, n) : 0.f; };
  for (int i = threadIdx.x; i < (UA_TZ + UA_TY + UA_TX) * 4; i += BLOCK) {
    const int o = i / 4, k = i % 4;
    if (o < UA_TZ) {
      wz[o][k] = weight(fz0 + 2 * o + k, cz0 + o, D);
    } else if (o < UA_TZ + UA_TY) {
      const int q = o - UA_TZ;
      wy[q][k] = weight(fy0 + 2 * q + k, cy0 + q, H);
    } else {
      const int q = o - UA_TZ - UA_TY;
      wx[q][k] = weight(fx0 + 2 * q + k, cx0 + q, W);
    }
  }
  const cgfloat* __restrict__ g = gp(it.src);
  gfloat* __restrict__ out = gp(it.dst);
  // the columns of the fine region that this thread stages
  constexpr int NC = (FY * FX + BLOCK - 1) / BLOCK;
  uint32_t off[NC];
  bool col[NC], in[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int q = threadIdx.x + k * BLOCK, ly = q / FX, lx = q - ly * FX;
    const int fy = fy0 + ly, fx = fx0 + lx;
    col[k] = q < FY * FX;
    in[k] = col[k] && fy >= 0 && fy < H2 && fx >= 0 && fx < W2;
    off[k] = in[k] ? (uint32_t)(fy * W2 + fx) : 0u;
  }
  for (int c = 0; c < 3; ++c) {
    // a column of the region per thread and round, all its planes in flight
    // before they land in LDS
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      if (!col[k]) continue;
      float v[FZ];
#pragma unroll
      for (int lz = 0; lz < FZ; ++lz) {
        const int fz = fz0 + lz;
        v[lz] = in[k] && fz >= 0 && fz < D2 ? ldo(g + c * n2, (uint32_t)(fz * (H2 * W2)) + off[k]) : 0.f;
      }
#pragma unroll
      for (int lz = 0; lz < FZ; ++lz) fine[lz * (FY * FX) + threadIdx.x + k * BLOCK] = v[lz];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < S1; i += BLOCK) {
      const int row = i / UA_TX, ox = i - row * UA_TX;
      const float* f = fine + row * FX + 2 * ox;
      s1[i] = fmaf(wx[ox][3], f[3], fmaf(wx[ox][2], f[2], fmaf(wx[ox][1], f[1], wx[ox][0] * f[0])));
    }
    __syncthreads();
    float* s2 = fine;
    for (int i = threadIdx.x; i < S2; i += BLOCK) {
      const int lz = i / (UA_TY * UA_TX), r = i - lz * (UA_TY * UA_TX);
      const int oy = r / UA_TX, ox = r - oy * UA_TX;
      const float* f = s1 + (lz * FY + 2 * oy) * UA_TX + ox;
      s2[i] = fmaf(wy[oy][3], f[3 * UA_TX],
                   fmaf(wy[oy][2], f[2 * UA_TX], fmaf(wy[oy][1], f[UA_TX], wy[oy][0] * f[0])));
    }
    __syncthreads();
    for (int i = threadIdx.x; i < TN; i += BLOCK) {
      const int oz = i / (UA_TY * UA_TX), r = i - oz * (UA_TY * UA_TX);
      const int oy = r / UA_TX, ox = r - oy * UA_TX;
      const int z = cz0 + oz, y = cy0 + oy, x = cx0 + ox;
      if (z >= D || y >= H || x >= W) continue;
      const float* f = s2 + (2 * oz) * (UA_TY * UA_TX) + oy * UA_TX + ox;
      constexpr int SZ = UA_TY * UA_TX;
      const float v = fmaf(wz[oz][3], f[3 * SZ],
                           fmaf(wz[oz][2], f[2 * SZ], fmaf(wz[oz][1], f[SZ], wz[oz][0] * f[0])));
      out[c * V + (z * H + y) * W + x] = 2.f * v;
    }
    __syncthreads();  // before the next component overwrites the fine region
  }
}

// ---------------------------------------------------------------------------
// Single-step helpers for the unit entry points
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(BLOCK) void k_adam_flat(int64_t n, float* x, const float* g, float* m,
                                                     float* v, float step_size, float bc2s,
                                                     float b1, float b2, float eps) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i >= n) return;
  const float gg = g[i];
  float mm = m[i], vv = v[i];
  mm = fmaf(1.f - b1, gg - mm, mm);
  vv = fmaf(1.f - b2, gg * gg, vv * b2);
  const float den = sqrtf(vv) / bc2s + eps;
  x[i] -= step_size * (mm / den);
  m[i] = mm;
  v[i] = vv;
}

__global__ void k_fill(float* p, int64_t n, float v) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Optional start / stop events of the next launches on this thread (the
// runtime's kernel timing): recorded by the launch packet itself, so a timed
// launch costs one API call and the events bracket the kernel alone.
static thread_local hipEvent_t t_launch_start = nullptr, t_launch_stop = nullptr;

void set_launch_events(hipEvent_t start, hipEvent_t stop) {
  t_launch_start = start;
  t_launch_stop = stop;
}

#define MUSTER_LAUNCH(kernel, grid, block, shm, stream, ...)                                  \
  do {                                                                                         \
    if (t_launch_start)                                                                        \
      hipExtLaunchKernelGGL(kernel, grid, block, shm, stream, t_launch_start, t_launch_stop, 0, \
                            __VA_ARGS__);                                                      \
    else                                                                                       \
      hipLaunchKernelGGL(kernel, grid, block, shm, stream, __VA_ARGS__);                      \
  } while (0)

template <class Items>
static hipError_t exp_fwd_(const Items& items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_exp_fwd<Items>, dim3(n_tiles), dim3(MT_NT), 0, s, items, n_tiles);
  return hipGetLastError();
}

template <class Items>
static hipError_t compose_fwd_(const Items& items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_compose_fwd<Items>, dim3(n_tiles), dim3(BLOCK), 0, s, items, n_tiles);
  return hipGetLastError();
}

// Marks per block of k_exp_far: a launch is about as many blocks as walk at
// once (97 to 110 VGPRs: four per CU), up to the 64 marks that one load of a wave
// holds.  With eight marks per block, side by side, 28800 unset ones took 6.9
// us against 4.9, half a million 142 against 26, and the adjoint of a
// 160x192x160 field of up to 8 voxels 971 us against 949.
template <bool DETMAX, class Items>
static hipError_t exp_far_(const Items& items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  const int group = std::min(64, std::max(1, n_tiles / 1024));
  MUSTER_LAUNCH((k_exp_far<DETMAX, Items>), dim3(ceil_div(n_tiles, group)), dim3(BLOCK), 0, s, items,
                n_tiles, group);
  return hipGetLastError();
}

template <class Items>
static hipError_t exp_bwd_(const Items& items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_exp_bwd<Items>, dim3(n_tiles), dim3(MT_NT), 0, s, items, n_tiles);
  return hipGetLastError();
}

template <class Items>
static hipError_t combine_(const Items& items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_combine<Items>, dim3(n_tiles), dim3(CT_Y * CT_X), 0, s, items, n_tiles);
  return hipGetLastError();
}

template <bool DETMAX, class Items>
static hipError_t compose_bwd_(const Items& items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH((k_compose_bwd<DETMAX, Items>), dim3(n_tiles), dim3(CB_NT), 0, s, items, n_tiles);
  return hipGetLastError();
}

hipError_t launch_det_fold(const DetFoldItem* items, int n_items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_det_fold, dim3(n_tiles), dim3(BLOCK), 0, s, items, n_items, n_tiles);
  return hipGetLastError();
}

hipError_t launch_det_clear(JobState* const* states, int n_jobs, hipStream_t s) {
  if (n_jobs <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_det_clear, dim3(n_jobs), dim3(64), 0, s, states, n_jobs);
  return hipGetLastError();
}

template <int R, int TY, int TX, class Items>
static void sim_launch(bool grad, const Items& items, int n_tiles, int metric, hipStream_t s) {
  if (grad)
    MUSTER_LAUNCH((k_sim_grad<R, TY, TX, Items>), dim3(n_tiles), dim3(TY * TX), 0, s, items, n_tiles);
  else
    MUSTER_LAUNCH((k_sim_stats<R, TY, TX, Items>), dim3(n_tiles), dim3(TY * TX), 0, s, items, n_tiles,
                  metric);
}

template <int R, class Items>
static hipError_t sim_shape(bool grad, const Items& items, int n_tiles, int metric, int shape,
                            hipStream_t s) {
  switch (shape) {
    case 0: sim_launch<R, 8, 32>(grad, items, n_tiles, metric, s); break;
    case 1: sim_launch<R, 16, 32>(grad, items, n_tiles, metric, s); break;
    case 2: sim_launch<R, 8, 64>(grad, items, n_tiles, metric, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class Items>
static hipError_t sim_window(bool grad, const Items& items, int n_tiles, int window, int metric,
                             int shape, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  switch (window) {
    case 3: return sim_shape<1>(grad, items, n_tiles, metric, shape, s);
    case 5: return sim_shape<2>(grad, items, n_tiles, metric, shape, s);
    case 7: return sim_shape<3>(grad, items, n_tiles, metric, shape, s);
    default: return hipErrorInvalidValue;
  }
}

template <class Items>
static hipError_t warp_(const Items& items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_warp<Items>, dim3(n_tiles), dim3(BLOCK), 0, s, items, n_tiles);
  return hipGetLastError();
}

template <class Items>
static hipError_t pool2_(const Items& items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_pool2<Items>, dim3(n_tiles), dim3(BLOCK), 0, s, items, n_tiles);
  return hipGetLastError();
}

template <class Items>
static hipError_t upsample2_(const Items& items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_upsample2<Items>, dim3(n_tiles), dim3(BLOCK), 0, s, items, n_tiles);
  return hipGetLastError();
}

template <class Items>
static hipError_t upsample2_adj_(const Items& items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_upsample2_adj<Items>, dim3(n_tiles), dim3(BLOCK), 0, s, items, n_tiles);
  return hipGetLastError();
}

// Each launcher for a table of items in device memory, and for one item that
// travels with the launch.
#define MUSTER_BOTH(name, Item, call)                                                              \
  hipError_t launch_##name(const Item* items, int n_items, int n_tiles, hipStream_t s) {           \
    return call(Table<Item>{items, n_items}, n_tiles, s);                                          \
  }                                                                                                \
  hipError_t launch_##name(const Item& one, int n_tiles, hipStream_t s) {                          \
    return call(One<Item>{one}, n_tiles, s);                                                       \
  }
MUSTER_BOTH(exp_fwd, ExpFwdItem, exp_fwd_)
MUSTER_BOTH(compose_fwd, ComposeItem, compose_fwd_)
MUSTER_BOTH(exp_bwd, ExpBwdItem, exp_bwd_)
MUSTER_BOTH(exp_far, ExpBwdItem, exp_far_<false>)
MUSTER_BOTH(combine, CombineItem, combine_)
MUSTER_BOTH(compose_bwd, ComposeBwdItem, compose_bwd_<false>)
MUSTER_BOTH(warp, SimItem, warp_)
MUSTER_BOTH(pool2, PoolItem, pool2_)
MUSTER_BOTH(upsample2, UpItem, upsample2_)
MUSTER_BOTH(upsample2_adj, UpItem, upsample2_adj_)
#undef MUSTER_BOTH

hipError_t launch_exp_far_detmax(const ExpBwdItem* items, int n_items, int n_tiles, hipStream_t s) {
  return exp_far_<true>(Table<ExpBwdItem>{items, n_items}, n_tiles, s);
}

hipError_t launch_compose_bwd_detmax(const ComposeBwdItem* items, int n_items, int n_tiles,
                                     hipStream_t s) {
  return compose_bwd_<true>(Table<ComposeBwdItem>{items, n_items}, n_tiles, s);
}

hipError_t launch_sim_stats(const SimItem* items, int n_items, int n_tiles, int window, int metric,
                            int shape, hipStream_t s) {
  return sim_window(false, Table<SimItem>{items, n_items}, n_tiles, window, metric, shape, s);
}

hipError_t launch_sim_stats(const SimItem& one, int n_tiles, int window, int metric, int shape,
                            hipStream_t s) {
  return sim_window(false, One<SimItem>{one}, n_tiles, window, metric, shape, s);
}

hipError_t launch_sim_grad(const SimItem* items, int n_items, int n_tiles, int window, int shape,
                           hipStream_t s) {
  return sim_window(true, Table<SimItem>{items, n_items}, n_tiles, window, 0, shape, s);
}

hipError_t launch_sim_grad(const SimItem& one, int n_tiles, int window, int shape, hipStream_t s) {
  return sim_window(true, One<SimItem>{one}, n_tiles, window, 0, shape, s);
}

hipError_t launch_adam(const AdamItem* items, int n_items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_adam, dim3(n_tiles), dim3(BLOCK), 0, s, items, n_items, n_tiles);
  return hipGetLastError();
}

hipError_t launch_smooth(const SmoothItem* items, int n_items, int n_tiles, int lds_floats,
                         hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  if (lds_floats <= 0 || lds_floats > SMOOTH_LDS) return hipErrorInvalidValue;
  MUSTER_LAUNCH(k_smooth, dim3(n_tiles), dim3(BLOCK), lds_floats * sizeof(float), s, items,
                     n_items, n_tiles);
  return hipGetLastError();
}

__global__ void k_pattern(float* __restrict__ p, int64_t n, int D, int H, int W, float off,
                          float amp, float phase) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t V = (int64_t)D * H * W;
  const int c = (int)(i / V);
  const int q = (int)(i - c * V);
  const int x = q % W, y = (q / W) % H, z = q / (W * H);
  p[i] = off + amp * sinf(0.21f * x + 0.13f * y + 0.17f * z + phase + 1.7f * c) *
                   cosf(0.05f * x - 0.09f * z + phase);
}

hipError_t launch_pattern(float* p, int64_t n, const int dims[3], float off, float amp,
                          float phase, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_pattern, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, dims[0],
                     dims[1], dims[2], off, amp, phase);
  return hipGetLastError();
}

hipError_t launch_finish(JobState* const* states, int n_jobs, hipStream_t s) {
  if (n_jobs <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_finish, dim3(ceil_div(n_jobs, 64)), dim3(64), 0, s, states, n_jobs);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Outputs and evaluation (Sec. 2.8): Jacobian determinants of Omega + U, and
// the sums from which Eu, the vector PCC and the regression slope follow.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float fd_axis(const cgfloat* __restrict__ f, int p, int i, int n,
                                         int stride) {
  // central difference inside, one-sided at the two faces
  if (i == 0) return f[p + stride] - f[p];
  if (i == n - 1) return f[p] - f[p - stride];
  return 0.5f * (f[p + stride] - f[p - stride]);
}

__global__ __launch_bounds__(BLOCK) void k_jacobian_det(GridDims d, const float* __restrict__ U_,
                                                        float* __restrict__ out) {
  const int D = d.D, H = d.H, W = d.W, HW = H * W, V = D * HW;
  const cgfloat* __restrict__ U = gp(U_);
  for (int p = blockIdx.x * BLOCK + threadIdx.x; p < V; p += gridDim.x * BLOCK) {
    const int x = p % W, y = (p / W) % H, z = p / HW;
    float J[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const cgfloat* __restrict__ f = U + (size_t)c * V;
      J[c][0] = fd_axis(f, p, z, D, HW) + (c == 0 ? 1.f : 0.f);
      J[c][1] = fd_axis(f, p, y, H, W) + (c == 1 ? 1.f : 0.f);
      J[c][2] = fd_axis(f, p, x, W, 1) + (c == 2 ? 1.f : 0.f);
    }
    gp(out)[p] = J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) -
                 J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
                 J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
  }
}

// Sums over the region of interest (roi may be NULL: every voxel): count,
// sum |b - a|, sum a (3), sum b (3), sum a a^T (9), sum b a^T (9), sum b.b.
constexpr int FIELD_STATS = 27;

__global__ __launch_bounds__(BLOCK) void k_field_stats(int V, const float* __restrict__ a_,
                                                       const float* __restrict__ b_,
                                                       const unsigned char* __restrict__ roi,
                                                       double* __restrict__ out) {
  __shared__ double red[BLOCK / 64];
  const cgfloat* __restrict__ a = gp(a_);
  const cgfloat* __restrict__ b = gp(b_);
  double acc[FIELD_STATS];
#pragma unroll
  for (int k = 0; k < FIELD_STATS; ++k) acc[k] = 0.0;
  for (int p = blockIdx.x * BLOCK + threadIdx.x; p < V; p += gridDim.x * BLOCK) {
    if (roi && !roi[p]) continue;
    double av[3], bv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      av[c] = a[(size_t)c * V + p];
      bv[c] = b[(size_t)c * V + p];
    }
    acc[0] += 1.0;
    acc[1] += sqrt((bv[0] - av[0]) * (bv[0] - av[0]) + (bv[1] - av[1]) * (bv[1] - av[1]) +
                   (bv[2] - av[2]) * (bv[2] - av[2]));
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      acc[2 + c] += av[c];
      acc[5 + c] += bv[c];
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        acc[8 + 3 * c + e] += av[c] * av[e];
        acc[17 + 3 * c + e] += bv[c] * av[e];
      }
    }
    acc[26] += bv[0] * bv[0] + bv[1] * bv[1] + bv[2] * bv[2];
  }
#pragma unroll
  for (int k = 0; k < FIELD_STATS; ++k) {
    const double t = block_sum(acc[k], red);
    if (threadIdx.x == 0) unsafeAtomicAdd(out + k, t);
    __syncthreads();
  }
}

hipError_t launch_jacobian_det(GridDims d, const float* U, float* out, hipStream_t s) {
  const int V = d.D * d.H * d.W;
  if (V <= 0) return hipSuccess;
  const int blocks = ceil_div(V, BLOCK) < 4096 ? ceil_div(V, BLOCK) : 4096;
  MUSTER_LAUNCH(k_jacobian_det, dim3(blocks), dim3(BLOCK), 0, s, d, U, out);
  return hipGetLastError();
}

hipError_t launch_field_stats(int V, const float* a, const float* b, const unsigned char* roi,
                              double* out, hipStream_t s) {
  if (V <= 0) return hipSuccess;
  const int blocks = ceil_div(V, BLOCK) < 1024 ? ceil_div(V, BLOCK) : 1024;
  MUSTER_LAUNCH(k_field_stats, dim3(blocks), dim3(BLOCK), 0, s, V, a, b, roi, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Rigid adjustment (Sec. 2.5)
// ---------------------------------------------------------------------------
// sum_p G(p) and sum_p G(p) (p - c)^T over one pair's gradient, into the
// source session's accumulators.
__global__ __launch_bounds__(BLOCK) void k_rigid_grad(const RigidGradItem* __restrict__ items,
                                                      int n_items, int n_tiles) {
  __shared__ double red[BLOCK / 64][12];
  const int tile = blockIdx.x;
  const RigidGradItem it = items[find_item(items, n_items, tile)];
  const int D = it.D, H = it.H, W = it.W, V = D * H * W;
  const float cz = 0.5f * (D - 1), cy = 0.5f * (H - 1), cx = 0.5f * (W - 1);
  const cgfloat* __restrict__ G = gp(it.G);
  double acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = 0.0;
  const int q0 = (tile - it.tile0) * ELEM_PER_BLOCK;
  for (int k = threadIdx.x; k < ELEM_PER_BLOCK; k += BLOCK) {
    const int q = q0 + k;
    if (q >= V) break;
    const int x = q % W, y = (q / W) % H, z = q / (W * H);
    const double pz = (double)z - cz, py = (double)y - cy, px = (double)x - cx;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double g = G[(size_t)c * V + q];
      acc[c] += g;
      acc[3 + 3 * c] += g * pz;
      acc[4 + 3 * c] += g * py;
      acc[5 + 3 * c] += g * px;
    }
  }
#pragma unroll
  for (int k = 0; k < 12; ++k)
    for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o);
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < 12; ++k) red[threadIdx.x >> 6][k] = acc[k];
  __syncthreads();
  if (threadIdx.x < 12) {
    double t = 0.0;
    for (int w = 0; w < BLOCK / 64; ++w) t += red[w][threadIdx.x];
    double* dst = threadIdx.x < 3 ? &it.rg->gsum[threadIdx.x] : &it.rg->gmom[threadIdx.x - 3];
    unsafeAtomicAdd(dst, t);
  }
}

// One Adam step of a session's rigid parameters (PyTorch semantics, the
// job's schedule; the angles' step scaled by rot_lr), then the displacement
// the kernels apply, and the sums cleared for the next iteration.
__global__ void k_rigid_step(const RigidStepItem* __restrict__ items, int n_items) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_items) return;
  const RigidStepItem it = items[i];
  RigidState* rg = it.rg;
  const JobState* js = it.js;
  const int step = js->t + 1;
  const double lr = schedule_lr(js, step);
  const double bc1 = 1.0 - pow((double)js->b1, (double)step);
  const double bc2 = 1.0 - pow((double)js->b2, (double)step);
  float g[6];
  for (int k = 0; k < 3; ++k) {
    float dR[9];
    rigid_rotation(rg->theta, k, dR);
    double acc = 0.0;
    for (int e = 0; e < 9; ++e) acc += (double)dR[e] * rg->gmom[e];
    g[k] = (float)acc;
    g[3 + k] = (float)rg->gsum[k];
  }
  const float b1 = js->b1, b2 = js->b2, eps = js->eps;
  float prm[6] = {rg->theta[0], rg->theta[1], rg->theta[2], rg->t[0], rg->t[1], rg->t[2]};
  for (int k = 0; k < 6; ++k) {
    const float m = fmaf(1.f - b1, g[k] - rg->m[k], rg->m[k]);
    const float v = fmaf(1.f - b2, g[k] * g[k], rg->v[k] * b2);
    rg->m[k] = m;
    rg->v[k] = v;
    const float scale = k < 3 ? it.rot_lr : 1.f;
    const float den = sqrtf(v) / (float)sqrt(bc2) + eps;
    prm[k] -= (float)(lr * scale / bc1) * (m / den);
  }
  for (int k = 0; k < 3; ++k) {
    rg->theta[k] = prm[k];
    rg->t[k] = prm[3 + k];
  }
  float R[9];
  rigid_rotation(rg->theta, -1, R);
  for (int a = 0; a < 3; ++a) {
    float rc = 0.f;
    for (int b = 0; b < 3; ++b) {
      rg->A[3 * a + b] = R[3 * a + b] - (a == b ? 1.f : 0.f);
      rc += R[3 * a + b] * it.c[b];
    }
    rg->off[a] = it.c[a] + rg->t[a] - rc;
  }
  for (int k = 0; k < 3; ++k) rg->gsum[k] = 0.0;
  for (int k = 0; k < 9; ++k) rg->gmom[k] = 0.0;
}

__global__ __launch_bounds__(BLOCK) void k_add_rigid(GridDims d, float* __restrict__ f_,
                                                     const RigidState* __restrict__ rg) {
  const int V = d.D * d.H * d.W;
  gfloat* __restrict__ f = gp(f_);
  for (int p = blockIdx.x * BLOCK + threadIdx.x; p < V; p += gridDim.x * BLOCK) {
    const float x = (float)(p % d.W), y = (float)((p / d.W) % d.H), z = (float)(p / (d.W * d.H));
#pragma unroll
    for (int c = 0; c < 3; ++c)
      f[(size_t)c * V + p] += fmaf(rg->A[3 * c], z, fmaf(rg->A[3 * c + 1], y,
                                                         fmaf(rg->A[3 * c + 2], x, rg->off[c])));
  }
}

hipError_t launch_rigid_grad(const RigidGradItem* items, int n_items, int n_tiles, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_rigid_grad, dim3(n_tiles), dim3(BLOCK), 0, s, items, n_items, n_tiles);
  return hipGetLastError();
}

hipError_t launch_rigid_step(const RigidStepItem* items, int n_items, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  MUSTER_LAUNCH(k_rigid_step, dim3(ceil_div(n_items, 64)), dim3(64), 0, s, items, n_items);
  return hipGetLastError();
}

hipError_t launch_add_rigid(GridDims d, float* field, const RigidState* rg, hipStream_t s) {
  const int V = d.D * d.H * d.W;
  if (V <= 0) return hipSuccess;
  const int blocks = ceil_div(V, BLOCK) < 2048 ? ceil_div(V, BLOCK) : 2048;
  MUSTER_LAUNCH(k_add_rigid, dim3(blocks), dim3(BLOCK), 0, s, d, field, rg);
  return hipGetLastError();
}

hipError_t launch_adam_flat(int64_t n, float* x, const float* g, float* m, float* v, int t,
                            float lr, float b1, float b2, float eps, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const double bc1 = 1.0 - std::pow((double)b1, (double)t);
  const double bc2 = 1.0 - std::pow((double)b2, (double)t);
  const float step_size = (float)(lr / bc1);
  const float bc2s = (float)std::sqrt(bc2);
  const int64_t blocks = (n + BLOCK - 1) / BLOCK;
  MUSTER_LAUNCH(k_adam_flat, dim3((unsigned)blocks), dim3(BLOCK), 0, s, n, x, g, m, v,
                     step_size, bc2s, b1, b2, eps);
  return hipGetLastError();
}

// Scratch of the allocation-free similarity entry point (see
// NOALLOC_SCRATCH_BYTES).  Host code never passes the array's name to a
// kernel or a copy: only the address hipGetSymbolAddress returns for the
// current device.
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch_address(int device, void** ptr) {
  static std::mutex mu;
  static std::map<int, void*> addr;
  std::lock_guard<std::mutex> lk(mu);
  auto it = addr.find(device);
  if (it != addr.end()) {
    *ptr = it->second;
    return hipSuccess;
  }
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (!p) return hipErrorInvalidSymbol;
  addr.emplace(device, p);
  *ptr = p;
  return hipSuccess;
}

hipError_t launch_fill(float* p, int64_t n, float v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + BLOCK - 1) / BLOCK;
  MUSTER_LAUNCH(k_fill, dim3((unsigned)blocks), dim3(BLOCK), 0, s, p, n, v);
  return hipGetLastError();
}

}  // namespace muster
