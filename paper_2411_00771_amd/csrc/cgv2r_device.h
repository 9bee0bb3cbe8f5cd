// Device-side helpers shared by the gfx950 kernels of the surfel rasterizer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/cgv2r.h"
#include "reach.h"

namespace cgv2 {

constexpr int kTile = CGV2_TILE;
constexpr int kRec = CGV2_REC_FLOATS;
constexpr int kGradFields = 19;  // per-surfel, per-view record gradients accumulated by render_bwd

// record field offsets
enum : int {
  R_CXH = 0, R_CYH, R_CXL, R_CYL, R_A11, R_A12, R_A21, R_A22, R_W0, R_W1, R_W2,
  R_ZC, R_OP, R_R, R_G, R_B, R_NX, R_NY, R_NZ, R_K2, R_PXR, R_PYR
};

// record-gradient fields accumulated by the reverse pass; the first 16 are the slots of its wave
// reduce-scatter
enum : int {
  G_CX = 0, G_CY, G_A11, G_A12, G_A21, G_A22, G_W0, G_W1, G_W2, G_OP, G_R, G_G, G_B, G_SCX, G_SCY, G_ZC,
  G_NX, G_NY, G_NZ
};

// Record gradients in the backward workspace.  Fields G_CX..G_ZC of (view v, surfel i) form one 64-B
// row row[(v n + i) 16 + f], so the 16 atomics a wave issues for a (surfel, tile) fall in one cache
// line; the normal fields follow all views' rows as 16-B rows nrm[(v n + i) 4 + c] (c < 3).
constexpr int kGradRow = 16;
constexpr int kGradNrm = 4;
struct RecGrads {
  float* row;
  float* nrm;
};

constexpr float kAlphaMin = 1.0f / 255.0f;
constexpr float kAlphaMax = 0.99f;
constexpr float kTmin = 1e-4f;
constexpr float kNegHalfLog2e = -0.72134752044448170368f;  // -0.5 / ln 2

struct DevCam {
  int W, H;
  float fx, fy, cx, cy, R[9], t[3], znear, bg[3];
};

// Cameras travel as kernel arguments (the library allocates nothing): up to kMaxViews per launch,
// views [v0, v0 + count) of the call.
constexpr int kMaxViews = 32;
struct CamPack {
  DevCam c[kMaxViews];
  int v0, count;
};

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// DPP move (gfx9 encodings); lanes of rows outside kRowMask receive 0.
template <int kCtrl, int kRowMask = 0xf>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, kRowMask, 0xf, false));
}

// Sum over the 64 lanes of a wave with DPP row operations only (no LDS traffic); the total is
// valid in lane 63.
__device__ __forceinline__ float wave_sum_lane63(float v) {
  v += dpp<0xB1>(v);        // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);        // quad_perm [2,3,0,1]
  v += dpp<0x141>(v);       // row_half_mirror: 4-lane groups -> 8
  v += dpp<0x140>(v);       // row_mirror: 8 -> 16 (every lane holds its row's sum)
  v += dpp<0x142, 0xa>(v);  // row_bcast:15 -> rows 1 and 3 add rows 0 and 2
  v += dpp<0x143, 0xc>(v);  // row_bcast:31 -> rows 2 and 3 add rows 0+1
  return v;
}

// Reduce-scatter of 16 per-lane values over a wave: on return every lane holds the wave total of
// value index reduce16_index(lane).  Lane bits 3 and 2 go first, with DPP adds whose bank masks write only
// the lanes that keep a value (two instructions per pair, no select); bits 5 and 4 with the row-swap
// instructions (x' + y' after a swap is already the pairwise sum of the kept half), on the three pairs that
// are left; the quads are summed last.  The row swaps issue slower than DPP adds: with bits 5 and 4 first
// (twelve swaps, 35 instead of 33 instructions) k_render_bwd took 349 us against 334 (1 M surfels, 1600x1066)
// and 4991 against 4718 (10 M, 8 views).  The DPP adds are one asm block because the compiler does not form
// them under a bank mask; its first s_nop separates them from the writes of their sources, its last from the
// swaps, and inside it no source is written less than two instructions before.
__device__ __forceinline__ int reduce16_index(int lane) {
  return ((lane >> 4) & 1) | (((lane >> 5) & 1) << 1) | (((lane >> 2) & 1) << 2) | (((lane >> 3) & 1) << 3);
}

__device__ __forceinline__ float reduce16_scatter(float (&v)[16]) {
  asm("s_nop 1\n"
      "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %3, %3, %3 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %4, %4, %4 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %5, %5, %5 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %6, %6, %6 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %7, %7, %7 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %0, %8, %8 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %1, %9, %9 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %2, %10, %10 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %3, %11, %11 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %4, %12, %12 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %5, %13, %13 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %6, %14, %14 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %7, %15, %15 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n"
      "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0x5\n"
      "v_add_f32_dpp %2, %2, %2 row_half_mirror row_mask:0xf bank_mask:0x5\n"
      "v_add_f32_dpp %3, %3, %3 row_half_mirror row_mask:0xf bank_mask:0x5\n"
      "v_add_f32_dpp %0, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xa\n"
      "v_add_f32_dpp %1, %5, %5 row_half_mirror row_mask:0xf bank_mask:0xa\n"
      "v_add_f32_dpp %2, %6, %6 row_half_mirror row_mask:0xf bank_mask:0xa\n"
      "v_add_f32_dpp %3, %7, %7 row_half_mirror row_mask:0xf bank_mask:0xa\n"
      "s_nop 1"
      : "+&v"(v[0]), "+&v"(v[1]), "+&v"(v[2]), "+&v"(v[3]), "+&v"(v[4]), "+&v"(v[5]), "+&v"(v[6]), "+&v"(v[7])
      : "v"(v[8]), "v"(v[9]), "v"(v[10]), "v"(v[11]), "v"(v[12]), "v"(v[13]), "v"(v[14]), "v"(v[15]));
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[j]), __float_as_uint(v[j + 2]), false, false);
    v[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[0]), __float_as_uint(v[1]), false, false);
  float t = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  t += dpp<0xB1>(t);  // quad_perm [1,0,3,2]
  t += dpp<0x4E>(t);  // quad_perm [2,3,0,1]
  return t;
}

// As reduce16_scatter, but over the sixteen lanes of equal lane % 4: on return every lane holds, for its lane % 4, the
// total of value reduce16_index(lane).  Lane bits 3 and 2 by DPP adds that keep the place in the quad.
__device__ __forceinline__ float reduce16_scatter_quads(float (&v)[16]) {
  asm("s_nop 1\n"
      "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %3, %3, %3 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %4, %4, %4 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %5, %5, %5 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %6, %6, %6 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %7, %7, %7 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %0, %8, %8 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %1, %9, %9 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %2, %10, %10 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %3, %11, %11 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %4, %12, %12 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %5, %13, %13 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %6, %14, %14 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %7, %15, %15 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "v_add_f32_dpp %0, %0, %0 row_shl:4 row_mask:0xf bank_mask:0x5\n"
      "v_add_f32_dpp %1, %1, %1 row_shl:4 row_mask:0xf bank_mask:0x5\n"
      "v_add_f32_dpp %2, %2, %2 row_shl:4 row_mask:0xf bank_mask:0x5\n"
      "v_add_f32_dpp %3, %3, %3 row_shl:4 row_mask:0xf bank_mask:0x5\n"
      "v_add_f32_dpp %0, %4, %4 row_shr:4 row_mask:0xf bank_mask:0xa\n"
      "v_add_f32_dpp %1, %5, %5 row_shr:4 row_mask:0xf bank_mask:0xa\n"
      "v_add_f32_dpp %2, %6, %6 row_shr:4 row_mask:0xf bank_mask:0xa\n"
      "v_add_f32_dpp %3, %7, %7 row_shr:4 row_mask:0xf bank_mask:0xa\n"
      "s_nop 1"
      : "+&v"(v[0]), "+&v"(v[1]), "+&v"(v[2]), "+&v"(v[3]), "+&v"(v[4]), "+&v"(v[5]), "+&v"(v[6]), "+&v"(v[7])
      : "v"(v[8]), "v"(v[9]), "v"(v[10]), "v"(v[11]), "v"(v[12]), "v"(v[13]), "v"(v[14]), "v"(v[15]));
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[j]), __float_as_uint(v[j + 2]), false, false);
    v[j] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[0]), __float_as_uint(v[1]), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sum over the sixteen lanes of equal lane % 4, in all of them.
__device__ __forceinline__ float sum_quads(float x) {
  x += dpp<0x128>(x);  // row_ror:8
  x += dpp<0x124>(x);  // row_ror:4
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// The same for three values: on return lanes with (lane & 12) == 0 hold the wave total of a, (lane & 4) that of
// b, (lane & 12) == 8 that of c.  11 operations against 18 for three separate sums.
__device__ __forceinline__ float reduce3_scatter(float a, float b, float c) {
  asm("s_nop 1\n"
      "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n"
      "v_add_f32_dpp %1, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n"
      "v_add_f32_dpp %0, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xc\n"
      "s_nop 1\n"
      "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n"
      "v_add_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xa\n"
      "s_nop 1"
      : "+&v"(a), "+&v"(b)
      : "v"(c));
  a += dpp<0xB1>(a);  // quad_perm [1,0,3,2]
  a += dpp<0x4E>(a);  // quad_perm [2,3,0,1]
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(a), false, false);
  a = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(a), false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

template <typename T>
__global__ __launch_bounds__(256) void k_fill(T* p, int64_t count, T v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// Zeroes count elements of a and of b (either may be null) in one launch.
template <typename T>
__global__ __launch_bounds__(256) void k_zero2(T* a, T* b, int64_t count) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) {
    if (a) a[i] = T(0);
    if (b) b[i] = T(0);
  }
}

// Exclusive scan over a workgroup of kThreads threads (a multiple of 64); lds holds kThreads / 64
// values; 'total' receives the workgroup sum.  Every thread of the workgroup must call it.
template <int kThreads, typename T>
__device__ __forceinline__ T block_exscan(T v, T* lds, T& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  T x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const T y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) lds[w] = x;
  __syncthreads();
  T off = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kThreads / 64; ++k) {
    if (k < w) off += lds[k];
    tot += lds[k];
  }
  __syncthreads();
  total = tot;
  return off + x - v;
}

// Block -> tile mapping.  Hardware dispatches workgroup b to XCD b % 8.  Here XCD x receives the
// runs of kXcdChunk consecutive tiles with run index = x (mod 8): neighbouring tiles of a run share
// that XCD's L2, while the runs of every XCD are spread over the whole image.  (Giving each XCD one
// contiguous band instead leaves the XCD with the densest band -- the far field of an oblique view --
// with up to twice the mean work.)  Blocks past the last full round of 8 runs map to themselves.
constexpr uint32_t kXcdChunk = 4;
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t nb) {
  const uint32_t span = 8u * kXcdChunk;
  const uint32_t full = nb - nb % span;
  if (b >= full) return b;
  const uint32_t x = b % 8u, k = b / 8u;  // XCD and the block's rank on it
  return (x + 8u * (k / kXcdChunk)) * kXcdChunk + k % kXcdChunk;
}

}  // namespace cgv2
