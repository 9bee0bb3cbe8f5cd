// Photometric loss of CityGaussianV2 Sec. 3.1: L = (1 - lambda) L1 + lambda (1 - SSIM), with the
// SSIM-only part of the gradient kept apart as the source of the decomposed densification
// gradient (Sec. 3.2, Eq. 2).
//
// SSIM (Wang et al. 2004): 11x11 separable Gaussian window (sigma 1.5), zero padding,
// C1 = 0.01^2, C2 = 0.03^2.  Both kernels run one wave per strip of 64 columns of one image plane and walk
// down the strip: each input row (the 64 columns and a 5-column halo on either side) goes through LDS once,
// its 11-tap horizontal sums enter a ring of the last 11 rows held in registers, and each new row completes
// the vertical sums of one output row -- the only recomputation is the 10-row halo at the strip's top.  The
// forward kernel sums four moments (x, y, x^2 + y^2, xy: SSIM needs the variances only added up), formed once
// per pixel on the way into LDS, and computes the SSIM map and its three partial derivatives (w.r.t. the
// local mean, E[x^2] and E[xy]) and deterministic per-wave sums; the backward kernel correlates the three
// partial maps with the same window and combines them with the L1 sign into dL/dI and
// d(lambda (1 - SSIM))/dI.
//
// Both are bound by vector instructions and LDS reads (and, where a SIMD holds a single wave, by the latency of
// a row's chain): a launch takes as long as the SIMD with the most rows, see strip_grid().
#include "cgv2r_device.h"
#include "cgv2r_kernels.h"

#include <algorithm>

namespace cgv2 {

constexpr int kR = 5;
constexpr int kTaps = 2 * kR + 1;       // 11
constexpr int kStripW = 64;             // output columns per wave (one per lane)
constexpr int kRowW = kStripW + 2 * kR;
constexpr float kC1 = 0.0001f, kC2 = 0.0009f;
// The moments of a strip are taken about mid-grey or about zero, whichever is nearer to the middle of its values:
// the variances do not change, and least cancels in them (see strip_mid).
constexpr float kMid = 0.5f;

struct Win { float g[kTaps]; };

// Block -> (strip column, strip row, plane vc = v * 3 + channel).
struct StripGrid {
  int nx, ny, rows;  // strips per plane across and down, output rows per strip
};

// Hardware sends workgroup b to XCD b % 8: XCD x takes the x-th contiguous eighth of the strips (row-major
// over strip columns, then strip rows, then planes), so the halo columns and rows that neighbouring
// strips share are fetched into one L2.  Blocks past the last full round of 8 map to themselves.
// Returns the strip index (the slot of its per-wave sums).
__device__ __forceinline__ int strip_of_block(const StripGrid& sg, int& x0, int& y0, int& vc) {
  const uint32_t nb = gridDim.x, full = nb - nb % 8u, bb = blockIdx.x;
  const int b = (int)(bb < full ? (bb % 8u) * (full / 8u) + bb / 8u : bb);
  const int r = b / sg.nx;
  x0 = (b - r * sg.nx) * kStripW;
  y0 = (r % sg.ny) * sg.rows;
  vc = r / sg.ny;
  return b;
}

// Orders a wave's own LDS writes and reads (the workgroup is that one wave, and a wave's LDS operations
// execute in program order): a compiler barrier only.  __syncthreads() would also wait for every
// outstanding global store of the wave, putting the output rows' store latency on the row loop.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_sched_barrier(0);  // also keeps the scheduler from hoisting later rows' loads (registers)
  __builtin_amdgcn_wave_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Loads and stores through buffer resources: an offset past the plane's end (kDrop) reads 0 (the zero
// padding of the window) and drops a store (an output outside the image), so the row loop has no
// branches and its only waits are for the loads of the row it is about to use, not for earlier stores.
constexpr uint32_t kDrop = 0xfffffff0u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const float* base, int64_t floats) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, (int)(floats * 4), 0x00020000);
}
__device__ __forceinline__ float load_or_zero(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, 0));
}
__device__ __forceinline__ void store_or_drop(__amdgpu_buffer_rsrc_t r, float v, uint32_t byte_off) {
  // the builtin stores a 32-bit integer: pass the float's bits, not its value
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, byte_off, 0, 0);
}

// Byte offsets of row yy at columns x0 - 5 + lane (a) and x0 + 59 + lane for lane < 10 (b), kDrop
// outside the image.
__device__ __forceinline__ void row_offsets(int W, int H, int x0, int yy, int lane, uint32_t& a,
                                            uint32_t& b) {
  const bool row = yy >= 0 && yy < H;
  const int c0 = x0 - kR + lane, c1 = x0 - kR + kStripW + lane;
  a = (row && c0 >= 0 && c0 < W) ? (uint32_t)((int64_t)yy * W + c0) * 4u : kDrop;
  b = (row && lane < 2 * kR && c1 < W) ? (uint32_t)((int64_t)yy * W + c1) * 4u : kDrop;
}

// Vertical sum of ring slot values for the output whose newest input row sits in slot j (oldest first).
template <int N, int J>
__device__ __forceinline__ void vsum(const float (&ring)[kTaps][N], const Win& win, float (&o)[N]) {
#pragma unroll
  for (int q = 0; q < N; ++q) o[q] = 0.f;
#pragma unroll
  for (int b = 0; b < kTaps; ++b) {
    const int k = (J + 1 + b) % kTaps;
#pragma unroll
    for (int q = 0; q < N; ++q) o[q] = fmaf(win.g[b], ring[k][q], o[q]);
  }
}

// The value that the strip's moments are taken about, from both images at four rows spread over its output rows.
// What cancels grows with the square of the distance of the values from it.  Relative error of the SSIM gradient
// against float64 on smooth images in [0, 1] / [0.45, 0.55] / [0, 0.2] / [0, 0.004] and a photograph-like one: about
// mid-grey 3.3e-6 / 2.0e-5 / 1.3e-5 / 3.7e-5 and 3.6e-5, about zero 1.1e-5 / 2.8e-5 / 2.0e-6 / 3.1e-7 and 9.0e-5,
// chosen per strip the smaller of the two in each.
struct StripSample {
  float x[4], y[4];
};

__device__ __forceinline__ void sample_load(StripSample& q, __amdgpu_buffer_rsrc_t rx, __amdgpu_buffer_rsrc_t ry,
                                            int W, int H, int x0, int y0, int rows, int lane) {
  const int col = min(x0 + lane, W - 1), last = min(rows, H - y0) - 1;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t off = (uint32_t)((int64_t)(y0 + last * k / 3) * W + col) * 4u;
    q.x[k] = load_or_zero(rx, off);
    q.y[k] = load_or_zero(ry, off);
  }
}

__device__ __forceinline__ float strip_mid(const StripSample& q) {
  float lo = INFINITY, hi = -INFINITY;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    lo = fminf(lo, fminf(q.x[k], q.y[k]));
    hi = fmaxf(hi, fmaxf(q.x[k], q.y[k]));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = fminf(lo, __shfl_xor(lo, o, 64));
    hi = fmaxf(hi, __shfl_xor(hi, o, 64));
  }
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(lo + hi < kMid ? 0.f : kMid)));
}

// Rows are loaded kTaps ahead of their use: the queue slot of a row is then its ring slot (row % 11), fixed at
// every position of the unrolled loop.  (Two rows ahead: a wave alone on its SIMD waits on every row.)
struct FwdStrip {
  __amdgpu_buffer_rsrc_t rx, ry, rm;
  int W, H, x0, y0, lane, rows;  // rows: input rows of the strip
  int64_t HW;
  float mid;                                         // of the moments
  float xa[kTaps], xb[kTaps], ya[kTaps], yb[kTaps];  // the next rows' own and halo columns
  float ring[kTaps][4];                              // horizontal sums of the last 11 input rows
  double m_sum, l1_sum;
};

// Loads input row rn of the strip into queue slot Q (rows past the strip are loaded too, and not used).
template <int Q>
__device__ __forceinline__ void fwd_load(FwdStrip& f, int rn) {
  uint32_t oa, ob;
  row_offsets(f.W, f.H, f.x0, f.y0 - kR + rn, f.lane, oa, ob);
  f.xa[Q] = load_or_zero(f.rx, oa);
  f.xb[Q] = load_or_zero(f.rx, ob);
  f.ya[Q] = load_or_zero(f.ry, oa);
  f.yb[Q] = load_or_zero(f.ry, ob);
}

// Input row r (image row y0 - 5 + r) into the ring; from row 10 on, output row y0 + r - 10 from the ring.
template <int J>
__device__ __forceinline__ void fwd_step(FwdStrip& f, float4* s, const Win& win, int r) {
  wave_lds_order();  // the previous row is no longer read
  const float x = f.xa[J] - f.mid, y = f.ya[J] - f.mid;
  s[f.lane] = make_float4(x, y, fmaf(x, x, y * y), x * y);
  if (f.lane < 2 * kR) {
    const float u = f.xb[J] - f.mid, v = f.yb[J] - f.mid;
    s[kStripW + f.lane] = make_float4(u, v, fmaf(u, u, v * v), u * v);
  }
  // L1 of the row where it is one of the strip's outputs, from the raw values: lanes 5 to 63 loaded columns x0 to
  // x0 + 58 with their own, lanes 0 to 4 the other five with the halo (both images read 0 outside)
  float l1 = f.xa[J] - f.ya[J];
  if (f.lane < kR) l1 = f.xb[J] - f.yb[J];
  asm volatile("" : "+v"(l1));  // taken here: left to the scheduler, the kernel needs 184 registers instead of 162
  f.l1_sum += r >= kR && r < f.rows - kR ? (double)fabsf(l1) : 0.0;
  wave_lds_order();
  fwd_load<J>(f, r + kTaps);  // the slot is free again
  float m0 = 0, m1 = 0, m2 = 0, m3 = 0;
#pragma unroll
  for (int a = 0; a < kTaps; ++a) {
    const float4 q = s[f.lane + a];
    const float g = win.g[a];
    m0 = fmaf(g, q.x, m0);
    m1 = fmaf(g, q.y, m1);
    m2 = fmaf(g, q.z, m2);
    m3 = fmaf(g, q.w, m3);
  }
  f.ring[J][0] = m0; f.ring[J][1] = m1; f.ring[J][2] = m2; f.ring[J][3] = m3;
  if (r < 2 * kR) return;
  float v[4];
  vsum<4, J>(f.ring, win, v);
  const float sx = v[0], sy = v[1], mx = sx + f.mid, my = sy + f.mid;  // the means, shifted and true
  const int px = f.x0 + f.lane, py = f.y0 + r - 2 * kR;
  const bool in = px < f.W && py < f.H;
  const float A1 = fmaf(2.f * mx, my, kC1), A2 = fmaf(2.f, fmaf(-sx, sy, v[3]), kC2);
  const float B1 = fmaf(mx, mx, fmaf(my, my, kC1)), B2 = (v[2] - fmaf(sx, sx, sy * sy)) + kC2;
  // single-precision reciprocals (1 ulp) in place of IEEE divisions
  const float iB1 = __builtin_amdgcn_rcpf(B1), iB2 = __builtin_amdgcn_rcpf(B2);
  const float iB = iB1 * iB2;
  const float m = A1 * A2 * iB;
  const uint32_t o = (uint32_t)((int64_t)py * f.W + px) * 4u, hw = (uint32_t)f.HW * 4u;
  store_or_drop(f.rm, 2.f * my * (A2 - A1) * iB - 2.f * m * mx * (iB1 - iB2), in ? o : kDrop);
  store_or_drop(f.rm, -m * iB2, in ? o + hw : kDrop);
  store_or_drop(f.rm, 2.f * A1 * iB, in ? o + 2u * hw : kDrop);
  f.m_sum += in ? (double)m : 0.0;
}

// The strip's rows in groups of kTaps, the first slot of each group first; ends after row f.rows - 1.
#define CGV2_STRIP_ROWS(STEP)                    \
  for (int r = 0;; r += kTaps) {                 \
    STEP(0) STEP(1) STEP(2) STEP(3) STEP(4) STEP(5) STEP(6) STEP(7) STEP(8) STEP(9) STEP(10) \
  }

template <int J>
__device__ __forceinline__ void fwd_fill(FwdStrip& f) {
  fwd_load<J>(f, J);
  if constexpr (J + 1 < kTaps) fwd_fill<J + 1>(f);
}

__device__ __forceinline__ void fwd_rows(FwdStrip& f, float4* s, const Win& win) {
#define CGV2_STEP(J)              \
  if (r + J >= f.rows) return;    \
  fwd_step<J>(f, s, win, r + J);
  CGV2_STRIP_ROWS(CGV2_STEP)
#undef CGV2_STEP
}

__global__ __launch_bounds__(64) void k_ssim_fwd(const float* __restrict__ img, const float* __restrict__ tgt, int W,
                                                 int H, Win win, StripGrid sg, float* __restrict__ maps,
                                                 double* __restrict__ partial) {
  __shared__ float4 s[kRowW];
  FwdStrip f;
  int vc;
  const int strip = strip_of_block(sg, f.x0, f.y0, vc);
  f.W = W;
  f.H = H;
  f.lane = (int)threadIdx.x;
  f.rows = min(sg.rows, H - f.y0) + 2 * kR;
  f.HW = (int64_t)W * H;
  f.rx = plane_rsrc(img + vc * f.HW, f.HW);
  f.ry = plane_rsrc(tgt + vc * f.HW, f.HW);
  f.rm = plane_rsrc(maps + (int64_t)vc * 3 * f.HW, 3 * f.HW);
  f.m_sum = f.l1_sum = 0.0;
  StripSample q;
  sample_load(q, f.rx, f.ry, W, H, f.x0, f.y0, sg.rows, f.lane);
  fwd_fill<0>(f);
  f.mid = strip_mid(q);
  fwd_rows(f, s, win);
  // per-wave sums in FP64, fixed order (butterfly)
  double m_sum = f.m_sum, l1_sum = f.l1_sum;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    m_sum += __shfl_xor(m_sum, o, 64);
    l1_sum += __shfl_xor(l1_sum, o, 64);
  }
  if (f.lane == 0) {
    partial[2 * (int64_t)strip] = m_sum;
    partial[2 * (int64_t)strip + 1] = l1_sum;
  }
}

struct BwdStrip {
  __amdgpu_buffer_rsrc_t rm, rx, ry, rs, ri;
  int W, H, x0, y0, lane, rows;
  int64_t HW;
  float ninv, lambda;
  float va[kTaps][3], vb[kTaps][3];  // the next rows of the three maps
  float xv[kTaps], yv[kTaps];        // image and target at those rows' output pixels
  float ring[kTaps][3];
};

// Loads input row rn of the strip (three maps) and the image / target at its output pixel into slot k.
template <int k>
__device__ __forceinline__ void bwd_load(BwdStrip& f, int rn) {
  uint32_t oa, ob;
  row_offsets(f.W, f.H, f.x0, f.y0 - kR + rn, f.lane, oa, ob);
  const uint32_t hw = (uint32_t)f.HW * 4u;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    f.va[k][q] = load_or_zero(f.rm, oa == kDrop ? kDrop : oa + (uint32_t)q * hw);
    f.vb[k][q] = load_or_zero(f.rm, ob == kDrop ? kDrop : ob + (uint32_t)q * hw);
  }
  const int px = f.x0 + f.lane, pyn = f.y0 + rn - 2 * kR;
  const bool ok = rn >= 2 * kR && px < f.W && pyn < f.H;
  const uint32_t on = ok ? (uint32_t)((int64_t)pyn * f.W + px) * 4u : kDrop;
  f.xv[k] = load_or_zero(f.rx, on);
  f.yv[k] = load_or_zero(f.ry, on);
}

template <int J>
__device__ __forceinline__ void bwd_step(BwdStrip& f, float4* s, const Win& win, int r) {
  wave_lds_order();
  s[f.lane] = make_float4(f.va[J][0], f.va[J][1], f.va[J][2], 0.f);
  if (f.lane < 2 * kR) s[kStripW + f.lane] = make_float4(f.vb[J][0], f.vb[J][1], f.vb[J][2], 0.f);
  wave_lds_order();
  const float xc = f.xv[J], yc = f.yv[J];  // this row's output pixel
  bwd_load<J>(f, r + kTaps);
  float m0 = 0, m1 = 0, m2 = 0;
#pragma unroll
  for (int a = 0; a < kTaps; ++a) {
    const float4 q = s[f.lane + a];
    const float g = win.g[a];
    m0 = fmaf(g, q.x, m0);
    m1 = fmaf(g, q.y, m1);
    m2 = fmaf(g, q.z, m2);
  }
  f.ring[J][0] = m0; f.ring[J][1] = m1; f.ring[J][2] = m2;
  if (r < 2 * kR) return;
  float sv[3];
  vsum<3, J>(f.ring, win, sv);
  const int px = f.x0 + f.lane, py = f.y0 + r - 2 * kR;
  const bool in = px < f.W && py < f.H;
  const uint32_t o = in ? (uint32_t)((int64_t)py * f.W + px) * 4u : kDrop;
  const float dssim = f.ninv * (sv[0] + 2.f * xc * sv[1] + yc * sv[2]);
  const float d = xc - yc;
  const float sgn = d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f);
  store_or_drop(f.rs, -f.lambda * dssim, o);
  store_or_drop(f.ri, (1.f - f.lambda) * sgn * f.ninv - f.lambda * dssim, o);
}

template <int J>
__device__ __forceinline__ void bwd_fill(BwdStrip& f) {
  bwd_load<J>(f, J);
  if constexpr (J + 1 < kTaps) bwd_fill<J + 1>(f);
}

__device__ __forceinline__ void bwd_rows(BwdStrip& f, float4* s, const Win& win) {
#define CGV2_STEP(J)              \
  if (r + J >= f.rows) return;    \
  bwd_step<J>(f, s, win, r + J);
  CGV2_STRIP_ROWS(CGV2_STEP)
#undef CGV2_STEP
}
#undef CGV2_STRIP_ROWS

__device__ __noinline__ void loss_final(const double* __restrict__ partial, int64_t blocks_per_view, int V, int64_t HW,
                                        float lambda, float* __restrict__ loss);

__global__ __launch_bounds__(64) void k_ssim_bwd(const float* __restrict__ img, const float* __restrict__ tgt, int W,
                                                 int H, Win win, StripGrid sg, float lambda,
                                                 const float* __restrict__ maps, float* __restrict__ d_img,
                                                 float* __restrict__ d_ssim, const double* __restrict__ partial,
                                                 int V, float* __restrict__ loss) {
  __shared__ float4 s[kRowW];
  if (blockIdx.x == 0) loss_final(partial, (int64_t)sg.nx * sg.ny * 3, V, (int64_t)W * H, lambda, loss);
  BwdStrip f;
  int vc;
  strip_of_block(sg, f.x0, f.y0, vc);
  f.W = W;
  f.H = H;
  f.lane = (int)threadIdx.x;
  f.rows = min(sg.rows, H - f.y0) + 2 * kR;
  f.HW = (int64_t)W * H;
  f.ninv = 1.f / (3.f * (float)f.HW);
  f.lambda = lambda;
  f.rm = plane_rsrc(maps + (int64_t)vc * 3 * f.HW, 3 * f.HW);
  f.rx = plane_rsrc(img + vc * f.HW, f.HW);
  f.ry = plane_rsrc(tgt + vc * f.HW, f.HW);
  f.rs = plane_rsrc(d_ssim + vc * f.HW, f.HW);
  f.ri = plane_rsrc(d_img + vc * f.HW, f.HW);
  bwd_fill<0>(f);
  bwd_rows(f, s, win);
}

// The loss values of every view from the forward's per-wave sums, in a fixed order: run by the first
// workgroup of k_ssim_bwd (the forward has completed by then).
__device__ __noinline__ void loss_final(const double* __restrict__ partial, int64_t blocks_per_view, int V, int64_t HW,
                                        float lambda, float* __restrict__ loss) {
  const int lane = (int)threadIdx.x;
  for (int v = 0; v < V; ++v) {
    double a = 0, b = 0;
    const double2* pv = (const double2*)partial + v * blocks_per_view;
#pragma unroll 4
    for (int64_t k = lane; k < blocks_per_view; k += 64) {
      const double2 q = pv[k];
      a += q.x;
      b += q.y;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      a += __shfl_xor(a, o, 64);
      b += __shfl_xor(b, o, 64);
    }
    if (lane == 0) {
      const double ssim = a / (3.0 * HW), l1 = b / (3.0 * HW);
      loss[3 * v] = (float)((1.0 - lambda) * l1 + lambda * (1.0 - ssim));
      loss[3 * v + 1] = (float)l1;
      loss[3 * v + 2] = (float)ssim;
    }
  }
}

}  // namespace cgv2

// Output rows per strip: a launch lasts as long as the SIMD with the most strips, whose input rows (the output
// rows and a 10-row halo each) cost about 0.35 us per strip when two or more share the SIMD and 0.52 us for a
// strip alone (forward and reverse: 82 output rows, one strip per SIMD, 96 us at 1600x1066; 40 rows, two, 71;
// 27 rows, three, 78; 45 rows, as before, 1.8 per SIMD, 80).  The cheapest height is taken, the largest of
// equals (fewer halo rows read); small images take short strips (128x128: 50 -> 23 us).
constexpr int kMinRows = 4;
static cgv2::StripGrid strip_grid(int W, int H, int V) {
  constexpr int64_t kSimds = 1024;
  cgv2::StripGrid g;
  g.nx = (W + cgv2::kStripW - 1) / cgv2::kStripW;
  int64_t best = INT64_MAX;
  for (int rows = kMinRows; rows <= 128; ++rows) {
    const int ny = (H + rows - 1) / rows;
    const int64_t strips = (int64_t)g.nx * ny * 3 * V;
    const int64_t per = (strips + kSimds - 1) / kSimds;
    const int64_t cost = (per == 1 ? 52 : 35 * per) * (rows + 2 * cgv2::kR);
    if (cost > best) continue;
    best = cost;
    g.rows = rows;
    g.ny = ny;
  }
  return g;
}

size_t cgv2_loss_ws_layout(int W, int H, int V, size_t* off) {
  // room for the most strips: a workspace sized for a larger image, whose strips may be taller, serves this one too
  const int64_t nx = (W + cgv2::kStripW - 1) / cgv2::kStripW, ny = ((int64_t)H + kMinRows - 1) / kMinRows;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t r = o; o += (bytes + 255) & ~(size_t)255; return r; };
  off[0] = take(sizeof(float) * 9 * (size_t)W * H * V);     // partial maps [V][3][3][H][W]
  off[1] = take(sizeof(double) * 2 * (size_t)(nx * ny * 3 * V));  // per-wave sums
  return o;
}

hipError_t cgv2_launch_loss(const float* img, const float* tgt, int V, int W, int H, float lambda, float* d_img,
                            float* d_ssim, float* loss, void* ws, hipStream_t st) {
  size_t off[kLossOffs];
  cgv2_loss_ws_layout(W, H, V, off);
  float* maps = (float*)((char*)ws + off[0]);
  double* partial = (double*)((char*)ws + off[1]);
  cgv2::Win win;
  double g[11], gs = 0;
  for (int a = -5; a <= 5; ++a) { g[a + 5] = exp(-(double)(a * a) / (2 * 1.5 * 1.5)); gs += g[a + 5]; }
  for (int a = 0; a < 11; ++a) win.g[a] = (float)(g[a] / gs);
  const cgv2::StripGrid sg = strip_grid(W, H, V);
  const unsigned blocks = (unsigned)(sg.nx * sg.ny * 3 * V);
  hipLaunchKernelGGL(cgv2::k_ssim_fwd, dim3(blocks), dim3(64), 0, st, img, tgt, W, H, win, sg, maps, partial);
  hipLaunchKernelGGL(cgv2::k_ssim_bwd, dim3(blocks), dim3(64), 0, st, img, tgt, W, H, win, sg, lambda, maps, d_img,
                     d_ssim, partial, V, loss);
  return hipGetLastError();
}
