// Visibility-frequency crop volume of the CityGaussianV2 evaluation protocol (Sec. 4): every
// ground-truth point is a small isotropic Gaussian; over all views, count the views in which its visible
// mask is set; keep the points seen often enough, take their height range and their ground-plane
// coordinates (for the alpha shape, which runs on the host).
//
// A point's footprint is the image of the sphere of radius rho around it, hulled with a disc of rf
// pixels around its projected centre; it is visible when its centre depth exceeds znear and a pixel
// sample (i + 0.5, j + 0.5) lies in the footprint's box (a sphere reaching the camera plane, depth <=
// rho, is visible).  Every decision is taken in FP64.
//
//   k_vis_table  per view: the camera in FP64 (a row) and, as columns across the views, its depth row, znear and
//                the planes through the camera and the four image edges
//   k_vis_count  per workgroup of up to 4,096 consecutive points: the box of its points is classified against 256
//                views at a time, one view per thread; then each wave classifies the views left undecided, one
//                per lane, against each of its boxes of 128 points.  A view that cannot see any point of a box is
//                skipped; a view in which every centre projects inside the sample range counts for all points at
//                once (rf >= 0.5 guarantees the nearest sample is covered); only the remaining views test the
//                points one by one, and most of them by the sign of a single plane.
//                Points in spatially coherent order make the boxes small; any order gives the same counts.
//   k_crop_*     threshold, FP64 ground transform, height range, order-preserving compaction
#include "cgv2r_device.h"
#include "cgv2r_kernels.h"

#include <algorithm>
#include <cmath>

namespace cgv2 {

constexpr int kVisThreads = 256;
constexpr int kVisWaves = kVisThreads / 64;
constexpr int kVisPts = 2;              // points per lane of a wave's box
constexpr int kVisRun = 64 * kVisPts;   // points per wave box
constexpr int kVisRuns = 8;             // most boxes per wave
// Per-view table in the workspace: an FP64 camera row per view (read with scalar loads by the general per-point
// test) and one column per coefficient across the views (one view per lane: coalesced loads).
constexpr int kRow = 36;                 // doubles of room per camera row (19 used)
constexpr int kCols = 37;                // doubles of room per view in the columns (25 used)
constexpr double kEdgeMarginPx = 1e-2;   // the plane tests keep this far from every decision edge
constexpr double kDepthMargin = 1e-7;

enum : int { T_R = 0, T_T = 9, T_FX = 12, T_FY, T_CX, T_CY, T_ZN, T_W, T_H };  // row of the general test
enum : int { C_Z = 0, C_ZN = 4, C_PL = 5, C_N = 21 };  // columns: depth row, znear, side q's plane at C_PL + 4 q, reach

struct VisTable {
  double* row;  // [V][kRow]
  double* col;  // [kCols][V]
  int V;
};

__global__ void k_vis_table(CamPack cams, double rho, VisTable tab) {
  const int k = threadIdx.x;
  if (k >= cams.count) return;
  const DevCam& c = cams.c[k];
  const int v = cams.v0 + k;
  double* T = tab.row + (int64_t)v * kRow;
  auto col = [&](int q) -> double& { return tab.col[(int64_t)q * tab.V + v]; };
  double R[9], t[3];
  for (int i = 0; i < 9; ++i) R[i] = T[T_R + i] = (double)c.R[i];
  for (int i = 0; i < 3; ++i) t[i] = T[T_T + i] = (double)c.t[i];
  const double fx = c.fx, fy = c.fy, cx = c.cx, cy = c.cy, W = c.W, H = c.H, zn = c.znear;
  T[T_FX] = fx, T[T_FY] = fy, T[T_CX] = cx, T[T_CY] = cy, T[T_ZN] = zn, T[T_W] = W, T[T_H] = H;
  for (int i = 0; i < 3; ++i) col(C_Z + i) = R[6 + i];
  col(C_Z + 3) = t[2];
  col(C_ZN) = zn;
  // u >= k  <=>  fx Xc + (cx - k) Zc >= 0 (Zc > 0); world plane w . p + off with w = fx R0 + (cx - k) R2, and a
  // sphere of radius rho reaches rho |(fx, cx - k)| beyond it in its own units
  auto side = [&](int q, int row, double f, double cc, double kk, double sign) {
    for (int i = 0; i < 3; ++i) col(C_PL + 4 * q + i) = sign * (f * R[3 * row + i] + (cc - kk) * R[6 + i]);
    col(C_PL + 4 * q + 3) = sign * (f * t[row] + (cc - kk) * t[2]);
    col(C_N + q) = rho * sqrt(f * f + (cc - kk) * (cc - kk));
  };
  side(0, 0, fx, cx, 0.5, 1.0);
  side(1, 0, fx, cx, W - 0.5, -1.0);
  side(2, 1, fy, cy, 0.5, 1.0);
  side(3, 1, fy, cy, H - 0.5, -1.0);
}

// A view's coefficients: depth row, znear, the planes through the camera and the first and last sample column and
// row (inside is positive), and the reach of the sphere beyond each.
struct ViewPlanes {
  double z[4], zn, p[4][4], n[4];
};

__device__ __forceinline__ void load_planes(const VisTable& tab, int v, ViewPlanes& k) {
  auto at = [&](int q) { return tab.col[(int64_t)q * tab.V + v]; };
#pragma unroll
  for (int i = 0; i < 4; ++i) k.z[i] = at(C_Z + i);
  k.zn = at(C_ZN);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
#pragma unroll
    for (int i = 0; i < 4; ++i) k.p[q][i] = at(C_PL + 4 * q + i);
    k.n[q] = at(C_N + q);
  }
}

// What a box of points c +- h (world, FP64) leaves undecided of a view: 0 every centre projects inside the sample
// range (all visible), else a bit per image side that crosses the box and kDepthBit when its depths need a test;
// kViewOut when no point can be visible, kDepthOnly when only those can whose sphere reaches the camera plane (the
// boxes beside an oblique camera: half of all that are left undecided).  'wide' (rf >= 0.5): a centre in the sample range covers a sample.
// With L the value of a side's plane at a point, no sample is covered beyond that side when L < -max(rf Z, reach).
constexpr uint32_t kDepthBit = 16u, kAllBits = 31u, kViewOut = 32u, kDepthOnly = 64u;

struct Depths {
  double lo, hi;  // of the box in the view
};

__device__ __forceinline__ uint32_t classify(const ViewPlanes& k, const double c[3], const double h[3], double rho,
                                             double rf, bool wide, Depths& z) {
  const double zc = fma(k.z[0], c[0], fma(k.z[1], c[1], fma(k.z[2], c[2], k.z[3])));
  const double zr = fma(fabs(k.z[0]), h[0], fma(fabs(k.z[1]), h[1], fabs(k.z[2]) * h[2]));
  z.lo = zc - zr;
  z.hi = zc + zr;
  const bool behind = z.hi < k.zn - kDepthMargin;  // every centre at or before znear
  const bool far = z.lo > rho + kDepthMargin;      // no sphere reaches the camera plane
  const bool front = z.lo > k.zn + kDepthMargin;
  const double disc = rf * z.hi, margin = kEdgeMarginPx * z.hi;
  bool out = false;
  uint32_t sides = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double* P = k.p[q];
    const double s = fma(P[0], c[0], fma(P[1], c[1], fma(P[2], c[2], P[3])));
    const double r = fma(fabs(P[0]), h[0], fma(fabs(P[1]), h[1], fabs(P[2]) * h[2]));
    out = out || s + r < -(margin + (disc > k.n[q] ? disc : k.n[q]));
    if (!(s - r > margin)) sides |= 1u << q;
  }
  if (behind || (far && out)) return kViewOut;
  if (out) return kDepthOnly;
  if (!wide || !front) return kAllBits;
  return sides == 0u || far ? sides : sides | kDepthBit;
}

// The visible mask of one point in one view, as defined (FP64): any filter reach.
__device__ __forceinline__ bool vis_exact(const double* T, double x, double y, double z, double rho,
                                          double rf) {
  const double X = T[0] * x + T[1] * y + T[2] * z + T[9];
  const double Y = T[3] * x + T[4] * y + T[5] * z + T[10];
  const double Z = T[6] * x + T[7] * y + T[8] * z + T[11];
  if (!(Z > T[T_ZN])) return false;
  if (Z <= rho) return true;
  const double fx = T[T_FX], fy = T[T_FY], cx = T[T_CX], cy = T[T_CY];
  const double iden = 1.0 / (Z * Z - rho * rho), iz = 1.0 / Z;
  const double sx = sqrt(X * X + Z * Z - rho * rho), sy = sqrt(Y * Y + Z * Z - rho * rho);
  const double u0 = fx * ((X * Z - rho * sx) * iden) + cx, u1 = fx * ((X * Z + rho * sx) * iden) + cx;
  const double v0 = fy * ((Y * Z - rho * sy) * iden) + cy, v1 = fy * ((Y * Z + rho * sy) * iden) + cy;
  const double uc = fx * (X * iz) + cx, vc = fy * (Y * iz) + cy;
  const double ulo = fmin(u0, uc - rf), uhi = fmax(u1, uc + rf);
  const double vlo = fmin(v0, vc - rf), vhi = fmax(v1, vc + rf);
  const double i0 = fmax(0.0, ceil(ulo - 0.5)), i1 = fmin(T[T_W] - 1.0, floor(uhi - 0.5));
  const double j0 = fmax(0.0, ceil(vlo - 0.5)), j1 = fmin(T[T_H] - 1.0, floor(vhi - 0.5));
  return i0 <= i1 && j0 <= j1;
}

// The same mask when rf >= 0.5, tested on the given sides only (the others hold for every point of the box).  The
// footprint's extent along an axis is then at least one pixel, so it holds a sample exactly when it overlaps
// [0.5, W - 0.5]: on x, max(u1, uc + rf) >= 0.5 and min(u0, uc - rf) <= W - 0.5.  Let L = fx X + (cx - 0.5) Z.
// With Z > rho, uc + rf >= 0.5 says L >= -rf Z, and u1 >= 0.5 says that the sphere reaches the plane L = 0 through
// the camera: L >= -rho |(fx, cx - 0.5)|.  So each side is one plane against the larger of the two reaches: no
// root, no division.  A point at infinity stays as the comparisons of the bounds have it (a plane value of -inf
// fails, NaN passes).
// The view is lane l's: its coefficients are read from that lane's registers (a wave alone waits about 1,000 cycles
// for a row of the table by scalar loads).
__device__ __forceinline__ double lane_value(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}

__device__ __forceinline__ void vis_exact_wide(const ViewPlanes& v, int l, uint32_t bits, const double (&p)[kVisPts][3],
                                               double rho, double rf, uint32_t (&cnt)[kVisPts]) {
  const double z0 = lane_value(v.z[0], l), z1 = lane_value(v.z[1], l), z2 = lane_value(v.z[2], l),
               z3 = lane_value(v.z[3], l);
  double Z[kVisPts], rz[kVisPts];
  bool ok[kVisPts];
#pragma unroll
  for (int k = 0; k < kVisPts; ++k) {
    Z[k] = fma(z0, p[k][0], fma(z1, p[k][1], fma(z2, p[k][2], z3)));
    rz[k] = rf * fmin(Z[k], 1e300);
    ok[k] = true;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (!(bits & (1u << q))) continue;
    const double p0 = lane_value(v.p[q][0], l), p1 = lane_value(v.p[q][1], l), p2 = lane_value(v.p[q][2], l),
                 p3 = lane_value(v.p[q][3], l), n = lane_value(v.n[q], l);
#pragma unroll
    for (int k = 0; k < kVisPts; ++k) {
        const double L = fma(p0, p[k][0], fma(p1, p[k][1], fma(p2, p[k][2], p3)));
      ok[k] = ok[k] && !(L < -fmax(rz[k], n));
    }
  }
  if (bits & kDepthBit) {
    const double zn = lane_value(v.zn, l);
#pragma unroll
    for (int k = 0; k < kVisPts; ++k) ok[k] = Z[k] > zn && (ok[k] || Z[k] <= rho);
  }
#pragma unroll
  for (int k = 0; k < kVisPts; ++k) cnt[k] += ok[k] ? 1u : 0u;
}

// Box lo, hi of the wave's points over all lanes.
__device__ __forceinline__ void wave_box(float (&lo)[3], float (&hi)[3]) {
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      lo[d] = fminf(lo[d], __shfl_xor(lo[d], s, 64));
      hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], s, 64));
    }
  }
}

constexpr uint32_t kNanPoint = 0x80000000u;

// Workgroup (x, y): kVisWaves * runs * kVisRun consecutive points, a slice of the views.
// Bound by FP64 instructions and the waits between its phases (118 registers, 4 waves per SIMD).  31.4 M points in
// octree order, 958 views: 2,820 us with boxes of 512 points per workgroup and every undecided view tested by all
// four sides, roots and divisions where one failed -> 870 (a point is left 14 undecided views instead of 26, 5 of
// them by depth only, 5.5 by one plane).  Boxes of 64 points 1,070 us; 2,048 or 8,192 points per workgroup 930
// and 1,020; 5 waves per SIMD spill (1,120).
template <bool kWide>
__global__ __launch_bounds__(kVisThreads, 4) void k_vis_count(const float* __restrict__ pts, int64_t m, VisTable tab,
                                                              int v_begin, int V, int slice, int runs, double rho,
                                                              double rf, uint32_t* __restrict__ count) {
  __shared__ float box[kVisWaves][kVisRuns][6];
  __shared__ uint32_t s_cnt[kVisWaves][kVisRuns][kVisRun];
  __shared__ uint16_t edge[kVisMaxViews];
  __shared__ uint32_t n_edge, n_in;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * kVisWaves * runs * kVisRun;
  const int64_t wbase = base + (int64_t)w * runs * kVisRun;
  const int va = (int)blockIdx.y * slice, vb = min(V, va + slice);

  if (threadIdx.x == 0) n_edge = n_in = 0;
  // a NaN coordinate is in no box: its point is not visible in any view (kNanPoint in its counter)
  auto first_pass = [&](int r, const float (&x)[kVisPts][3]) {
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int k = 0; k < kVisPts; ++k) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        lo[d] = fminf(lo[d], x[k][d]);
        hi[d] = fmaxf(hi[d], x[k][d]);
      }
      s_cnt[w][r][k * 64 + lane] = isnan(x[k][0]) || isnan(x[k][1]) || isnan(x[k][2]) ? kNanPoint : 0u;
    }
    wave_box(lo, hi);
    if (lane == 0) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        box[w][r][d] = lo[d];
        box[w][r][3 + d] = hi[d];
      }
    }
  };
  auto load_run = [&](int r, float (&x)[kVisPts][3]) {  // past the end: the last point once more
#pragma unroll
    for (int k = 0; k < kVisPts; ++k) {
      const int64_t i = min(wbase + (int64_t)r * kVisRun + k * 64 + lane, m - 1);
#pragma unroll
      for (int d = 0; d < 3; ++d) x[k][d] = pts[d * m + i];
    }
  };
  for (int r0 = 0; r0 < runs; r0 += 4) {  // four runs' points in flight
    float x[4][kVisPts][3];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (r0 + j < runs) load_run(r0 + j, x[j]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (r0 + j < runs) first_pass(r0 + j, x[j]);
  }
  __syncthreads();
  double c[3], h[3];
  auto middle = [&](const float* lo, const float* hi) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      c[d] = 0.5 * ((double)lo[d] + (double)hi[d]);
      h[d] = 0.5 * ((double)hi[d] - (double)lo[d]);
    }
  };
  {
    // the workgroup's box: its kVisWaves * runs <= 64 wave boxes, one per lane
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (lane < kVisWaves * runs) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        lo[d] = box[lane / runs][lane % runs][d];
        hi[d] = box[lane / runs][lane % runs][3 + d];
      }
    }
    wave_box(lo, hi);
    middle(lo, hi);
  }
  for (int q0 = va; q0 < vb; q0 += kVisThreads) {
    const int q = q0 + (int)threadIdx.x;
    uint32_t bits = kViewOut;
    if (q < vb) {
      ViewPlanes k;
      load_planes(tab, v_begin + q, k);
      Depths z;
      bits = classify(k, c, h, rho, rf, kWide, z);
    }
    const unsigned long long in_mask = __ballot(bits == 0u);
    const unsigned long long ed_mask = __ballot(bits != 0u && bits != kViewOut);
    uint32_t at = 0;
    if (lane == 0) {
      if (in_mask) atomicAdd(&n_in, (uint32_t)__popcll(in_mask));
      if (ed_mask) at = atomicAdd(&n_edge, (uint32_t)__popcll(ed_mask));
    }
    at = __shfl(at, 0, 64);
    if (bits != 0u && bits != kViewOut) edge[at + __popcll(ed_mask & ((1ull << lane) - 1ull))] = (uint16_t)q;
  }
  __syncthreads();

  const int na = (int)n_edge;
  for (int e0 = 0; e0 < na; e0 += 64) {
    // a lane keeps one edge view's planes for all runs of its wave
    const int v = v_begin + (e0 + lane < na ? (int)edge[e0 + lane] : (int)edge[e0]);
    ViewPlanes kp;
    load_planes(tab, v, kp);
    float x[kVisPts][3];
    load_run(0, x);
    for (int r = 0; r < runs; ++r) {
      if (wbase + (int64_t)r * kVisRun >= m) break;
      double p[kVisPts][3];
#pragma unroll
      for (int k = 0; k < kVisPts; ++k)
#pragma unroll
        for (int d = 0; d < 3; ++d) p[k][d] = x[k][d];
      if (r + 1 < runs) load_run(r + 1, x);  // in flight during this run's tests
      middle(&box[w][r][0], &box[w][r][3]);
      Depths z;
      uint32_t bits = classify(kp, c, h, rho, rf, kWide, z);
      if (e0 + lane >= na) bits = kViewOut;
      uint32_t cnt[kVisPts];
#pragma unroll
      for (int k = 0; k < kVisPts; ++k) cnt[k] = (uint32_t)__popcll(__ballot(bits == 0u));
      if constexpr (kWide) {
        // Most views have one side crossing the box and one of the two reaches the larger over all of it: their
        // test is the sign of one plane.
        double a[4], n = kp.n[0];
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = kp.p[0][i];
#pragma unroll
        for (int q = 1; q < 4; ++q) {
          const bool is = bits == (1u << q);
#pragma unroll
          for (int i = 0; i < 4; ++i) a[i] = is ? kp.p[q][i] : a[i];
          n = is ? kp.n[q] : n;
        }
        const bool sphere = rf * z.hi < n * (1.0 - 1e-9), disc = rf < 1e300 && rf * z.lo > n * (1.0 + 1e-9);
        const bool one = (bits == 1u || bits == 2u || bits == 4u || bits == 8u) && (sphere || disc);
        a[3] = sphere ? a[3] + n : fma(rf, kp.z[3], a[3]);
#pragma unroll
        for (int i = 0; i < 3; ++i) a[i] = sphere ? a[i] : fma(rf, kp.z[i], a[i]);
        for (unsigned long long ed = __ballot(one); ed; ed &= ed - 1) {
          const int l = __builtin_ctzll(ed);
          const double a0 = lane_value(a[0], l), a1 = lane_value(a[1], l), a2 = lane_value(a[2], l),
                       a3 = lane_value(a[3], l);
#pragma unroll
          for (int k = 0; k < kVisPts; ++k)
            cnt[k] += fma(a0, p[k][0], fma(a1, p[k][1], fma(a2, p[k][2], a3))) >= 0.0 ? 1u : 0u;
        }
        for (unsigned long long ed = __ballot(bits == kDepthOnly); ed; ed &= ed - 1) {
          const int l = __builtin_ctzll(ed);
          const double z0 = lane_value(kp.z[0], l), z1 = lane_value(kp.z[1], l), z2 = lane_value(kp.z[2], l),
                       z3 = lane_value(kp.z[3], l), zn = lane_value(kp.zn, l);
#pragma unroll
          for (int k = 0; k < kVisPts; ++k) {
            const double Z = fma(z0, p[k][0], fma(z1, p[k][1], fma(z2, p[k][2], z3)));
            cnt[k] += Z > zn && Z <= rho ? 1u : 0u;
          }
        }
        for (unsigned long long ed = __ballot(bits != 0u && bits < kViewOut && !one); ed; ed &= ed - 1) {
          const int l = __builtin_ctzll(ed);
          vis_exact_wide(kp, l, __builtin_amdgcn_readlane(bits, l), p, rho, rf, cnt);
        }
      } else {
        for (unsigned long long ed = __ballot(bits != kViewOut); ed; ed &= ed - 1) {
          // the view is uniform: its camera row is read with scalar loads
          const double* T = tab.row + (int64_t)__builtin_amdgcn_readlane(v, __builtin_ctzll(ed)) * kRow;
#pragma unroll
          for (int k = 0; k < kVisPts; ++k) cnt[k] += vis_exact(T, p[k][0], p[k][1], p[k][2], rho, rf) ? 1u : 0u;
        }
      }
#pragma unroll
      for (int k = 0; k < kVisPts; ++k) s_cnt[w][r][k * 64 + lane] += cnt[k];
    }
  }
  const uint32_t ia = n_in;
#pragma unroll 4
  for (int r = 0; r < runs; ++r) {
#pragma unroll
    for (int k = 0; k < kVisPts; ++k) {
      const int64_t i = wbase + (int64_t)r * kVisRun + k * 64 + lane;
      if (i >= m) continue;
      const uint32_t own = s_cnt[w][r][k * 64 + lane];
      const uint32_t t = own & kNanPoint ? 0u : ia + own;
      if (gridDim.y > 1) {
        if (t) atomicAdd(&count[i], t);
      } else {
        count[i] += t;
      }
    }
  }
}

// ---- crop: threshold, ground transform, height range, compaction ---------------------------------

constexpr int kCropBlock = 256;
constexpr int kCropItems = 8;
constexpr int kCropChunk = kCropBlock * kCropItems;

struct Ground {
  double T[12];
};

__device__ __forceinline__ void ground_of(const Ground& g, const float* pts, int64_t m, int64_t i, double& gx,
                                          double& gy, double& gh) {
  const double x = pts[i], y = pts[m + i], z = pts[2 * m + i];
  gx = g.T[0] * x + g.T[1] * y + g.T[2] * z + g.T[3];
  gy = g.T[4] * x + g.T[5] * y + g.T[6] * z + g.T[7];
  gh = g.T[8] * x + g.T[9] * y + g.T[10] * z + g.T[11];
}

// per workgroup: kept count, height min and max of its kept points
__global__ __launch_bounds__(kCropBlock) void k_crop_count(const float* __restrict__ pts, int64_t m,
                                                           const uint32_t* __restrict__ count, uint32_t tau, Ground g,
                                                           uint8_t* __restrict__ keep, uint32_t* __restrict__ kpart,
                                                           double* __restrict__ hpart) {
  __shared__ uint32_t lds[kCropBlock / 64];
  __shared__ double hred[2][kCropBlock / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * kCropChunk + threadIdx.x;
  uint32_t k_local = 0;
  double hmin = INFINITY, hmax = -INFINITY;
#pragma unroll
  for (int k = 0; k < kCropItems; ++k) {
    const int64_t i = base + (int64_t)k * kCropBlock;
    if (i >= m) break;
    const bool kp = count[i] >= tau;
    keep[i] = kp ? 1 : 0;
    if (kp) {
      double gx, gy, gh;
      ground_of(g, pts, m, i, gx, gy, gh);
      hmin = fmin(hmin, gh);
      hmax = fmax(hmax, gh);
      ++k_local;
    }
  }
  uint32_t tot;
  block_exscan<kCropBlock>(k_local, lds, tot);
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) {
    hmin = fmin(hmin, __shfl_xor(hmin, s, 64));
    hmax = fmax(hmax, __shfl_xor(hmax, s, 64));
  }
  if (lane == 0) {
    hred[0][w] = hmin;
    hred[1][w] = hmax;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = hred[0][0], b = hred[1][0];
    for (int q = 1; q < kCropBlock / 64; ++q) {
      a = fmin(a, hred[0][q]);
      b = fmax(b, hred[1][q]);
    }
    kpart[blockIdx.x] = tot;
    hpart[2 * blockIdx.x] = a;
    hpart[2 * blockIdx.x + 1] = b;
  }
}

constexpr int kScanBlock = 1024;
constexpr int kScanItems = 8;

// Latency bound: 8,192 partials a round (15,332 of them: 59 us in rounds of 256 -> 22).
// one workgroup: exclusive offsets of the kept points per workgroup, the kept total, the height range
__global__ __launch_bounds__(kScanBlock) void k_crop_scan(uint32_t* __restrict__ kpart, const double* __restrict__ hpart,
                                                          int nb, int64_t* __restrict__ kept,
                                                          double* __restrict__ hrange) {
  __shared__ unsigned long long lds[kScanBlock / 64];
  __shared__ double hred[2][kScanBlock / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  unsigned long long carry = 0;
  double hmin = INFINITY, hmax = -INFINITY;
  for (int b0 = 0; b0 < nb; b0 += kScanBlock * kScanItems) {
    const int b = b0 + (int)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    unsigned long long own = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      v[k] = b + k < nb ? kpart[b + k] : 0u;
      own += v[k];
      // (the heights in any order: coalesced)
      const int c = b0 + k * kScanBlock + (int)threadIdx.x;
      if (c < nb) {
        hmin = fmin(hmin, hpart[2 * (int64_t)c]);
        hmax = fmax(hmax, hpart[2 * (int64_t)c + 1]);
      }
    }
    unsigned long long tot;
    unsigned long long ex = block_exscan<kScanBlock>(own, lds, tot) + carry;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      if (b + k < nb) kpart[b + k] = (uint32_t)ex;
      ex += v[k];
    }
    carry += tot;
  }
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) {
    hmin = fmin(hmin, __shfl_xor(hmin, s, 64));
    hmax = fmax(hmax, __shfl_xor(hmax, s, 64));
  }
  if (lane == 0) {
    hred[0][w] = hmin;
    hred[1][w] = hmax;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = hred[0][0], b = hred[1][0];
    for (int q = 1; q < kScanBlock / 64; ++q) {
      a = fmin(a, hred[0][q]);
      b = fmax(b, hred[1][q]);
    }
    *kept = (int64_t)carry;
    hrange[0] = carry ? a : NAN;
    hrange[1] = carry ? b : NAN;
  }
}

// per workgroup: ground coordinates of its kept points at their slots (id order)
// Bound by memory: consecutive lanes take consecutive points, so loads and stores are coalesced (31.4 M points, 95 %
// kept: 669 us with eight consecutive points per thread -> 146, 5.9 TB/s).
__global__ __launch_bounds__(kCropBlock) void k_crop_write(const float* __restrict__ pts, int64_t m,
                                                           const uint8_t* __restrict__ keep, Ground g,
                                                           const uint32_t* __restrict__ koff,
                                                           double* __restrict__ ground) {
  constexpr int kW = kCropBlock / 64;
  __shared__ uint32_t s_kept[kCropItems][kW];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * kCropChunk + threadIdx.x;
  uint8_t kp[kCropItems];
  uint32_t rank[kCropItems];  // among the kept points of the wave's 64
#pragma unroll
  for (int k = 0; k < kCropItems; ++k) {
    const int64_t i = base + (int64_t)k * kCropBlock;
    kp[k] = i < m ? keep[i] : (uint8_t)0;
  }
#pragma unroll
  for (int k = 0; k < kCropItems; ++k) {
    const unsigned long long kept = __ballot(kp[k] != 0);
    rank[k] = (uint32_t)__popcll(kept & ((1ull << lane) - 1ull));
    if (lane == 0) s_kept[k][w] = (uint32_t)__popcll(kept);
  }
  __syncthreads();
  uint32_t at = koff[blockIdx.x];
#pragma unroll
  for (int k = 0; k < kCropItems; ++k) {
#pragma unroll
    for (int q = 0; q < kW; ++q) {
      if (q == w && kp[k]) {
        double gx, gy, gh;
        ground_of(g, pts, m, base + (int64_t)k * kCropBlock, gx, gy, gh);
        ground[at + rank[k]] = gx;
        ground[m + at + rank[k]] = gy;
      }
      at += s_kept[k][q];
    }
  }
}

}  // namespace cgv2

size_t cgv2_vis_ws_layout(int V) {
  return (((size_t)V * (cgv2::kRow + cgv2::kCols) * sizeof(double)) + 255) & ~(size_t)255;
}

static cgv2::VisTable vis_table(void* ws, int V) {
  cgv2::VisTable t;
  t.row = (double*)ws;
  t.col = t.row + (size_t)V * cgv2::kRow;
  t.V = V;
  return t;
}

hipError_t cgv2_launch_vis_table(const cgv2::CamPack& cams, int V, double rho, void* ws, hipStream_t st) {
  hipLaunchKernelGGL(cgv2::k_vis_table, dim3(1), dim3(64), 0, st, cams, rho, vis_table(ws, V));
  return hipGetLastError();
}

// Workgroups that fill the chip twice: fewer points per workgroup, then slices of the views (their counts are added
// atomically) until there are that many (us: 20,000 points, 958 views 5,930 -> 127; 200,000 points, 60 views 243 -> 42).
constexpr int64_t kVisGroups = 2048;

hipError_t cgv2_launch_vis_count(const float* pts, int64_t m, int V, double rho, double rf, uint32_t* count,
                                 void* ws, hipStream_t st) {
  if (m == 0) return hipGetLastError();
  for (int v0 = 0; v0 < V; v0 += kVisMaxViews) {
    const int vc = std::min(V - v0, kVisMaxViews);
    const int64_t boxes = (m + cgv2::kVisWaves * cgv2::kVisRun - 1) / (cgv2::kVisWaves * cgv2::kVisRun);
    const int runs = (int)std::max<int64_t>(1, std::min<int64_t>(boxes / kVisGroups, cgv2::kVisRuns));
    const int64_t gx = (boxes + runs - 1) / runs;
    const int64_t gy = std::max<int64_t>(1, std::min<int64_t>(kVisGroups / gx, (vc + 63) / 64));
    const int slice = (int)(((vc + gy - 1) / gy + 63) / 64 * 64);
    const dim3 grid((unsigned)gx, (unsigned)((vc + slice - 1) / slice));
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(cgv2::kVisThreads), 0, st, pts, m, vis_table(ws, V), v0, vc, slice, runs, rho,
                         rf, count);
    };
    if (rf >= 0.5)
      go(cgv2::k_vis_count<true>);
    else
      go(cgv2::k_vis_count<false>);
  }
  return hipGetLastError();
}

size_t cgv2_crop_ws_layout(int64_t m, size_t* off) {
  const int64_t nb = std::max<int64_t>((m + cgv2::kCropChunk - 1) / cgv2::kCropChunk, 1);
  // off: [0] kept count / offset per workgroup (u32), [1] height min / max per workgroup (f64 x 2)
  off[0] = 0;
  off[1] = ((size_t)4 * (size_t)nb + 255) & ~(size_t)255;
  return off[1] + (((size_t)16 * (size_t)nb + 255) & ~(size_t)255);
}

hipError_t cgv2_launch_crop(const float* pts, int64_t m, const uint32_t* count, uint32_t tau, const double* T,
                            uint8_t* keep, double* ground, double* hrange, int64_t* kept, void* ws, hipStream_t st) {
  size_t off[kCropOffs];
  cgv2_crop_ws_layout(m, off);
  const int nb = (int)std::max<int64_t>((m + cgv2::kCropChunk - 1) / cgv2::kCropChunk, 1);
  uint32_t* kpart = (uint32_t*)((char*)ws + off[0]);
  double* hpart = (double*)((char*)ws + off[1]);
  cgv2::Ground g;
  for (int i = 0; i < 12; ++i) g.T[i] = T[i];
  if (m > 0) {
    hipLaunchKernelGGL(cgv2::k_crop_count, dim3((unsigned)nb), dim3(cgv2::kCropBlock), 0, st, pts, m, count, tau, g,
                       keep, kpart, hpart);
  } else {
    hipLaunchKernelGGL((cgv2::k_fill<uint32_t>), dim3(1), dim3(64), 0, st, kpart, (int64_t)1, 0u);
    hipLaunchKernelGGL((cgv2::k_fill<double>), dim3(1), dim3(64), 0, st, hpart, (int64_t)2, 0.0);
  }
  hipLaunchKernelGGL(cgv2::k_crop_scan, dim3(1), dim3(cgv2::kScanBlock), 0, st, kpart, hpart, nb, kept, hrange);
  if (m > 0)
    hipLaunchKernelGGL(cgv2::k_crop_write, dim3((unsigned)nb), dim3(cgv2::kCropBlock), 0, st, pts, m, keep, g, kpart,
                       ground);
  return hipGetLastError();
}
