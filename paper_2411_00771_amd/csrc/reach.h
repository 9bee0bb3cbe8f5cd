// Where a surfel can reach alpha >= 1/255: the test of the tile lists and of the quadrant masks.  Also compiled by
// the host compiler, for its check against the renderer's evaluation on thin surfels.
#pragma once
#include <math.h>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define CGV2_FN __device__ __forceinline__
#else
#define CGV2_FN inline
#endif

namespace cgv2 {

// Where a surfel can reach alpha >= 1/255 (Sec. 3.1 cutoff).  rho is the smaller of the ray-splat
// distance |A x|^2 / w(x)^2 and the screen-filter distance |x|^2, both halved (x relative to the
// projected centre; A = the record's a_ij / sqrt 2, w(x) = w0 + w1 x + w2 y as the renderer stages
// them, so this is the function its evaluation rounds), and the cutoff is rho <= ln(255 o) = k2 / 2.
// {|A x|^2 <= c w(x)^2} is the conic g(x) = x'Gx + 2 b'x + d <= 0; when G is positive definite it is an
// ellipse, met by a box iff g <= 0 at its smallest there (see reach_box).  FP64, with the cutoff
// enlarged to c = 0.5 k2 (1 + 2e-3) + 1e-3 and every box padded by kReachPad, against the FP32 error of
// the evaluation.  A conic that is not an ellipse reaches every box, and so does one whose long axis that error can
// stretch by more than this slack: a long thin surfel seen edge-on, with det G below kReachCond G00 G11.  (650 M
// pixel samples on the long axes of surfels with ratios up to 1,000, tilted against the ray by 1.5 to 1e-7 rad, that
// the evaluation takes: none in a box reported unreachable, none either with a limit of 1e-12, 17 with 1e-13, 330,000
// without limit.  With single-precision reciprocals, whose error the centre and the line minima of such a conic
// magnify by its condition, 7 M.  The Newton steps cost a 4K view of 5 M surfels 1,951 -> 1,975 us, the step of 1 M
// at 1600x1066 nothing.)
constexpr float kInvSqrt2 = 0.70710678118654752440f;
constexpr double kReachPad = 1.0 / 64.0;
constexpr double kReachCond = 1e-11;

struct Reach {
  double G00, G01, G11, b0, b1, d, c, i00, i11, xs, ys;
  bool ellipse;
};

CGV2_FN float reach_rcp(float x) {
#ifdef __HIPCC__
  return __builtin_amdgcn_rcpf(x);
#else
  return 1.0f / x;
#endif
}

CGV2_FN void reach_setup(float a11, float a12, float a21, float a22, float w0f, float w1f, float w2f, float k2,
                         Reach& q) {
  q.c = 0.5 * (double)k2 * (1.0 + 2e-3) + 1e-3;
  const double A11 = a11, A12 = a12, A21 = a21, A22 = a22, w0 = w0f, w1 = w1f, w2 = w2f, c = q.c;
  q.G00 = A11 * A11 + A21 * A21 - c * w1 * w1;
  q.G01 = A11 * A12 + A21 * A22 - c * w1 * w2;
  q.G11 = A12 * A12 + A22 * A22 - c * w2 * w2;
  const double pp = q.G00 * q.G11, det = pp - q.G01 * q.G01;
  q.b0 = -c * w0 * w1;
  q.b1 = -c * w0 * w2;
  q.d = -c * w0 * w0;
  // single-precision reciprocals and a Newton step (error about 1e-14)
  const float r00 = reach_rcp((float)q.G00), r11 = reach_rcp((float)q.G11), rdet = reach_rcp((float)det);
  // (a reciprocal that overflows or underflows in single precision leaves the conic unused)
  const bool fin = isfinite(r00) && isfinite(r11) && isfinite(rdet) && r00 > 0.f && r11 > 0.f && rdet > 0.f;
  q.ellipse = q.G00 > 0.0 && q.G11 > 0.0 && det > kReachCond * pp && det < 1e300 && fin;
  auto newton = [](double r, double x) { return fma(r, fma(-x, r, 1.0), r); };
  q.i00 = q.ellipse ? newton(r00, q.G00) : 0.0;
  q.i11 = q.ellipse ? newton(r11, q.G11) : 0.0;
  const double idet = q.ellipse ? newton(rdet, det) : 0.0;
  q.xs = -(q.G11 * q.b0 - q.G01 * q.b1) * idet;
  q.ys = -(q.G00 * q.b1 - q.G01 * q.b0) * idet;
}

// Does the box [xl, xh] x [yl, yh] (centre-relative, already padded) hold a point with rho <= c?
// The minimum of the convex g over a box that does not hold the ellipse's centre lies on an edge facing the
// centre, so two evaluations decide: the best point of the vertical through the centre's x clamped to the
// box, and of the horizontal through its clamped y (with the centre inside, either is the centre).
// Against all four edges: 10 M surfels in 8 views, k_stage_big 396 -> 313 us, forward 2716 -> 2624, contribution
// pass 2778 -> 2535; 1 M at 1600x1066, k_stage 27.5 -> 25.6, forward 194 -> 190.
CGV2_FN bool reach_box(const Reach& q, double xl, double xh, double yl, double yh) {
  auto clamp = [](double v, double lo, double hi) { return fmin(fmax(v, lo), hi); };
  // screen-filter disc |x|^2 <= c
  const double dx = clamp(0.0, xl, xh), dy = clamp(0.0, yl, yh);
  if (fma(dx, dx, dy * dy) <= q.c) return true;
  if (!q.ellipse) return true;
  const double X = clamp(q.xs, xl, xh), Y = clamp(q.ys, yl, yh);
  const double p = fma(q.G01, X, q.b1), r = fma(q.G01, Y, q.b0);
  const double y = clamp(-p * q.i11, yl, yh), x = clamp(-r * q.i00, xl, xh);
  const double gx = fma(fma(q.G11, y, p + p), y, fma(fma(q.G00, X, 2.0 * q.b0), X, q.d));
  const double gy = fma(fma(q.G00, x, r + r), x, fma(fma(q.G11, Y, 2.0 * q.b1), Y, q.d));
  return fmin(gx, gy) <= 0.0;
}

// Box of the pixel samples [x0 + 0.5, x0 + span - 0.5] x [y0 + ...] of a tile-relative cell, relative to
// the tile-relative centre (cxt, cyt), padded.
CGV2_FN bool reach_cell(const Reach& q, float cxt, float cyt, int x0, int y0, int span) {
  const double xl = (double)x0 + 0.5 - (double)cxt - kReachPad, xh = xl + (double)(span - 1) + 2.0 * kReachPad;
  const double yl = (double)y0 + 0.5 - (double)cyt - kReachPad, yh = yl + (double)(span - 1) + 2.0 * kReachPad;
  return reach_box(q, xl, xh, yl, yh);
}

}  // namespace cgv2
