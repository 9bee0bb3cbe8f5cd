// Pixel samples on the long axes of thin, near edge-on surfels: prints, for each (axis ratio, largest tilt), the
// samples that the renderer's float32 evaluation takes and those of them in a tile or quadrant that the reach test
// reports unreachable.
#include <math.h>
#include <stdio.h>

#include <algorithm>
#include <random>

#include "reach.h"

namespace {

struct Record {
  float cx_hi, cy_hi, cx_lo, cy_lo, a[4], w[3], k2, o;
};

// The projection's record (float64 homography of M = K [su tu | sv tv | pc], rounded once) for a centre anywhere.
bool record(const double* tu, const double* tv, double su, double sv, const double* pc, double o, Record& r) {
  const double f = 1000, c[2] = {800, 533};
  double M[9];
  const double cols[3][3] = {{su * tu[0], su * tu[1], su * tu[2]}, {sv * tv[0], sv * tv[1], sv * tv[2]},
                             {pc[0], pc[1], pc[2]}};
  for (int k = 0; k < 3; ++k) {
    M[k] = f * cols[k][0] + c[0] * cols[k][2];
    M[3 + k] = f * cols[k][1] + c[1] * cols[k][2];
    M[6 + k] = cols[k][2];
  }
  const double k2 = 2 * log(255 * o);
  if (!(k2 > 0) || !(M[6] * M[6] + M[7] * M[7] - M[8] * M[8] / k2 < 0)) return false;
  const double cx = M[2] / M[8], cy = M[5] / M[8];
  const double al1 = M[0] - cx * M[6], al2 = M[1] - cx * M[7], be1 = M[3] - cy * M[6], be2 = M[4] - cy * M[7];
  const double A[4] = {M[8] * be2, -M[8] * al2, -M[8] * be1, M[8] * al1};
  const double W[3] = {al1 * be2 - al2 * be1, be1 * M[7] - be2 * M[6], M[6] * al2 - M[7] * al1};
  double m = 0;
  for (double x : A) m = fmax(m, fabs(x));
  for (double x : W) m = fmax(m, fabs(x));
  for (int k = 0; k < 4; ++k) r.a[k] = (float)(A[k] / m);
  for (int k = 0; k < 3; ++k) r.w[k] = (float)(W[k] / m);
  r.k2 = (float)k2;
  r.o = (float)o;
  return true;
}

// The renderer's evaluation at pixel (px, py): the terms of the quadrant-0 pixel, then 8 columns and rows further.
bool takes(const Record& r, int px, int py) {
  const int ox = px / 16 * 16, oy = py / 16 * 16, lx = (px - ox) & 7, ly = (py - oy) & 7;
  float a[4];
  for (int k = 0; k < 4; ++k) a[k] = r.a[k] * cgv2::kInvSqrt2;
  float x = ((float)lx + 0.5f) - ((r.cx_hi - (float)ox) + r.cx_lo);
  float y = ((float)ly + 0.5f) - ((r.cy_hi - (float)oy) + r.cy_lo);
  float p1 = fmaf(a[0], x, a[1] * y), p2 = fmaf(a[2], x, a[3] * y), w = fmaf(r.w[1], x, fmaf(r.w[2], y, r.w[0]));
  if ((px - ox) & 8) {
    p1 = fmaf(8.f, a[0], p1);
    p2 = fmaf(8.f, a[2], p2);
    w = fmaf(8.f, r.w[1], w);
    x += 8.f;
  }
  if ((py - oy) & 8) {
    p1 = fmaf(8.f, a[1], p1);
    p2 = fmaf(8.f, a[3], p2);
    w = fmaf(8.f, r.w[2], w);
    y += 8.f;
  }
  const float iw = 1.f / w, r2 = fmaf(x, x, y * y), r3 = fmaf(p1, p1, p2 * p2) * (iw * iw);
  const float rho = r3 <= r2 ? r3 : r2;
  return exp2f(fmaf(rho, -1.44269504088896340736f, log2f(r.o))) >= 1.f / 255.f;
}

}  // namespace

int main() {
  std::mt19937_64 rng(7);
  auto uni = [&](double a, double b) { return a + (b - a) * (double)(rng() >> 11) * 0x1p-53; };
  for (double ratio : {1.0, 50.0, 1000.0})
    for (double most : {1.5, 1e-2, 1e-3, 1e-4, 1e-5, 1e-6}) {
      long taken = 0, missed = 0;
      for (int s = 0; s < 6000; ++s) {
        // a surfel whose first axis lies across the view ray and whose second is tilted against it by 'tilt'
        const double z = exp(uni(log(2.0), log(300.0)));
        const double pc[3] = {uni(-0.7, 0.7) * z, uni(-0.43, 0.43) * z, z};
        const double n = sqrt(pc[0] * pc[0] + pc[1] * pc[1] + pc[2] * pc[2]);
        const double v[3] = {pc[0] / n, pc[1] / n, pc[2] / n};
        double e1[3] = {1 - v[0] * v[0], -v[0] * v[1], -v[0] * v[2]};
        const double l = sqrt(e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2]);
        for (double& x : e1) x /= l;
        const double e2[3] = {v[1] * e1[2] - v[2] * e1[1], v[2] * e1[0] - v[0] * e1[2], v[0] * e1[1] - v[1] * e1[0]};
        const double turn = uni(0, 6.2831853), tilt = uni(0, 1) * most, spin = s & 1 ? uni(0, 6.2831853) : 0;
        double tu[3], tv[3];
        for (int k = 0; k < 3; ++k) {
          const double u = cos(turn) * e1[k] + sin(turn) * e2[k];
          const double w = cos(tilt) * v[k] + sin(tilt) * (cos(turn) * e2[k] - sin(turn) * e1[k]);
          tu[k] = (float)(cos(spin) * u + sin(spin) * w);
          tv[k] = (float)(cos(spin) * w - sin(spin) * u);
        }
        const double su = exp(uni(log(10.0), log(400.0))) / 3000 * z;
        Record r;
        if (!record(tu, tv, su, su / ratio, pc, uni(0.02, 0.99), r)) continue;
        cgv2::Reach q;
        cgv2::reach_setup(r.a[0] * cgv2::kInvSqrt2, r.a[1] * cgv2::kInvSqrt2, r.a[2] * cgv2::kInvSqrt2,
                          r.a[3] * cgv2::kInvSqrt2, r.w[0], r.w[1], r.w[2], r.k2, q);
        // centre, direction and half length of the conic's long axis
        const long double G00 = q.G00, G01 = q.G01, G11 = q.G11, det = G00 * G11 - G01 * G01;
        if (!(G00 > 0 && G11 > 0 && det > 0)) continue;
        const long double xs = -(G11 * q.b0 - G01 * q.b1) / det, ys = -(G00 * q.b1 - G01 * q.b0) / det;
        const long double most_g = q.d + q.b0 * xs + q.b1 * ys;
        const long double root = sqrtl((G00 - G11) * (G00 - G11) + 4 * G01 * G01);
        const long double half = sqrtl(-most_g * (G00 + G11 + root) / (2 * det));
        const long double angle = 0.5L * atan2l(2 * G01, G00 - G11);
        if (!(half < 2000)) continue;
        for (int j = 0; j < 24; ++j) {
          const double t = uni(-1, 1);
          const double x = (double)(xs - t * half * sinl(angle)), y = (double)(ys + t * half * cosl(angle));
          if (fabs(x) > 2000 || fabs(y) > 2000) continue;
          // the centre that puts pixel sample (px, py) there
          const int px = (int)uni(0, 1600), py = (int)uni(0, 1066), ox = px / 16 * 16, oy = py / 16 * 16;
          r.cx_hi = (float)rint(px + 0.5 - x);
          r.cy_hi = (float)rint(py + 0.5 - y);
          r.cx_lo = (float)(px + 0.5 - x - r.cx_hi);
          r.cy_lo = (float)(py + 0.5 - y - r.cy_hi);
          if (!takes(r, px, py)) continue;
          ++taken;
          const float cx = (r.cx_hi - (float)ox) + r.cx_lo, cy = (r.cy_hi - (float)oy) + r.cy_lo;
          if (!cgv2::reach_cell(q, cx, cy, 0, 0, 16) || !cgv2::reach_cell(q, cx, cy, (px - ox) & 8, (py - oy) & 8, 8))
            ++missed;
        }
      }
      printf("%g %g %ld %ld\n", ratio, most, taken, missed);
    }
}
