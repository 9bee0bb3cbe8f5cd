// Tile renderer: forward (Eq. 1 alpha blending of CityGaussianV2 Sec. 3.1, with the depth,
// median-depth and normal renders of Sec. 3.2 / 5.1) and its reverse.
//
// One 64-lane wave per 16x16 tile.  Lane (x, y) = (lane & 7, lane >> 3) owns one pixel in each 8x8
// quadrant of the tile: (x, y), (x + 8, y), (x, y + 8) and (x + 8, y + 8).  The records of a tile
// list are staged 64 at a time into LDS (one per lane, as five float4), converting the centre to
// tile-relative coordinates exactly ((cx_hi - tile_x0) + cx_lo), pre-scaling the homography
// numerator by 1/sqrt(2) (so rho/2 comes out directly), replacing the opacity by log2(o) and 1/o,
// and reducing the surfel's pixel rect to a 4-bit mask of the quadrants it reaches, less those its
// alpha >= 1/255 region (an ellipse, plus the screen-filter disc) misses.  A quadrant outside the mask
// is skipped wave-uniformly, as is a quadrant whose pixels have all stopped; within a quadrant the
// evaluation is branch-free, and the homography terms of a lane's four pixels are one add apart.  A heavy tile, or
// one of a small launch, runs as halves, quadrants or sixteen 4x4 blocks in waves of their own (tile_of_block).
//
// The reverse walks each pixel's list from its checkpointed 'last' entry downwards, recovers T by
// division, sums the per-surfel gradients of its four pixels in registers, reduces them over the
// wave with a reduce-scatter (row swaps + DPP) and adds them with one atomic instruction per
// (surfel, tile).
#include "cgv2r_device.h"
#include "cgv2r_kernels.h"

#include <algorithm>
#include <type_traits>

namespace cgv2 {

constexpr float kLog2e = 1.44269504088896340736f;

struct RenderArgs {
  const float* rec;
  const uint32_t* ids;
  const uint32_t* ranges;
  const int32_t* status;
  CamPack cams;
  int64_t n;
  int tiles_x, tiles_y, tiles;
  cgv2_image img;
  unsigned long long* counters;
  float* cws;   // contribution mode: [V][n] pairs (sum of alpha^gamma T^(1-gamma), pixel count)
  float gamma;
  const uint32_t* order;  // launch order of this view chunk (heaviest tiles first), or null
  // the first n_b tiles of 'order' run as sixteen 4x4 blocks, the next n_m as sixteen blocks where the tile is long and
  // as four quadrant blocks elsewhere (neither in the counting and contribution passes), the next n_q as four quadrant
  // blocks, the next n_h as two halves
  uint32_t n_b, n_m, n_q, n_h;
};

// Block -> (local view, tile) index and quadrant subset.  Without a launch order: the XCD-aware spatial
// mapping, whole tiles.  With one (the bin_sort's heaviest-first order; bounded, so a stale order cannot
// leave the launch), the n_b heaviest tiles run as sixteen blocks each (bit kBlockBit of sub, the block's
// row-major number below it), the next n_m likewise with kMaybeBit (only the first four here), the next n_q as four
// single-quadrant blocks, the next n_h as two halves (top 0x3, bottom 0xc), the rest whole; then come the other
// twelve of each of the n_m, where the launch's work hides their dispatch if they find nothing to do.  The launch has
// 15 n_b + 15 n_m + 3 n_q + n_h blocks more than tiles.
constexpr uint32_t kBlockBit = 16u, kMaybeBit = 32u;
constexpr uint32_t kLongFwd = 512, kLongFwdHalves = 5, kLongBwd = 256;  // see split_blocks
__device__ __forceinline__ uint32_t tile_of_block(const RenderArgs& a, uint32_t& sub) {
  const uint32_t tiles = gridDim.x - 15u * (a.n_b + a.n_m) - 3u * a.n_q - a.n_h;
  uint32_t bid = blockIdx.x;
  sub = 0xfu;
  if (!a.order) return xcd_remap(bid, tiles);
  const uint32_t late = gridDim.x - 12u * a.n_m;
  uint32_t i;
  if (bid < 16u * a.n_b) {
    i = bid >> 4;
    sub = kBlockBit | (bid & 15u);
  } else if (bid >= late) {
    bid -= late;
    const uint32_t k = bid / 12u;
    i = a.n_b + k;
    sub = kMaybeBit | kBlockBit | (4u + bid - 12u * k);
  } else {
    bid -= 16u * a.n_b;
    const uint32_t n4 = 4u * (a.n_m + a.n_q);
    if (bid < n4) {
      i = bid >> 2;
      sub = i < a.n_m ? kMaybeBit | kBlockBit | (bid & 3u) : 1u << (bid & 3u);
    } else if (bid < n4 + 2u * a.n_h) {
      const uint32_t r = bid - n4;
      i = a.n_m + a.n_q + (r >> 1);
      sub = (r & 1u) ? 0xcu : 0x3u;
    } else {
      i = bid - 3u * (a.n_m + a.n_q) - a.n_h;
    }
    i += a.n_b;
  }
  const uint32_t b = a.order[i];
  return b < tiles ? b : tiles - 1u;
}

// Is tile b's list long: at least 'least' entries and 'halves' / 2 times the mean of the launch?
__device__ __forceinline__ bool long_list(const RenderArgs& a, uint32_t b, uint32_t least, uint32_t halves) {
  const uint32_t all = (uint32_t)a.cams.count * (uint32_t)a.tiles, *r = a.ranges + (int64_t)a.cams.v0 * a.tiles;
  const uint32_t len = r[b + 1] - r[b];
  return len >= least && 2ull * len * all >= (uint64_t)halves * (r[all] - r[0]);
}

// What a block of a kMaybeBit tile does: its block of a long tile, else one quadrant (the first four) or nothing (0).
__device__ __forceinline__ uint32_t maybe_block(uint32_t sub, bool tile_is_long) {
  if (tile_is_long) return sub & ~kMaybeBit;
  return (sub & 15u) < 4u ? 1u << (sub & 3u) : 0u;
}

// LDS record, five float4 (the quadrant masks of the 64 staged entries travel as wave ballots):
//   q0 = (cx, cy, a11 / sqrt2, a12 / sqrt2)     q1 = (a21 / sqrt2, a22 / sqrt2, w0, w1)
//   q2 = (w2, log2 o, z_c, z_c * w0)           q3 = (r, g, b, id)      q4 = (nx, ny, nz, 1 / o)
struct Stage {
  float4 q[64][5];
};

// The 4-bit quadrant masks of the 64 staged entries as nibbles in scalar registers: entry j's mask is
// bits 4 (j % 16) .. 4 (j % 16) + 3 of w[j / 16].  Built with one OR reduction over each row of 16 lanes
// (DPP row shifts) and four lane reads per half; reading one entry's mask is then a shift and a mask.
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_or_in(uint32_t v) {
  return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, false);
}
struct QuadBits {
  uint64_t w[4];
  __device__ __forceinline__ void from_lanes(uint32_t m) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t sh = 4u * (lane & 7u);
    uint32_t lo = (lane & 8u) ? 0u : (m & 0xfu) << sh, hi = (lane & 8u) ? (m & 0xfu) << sh : 0u;
    lo = dpp_or_in<0x111>(lo);  // row_shr:1
    hi = dpp_or_in<0x111>(hi);
    lo = dpp_or_in<0x112>(lo);  // row_shr:2
    hi = dpp_or_in<0x112>(hi);
    lo = dpp_or_in<0x114>(lo);  // row_shr:4
    hi = dpp_or_in<0x114>(hi);
    lo = dpp_or_in<0x118>(lo);  // row_shr:8: lane 15 of each row holds the row's OR
    hi = dpp_or_in<0x118>(hi);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      w[r] = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, 16 * r + 15) << 32 |
             (uint32_t)__builtin_amdgcn_readlane((int)lo, 16 * r + 15);
  }
  // the nibbles of entries 16 i .. 16 i + 15 (i wave-uniform)
  __device__ __forceinline__ uint64_t word(int i) const { return i == 0 ? w[0] : i == 1 ? w[1] : i == 2 ? w[2] : w[3]; }
};

// Quadrants (bits of 'm') in which some pixel sample can reach alpha >= 1/255 (reach_setup / reach_cell).
__device__ __forceinline__ uint32_t reach_quadrants(uint32_t m, const float4& q0, const float4& q1, float w2, float k2) {
  Reach r;
  reach_setup(q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, w2, k2, r);
  uint32_t out = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (((m >> k) & 1u) && reach_cell(r, q0.x, q0.y, 8 * (k & 1), 8 * (k >> 1), 8)) out |= 1u << k;
  return out;
}

// A list entry on its way to LDS: its record, as loaded.  qm: the quadrants the entry may reach (0: its
// record is not read).
struct StageIn {
  float4 r[6];
  uint32_t id, qm;
  bool valid;
};

__device__ __forceinline__ void stage_load(StageIn& in, const float* rec, int64_t vn, int64_t n, uint32_t id,
                                           uint32_t qm) {
  // an id outside [0, n) (never produced by the binning) stages a record that reaches no quadrant
  in.valid = (int64_t)id < n;
  in.id = in.valid ? id : 0u;
  in.qm = qm;
  if (qm == 0u) return;
  const float4* r = (const float4*)(rec + (size_t)(vn + in.id) * kRec);
#pragma unroll
  for (int k = 0; k < 6; ++k) in.r[k] = r[k];
}

// Writes the entry's LDS record and returns its mask among the quadrants in.qm: those its pixel rect
// meets and, with 'reach', that some pixel sample of the surfel can reach (reach_quadrants; without it
// in.qm is the forward's mask of the quadrants with a contributing pixel).
// kBlock: instead, whether the pixel rect meets the 4x4 block at (bx, by) of a reached quadrant.
template <bool kBlock = false>
__device__ __forceinline__ uint32_t stage_put(Stage& s, int lane, const StageIn& in, int ox, int oy, bool reach,
                                              int bx = 0, int by = 0) {
  // an entry no pixel takes reaches no quadrant here
  if (in.qm == 0u) return 0u;
  const float4 r0 = in.r[0], r1 = in.r[1], r2 = in.r[2], r3 = in.r[3], r4 = in.r[4], r5 = in.r[5];
  const float fox = (float)ox, foy = (float)oy;
  const float4 q0 = make_float4((r0.x - fox) + r0.z, (r0.y - foy) + r0.w, r1.x * kInvSqrt2, r1.y * kInvSqrt2);
  const float4 q1 = make_float4(r1.z * kInvSqrt2, r1.w * kInvSqrt2, r2.x, r2.y);
  s.q[lane][0] = q0;
  s.q[lane][1] = q1;
  s.q[lane][2] = make_float4(r2.z, in.valid ? log2f(r3.x) : -INFINITY, r2.w, r2.w * r2.x);
  s.q[lane][3] = make_float4(r3.y, r3.z, r3.w, __uint_as_float(in.id));
  s.q[lane][4] = make_float4(r4.x, r4.y, r4.z, in.valid ? 1.f / r3.x : 0.f);
  // pixel rect relative to the tile origin
  const uint32_t px = __float_as_uint(r5.x), py = __float_as_uint(r5.y);
  const int i0 = (int)(px & 0xffffu) - ox, i1 = (int)(px >> 16) - ox;
  const int j0 = (int)(py & 0xffffu) - oy, j1 = (int)(py >> 16) - oy;
  uint32_t m = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int x0 = 8 * (k & 1), y0 = 8 * (k >> 1);
    if (i0 <= x0 + 7 && i1 >= x0 && j0 <= y0 + 7 && j1 >= y0) m |= 1u << k;
  }
  m &= in.qm;
  if (kBlock && !(i0 <= bx + 3 && i1 >= bx && j0 <= by + 3 && j1 >= by)) m = 0u;
  if (reach && m) m = reach_quadrants(m, q0, q1, r2.z, r4.w);
  return in.valid ? m : 0u;
}

__device__ __forceinline__ uint32_t stage_record(Stage& s, int lane, const float* rec, int64_t vn, int64_t n,
                                                 uint32_t id, uint32_t qm, int ox, int oy, bool reach) {
  // an entry no pixel of the forward took reaches no quadrant here: its record is not read at all
  if (qm == 0u) return 0u;
  StageIn in;
  stage_load(in, rec, vn, n, id, qm);
  return stage_put(s, lane, in, ox, oy, reach);
}

// Per-surfel terms of a lane at its quadrant-0 pixel; pixel k sits at (xr0 + 8 (k & 1), yr0 + 8 (k >> 1))
// relative to the projected centre (xr1 = xr0 + 8, yr1 = yr0 + 8).
// (c1x, c1y, c2x, c2y, cwx, cwy) are the coefficients of x' and y' in P1, P2 and w: a pixel 8 columns or
// rows further adds 8 times them (exact in FP32, so one FMA per term).
struct LaneTerms {
  float xr0, yr0, xr1, yr1, p1, p2, wb, c1x, c1y, c2x, c2y, cwx, cwy;
};

__device__ __forceinline__ void lane_terms(float lx0, float ly0, const float4& q0, const float4& q1, const float4& q2,
                                           LaneTerms& t) {
  t.xr0 = lx0 - q0.x;
  t.yr0 = ly0 - q0.y;
  t.xr1 = t.xr0 + 8.f;
  t.yr1 = t.yr0 + 8.f;
  t.p1 = fmaf(q0.z, t.xr0, q0.w * t.yr0);
  t.p2 = fmaf(q1.x, t.xr0, q1.y * t.yr0);
  t.wb = fmaf(q1.w, t.xr0, fmaf(q2.x, t.yr0, q1.z));
  t.c1x = q0.z;
  t.c1y = q0.w;
  t.c2x = q1.x;
  t.c2y = q1.y;
  t.cwx = q1.w;
  t.cwy = q2.x;
}

// Evaluation of one staged surfel at pixel k of a lane, shared by the forward and the reverse so that
// both take bit-identical decisions.  rho is half the Mahalanobis-type distance:
// rho = min(rho_3d, rho_2d) / 2, alpha_raw = o exp(-rho).
struct Px {
  float xr, yr, P1, P2, w, iw, rho, arg, araw, alpha;
  bool is3d;
};

template <int k>
__device__ __forceinline__ void eval_px(const LaneTerms& t, float lo, Px& e) {
  e.xr = (k & 1) ? t.xr1 : t.xr0;
  e.yr = (k >> 1) ? t.yr1 : t.yr0;
  e.P1 = t.p1;
  e.P2 = t.p2;
  e.w = t.wb;
  if (k & 1) {
    e.P1 = fmaf(8.f, t.c1x, e.P1);
    e.P2 = fmaf(8.f, t.c2x, e.P2);
    e.w = fmaf(8.f, t.cwx, e.w);
  }
  if (k >> 1) {
    e.P1 = fmaf(8.f, t.c1y, e.P1);
    e.P2 = fmaf(8.f, t.c2y, e.P2);
    e.w = fmaf(8.f, t.cwy, e.w);
  }
  const float r2 = fmaf(e.xr, e.xr, e.yr * e.yr);
  const float nn = fmaf(e.P1, e.P1, e.P2 * e.P2);
  // w == 0: the ray runs parallel to the plane; rcp gives inf (or NaN for nn == 0) and the
  // comparison below then selects the screen filter
  e.iw = __builtin_amdgcn_rcpf(e.w);
  const float r3 = nn * (e.iw * e.iw);
  e.is3d = r3 <= r2;
  e.rho = e.is3d ? r3 : r2;
  e.arg = fmaf(e.rho, -kLog2e, lo);  // log2(alpha_raw)
  e.araw = __builtin_amdgcn_exp2f(e.arg);
  e.alpha = fminf(kAlphaMax, e.araw);
}

__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// T carries the pixel's state in its sign: T > 0 while the pixel runs (T >= 1e-4 then), -T once it has
// stopped (or lies outside the image); the transmittance itself is |T|.  'last' holds the index of the
// last entry blended (start - 1 before the first); the image stores last + 1.
struct FwdState {
  float T, C[3], D, Dm, N[3];
  uint32_t last, med;
};

// The entry index as a per-lane register, for the selects of 'last' and 'med' (which cannot take it from
// a scalar register next to their lane mask).
__device__ __forceinline__ uint32_t lane_copy(uint32_t x) {
  uint32_t v;
  asm("v_mov_b32 %0, %1" : "=v"(v) : "s"(x));
  return v;
}

// Returns false when no pixel of the quadrant takes the entry (wave-uniform); true otherwise, which
// covers every entry with a contributing fragment (a superset is all the reverse pass needs).
// kContrib: also add the fragment's alpha^gamma T^(1-gamma) (T in front of it) to csum and the quadrant's
// number of blended pixels to ccnt.  kHalfGamma (the usual gamma = 1/2) is sqrt(alpha T): one transcendental
// instead of two.
constexpr float kLog2AlphaMax = -0.014499569695115089f;  // log2(0.99)

enum : int { kNoContrib = 0, kAnyGamma = 1, kHalfGamma = 2 };

template <int kContrib>
__device__ __forceinline__ bool fwd_px(const Px& e, const float4& q2, const float4& q3, const float4& q4,
                                       uint32_t e_idx, FwdState& f, unsigned long long& n_con, float gamma,
                                       float& csum, uint32_t& ccnt) {
  // wave-uniform skip when no pixel of the quadrant takes this surfel; otherwise branch-free: a
  // contribution is a zero-weight no-op for pixels that skip or stop here
  const bool take = f.T > 0.f && e.alpha >= kAlphaMin;
  if (__ballot(take) == 0) return false;
  // Tn is used only where the pixel takes the entry
  const float Tn = f.T * (1.f - e.alpha);
  const bool upd = take && !(Tn < kTmin);
  n_con += upd ? 1u : 0u;
  if (kContrib) {
    float c;
    if (kContrib == kHalfGamma) {
      c = __builtin_amdgcn_sqrtf(e.alpha * f.T);
    } else {
      // log2(alpha) = min(log2(alpha_raw), log2(0.99))
      const float la = fminf(e.arg, kLog2AlphaMax);
      c = __builtin_amdgcn_exp2f(fmaf(gamma, la, (1.f - gamma) * __builtin_amdgcn_logf(f.T)));
    }
    csum += upd ? c : 0.f;
    ccnt += (uint32_t)__popcll(__ballot(upd));
  }
  const float wgt = upd ? e.alpha * f.T : 0.f;
  const float zf = e.is3d ? q2.w * e.iw : q2.z;
  f.C[0] = fmaf(wgt, q3.x, f.C[0]);
  f.C[1] = fmaf(wgt, q3.y, f.C[1]);
  f.C[2] = fmaf(wgt, q3.z, f.C[2]);
  f.N[0] = fmaf(wgt, q4.x, f.N[0]);
  f.N[1] = fmaf(wgt, q4.y, f.N[1]);
  f.N[2] = fmaf(wgt, q4.z, f.N[2]);
  f.D = fmaf(wgt, zf, f.D);
  const bool m = upd && f.T > 0.5f;
  f.Dm = m ? zf : f.Dm;
  f.med = m ? e_idx : f.med;
  f.last = upd ? e_idx : f.last;
  // a pixel that takes the entry but would fall below 1e-4 stops in front of it
  f.T = upd ? Tn : (take ? -f.T : f.T);
  return true;
}

// Quadrants (of the subset kSub) with a running pixel (wave-uniform bit mask).
template <uint32_t kSub>
__device__ __forceinline__ uint32_t live_quadrants(const FwdState (&f)[4]) {
  uint32_t m = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if ((kSub >> k) & 1u) m |= (__ballot(f[k].T > 0.f) != 0 ? 1u : 0u) << k;
  return m;
}

// Forward of the quadrants kSub of one tile (bit k: 8x8 quadrant k).  kSub = 0xf is the whole tile, a lane
// holding one pixel in each quadrant; a heavy tile runs as two halves (0x3, 0xc) or four single quadrants
// in separate waves.  Every subset runs the per-quadrant arithmetic of the whole tile (eval_px<k> from
// the lane terms at the quadrant-0 pixel), so the decisions do not depend on the split.  The reverse
// pass's per-entry quadrant bits go to img.qmask: a plain byte store for a whole tile, an atomic OR on
// the entry's word for a split one (its waves share the byte, which is cleared before the launch).
// kCount: instead of images, count the (pixel, list entry) pairs of the method (every entry a running
// pixel meets, quadrant mask or not), the contributing pairs, and the pairs the reverse walks.
// kContrib: instead of images, add each surfel's contribution sums (Sec. 3.3, Eq. 3) of this view into
// a.cws, one wave reduction and one atomic pair per (surfel, tile or split block).
template <bool kCount, bool kMask, int kContrib, uint32_t kSub>
__device__ __forceinline__ void render_fwd_tile(const RenderArgs& a, Stage& s, uint32_t b) {
  const int lv = (int)(b / (uint32_t)a.tiles);
  const int v = a.cams.v0 + lv;
  const int t = (int)(b % (uint32_t)a.tiles);
  const int tx = t % a.tiles_x, ty = t / a.tiles_x;
  const DevCam& c = a.cams.c[lv];
  const int W = c.W, H = c.H;
  const int lane = threadIdx.x;
  const int lx = lane & 7, ly = lane >> 3;
  const int ox = tx * kTile, oy = ty * kTile;
  const uint32_t start = a.ranges[(int64_t)v * a.tiles + t], end = a.ranges[(int64_t)v * a.tiles + t + 1];
  const int64_t vn = (int64_t)v * a.n;
  constexpr bool kOne = (kSub & (kSub - 1u)) == 0u;  // a single quadrant

  FwdState f[4];
  unsigned long long n_eval = 0, n_con = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int px = ox + lx + 8 * (k & 1), py = oy + ly + 8 * (k >> 1);
    f[k].T = ((kSub >> k) & 1u) && px < W && py < H ? 1.f : -1.f;
    f[k].D = 0.f;
    f[k].Dm = 0.f;
    f[k].last = start - 1u;
    f[k].med = 0xffffffffu;
    f[k].C[0] = f[k].C[1] = f[k].C[2] = 0.f;
    f[k].N[0] = f[k].N[1] = f[k].N[2] = 0.f;
  }
  const float lx0 = (float)lx + 0.5f, ly0 = (float)ly + 0.5f;
  uint8_t* qmask = kMask ? a.img.qmask : nullptr;
  uint32_t qlive = live_quadrants<kSub>(f);
  // the list ids of the next chunk are loaded one chunk ahead: staging then waits on one load round trip
  // (the records) instead of two
  uint32_t nid = start + lane < end ? a.ids[start + lane] : 0u;
  [[maybe_unused]] StageIn in;
  if constexpr (kOne) {
    stage_load(in, a.rec, vn, a.n, nid, start + lane < end ? kSub : 0u);
    nid = start + 64u + lane < end ? a.ids[start + 64u + lane] : 0u;
  }
  for (uint32_t base = start; base < end && qlive != 0; base += 64) {
    const uint32_t idx = base + lane;
    uint32_t m4;
    if constexpr (!kOne) {
      m4 = stage_record(s, lane, a.rec, vn, a.n, nid, idx < end ? kSub : 0u, ox, oy, true);
      nid = idx + 64u < end ? a.ids[idx + 64u] : 0u;
    } else {
      m4 = stage_put(s, lane, in, ox, oy, true);
      // a quadrant block holds one pixel's state per lane, so there are registers for the next chunk's
      // records too: their round trip runs under this chunk's entries
      stage_load(in, a.rec, vn, a.n, nid, idx + 64u < end ? kSub : 0u);
      nid = idx + 128u < end ? a.ids[idx + 128u] : 0u;
    }
    __syncthreads();
    const int cnt = (int)min(64u, end - base);
    int reached = cnt;  // entries of this chunk the wave evaluated
    // bit j of cq[k]: quadrant k had a taking pixel at entry base + j (scalar registers)
    uint64_t cq[4] = {0, 0, 0, 0};
    auto entry = [&](int j, uint32_t m) {
      const float4 q0 = s.q[j][0], q1 = s.q[j][1], q2 = s.q[j][2], q3 = s.q[j][3], q4 = s.q[j][4];
      LaneTerms lt;
      lane_terms(lx0, ly0, q0, q1, q2, lt);
      const uint32_t e_idx = lane_copy(base + (uint32_t)j);
      float csum = 0.f;
      uint32_t ccnt = 0;  // wave-uniform
      bool took = false;
      Px e[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (!((kSub >> k) & 1u)) continue;
        // (evaluated where it is used: the compiler sinks each pixel's evaluation into its branch)
        if (k == 0) eval_px<0>(lt, q2.y, e[0]);
        if (k == 1) eval_px<1>(lt, q2.y, e[1]);
        if (k == 2) eval_px<2>(lt, q2.y, e[2]);
        if (k == 3) eval_px<3>(lt, q2.y, e[3]);
        if (((m >> k) & 1u) && fwd_px<kContrib>(e[k], q2, q3, q4, e_idx, f[k], n_con, a.gamma, csum, ccnt)) {
          took = true;
          if (kMask) cq[k] |= 1ull << j;
        }
      }
      if (kContrib && took && ccnt != 0) {
        // the sum from lane 63, the count from lane 62: one atomic instruction
        const float ts = wave_sum_lane63(csum);
        if (lane >= 62)
          atomicAdd(a.cws + 2 * (vn + (int64_t)__float_as_uint(q3.w)) + (63 - lane), lane == 63 ? ts : (float)ccnt);
      }
    };
    if constexpr (kOne && !kCount) {
      // one quadrant: walk the set bits of its ballot
      uint64_t todo = __ballot((m4 & kSub) != 0u);
      for (int seen = 1; todo != 0; ++seen) {
        const int j = __builtin_ctzll(todo);
        todo &= todo - 1;
        entry(j, kSub);
        if ((seen & 15) == 0 && live_quadrants<kSub>(f) == 0) {
          reached = j + 1;
          break;
        }
      }
    } else {
      QuadBits qb;
      qb.from_lanes(m4);
      uint64_t cur = qb.w[0];  // entry j's nibble in bits 0-3
      for (int j = 0; j < cnt; ++j) {
        if (kCount) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if ((kSub >> k) & 1u) n_eval += f[k].T > 0.f ? 1u : 0u;
        }
        const uint32_t m = (uint32_t)cur & 0xfu & qlive;
        cur >>= 4;
        if (m != 0) entry(j, m);
        if ((j & 15) == 15) {
          qlive = live_quadrants<kSub>(f);
          if (qlive == 0) {
            reached = j + 1;
            break;
          }
          cur = qb.word((j + 1) >> 4);
        }
      }
    }
    // entries past 'reached' lie beyond every pixel's 'last': the reverse pass never reads them
    if (kMask && lane < reached) {
      const uint32_t bits = (uint32_t)((cq[0] >> lane) & 1u) | (uint32_t)((cq[1] >> lane) & 1u) << 1 |
                            (uint32_t)((cq[2] >> lane) & 1u) << 2 | (uint32_t)((cq[3] >> lane) & 1u) << 3;
      if (kSub == 0xfu) qmask[idx] = (uint8_t)bits;
      else if (bits) atomicOr((uint32_t*)(qmask + (idx & ~3u)), bits << (8u * (idx & 3u)));
    }
    qlive = live_quadrants<kSub>(f);
    __syncthreads();
  }
  if (kContrib) return;
  if (kCount) {
    unsigned long long n_bwd = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int px = ox + lx + 8 * (k & 1), py = oy + ly + 8 * (k >> 1);
      if (((kSub >> k) & 1u) && px < W && py < H) n_bwd += f[k].last + 1u - start;
    }
    atomicAdd(a.counters + 0, n_eval);
    atomicAdd(a.counters + 1, n_con);
    atomicAdd(a.counters + 2, n_bwd);
    return;
  }
  const int64_t HW = (int64_t)W * H;
  const cgv2_image& im = a.img;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int px = ox + lx + 8 * (k & 1), py = oy + ly + 8 * (k >> 1);
    if (!((kSub >> k) & 1u) || !(px < W && py < H)) continue;
    const int64_t p = (int64_t)py * W + px;
    const float T = fabsf(f[k].T);
    if (im.rgb) {
      float* o = im.rgb + (int64_t)v * 3 * HW + p;
      o[0] = fmaf(T, c.bg[0], f[k].C[0]);
      o[HW] = fmaf(T, c.bg[1], f[k].C[1]);
      o[2 * HW] = fmaf(T, c.bg[2], f[k].C[2]);
    }
    if (im.normal) {
      float* o = im.normal + (int64_t)v * 3 * HW + p;
      o[0] = f[k].N[0];
      o[HW] = f[k].N[1];
      o[2 * HW] = f[k].N[2];
    }
    const int64_t vp = (int64_t)v * HW + p;
    if (im.depth) im.depth[vp] = f[k].D;
    if (im.depth_med) im.depth_med[vp] = f[k].Dm;
    if (im.alpha) im.alpha[vp] = 1.f - T;
    if (im.T_final) im.T_final[vp] = T;
    if (im.last) im.last[vp] = f[k].last + 1u;
    if (im.med) im.med[vp] = f[k].med;
  }
}

// Quad-lane broadcast of lane s's value (0 to 3).
template <int s>
__device__ __forceinline__ float quad_lane(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), s * 0x55, 0xf, 0xf, true));
}
template <int kCtrl>
__device__ __forceinline__ float quad_swap(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), kCtrl, 0xf, 0xf, true));
}

// Forward of one 4x4 block (of quadrant k) of a heavy tile or of a small launch.  The walk of a long list is one chain of dependent
// entries, bound by the wave's own instruction issue, and its small surfels meet few blocks; here the four lanes of
// a pixel evaluate four entries of the block's list at a time, the transmittance runs through them by quad-lane
// broadcasts, and each lane adds two of the images' channels over the four: every operation and its order are those
// of the tile's walk, bit for bit.
template <bool kMask, int k>
__device__ __forceinline__ void render_fwd_block(const RenderArgs& a, Stage& s, uint32_t b, int bx, int by) {
  const int lv = (int)(b / (uint32_t)a.tiles);
  const int v = a.cams.v0 + lv;
  const int t = (int)(b % (uint32_t)a.tiles);
  const DevCam& c = a.cams.c[lv];
  const int W = c.W, H = c.H;
  const int lane = threadIdx.x, part = lane & 3;
  const int ox = t % a.tiles_x * kTile, oy = t / a.tiles_x * kTile;
  const int px = ox + bx + ((lane >> 2) & 3), py = oy + by + (lane >> 4);
  const uint32_t start = a.ranges[(int64_t)v * a.tiles + t], end = a.ranges[(int64_t)v * a.tiles + t + 1];
  const int64_t vn = (int64_t)v * a.n;
  const bool inside = px < W && py < H;
  // the pixel of quadrant 0 whose terms the evaluation starts from
  const float lx0 = (float)(px - ox - 8 * (k & 1)) + 0.5f, ly0 = (float)(py - oy - 8 * (k >> 1)) + 0.5f;

  float T = inside ? 1.f : -1.f;  // as FwdState's, the same in the pixel's four lanes
  float A0 = 0.f, A1 = 0.f;       // lane 0: r, g; 1: b, depth; 2: nx, ny; 3: nz
  float Dm = 0.f;
  uint32_t last = start, med = 0;  // one past the entry
  uint32_t nid = start + lane < end ? a.ids[start + lane] : 0u;
  StageIn in;
  stage_load(in, a.rec, vn, a.n, nid, start + lane < end ? 1u << k : 0u);
  nid = start + 64u + lane < end ? a.ids[start + 64u + lane] : 0u;
  bool live = __ballot(T > 0.f) != 0;
  for (uint32_t base = start; base < end && live; base += 64) {
    const uint32_t idx = base + lane;
    const bool here = stage_put<true>(s, lane, in, ox, oy, true, bx, by) != 0u;
    uint64_t todo = __ballot(here);
    // Entries of an infinite colour (colours are never negative or NaN) are taken alone: zero times it is not zero, so
    // one that no pixel takes may not share in the others' sums.
    const uint64_t inf = __ballot(here && !(in.r[3].y + in.r[3].z + in.r[3].w < INFINITY));
    stage_load(in, a.rec, vn, a.n, nid, idx + 64u < end ? 1u << k : 0u);
    nid = idx + 128u < end ? a.ids[idx + 128u] : 0u;
    __syncthreads();
    uint64_t cq = 0;
    while (todo != 0) {
      int at[4];
      bool has[4];
      uint64_t now = todo;
      if (inf != 0) {
        const uint64_t first = todo & (0ull - todo), next = todo & inf;
        now = (first & inf) ? first : todo & ((next & (0ull - next)) - 1ull);
      }
      todo &= ~now;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        has[q] = now != 0;
        at[q] = has[q] ? __builtin_ctzll(now) : at[0];
        now &= now - 1;
      }
      todo |= now;
      const int j = part == 0 ? at[0] : part == 1 ? at[1] : part == 2 ? at[2] : at[3];
      const bool act = part == 0 || (part == 1 ? has[1] : part == 2 ? has[2] : has[3]);
      const float4 q0 = s.q[j][0], q1 = s.q[j][1], q2 = s.q[j][2];
      float2 ch[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) ch[q] = ((const float2*)&s.q[at[q]][3])[part];
      LaneTerms lt;
      lane_terms(lx0, ly0, q0, q1, q2, lt);
      Px e;
      eval_px<k>(lt, q2.y, e);
      bool upd = act && T > 0.f && e.alpha >= kAlphaMin;
      const uint64_t taken = __ballot(upd);
      if (taken == 0) continue;
      if (kMask) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (taken & (0x1111111111111111ull << q)) cq |= 1ull << at[q];
      }
      const float al = upd ? e.alpha : 0.f;
      const float om = 1.f - al;
      const float o0 = quad_lane<0>(om), o1 = quad_lane<1>(om), o2 = quad_lane<2>(om), o3 = quad_lane<3>(om);
      const float T1 = T * o0, T2 = T1 * o1, T3 = T2 * o2, T4 = T3 * o3;
      float Tf = part == 0 ? T : part == 1 ? T1 : part == 2 ? T2 : T3;  // in front of this lane's entry
      if (__ballot(T > 0.f && T4 < kTmin) == 0) {
        T = T4;
      } else {
        // some pixel stops within these entries: one after the other
        float cur = T;
        auto step = [&](int q, float o) {
          const float Tn = cur * o;
          const bool takes = cur > 0.f && o < 1.f, stops = Tn < kTmin;
          if (part == q) {
            Tf = cur;
            upd = upd && takes && !stops;
          }
          cur = takes ? (stops ? -cur : Tn) : cur;
        };
        step(0, o0);
        step(1, o1);
        step(2, o2);
        step(3, o3);
        T = cur;
        live = __ballot(T > 0.f) != 0;
        if (!live) todo = 0;
      }
      const float wgt = upd ? al * Tf : 0.f;
      const float zf = e.is3d ? q2.w * e.iw : q2.z;
      auto add = [&](const float2& x, float w, float z) {
        A0 = fmaf(w, x.x, A0);
        A1 = fmaf(w, part == 1 ? z : x.y, A1);
      };
      add(ch[0], quad_lane<0>(wgt), quad_lane<0>(zf));
      add(ch[1], quad_lane<1>(wgt), quad_lane<1>(zf));
      add(ch[2], quad_lane<2>(wgt), quad_lane<2>(zf));
      add(ch[3], quad_lane<3>(wgt), quad_lane<3>(zf));
      const uint32_t next = base + (uint32_t)j + 1u;
      const bool m = upd && Tf > 0.5f;
      Dm = m ? zf : Dm;
      med = m ? next : med;
      last = upd ? next : last;
    }
    if (kMask && ((cq >> lane) & 1u))
      atomicOr((uint32_t*)(a.img.qmask + (idx & ~3u)), (1u << k) << (8u * (idx & 3u)));
    __syncthreads();
  }
  // the latest of the four lanes' entries
  auto over = [&](auto ctrl) {
    constexpr int kC = decltype(ctrl)::value;
    const float od = quad_swap<kC>(Dm);
    const uint32_t om = __float_as_uint(quad_swap<kC>(__uint_as_float(med)));
    Dm = om > med ? od : Dm;
    med = max(med, om);
    last = max(last, __float_as_uint(quad_swap<kC>(__uint_as_float(last))));
  };
  over(std::integral_constant<int, 0xb1>{});  // lanes 1 0 3 2
  over(std::integral_constant<int, 0x4e>{});  // lanes 2 3 0 1
  if (!inside) return;
  const int64_t HW = (int64_t)W * H;
  const cgv2_image& im = a.img;
  const int64_t p = (int64_t)py * W + px, vp = (int64_t)v * HW + p;
  T = fabsf(T);
  float* o = part < 2 ? im.rgb : im.normal;
  if (o) {
    o += (int64_t)v * 3 * HW + p + (part & 1 ? 2 * HW : 0);
    o[0] = part < 2 ? fmaf(T, c.bg[part == 0 ? 0 : 2], A0) : A0;
    if (!(part & 1)) o[HW] = part < 2 ? fmaf(T, c.bg[1], A1) : A1;
  }
  if (part == 1 && im.depth) im.depth[vp] = A1;
  if (part != 0) return;
  if (im.depth_med) im.depth_med[vp] = Dm;
  if (im.alpha) im.alpha[vp] = 1.f - T;
  if (im.T_final) im.T_final[vp] = T;
  if (im.last) im.last[vp] = last;
  if (im.med) im.med[vp] = med - 1u;
}

template <bool kCount, bool kMask, int kContrib>
__global__ __launch_bounds__(64) void k_render_fwd(RenderArgs a) {
  __shared__ Stage s;
  uint32_t sub;
  const uint32_t b = tile_of_block(a, sub);
  if (*a.status != 0) return;
  if constexpr (!kCount && kContrib == kNoContrib) {
    if (sub & kMaybeBit) {
      sub = maybe_block(sub, long_list(a, b, kLongFwd, kLongFwdHalves));
      if (sub == 0u) return;
    }
    if (sub & kBlockBit) {
      const int bx = 4 * (int)(sub & 3u), by = (int)(sub & 12u);
      switch ((bx >> 3) + 2 * (by >> 3)) {
        case 0: render_fwd_block<kMask, 0>(a, s, b, bx, by); break;
        case 1: render_fwd_block<kMask, 1>(a, s, b, bx, by); break;
        case 2: render_fwd_block<kMask, 2>(a, s, b, bx, by); break;
        default: render_fwd_block<kMask, 3>(a, s, b, bx, by); break;
      }
      return;
    }
  }
  switch (sub) {
    case 0x1u: render_fwd_tile<kCount, kMask, kContrib, 0x1u>(a, s, b); break;
    case 0x2u: render_fwd_tile<kCount, kMask, kContrib, 0x2u>(a, s, b); break;
    case 0x4u: render_fwd_tile<kCount, kMask, kContrib, 0x4u>(a, s, b); break;
    case 0x8u: render_fwd_tile<kCount, kMask, kContrib, 0x8u>(a, s, b); break;
    case 0x3u: render_fwd_tile<kCount, kMask, kContrib, 0x3u>(a, s, b); break;
    case 0xcu: render_fwd_tile<kCount, kMask, kContrib, 0xcu>(a, s, b); break;
    default: render_fwd_tile<kCount, kMask, kContrib, 0xfu>(a, s, b); break;
  }
}

struct BwdArgs {
  RenderArgs r;
  cgv2_image_grad up;
  RecGrads rg;
};

__device__ __forceinline__ float ldg0(const float* p, int64_t i) { return p ? p[i] : 0.f; }

// Per-pixel state of the reverse walk.  The upstream gradients are held multiplied by -2 (exact), which
// makes 2 d rho come out of the chain directly (rho is half the distance, and d alpha_raw / d rho =
// -alpha_raw); the fields that take them linearly (colour, normal, opacity) are scaled back once per
// (surfel, tile) at the atomics.  Instead of the colour (normal, depth) sums of the fragments behind,
// the walk keeps their dot products with the upstream gradients: sA for the total upstream, sS for the
// SSIM-only one; the background (and the alpha-image term) starts them.
struct BwdState {
  float T, sA, sS, GC[3], GS[3], GN[3], GD2, GD, GM;
  uint32_t last, med;
};

// Pixel (px, py) of view v: its checkpoint (T, last, median id) and upstream gradients.
template <bool kGeom>
__device__ __forceinline__ void bwd_init(const BwdArgs& A, const DevCam& c, int v, int px, int py, uint32_t start,
                                         uint32_t end, BwdState& p) {
  const int W = c.W, H = c.H;
  const int64_t HW = (int64_t)W * H;
  const bool in = px < W && py < H;
  const int64_t pp = in ? (int64_t)py * W + px : 0;
  const int64_t vp = (int64_t)v * HW + pp;
  const int64_t v3 = (int64_t)v * 3 * HW + pp;
  p.last = in ? min(max(A.r.img.last[vp], start), end) : start;
  p.med = in ? A.r.img.med[vp] : 0xffffffffu;
  const float Tf = in ? A.r.img.T_final[vp] : 1.f;
  p.T = Tf;
  float bA = 0.f, bS = 0.f;
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) {
    p.GC[ch] = -2.f * (in ? ldg0(A.up.d_rgb, v3 + ch * HW) : 0.f);
    p.GS[ch] = -2.f * (in ? ldg0(A.up.d_rgb_ssim, v3 + ch * HW) : 0.f);
    p.GN[ch] = -2.f * (kGeom && in ? ldg0(A.up.d_normal, v3 + ch * HW) : 0.f);
    bA = fmaf(p.GC[ch], c.bg[ch], bA);
    bS = fmaf(p.GS[ch], c.bg[ch], bS);
  }
  p.GD = kGeom && in ? ldg0(A.up.d_depth, vp) : 0.f;
  p.GM = kGeom && in ? ldg0(A.up.d_depth_med, vp) : 0.f;
  p.GD2 = -2.f * p.GD;
  // alpha = 1 - T_final: d alpha / d alpha_i = T_final / (1 - alpha_i), the same factor as the blend terms
  const float GA = kGeom && in ? ldg0(A.up.d_alpha, vp) : 0.f;
  p.sA = fmaf(2.f * GA, Tf, Tf * bA);
  p.sS = Tf * bS;
}

// What a pixel takes from a staged surfel, before its transmittance and sums come in.
struct BwdTake {
  float rom, ar, g, gs, zf;  // 1 / (1 - alpha), alpha / (1 - alpha), upstream . attributes (total, SSIM-only), depth
  bool con;
};

template <bool kGeom>
__device__ __forceinline__ void bwd_take(const Px& e, bool con, const float4& q2, const float4& q3, const float4& q4,
                                         const BwdState& p, BwdTake& t) {
  t.con = con;
  const float al = con ? e.alpha : 0.f;
  t.rom = __builtin_amdgcn_rcpf(1.f - al);
  t.ar = al * t.rom;
  t.g = fmaf(p.GC[0], q3.x, fmaf(p.GC[1], q3.y, p.GC[2] * q3.z));
  t.gs = fmaf(p.GS[0], q3.x, fmaf(p.GS[1], q3.y, p.GS[2] * q3.z));
  t.zf = 0.f;
  if (kGeom) {
    t.zf = e.is3d ? q2.w * e.iw : q2.z;
    t.g = fmaf(p.GN[0], q4.x, t.g);
    t.g = fmaf(p.GN[1], q4.y, t.g);
    t.g = fmaf(p.GN[2], q4.z, t.g);
    t.g = fmaf(p.GD2, t.zf, t.g);
  }
}

// Its share of the record gradients: wgt = alpha T, nA and nS = 2 (1 - alpha) dL/dalpha of the total and the SSIM-only
// upstream (what lies behind minus T in front times this fragment's attributes).
// acc[G_OP] collects 2 d rho (the opacity gradient is -alpha_raw d rho / o, formed at the atomics);
// acc[G_R..G_B] and the normal sums collect -2 times their gradients.
template <bool kGeom>
__device__ __forceinline__ void bwd_terms(const Px& e, const BwdTake& t, const float4& q0, const float4& q1,
                                          const float4& q2, uint32_t e_idx, const BwdState& p, float wgt, float nA,
                                          float nS, float (&acc)[kGradFields]) {
  const float a11 = q0.z, a12 = q0.w, a21 = q1.x, a22 = q1.y, w0 = q1.z, w1 = q1.w, w2 = q2.x;
  const float zc = q2.z;
  // d alpha / d alpha_raw / (1 - alpha): the 0.99 clamp blocks the path to o and rho; below it alpha is
  // alpha_raw, and a pixel that does not take the entry has al = 0
  const float rA = e.araw > kAlphaMax ? 0.f : t.ar;
  acc[G_R] = fmaf(p.GC[0], wgt, acc[G_R]);
  acc[G_G] = fmaf(p.GC[1], wgt, acc[G_G]);
  acc[G_B] = fmaf(p.GC[2], wgt, acc[G_B]);
  float dz = 0.f;
  if (kGeom) {
    acc[G_NX] = fmaf(p.GN[0], wgt, acc[G_NX]);
    acc[G_NY] = fmaf(p.GN[1], wgt, acc[G_NY]);
    acc[G_NZ] = fmaf(p.GN[2], wgt, acc[G_NZ]);
    dz = fmaf(p.GD, wgt, t.con && e_idx == p.med ? p.GM : 0.f);
  }
  // -2 d rho of either upstream
  const float ndr = rA * nA;
  const float nds = rA * nS;
  acc[G_OP] -= ndr;
  // (vx, vy) = d rho / d(x', y') / 2: the centre gradient of either upstream is -2 d rho * (vx, vy)
  float vx, vy;
  if (e.is3d) {
    // rho = |P|^2 / (2 w^2) with P = (P1, P2), so d rho = (P . dP) / w^2 - 2 rho dw / w
    const float iw = e.iw, iww = iw * iw;
    const float u1 = e.P1 * iww, u2 = e.P2 * iww, uw = e.rho * iw;
    const float nP1 = ndr * u1, nP2 = ndr * u2;
    // the intersection depth z_c w0 / w also depends on w
    const float dzw = kGeom ? dz * t.zf * iw : 0.f;
    const float gw = kGeom ? fmaf(ndr, uw, -dzw) : ndr * uw;
    acc[G_A11] = fmaf(-nP1, e.xr, acc[G_A11]);
    acc[G_A12] = fmaf(-nP1, e.yr, acc[G_A12]);
    acc[G_A21] = fmaf(-nP2, e.xr, acc[G_A21]);
    acc[G_A22] = fmaf(-nP2, e.yr, acc[G_A22]);
    acc[G_W0] += kGeom ? fmaf(dz * zc, iw, gw) : gw;
    acc[G_W1] = fmaf(gw, e.xr, acc[G_W1]);
    acc[G_W2] = fmaf(gw, e.yr, acc[G_W2]);
    if (kGeom) {
      acc[G_ZC] = fmaf(dz, w0 * iw, acc[G_ZC]);
      acc[G_CX] = fmaf(dzw, w1, acc[G_CX]);
      acc[G_CY] = fmaf(dzw, w2, acc[G_CY]);
    }
    vx = fmaf(u1, a11, fmaf(u2, a21, -uw * w1));
    vy = fmaf(u1, a12, fmaf(u2, a22, -uw * w2));
  } else {
    vx = e.xr;
    vy = e.yr;
    if (kGeom) acc[G_ZC] += dz;
  }
  acc[G_CX] = fmaf(ndr, vx, acc[G_CX]);
  acc[G_CY] = fmaf(ndr, vy, acc[G_CY]);
  acc[G_SCX] = fmaf(nds, vx, acc[G_SCX]);
  acc[G_SCY] = fmaf(nds, vy, acc[G_SCY]);
}

// One pixel's share of the record gradients of a staged surfel.  Branch-free: a pixel that does not
// take this surfel (entry at or past its 'last', or alpha below 1/255) adds zero and keeps its T.
template <int k, bool kGeom>
__device__ __forceinline__ void bwd_px(const LaneTerms& lt, const float4& q0, const float4& q1, const float4& q2,
                                       const float4& q3, const float4& q4, uint32_t e_idx, BwdState& p,
                                       float (&acc)[kGradFields], bool& any) {
  Px e;
  eval_px<k>(lt, q2.y, e);
  const bool con = e_idx < p.last && e.alpha >= kAlphaMin;
  // for a quadrant without a contributing pixel every update below is the identity
  if (__ballot(con) == 0) return;
  any = true;  // wave-uniform: some pixel takes the entry
  BwdTake t;
  bwd_take<kGeom>(e, con, q2, q3, q4, p, t);
  // Tn = the transmittance after this fragment (its last use is the step back to the one in front, so
  // the step writes in place)
  const float Tn = p.T;
  const float nA = fmaf(-Tn, t.g, p.sA);
  const float nS = fmaf(-Tn, t.gs, p.sS);
  const float wgt = Tn * t.ar;  // alpha T_i
  p.T = Tn * t.rom;             // T_i, in front of it
  p.sA = fmaf(wgt, t.g, p.sA);
  p.sS = fmaf(wgt, t.gs, p.sS);
  bwd_terms<kGeom>(e, t, q0, q1, q2, e_idx, p, wgt, nA, nS, acc);
}

// Factor that turns the reduced value of field 'slot' into its record gradient: the staged numerator
// coefficients carry 1/sqrt(2), the colour fields -2.  (The opacity field, 2 d rho, takes -1 / (2 o) of
// its surfel instead.)
__device__ __forceinline__ float slot_scale(int slot) {
  if (slot >= G_A11 && slot <= G_A22) return kInvSqrt2;
  return slot >= G_R && slot <= G_B ? -0.5f : 1.f;
}

// Adds one staged entry's wave-summed record gradients (acc of every lane) into (view, surfel) 'id':
// fields G_CX..G_ZC by reduce-scatter (one atomic instruction, one lane per field), the normals (kGeom)
// likewise.  sc = slot_scale of the lane's field.
template <bool kGeom>
__device__ __forceinline__ void bwd_commit(float (&acc)[kGradFields], int lane, int slot, float sc, float io,
                                           float* rgv, float* rgn, uint32_t id) {
  float red[16];
#pragma unroll
  for (int f = 0; f < 16; ++f) red[f] = acc[f];
  const float tot = reduce16_scatter(red);
  if ((lane & 3) == 0 && (kGeom || slot != G_ZC))
    atomicAdd(rgv + (int64_t)id * kGradRow + slot, tot * (slot == G_OP ? -0.5f * io : sc));
  if (kGeom) {
    const float nrm = reduce3_scatter(acc[G_NX], acc[G_NY], acc[G_NZ]);
    // lanes 0, 4 and 8: nx, ny, nz
    if ((lane & 0x33) == 0 && lane < 12) atomicAdd(rgn + (int64_t)id * kGradNrm + (lane >> 2), -0.5f * nrm);
  }
}

// Reverse pass over the quadrants kSub of one tile (as render_fwd_tile): each entry's record gradients
// summed over the block's pixels and added per (surfel, tile or split block).
// kGeom: depth, median-depth, normal or alpha upstream gradients are present.  Without them (the
// photometric-loss-only case) their per-pixel state, terms and four of the reductions drop out.
template <bool kGeom, uint32_t kSub>
__device__ __forceinline__ void render_bwd_tile(const BwdArgs& A, Stage& s, uint32_t b) {
  const RenderArgs& a = A.r;
  const int lv = (int)(b / (uint32_t)a.tiles);
  const int v = a.cams.v0 + lv;
  const int t = (int)(b % (uint32_t)a.tiles);
  const int tx = t % a.tiles_x, ty = t / a.tiles_x;
  const DevCam& c = a.cams.c[lv];
  const int lane = threadIdx.x;
  const int lx = lane & 7, ly = lane >> 3;
  const int ox = tx * kTile, oy = ty * kTile;
  const uint32_t start = a.ranges[(int64_t)v * a.tiles + t], end = a.ranges[(int64_t)v * a.tiles + t + 1];
  const int64_t vn = (int64_t)v * a.n;
  float* rgv = A.rg.row + (int64_t)v * a.n * kGradRow;
  float* rgn = A.rg.nrm + (int64_t)v * a.n * kGradNrm;

  BwdState p[4];
  // per-quadrant wave maxima of 'last': quadrant k has nothing to walk at or above qhi[k]
  uint32_t qhi[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    qhi[k] = start;
    if (!((kSub >> k) & 1u)) continue;
    bwd_init<kGeom>(A, c, v, ox + lx + 8 * (k & 1), oy + ly + 8 * (k >> 1), start, end, p[k]);
    uint32_t h = p[k].last;
    for (int off = 1; off < 64; off <<= 1) h = max(h, __shfl_xor(h, off));
    qhi[k] = uniform(h);
  }
  const uint32_t hi = max(max(qhi[0], qhi[1]), max(qhi[2], qhi[3]));
  const float lx0 = (float)lx + 0.5f, ly0 = (float)ly + 0.5f;
  const int slot = reduce16_index(lane);
  const float sc = slot_scale(slot);

  constexpr bool kOne = (kSub & (kSub - 1u)) == 0u;  // a single quadrant
  // quadrants of the subset in which list entry idx of the chunk below 'top' may contribute: each only
  // below its walk bound, and where the forward found a contributing pixel
  auto wanted = [&](uint32_t idx, uint32_t top) -> uint32_t {
    uint32_t allow = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) allow |= (((kSub >> k) & 1u) && idx < qhi[k] ? 1u : 0u) << k;
    if (idx >= top) allow = 0u;
    return allow && a.img.qmask ? a.img.qmask[idx] & allow : allow;
  };
  auto below = [&](uint32_t x) { return x - start > 64u ? x - 64u : start; };
  uint32_t nlo = below(hi);
  if constexpr (kOne) {
    // as the forward: the next chunk's records are loaded under this chunk's entries, and only the set
    // bits of the quadrant's ballot are walked
    StageIn in;
    uint32_t nid, nqm;
    {
      const uint32_t idx = nlo + lane;
      stage_load(in, a.rec, vn, a.n, idx < hi ? a.ids[idx] : 0u, wanted(idx, hi));
      const uint32_t l2 = below(nlo);
      nid = l2 + lane < nlo ? a.ids[l2 + lane] : 0u;
      nqm = wanted(l2 + lane, nlo);
    }
    for (uint32_t top = hi; top > start;) {
      const uint32_t lo = nlo;
      uint64_t todo = __ballot(stage_put(s, lane, in, ox, oy, !a.img.qmask) != 0u);
      nlo = below(lo);
      stage_load(in, a.rec, vn, a.n, nid, nqm);
      const uint32_t l2 = below(nlo);
      nid = l2 + lane < nlo ? a.ids[l2 + lane] : 0u;
      nqm = wanted(l2 + lane, nlo);
      __syncthreads();
      while (todo != 0) {
        const int j = 63 - __builtin_clzll(todo);
        todo &= ~(1ull << j);
        const uint32_t e_idx = lo + (uint32_t)j;
        const float4 q0 = s.q[j][0], q1 = s.q[j][1], q2 = s.q[j][2], q3 = s.q[j][3], q4 = s.q[j][4];
        LaneTerms lt;
        lane_terms(lx0, ly0, q0, q1, q2, lt);
        float acc[kGradFields];
#pragma unroll
        for (int f = 0; f < kGradFields; ++f) acc[f] = 0.f;
        bool any = false;
        if (kSub == 1u) bwd_px<0, kGeom>(lt, q0, q1, q2, q3, q4, e_idx, p[0], acc, any);
        if (kSub == 2u) bwd_px<1, kGeom>(lt, q0, q1, q2, q3, q4, e_idx, p[1], acc, any);
        if (kSub == 4u) bwd_px<2, kGeom>(lt, q0, q1, q2, q3, q4, e_idx, p[2], acc, any);
        if (kSub == 8u) bwd_px<3, kGeom>(lt, q0, q1, q2, q3, q4, e_idx, p[3], acc, any);
        if (any) bwd_commit<kGeom>(acc, lane, slot, sc, q4.w, rgv, rgn, __float_as_uint(q3.w));
      }
      __syncthreads();
      top = lo;
    }
  } else {
    // the list ids of the next (lower) chunk are loaded one chunk ahead, as in the forward
    uint32_t nid = nlo + lane < hi ? a.ids[nlo + lane] : 0u;
    for (uint32_t top = hi; top > start;) {
      const uint32_t lo = nlo;
      const uint32_t id = nid;
      QuadBits qb;
      qb.from_lanes(stage_record(s, lane, a.rec, vn, a.n, id, wanted(lo + lane, top), ox, oy, !a.img.qmask));
      nlo = below(lo);
      nid = nlo + lane < lo ? a.ids[nlo + lane] : 0u;
      __syncthreads();
      const int j0 = (int)(top - lo) - 1;
      uint64_t cur = qb.word(j0 >> 4) << (4 * (15 - (j0 & 15)));  // entry j's nibble in bits 60-63
      for (int j = (int)(top - lo) - 1; j >= 0; --j) {
        const uint32_t e_idx = lo + (uint32_t)j;
        if ((j & 15) == 15) cur = qb.word(j >> 4);
        const uint32_t m = (uint32_t)(cur >> 60);  // quadrant bits, kSub and the quadrants' walk bounds applied
        cur <<= 4;
        if (m == 0) continue;
        const float4 q0 = s.q[j][0], q1 = s.q[j][1], q2 = s.q[j][2], q3 = s.q[j][3], q4 = s.q[j][4];
        LaneTerms lt;
        lane_terms(lx0, ly0, q0, q1, q2, lt);
        float acc[kGradFields];
#pragma unroll
        for (int f = 0; f < kGradFields; ++f) acc[f] = 0.f;
        bool any = false;
        if ((kSub & 1u) && (m & 1u)) bwd_px<0, kGeom>(lt, q0, q1, q2, q3, q4, e_idx, p[0], acc, any);
        if ((kSub & 2u) && (m & 2u)) bwd_px<1, kGeom>(lt, q0, q1, q2, q3, q4, e_idx, p[1], acc, any);
        if ((kSub & 4u) && (m & 4u)) bwd_px<2, kGeom>(lt, q0, q1, q2, q3, q4, e_idx, p[2], acc, any);
        if ((kSub & 8u) && (m & 8u)) bwd_px<3, kGeom>(lt, q0, q1, q2, q3, q4, e_idx, p[3], acc, any);
        if (!any) continue;
        bwd_commit<kGeom>(acc, lane, slot, sc, q4.w, rgv, rgn, __float_as_uint(q3.w));
      }
      __syncthreads();
      top = lo;
    }
  }
}

// Reverse pass of one 4x4 block (of quadrant k): as render_fwd_block, the four lanes of a pixel take four entries at a
// time, from the back.  Each pixel's terms are those of the tile's walk bit for bit; the record gradients of the four
// entries are summed over the block's pixels at once and leave in one atomic instruction.
template <bool kGeom, int k>
__device__ __forceinline__ void render_bwd_block(const BwdArgs& A, Stage& s, uint32_t b, int bx, int by) {
  const RenderArgs& a = A.r;
  const int lv = (int)(b / (uint32_t)a.tiles);
  const int v = a.cams.v0 + lv;
  const int t = (int)(b % (uint32_t)a.tiles);
  const DevCam& c = a.cams.c[lv];
  const int lane = threadIdx.x, part = lane & 3;
  const int ox = t % a.tiles_x * kTile, oy = t / a.tiles_x * kTile;
  const int px = ox + bx + ((lane >> 2) & 3), py = oy + by + (lane >> 4);
  const uint32_t start = a.ranges[(int64_t)v * a.tiles + t], end = a.ranges[(int64_t)v * a.tiles + t + 1];
  const int64_t vn = (int64_t)v * a.n;
  float* rgv = A.rg.row + (int64_t)v * a.n * kGradRow;
  float* rgn = A.rg.nrm + (int64_t)v * a.n * kGradNrm;
  const float lx0 = (float)(px - ox - 8 * (k & 1)) + 0.5f, ly0 = (float)(py - oy - 8 * (k >> 1)) + 0.5f;
  BwdState p;  // the same in the pixel's four lanes
  bwd_init<kGeom>(A, c, v, px, py, start, end, p);
  uint32_t hi = p.last;
  for (int off = 4; off < 64; off <<= 1) hi = max(hi, __shfl_xor(hi, off));
  hi = uniform(hi);
  const int slot = reduce16_index(lane);
  const float sc = slot_scale(slot);
  auto wanted = [&](uint32_t idx, uint32_t top) -> uint32_t {
    const uint32_t allow = idx < top ? 1u << k : 0u;
    return allow && a.img.qmask ? a.img.qmask[idx] & allow : allow;
  };
  auto below = [&](uint32_t x) { return x - start > 64u ? x - 64u : start; };
  uint32_t nlo = below(hi), nid, nqm;
  StageIn in;
  {
    const uint32_t idx = nlo + lane, l2 = below(nlo);
    stage_load(in, a.rec, vn, a.n, idx < hi ? a.ids[idx] : 0u, wanted(idx, hi));
    nid = l2 + lane < nlo ? a.ids[l2 + lane] : 0u;
    nqm = wanted(l2 + lane, nlo);
  }
  for (uint32_t top = hi; top > start;) {
    const uint32_t lo = nlo;
    uint64_t todo = __ballot(stage_put<true>(s, lane, in, ox, oy, !a.img.qmask, bx, by) != 0u);
    nlo = below(lo);
    stage_load(in, a.rec, vn, a.n, nid, nqm);
    const uint32_t l2 = below(nlo);
    nid = l2 + lane < nlo ? a.ids[l2 + lane] : 0u;
    nqm = wanted(l2 + lane, nlo);
    __syncthreads();
    while (todo != 0) {
      int at[4];
      bool has[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        has[q] = todo != 0;
        at[q] = has[q] ? 63 - __builtin_clzll(todo) : at[0];
        if (has[q]) todo &= ~(1ull << at[q]);
      }
      const int j = part == 0 ? at[0] : part == 1 ? at[1] : part == 2 ? at[2] : at[3];
      const bool act = part == 0 || (part == 1 ? has[1] : part == 2 ? has[2] : has[3]);
      const uint32_t e_idx = lo + (uint32_t)j;
      const float4 q0 = s.q[j][0], q1 = s.q[j][1], q2 = s.q[j][2], q3 = s.q[j][3], q4 = s.q[j][4];
      LaneTerms lt;
      lane_terms(lx0, ly0, q0, q1, q2, lt);
      Px e;
      eval_px<k>(lt, q2.y, e);
      const bool con = act && e_idx < p.last && e.alpha >= kAlphaMin;
      const uint64_t taken = __ballot(con);
      if (taken == 0) continue;
      BwdTake u;
      bwd_take<kGeom>(e, con, q2, q3, q4, p, u);
      u.g = con ? u.g : 0.f;  // (of an entry that is not taken it may be infinite)
      u.gs = con ? u.gs : 0.f;
      // the transmittance behind each of the four entries, from the last one on
      const float T1 = p.T * quad_lane<0>(u.rom), T2 = T1 * quad_lane<1>(u.rom), T3 = T2 * quad_lane<2>(u.rom);
      const float Tn = part == 0 ? p.T : part == 1 ? T1 : part == 2 ? T2 : T3;
      p.T = T3 * quad_lane<3>(u.rom);
      const float wgt = Tn * u.ar;
      const float w0 = quad_lane<0>(wgt), w1 = quad_lane<1>(wgt), w2 = quad_lane<2>(wgt), w3 = quad_lane<3>(wgt);
      // an entry the pixel does not take leaves the sums as they are
      auto sums = [&](float& sum, float g) {
        const float s1 = fmaf(w0, quad_lane<0>(g), sum), s2 = fmaf(w1, quad_lane<1>(g), s1),
                    s3 = fmaf(w2, quad_lane<2>(g), s2);
        const float own = part == 0 ? sum : part == 1 ? s1 : part == 2 ? s2 : s3;
        sum = fmaf(w3, quad_lane<3>(g), s3);
        return own;
      };
      const float sA = sums(p.sA, u.g), sS = sums(p.sS, u.gs);
      float acc[kGradFields];
#pragma unroll
      for (int f = 0; f < kGradFields; ++f) acc[f] = 0.f;
      bwd_terms<kGeom>(e, u, q0, q1, q2, e_idx, p, wgt, fmaf(-Tn, u.g, sA), fmaf(-Tn, u.gs, sS), acc);
      float red[16];
#pragma unroll
      for (int f = 0; f < 16; ++f) red[f] = acc[f];
      const float tot = reduce16_scatter_quads(red);
      const bool any = (taken & (0x1111111111111111ull << part)) != 0;  // some pixel takes this lane's entry
      const int64_t id = (int64_t)__float_as_uint(q3.w);
      if (any && (kGeom || slot != G_ZC))
        atomicAdd(rgv + id * kGradRow + slot, tot * (slot == G_OP ? -0.5f * q4.w : sc));
      if (kGeom) {
        const float n0 = sum_quads(acc[G_NX]), n1 = sum_quads(acc[G_NY]), n2 = sum_quads(acc[G_NZ]);
        if (any && lane < 12)
          atomicAdd(rgn + id * kGradNrm + (lane >> 2), -0.5f * (lane < 4 ? n0 : lane < 8 ? n1 : n2));
      }
    }
    __syncthreads();
    top = lo;
  }
}

template <bool kGeom>
__global__ __launch_bounds__(64) void k_render_bwd(BwdArgs A) {
  __shared__ Stage s;
  uint32_t sub;
  const uint32_t b = tile_of_block(A.r, sub);
  if (*A.r.status != 0) return;
  if (sub & kMaybeBit) {
    sub = maybe_block(sub, long_list(A.r, b, kLongBwd, 0u));
    if (sub == 0u) return;
  }
  if (sub & kBlockBit) {
    const int bx = 4 * (int)(sub & 3u), by = (int)(sub & 12u);
    switch ((bx >> 3) + 2 * (by >> 3)) {
      case 0: render_bwd_block<kGeom, 0>(A, s, b, bx, by); break;
      case 1: render_bwd_block<kGeom, 1>(A, s, b, bx, by); break;
      case 2: render_bwd_block<kGeom, 2>(A, s, b, bx, by); break;
      default: render_bwd_block<kGeom, 3>(A, s, b, bx, by); break;
    }
    return;
  }
  switch (sub) {
    case 0x1u: render_bwd_tile<kGeom, 0x1u>(A, s, b); break;
    case 0x2u: render_bwd_tile<kGeom, 0x2u>(A, s, b); break;
    case 0x4u: render_bwd_tile<kGeom, 0x4u>(A, s, b); break;
    case 0x8u: render_bwd_tile<kGeom, 0x8u>(A, s, b); break;
    case 0x3u: render_bwd_tile<kGeom, 0x3u>(A, s, b); break;
    case 0xcu: render_bwd_tile<kGeom, 0xcu>(A, s, b); break;
    default: render_bwd_tile<kGeom, 0xfu>(A, s, b); break;
  }
}

// Clears the record gradients of the surfels in view v's visible list (the atomics add into them).
__global__ __launch_bounds__(256) void k_zero_visible(const uint32_t* __restrict__ visible,
                                                     const uint32_t* __restrict__ vstart, int64_t n, RecGrads rg,
                                                     int v0) {
  const int v = v0 + (int)blockIdx.y;
  const uint32_t e0 = vstart[v], e1 = vstart[v + 1];
  const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  for (uint32_t e = e0 + blockIdx.x * blockDim.x + threadIdx.x; e < e1; e += gridDim.x * blockDim.x) {
    const int64_t vi = (int64_t)v * n + visible[e];
    float4* r = (float4*)(rg.row + vi * kGradRow);
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = z;
    *(float4*)(rg.nrm + vi * kGradNrm) = z;
  }
}

}  // namespace cgv2

// Heavy tiles split over several waves: the 1 / kSplitDiv heaviest of a launch's tiles (at most
// kSplitMax) into four quadrant blocks, the next 1 / kHalfDiv (at most kSplitMax; none for 0) into two
// halves.  A launch with fewer tiles than the chip holds waves of the kernel ('resident': 1,024 SIMDs
// times its waves per SIMD) is split further, because its time is then one wave's walk of one list:
//   2 tiles <= 1.25 resident   every tile, into halves, and the heaviest into quadrants as far as 1.25
//                              resident blocks go (all of them up to 0.31 resident tiles)
//   up to 'fill_below' tiles   the heaviest into quadrants, up to 'resident' blocks
// Measured (us, before -> after): 64 tiles (4,096 surfels, 128x128) forward 121 -> 47, reverse 181 -> 68;
// 1,200 tiles (5 M surfels, 640x480) 4067 -> 1932 and 3232 -> 1702; 1,900 tiles (1 M, 800x600) 109 -> 83
// and 160 -> 128; 2,304 tiles (2 M, 1024x576) 302 -> 222 and 440 -> 338; 3,072 tiles (2 M, 1024x768)
// 302 -> 243 and 442 -> 386; 3,600 tiles (5 M, 1280x720) forward 1744 -> 1229, but the reverse 1604 ->
// 1703 and 242 -> 262 (1 M), so the reverse stops at 3/4 resident.  At 6,700 tiles more splitting is
// slower in both (forward 197 -> 201 and reverse 353 -> 358 with 5,120 to 8,192 blocks).
#ifndef CGV2_SPLIT_DIV
#define CGV2_SPLIT_DIV 48
#endif
#ifndef CGV2_HALF_DIV
#define CGV2_HALF_DIV 12
#endif
constexpr int kSplitDiv = CGV2_SPLIT_DIV;
constexpr int kHalfDiv = CGV2_HALF_DIV;
constexpr int kSplitMax = 1024;

namespace cgv2 {
// Clears the quadrant-mask bytes of the split tiles' lists (their blocks OR their bits in).
__global__ __launch_bounds__(256) void k_clear_split_qmask(RenderArgs a) {
  if (*a.status != 0) return;  // overflowed bins: ranges may lie beyond the list arrays
  const uint32_t tiles = (uint32_t)a.cams.count * (uint32_t)a.tiles;
  const uint32_t b0 = a.order[blockIdx.x];
  const uint32_t b = b0 < tiles ? b0 : tiles - 1u;
  const int v = a.cams.v0 + (int)(b / (uint32_t)a.tiles), t = (int)(b % (uint32_t)a.tiles);
  const uint32_t start = a.ranges[(int64_t)v * a.tiles + t], end = a.ranges[(int64_t)v * a.tiles + t + 1];
  for (uint32_t e = start + threadIdx.x; e < end; e += blockDim.x) a.img.qmask[e] = 0;
}
}  // namespace cgv2

static void split_tiles(cgv2::RenderArgs& a, int64_t resident, int64_t fill_below) {
  a.n_b = a.n_m = a.n_q = a.n_h = 0;
  if (!a.order) return;
  const int64_t all = (int64_t)a.cams.count * a.tiles;
  int64_t q = std::min<int64_t>(all / kSplitDiv, kSplitMax);
  int64_t h = kHalfDiv > 0 ? std::min<int64_t>(all / std::max(kHalfDiv, 1), kSplitMax) : 0;
  const int64_t most = resident + resident / 4;
  if (2 * all <= most) {
    q = std::max(q, (most - 2 * all) / 2);
    h = all;
  } else if (all < fill_below) {
    q = std::max(q, (resident - all) / 3);
  }
  a.n_q = (uint32_t)std::min(q, all);
  a.n_h = (uint32_t)std::min(h, all - (int64_t)a.n_q);
}
constexpr int64_t kSimds = 1024;

static cgv2::RenderArgs make_args(const cgv2_proj& p, const cgv2_bins& b, const cgv2::CamPack& cams, int64_t n,
                                  int tiles_x, int tiles_y, const cgv2_image* img, unsigned long long* counters) {
  cgv2::RenderArgs a;
  a.rec = p.rec;
  a.ids = b.ids;
  a.ranges = b.ranges;
  a.order = b.order ? b.order + (int64_t)cams.v0 * tiles_x * tiles_y : nullptr;
  a.status = b.status;
  a.cams = cams;
  a.n = n;
  a.tiles_x = tiles_x;
  a.tiles_y = tiles_y;
  a.tiles = tiles_x * tiles_y;
  if (img) a.img = *img; else a.img = cgv2_image{};
  a.counters = counters;
  a.cws = nullptr;
  a.gamma = 0.f;
  a.n_b = a.n_m = a.n_q = a.n_h = 0;
  return a;
}

// the forward kernels hold at least 4 waves per SIMD, the reverse 4 without and 3 with geometry terms
static void split_fwd(cgv2::RenderArgs& a) { split_tiles(a, 4 * kSimds, 4 * kSimds); }
static void split_bwd(cgv2::RenderArgs& a, bool geom) {
  const int64_t resident = (geom ? 3 : 4) * kSimds;
  split_tiles(a, resident, resident * 3 / 4 + 1);
}

// Of the quadrant tiles, the heaviest run as blocks while the launch is small: a block tile issues up to twice the
// instructions of four quadrants (in the reverse about as many: its reductions take four entries at once), but in
// sixteen chains a quarter to an eighth as long.  With quadrants -> with blocks, forward / reverse / reverse with
// geometry terms, us:
//   64 tiles                             43 -> 26      63 -> 30      79 -> 34
//   260 tiles                            65 -> 42      98 -> 47     128 -> 58
//   260 tiles, lists to 67,521         4370 -> 1940  2855 -> 1290  3463 -> 1440
//   475 tiles                            89 -> 66     130 -> 73     166 -> 98
//   600 tiles                           100 -> 78     141 -> 88     186 -> 117   (26 % of them: 85, 127, 172)
// Up to kAllBlocks tiles all of them do.  Beyond, the heaviest do as far as kBlockWaves waves go, and further ones, as
// far as kMaybeWaves go, where the device finds their lists long (maybe_block): in the forward kLongFwd entries and
// kLongFwdHalves / 2 times the mean, since blocks help only where single tiles' chains bound the launch, in the reverse
// kLongBwd entries.  The twelve waves too many of a short tile come last in the launch, where they cost nothing (in
// front of the others: reverse 196 -> 240 at 300 k opaque surfels).  Measured, first with an allowance by the bins'
// capacity (fitted to the scene, then the engine's own default), then by the lists:
//   1,200 tiles, 5 M surfels, lists to 16,504, mean 2,407  forward 850, 849 -> 704   reverse 532, 531 -> 544
//                1 M, to 3,938, mean 675                           324, 270 -> 251           410, 257 -> 265
//                300 k opaque, to 2,295, mean 996                  110, 139 -> 110           192, 196 -> 205
//                1 M faint, to 2,971, mean 1,214                   333, 477 -> 333           537, 383 -> 389
//                300 k, to 679, mean 163                            92, 118 ->  93           144, 133 -> 137
//   1,900 tiles, 1 M opaque, to 6,078, mean 2,661                  167, 166 -> 168           331, 322 -> 250
//                1 M, to 1,043, mean 224                           139, 142 -> 142           224, 272 -> 204
//   3,600 tiles, 2 M, 1280x720                                     376 -> 361                517 -> 533
// (the forward by kLongFwd alone: 110 -> 136 at 300 k opaque, 333 -> 398 at 1 M faint.)  At 6,700 tiles blocks for the
// heaviest 1/64 cost the forward 152 -> 170, for 1/8 the reverse 297 -> 375.
constexpr int64_t kAllBlocks = 640, kBlockWaves = 5120, kMaybeWavesFwd = 8192, kMaybeWavesBwd = 20480;
static void split_blocks(cgv2::RenderArgs& a, int64_t maybe_waves) {
  const int64_t all = (int64_t)a.cams.count * a.tiles;
  auto tiles_of = [&](int64_t waves) {
    return (uint32_t)std::min<int64_t>(std::max<int64_t>((waves - 4 * all) / 12, 0), a.n_q);
  };
  a.n_b = all > kAllBlocks ? tiles_of(kBlockWaves) : a.n_q;
  a.n_m = all > kAllBlocks ? tiles_of(maybe_waves) - a.n_b : 0;
  a.n_q -= a.n_b + a.n_m;
}
static unsigned launch_blocks(const cgv2::RenderArgs& a) {
  return (unsigned)((int64_t)a.cams.count * a.tiles + 15 * (int64_t)(a.n_b + a.n_m) + 3 * a.n_q + a.n_h);
}

hipError_t cgv2_launch_render_fwd(const cgv2_proj& p, const cgv2_bins& b, const cgv2::CamPack& cams, int64_t n,
                                  int tiles_x, int tiles_y, const cgv2_image& img, hipStream_t st) {
  cgv2::RenderArgs a = make_args(p, b, cams, n, tiles_x, tiles_y, &img, nullptr);
  split_fwd(a);
  split_blocks(a, kMaybeWavesFwd);
  const unsigned grid = launch_blocks(a), split = a.n_b + a.n_m + a.n_q + a.n_h;
  if (img.qmask && split) hipLaunchKernelGGL(cgv2::k_clear_split_qmask, dim3(split), dim3(256), 0, st, a);
  if (img.qmask) hipLaunchKernelGGL((cgv2::k_render_fwd<false, true, cgv2::kNoContrib>), dim3(grid), dim3(64), 0, st, a);
  else hipLaunchKernelGGL((cgv2::k_render_fwd<false, false, cgv2::kNoContrib>), dim3(grid), dim3(64), 0, st, a);
  return hipGetLastError();
}

hipError_t cgv2_launch_render_count(const cgv2_proj& p, const cgv2_bins& b, const cgv2::CamPack& cams, int64_t n,
                                    int tiles_x, int tiles_y, unsigned long long* counters, hipStream_t st) {
  cgv2::RenderArgs a = make_args(p, b, cams, n, tiles_x, tiles_y, nullptr, counters);
  split_fwd(a);
  const unsigned grid = launch_blocks(a);
  hipLaunchKernelGGL((cgv2::k_render_fwd<true, false, cgv2::kNoContrib>), dim3(grid), dim3(64), 0, st, a);
  return hipGetLastError();
}

hipError_t cgv2_launch_render_bwd(const cgv2_proj& p, const cgv2_bins& b, const cgv2::CamPack& cams, int64_t n,
                                  int tiles_x, int tiles_y, const cgv2_image& img, const cgv2_image_grad& up,
                                  const cgv2::RecGrads& rg, hipStream_t st) {
  if (n > 0) {
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 1024);
    hipLaunchKernelGGL(cgv2::k_zero_visible, dim3(blocks, (unsigned)cams.count), dim3(256), 0, st, p.visible,
                       p.visible_start, n, rg, cams.v0);
  }
  cgv2::BwdArgs A;
  A.r = make_args(p, b, cams, n, tiles_x, tiles_y, &img, nullptr);
  A.up = up;
  A.rg = rg;
  const bool geom = up.d_depth || up.d_depth_med || up.d_normal || up.d_alpha;
  split_bwd(A.r, geom);
  split_blocks(A.r, kMaybeWavesBwd);
  const unsigned grid = launch_blocks(A.r);
  if (geom) hipLaunchKernelGGL(cgv2::k_render_bwd<true>, dim3(grid), dim3(64), 0, st, A);
  else hipLaunchKernelGGL(cgv2::k_render_bwd<false>, dim3(grid), dim3(64), 0, st, A);
  return hipGetLastError();
}

hipError_t cgv2_launch_contribution(const cgv2_proj& p, const cgv2_bins& b, const cgv2::CamPack& cams, int64_t n,
                                    int tiles_x, int tiles_y, float gamma, float* cws, hipStream_t st) {
  cgv2::RenderArgs a = make_args(p, b, cams, n, tiles_x, tiles_y, nullptr, nullptr);
  split_fwd(a);
  a.cws = cws;
  a.gamma = gamma;
  const unsigned grid = launch_blocks(a);
  if (gamma == 0.5f)
    hipLaunchKernelGGL((cgv2::k_render_fwd<false, false, cgv2::kHalfGamma>), dim3(grid), dim3(64), 0, st, a);
  else
    hipLaunchKernelGGL((cgv2::k_render_fwd<false, false, cgv2::kAnyGamma>), dim3(grid), dim3(64), 0, st, a);
  return hipGetLastError();
}
