// Tile binning and per-tile depth sort.
//
// Instead of a global LSD radix sort over (view | tile | depth) keys, intersections are bucketed
// by tile directly:
//   surfel scan   one fused pass of three kernels (two up to kSurfLocal chunks) over every (view,
//                 surfel): the exclusive prefix sum of its tile count (from its rect) and the compaction
//                 of the visible ones into per-view lists, plus the capacity check
//   k_stage       a workgroup per run of consecutive visible surfels: for each tile of a surfel's rect that
//                 its alpha >= 1/255 region reaches (reach_cell over the tile's pixel samples), a returning
//                 atomic on the tile's counter gives the entry's rank within the tile; the entry (counter, rank)
//                 is packed, with large rects at the start of the surfel's rect slots, with small ones at the
//                 start of the run's; each visible surfel's depth, number of entries and first slot go beside
//   k_tile_scan_order   one workgroup up to kScanChunk tiles: exclusive prefix sum of the counters ->
//                 ranges and each counter's first slot; for at most kMaxViews views also the launch order
//                 (k_tile_sums / k_tile_apply and the multi-workgroup order kernels otherwise)
//   k_place       a workgroup per run: keys[first slot of the counter + rank] = depth bits << 32 | id of the
//                 entry's surfel (no atomics)
//   k_sort_wave   one wave per tile: bitonic sort of lists up to kWaveSort entries in registers; a longer
//                 list is cut into equal chunks of at most kWaveSort, one wave each
//   k_merge       one workgroup per chunk: each key's place among the other chunks of its list (binary
//                 searches in LDS) gives its slot
// (depth bits, id) is unique within a tile, so the order in which the atomics hand out ranks does not
// matter: the result is deterministic and bit-exact.  HBM traffic is about 8 B staged + 8 B read + 8 B placed +
// 8 B read + 4 B written per listed entry and 10 B written and read per visible surfel, nothing per rect tile out
// of reach.
#include "cgv2r_device.h"
#include "cgv2r_kernels.h"

#include <algorithm>

namespace cgv2 {

constexpr int kWaveSort = 1024;  // longest list one wave sorts in its registers (16 keys per lane)

// The chunks of lists longer than kWaveSort, as (tile, chunk): a list of length len in chunks of equal size
// (the last one shorter), as few as hold at most kWaveSort entries each.  Each such list holds more than
// kWaveSort entries, so capacity / (kWaveSort / 2) + 1 items hold all chunks.
struct SortItems {
  uint2* item;
  uint32_t* count;
};
__device__ __forceinline__ uint32_t chunk_size(uint32_t len) {
  const uint32_t nc = (len + kWaveSort - 1) / kWaveSort;
  return (len + nc - 1) / nc;
}
__device__ __forceinline__ uint32_t chunk_count(uint32_t len) {
  const uint32_t cs = chunk_size(len);
  return (len + cs - 1) / cs;
}

constexpr int kScanBlock = 1024;
constexpr int kScanItems = 8;  // elements per thread per scan block
constexpr int kScanChunk = kScanBlock * kScanItems;

__device__ __forceinline__ void tile_rect(const uint16_t* r4, uint32_t& tx0, uint32_t& ty0, uint32_t& tx1,
                                          uint32_t& ty1) {
  const uint2 r = *(const uint2*)r4;
  tx0 = r.x & 0xffffu; ty0 = r.x >> 16; tx1 = r.y & 0xffffu; ty1 = r.y >> 16;
}

__device__ __forceinline__ uint32_t rect_count(const uint16_t* r4) {
  uint32_t tx0, ty0, tx1, ty1;
  tile_rect(r4, tx0, ty0, tx1, ty1);
  return (tx1 - tx0) * (ty1 - ty0);
}

__device__ __forceinline__ uint64_t shfl_up64(uint64_t x, unsigned d) {
  const uint32_t lo = __shfl_up((uint32_t)x, d, 64), hi = __shfl_up((uint32_t)(x >> 32), d, 64);
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl_xor64(uint64_t x, int m) {
  const uint32_t lo = __shfl_xor((uint32_t)x, m, 64), hi = __shfl_xor((uint32_t)(x >> 32), m, 64);
  return ((uint64_t)hi << 32) | lo;
}

// inclusive prefix sum over the 64 lanes of a wave
__device__ __forceinline__ uint64_t wave_scan(uint64_t x) {
  const unsigned lane = threadIdx.x & 63u;
#pragma unroll
  for (unsigned d = 1; d < 64; d <<= 1) {
    const uint64_t y = shfl_up64(x, d);
    if (lane >= d) x += y;
  }
  return x;
}

// inclusive prefix sum over the 64 lanes of a wave (32-bit) with DPP row shifts and row broadcasts
// only: each row of 16 lanes scans itself, then rows 1 and 3 add the total of the row before, then
// rows 2 and 3 that of rows 0-1 (lanes a shift or broadcast does not reach receive 0)
template <int kCtrl, int kRowMask = 0xf>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, kRowMask, 0xf, false);
}

__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t x) {
  x += dpp_u32<0x111>(x);       // row_shr:1
  x += dpp_u32<0x112>(x);       // row_shr:2
  x += dpp_u32<0x114>(x);       // row_shr:4
  x += dpp_u32<0x118>(x);       // row_shr:8
  x += dpp_u32<0x142, 0xa>(x);  // row_bcast:15
  x += dpp_u32<0x143, 0xc>(x);  // row_bcast:31
  return x;
}

// Appends the chunks of the long lists among a lane's N tiles (tile[k] of length len[k]) with one atomic per
// wave.  Every lane of the wave must call it.
template <int N>
__device__ __forceinline__ void list_items(const SortItems& it, const uint32_t (&tile)[N], const uint32_t (&len)[N]) {
  uint32_t mine = 0;
#pragma unroll
  for (int k = 0; k < N; ++k) mine += len[k] > (uint32_t)kWaveSort ? chunk_count(len[k]) : 0u;
  const uint32_t inc = wave_scan_u32(mine);
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
  if (total == 0) return;
  uint32_t base = 0;
  if ((threadIdx.x & 63u) == 0u) base = atomicAdd(it.count, total);
  uint2* out = it.item + (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + inc - mine;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (len[k] <= (uint32_t)kWaveSort) continue;
    const uint32_t nc = chunk_count(len[k]);
    for (uint32_t c = 0; c < nc; ++c) *out++ = make_uint2(tile[k], c);
  }
}

// the value of lane 63 (a wave total after wave_scan_u32)
__device__ __forceinline__ uint32_t lane63(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }

constexpr int kScanWaves = kScanBlock / 64;

// block-wide exclusive scan of kScanChunk values held kScanItems per thread (consecutive items per
// thread); returns the total.  Lane scans in registers, one LDS round for the 16 wave totals; lds
// holds at least 2 * kScanWaves entries.
__device__ __forceinline__ uint64_t block_scan(uint64_t (&vals)[kScanItems], uint64_t* lds) {
  uint64_t s = 0;
  for (int k = 0; k < kScanItems; ++k) { const uint64_t t = vals[k]; vals[k] = s; s += t; }
  const unsigned lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  const uint64_t inc = wave_scan(s);
  if (lane == 63u) lds[w] = inc;
  __syncthreads();
  if (w == 0) {
    const uint64_t x = wave_scan(lane < (unsigned)kScanWaves ? lds[lane] : 0);
    if (lane < (unsigned)kScanWaves) lds[kScanWaves + lane] = x;
  }
  __syncthreads();
  const uint64_t excl = (w > 0 ? lds[kScanWaves + w - 1] : 0) + inc - s;
  const uint64_t total = lds[2 * kScanWaves - 1];
  for (int k = 0; k < kScanItems; ++k) vals[k] += excl;
  __syncthreads();
  return total;
}

// block-wide sum, valid in thread 0; lds holds at least kScanWaves entries (a second call right after
// needs another lds array: thread 0 may still be reading this one)
__device__ __forceinline__ uint64_t block_sum(uint64_t x, uint64_t* lds) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) x += shfl_xor64(x, m);
  if ((threadIdx.x & 63u) == 0) lds[threadIdx.x >> 6] = x;
  __syncthreads();
  uint64_t t = 0;
  if (threadIdx.x == 0)
    for (int q = 0; q < kScanWaves; ++q) t += lds[q];
  return t;
}

// pass 2 of the surfel scan: workgroup 0 scans the chunk sums of the counts in place, workgroup 1
// those of the visible flags (any count, kScanChunk at a time); totals[blockIdx.x] = grand total
__global__ __launch_bounds__(kScanBlock) void k_scan_top(uint64_t* __restrict__ sums0, uint64_t* __restrict__ sums1,
                                                         int64_t nb, uint64_t* __restrict__ totals) {
  __shared__ uint64_t lds[2 * kScanWaves];
  uint64_t* sums = blockIdx.x == 0 ? sums0 : sums1;
  uint64_t carry = 0;
  for (int64_t base = 0; base < nb; base += kScanChunk) {
    const int64_t b0 = base + (int64_t)threadIdx.x * kScanItems;
    uint64_t vals[kScanItems];
    for (int k = 0; k < kScanItems; ++k) vals[k] = b0 + k < nb ? sums[b0 + k] : 0;
    const uint64_t tot = block_scan(vals, lds);
    for (int k = 0; k < kScanItems; ++k)
      if (b0 + k < nb) sums[b0 + k] = vals[k] + carry;
    carry += tot;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// The surfel scan runs over chunks of kSurfChunk (view, surfel) entries, one 256-thread workgroup each;
// a wave owns kSurfRows consecutive rows of 64 entries (coalesced loads), scans them with shuffles and
// ballots, and only the wave totals go through LDS.
constexpr int kSurfBlock = 256;
constexpr int kSurfWaves = kSurfBlock / 64;
constexpr int kSurfRows = 8;
constexpr int kSurfChunk = kSurfBlock * kSurfRows;
constexpr int kSurfLocal = 4 * kSurfBlock;  // up to this many chunks, each apply workgroup adds up those before it

// pass 1 of the surfel scan: per-chunk sums of the tile counts and of the visible flags; the workgroups
// also zero the nz tile counters (and the counts after them), which the staging uses two launches later
__global__ __launch_bounds__(kSurfBlock) void k_surfel_sums(const uint16_t* __restrict__ rect, int64_t m,
                                                            uint64_t* __restrict__ sums_cnt,
                                                            uint64_t* __restrict__ sums_vis,
                                                            uint32_t* __restrict__ zero, int64_t nz) {
  __shared__ uint64_t red[2][kSurfWaves];
  for (int64_t z = (int64_t)blockIdx.x * kSurfBlock + threadIdx.x; z < nz; z += (int64_t)gridDim.x * kSurfBlock)
    zero[z] = 0u;
  const int64_t base = (int64_t)blockIdx.x * kSurfChunk;
  uint64_t c = 0, f = 0;
  for (int k = 0; k < kSurfRows; ++k) {
    const int64_t idx = base + (int64_t)k * kSurfBlock + threadIdx.x;
    if (idx < m) {
      const uint32_t t = rect_count(rect + 4 * idx);
      c += t;
      f += t != 0u;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    c += shfl_xor64(c, o);
    f += shfl_xor64(f, o);
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    red[0][w] = c;
    red[1][w] = f;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t sc = 0, sf = 0;
    for (int q = 0; q < kSurfWaves; ++q) {
      sc += red[0][q];
      sf += red[1][q];
    }
    sums_cnt[blockIdx.x] = sc;
    sums_vis[blockIdx.x] = sf;
  }
}

// pass 3 of the surfel scan: visible[pos] = surfel id of every (view, surfel) with a non-empty rect in
// (view, id) order, voff[pos] = its first rect slot (for pos < max_vis; more are visible only when the
// slots exceed the capacity too), vstart[v] = first entry of view v, vstart[V] = total; the total is
// checked against the capacity.
// local_nsb > 0 (at most kSurfLocal chunks): the sums are pass 1's raw chunk sums and each workgroup
// adds up those before it (pass 2 is skipped); 0: the sums are pass 2's scanned ones, totals its totals.
__global__ __launch_bounds__(kSurfBlock) void k_surfel_apply(
    const uint16_t* __restrict__ rect, int64_t m, int64_t n, const uint64_t* __restrict__ sums_cnt,
    const uint64_t* __restrict__ sums_vis, const uint64_t* __restrict__ totals, int local_nsb,
    uint32_t* __restrict__ voff, int64_t max_vis, uint32_t* __restrict__ visible, uint32_t* __restrict__ vstart,
    int V, int64_t capacity, int32_t* __restrict__ status, int64_t* __restrict__ needed) {
  __shared__ uint64_t red[4][kSurfWaves];
  __shared__ uint32_t wt[2][kSurfWaves];
  __shared__ uint64_t carry[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (local_nsb > 0) {
    uint64_t r[4] = {0, 0, 0, 0};  // counts and flags before this chunk, then their totals
    for (int j = threadIdx.x; j < local_nsb; j += kSurfBlock) {
      const uint64_t sc = sums_cnt[j], sv = sums_vis[j];
      if (j < (int)blockIdx.x) {
        r[0] += sc;
        r[1] += sv;
      }
      r[2] += sc;
      r[3] += sv;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) r[k] += shfl_xor64(r[k], o);
      if (lane == 0) red[k][w] = r[k];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
      uint64_t t = 0;
      for (int q = 0; q < kSurfWaves; ++q) t += red[threadIdx.x][q];
      carry[threadIdx.x] = t;
    }
  } else if (threadIdx.x == 0) {
    carry[0] = sums_cnt[blockIdx.x];
    carry[1] = sums_vis[blockIdx.x];
    carry[2] = totals[0];
    carry[3] = totals[1];
  }
  // wave scans of the counts and of the visible flags over the wave's rows (32-bit: a chunk's counts
  // stay far below 2^32)
  const int64_t wbase = (int64_t)blockIdx.x * kSurfChunk + (int64_t)w * (64 * kSurfRows);
  const unsigned long long lt = (1ull << lane) - 1ull;
  uint32_t c[kSurfRows], ex[kSurfRows], fx[kSurfRows];
  uint32_t cc = 0, fc = 0;
#pragma unroll
  for (int r = 0; r < kSurfRows; ++r) {
    const int64_t idx = wbase + 64 * r + lane;
    c[r] = idx < m ? rect_count(rect + 4 * idx) : 0u;
  }
#pragma unroll
  for (int r = 0; r < kSurfRows; ++r) {
    const uint32_t inc = wave_scan_u32(c[r]);
    ex[r] = cc + inc - c[r];
    cc += lane63(inc);
    const unsigned long long fb = __ballot(c[r] != 0u);
    fx[r] = fc + (uint32_t)__popcll(fb & lt);
    fc += (uint32_t)__popcll(fb);
  }
  if (lane == 0) {
    wt[0][w] = cc;
    wt[1][w] = fc;
  }
  __syncthreads();
  uint64_t oc = carry[0], ov = carry[1];
  for (int q = 0; q < w; ++q) {
    oc += wt[0][q];
    ov += wt[1][q];
  }
#pragma unroll
  for (int r = 0; r < kSurfRows; ++r) {
    const int64_t e = wbase + 64 * r + lane;
    if (e >= m) continue;
    const uint32_t pos = (uint32_t)(ov + fx[r]);
    const int64_t i = e % n;
    if (c[r] != 0u) {
      visible[pos] = (uint32_t)i;
      const uint64_t cs = oc + ex[r];
      if (pos < max_vis) voff[pos] = (uint32_t)(cs > 0xffffffffull ? 0xffffffffull : cs);
    }
    if (i == 0) vstart[e / n] = pos;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const uint64_t K = carry[2];
    vstart[V] = (uint32_t)carry[3];
    *needed = (int64_t)K;
    if ((int64_t)K > capacity) *status = 1;
  }
}

// How a workgroup of k_stage takes the visible surfels of view blockIdx.y depends on the call's rects:
//   large rects  runs of kGroups surfels, a group of 32 lanes spread over the rect tiles of each
//   small rects  (on average at most kSmallRect tiles: distant surfels, one or two tiles each, and at least
//                kLaneMin visible per view, so that the runs cover the chip) runs of a surfel per lane.  A
//                lane stages its own surfel when the rect holds at most kLaneTiles tiles; the groups then
//                take the run's others.  (With a group for each, a 640x480 view of 5 M surfels, 2.6 M
//                visible with 1.6 rect tiles each, kept 5 % of the lanes busy.)
// The tile counters lie row by row for large rects, whose rows then touch one cache line, and column by
// column for small ones: atomics on one 128-byte line complete every 4 ns, and the horizon's row of long
// lists would share few lines (5 M surfels at 1920x1080: 854 us row by row, 510 column by column; 1 M at
// 1600x1066, 52 tiles per rect, 33 us column by column, 26 row by row).
// A group stages at most the first kFirstTiles tiles of a surfel; the rest of a larger rect (a surfel near
// the camera, or a long thin one) goes to a queue of kChunkTiles-tile chunks that k_stage_big spreads over
// all groups, so no group walks one rect for long while the others idle.  (Measured: 8 or 16 lanes per
// surfel are slower on the training views, 64 saves 7 us there but costs 20 % of the served latency on the
// 5 M-surfel 4K views; up to 8192 workgroups per view instead of 2048 saves 3 us.)
constexpr int kGroup = 32;
constexpr int kStageBlock = 256;
constexpr uint32_t kGroups = kStageBlock / kGroup;
constexpr uint32_t kLaneMin = 32768;
constexpr uint32_t kSmallRect = 6;
constexpr uint32_t kLaneTiles = 8;
constexpr int kLaneStep = 4;             // tiles of a lane in flight
constexpr uint32_t kRunBig = 0x8000u;    // a long run's count: of a surfel with slots of its own
constexpr uint32_t kChunkTiles = 4 * kGroup;
#ifndef CGV2_FIRST_CHUNKS
#define CGV2_FIRST_CHUNKS 2
#endif
constexpr uint32_t kFirstTiles = CGV2_FIRST_CHUNKS * kChunkTiles;
// Atomics on one address complete every 13 ns, whichever XCD they come from: a tile of 32,767 entries (the
// horizon of a 640x480 view of 5 M surfels) alone takes 0.43 ms.  Launches of few tiles, whose lists can be
// that long, count into kSets counters per tile (workgroup b into set b % kSets), where the bins have room for
// lists that can queue on one counter (kSetsSlots slots a tile: 0.8 us).
constexpr int kSets = 8;
constexpr int64_t kSetsMaxTiles = 4096;
constexpr int64_t kSetsSlots = 64;

// Small-rect runs pack a surfel's index within its run into the top 8 bits of an entry's rank (a tile lists
// each of a view's n surfels at most once).
constexpr int kRankBits = 24;
static_assert(kStageBlock == 256, "a run's index takes 8 bits of the rank");
__device__ __forceinline__ bool small_rects(const uint32_t* vstart, const int64_t* needed, int V, int64_t n) {
  const uint64_t vis = vstart[V];
  return vis >= (uint64_t)kLaneMin * (uint32_t)V && (uint64_t)*needed <= kSmallRect * vis &&
         n <= ((int64_t)1 << kRankBits);
}

// A view's tiles and their counters.
struct TileMap {
  uint32_t tiles_x, tiles_y, m;  // m: tiles of all views
  int sets;
  __device__ __forceinline__ uint32_t counter(uint32_t tx, uint32_t ty, bool small) const {
    return small ? tx * tiles_y + ty : ty * tiles_x + tx;
  }
  // the counter of tile i of the call's views
  __device__ __forceinline__ uint32_t counter_of(uint32_t i, bool small) const {
    if (!small) return i;
    const uint32_t tiles = tiles_x * tiles_y, v = i / tiles, t = i - v * tiles, ty = t / tiles_x;
    return v * tiles + counter(t - ty * tiles_x, ty, true);
  }
  // the first counter of view v in the set of this workgroup
  __device__ __forceinline__ uint32_t base(int v) const {
    return (uint32_t)v * tiles_x * tiles_y + (sets > 1 ? blockIdx.x % kSets * m : 0u);
  }
};

// One visible surfel as the staging sees it.
struct StageSurfel {
  uint32_t tx0, ty0, w, total;
  float4 r0;
  float depth;
  Reach q;
};

__device__ __forceinline__ void stage_rect(const uint16_t* rect, int64_t vi, StageSurfel& u) {
  uint32_t tx1, ty1;
  tile_rect(rect + 4 * vi, u.tx0, u.ty0, tx1, ty1);
  u.w = tx1 - u.tx0;
  u.total = u.w * (ty1 - u.ty0);
}

__device__ __forceinline__ void stage_surfel(const float* rec, int64_t vi, StageSurfel& u) {
  const float4* rp = (const float4*)(rec + vi * kRec);
  const float4 r1 = rp[1], r2 = rp[2], r4 = rp[4];
  u.r0 = rp[0];
  u.depth = r2.w;
  reach_setup(r1.x * kInvSqrt2, r1.y * kInvSqrt2, r1.z * kInvSqrt2, r1.w * kInvSqrt2, r2.x, r2.y, r2.z, r4.w, u.q);
}

// Does the surfel reach rect tile k (counter c of its view)?
__device__ __forceinline__ bool stage_tile(const StageSurfel& u, uint32_t k, const TileMap& tm, bool small,
                                           uint32_t& c) {
  const uint32_t tx = u.tx0 + k % u.w, ty = u.ty0 + k / u.w;
  c = tm.counter(tx, ty, small);
  // the tile-relative centre exactly as the renderer stages it
  const float fox = (float)(tx * kTile), foy = (float)(ty * kTile);
  return reach_cell(u.q, (u.r0.x - fox) + u.r0.z, (u.r0.y - foy) + u.r0.w, 0, 0, kTile);
}

// A staged entry is (counter, rank there | tag).
//
// Stages up to N tiles per lane (keep[j]: tile counter c[j] is reached) of a run's lanes: the ranks by
// returning atomics, all in flight before their results are used, and the entries packed from *slots (LDS) on.
template <int N>
__device__ __forceinline__ void stage_packed(const bool (&keep)[N], const uint32_t (&c)[N], uint32_t tag,
                                             uint32_t* __restrict__ cnt, uint32_t* slots, uint2* __restrict__ out) {
  const unsigned lane = threadIdx.x & 63u;
  const unsigned long long lt = (1ull << lane) - 1ull;
  uint32_t r[N];
#pragma unroll
  for (int j = 0; j < N; ++j) r[j] = keep[j] ? atomicAdd(cnt + c[j], 1u) : 0u;
  uint32_t total = 0;
#pragma unroll
  for (int j = 0; j < N; ++j) total += (uint32_t)__popcll(__ballot(keep[j]));
  if (total == 0) return;
  uint32_t base = 0;
  if ((__ballot(true) & lt) == 0) base = atomicAdd(slots, total);
  base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const unsigned long long b = __ballot(keep[j]);
    if (keep[j]) out[base + (uint32_t)__popcll(b & lt)] = make_uint2(c[j], r[j] | tag);
    base += (uint32_t)__popcll(b);
  }
}

// Rect tiles [kb, ke) of surfel u by the kGroup lanes of a group, tile kb + g + 32 j on lane g: the entries
// packed from out[0] on; returns their number.  Four returning atomics are in flight per lane.
__device__ __forceinline__ uint32_t stage_group(const StageSurfel& u, uint32_t kb, uint32_t ke, const TileMap& tm,
                                                bool small, uint32_t tbase, uint32_t tag, uint32_t* __restrict__ cnt,
                                                uint2* __restrict__ out) {
  uint32_t at = 0;
  const uint32_t g = threadIdx.x % kGroup;
  const uint32_t shift = threadIdx.x & 63u & ~(uint32_t)(kGroup - 1);  // the group's lanes in its wave
  for (uint32_t k0 = kb; k0 < ke; k0 += 4 * kGroup) {
    uint32_t c[4] = {0, 0, 0, 0}, r[4];
    bool keep[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t k = k0 + g + (uint32_t)j * kGroup;
      keep[j] = k < ke && stage_tile(u, k, tm, small, c[j]);
      c[j] += tbase;
      r[j] = keep[j] ? atomicAdd(cnt + c[j], 1u) : 0u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t b = (uint32_t)(__ballot(keep[j]) >> shift);
      if (keep[j]) out[at + (uint32_t)__popc(b & ((1u << g) - 1u))] = make_uint2(c[j], r[j] | tag);
      at += (uint32_t)__popc(b);
    }
  }
  return at;
}

// chunk queue entry: (index into 'visible', view << 16 | chunk, first staged slot, entries staged there by
// k_stage_big); chunk c covers rect tiles [kFirstTiles + c kChunkTiles, ... + kChunkTiles).  A surfel with
// T > kFirstTiles tiles queues ceil((T - kFirstTiles) / kChunkTiles) < T / kChunkTiles chunks, so
// capacity / kChunkTiles + 1 entries hold every queue whose rect slots fit the capacity (the staging does
// not run otherwise).  Called by the lanes of one group together.
__device__ __forceinline__ void queue_chunks(uint32_t vis, int v, uint32_t total, uint32_t at,
                                             uint4* __restrict__ chunks, uint32_t* __restrict__ n_chunks,
                                             uint32_t max_chunks) {
  const uint32_t g = threadIdx.x % kGroup;
  const uint32_t nc = (total - kFirstTiles + kChunkTiles - 1) / kChunkTiles;
  uint32_t base = 0;
  if (g == 0) base = atomicAdd(n_chunks, nc);
  base = __shfl(base, (int)(threadIdx.x & 63u & ~(uint32_t)(kGroup - 1)), 64);
  for (uint32_t c = g; c < nc; c += kGroup)
    if (base + c < max_chunks) chunks[base + c] = make_uint4(vis, ((uint32_t)v << 16) | c, at + c * kChunkTiles, 0u);
}

// Every visible entry's depth goes to depth[].  A short run's surfels each pack their entries at the start
// of their own rect slots (count[entry]).  A long run's rect slots hold the lanes' entries, packed, then the
// slots of each surfel for the groups; of its b such surfels, number k has its entries at voff[first + k]
// and kRunBig | their count in count[first + k], and the lanes' follow at index b (when b is not all of them).
__global__ __launch_bounds__(kStageBlock, 5) void k_stage(const uint16_t* __restrict__ rect,
                                                       const float* __restrict__ rec, int64_t n, TileMap tm, int V,
                                                       const int64_t* __restrict__ needed,
                                                       const uint32_t* __restrict__ visible,
                                                       const uint32_t* __restrict__ vstart, uint32_t* voff,
                                                       uint32_t* __restrict__ cnt,
                                                       uint2* __restrict__ st, uint16_t* __restrict__ count,
                                                       float* __restrict__ depth, uint4* __restrict__ chunks,
                                                       uint32_t* __restrict__ n_chunks, uint32_t max_chunks,
                                                       const int32_t* __restrict__ status) {
  __shared__ uint32_t big[kStageBlock];  // a long run's surfels for the groups
  __shared__ uint32_t n_big, slots, own;
  const int v = blockIdx.y;
  if (*status != 0) return;
  const uint32_t vs = vstart[v], nv = vstart[v + 1] - vs;
  const uint32_t* list = visible + vs;
  const uint32_t g = threadIdx.x % kGroup, grp = threadIdx.x / kGroup;
  const uint32_t tbase = tm.base(v);
  if (!small_rects(vstart, needed, V, n)) {
    for (uint32_t e = blockIdx.x * kGroups + grp; e < nv; e += gridDim.x * kGroups) {
      const uint32_t at = voff[vs + e];
      const int64_t vi = (int64_t)v * n + list[e];
      StageSurfel u;
      stage_rect(rect, vi, u);
      stage_surfel(rec, vi, u);
      const uint32_t k = stage_group(u, 0u, min(u.total, kFirstTiles), tm, false, tbase, 0u, cnt, st + at);
      if (g == 0) {
        count[vs + e] = (uint16_t)k;
        depth[vs + e] = u.depth;
      }
      if (u.total > kFirstTiles) queue_chunks(vs + e, v, u.total, at + kFirstTiles, chunks, n_chunks, max_chunks);
    }
    return;
  }
  for (uint32_t e0 = blockIdx.x * kStageBlock; e0 < nv; e0 += gridDim.x * kStageBlock) {
    const uint32_t e = e0 + threadIdx.x;
    const bool live = e < nv;
    if (threadIdx.x == 0) n_big = slots = own = 0u;
    __syncthreads();
    const int64_t vi = (int64_t)v * n + (live ? list[e] : 0u);
    const uint32_t at = voff[vs + e0];
    StageSurfel u;
    u.total = 0;
    if (live) stage_rect(rect, vi, u);
    const bool mine = live && u.total <= kLaneTiles;
    if (mine) {
      stage_surfel(rec, vi, u);
      depth[vs + e] = u.depth;
      atomicAdd(&own, u.total);
    } else if (live) {
      big[atomicAdd(&n_big, 1u)] = threadIdx.x;
    }
    for (uint32_t k0 = 0; __ballot(mine && k0 < u.total) != 0; k0 += kLaneStep) {
      bool keep[kLaneStep];
      uint32_t c[kLaneStep] = {};
#pragma unroll
      for (int j = 0; j < kLaneStep; ++j) {
        keep[j] = mine && k0 + j < u.total && stage_tile(u, k0 + j, tm, true, c[j]);
        c[j] += tbase;
      }
      stage_packed<kLaneStep>(keep, c, threadIdx.x << kRankBits, cnt, &slots, st + at);
    }
    __syncthreads();
    const uint32_t nb = n_big;
    if (live && threadIdx.x >= nb) count[vs + e] = (uint16_t)(threadIdx.x == nb ? slots : 0u);
    if (live && threadIdx.x == nb) voff[vs + e] = at;
    for (uint32_t b = grp; b < nb; b += kGroups) {
      const uint32_t eb = e0 + big[b];
      const int64_t vb = (int64_t)v * n + list[eb];
      stage_rect(rect, vb, u);
      stage_surfel(rec, vb, u);
      uint32_t to = 0;
      if (g == 0) to = atomicAdd(&own, u.total);
      to = at + __shfl(to, (int)(threadIdx.x & 63u & ~(uint32_t)(kGroup - 1)), 64);
      const uint32_t k = stage_group(u, 0u, min(u.total, kFirstTiles), tm, true, tbase, big[b] << kRankBits,
                                     cnt, st + to);
      if (g == 0) {
        voff[vs + e0 + b] = to;
        count[vs + e0 + b] = (uint16_t)(kRunBig | k);
        depth[vs + eb] = u.depth;
      }
      if (u.total > kFirstTiles) queue_chunks(vs + eb, v, u.total, to + kFirstTiles, chunks, n_chunks, max_chunks);
    }
    __syncthreads();  // the list and the counters are rewritten by the next run
  }
}

// The queued chunks of the large rects, one chunk per group.
__global__ __launch_bounds__(kStageBlock) void k_stage_big(const uint16_t* __restrict__ rect,
                                                           const float* __restrict__ rec, int64_t n, TileMap tm, int V,
                                                           const int64_t* __restrict__ needed,
                                                           const uint32_t* __restrict__ visible,
                                                           const uint32_t* __restrict__ vstart,
                                                           uint32_t* __restrict__ cnt,
                                                           uint2* __restrict__ st, uint4* __restrict__ chunks,
                                                           const uint32_t* __restrict__ n_chunks, uint32_t max_chunks,
                                                           const int32_t* __restrict__ status) {
  if (*status != 0) return;
  const uint32_t nc = min(*n_chunks, max_chunks);
  const bool small = small_rects(vstart, needed, V, n);
  for (uint32_t it = (blockIdx.x * blockDim.x + threadIdx.x) / kGroup; it < nc;
       it += gridDim.x * blockDim.x / kGroup) {
    const uint4 q = chunks[it];
    const int v = (int)(q.y >> 16);
    const int64_t vi = (int64_t)v * n + visible[q.x];
    StageSurfel u;
    stage_rect(rect, vi, u);
    stage_surfel(rec, vi, u);
    const uint32_t kb = kFirstTiles + (q.y & 0xffffu) * kChunkTiles;
    const uint32_t k = stage_group(u, kb, min(u.total, kb + kChunkTiles), tm, small, tm.base(v), 0u, cnt, st + q.z);
    if (threadIdx.x % kGroup == 0) chunks[it].w = k;
  }
}

// Multi-workgroup form of the tile scan for more than kScanChunk tiles: chunk sums, then each chunk scanned
// with the sum of those before it (us, two launches against one workgroup: 32,400 tiles 31 -> 10, 53,600
// tiles 50 -> 10).
__global__ __launch_bounds__(kScanBlock) void k_tile_sums(const uint32_t* __restrict__ cnt, TileMap tm, int V,
                                                          int64_t n, const uint32_t* __restrict__ vstart,
                                                          const int64_t* __restrict__ needed,
                                                          uint64_t* __restrict__ sums) {
  __shared__ uint64_t lds[2 * kScanWaves];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk;
  const bool small = small_rects(vstart, needed, V, n);
  uint64_t c = 0;
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t idx = base + (int64_t)k * kScanBlock + threadIdx.x;
    if (idx < tm.m) c += cnt[tm.counter_of((uint32_t)idx, small)];
  }
  const uint64_t t = block_sum(c, lds);
  if (threadIdx.x == 0) sums[blockIdx.x] = t;
}

// (column-major counters become their first slots; row-major ones have them in ranges)
__global__ __launch_bounds__(kScanBlock) void k_tile_apply(uint32_t* __restrict__ cnt, TileMap tm, int V, int64_t n,
                                                           const uint32_t* __restrict__ vstart,
                                                           const int64_t* __restrict__ needed, SortItems items,
                                                           const uint64_t* __restrict__ sums,
                                                           uint32_t* __restrict__ ranges) {
  __shared__ uint64_t lds[2 * kScanWaves], red[2][kScanWaves], tot[2];
  {
    // the totals of the chunks before this one, and of all
    uint64_t before = 0, all = 0;
    for (uint32_t j = threadIdx.x; j < gridDim.x; j += kScanBlock) {
      const uint64_t x = sums[j];
      before += j < blockIdx.x ? x : 0;
      all += x;
    }
    before = block_sum(before, red[0]);
    all = block_sum(all, red[1]);
    if (threadIdx.x == 0) {
      tot[0] = before;
      tot[1] = all;
    }
    __syncthreads();
  }
  const uint64_t carry = tot[0];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
  uint64_t vals[kScanItems];
  const bool small = small_rects(vstart, needed, V, n);
  uint32_t at[kScanItems];
  for (int k = 0; k < kScanItems; ++k) {
    at[k] = base + k < tm.m ? tm.counter_of((uint32_t)(base + k), small) : 0u;
    vals[k] = base + k < tm.m ? cnt[at[k]] : 0;
  }
  uint32_t tile[kScanItems], len[kScanItems];
  for (int k = 0; k < kScanItems; ++k) {
    tile[k] = (uint32_t)(base + k);
    len[k] = (uint32_t)vals[k];
  }
  list_items(items, tile, len);
  block_scan(vals, lds);
  for (int k = 0; k < kScanItems; ++k)
    if (base + k < tm.m) {
      ranges[base + k] = (uint32_t)(vals[k] + carry);
      if (small) cnt[at[k]] = (uint32_t)(vals[k] + carry);
    }
  if (blockIdx.x == 0 && threadIdx.x == 0) ranges[tm.m] = (uint32_t)tot[1];
}

// Staged entries to their tiles: a group per surfel of short runs, a workgroup per long run, then a group
// per queued chunk.
__global__ __launch_bounds__(kStageBlock) void k_place(const uint32_t* __restrict__ visible,
                                                       const uint32_t* __restrict__ vstart, int V, int64_t n,
                                                       const int64_t* __restrict__ needed,
                                                       const uint32_t* __restrict__ voff,
                                                       const uint16_t* __restrict__ count,
                                                       const float* __restrict__ depth, const uint2* __restrict__ st,
                                                       const uint32_t* __restrict__ cnt, int sets,
                                                       const uint32_t* __restrict__ ranges,
                                                       const uint4* __restrict__ chunks,
                                                       const uint32_t* __restrict__ n_chunks, uint32_t max_chunks,
                                                       uint64_t* __restrict__ keys, const int32_t* __restrict__ status) {
  __shared__ uint64_t key[kStageBlock];
  __shared__ uint32_t at_s[kStageBlock], cnt_s[kStageBlock];
  __shared__ uint32_t n_big;
  if (*status != 0) return;
  const int v = blockIdx.y;
  const uint32_t vs = vstart[v], nv = vstart[v + 1] - vs;
  const uint32_t g = threadIdx.x % kGroup, grp = threadIdx.x / kGroup;
  const bool small = small_rects(vstart, needed, V, n);
  const uint32_t* __restrict__ first = sets == 1 && !small ? ranges : cnt;  // first slot of each counter
  auto key_of = [&](uint32_t e) { return (uint64_t)__float_as_uint(depth[e]) << 32 | visible[e]; };
  if (!small) {
    for (uint32_t e = blockIdx.x * kGroups + grp; e < nv; e += gridDim.x * kGroups) {
      const uint32_t k = count[vs + e];
      const uint2* p = st + voff[vs + e];
      const uint64_t x = key_of(vs + e);
      for (uint32_t j = g; j < k; j += kGroup) keys[first[p[j].x] + p[j].y] = x;
    }
  } else {
    auto put = [&](const uint2& q) {
      keys[first[q.x] + (q.y & ((1u << kRankBits) - 1u))] = key[q.y >> kRankBits];
    };
    for (uint32_t e0 = blockIdx.x * kStageBlock; e0 < nv; e0 += gridDim.x * kStageBlock) {
      const uint32_t e = vs + e0 + threadIdx.x;
      const bool live = e0 + threadIdx.x < nv;
      if (threadIdx.x == 0) n_big = 0u;
      __syncthreads();
      if (live) {
        key[threadIdx.x] = key_of(e);
        at_s[threadIdx.x] = voff[e];
        cnt_s[threadIdx.x] = count[e];
      }
      const unsigned long long flagged = __ballot(live && (cnt_s[threadIdx.x] & kRunBig) != 0u);
      if ((threadIdx.x & 63u) == 0u && flagged) atomicAdd(&n_big, (uint32_t)__popcll(flagged));
      __syncthreads();
      const uint32_t nb = n_big;
      if (e0 + nb < nv && nb < kStageBlock) {
        const uint2* p = st + at_s[nb];
        const uint32_t k = cnt_s[nb];
        for (uint32_t j = threadIdx.x; j < k; j += kStageBlock) put(p[j]);
      }
      for (uint32_t b = grp; b < nb; b += kGroups) {
        const uint2* p = st + at_s[b];
        const uint32_t k = cnt_s[b] & (kRunBig - 1u);
        for (uint32_t j = g; j < k; j += kGroup) put(p[j]);
      }
      __syncthreads();
    }
  }
  const uint32_t nc = min(*n_chunks, max_chunks);
  for (uint32_t it = ((blockIdx.y * gridDim.x + blockIdx.x) * kStageBlock + threadIdx.x) / kGroup; it < nc;
       it += gridDim.y * gridDim.x * kGroups) {
    const uint4 q = chunks[it];
    const uint64_t x = key_of(q.x);
    for (uint32_t j = g; j < q.w; j += kGroup) keys[first[st[q.z + j].x] + st[q.z + j].y] = x;
  }
}

// ---- per-tile sort of up to kWaveSort keys in one wave's registers ----------------------------------
// A bitonic network over 64 E keys, E per lane in blocked order (key x = E lane + e).  Steps whose partner
// distance j is below E pair two registers of a lane; the others pair register e of lanes l and l ^ j / E,
// exchanged with DPP (distances 1, 2, 4, 8) or the gfx950 row-swap instructions (16, 32), so the sort
// touches neither LDS nor a barrier.  A compare-exchange keeps the minimum where the lane holds the
// lower index of an ascending pair or the upper one of a descending pair.

// value of lane l ^ D for D = 1, 2, 4, 8 (DPP within rows of 16)
template <int D>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
  const int i = (int)x;
  if constexpr (D == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, i, 0xB1, 0xf, 0xf, false);   // [1,0,3,2]
  if constexpr (D == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, i, 0x4E, 0xf, 0xf, false);   // [2,3,0,1]
  if constexpr (D == 4) {  // l ^ 7 (row_half_mirror), then ^ 3 (quad_perm [3,2,1,0])
    const int h = __builtin_amdgcn_update_dpp(0, i, 0x141, 0xf, 0xf, false);
    return (uint32_t)__builtin_amdgcn_update_dpp(0, h, 0x1B, 0xf, 0xf, false);
  }
  if constexpr (D == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, i, 0x128, 0xf, 0xf, false);  // row_ror:8
}

// register e of lanes l and l ^ D: keep the smaller key where keep_min, else the larger
template <int D>
__device__ __forceinline__ void cx_lanes(uint64_t& v, bool keep_min) {
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  uint64_t a, b;  // the two keys of the pair (which one is this lane's does not matter)
  if constexpr (D <= 8) {
    a = v;
    b = ((uint64_t)lane_xor<D>(hi) << 32) | lane_xor<D>(lo);
  } else {
    // a row swap of a register with itself leaves this lane's key in one result and its partner's in
    // the other
    const auto rl = D == 16 ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false)
                            : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto rh = D == 16 ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false)
                            : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    a = ((uint64_t)rh[0] << 32) | rl[0];
    b = ((uint64_t)rh[1] << 32) | rl[1];
  }
  v = ((a < b) == keep_min) ? a : b;
}

// registers x (lower index) and y of one lane, ascending or descending
__device__ __forceinline__ void cx_regs(uint64_t& x, uint64_t& y, bool asc) {
  const bool c = (x < y) == asc;
  const uint64_t p = c ? x : y, q = c ? y : x;
  x = p;
  y = q;
}

template <int E, int K, int J>
__device__ __forceinline__ void bitonic_step(uint64_t (&v)[E], unsigned lane) {
  if constexpr (J >= E) {
    // K >= 2 J >= 2 E: the direction follows bit K / E of the lane (all ascending in the last merge)
    const bool asc = K >= 64 * E || (lane & (unsigned)(K / E)) == 0u;
    const bool keep_min = ((lane & (unsigned)(J / E)) == 0u) == asc;
#pragma unroll
    for (int e = 0; e < E; ++e) cx_lanes<J / E>(v[e], keep_min);
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (e & J) continue;
      const bool asc = K < E ? (e & K) == 0 : (K >= 64 * E || (lane & (unsigned)(K / E)) == 0u);
      cx_regs(v[e], v[e | J], asc);
    }
  }
  if constexpr (J > 1) bitonic_step<E, K, J / 2>(v, lane);
}

template <int E, int K = 2>
__device__ __forceinline__ void wave_bitonic(uint64_t (&v)[E], unsigned lane) {
  bitonic_step<E, K, K / 2>(v, lane);
  if constexpr (K < 64 * E) wave_bitonic<E, 2 * K>(v, lane);
}

// keys[a, a + len) sorted by one wave (len <= 64 E): the ids written in order, or (kBack) the keys; the
// tail is padded with the largest key
template <int E, bool kBack>
__device__ __forceinline__ void sort_list_wave(uint64_t* keys, uint32_t* __restrict__ ids, uint32_t a, int len,
                                               unsigned lane) {
  uint64_t v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int x = E * (int)lane + e;
    v[e] = x < len ? keys[a + x] : ~0ull;
  }
  wave_bitonic<E>(v, lane);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int x = E * (int)lane + e;
    if (x >= len) continue;
    if (kBack) keys[a + x] = v[e];
    else ids[a + x] = (uint32_t)v[e];
  }
}

// One wave per tile for lists up to kWaveSort entries, with the smallest E that holds them; the waves of
// the workgroups past the tiles sort the chunks of the longer lists (the keys stay in place for k_merge).
__global__ __launch_bounds__(256, 5) void k_sort_wave(const uint32_t* __restrict__ ranges, int num_tiles,
                                                      SortItems items, uint64_t* keys, uint32_t* __restrict__ ids,
                                                      const int32_t* __restrict__ status) {
  if (*status != 0) return;
  const unsigned lane = threadIdx.x & 63u;
  const uint32_t t = blockIdx.x * 4u + (threadIdx.x >> 6);
  const uint32_t first = ((uint32_t)num_tiles + 3u) / 4u * 4u;  // the tiles' waves
  if (t < first) {
    if (t >= (uint32_t)num_tiles) return;
    const uint32_t a = ranges[t];
    const int len = (int)(ranges[t + 1] - a);
    if (len == 0 || len > kWaveSort) return;
    if (len <= 64) sort_list_wave<1, false>(keys, ids, a, len, lane);
    else if (len <= 128) sort_list_wave<2, false>(keys, ids, a, len, lane);
    else if (len <= 256) sort_list_wave<4, false>(keys, ids, a, len, lane);
    else if (len <= 512) sort_list_wave<8, false>(keys, ids, a, len, lane);
    else sort_list_wave<16, false>(keys, ids, a, len, lane);
    return;
  }
  const uint32_t n = *items.count;
  for (uint32_t k = t - first; k < n; k += gridDim.x * 4u - first) {
    const uint2 it = items.item[k];
    const uint32_t a = ranges[it.x], len = ranges[it.x + 1] - a, cs = chunk_size(len);
    sort_list_wave<16, true>(keys, ids, a + it.y * cs, (int)min(cs, len - it.y * cs), lane);
  }
}

// Merge of a long list's sorted chunks, one workgroup per chunk: its keys (four per thread) are ranked in
// every other chunk of the list, staged through LDS with the next one's loads in flight; a key's slot is
// its index plus those ranks (the keys differ).  Long lists thus spread over as many workgroups as they have
// chunks: for a 640x480 view of 5 M surfels (659 lists above 1,024, up to 32,767) both sorts take 173 us,
// against 693 with one workgroup per list (LDS bitonic sort up to 16,384 entries, then pairwise merges);
// 10 M surfels in 8 views (4,768 lists up to 3,810) 348 against 640.
constexpr int kMergeBlock = 256;
constexpr int kMergeKeys = kWaveSort / kMergeBlock;

__global__ __launch_bounds__(kMergeBlock) void k_merge(const uint32_t* __restrict__ ranges, SortItems items,
                                                       const uint64_t* __restrict__ keys, uint32_t* __restrict__ ids,
                                                       const int32_t* __restrict__ status) {
  __shared__ uint64_t s[2][kWaveSort];
  if (*status != 0) return;
  const uint32_t n = *items.count;
  for (uint32_t k = blockIdx.x; k < n; k += gridDim.x) {
    const uint2 it = items.item[k];
    const uint32_t a = ranges[it.x], len = ranges[it.x + 1] - a, cs = chunk_size(len), nc = chunk_count(len);
    const uint32_t own = it.y * cs, ol = min(cs, len - own);
    uint64_t x[kMergeKeys], next[kMergeKeys];
    uint32_t pos[kMergeKeys];
#pragma unroll
    for (int j = 0; j < kMergeKeys; ++j) {
      const uint32_t e = threadIdx.x + (uint32_t)j * kMergeBlock;
      x[j] = e < ol ? keys[a + own + e] : ~0ull;
      pos[j] = e;
    }
    // keys of chunk c (padded with the largest key: above every key)
    auto load = [&](uint32_t c) {
#pragma unroll
      for (int j = 0; j < kMergeKeys; ++j) {
        const uint32_t e = threadIdx.x + (uint32_t)j * kMergeBlock;
        next[j] = c < nc && e < cs && c * cs + e < len ? keys[a + c * cs + e] : ~0ull;
      }
    };
    uint32_t c = it.y == 0 ? 1u : 0u;
    load(c);
    for (int buf = 0; c < nc; buf ^= 1) {
#pragma unroll
      for (int j = 0; j < kMergeKeys; ++j) s[buf][threadIdx.x + j * kMergeBlock] = next[j];
      __syncthreads();  // (the other buffer's readers are behind the barrier before)
      c += c + 1u == it.y ? 2u : 1u;
      load(c);
      // number of keys below x[j]: kWaveSort is a power of two and the chunk padded to it
      uint32_t r[kMergeKeys] = {};
#pragma unroll
      for (int step = kWaveSort / 2; step > 0; step >>= 1) {
#pragma unroll
        for (int j = 0; j < kMergeKeys; ++j) r[j] += s[buf][r[j] + (uint32_t)step - 1u] < x[j] ? (uint32_t)step : 0u;
      }
#pragma unroll
      for (int j = 0; j < kMergeKeys; ++j) pos[j] += r[j] + (s[buf][r[j]] < x[j] ? 1u : 0u);
    }
#pragma unroll
    for (int j = 0; j < kMergeKeys; ++j) {
      const uint32_t e = threadIdx.x + (uint32_t)j * kMergeBlock;
      if (e < ol) ids[a + pos[j]] = (uint32_t)x[j];
    }
    __syncthreads();  // the next item rewrites the buffers
  }
}

// ---- launch order of the render kernels --------------------------------------------------------
// A render launch holds few tiles per wave slot and tile costs vary by orders of magnitude, so the
// heaviest tiles go first (longest-processing-time order): a stable counting sort of a view chunk's
// tiles by a log-scale bucket of their list length, descending, tiles in index order within a bucket.
constexpr int kOrdBuckets = 64;
static_assert(kOrdBuckets == 64, "the order kernels keep one bucket per lane");
constexpr int kOrdChunk = 1024;  // tiles per workgroup (16 waves)

__device__ __forceinline__ int order_bucket(uint32_t len) {
  if (len == 0) return 0;
  const int e = 31 - __clz(len);  // floor(log2 len)
  const int half = e >= 1 ? (int)((len >> (e - 1)) & 1u) : 0;
  const int b = 2 * e + 1 + half;
  return b < kOrdBuckets ? b : kOrdBuckets - 1;
}

// lanes of this wave whose bucket equals the calling lane's (bk in [0, kOrdBuckets), -1 for none; the
// result is meaningful for bk >= 0): one ballot per bit of the 6-bit bucket
__device__ __forceinline__ unsigned long long same_bucket(int bk) {
  unsigned long long same = __ballot(bk >= 0);
#pragma unroll
  for (int b = 0; b < 6; ++b) {
    const bool bit = bk >= 0 && ((bk >> b) & 1);
    const unsigned long long B = __ballot(bit);
    same &= bit ? B : ~B;
  }
  return same;
}

__global__ __launch_bounds__(kOrdChunk) void k_order_hist(const uint32_t* __restrict__ ranges, int64_t base, int T,
                                                          uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[kOrdBuckets];
  if (threadIdx.x < kOrdBuckets) h[threadIdx.x] = 0;
  __syncthreads();
  const int t = blockIdx.x * kOrdChunk + threadIdx.x;
  if (t < T) atomicAdd(&h[order_bucket(ranges[base + t + 1] - ranges[base + t])], 1u);
  __syncthreads();
  if (threadIdx.x < kOrdBuckets) hist[(int64_t)blockIdx.x * kOrdBuckets + threadIdx.x] = h[threadIdx.x];
}

// one wave: hist[c][k] -> first slot of bucket k's tiles of chunk c, buckets in descending order
__global__ __launch_bounds__(64) void k_order_scan(uint32_t* __restrict__ hist, int nc) {
  const int k = threadIdx.x;  // bucket
  uint32_t tot = 0;
#pragma unroll 16
  for (int c = 0; c < nc; ++c) tot += hist[(int64_t)c * kOrdBuckets + k];
  // inclusive suffix sum over the buckets k and above, then exclusive
  uint32_t x = tot;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = __shfl_down(x, d, 64);
    if (k + d < 64) x += y;
  }
  uint32_t run = x - tot;
#pragma unroll 16
  for (int c = 0; c < nc; ++c) {
    const uint32_t v = hist[(int64_t)c * kOrdBuckets + k];
    hist[(int64_t)c * kOrdBuckets + k] = run;
    run += v;
  }
}

__global__ __launch_bounds__(kOrdChunk) void k_order_place(const uint32_t* __restrict__ ranges, int64_t base, int T,
                                                           const uint32_t* __restrict__ hist,
                                                           uint32_t* __restrict__ order) {
  constexpr int kWaves = kOrdChunk / 64;
  __shared__ uint32_t wc[kWaves][kOrdBuckets];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int t = blockIdx.x * kOrdChunk + threadIdx.x;
  const int bk = t < T ? order_bucket(ranges[base + t + 1] - ranges[base + t]) : -1;
  const unsigned long long lt = (1ull << lane) - 1ull;
  const unsigned long long same = same_bucket(bk);
  const uint32_t rank = bk >= 0 ? (uint32_t)__popcll(same & lt) : 0u;
  wc[w][lane] = 0;  // kOrdBuckets == 64: one bucket per lane
  // the first lane of each bucket present writes its count (after the zeroing: one wave, LDS in order)
  if (bk >= 0 && rank == 0) wc[w][bk] = (uint32_t)__popcll(same);
  __syncthreads();
  if (threadIdx.x < kOrdBuckets) {
    uint32_t run = 0;
    for (int q = 0; q < kWaves; ++q) {
      const uint32_t v = wc[q][threadIdx.x];
      wc[q][threadIdx.x] = run;
      run += v;
    }
  }
  __syncthreads();
  if (bk >= 0) order[hist[(int64_t)blockIdx.x * kOrdBuckets + bk] + wc[w][bk] + rank] = (uint32_t)t;
}

// One workgroup for up to kScanChunk tiles of at most kMaxViews views (the common single-view case):
// the tile scan and the launch order of k_order_hist / k_order_scan / k_order_place in
// one launch, the same results.  Wave w owns the contiguous tiles [w per, (w + 1) per) and loads their
// counts once, all at the same time (lane l holds tiles w per + 64 k + l); the scan runs over those
// registers (wave scans in k order, one LDS exchange of the 16 wave totals); the order takes LDS counts
// per (wave, bucket), one exchange of the 16 x 64 counts into first slots, and a placing pass with
// stable ranks from the lanes that share a bucket (same_bucket).

// A tile's count is the sum over its counters (one per set), which become their first slots (unless they are
// one set in row order: ranges holds those).  order may be null.
__global__ __launch_bounds__(kScanBlock) void k_tile_scan_order(uint32_t* __restrict__ cnt, TileMap tm, int V,
                                                                int64_t n, const uint32_t* __restrict__ vstart,
                                                                const int64_t* __restrict__ needed, SortItems items,
                                                                uint32_t* __restrict__ ranges,
                                                                uint32_t* __restrict__ order) {
  const int m = (int)tm.m;
  const bool small = small_rects(vstart, needed, V, n);
  __shared__ uint32_t wtot[kScanWaves];
  __shared__ uint32_t wc[kScanWaves][kOrdBuckets];
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6;
  // kScanWaves * per >= m, per a multiple of 64 and at most 64 kScanItems (m <= kScanChunk)
  const int per = ((m + kScanBlock - 1) / kScanBlock) * 64;
  const int i0 = w * per, i1 = min(m, i0 + per);
  uint32_t c[kScanItems], at[kScanItems];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int i = i0 + 64 * k + lane;
    const bool in = 64 * k < per && i < i1;
    at[k] = in ? tm.counter_of((uint32_t)i, small) : 0u;
    c[k] = in ? cnt[at[k]] : 0u;
  }
  if (tm.sets > 1) {
    // (at most kSetsMaxTiles tiles)
#pragma unroll
    for (int k = 0; k < kSetsMaxTiles / kScanBlock; ++k) {
      if (64 * k >= per || i0 + 64 * k + lane >= i1) continue;
#pragma unroll
      for (int q = 1; q < kSets; ++q) c[k] += cnt[q * m + at[k]];
    }
  }
  // tile scan: exclusive prefix sums within the wave's tiles, then the wave offsets
  uint32_t ex[kScanItems];
  uint32_t carry = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const uint32_t inc = wave_scan_u32(c[k]);
    ex[k] = carry + inc - c[k];
    carry += lane63(inc);
  }
  if (lane == 0) wtot[w] = carry;
  const unsigned long long lt = (1ull << lane) - 1ull;
  wc[w][lane] = 0;  // kOrdBuckets == 64: one bucket per lane
  __syncthreads();
  uint32_t off = 0, total = 0;
  for (int q = 0; q < kScanWaves; ++q) {
    const uint32_t v = wtot[q];
    off += q < w ? v : 0u;
    total += v;
  }
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int i = i0 + 64 * k + lane;
    if (64 * k >= per || i >= i1) continue;
    ranges[i] = off + ex[k];
    if (tm.sets == 1 && small) cnt[at[k]] = off + ex[k];
  }
  if (tm.sets > 1) {
#pragma unroll
    for (int k = 0; k < kSetsMaxTiles / kScanBlock; ++k) {
      if (64 * k >= per || i0 + 64 * k + lane >= i1) continue;
      uint32_t x[kSets], first = off + ex[k];
#pragma unroll
      for (int q = 0; q < kSets; ++q) x[q] = cnt[q * m + at[k]];
#pragma unroll
      for (int q = 0; q < kSets; ++q) {
        cnt[q * m + at[k]] = first;
        first += x[q];
      }
    }
  }
  if (t == 0) ranges[m] = total;
  uint32_t tile[kScanItems];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) tile[k] = (uint32_t)(i0 + 64 * k + lane);
  list_items(items, tile, c);
  if (!order) return;
  // counts per (wave, bucket), by LDS atomics that return nothing (no wait between the rows)
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (i0 + 64 * k >= i1) break;
    const int i = i0 + 64 * k + lane;
    if (i < i1) atomicAdd(&wc[w][order_bucket(c[k])], 1u);
  }
  __syncthreads();
  if (t < kOrdBuckets) {
    uint32_t tot = 0;
    for (int q = 0; q < kScanWaves; ++q) tot += wc[q][t];
    // buckets in descending order: bucket t starts after the tiles of the buckets above it
    const uint32_t inc = wave_scan_u32(tot);
    uint32_t run = lane63(inc) - inc;
    for (int q = 0; q < kScanWaves; ++q) {
      const uint32_t v = wc[q][t];
      wc[q][t] = run;
      run += v;
    }
  }
  __syncthreads();
  // wc[w][k]: next slot of bucket k for this wave's tiles
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (i0 + 64 * k >= i1) break;
    const int i = i0 + 64 * k + lane;
    const int bk = i < i1 ? order_bucket(c[k]) : -1;
    const unsigned long long same = same_bucket(bk);
    const uint32_t rank = (uint32_t)__popcll(same & lt);
    const uint32_t first = bk >= 0 ? wc[w][bk] : 0u;
    if (bk >= 0) order[first + rank] = (uint32_t)i;
    // after every lane's read above
    if (bk >= 0 && rank == 0) wc[w][bk] = first + (uint32_t)__popcll(same);
  }
}

}  // namespace cgv2

static int64_t scan_blocks(int64_t m) { return (m + cgv2::kScanChunk - 1) / cgv2::kScanChunk; }
static int64_t surf_blocks(int64_t m) { return (m + cgv2::kSurfChunk - 1) / cgv2::kSurfChunk; }

static int counter_sets(int64_t m, int64_t capacity) {
  return m <= cgv2::kSetsMaxTiles && capacity >= cgv2::kSetsSlots * m ? cgv2::kSets : 1;
}
// Counters that the workspace holds: of m tiles, and of any fewer (a workspace sized for an engine's largest image
// serves its smaller ones too).
static int64_t counter_room(int64_t m, int64_t capacity) {
  return std::max(m, cgv2::kSets * std::min(std::min(m, cgv2::kSetsMaxTiles), capacity / cgv2::kSetsSlots));
}

size_t cgv2_binsort_ws_layout(int64_t capacity, int V, int tiles, int64_t n, size_t* off) {
  // off: [0] tile counters (u32, counter_room) and, after those in use, the sort-item and chunk-queue
  //      counts, [1] chunk sums of the surfel scan (2 x u64 arrays), [2] chunks of the long lists (uint2), [3] scan totals
  //      (u64 x 2), [4] keys (u64, capacity), [5] staged entries (8 B, capacity), [11], [6], [7] per visible
  //      surfel: depth (f32), staged count (u16), first slot (u32, capacity), [8] chunk sums of the tile scan (u64)
  const int64_t m = (int64_t)V * tiles;
  const int64_t vn = (int64_t)V * n;
  const int64_t nsb = surf_blocks(vn > 0 ? vn : 1);
  const int64_t vis = std::min(vn, capacity);  // most visible surfels that are staged
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t r = o; o += (bytes + 255) & ~(size_t)255; return r; };
  off[0] = take(4 * (size_t)(counter_room(m, capacity) + 2));
  off[1] = take(16 * (size_t)(nsb + 1));
  off[2] = take(8 * (size_t)(capacity / (cgv2::kWaveSort / 2) + 1));
  off[3] = take(64);
  off[4] = take(8 * (size_t)capacity);
  off[5] = take(8 * (size_t)capacity);
  off[11] = take(6 * (size_t)vis);
  off[6] = off[11] + 4 * (size_t)vis;
  off[7] = take(4 * (size_t)(capacity + 1));
  off[8] = take(8 * (size_t)(scan_blocks(m) + 1));
  // [9] per-chunk bucket counts of the launch order (one view chunk at a time)
  const int64_t per = (int64_t)std::min(V, cgv2::kMaxViews) * tiles;
  off[9] = take(4 * (size_t)cgv2::kOrdBuckets * (size_t)((per + cgv2::kOrdChunk - 1) / cgv2::kOrdChunk + 1));
  // [10] the chunk queue of the large rects (see k_stage)
  off[10] = take(16 * (size_t)(capacity / cgv2::kChunkTiles + 1));
  return o;
}

hipError_t cgv2_launch_bin_sort(const cgv2_proj& p, int64_t n, int V, int tiles_x, int tiles_y, const cgv2_bins& b,
                                void* ws, hipStream_t st) {
  using namespace cgv2;
  const int tiles = tiles_x * tiles_y;
  const int64_t m = (int64_t)V * tiles;
  const int64_t vn = (int64_t)V * n;
  const int sets = counter_sets(m, b.capacity);
  size_t off[kBinsortOffs];
  cgv2_binsort_ws_layout(b.capacity, V, tiles, n, off);
  char* w = (char*)ws;
  uint32_t* cnt = (uint32_t*)(w + off[0]);
  SortItems items;
  items.count = cnt + m * sets;
  const int64_t nsb = surf_blocks(vn > 0 ? vn : 1);
  uint64_t* sums_cnt = (uint64_t*)(w + off[1]);
  uint64_t* sums_vis = sums_cnt + nsb + 1;
  items.item = (uint2*)(w + off[2]);
  uint64_t* totals = (uint64_t*)(w + off[3]);
  uint64_t* keys = (uint64_t*)(w + off[4]);
  uint2* staged = (uint2*)(w + off[5]);
  uint16_t* count = (uint16_t*)(w + off[6]);
  float* depth = (float*)(w + off[11]);
  uint32_t* voff = (uint32_t*)(w + off[7]);
  uint32_t* n_chunks = items.count + 1;
  uint4* chunks = (uint4*)(w + off[10]);
  const uint32_t max_chunks = (uint32_t)std::min<int64_t>(b.capacity / kChunkTiles + 1, 0xffffffffll);
  TileMap tm;
  tm.tiles_x = (uint32_t)tiles_x;
  tm.tiles_y = (uint32_t)tiles_y;
  tm.m = (uint32_t)m;
  tm.sets = sets;
  // workgroups per view of the staging and the placement: up to 8192, one run each (a multiple of kSets)
  const unsigned runs =
      (unsigned)std::min<int64_t>((std::max<int64_t>(n, 1) + kGroups * kSets - 1) / (kGroups * kSets) * kSets, 8192);
  if (n > 0) {
    // first rect slots and visible lists (consumed by the staging here and by the reverse pass), total and
    // overflow check; the tile counters and the two counts after them are zeroed on the way
    hipLaunchKernelGGL(k_surfel_sums, dim3((unsigned)nsb), dim3(kSurfBlock), 0, st, p.rect, vn, sums_cnt, sums_vis,
                       cnt, m * sets + 2);
    // up to kSurfLocal chunks each apply workgroup adds up the chunk sums before it itself
    const int local_nsb = nsb <= kSurfLocal ? (int)nsb : 0;
    if (!local_nsb) hipLaunchKernelGGL(k_scan_top, dim3(2), dim3(kScanBlock), 0, st, sums_cnt, sums_vis, nsb, totals);
    hipLaunchKernelGGL(k_surfel_apply, dim3((unsigned)nsb), dim3(kSurfBlock), 0, st, p.rect, vn, n, sums_cnt,
                       sums_vis, totals, local_nsb, voff, std::min(vn, b.capacity), p.visible, p.visible_start, V,
                       b.capacity, b.status, b.needed);
    hipLaunchKernelGGL(k_stage, dim3(runs, (unsigned)V), dim3(kStageBlock), 0, st, p.rect, p.rec, n, tm, V, b.needed,
                       p.visible, p.visible_start, voff, cnt, staged, count, depth, chunks, n_chunks,
                       max_chunks, b.status);
    hipLaunchKernelGGL(k_stage_big, dim3(1024), dim3(kStageBlock), 0, st, p.rect, p.rec, n, tm, V, b.needed,
                       p.visible, p.visible_start, cnt, staged, chunks, n_chunks, max_chunks, b.status);
  } else {
    // no surfels: empty lists, zero intersections
    hipLaunchKernelGGL(k_fill<uint32_t>, dim3((unsigned)std::min<int64_t>((m * sets + 257) / 256, 65535)), dim3(256),
                       0, st, cnt, m * sets + 2, 0u);
    hipLaunchKernelGGL(k_fill<uint32_t>, dim3(1), dim3(256), 0, st, p.visible_start, (int64_t)V + 1, 0u);
    hipLaunchKernelGGL(k_fill<int64_t>, dim3(1), dim3(256), 0, st, b.needed, (int64_t)1, (int64_t)0);
  }
  const int64_t nbt = scan_blocks(m);
  const bool fused_order = b.order && m <= kScanChunk && V <= kMaxViews;
  if (nbt <= 1) {
    hipLaunchKernelGGL(k_tile_scan_order, dim3(1), dim3(kScanBlock), 0, st, cnt, tm, V, n, p.visible_start,
                       b.needed, items, b.ranges,
                       fused_order ? b.order : nullptr);
  } else {
    uint64_t* ts = (uint64_t*)(w + off[8]);
    hipLaunchKernelGGL(k_tile_sums, dim3((unsigned)nbt), dim3(kScanBlock), 0, st, cnt, tm, V, n,
                       p.visible_start, b.needed, ts);
    hipLaunchKernelGGL(k_tile_apply, dim3((unsigned)nbt), dim3(kScanBlock), 0, st, cnt, tm, V, n,
                       p.visible_start, b.needed, items, ts, b.ranges);
  }
  hipLaunchKernelGGL(k_place, dim3(runs, (unsigned)V), dim3(kStageBlock), 0, st, p.visible, p.visible_start, V, n,
                     b.needed, voff,
                     count, depth, staged, cnt, sets, b.ranges, chunks, n_chunks, max_chunks, keys, b.status);
  // (512 workgroups more than the tiles need, for the chunks of long lists)
  hipLaunchKernelGGL(k_sort_wave, dim3((unsigned)((m + 3) / 4 + 512)), dim3(256), 0, st, b.ranges, (int)m, items, keys,
                     b.ids, b.status);
  hipLaunchKernelGGL(k_merge, dim3(1024), dim3(kMergeBlock), 0, st, b.ranges, items, keys, b.ids, b.status);
  if (b.order && !fused_order) {
    uint32_t* hist = (uint32_t*)(w + off[9]);
    for (int v0 = 0; v0 < V; v0 += kMaxViews) {
      const int T = std::min(V - v0, kMaxViews) * tiles;
      const int nc = (T + kOrdChunk - 1) / kOrdChunk;
      const int64_t base = (int64_t)v0 * tiles;
      hipLaunchKernelGGL(k_order_hist, dim3((unsigned)nc), dim3(kOrdChunk), 0, st, b.ranges, base, T, hist);
      hipLaunchKernelGGL(k_order_scan, dim3(1), dim3(64), 0, st, hist, nc);
      hipLaunchKernelGGL(k_order_place, dim3((unsigned)nc), dim3(kOrdChunk), 0, st, b.ranges, base, T, hist,
                         b.order + base);
    }
  }
  return hipGetLastError();
}
