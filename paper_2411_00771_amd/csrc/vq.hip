// Serving storage of CityGaussianV2 (Sec. 3.3: SH degree 2; the appendix's vector-tree quantization):
// the least important surfels' SH vectors are replaced by the nearest row of a k-means codebook, the rest
// of the set is stored in float16.
//
//   k_part_*      stable partition by the quantize mask: kept surfels first, both groups in id order
//   k_vq_init     codeword j = row floor(j m / K) of the quantized vectors
//   k_vq_assign   nearest codeword: |c|^2 - 2 x.c on the matrix cores (FP32 MFMA 16x16x4), the argmin
//                 fused into the epilogue; codewords stream through LDS in chunks
//   k_vq_accum / k_vq_final   Lloyd update: FP64 sums per codeword, mean, empty codewords kept
//   k_compact_*   the stored arrays in partition order (float16 by round-to-nearest-even)
#include "cgv2r_device.h"
#include "cgv2r_kernels.h"

#include <algorithm>

namespace cgv2 {

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t to_half_bits(float x) { return __builtin_bit_cast(uint16_t, (_Float16)x); }
__device__ __forceinline__ float from_half_bits(uint16_t b) { return (float)__builtin_bit_cast(_Float16, b); }

// ---- stable partition --------------------------------------------------------------------------

constexpr int kPBlock = 256;
constexpr int kPItems = 8;
constexpr int kPChunk = kPBlock * kPItems;

__global__ __launch_bounds__(kPBlock) void k_part_count(const uint8_t* __restrict__ q, int64_t n,
                                                        uint32_t* __restrict__ part) {
  __shared__ uint32_t lds[kPBlock / 64];
  const int64_t base = (int64_t)blockIdx.x * kPChunk + threadIdx.x;
  uint32_t keep = 0;
#pragma unroll
  for (int k = 0; k < kPItems; ++k) {
    const int64_t i = base + (int64_t)k * kPBlock;
    if (i < n && !q[i]) ++keep;
  }
  uint32_t tot;
  block_exscan<kPBlock>(keep, lds, tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kPBlock) void k_part_scan(uint32_t* __restrict__ part, int nb, int64_t* __restrict__ n_full) {
  __shared__ unsigned long long lds[kPBlock / 64];
  unsigned long long carry = 0;
  for (int b0 = 0; b0 < nb; b0 += kPBlock) {
    const int b = b0 + (int)threadIdx.x;
    const unsigned long long v = b < nb ? part[b] : 0ull;
    unsigned long long tot;
    const unsigned long long ex = block_exscan<kPBlock>(v, lds, tot) + carry;
    if (b < nb) part[b] = (uint32_t)ex;
    carry += tot;
  }
  if (threadIdx.x == 0) *n_full = (int64_t)carry;
}

__global__ __launch_bounds__(kPBlock) void k_part_write(const uint8_t* __restrict__ q, int64_t n,
                                                        const uint32_t* __restrict__ koff,
                                                        const int64_t* __restrict__ n_full,
                                                        uint32_t* __restrict__ order) {
  __shared__ uint32_t lds[kPBlock / 64];
  const int64_t chunk = (int64_t)blockIdx.x * kPChunk;
  const int64_t base = chunk + (int64_t)threadIdx.x * kPItems;
  uint32_t qq[kPItems], keep = 0;
#pragma unroll
  for (int k = 0; k < kPItems; ++k) {
    qq[k] = base + k < n ? (q[base + k] ? 1u : 0u) : 1u;
    keep += base + k < n ? 1u - qq[k] : 0u;
  }
  uint32_t tot;
  const uint32_t ex = block_exscan<kPBlock>(keep, lds, tot);
  // kept before this thread's first item, over the whole set; quantized before it = index - kept
  uint32_t kept_before = koff[blockIdx.x] + ex;
  const int64_t nf = *n_full;
#pragma unroll
  for (int k = 0; k < kPItems; ++k) {
    const int64_t i = base + k;
    if (i >= n) break;
    if (!qq[k]) {
      order[kept_before] = (uint32_t)i;
      ++kept_before;
    } else {
      order[nf + (i - kept_before)] = (uint32_t)i;
    }
  }
}

// ---- codebook ------------------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_vq_init(const float* __restrict__ x, int D, const uint32_t* __restrict__ rows,
                                                 int64_t m, int K, float* __restrict__ cb) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)K * D) return;
  const int j = (int)(t / D), d = (int)(t - (int64_t)j * D);
  const int64_t r = ((int64_t)j * m) / K;
  cb[t] = x[(int64_t)rows[r] * D + d];
}

// Nearest codeword for kVqRows query vectors per workgroup (kVqRowsWave per wave: two 16-row MFMA
// tiles), against codewords staged kVqCols at a time in LDS.
// MFMA 16x16x4 f32 operand layout (wave64): A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k, and
// D[4 (lane / 16) + r][lane % 16] in accumulator element r.
constexpr int kVqThreads = 256;
constexpr int kVqRowsWave = 32;
constexpr int kVqRows = kVqRowsWave * (kVqThreads / 64);
constexpr int kVqCols = 128;

// |c|^2 of every codeword (of its float16 rounding when half_cb), FP32.
__global__ __launch_bounds__(256) void k_vq_norms(const float* __restrict__ cb, int K, int D, int half_cb,
                                                  float* __restrict__ norms) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= K) return;
  float s2 = 0.f;
  for (int d = 0; d < D; ++d) {
    float v = cb[(int64_t)j * D + d];
    if (half_cb) v = (float)(_Float16)v;
    s2 = fmaf(v, v, s2);
  }
  norms[j] = s2;
}

// The codewords lie in LDS as the lanes read them (a lane's values of all steps together, wide reads), in two buffers:
// the next chunk's loads, one contiguous stream of the codebook, are in flight while this one is multiplied.
// The first 'full' workgroups take kVqRows queries each.  The rest take kVqRowsWave each: their waves multiply the
// same queries with a quarter of the column tiles each.
// Bound by the FP32 matrix rate and the argmin's vector instructions beside it (matrix cores busy 1.2 ms of 1.8 at
// 400 k queries, 8,192 codewords of 27 dimensions): 2,130 us with strided codebook loads, a transposed single buffer
// (four-way bank conflicts) and accumulators copied out of the accumulation registers -> 1,785; 48 dimensions 3,970
// -> 2,765; 2 M queries 9,300 -> 8,240.  The column tiles unrolled by 8 spill (3,660); wave priorities give nothing.
template <int DP>  // dimensions padded to a multiple of 4
__global__ __launch_bounds__(kVqThreads, DP > 28 ? 3 : 4) void k_vq_assign(
    const float* __restrict__ x, int D, const uint32_t* __restrict__ rows, int64_t m, const float* __restrict__ cb,
    const float* __restrict__ norms, int K, int half_cb, uint16_t* __restrict__ code, unsigned full) {
  constexpr int kSteps = DP / 4;
  constexpr int kPad = kSteps == 1 ? 1 : (kSteps + 3) / 4 * 4;  // floats per lane and column tile
  constexpr int kTiles = kVqCols / 16;
  constexpr int kWaves = kVqThreads / 64;
  constexpr int kLoads = (kVqCols * DP + kVqThreads - 1) / kVqThreads;
  constexpr int kSure = kVqCols * (DP - 3) / kVqThreads;  // loads that every thread has for every D
  const int count = kVqCols * D;
  __shared__ __align__(16) float frag[2][kTiles][64][kPad];
  __shared__ float norm[2][kVqCols];
  __shared__ float s_best[kWaves][kVqRowsWave];
  __shared__ int s_idx[kWaves][kVqRowsWave];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const bool split = blockIdx.x >= full;
  const int64_t row0 = split ? (int64_t)full * kVqRows + (int64_t)(blockIdx.x - full) * kVqRowsWave
                             : (int64_t)blockIdx.x * kVqRows + (int64_t)w * kVqRowsWave;
  const int ct_begin = split ? w * (kTiles / kWaves) : 0, ct_end = split ? ct_begin + kTiles / kWaves : kTiles;
  // A operands: query (row0 + 16 t + li), dimension 4 s + lk
  float a[2][kSteps];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int64_t r = row0 + 16 * t + li;
    const float* xr = r < m ? x + (int64_t)rows[r] * D : nullptr;
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const int d = 4 * s + lk;
      a[t][s] = (xr && d < D) ? xr[d] : 0.f;
    }
  }
  float best[2][4];
  int bidx[2][4];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      best[t][r] = INFINITY;
      bidx[t][r] = 0x7fffffff;
    }
  // the dimensions past D stay zero
  if (D < DP)
    for (int e = threadIdx.x; e < 2 * kTiles * 64 * kPad; e += kVqThreads) (&frag[0][0][0][0])[e] = 0.f;
  // value e = thread + 256 k of a chunk: codeword e / D of it, dimension e % D
  float v[kLoads], nv = INFINITY;
  int at[kLoads];
  int j = (int)threadIdx.x / D, d = (int)threadIdx.x - j * D;
  const int dj = kVqThreads / D, dd = kVqThreads - dj * D;
#pragma unroll
  for (int k = 0; k < kLoads; ++k) {  // (past the chunk: not stored)
    at[k] = ((j >> 4) * 64 + (j & 15) + 16 * (d & 3)) * kPad + (d >> 2);
    j += dj;
    d += dd;
    if (d >= D) {
      d -= D;
      ++j;
    }
  }
  auto mine = [&](int k) { return k < kSure || (int)threadIdx.x + k * kVqThreads < count; };
  auto load = [&](int c0) {
    const float* src = cb + (int64_t)c0 * D + threadIdx.x;
    if (c0 + kVqCols <= K) {
#pragma unroll
      for (int k = 0; k < kLoads; ++k)
        if (mine(k)) v[k] = src[k * kVqThreads];
      if (threadIdx.x < kVqCols) nv = norms[c0 + threadIdx.x];
    } else {
      const int live = (K - c0) * D - (int)threadIdx.x;
#pragma unroll
      for (int k = 0; k < kLoads; ++k) v[k] = mine(k) && k * kVqThreads < live ? src[k * kVqThreads] : 0.f;
      if (threadIdx.x < kVqCols) nv = c0 + (int)threadIdx.x < K ? norms[c0 + threadIdx.x] : INFINITY;
    }
  };
  auto put = [&](int buf) {
    float* to = &frag[buf][0][0][0];
    if (half_cb) {
#pragma unroll
      for (int k = 0; k < kLoads; ++k) v[k] = (float)(_Float16)v[k];
    }
#pragma unroll
    for (int k = 0; k < kLoads; ++k)
      if (mine(k)) to[at[k]] = v[k];
    if (threadIdx.x < kVqCols) norm[buf][threadIdx.x] = nv;
  };
  load(0);
  __syncthreads();  // the zeros are written
  put(0);
  __syncthreads();
  for (int c0 = 0, buf = 0; c0 < K; c0 += kVqCols, buf ^= 1) {
    const bool more = c0 + kVqCols < K;
    if (more) load(c0 + kVqCols);
    for (int ct = ct_begin; ct < ct_end; ++ct) {
      floatx4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
      float b[kPad];
#pragma unroll
      for (int s = 0; s < kPad; ++s) b[s] = frag[buf][ct][lane][s];
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0][s], b[s], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1][s], b[s], acc1, 0, 0, 0);
      }
      const int j = 16 * ct + li;
      const float nj = norm[buf][j];
      const int idx = c0 + j;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float s0 = fmaf(-2.f, acc0[r], nj), s1 = fmaf(-2.f, acc1[r], nj);
        if (s0 < best[0][r]) { best[0][r] = s0; bidx[0][r] = idx; }
        if (s1 < best[1][r]) { best[1][r] = s1; bidx[1][r] = idx; }
      }
    }
    if (more) put(buf ^ 1);
    __syncthreads();  // the next chunk is written and this one no longer read
  }
  // reduce over the 16 lanes that hold the same rows (lane % 16 = codeword column)
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float b = best[t][r];
      int bi = bidx[t][r];
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) {
        const float ob = __shfl_xor(b, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (ob < b || (ob == b && oi < bi)) { b = ob; bi = oi; }
      }
      const int row = 16 * t + 4 * lk + r;
      if (li == 0) {
        if (split) {
          s_best[w][row] = b;
          s_idx[w][row] = bi;
        } else if (row0 + row < m) {
          code[row0 + row] = (uint16_t)bi;
        }
      }
    }
  if (!split) return;
  __syncthreads();
  if (threadIdx.x < kVqRowsWave && row0 + (int64_t)threadIdx.x < m) {
    float b = s_best[0][threadIdx.x];
    int bi = s_idx[0][threadIdx.x];
#pragma unroll
    for (int q = 1; q < kWaves; ++q) {
      const float ob = s_best[q][threadIdx.x];
      const int oi = s_idx[q][threadIdx.x];
      if (ob < b || (ob == b && oi < bi)) { b = ob; bi = oi; }
    }
    code[row0 + threadIdx.x] = (uint16_t)bi;
  }
}

constexpr int kAccRows = 64;  // rows per workgroup

// One value per thread: a row's D sums lie on two or three cache lines, and the lanes of a wave that add to one line
// share its request: 400 k rows of 27 700 us with a row per thread (27 requests a row) -> 145.
__global__ __launch_bounds__(256) void k_vq_accum(const float* __restrict__ x, int D, const uint32_t* __restrict__ rows,
                                                  int64_t m, const uint16_t* __restrict__ code, int K,
                                                  double* __restrict__ sums, uint32_t* __restrict__ counts) {
  const int64_t q0 = (int64_t)blockIdx.x * kAccRows;
  const int live = (int)(m - q0 < kAccRows ? m - q0 : kAccRows) * D;
  for (int t = threadIdx.x; t < live; t += 256) {
    const int q = t / D, d = t - q * D;
    const int c = code[q0 + q];
    if (c >= K) continue;
    atomicAdd(&sums[(int64_t)c * D + d], (double)x[(int64_t)rows[q0 + q] * D + d]);
    if (d == 0) atomicAdd(&counts[c], 1u);
  }
}

__global__ __launch_bounds__(256) void k_vq_final(const double* __restrict__ sums,
                                                  const uint32_t* __restrict__ counts, int K, int D,
                                                  float* __restrict__ cb) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)K * D) return;
  const uint32_t c = counts[t / D];
  if (c) cb[t] = (float)(sums[t] / (double)c);
}

// ---- stored arrays ---------------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_compact_geom(cgv2_surfels s, const uint32_t* __restrict__ order,
                                                      cgv2_compact_out out) {
  const int64_t n = s.n;
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const int64_t i = order[j];
  if (i >= n) return;
#pragma unroll
  for (int c = 0; c < 3; ++c) out.mean[c * n + j] = s.mean[c * n + i];
#pragma unroll
  for (int c = 0; c < 2; ++c) out.log_scale[c * n + j] = to_half_bits(s.log_scale[c * n + i]);
#pragma unroll
  for (int c = 0; c < 4; ++c) out.quat[c * n + j] = to_half_bits(s.quat[c * n + i]);
  out.opacity_logit[j] = to_half_bits(s.opacity_logit[i]);
}

// SH of the kept slots [0, n_full), one value per thread (coalesced writes)
__global__ __launch_bounds__(256) void k_compact_sh(const float* __restrict__ sh, int64_t n, int F,
                                                    const uint32_t* __restrict__ order,
                                                    const int64_t* __restrict__ n_full, uint16_t* __restrict__ out) {
  const int64_t lim = *n_full * F;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < lim; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = t / F;
    const int k = (int)(t - j * F);
    const int64_t i = order[j];
    if (i < n) out[t] = to_half_bits(sh[i * F + k]);
  }
}

__global__ __launch_bounds__(256) void k_to_half(const float* __restrict__ x, int64_t count, uint16_t* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < count) out[t] = to_half_bits(x[t]);
}

inline unsigned blocks_for(int64_t items, int64_t cap = 1 << 20) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>((items + 255) / 256, cap));
}

}  // namespace cgv2

size_t cgv2_part_ws_layout(int64_t n) {
  const int64_t nb = std::max<int64_t>((n + cgv2::kPChunk - 1) / cgv2::kPChunk, 1);
  return ((size_t)4 * (size_t)nb + 255) & ~(size_t)255;
}

hipError_t cgv2_launch_compact_order(const uint8_t* q, int64_t n, uint32_t* order, int64_t* n_full, void* ws,
                                     hipStream_t st) {
  const int nb = (int)std::max<int64_t>((n + cgv2::kPChunk - 1) / cgv2::kPChunk, 1);
  uint32_t* part = (uint32_t*)ws;
  if (n > 0)
    hipLaunchKernelGGL(cgv2::k_part_count, dim3((unsigned)nb), dim3(cgv2::kPBlock), 0, st, q, n, part);
  else
    hipLaunchKernelGGL((cgv2::k_fill<uint32_t>), dim3(1), dim3(64), 0, st, part, (int64_t)1, 0u);
  hipLaunchKernelGGL(cgv2::k_part_scan, dim3(1), dim3(cgv2::kPBlock), 0, st, part, nb, n_full);
  if (n > 0)
    hipLaunchKernelGGL(cgv2::k_part_write, dim3((unsigned)nb), dim3(cgv2::kPBlock), 0, st, q, n, part, n_full, order);
  return hipGetLastError();
}

hipError_t cgv2_launch_vq_init(const float* x, int D, const uint32_t* rows, int64_t m, int K, float* cb,
                               hipStream_t st) {
  hipLaunchKernelGGL(cgv2::k_vq_init, dim3(cgv2::blocks_for((int64_t)K * D)), dim3(256), 0, st, x, D, rows, m, K, cb);
  return hipGetLastError();
}

size_t cgv2_vq_assign_ws_layout(int K) { return (((size_t)K * sizeof(float)) + 255) & ~(size_t)255; }

// A rest of up to so many workgroups, half of the CUs, is split four ways, so that it ends with the last round (us:
// 400 k queries, rest 53: 1,881 -> 1,773; 3,000 queries, rest 24: 200 -> 89; 60 k, rest 469: 94, split 124).
constexpr int64_t kVqSplit = 128;

hipError_t cgv2_launch_vq_assign(const float* x, int D, const uint32_t* rows, int64_t m, const float* cb, int K,
                                 int half_cb, uint16_t* code, void* ws, hipStream_t st) {
  if (m == 0) return hipGetLastError();
  float* norms = (float*)ws;
  hipLaunchKernelGGL(cgv2::k_vq_norms, dim3((unsigned)((K + 255) / 256)), dim3(256), 0, st, cb, K, D, half_cb, norms);
  // Whole rounds of the workgroups that run at once, and the rest split when it is small
  const int64_t nb = (m + cgv2::kVqRows - 1) / cgv2::kVqRows, round = 256 * (D > 28 ? 3 : 4);
  const int64_t rest = nb % round;
  const int64_t full = rest <= kVqSplit ? nb - rest : nb;
  const int64_t part = m > full * cgv2::kVqRows ? (m - full * cgv2::kVqRows + cgv2::kVqRowsWave - 1) / cgv2::kVqRowsWave : 0;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(full + part)), dim3(cgv2::kVqThreads), 0, st, x, D, rows, m, cb, norms,
                       K, half_cb, code, (unsigned)full);
  };
  switch ((D + 3) & ~3) {
    case 4: go(cgv2::k_vq_assign<4>); break;
    case 12: go(cgv2::k_vq_assign<12>); break;
    case 28: go(cgv2::k_vq_assign<28>); break;
    case 48: go(cgv2::k_vq_assign<48>); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

size_t cgv2_vq_update_ws_layout(int K, int D) {
  return (((size_t)K * D * sizeof(double)) + 255) & ~(size_t)255;
}

hipError_t cgv2_launch_vq_update(const float* x, int D, const uint32_t* rows, int64_t m, const uint16_t* code, int K,
                                 float* cb, uint32_t* counts, void* ws, hipStream_t st) {
  double* sums = (double*)ws;
  hipLaunchKernelGGL((cgv2::k_fill<double>), dim3(cgv2::blocks_for((int64_t)K * D, 4096)), dim3(256), 0, st, sums,
                     (int64_t)K * D, 0.0);
  hipLaunchKernelGGL((cgv2::k_fill<uint32_t>), dim3(cgv2::blocks_for(K, 4096)), dim3(256), 0, st, counts, (int64_t)K, 0u);
  if (m > 0)
    hipLaunchKernelGGL(cgv2::k_vq_accum, dim3((unsigned)((m + cgv2::kAccRows - 1) / cgv2::kAccRows)), dim3(256), 0, st, x, D, rows, m, code, K, sums,
                       counts);
  hipLaunchKernelGGL(cgv2::k_vq_final, dim3(cgv2::blocks_for((int64_t)K * D)), dim3(256), 0, st, sums, counts, K, D, cb);
  return hipGetLastError();
}

hipError_t cgv2_launch_compact_write(const cgv2_surfels& s, const uint32_t* order, const int64_t* n_full,
                                     const float* cb, int K, const cgv2_compact_out& out, hipStream_t st) {
  const int64_t n = s.n;
  const int F = 3 * (s.sh_degree + 1) * (s.sh_degree + 1);
  if (n > 0) {
    hipLaunchKernelGGL(cgv2::k_compact_geom, dim3(cgv2::blocks_for(n)), dim3(256), 0, st, s, order, out);
    hipLaunchKernelGGL(cgv2::k_compact_sh, dim3(cgv2::blocks_for(n * F, 16384)), dim3(256), 0, st, s.sh, n, F, order,
                       n_full, out.sh);
  }
  if (K > 0 && cb)
    hipLaunchKernelGGL(cgv2::k_to_half, dim3(cgv2::blocks_for((int64_t)K * F)), dim3(256), 0, st, cb, (int64_t)K * F,
                       out.codebook);
  return hipGetLastError();
}
