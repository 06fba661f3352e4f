// recon_kernels.hip - control-matrix product and pure integrator of the closed loop (Sec. 3:
// the slope vectors are multiplied by the control matrix, the modal increments integrated).
//
// The product streams the whole matrix from HBM once; it is bandwidth-bound.  A block owns a
// tile of 16 rows x 4096 columns: the 16 KB slope chunk is staged in LDS once per block, each
// wave streams 4 rows with 16-byte loads (64 lanes cover 1 KB of a row per step, 8 loads in
// flight per lane) past the caches, since a call reads nothing twice, and per-row sums are
// reduced across the wave.  Chunk sums go to a partial buffer and a second pass adds them in a fixed
// order, so results do not depend on scheduling.
// 8219 x 59,136 (1.94 GB): 289 us, 6.7 TB/s; 413 us with 16 rows a wave and cached loads behind a test
// of the row number.  A bare read of the matrix in this order takes 284 us (322 us with cached loads),
// in 16 KB runs of one row after the other 278 us.  A loop reads the same matrix at every step; where the caches
// could keep it, uncached and cached loads take 9.0 and 8.0 us (16 MB), 10.8 and 9.7 (32 MB), 15.5 and 17.7 (64 MB),
// 30.8 and 31.0 (160 MB), 43.4 and 41.8 (240 MB), 51.5 and 54.7 (320 MB), 73.9 and 84.7 us (480 MB).
#include <hip/hip_runtime.h>

#include "recon_internal.h"

namespace shw {
namespace {

constexpr int kFill = 2048;   // blocks that fill the GPU (8 per CU)
constexpr int kLoads = 8;     // 16-byte loads in flight per lane: R rows x 8 / R steps
typedef float Vec4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// R rows per wavefront, 4 R per block.
template <int R>
__global__ __launch_bounds__(256) void recon_partial_kernel(const float* __restrict__ cm, int64_t ld, int32_t n_modes,
                                                            int32_t n_slopes, const float* __restrict__ slopes,
                                                            float* __restrict__ partial) {
  __shared__ float4 s_sl[kReconCols / 4];
  // one dimension of blocks (row blocks alone may pass the 65535 of a second one), chunks of a row block
  // next to each other
  const int n_chunks = recon_chunks(n_slopes);
  const int row_block = blockIdx.x / n_chunks;
  const int chunk = blockIdx.x - row_block * n_chunks;
  const int64_t c0 = (int64_t)chunk * kReconCols;
  const int ncol = (int)((int64_t)n_slopes - c0 < kReconCols ? (int64_t)n_slopes - c0 : kReconCols);
  for (int k = threadIdx.x; k < kReconCols / 4; k += 256) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (4 * k + e < ncol) ? slopes[c0 + 4 * k + e] : 0.0f;
    s_sl[k] = make_float4(v[0], v[1], v[2], v[3]);
  }
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int row0 = (row_block * 4 + wave) * R;
  // rows past the last one read it again (no test between the loads); their sums are not stored
  const float* rows[R];
  float acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    rows[r] = cm + (int64_t)min(row0 + r, n_modes - 1) * ld + c0;
    acc[r] = 0.0f;
  }
  const int nfull = ncol / 4;  // float4 columns entirely inside the matrix
  auto load = [&](int r, int k) {
    return __builtin_nontemporal_load(reinterpret_cast<const Vec4*>(rows[r]) + k);
  };
  auto add = [&](int r, const Vec4& a, const float4& x) { acc[r] += a.x * x.x + a.y * x.y + a.z * x.z + a.w * x.w; };
  constexpr int kSteps = kLoads / R;
  int k = lane;
  for (; k + 64 * (kSteps - 1) < nfull; k += 64 * kSteps) {
    Vec4 a[kSteps][R];
#pragma unroll
    for (int h = 0; h < kSteps; ++h)
#pragma unroll
      for (int r = 0; r < R; ++r) a[h][r] = load(r, k + 64 * h);
#pragma unroll
    for (int h = 0; h < kSteps; ++h) {
      const float4 x = s_sl[k + 64 * h];
#pragma unroll
      for (int r = 0; r < R; ++r) add(r, a[h][r], x);
    }
  }
  for (; k < nfull; k += 64) {
    const float4 x = s_sl[k];
#pragma unroll
    for (int r = 0; r < R; ++r) add(r, load(r, k), x);
  }
  // ragged tail of the last chunk: at most 3 columns, one lane each
  if (lane < ncol - 4 * nfull) {
    const int c = 4 * nfull + lane;
    const float x = slopes[c0 + c];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] += rows[r][c] * x;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const float s = wave_sum(acc[r]);
    const int m = row0 + r;
    if (lane == 0 && m < n_modes) partial[(int64_t)chunk * n_modes + m] = s;
  }
}

// One mode per lane; the chunk sums of a mode are read 16 at a time and added in order.  Small blocks:
// the time is one lane's chain of reads, so the modes are spread over the CUs.
__global__ __launch_bounds__(64) void recon_integrate_kernel(const float* __restrict__ partial, int32_t n_chunks,
                                                              int32_t n_modes, float gain, float* __restrict__ coefs,
                                                              float* __restrict__ delta_out) {
  const int m = blockIdx.x * 64 + threadIdx.x;
  if (m >= n_modes) return;
  float d = 0.0f;
  for (int c0 = 0; c0 < n_chunks; c0 += 16) {
    float p[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) p[c] = partial[(int64_t)min(c0 + c, n_chunks - 1) * n_modes + m];
#pragma unroll
    for (int c = 0; c < 16; ++c)
      if (c0 + c < n_chunks) d += p[c];
  }
  coefs[m] += gain * d;
  if (delta_out) delta_out[m] = d;
}

}  // namespace

hipError_t launch_recon_partial(const float* cm, int64_t ld, int32_t n_modes, int32_t n_slopes, const float* slopes,
                                float* partial, hipStream_t st) {
  if (n_modes <= 0 || n_slopes <= 0) return hipSuccess;
  const int64_t chunks = recon_chunks(n_slopes);
  auto blocks = [&](int r) { return chunks * ((n_modes + 4 * r - 1) / (4 * r)); };
  // 4 rows a wavefront where that makes at least kFill blocks, fewer for smaller matrices, which would leave
  // CUs idle: 500 x 8000 takes 10.2 us with 1 row (63 blocks with 4 rows, 12.9 us and 86 us with the 16 rows
  // of one size of tile for all), 2000 x 20,000 32.6 us (130).  The line at 1024 or 4096 blocks moves no
  // measured size by more than 3 %.
  int r = 4;
  while (r > 1 && blocks(r) < kFill) r >>= 1;
  if (blocks(r) > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks(r));
  switch (r) {
    case 4: hipLaunchKernelGGL(recon_partial_kernel<4>, grid, dim3(256), 0, st, cm, ld, n_modes, n_slopes, slopes, partial); break;
    case 2: hipLaunchKernelGGL(recon_partial_kernel<2>, grid, dim3(256), 0, st, cm, ld, n_modes, n_slopes, slopes, partial); break;
    default: hipLaunchKernelGGL(recon_partial_kernel<1>, grid, dim3(256), 0, st, cm, ld, n_modes, n_slopes, slopes, partial); break;
  }
  return hipGetLastError();
}

hipError_t launch_recon_integrate(const float* partial, int32_t n_chunks, int32_t n_modes, float gain, float* coefs,
                                  float* delta_out, hipStream_t st) {
  if (n_modes <= 0) return hipSuccess;
  hipLaunchKernelGGL(recon_integrate_kernel, dim3((unsigned)((n_modes + 63) / 64)), dim3(64), 0, st, partial,
                     n_chunks, n_modes, gain, coefs, delta_out);
  return hipGetLastError();
}

}  // namespace shw
