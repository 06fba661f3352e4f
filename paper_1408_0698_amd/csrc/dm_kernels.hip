// dm_kernels.hip - DM surfaces and residual OPD (Sec. 3 closed-loop block: residual =
// open-loop wavefront minus the DM; Sec. 2 DM mode counts; analytic influence functions).
//
// Surface: tiles of pixels.  The actuators sit on a square grid of pitch P,
// so the actuators whose patches reach a tile form a small index box; a
// grid-index table maps each box entry to its actuator (or -1 outside the
// metapupil).  Residual: four consecutive pixels per lane, looping over the
// outputs.
#include <hip/hip_runtime.h>

#include "dm_internal.h"

namespace shw {

namespace {

__device__ __forceinline__ int floor_div(int a, int b) {  // b > 0
  int q = a / b;
  return (a % b != 0 && a < 0) ? q - 1 : q;
}

// Surface tile of 64 x 16 pixels.  The influence function is a product of two one-dimensional
// Gaussians on a square patch, so the tile's sum over actuators splits: along x first,
// A[gy][x] = sum_gx c[gy][gx] e(x - gx), for the grid rows gy that reach the tile, then
// S[y][x] = sum_gy e(y - gy) A[gy][x].  A pixel of the 10-px-pitch DM (patch 64) then takes about
// 4 + 7 FMAs instead of 41 exponentials; the Gaussian is tabulated once per block.
// Actuators go in chunks of kGy x kGx, so any patch and pitch fits the LDS.  Bound by the latency of
// its steps (grid table, coefficients, two passes): 6.4 us for the 800^2 surface of 5025 actuators and
// 7.3 us on average over the three mirrors of the 39 m telescope, against 11.6 and 17.1 us for one
// exponential per pixel and actuator.
constexpr int kTileX = 64, kTileY = 16;
constexpr int kGy = 16, kGx = 32;
constexpr int kMaxPatch = 1024;

__global__ __launch_bounds__(256) void dm_surface_kernel(const DmLaunch a, const float* __restrict__ coefs,
                                                         float* __restrict__ surf) {
  __shared__ float s_e[kMaxPatch];
  __shared__ float s_c[kGy][kGx];
  __shared__ float s_a[kGy][kTileX];
  const int tid = threadIdx.x;
  const int lx = tid & 63, ly = tid >> 6;
  const int half = a.size / 2, h = a.half_patch, patch = 2 * h;
  const int j0 = blockIdx.x * kTileX, i0 = blockIdx.y * kTileY;
  for (int d = tid; d < patch; d += 256) {
    const float x = (float)(d - h) + 0.5f;  // pixel centre minus actuator
    s_e[d] = expf(-x * x * a.inv_2s2);
  }
  // grid index g (position g * pitch from the centre) covers pixel j iff 0 <= j - half - g*pitch + h < patch
  const int gx0 = max(floor_div(j0 - half - h, a.pitch) + 1, -a.m);
  const int gx1 = min(floor_div(j0 + kTileX - 1 - half + h, a.pitch), a.m);
  const int gy0 = max(floor_div(i0 - half - h, a.pitch) + 1, -a.m);
  const int gy1 = min(floor_div(i0 + kTileY - 1 - half + h, a.pitch), a.m);
  const int side = 2 * a.m + 1;
  const int jr = j0 + lx - half + h;  // minus g * pitch: the pixel's place in the patch of g
  const int ir = i0 - half + h;
  float s[kTileY / 4];
#pragma unroll
  for (int r = 0; r < kTileY / 4; ++r) s[r] = 0.0f;
  for (int gyc = gy0; gyc <= gy1; gyc += kGy) {
    float acc[kGy / 4];
#pragma unroll
    for (int r = 0; r < kGy / 4; ++r) acc[r] = 0.0f;
    for (int gxc = gx0; gxc <= gx1; gxc += kGx) {
      // coefficients of the chunk, 0 where there is no actuator
      for (int e = tid; e < kGy * kGx; e += 256) {
        const int gy = gyc + e / kGx, gx = gxc + e % kGx;
        float c = 0.0f;
        if (gy <= gy1 && gx <= gx1) {
          const int k = a.grid[(gy + a.m) * side + gx + a.m];
          if (k >= 0) c = coefs[k];
        }
        s_c[e / kGx][e % kGx] = c;
      }
      __syncthreads();
      // the chunk's grid columns that cover this lane's pixel column
      const int lo = max(floor_div(jr - patch, a.pitch) + 1, gxc) - gxc;
      const int hi = min(min(floor_div(jr, a.pitch), gx1), gxc + kGx - 1) - gxc;
      for (int g = lo; g <= hi; ++g) {
        const float e = s_e[jr - (gxc + g) * a.pitch];
#pragma unroll
        for (int r = 0; r < kGy / 4; ++r) acc[r] = fmaf(s_c[ly + 4 * r][g], e, acc[r]);
      }
      __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < kGy / 4; ++r) s_a[ly + 4 * r][lx] = acc[r];
    __syncthreads();
    const int n = min(kGy, gy1 - gyc + 1);
#pragma unroll
    for (int r = 0; r < kTileY / 4; ++r) {
      const int y = ir + ly + 4 * r;  // uniform over the wavefront, like the test below
      for (int g = 0; g < n; ++g) {
        const int d = y - (gyc + g) * a.pitch;
        if (d >= 0 && d < patch) s[r] = fmaf(s_e[d], s_a[g][lx], s[r]);
      }
    }
    __syncthreads();
  }
  const int j = j0 + lx;
#pragma unroll
  for (int r = 0; r < kTileY / 4; ++r) {
    const int i = i0 + ly + 4 * r;
    if (i < a.size && j < a.size) surf[(int64_t)i * a.size + j] = s[r];
  }
}

// Four consecutive floats at any 4-byte alignment (one 16-byte access).
struct __attribute__((packed, aligned(4))) Quad {
  float v[4];
};
typedef float QuadV __attribute__((ext_vector_type(4), aligned(4)));

// Each thread owns four consecutive pixels of the pupil and goes through per_block outputs; the
// mirrors' pixels stay in registers while the outputs keep the same mirror windows (the frames of
// one direction; the host orders the outputs by their windows), so a further frame costs one read
// of the screen and one write.  Bound by the writes: 60 outputs of 800^2 with three mirrors (154 MB)
// take 29 us = 5.2 TB/s; one pixel per thread and output, reading every mirror for every output,
// took 53-97 us for 32 of them.
template <int NDM>
__global__ __launch_bounds__(256) void residual_kernel(const ResidualLaunch a, float* __restrict__ out) {
  // consecutive blocks go to the 8 XCDs in turn: XCD c takes the c-th eighth of the pupil's tiles
  // for every output, so that its L2 keeps that part of the screen and of the mirrors
  const int slot = blockIdx.x >> 3;
  const int group = slot / a.xcd_tiles;
  const int tile = (blockIdx.x & 7) * a.xcd_tiles + slot - group * a.xcd_tiles;
  const int e = tile * 256 + threadIdx.x;
  const int y = e / a.quads;
  const int x = 4 * (e - y * a.quads);
  if (y >= (int)a.rows) return;
  const int k0 = group * a.per_block;
  const int k1 = min(k0 + a.per_block, a.n_out);
  const int64_t scr = (int64_t)y * a.screen_pitch + x;
  const int64_t dst = (int64_t)y * a.out_pitch + x;
  if (x + 4 <= a.pupil_n) {
    Quad m[NDM > 0 ? NDM : 1];
    Quad next = *reinterpret_cast<const Quad*>(a.screen + a.o[k0].scr_off + scr);
    for (int k = k0; k < k1; ++k) {
      const ResidualOut& o = a.o[k];
      bool same = k > k0;
#pragma unroll
      for (int d = 0; d < NDM; ++d) same = same && o.dm_off[d] == a.o[k - 1].dm_off[d];
      if (!same) {
#pragma unroll
        for (int d = 0; d < NDM; ++d)
          m[d] = *reinterpret_cast<const Quad*>(a.surf[d] + o.dm_off[d] + (int64_t)y * a.surf_size[d] + x);
      }
      Quad v = next;
      if (k + 1 < k1) next = *reinterpret_cast<const Quad*>(a.screen + a.o[k + 1].scr_off + scr);
#pragma unroll
      for (int d = 0; d < NDM; ++d)
#pragma unroll
        for (int q = 0; q < 4; ++q) v.v[q] -= m[d].v[q];
      QuadV* po = reinterpret_cast<QuadV*>(out + o.out * a.out_stride + dst);
      const QuadV w = {v.v[0], v.v[1], v.v[2], v.v[3]};
      if (a.streaming)
        __builtin_nontemporal_store(w, po);
      else
        *po = w;
    }
  } else {
    for (int k = k0; k < k1; ++k) {
      const ResidualOut& o = a.o[k];
      const float* ps = a.screen + o.scr_off + scr;
      float* po = out + o.out * a.out_stride + dst;
      for (int q = 0; x + q < a.pupil_n; ++q) {
        float v = ps[q];
#pragma unroll
        for (int d = 0; d < NDM; ++d) v -= a.surf[d][o.dm_off[d] + (int64_t)y * a.surf_size[d] + x + q];
        po[q] = v;
      }
    }
  }
}

// One lane per output pixel; the pixel is inside the actuator's patch or the value is 0.
__global__ __launch_bounds__(256) void influence_kernel(const InfluenceLaunch a, float* __restrict__ out) {
  const int x = blockIdx.x * 256 + threadIdx.x;
  const int y = blockIdx.y;
  const int k = blockIdx.z;
  if (x >= a.pupil_n) return;
  const int act = a.act[k];
  if (act < 0 || act >= a.n_act) {  // an index off the grid yields a NaN frame, never a stray read
    out[(int64_t)k * a.out_stride + (int64_t)y * a.out_pitch + x] = __builtin_nanf("");
    return;
  }
  const float ax = a.act_xy[2 * act], ay = a.act_xy[2 * act + 1];
  const int half = a.size / 2;
  const int i = a.row0 + y, j = a.col0 + x;  // surface pixel
  const int cx = half + (int)ax, cy = half + (int)ay;
  float v = 0.0f;
  if (j >= cx - a.half_patch && j < cx + a.half_patch && i >= cy - a.half_patch && i < cy + a.half_patch) {
    const float dx = (float)j + 0.5f - (float)half - ax;
    const float dy = (float)i + 0.5f - (float)half - ay;
    v = influence(a.amp[k], dx, dy, a.inv_2s2);
  }
  out[(int64_t)k * a.out_stride + (int64_t)y * a.out_pitch + x] = v;
}

// Interaction-matrix columns from push/pull slope pairs: a 32 x 32 tile transpose through LDS.
__global__ __launch_bounds__(256) void push_pull_kernel(const float* __restrict__ slopes, int32_t n_modes,
                                                        int32_t n_slopes, float scale, float* __restrict__ im,
                                                        int64_t ld) {
  __shared__ float tile[32][33];
  const int s0 = blockIdx.x * 32, m0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    const int m = m0 + r, s = s0 + tx;
    float v = 0.0f;
    if (m < n_modes && s < n_slopes)
      v = (slopes[(int64_t)(2 * m) * n_slopes + s] - slopes[(int64_t)(2 * m + 1) * n_slopes + s]) * scale;
    tile[r][tx] = v;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int s = s0 + r, m = m0 + tx;
    if (s < n_slopes && m < n_modes) im[(int64_t)s * ld + m] = tile[tx][r];
  }
}

// Four elements of a row per thread.
__global__ __launch_bounds__(256) void fill_matrix_kernel(float* __restrict__ im, int64_t quads, int32_t row_quads,
                                                           int32_t cols, int64_t ld, float v) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= quads) return;
  const int64_t r = e / row_quads;
  const int32_t c = 4 * (int32_t)(e - r * row_quads);
  float* p = im + r * ld + c;
  if (c + 4 <= cols) {
    *reinterpret_cast<QuadV*>(p) = QuadV{v, v, v, v};
  } else {
    for (int k = 0; c + k < cols; ++k) p[k] = v;
  }
}

}  // namespace

hipError_t launch_fill_matrix(float* im, int64_t rows, int32_t cols, int64_t ld, float v, hipStream_t st) {
  const int32_t rq = (cols + 3) / 4;
  // rows per launch: fewer than the 2^32 lanes that one may have
  const int64_t band = ((int64_t)1 << 31) / rq;
  for (int64_t r0 = 0; r0 < rows; r0 += band) {
    const int64_t quads = (rows - r0 < band ? rows - r0 : band) * rq;
    hipLaunchKernelGGL(fill_matrix_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st, im + r0 * ld, quads, rq,
                       cols, ld, v);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_influence_opd(const InfluenceLaunch& a, float* out, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  dim3 grid((a.pupil_n + 255) / 256, a.pupil_n, a.n);
  hipLaunchKernelGGL(influence_kernel, grid, dim3(256), 0, st, a, out);
  return hipGetLastError();
}

hipError_t launch_push_pull(const float* slopes, int32_t n_modes, int32_t n_slopes, float scale, float* im,
                            int64_t ld, hipStream_t st) {
  if (n_modes <= 0 || n_slopes <= 0) return hipSuccess;
  dim3 grid((n_slopes + 31) / 32, (n_modes + 31) / 32);
  hipLaunchKernelGGL(push_pull_kernel, grid, dim3(256), 0, st, slopes, n_modes, n_slopes, scale, im, ld);
  return hipGetLastError();
}

hipError_t launch_dm_surface(const DmLaunch& a, const float* coefs, float* surf, hipStream_t st) {
  if (2 * a.half_patch > kMaxPatch) return hipErrorInvalidValue;
  dim3 grid((a.size + kTileX - 1) / kTileX, (a.size + kTileY - 1) / kTileY);
  hipLaunchKernelGGL(dm_surface_kernel, grid, dim3(256), 0, st, a, coefs, surf);
  return hipGetLastError();
}

static hipError_t launch_residual_rows(ResidualLaunch& a, int n_dm, float* out, hipStream_t st) {
  const int64_t tiles = (a.quads * a.rows + 255) / 256;
  // enough blocks to fill the GPU about twice (8 resident per CU), the rest of the outputs in the
  // blocks' loops
  int64_t pb = (int64_t)a.n_out * tiles / 4096;
  a.per_block = pb < 1 ? 1 : (pb > a.n_out ? a.n_out : (int)pb);
  a.xcd_tiles = (int32_t)((tiles + 7) / 8);
  const dim3 grid((unsigned)(8 * a.xcd_tiles * ((a.n_out + a.per_block - 1) / a.per_block)));
  switch (n_dm) {
    case 0: hipLaunchKernelGGL(residual_kernel<0>, grid, dim3(256), 0, st, a, out); break;
    case 1: hipLaunchKernelGGL(residual_kernel<1>, grid, dim3(256), 0, st, a, out); break;
    case 2: hipLaunchKernelGGL(residual_kernel<2>, grid, dim3(256), 0, st, a, out); break;
    case 3: hipLaunchKernelGGL(residual_kernel<3>, grid, dim3(256), 0, st, a, out); break;
    case 4: hipLaunchKernelGGL(residual_kernel<4>, grid, dim3(256), 0, st, a, out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_residual(ResidualLaunch& a, int n_dm, float* out, hipStream_t st) {
  a.quads = (a.pupil_n + 3) / 4;
  // results larger than twice the L2s (8 x 4 MB) leave them before anyone reads them: written past
  // the caches they leave the screen and the mirrors there (60 outputs of 800^2: 29.3 against 31.3 us)
  a.streaming = (int64_t)a.n_out * a.pupil_n * a.pupil_n * (int64_t)sizeof(float) > ((int64_t)64 << 20);
  // the kernel counts quads in 32 bits and a launch has at most 2^32 lanes: pupils above 65536 pixels go in
  // bands of rows
  const int64_t band = ((int64_t)1 << 30) / a.quads;
  for (int64_t y0 = 0; y0 < a.pupil_n; y0 += a.rows) {
    a.rows = a.pupil_n - y0 < band ? a.pupil_n - y0 : band;
    const hipError_t e = launch_residual_rows(a, n_dm, out + y0 * a.out_pitch, st);
    if (e != hipSuccess) return e;
    // to the next band, and back to the first row after the last one
    const int64_t step = y0 + a.rows < a.pupil_n ? a.rows : -y0;
    a.screen += step * a.screen_pitch;
    for (int d = 0; d < n_dm; ++d) a.surf[d] += step * a.surf_size[d];
  }
  return hipSuccess;
}

}  // namespace shw
