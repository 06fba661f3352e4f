// lgs_geometry_kernels.hip - open-loop wavefronts of finite-altitude sources (the cone effect)
// and the uplink tip-tilt of laser guide stars.
//
// Sec. 4 (open-loop generation): the shifted phase screens are piled up per source direction;
// for an LGS each sodium sub-layer is a source at its own altitude, whose beam crosses a layer
// at altitude h on a pupil footprint shrunk by (1 - h/H) and moved by h theta, and the spot on
// the sodium layer is displaced by the tip-tilt the laser beam picks up on its way up.
#include <hip/hip_runtime.h>

#include "geom_internal.h"

namespace shw {

namespace {

// Two neighbouring screen samples (8 bytes at 4-byte alignment: one access).
typedef float Pair __attribute__((ext_vector_type(2), aligned(4)));

// Sample pair `bytes` past p (device memory; a uniform p stays in scalar registers).
__device__ __forceinline__ Pair load_pair(const float* p, uint32_t bytes) {
  using GlobalC = __attribute__((address_space(1))) const char;
  using GlobalP = __attribute__((address_space(1))) const Pair;
  return *(const GlobalP*)((const GlobalC*)p + bytes);
}

// (1 - f) u + f v with g = 1 - f (two products: an infinite sample stays infinite)
__device__ __forceinline__ double lerp(double u, double v, double g, double f) { return fma(f, v, g * u); }

// Integer part of the screen coordinate X, kept in [0, n - 2] (the host checks the footprints; the
// clamp only guards rounding), and the fraction f from it.
__device__ __forceinline__ int split_coord(double X, int n, double& f) {
  int i = (int)floor(X);
  i = max(0, min(i, n - 2));
  f = X - (double)i;
  return i;
}

constexpr int kProjRows = 4;   // pupil rows per lane
constexpr int kProjCols = 2;   // column tiles of 64 per wavefront
constexpr int kProjWaves = 4;  // wavefronts per block, each on its own rows
constexpr int kRows = kProjWaves * kProjRows;

// v of lane r (uniform r), as a scalar
__device__ __forceinline__ int lane_i32(int v, int r) { return __builtin_amdgcn_readlane(v, r); }
__device__ __forceinline__ double lane_f64(double v, int r) {
  const int64_t b = __double_as_longlong(v);
  const uint32_t lo = (uint32_t)lane_i32((int)b, r);
  return __longlong_as_double(((int64_t)lane_i32((int)(b >> 32), r) << 32) | lo);
}

}  // namespace

// One wavefront: kProjRows rows of kProjCols tiles of 64 columns of one target's pupil.  The screen
// coordinates of a layer are affine in the pupil indices, X = ax + b (j + 1/2 - N/2) and Y likewise, so
// the column part of a lane serves all its rows, and the row part is uniform (lane r works it out
// for row r) and serves all tiles.  Where a wavefront's rows go on by at most one sample (the cone shrinks
// the footprint, and screens are rarely finer than the pupil), the screen row above a pupil row's
// point is the one above or below the previous row's point, so each row costs one new screen row;
// otherwise the rows above are read too.  Positions, weights and sums are FP64, FP32 out.
// Bound by FP64 issue (290 VALU instructions per lane for its 8 pixels through three layers, 4.6
// cycles each) and the row bookkeeping: 18 targets of 800^2 through three layers take 40 us traced,
// 108 us with one lane per pixel, its own row arithmetic, a division by the sample spacing per layer
// and the layers padded to groups of four.  4 x 1 and 8 x 2 rows x tiles per wavefront: 43 and 48 us;
// tiles of the screen staged in LDS: 55 us (two barriers per layer).
// MAPS: the maps come ready in the arguments, else the kernel makes them (6 more FP64 instructions a layer:
// 1-4 % where one launch does either way).  The line is at one launch: the maps of 18 targets of 800^2 through
// seven layers take two, 77 instead of 70 us; 18 of 200^2 through 16 layers take three, 52 instead of 25 us, the
// serial chain of 16 layers each time; 40 of 130^2 through 16 layers six, 98 instead of 24 us.
template <bool MAPS>
__global__ __launch_bounds__(64 * kProjWaves) void project_layers_kernel(const ProjectLaunch a) {
  // consecutive blocks go to the 8 XCDs in turn: XCD c takes the tile rows c mod 8, all targets of a
  // tile before the next one, because the targets' footprints on a layer largely overlap
  const int t = blockIdx.x >> 3;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i0 = (blockIdx.y * 8 + (blockIdx.x & 7)) * kRows + wave * kProjRows;
  const int n = a.pupil_n;
  if (i0 >= n) return;  // the whole wavefront
  const int j0 = blockIdx.z * 64, jstep = gridDim.z * 64;  // tile c starts at column j0 + c jstep
  const double centre = 0.5 - 0.5 * n;
  const double ic = (double)min(i0 + (lane & (kProjRows - 1)), n - 1) + centre;
  double acc[kProjCols][kProjRows];
#pragma unroll
  for (int c = 0; c < kProjCols; ++c)
#pragma unroll
    for (int r = 0; r < kProjRows; ++r) acc[c][r] = 0.0;
  for (int l = 0; l < a.n_layers; ++l) {
    const ProjectLayer& L = a.layer[l];
    const ProjectMap m = MAPS ? a.map[t * a.n_layers + l] : project_map(a.place[l], a.target[t], a.dx);
    double fyv;
    const int iyv = split_coord(fma(m.b, ic, m.ay), L.rows, fyv);
    const double gyv = 1.0 - fyv;
    int iy[kProjRows];
#pragma unroll
    for (int r = 0; r < kProjRows; ++r) iy[r] = lane_i32(iyv, r);
    // rows that go on by one sample at most (uniform).  Told by the steps and not by b <= 1: where Y passes a
    // power of two its rounding changes, and with b = 1 the row may then go on by two
    bool shared = true;
#pragma unroll
    for (int r = 1; r < kProjRows; ++r) shared = shared && iy[r] - iy[r - 1] <= 1;
    // the reads of every tile and row first
    Pair top[kProjCols], bot[kProjCols][kProjRows];
    double fx[kProjCols];
    int ix[kProjCols];
#pragma unroll
    for (int c = 0; c < kProjCols; ++c) {
      if (j0 + c * jstep >= n) break;  // uniform
      const double jc = (double)min(j0 + c * jstep + lane, n - 1) + centre;
      ix[c] = split_coord(fma(m.b, jc, m.ax), L.cols, fx[c]);
      const int ix0 = lane_i32(ix[c], 0);  // the lanes' columns follow lane 0's (b > 0)
      const uint32_t off = (uint32_t)(ix[c] - ix0) * (uint32_t)sizeof(float);
      const float* row = L.screen + ix0 + (int64_t)iy[0] * L.pitch;
      top[c] = load_pair(row, off);
      row += L.pitch;
#pragma unroll
      for (int r = 0; r < kProjRows; ++r) {
        if (r > 0) row += (int64_t)(iy[r] - iy[r - 1]) * L.pitch;
        bot[c][r] = load_pair(row, off);
      }
    }
#pragma unroll
    for (int c = 0; c < kProjCols; ++c) {
      if (j0 + c * jstep >= n) break;
      const double gx = 1.0 - fx[c];
      double up = lerp(top[c].x, top[c].y, gx, fx[c]), down = 0.0;
#pragma unroll
      for (int r = 0; r < kProjRows; ++r) {
        if (r > 0) {
          if (shared) {
            if (iy[r] != iy[r - 1]) {  // one row further
              up = down;
              asm volatile("" : "+v"(up));  // a uniform branch, not selects by a lane mask
            }
          } else {
            const Pair p = load_pair(L.screen + (int64_t)iy[r] * L.pitch + ix[c], 0);
            up = lerp(p.x, p.y, gx, fx[c]);
          }
        }
        down = lerp(bot[c][r].x, bot[c][r].y, gx, fx[c]);
        acc[c][r] += lerp(up, down, lane_f64(gyv, r), lane_f64(fyv, r));
      }
    }
  }
  double tilt_x = 0.0, tilt_y = 0.0;
  if (a.tilt) {
    tilt_x = a.tilt[2 * t] * a.dx;
    tilt_y = a.tilt[2 * t + 1] * a.dx;
  }
#pragma unroll
  for (int c = 0; c < kProjCols; ++c) {
    const int j = j0 + c * jstep + lane;
    if (j >= n) break;
    const double jc = (double)j + centre;
    float* out = a.out + t * a.out_stride + j;
#pragma unroll
    for (int r = 0; r < kProjRows; ++r) {
      const int i = i0 + r;
      if (i < n) out[(int64_t)i * a.out_pitch] = (float)(acc[c][r] + fma(tilt_x, jc, tilt_y * ((double)i + centre)));
    }
  }
}

hipError_t launch_project_layers(const ProjectLaunch& a, bool maps, hipStream_t st) {
  constexpr int k8 = 8 * kRows;
  const int tiles = (a.pupil_n + 63) / 64;
  const dim3 grid(8u * (unsigned)a.n_t, (unsigned)((a.pupil_n + k8 - 1) / k8), (unsigned)((tiles + kProjCols - 1) / kProjCols));
  if (maps)
    hipLaunchKernelGGL(project_layers_kernel<true>, grid, dim3(64 * kProjWaves), 0, st, a);
  else
    hipLaunchKernelGGL(project_layers_kernel<false>, grid, dim3(64 * kProjWaves), 0, st, a);
  return hipGetLastError();
}

// One block of 1024 threads per LGS: each thread takes samples of the launch beam in groups of
// kUpGroup (their reads of a layer in flight together), FP64 sums reduced in a fixed order.  A few
// blocks only, so the time is one thread's chain of reads: 6 LGS x 64^2 samples x 3 layers take
// 7 us (21 us with 256 threads, one sample at a time and two divisions per sample and layer).
constexpr int kUpThreads = 1024;
constexpr int kUpGroup = 4;
__global__ __launch_bounds__(kUpThreads) void uplink_tilt_kernel(const UplinkLaunch a) {
  __shared__ double s_cx[kMaxLayers], s_cy[kMaxLayers];
  __shared__ double red[3][kUpThreads / 64];
  const int k = blockIdx.x, tid = threadIdx.x;
  const double* g = a.lgs[k];
  if (tid < a.L.n_layers) {
    // the beam centre at altitude h: launcher (1 - h/H) + h theta; the beam keeps its diameter
    const LayerDesc& L = a.L.layer[tid];
    const double f = 1.0 - L.alt_m / g[4];
    s_cx[tid] = g[0] * f + L.alt_m * g[2];
    s_cy[tid] = g[1] * f + L.alt_m * g[3];
  }
  __syncthreads();
  const double step = a.d / a.n_s, r2 = 0.25 * a.d * a.d;
  const int total = a.n_s * a.n_s;
  double sxo = 0.0, syo = 0.0, sxx = 0.0;
  for (int e0 = tid; e0 < total; e0 += kUpThreads * kUpGroup) {
    double sx[kUpGroup], sy[kUpGroup], opd[kUpGroup];
    bool in[kUpGroup];
#pragma unroll
    for (int q = 0; q < kUpGroup; ++q) {
      const int e = e0 + q * kUpThreads;
      const int si = e / a.n_s, sj = e - si * a.n_s;
      sx[q] = ((double)sj + 0.5 - 0.5 * a.n_s) * step;
      sy[q] = ((double)si + 0.5 - 0.5 * a.n_s) * step;
      in[q] = e < total && sx[q] * sx[q] + sy[q] * sy[q] <= r2;
      // samples outside the disc read the beam centre and are left out of the sums
      if (!in[q]) sx[q] = sy[q] = 0.0;
      opd[q] = 0.0;
    }
    for (int l = 0; l < a.L.n_layers; ++l) {
      const LayerDesc& L = a.L.layer[l];
      Pair p[kUpGroup], w[kUpGroup];
      double fx[kUpGroup], fy[kUpGroup];
#pragma unroll
      for (int q = 0; q < kUpGroup; ++q) {
        const int ix = split_coord(fma(s_cx[l] + sx[q], L.inv_pitch, L.x0), L.cols, fx[q]);
        const int iy = split_coord(fma(s_cy[l] + sy[q], L.inv_pitch, L.y0), L.rows, fy[q]);
        const float* at = L.screen + (int64_t)iy * L.pitch + ix;
        p[q] = load_pair(at, 0);
        w[q] = load_pair(at + L.pitch, 0);
      }
#pragma unroll
      for (int q = 0; q < kUpGroup; ++q)
        opd[q] += lerp(lerp(p[q].x, p[q].y, 1.0 - fx[q], fx[q]), lerp(w[q].x, w[q].y, 1.0 - fx[q], fx[q]), 1.0 - fy[q],
                       fy[q]);
    }
#pragma unroll
    for (int q = 0; q < kUpGroup; ++q) {
      if (in[q]) {
        sxo += sx[q] * opd[q];
        syo += sy[q] * opd[q];
        sxx += sx[q] * sx[q];  // the sample set is symmetric: sum sy^2 = sum sx^2, sum sx = sum sy = sum sx sy = 0
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sxo += __shfl_xor(sxo, off);
    syo += __shfl_xor(syo, off);
    sxx += __shfl_xor(sxx, off);
  }
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = sxo;
    red[1][tid >> 6] = syo;
    red[2][tid >> 6] = sxx;
  }
  __syncthreads();
  if (tid == 0) {
    double x = 0.0, y = 0.0, den = 0.0;
#pragma unroll
    for (int v = 0; v < kUpThreads / 64; ++v) {
      x += red[0][v];
      y += red[1][v];
      den += red[2][v];
    }
    a.tilt[2 * k] = den > 0.0 ? x / den : 0.0;
    a.tilt[2 * k + 1] = den > 0.0 ? y / den : 0.0;
  }
}

hipError_t launch_uplink_tilt(const UplinkLaunch& a, hipStream_t st) {
  hipLaunchKernelGGL(uplink_tilt_kernel, dim3((unsigned)a.n), dim3(kUpThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace shw
