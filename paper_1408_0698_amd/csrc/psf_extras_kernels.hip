// psf_extras_kernels.hip - encircled energy of a PSF and resampling of a PSF to another
// wavelength's angular grid (Sec. 3 PSF block: PSFs at one or several wavelengths weighted by
// the object's colour; Strehl ratio and encircled energy in a chosen radius).
#include <hip/hip_runtime.h>

#include <mutex>

#include "geom_internal.h"

namespace shw {

// Workspace of the allocation-free encircled-energy entry point: one copy of this array per GPU,
// held until the process ends.  In host code the name stands for a host-side shadow, not a device
// address; kernels receive the address from ee_scratch_device() below.
static __device__ __align__(256) double scratch[kEeScratchDoubles];

// Largest integer w with w^2 <= q (q >= 0).
__device__ __forceinline__ int isqrt_floor(double q) {
  int w = (int)floor(sqrt(q));
  while ((double)(w + 1) * (w + 1) <= q) ++w;
  while (w > 0 && (double)w * w > q) --w;
  return w;
}

// Pass 1.  The pixels within radius r of a row at dv from the centre c = M/2 form the run |u - c| <= w,
// w = floor(sqrt(r^2 - dv^2)), the same for the rows c + dv and c - dv.  So the two rows are folded
// about the centre first, G[j] = P[c + dv][c + j] + P[c + dv][c - j] + P[c - dv][c + j] + P[c - dv][c - j],
// and their share of radius r is the prefix sum of G up to w: a quarter of the pixels to scan, one
// window for both rows, one prefix instead of a difference of two.
// A wavefront takes one pair of rows: lane l holds j = 256 i + 4 l .. 4 l + 3 (16-byte reads of both
// sides of both rows, all in flight together), FP64 sums, a scan over the lanes for every i, and the
// prefixes go to LDS, where lane k < n_r reads radius k's.  The column u = 0 of an even M (and any
// other without a mirror image) has j past the folded part and is added to the windows that
// reach it.  Block (g, s) takes the row distances g, g + G, ... of PSF s, one per wavefront at a time;
// its wavefronts are added in a fixed order.
// Bound by the read: 9 PSFs of 1600^2 (92 MB) take 21 us traced = 4.4 TB/s; a wavefront per single row,
// staged in LDS and scanned whole, took 52 us.
constexpr int kEeWaves = 4;
constexpr int kEeSteps = 4;  // 256-pixel steps that cover a folded half row: M <= 2048
static_assert(kMaxRadii <= 64, "one lane per radius");

// Pixels p .. p + 3 (16 bytes at 4-byte alignment).
typedef float EeQuad __attribute__((ext_vector_type(4), aligned(4)));

// Inclusive sums over the lanes of a wavefront, in a fixed order.
__device__ __forceinline__ double ee_scan(double v, int lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double t = __shfl_up(v, off);
    if (lane >= off) v += t;
  }
  return v;
}

__global__ __launch_bounds__(64 * kEeWaves) void ee_rows_kernel(const EeLaunch a) {
  extern __shared__ __align__(16) double ee_pre[];  // [wavefront][H rounded up to 4]
  __shared__ double fin[kEeWaves][kMaxRadii + 1];
  const int M = a.m, c = M / 2;
  // folded part: j < H has both c + j and c - j inside the row, in whole quads; pixels beyond it are
  // added one by one
  const int H = ((M - c) < (c + 1) ? (M - c) : (c + 1)) & ~3;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = blockIdx.x, s = blockIdx.y;
  double* pre = ee_pre + wave * H;
  const float* P = a.psf + s * a.psf_stride;
  const double r2 = lane < a.n_r ? a.r2[lane] : -1.0;
  double acc = 0.0, tot = 0.0;
  for (int dv = g + wave * kEeGroups; dv <= c; dv += kEeWaves * kEeGroups) {
    // rows c + dv and c - dv, or the one of them that is there (dv = 0: the centre row once)
    const bool pair = dv > 0 && c + dv < M;
    const float* hi = P + (int64_t)(c + dv < M ? c + dv : c - dv) * M;
    const float* lo = P + (int64_t)(c - dv) * M;
    EeQuad q[kEeSteps][4];
#pragma unroll
    for (int i = 0; i < kEeSteps; ++i) {
      const int j = 256 * i + 4 * lane;
#pragma unroll
      for (int k = 0; k < 4; ++k) q[i][k] = EeQuad{0.0f, 0.0f, 0.0f, 0.0f};
      if (j < H) {
        q[i][0] = *reinterpret_cast<const EeQuad*>(hi + c + j);
        q[i][1] = *reinterpret_cast<const EeQuad*>(hi + c - j - 3);
        if (pair) {
          q[i][2] = *reinterpret_cast<const EeQuad*>(lo + c + j);
          q[i][3] = *reinterpret_cast<const EeQuad*>(lo + c - j - 3);
        }
      }
    }
    // radius window of this row distance
    const double rem = r2 - (double)dv * (double)dv;
    const int w = rem >= 0.0 ? isqrt_floor(rem) : -1;
    // pixels outside the folded part, with the windows that reach them (few; uniform addresses)
    double edge = 0.0, edge_tot = 0.0;
    auto single = [&](int u) {
      double v = (double)hi[u];
      if (pair) v += (double)lo[u];
      edge_tot += v;
      if (abs(u - c) <= w) edge += v;
    };
    for (int u = c + H; u < M; ++u) single(u);
    for (int u = c - (H > 0 ? H : 1); u >= 0; --u) single(u);
    double carry = 0.0;
#pragma unroll
    for (int i = 0; i < kEeSteps; ++i) {
      double p[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        // the centre column (j = 0) has no mirror image
        const bool centre = i == 0 && k == 0 && lane == 0;
        double t = (double)q[i][0][k] + (double)q[i][2][k];
        const double f = (double)q[i][1][3 - k] + (double)q[i][3][3 - k];
        t += centre ? 0.0 : f;
        p[k] = k > 0 ? p[k - 1] + t : t;
      }
      const double inc = ee_scan(p[3], lane);
      const double base = carry + (inc - p[3]);
      const int j = 256 * i + 4 * lane;
      if (j < H) {
#pragma unroll
        for (int k = 0; k < 4; ++k) pre[j + k] = base + p[k];
      }
      carry += __shfl(inc, 63);
    }
    // the prefixes are written and read by this wavefront only: order its LDS accesses
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    tot += carry + edge_tot;
    if (w >= 0) acc += (H > 0 ? pre[min(w, H - 1)] : 0.0) + edge;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  if (lane < a.n_r) fin[wave][lane] = acc;
  if (lane == 0) fin[wave][a.n_r] = tot;
  __syncthreads();
  if ((int)threadIdx.x <= a.n_r) {
    double t = 0.0;
#pragma unroll
    for (int v = 0; v < kEeWaves; ++v) t += fin[v][threadIdx.x];
    a.ws[((int64_t)s * (a.n_r + 1) + threadIdx.x) * kEeGroups + g] = t;
  }
}

// Pass 2: block s adds the groups of PSF s and divides by the total.  Wavefront w takes entries
// k = w, w + 16, ... <= n_r; lane l adds groups l, l + 64, ... (read together), then a fixed tree over
// the lanes.
constexpr int kEeFinalWaves = 16;
__global__ __launch_bounds__(64 * kEeFinalWaves) void ee_final_kernel(const EeLaunch a) {
  __shared__ double s_tot[kMaxRadii + 1];
  const int s = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int kParts = (kEeGroups + 63) / 64;
  for (int k = wave; k <= a.n_r; k += kEeFinalWaves) {
    const double* w = a.ws + ((int64_t)s * (a.n_r + 1) + k) * kEeGroups;
    double v[kParts];
#pragma unroll
    for (int t = 0; t < kParts; ++t) v[t] = lane + 64 * t < kEeGroups ? w[lane + 64 * t] : 0.0;
    double x = 0.0;
#pragma unroll
    for (int t = 0; t < kParts; ++t) x += v[t];
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    if (lane == 0) s_tot[k] = x;
  }
  __syncthreads();
  if ((int)threadIdx.x < a.n_r) {
    const double tot = s_tot[a.n_r], in = s_tot[threadIdx.x];
    a.ee[(int64_t)s * a.n_r + threadIdx.x] = tot > 0.0 ? in / tot : 0.0;
  }
}

hipError_t launch_encircled_energy(const EeLaunch& a, hipStream_t st) {
  const int c = a.m / 2;
  const int h = (a.m - c < c + 1 ? a.m - c : c + 1) & ~3;
  const size_t lds = (size_t)kEeWaves * h * sizeof(double);
  const dim3 grid(kEeGroups, (unsigned)a.n_psf);
  if (h > kEeSteps * 256) return hipErrorInvalidValue;
  hipLaunchKernelGGL(ee_rows_kernel, grid, dim3(64 * kEeWaves), lds, st, a);
  hipLaunchKernelGGL(ee_final_kernel, dim3((unsigned)a.n_psf), dim3(64 * kEeFinalWaves), 0, st, a);
  return hipGetLastError();
}

hipError_t ee_scratch_device(int device, double** out) {
  static std::mutex mu;
  static double* addr[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[device]) {
    // the caller has made `device` current; each GPU holds its own copy at its own address
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[device] = static_cast<double*>(p);
  }
  *out = addr[device];
  return hipSuccess;
}

// dst[v][u] += w * src sampled bilinearly at (c + (v - c) s, c + (u - c) s), c = M/2; samples
// outside [0, M - 1]^2 add nothing.
__global__ __launch_bounds__(256) void psf_resample_kernel(const float* __restrict__ src, int32_t m, double s, float w,
                                                           float* __restrict__ dst) {
  const int u = blockIdx.x * 256 + threadIdx.x, v = blockIdx.y;
  if (u >= m) return;
  const int c = m / 2;
  const double X = c + (u - c) * s, Y = c + (v - c) * s;
  if (X < 0.0 || Y < 0.0 || X > (double)(m - 1) || Y > (double)(m - 1)) return;
  int ix = (int)floor(X), iy = (int)floor(Y);
  ix = ix > m - 2 ? m - 2 : ix;
  iy = iy > m - 2 ? m - 2 : iy;
  const double fx = X - ix, fy = Y - iy;
  const float* r0 = src + (int64_t)iy * m + ix;
  const float* r1 = r0 + m;
  const double top = (1.0 - fx) * (double)r0[0] + fx * (double)r0[1];
  const double bot = (1.0 - fx) * (double)r1[0] + fx * (double)r1[1];
  dst[(int64_t)v * m + u] += (float)((double)w * ((1.0 - fy) * top + fy * bot));
}

hipError_t launch_psf_resample(const float* src, int32_t m, double s, float w, float* dst, hipStream_t st) {
  hipLaunchKernelGGL(psf_resample_kernel, dim3((unsigned)((m + 255) / 256), (unsigned)m), dim3(256), 0, st, src, m,
                     s, w, dst);
  return hipGetLastError();
}

}  // namespace shw
