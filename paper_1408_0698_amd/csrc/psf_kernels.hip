// psf_kernels.hip - science PSF accumulation (Sec. 3 PSF block, Sec. 5 Strehl).
//
// P(v,u) = |sum_{y,x} A e^{i phi} e^{-2 pi i ((u - M/2) x + (v - M/2) y) / M}|^2 / (sum A)^2
// with M = 1600 = 40 x 40, computed as a row pass then a column pass.
// Each M-point transform is the four-step split n = 40 n1 + n2,
// k = k1 + 40 k2: 40-point transforms over n1 (one per lane n2), the twiddle
// W_M^(n2 k1), a transpose through LDS, 40-point transforms over n2 (one
// per lane k1).  Only the first pupil_n <= M/2 inputs are non-zero, so the
// first 40-point transforms see n1 < 20 only and run as two 20-point
// transforms.  The fftshift centring (-1)^(x+y) is folded into the FP64
// phase as (x + y)/2 waves.
//
// Every line (a row in the row pass, a column in the column pass) is
// transformed by 40 lane pairs (q, h).  First step: lane (n2 = q, h) runs the
// 20-point transform of residue h of the pruned 40-point transform over n1,
// giving Y[k1] for k1 = 2k + h, and applies its four-step twiddles.  After a
// transpose through LDS, lane (k1 = q, h) holds the samples n2 = 2t + h of
// row k1, and the 40-point transform over n2 is split radix-2 across the
// pair: 20-point transforms, twiddle, butterfly with the partner through
// DPP; lane h ends with outputs k2 = c + 20 h.  In both steps register j of an
// odd lane stands for k or t = j + 2 mod 20: 40 = 8 x 5 without a common factor, so with that rotation
// the odd lane's twiddles W_40^j become W_8^j, half of them trivial (80 of 950
// instructions per column: 678 -> 638 us for 9 x 20 star-frames of 203-pixel pupils, 1098 -> 1090 of
// 800-pixel ones on the same card).  A lane keeps 20 complex values instead of 40.
//
// Row pass: 4 rows per block of 320 lanes; each lane of a pair computes half
// of the row's phases (all its OPD loads issued first) and shares them with its partner.  The intermediate is
// stored in column blocks of 4: element (frame f, row y, column u) of T sits
// at ((f * M/4 + u/4) * pupil_n + y) * 4 + u % 4, and a wavefront holds 8 consecutive outputs of all four rows,
// so that every store writes whole 128-byte lines (runs of 64 bytes, one row at a time, are written
// at 3.4 TB/s on this card, whole lines at 5.8; the stores alone took 650 us of 9 x 20 star-frames).
// Column pass: 4 columns per block, which are one contiguous region of T.  Each wavefront reads the rows it
// transforms straight into LDS, 16 bytes a lane, before it needs them; the frames' sums stay in LDS
// (each lane owns its 20 outputs), then one read-modify-write of the accumulator per call, 16 bytes
// (the block's 4 columns) per row, the 8 blocks of a 32-column group (one 128-byte line of every
// accumulator row) launched 8 apart, so that the dispatcher places them on one XCD and its L2 merges
// their writes; the on-axis sample of each frame is the Strehl ratio.  With an 80-register target 3 blocks
// share a CU (at 96 they fit too, but not after every order in which blocks end).  With more (the sums in
// registers: 124) only 2 do, because a CU takes 5-wavefront blocks only while every SIMD has room for 2 more of
// their wavefronts: 0.81 to 0.85 instead of 0.71 ms, and as much with 3 barriers a frame (transposes of complex
// values) as with 4.
// 9 stars x 20 frames: 1.07 to 1.10 ms for both passes back to back, traced 0.50 ms for the rows (4.6 TB/s) and 0.61 for the
// columns once the card has run them for some 0.2 s.  Before that it is slower: the first 20 calls of a run average
// 0.56 and 0.70 ms, and the other traced times here are such averages.  The rows are
// bound by HBM; the columns by issue (with the reads taken out they took 0.66 ms, the reads alone 0.44).
// 1.51 ms with T in column blocks of 8, one row or column per 80 consecutive lanes and each lane reading its
// column with 64-byte strides.
// Both passes have a form for pupil_n = M/2 (the Nyquist-sampled PSF), where
// every sample of the pruned transforms lies in the pupil grid, so its loads
// need no bounds masks.
#include <hip/hip_runtime.h>

#include "psf_internal.h"
#include "regfft.h"

namespace shw {

namespace {

constexpr int kM = 1600;
constexpr int kQ = 40;            // M = kQ * kQ
constexpr int kNZ = kM / 2 / kQ;  // non-zero n1 (20) = outputs per lane of the second step
constexpr int kP = 2 * kQ;        // lanes per line
constexpr int kLines = 4;         // lines per block
// LDS plane of one line's transpose: element (row r, column n) at plane_at(r, n).  Lanes (q, h) write
// (2k + h, q) and read (q, 2t + h); the 32 lanes served together (8 q, both h, two lines) touch 32 different
// banks in both, because 84 = 20 mod 32 and the plane's size is 16 mod 32.
constexpr int kPlane = (kQ / 2) * 84;
// Sums of one line: output v = q + 40 (c + 20 h) at q + 40 c + kHalf h, lines kSumStride apart; 8 and 16
// mod 32, for the same reason.
constexpr int kHalf = kM / 2 + 8;
constexpr int kSumStride = kM + 16;
constexpr int kCB = kLines;       // columns per block of the intermediate
constexpr int kFetch = kM / 2 * kLines * (int)sizeof(float2) / (16 * kLines * kP);  // 16-byte reads per lane and frame
static_assert(kFetch * 16 * kLines * kP == kM / 2 * kLines * (int)sizeof(float2), "a frame's columns in whole reads");
static_assert(kLines * kP / 64 * kFetch * 16 * 64 <= kLines * kPlane * (int)sizeof(float), "the columns fit the transposes' planes");
constexpr int kGroupCols = 32;    // columns per 128-byte accumulator line (8 column-pass blocks)

typedef float float2v __attribute__((ext_vector_type(2)));

// Offset of element (star-frame sf, row y, column u) of the intermediate.
__device__ __forceinline__ int64_t t_index(int64_t sf, int pupil_n, int y, int u) {
  return ((sf * (kM / kCB) + u / kCB) * pupil_n + y) * kCB + (u & (kCB - 1));
}

// Values of the same register in other lanes of the pair: the partner's (DPP quad permutation
// 1, 0, 3, 2), the even lane's (0, 0, 2, 2) and the odd lane's (1, 1, 3, 3).
template <int CTRL>
__device__ __forceinline__ float2 pair_perm(float2 v) {
  return make_float2(__int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v.x), CTRL, 0xF, 0xF, true)),
                     __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v.y), CTRL, 0xF, 0xF, true)));
}
__device__ __forceinline__ float2 pair_swap(float2 v) { return pair_perm<0xB1>(v); }
__device__ __forceinline__ float2 pair_even(float2 v) { return pair_perm<0xA0>(v); }
__device__ __forceinline__ float2 pair_odd(float2 v) { return pair_perm<0xF5>(v); }
__device__ __forceinline__ int plane_at(int r, int n) { return (r >> 1) * 84 + (r & 1) * 2 + (n >> 1) * 4 + (n & 1); }

// Lane pair and line of a thread: a wavefront holds 8 consecutive q of all four lines, so that the 4 x 8
// values it moves at a time to or from the intermediate are whole 128-byte lines.
__device__ __forceinline__ void lane_place(int tid, int& q, int& h, int& line) {
  h = tid & 1;
  q = ((tid >> 6) << 3) | ((tid >> 1) & 7);
  line = (tid >> 4) & 3;
}

// First register of a lane pair's odd lane whose index k or t = j + 2 h wraps round to j + 2 h - 20.
constexpr int kWrap = kNZ - 2;

// Four-step twiddles W_M^(n2 k1) of lane (n2 = q, h), k1 = 2k + h, k = j + 2 h mod 20 in register j: exact every
// 4 registers and where k wraps, products of W_M^(2 n2) between.
struct LineTwiddles {
  float2 start[kNZ / 4], wrap, step;
};
__device__ __forceinline__ LineTwiddles line_twiddles(int q, int h) {
  LineTwiddles tw;
  constexpr float kInvM = 1.0f / (float)kM;
  const float sr = -(float)(2 * q) * kInvM;  // 2 q < M
  tw.step = make_float2(__builtin_amdgcn_cosf(sr), __builtin_amdgcn_sinf(sr));
#pragma unroll
  for (int b = 0; b < kNZ / 4; ++b) {
    const float rev = -(float)(q * (8 * b + 5 * h)) * kInvM;  // q (8 b + 5 h) < M
    tw.start[b] = make_float2(__builtin_amdgcn_cosf(rev), __builtin_amdgcn_sinf(rev));
  }
  const float wr = -(float)(q * (h ? 1 : 2 * kWrap)) * kInvM;
  tw.wrap = make_float2(__builtin_amdgcn_cosf(wr), __builtin_amdgcn_sinf(wr));
  return tw;
}

// One M-point transform of a line with at most M/2 non-zero inputs v[n1] (sample 40 n1 + q),
// on lane pair (q, h) of the line; pl is the line's LDS plane.  On return lane (q, h) holds
// X[q + 40 (c + 20 h)] in x[c], c < 20.  Every lane of the block must call it.
// `moved` runs once every lane of the block has read the plane.
template <class F>
__device__ __forceinline__ void line_transform(const float2 (&v)[kNZ], float2 (&x)[kNZ], float* pl,
                                               const LineTwiddles& tw, int q, int h, F moved) {
  float2 z[kNZ];
#pragma unroll
  for (int n1 = 0; n1 < kNZ; ++n1) z[n1] = v[n1];
  if (h) {  // lanes with odd outputs
#pragma unroll
    for (int n1 = 0; n1 < kNZ; ++n1) z[n1] = twiddle_mul<8, -1>(z[n1], n1);
  }
  RegFFT<kNZ, -1>::run(z);
  // four-step twiddle W_M^(n2 k1), k1 = 2k + h
  {
    float2 step = tw.step;
    // an opaque copy: in a loop over frames the products below are formed again rather than kept live
    asm volatile("" : "+v"(step.x), "+v"(step.y));
#pragma unroll
    for (int b = 0; b < kNZ / 4; ++b) {
      float2 t = tw.start[b];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (4 * b + e == kWrap) t = tw.wrap;
        z[4 * b + e] = cmul(z[4 * b + e], t);
        t = cmul(t, step);
      }
    }
  }
  // transpose: lane (n2, h) holds Y[2k + h]; lane (k1, h) takes samples n2 = 2t + h; k and t are j + 2 h mod 20
  float* wr = pl + plane_at(h, q) + 2 * 84 * h;           // row 2k + h is 84 k further on
  const float* rd = pl + plane_at(q, h) + 2 * 4 * h;      // column 2t + h is 4 t further on
  int hh = h;  // opaque: in a loop over frames the two are formed again rather than kept
  asm volatile("" : "+v"(hh));
  float* wr_wrap = wr - kNZ * 84 * hh;
  const float* rd_wrap = rd - kNZ * 4 * hh;
#pragma unroll
  for (int k = 0; k < kNZ; ++k) (k < kWrap ? wr : wr_wrap)[84 * k] = z[k].x;
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kNZ; ++t) x[t].x = (t < kWrap ? rd : rd_wrap)[4 * t];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kNZ; ++k) (k < kWrap ? wr : wr_wrap)[84 * k] = z[k].y;
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kNZ; ++t) x[t].y = (t < kWrap ? rd : rd_wrap)[4 * t];
  __syncthreads();
  moved();
  RegFFT<kNZ, -1>::run(x);
  __builtin_amdgcn_sched_barrier(0);  // the products below, moved up into the transform, cost registers
  if (h) {
#pragma unroll
    for (int c = 0; c < kNZ; ++c) x[c] = twiddle_mul<8, -1>(x[c], c);
  }
  // h = 0: X[c] = E + W O (partner holds W O); h = 1: X[c + 20] = E (partner) - W O, one fused operation
  // by the lane's sign for both
  const float sgn = h ? -1.0f : 1.0f;
#pragma unroll
  for (int c = 0; c < kNZ; ++c) {
    const float2 o = pair_swap(x[c]);
    x[c] = make_float2(fmaf(sgn, x[c].x, o.x), fmaf(sgn, x[c].y, o.y));
  }
}

}  // namespace

// FULL: pupil_n = M / 2, so every sample 40 n1 + q (n1 < 20) lies inside the grid.
template <bool FULL>
__global__ __launch_bounds__(kLines * kP) void psf_rows_kernel(const PsfLaunch a, int64_t f0, int nf,
                                                               float2* __restrict__ T) {
  __shared__ float s_pl[kLines * kPlane];
  const int tid = threadIdx.x;
  int q, h, line;
  lane_place(tid, q, h, line);
  // a block's rows belong to one star-frame, so its place is worked out on the scalar unit
  const uint32_t row_blocks = (uint32_t)(a.pupil_n + kLines - 1) / kLines;
  const uint32_t sf = blockIdx.x / row_blocks;  // star * nf + frame - f0
  const int y = (int)(blockIdx.x - sf * row_blocks) * kLines + line;
  const bool active = y < a.pupil_n;
  const uint32_t star = sf / (uint32_t)nf, fl = sf - star * (uint32_t)nf;
  float* pl = s_pl + line * kPlane;
  // field samples x = 40 n1 + q; lane h computes those with n1 = h (mod 2), then the pair swaps
  float2 v[kNZ];
  {
    const float* src = a.opd + star * a.star_stride + (f0 + fl) * a.frame_stride + (int64_t)(active ? y : 0) * a.row_pitch;
    const float by = (float)y + 0.5f - a.half_n;
    const float by2 = by * by;
    // (-1)^(x + y) in waves: x = 40 n1 + q has the parity of q
    const double centring = (q + y) & 1 ? 0.5 : 0.0;
    // every load is issued before any is used (at a clamped address), and the samples outside
    // the pupil, the annulus or the last block's rows are masked afterwards
    float ov[kNZ / 2];
#pragma unroll
    for (int i = 0; i < kNZ / 2; ++i) ov[i] = src[FULL ? kQ * (2 * i + h) + q : min(kQ * (2 * i + h) + q, a.pupil_n - 1)];
#pragma unroll
    for (int i = 0; i < kNZ / 2; ++i) {
      const int n1 = 2 * i + h;
      const int x = kQ * n1 + q;
      const float bx = (float)x + 0.5f - a.half_n;
      const float r2 = bx * bx + by2;
      const bool lit = active & (FULL || x < a.pupil_n) & (r2 <= a.r2_outer) & (r2 >= a.r2_inner);
      const double wv = __builtin_amdgcn_fract(fma((double)ov[i], a.inv_lambda, centring));  // wv - floor(wv)
      // hardware sine and cosine take revolutions: exp(2 pi i wv) after the FP64 reduction
      const float fw = (float)wv;
      // a select, not a product with a 0/1 amplitude: samples outside the pupil may hold anything
      const float cw = __builtin_amdgcn_cosf(fw), sw = __builtin_amdgcn_sinf(fw);
      const float2 e = make_float2(lit ? cw : 0.0f, lit ? sw : 0.0f);
      v[2 * i] = pair_even(e);
      v[2 * i + 1] = pair_odd(e);
    }
  }
  float2 x[kNZ];
  line_transform(v, x, pl, line_twiddles(q, h), q, h, [] {});
  if (active) {
    // column q + 40 (c + 20 h): its column block advances by 10 per c and its place in the block
    // stays q % 4, so the outputs are 40 pupil_n elements apart (a scalar step; a star-frame is 10 MB at most)
    using GlobalF2 = __attribute__((address_space(1))) float2v;
    __attribute__((address_space(1))) char* base = (__attribute__((address_space(1))) char*)(T + t_index(sf, a.pupil_n, 0, 0));
    const uint32_t at = (uint32_t)t_index(0, a.pupil_n, y, q + kQ * kNZ * h) * sizeof(float2);
    const uint32_t step = (uint32_t)(kQ / kCB) * a.pupil_n * kCB * sizeof(float2);
#pragma unroll
    for (int c = 0; c < kNZ; ++c) *(GlobalF2*)(base + c * (size_t)step + at) = float2v{x[c].x, x[c].y};
  }
}

// Column pass.  Block b = 64 j + 8 m + x takes columns 4 m .. 4 m + 3 of the 32-column group
// g = 8 j + x (groups past the last one leave at once).
template <bool FULL>
__global__ __launch_bounds__(kLines * kP) __attribute__((amdgpu_waves_per_eu(6))) void psf_cols_kernel(const PsfLaunch a, int64_t f0, int nf,
                                                               int n_groups, const float2* __restrict__ T,
                                                               float* __restrict__ acc, float* __restrict__ strehl) {
  // the transposes' planes; before them each wavefront's part of the columns of a frame
  extern __shared__ __align__(16) float s_pl[];
  // per-line sums over the frames; each lane owns its outputs'
  float* const s_sum = s_pl + kLines * kPlane;
  const int tid = threadIdx.x;
  int q, h, line;
  lane_place(tid, q, h, line);
  const int b = blockIdx.x;
  const int m = (b >> 3) & 7;
  const int g = (b >> 6) * 8 + (b & 7);
  if (g >= n_groups) return;  // the whole block
  constexpr int kGroups = kM / kGroupCols;
  const int star = g / kGroups;
  const int u0 = (g - star * kGroups) * kGroupCols + m * kLines;  // first column of the block
  const int u = u0 + line;
  float* pl = s_pl + line * kPlane;
  // Reads the rows 40 n1 + q of a frame's columns that this wavefront transforms straight into LDS, 16
  // bytes a lane (8 rows of the block's columns, 256 bytes, lie together).  A lane's place there is
  // its number, so it picks what to read: 16-byte unit P holds columns 2 ((P >> 3) & 1) .. + 1 of row
  // 40 (P >> 4) + 8 wave + (P & 7), and the 8 rows that a wavefront reads together below lie in 8 different
  // bank quads.
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rows = FULL ? kM / 2 : a.pupil_n;
  const int row0 = kQ * ((tid & 63) >> 4) + (wave * 8) + (tid & 7);  // row of the lane's first unit; the next ones are kFetchRows on
  constexpr int kFetchRows = 4 * kQ;
  constexpr int kFetchBytes = 16 * 64;  // of LDS per step of the wavefront
  float2* part = reinterpret_cast<float2*>(s_pl) + wave * (kFetch * kFetchBytes / (int)sizeof(float2));
  const uint32_t lane_off = (uint32_t)(row0 * kLines + 2 * ((tid >> 3) & 1)) * sizeof(float2);
  auto fetch = [&](int fl) {
    using GlobalC = __attribute__((address_space(1))) const char;
    const GlobalC* src = (const GlobalC*)(T + t_index((int64_t)star * nf + fl, a.pupil_n, 0, u0));
#pragma unroll
    for (int i = 0; i < kFetch; ++i) {
      constexpr int kBytes = kFetchRows * kLines * (int)sizeof(float2);
      if (FULL || i * kFetchRows + row0 < rows)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + i * kBytes + lane_off),
                                         (__attribute__((address_space(3))) void*)((char*)part + i * kFetchBytes),
                                         16, 0, 0);
    }
  };
  // row 40 n1 + q of the lane's column, 32 n1 further on
  const float2* in = part + (line >> 1) * 16 + (q & 7) * 2 + (line & 1);
  const LineTwiddles tw = line_twiddles(q, h);
  float* sum = s_sum + line * kSumStride + q + kHalf * h;  // output q + 40 (c + 20 h) is 40 c further on
#pragma unroll
  for (int c = 0; c < kNZ; ++c) sum[kQ * c] = 0.0f;
  fetch(0);
  for (int fl = 0; fl < nf; ++fl) {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's part of the columns is in LDS
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    // rows 40 n1 + q of column u; with FULL every row is inside the pupil
    float2 v[kNZ];
#pragma unroll
    for (int n1 = 0; n1 < kNZ; ++n1)
      v[n1] = FULL || kQ * n1 + q < rows ? in[32 * n1] : make_float2(0.0f, 0.0f);
    __syncthreads();  // every wavefront has read its part
    float2 x[kNZ];
    line_transform(v, x, pl, tw, q, h, [&] {
      if (fl + 1 < nf) fetch(fl + 1);
    });
#pragma unroll
    for (int c = 0; c < kNZ; ++c) sum[kQ * c] = fmaf(fmaf(x[c].x, x[c].x, x[c].y * x[c].y), a.inv_norm, sum[kQ * c]);
    // on-axis sample: v = u = M/2, i.e. k1 = 0, k2 = 20 (c = 0, h = 1) of column M/2
    if (strehl && u == kM / 2 && q == 0 && h == 1)
      strehl[(int64_t)star * a.n_frames + f0 + fl] = fmaf(x[0].x, x[0].x, x[0].y * x[0].y) * a.inv_norm;
  }
  __syncthreads();
  // accumulator rows v, columns u0 .. u0 + 3: one 16-byte read-modify-write per row when the
  // accumulator allows it (u0 is a multiple of 4), else four 4-byte ones
  float* ac = acc + star * a.acc_stride + u0;
  if ((reinterpret_cast<uintptr_t>(ac) & 15) == 0) {
    for (int vv = tid; vv < kM; vv += kLines * kP) {
      float4* pa = reinterpret_cast<float4*>(ac + (int64_t)vv * kM);
      const int at = vv < kM / 2 ? vv : vv + (kHalf - kM / 2);
      float4 o = *pa;
      o.x += s_sum[at];
      o.y += s_sum[kSumStride + at];
      o.z += s_sum[2 * kSumStride + at];
      o.w += s_sum[3 * kSumStride + at];
      *pa = o;
    }
  } else {
    for (int e = tid; e < kM * kLines; e += kLines * kP) {
      const int vv = e >> 2, l = e & 3;
      const int at = vv < kM / 2 ? vv : vv + (kHalf - kM / 2);
      float* pa = ac + (int64_t)vv * kM + l;
      *pa += s_sum[l * kSumStride + at];
    }
  }
}

bool psf_size_supported(int fft_m, int pupil_n) { return fft_m == kM && pupil_n >= 1 && pupil_n <= kM / 2; }

hipError_t launch_psf_rows(const PsfLaunch& a, int n_stars, int64_t f0, int nf, float2* T, hipStream_t st) {
  const int64_t rb = (int64_t)n_stars * nf * ((a.pupil_n + kLines - 1) / kLines);
  if (a.pupil_n == kM / 2)
    hipLaunchKernelGGL(psf_rows_kernel<true>, dim3((unsigned)rb), dim3(kLines * kP), 0, st, a, f0, nf, T);
  else
    hipLaunchKernelGGL(psf_rows_kernel<false>, dim3((unsigned)rb), dim3(kLines * kP), 0, st, a, f0, nf, T);
  return hipGetLastError();
}

hipError_t launch_psf_cols(const PsfLaunch& a, int n_stars, int64_t f0, int nf, const float2* T, float* acc,
                           float* strehl, hipStream_t st) {
  static_assert(kGroupCols == 8 * kLines && kM % kGroupCols == 0, "8 blocks per 32-column group");
  const int n_groups = n_stars * (kM / kGroupCols);
  const dim3 cg((unsigned)(((n_groups + 7) / 8) * 64));
  // the size is given here and not by static arrays: knowing it, the compiler counts 3 blocks as 4 wavefronts a
  // SIMD and claims the registers that 4 may have, with which only 2 blocks fit (0.85 instead of 0.71 ms)
  constexpr unsigned kLds = kLines * (kPlane + kSumStride) * sizeof(float);
  if (a.pupil_n == kM / 2)
    hipLaunchKernelGGL(psf_cols_kernel<true>, cg, dim3(kLines * kP), kLds, st, a, f0, nf, n_groups, T, acc, strehl);
  else
    hipLaunchKernelGGL(psf_cols_kernel<false>, cg, dim3(kLines * kP), kLds, st, a, f0, nf, n_groups, T, acc, strehl);
  return hipGetLastError();
}

}  // namespace shw
