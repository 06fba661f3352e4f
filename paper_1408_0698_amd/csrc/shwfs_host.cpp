// shwfs_host.cpp - host side of the C ABI (include/shwfs.h).
//
// Validation, sub-aperture geometry and the LGS kernel parameters are
// computed here in FP64 on the host; every per-frame step runs in the HIP
// kernels.  Validation touches no HIP API, so it runs without a GPU.
#include "../../include/shwfs.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <string>
#include <vector>

#include "geom_internal.h"
#include "internal.h"
#include "psf_internal.h"
#include "dm_internal.h"
#include "recon_internal.h"
#include "big_internal.h"
#include "mfma_internal.h"

using namespace shw;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

int ok() {
  g_err.clear();
  return SHW_OK;
}

int hip_fail(hipError_t e, const char* what) {
  if (e == hipErrorOutOfMemory) return fail(SHW_E_NOMEM, "%s: %s", what, hipGetErrorString(e));
  return fail(SHW_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

constexpr double kArcsec = 3.14159265358979323846 / (180.0 * 3600.0);

bool is_fin(double v) { return std::isfinite(v); }

}  // namespace

constexpr int kListRing = 4;  // host staging slots of the work lists

struct shw_wfs_plan {
  shw_wfs_config cfg;
  int32_t n_wfs = 0;
  int32_t n_valid = 0;
  int32_t npx = 0;
  WfsShape shape{};
  int device = 0;
  int32_t* d_valid = nullptr;
  int32_t* d_inv = nullptr;      // shapes with calibration pairs: number of each valid sub-aperture, in d_valid's block
  float* d_khat = nullptr;
  float* d_khat_band = nullptr;  // in-band K^ rows of the band-limited variants and the MFMA form, or null
  size_t bytes = 0;
  std::vector<int32_t> valid;
  int32_t variant = 0;
  int32_t noise_head = 4;        // lockstep inversion steps of det_noise_kernel: 2, 4 or 6
  int32_t prec = 0;              // SHW_PREC_*: 0 = FP32 register FFTs, else MFMA DFT GEMMs
  uint4* d_mfma_tab = nullptr;   // constant operands of the MFMA variant
  FrameWork* d_list = nullptr;   // work list of sh_wfs_measure_batch
  int32_t list_cap = 0;
  // pinned host staging of the work lists: kListRing slots of list_cap entries, each reusable once
  // the event recorded after its upload has completed
  FrameWork* h_ring = nullptr;
  hipEvent_t ring_ev[kListRing] = {};
  bool ring_pending[kListRing] = {};
  int32_t ring_next = 0;
  // large sub-apertures (FFT 512): row/column workspace for chunk_items work items
  bool big = false;
  int64_t chunk_items = 0;
  float2* d_T = nullptr;
  float* d_Jr = nullptr;
  // sodium sub-layers: [n_sub][2] (phase coefficient, weight) then [n_wfs][2] launcher pixels
  int32_t n_sub = 0;
  double* d_sub = nullptr;
  // detector values of the detector-split launch variants: det_ws_items items of det_n^2 floats
  float* d_det_ws = nullptr;
  int64_t det_ws_items = 0;
};



extern "C" const char* shw_last_error(void) { return g_err.c_str(); }

extern "C" int32_t shw_abi_version(void) { return SHW_ABI_VERSION; }

// ---------------------------------------------------------------- validation

static int check_config(const shw_wfs_config* c, int32_t n_wfs, const shw_lgs_geom* geom) {
  if (!c) return fail(SHW_E_INVALID, "config is NULL");
  if (c->abi_version != SHW_ABI_VERSION)
    return fail(SHW_E_ABI, "abi_version %d, library %d", c->abi_version, SHW_ABI_VERSION);
  if (n_wfs < 1 || n_wfs > 4096) return fail(SHW_E_INVALID, "n_wfs %d outside [1, 4096]", n_wfs);
  if (c->pupil_n < 1 || c->pupil_n > 16384) return fail(SHW_E_INVALID, "pupil_n %d outside [1, 16384]", c->pupil_n);
  if (!(is_fin(c->pupil_dx_m) && c->pupil_dx_m > 0)) return fail(SHW_E_INVALID, "pupil_dx_m must be > 0");
  if (!(is_fin(c->obstruction) && c->obstruction >= 0 && c->obstruction < 1))
    return fail(SHW_E_INVALID, "obstruction must be in [0, 1)");
  if (c->n_subap < 1 || c->pupil_n % c->n_subap != 0)
    return fail(SHW_E_INVALID, "n_subap %d must divide pupil_n %d", c->n_subap, c->pupil_n);
  const int npx = c->pupil_n / c->n_subap;
  if (c->fft_n < npx || c->fft_n > 4096)
    return fail(SHW_E_INVALID, "fft_n %d must be in [sub-aperture size %d, 4096]", c->fft_n, npx);
  if (c->conv_n < c->fft_n || (c->conv_n - c->fft_n) % 2 != 0)
    return fail(SHW_E_INVALID, "conv_n %d must be >= fft_n %d with an even difference", c->conv_n, c->fft_n);
  if (c->det_n < 1 || c->det_n > c->conv_n) return fail(SHW_E_INVALID, "det_n %d outside [1, conv_n]", c->det_n);
  if (c->lgs != 0 && c->lgs != 1) return fail(SHW_E_INVALID, "lgs must be 0 or 1");
  if (c->flags & ~(SHW_FLAG_NOISE | (0xFu << SHW_PRECISION_SHIFT))) return fail(SHW_E_INVALID, "unknown flag bits");
  const unsigned prec = (c->flags >> SHW_PRECISION_SHIFT) & 0xFu;
  if (prec > SHW_PREC_FP16X3) return fail(SHW_E_INVALID, "unknown precision %u", prec);
  if (!(is_fin(c->min_illum) && c->min_illum > 0 && c->min_illum <= 1))
    return fail(SHW_E_INVALID, "min_illum must be in (0, 1]");
  if (!(is_fin(c->wavelength_m) && c->wavelength_m > 0)) return fail(SHW_E_INVALID, "wavelength_m must be > 0");
  if (!(is_fin(c->photons_per_subap) && c->photons_per_subap >= 0))
    return fail(SHW_E_INVALID, "photons_per_subap must be >= 0");
  if (!(is_fin(c->ron_e) && c->ron_e >= 0)) return fail(SHW_E_INVALID, "ron_e must be >= 0");
  if (!is_fin(c->threshold_e)) return fail(SHW_E_INVALID, "threshold_e must be finite");
  if (c->lgs) {
    if (!geom) return fail(SHW_E_INVALID, "LGS geometry needs launch positions");
    if (!(is_fin(c->spot_fwhm_arcsec) && c->spot_fwhm_arcsec > 0))
      return fail(SHW_E_INVALID, "spot_fwhm_arcsec must be > 0");
    if (!is_fin(c->elong_max_arcsec)) return fail(SHW_E_INVALID, "elong_max_arcsec must be finite");
    if (c->elong_max_arcsec <= 0 &&
        !(is_fin(c->na_height_m) && c->na_height_m > 0 && is_fin(c->na_fwhm_m) && c->na_fwhm_m >= 0))
      return fail(SHW_E_INVALID, "geometric elongation needs na_height_m > 0 and na_fwhm_m >= 0");
    for (int w = 0; w < n_wfs; ++w)
      if (!is_fin(geom[w].launch_x_m) || !is_fin(geom[w].launch_y_m))
        return fail(SHW_E_INVALID, "launch position %d not finite", w);
  }
  if (prec != SHW_PREC_FP32) {
    if (!mfma_shape_supported(npx, c->fft_n, c->conv_n, c->det_n, (int)prec))
      return fail(SHW_E_UNSUPPORTED, "precision %u has no kernel for this shape", prec);
    return SHW_OK;
  }
  const WfsShape shape{npx, c->fft_n, c->conv_n, c->det_n, c->lgs};
  if (!wfs_shape_supported(shape) && !big_shape_supported(npx, c->fft_n, c->conv_n, c->det_n, c->lgs))
    return fail(SHW_E_UNSUPPORTED, "no kernel for npx %d, fft_n %d, conv_n %d, det_n %d, lgs %d", npx, c->fft_n,
                c->conv_n, c->det_n, c->lgs);
  return SHW_OK;
}

extern "C" int shw_wfs_config_check(const shw_wfs_config* cfg, int32_t n_wfs, const shw_lgs_geom* geom) {
  const int r = check_config(cfg, n_wfs, geom);
  return r == SHW_OK ? ok() : r;
}

// ---------------------------------------------------------------- geometry

// Lit pupil pixel: centre at half-integer pixel coordinates; the squared radius
// is exact in FP64, so the annulus test is exact.
static bool lit(const shw_wfs_config* c, int r, int col) {
  const double h = c->pupil_n / 2.0;
  const double a = col + 0.5 - h, b = r + 0.5 - h;
  const double r2 = a * a + b * b;
  const double ro = h * h;
  const double ri = (c->obstruction * h) * (c->obstruction * h);
  return r2 <= ro && r2 >= ri;
}

static void valid_table(const shw_wfs_config* c, std::vector<int32_t>& idx, std::vector<double>& illum) {
  const int n = c->pupil_n / c->n_subap;
  idx.clear();
  illum.clear();
  for (int sa = 0; sa < c->n_subap; ++sa)
    for (int sb = 0; sb < c->n_subap; ++sb) {
      int cnt = 0;
      for (int y = 0; y < n; ++y)
        for (int x = 0; x < n; ++x) cnt += lit(c, sa * n + y, sb * n + x) ? 1 : 0;
      const double frac = (double)cnt / (double)(n * n);
      if (frac >= c->min_illum) {
        idx.push_back(sa * c->n_subap + sb);
        illum.push_back(frac);
      }
    }
}

extern "C" int shw_wfs_geometry(const shw_wfs_config* cfg, int32_t* n_valid, int32_t* valid_idx, double* illum) {
  if (!cfg || !n_valid) return fail(SHW_E_INVALID, "NULL argument");
  if (cfg->abi_version != SHW_ABI_VERSION) return fail(SHW_E_ABI, "abi_version mismatch");
  if (cfg->pupil_n < 1 || cfg->n_subap < 1 || cfg->pupil_n % cfg->n_subap != 0 || !(cfg->min_illum > 0) ||
      !(cfg->obstruction >= 0 && cfg->obstruction < 1))
    return fail(SHW_E_INVALID, "bad pupil geometry");
  std::vector<int32_t> idx;
  std::vector<double> il;
  valid_table(cfg, idx, il);
  *n_valid = (int32_t)idx.size();
  for (size_t k = 0; k < idx.size(); ++k) {
    if (valid_idx) valid_idx[k] = idx[k];
    if (illum) illum[k] = il[k];
  }
  return ok();
}

// Gaussian parameters (sigma along, sigma across in FFT pixels; axis angle) of one sub-aperture.
static void elongation(const shw_wfs_config* c, const shw_lgs_geom& g, int32_t sidx, double out[3]) {
  const int n = c->pupil_n / c->n_subap;
  const int sa = sidx / c->n_subap, sb = sidx % c->n_subap;
  const double xs = ((sb + 0.5) * n - c->pupil_n / 2.0) * c->pupil_dx_m;
  const double ys = ((sa + 0.5) * n - c->pupil_n / 2.0) * c->pupil_dx_m;
  const double dx = xs - g.launch_x_m, dy = ys - g.launch_y_m;
  const double d = std::hypot(dx, dy);
  const double diam = c->pupil_n * c->pupil_dx_m;
  const double el = c->elong_max_arcsec > 0 ? c->elong_max_arcsec * d / diam
                                            : d * c->na_fwhm_m / (c->na_height_m * c->na_height_m) / kArcsec;
  const double fwhm_par = std::sqrt(el * el + c->spot_fwhm_arcsec * c->spot_fwhm_arcsec);
  const double px_arcsec = c->wavelength_m / (c->fft_n * c->pupil_dx_m) / kArcsec;
  const double to_sigma = 1.0 / (2.0 * std::sqrt(2.0 * std::log(2.0)));
  out[0] = fwhm_par * to_sigma / px_arcsec;
  out[1] = c->spot_fwhm_arcsec * to_sigma / px_arcsec;
  out[2] = std::atan2(dy, dx);
}

// ---------------------------------------------------------------- MFMA constant tables

static uint16_t bf16_rne(float x) {
  uint32_t u;
  std::memcpy(&u, &x, 4);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
static float bf16_to_float(uint16_t b) {
  const uint32_t u = (uint32_t)b << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

// hi/lo halves of v for the precision: bf16 hi + bf16 residual, or fp16 hi + fp16 of 2^11 x residual.
static void split_const(double v, int prec, uint16_t* hi, uint16_t* lo) {
  if (prec == SHW_PREC_FP16X3) {
    // no subnormal high part: below the fp16 normal range the scaled low part carries the value
    const _Float16 h = std::fabs(v) < 6.103515625e-05 ? (_Float16)0.0 : (_Float16)v;
    const _Float16 l = (_Float16)((v - (double)h) * 2048.0);
    std::memcpy(hi, &h, 2);
    std::memcpy(lo, &l, 2);
  } else {
    const uint16_t h = bf16_rne((float)v);
    *hi = h;
    *lo = bf16_rne((float)(v - (double)bf16_to_float(h)));
  }
}

static std::vector<uint16_t> mfma_tables(const shw_wfs_config* c, int prec) {
  const double pi = 3.14159265358979323846;
  const int N = 40, n = 10, nb = 19;
  const double cc = (N - 1) / 2.0;
  auto band_k = [](int j) { return j <= 9 ? j : j - 19; };
  auto Wm = [&](int comp, int x, int u) -> double {  // W^T[x][u]
    if (x >= n || u >= N) return 0.0;
    const double th = 2.0 * pi * (u - cc) * x / N;
    return comp == 0 ? std::cos(th) : (comp == 1 ? -std::sin(th) : std::sin(th));
  };
  auto Dm = [&](int comp, int v, int j) -> double {  // D^T[v][j] = exp(-2 pi i k(j) v / N)
    if (v >= N || j >= nb) return 0.0;
    const double th = 2.0 * pi * (double)(((band_k(j) * v) % N + N) % N) / N;
    return comp == 0 ? std::cos(th) : (comp == 1 ? -std::sin(th) : std::sin(th));
  };
  const double b = (double)c->conv_n / c->det_n;
  auto Wb = [&](int p, int k) -> double {  // area overlap of input pixel k with detector pixel p
    const double lo = std::max((double)k, b * p), hi = std::min((double)(k + 1), b * (p + 1));
    return hi > lo ? hi - lo : 0.0;
  };
  // M^T[j][p] = (1/N) sum_v Wb[p][v] exp(2 pi i k(j) v / N), times c_j (rows j < 10 only) when folded
  auto Mm = [&](int comp, int j, int p, bool folded) -> double {
    if (j >= (folded ? 10 : nb) || p >= c->det_n) return 0.0;
    double s = 0.0;
    for (int v = 0; v < N; ++v) {
      const double w = Wb(p, v);
      if (w == 0.0) continue;
      const double th = 2.0 * pi * (double)(((band_k(j) * v) % N + N) % N) / N;
      s += w * (comp == 0 ? std::cos(th) : (comp == 1 ? std::sin(th) : -std::sin(th)));
    }
    const double cj = folded && j > 0 ? 2.0 : 1.0;
    return cj * s / N;
  };
  // tiles: part (0 hi, 1 lo) of tile `tile` for lane `lane` = 4 halves at ((tile * 2 + part) * 64 + lane) * 4
  std::vector<uint16_t> t((size_t)kMfmaTableTiles * 2 * 64 * 4, 0);
  auto put = [&](int tile, int lane, int r, double v) {
    uint16_t h, l;
    split_const(v, prec, &h, &l);
    t[(((size_t)tile * 2 + 0) * 64 + lane) * 4 + r] = h;
    t[(((size_t)tile * 2 + 1) * 64 + lane) * 4 + r] = l;
  };
  for (int lane = 0; lane < 64; ++lane)
    for (int r = 0; r < 4; ++r) {
      const int kr = 4 * (lane / 16) + r, nc = lane % 16;
      for (int tc = 0; tc < 3; ++tc) {
        put(kTabWr + tc, lane, r, Wm(0, kr, 16 * tc + nc));
        put(kTabWi + tc, lane, r, Wm(1, kr, 16 * tc + nc));
        put(kTabWiNeg + tc, lane, r, Wm(2, kr, 16 * tc + nc));
      }
      for (int tb = 0; tb < 3; ++tb)
        for (int tc = 0; tc < 2; ++tc) {
          put(kTabDr + 2 * tb + tc, lane, r, Dm(0, 16 * tb + kr, 16 * tc + nc));
          put(kTabDi + 2 * tb + tc, lane, r, Dm(1, 16 * tb + kr, 16 * tc + nc));
          put(kTabDiNeg + 2 * tb + tc, lane, r, Dm(2, 16 * tb + kr, 16 * tc + nc));
        }
      put(kTabMvr, lane, r, Mm(0, kr, nc, true));
      put(kTabMvi, lane, r, Mm(1, kr, nc, true));
      put(kTabMviNeg, lane, r, Mm(2, kr, nc, true));
      for (int tb = 0; tb < 2; ++tb) {
        put(kTabMur + tb, lane, r, Mm(0, 16 * tb + kr, nc, false));
        put(kTabMuiNeg + tb, lane, r, Mm(2, 16 * tb + kr, nc, false));
      }
    }
  // operands: (tile a, part pa) then (tile b, part pb), 8 halves per lane
  std::vector<uint16_t> o((size_t)kMfmaOps * 64 * 8, 0);
  auto op = [&](int idx, int a, int pa, int b, int pb) {
    for (int lane = 0; lane < 64; ++lane)
      for (int r = 0; r < 4; ++r) {
        o[((size_t)idx * 64 + lane) * 8 + r] = t[(((size_t)a * 2 + pa) * 64 + lane) * 4 + r];
        o[((size_t)idx * 64 + lane) * 8 + 4 + r] = t[(((size_t)b * 2 + pb) * 64 + lane) * 4 + r];
      }
  };
  // a complex pair [A|B]: hi operand then lo operand
  auto pair = [&](int idx, int a, int b) {
    op(idx, a, 0, b, 0);
    op(idx + 1, a, 1, b, 1);
  };
  for (int c = 0; c < 3; ++c) {
    pair(kOpW + 4 * c, kTabWr + c, kTabWiNeg + c);
    pair(kOpW + 4 * c + 2, kTabWi + c, kTabWr + c);
  }
  for (int tt = 0; tt < 6; ++tt) {
    pair(kOpD + 4 * tt, kTabDr + tt, kTabDiNeg + tt);
    pair(kOpD + 4 * tt + 2, kTabDi + tt, kTabDr + tt);
  }
  for (int tv = 0; tv < 3; ++tv) {
    op(kOpDre + tv, kTabDr + 2 * tv, 1, kTabDr + 2 * tv, 0);
    op(kOpDre + 3 + tv, kTabDi + 2 * tv, 1, kTabDi + 2 * tv, 0);
  }
  pair(kOpMv, kTabMvr, kTabMviNeg);
  pair(kOpMv + 2, kTabMvi, kTabMvr);
  for (int tb = 0; tb < 2; ++tb) pair(kOpMu + 2 * tb, kTabMur + tb, kTabMuiNeg + tb);
  return o;
}

// ---------------------------------------------------------------- plan

extern "C" int shw_wfs_plan_destroy(shw_wfs_plan* p) {
  if (!p) return ok();
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != p->device) (void)hipSetDevice(p->device);
  if (p->d_valid) (void)hipFree(p->d_valid);
  if (p->d_khat) (void)hipFree(p->d_khat);
  if (p->d_khat_band) (void)hipFree(p->d_khat_band);
  if (p->d_T) (void)hipFree(p->d_T);
  for (int k = 0; k < kListRing; ++k) {
    if (p->ring_pending[k]) (void)hipEventSynchronize(p->ring_ev[k]);  // uploads out of the host ring done
    if (p->ring_ev[k]) (void)hipEventDestroy(p->ring_ev[k]);
  }
  if (p->h_ring) (void)hipHostFree(p->h_ring);
  if (p->d_list) (void)hipFree(p->d_list);
  if (p->d_mfma_tab) (void)hipFree(p->d_mfma_tab);
  if (p->d_Jr) (void)hipFree(p->d_Jr);
  if (p->d_sub) (void)hipFree(p->d_sub);
  if (p->d_det_ws) (void)hipFree(p->d_det_ws);
  if (cur != p->device) (void)hipSetDevice(cur);
  delete p;
  return ok();
}

// Sodium sub-layer tables: phase coefficient and normalised weight per sub-layer, launcher
// positions in pupil pixels.  A point of the beam at height h seen from pupil point r has the
// wavefront of a point source at (L, h); against the focus at the layer height H this adds
// -|r - L|^2 / 2 (1/h - 1/H) metres of OPD (Sec. 4: tip-tilt and defocus per sub-layer).
static int sodium_tables(const shw_wfs_config* c, int32_t n_wfs, const shw_lgs_geom* geom, int32_t n_sub,
                         const double* dh_m, const double* weight, std::vector<double>& t) {
  if (!c->lgs) return fail(SHW_E_INVALID, "sodium sub-layers need an LGS configuration");
  if (n_sub < 1 || n_sub > 16) return fail(SHW_E_INVALID, "n_sub %d outside [1, 16]", n_sub);
  if (!dh_m || !weight) return fail(SHW_E_INVALID, "NULL sub-layer table");
  const double H = c->na_height_m;
  if (!(is_fin(H) && H > 0)) return fail(SHW_E_INVALID, "na_height_m must be > 0");
  double wsum = 0.0;
  for (int j = 0; j < n_sub; ++j) {
    if (!(is_fin(dh_m[j]) && H + dh_m[j] > 0)) return fail(SHW_E_INVALID, "sub-layer %d height not > 0", j);
    if (!(is_fin(weight[j]) && weight[j] >= 0)) return fail(SHW_E_INVALID, "sub-layer %d weight not >= 0", j);
    wsum += weight[j];
  }
  if (!(wsum > 0)) return fail(SHW_E_INVALID, "sub-layer weights sum to 0");
  const unsigned prec = (c->flags >> SHW_PRECISION_SHIFT) & 0xFu;
  const WfsShape shape{c->pupil_n / c->n_subap, c->fft_n, c->conv_n, c->det_n, c->lgs, 1};
  if (prec != SHW_PREC_FP32 || !wfs_shape_supported(shape))
    return fail(SHW_E_UNSUPPORTED, "no sodium sub-layer kernel for this shape and precision");
  const double dx = c->pupil_dx_m;
  t.assign((size_t)2 * (n_sub + n_wfs), 0.0);
  for (int j = 0; j < n_sub; ++j) {
    const double kappa = 1.0 / (H + dh_m[j]) - 1.0 / H;
    t[2 * j] = -dx * dx * kappa / c->wavelength_m;
    t[2 * j + 1] = weight[j] / wsum;
  }
  for (int w = 0; w < n_wfs; ++w) {
    t[2 * (n_sub + w)] = geom[w].launch_x_m / dx;
    t[2 * (n_sub + w) + 1] = geom[w].launch_y_m / dx;
  }
  return SHW_OK;
}

static int plan_create(const shw_wfs_config* cfg, int32_t n_wfs, const shw_lgs_geom* geom, int32_t n_sub,
                       const double* dh_m, const double* weight, shw_wfs_plan** out) {
  if (!out) return fail(SHW_E_INVALID, "out is NULL");
  *out = nullptr;
  int r = check_config(cfg, n_wfs, geom);
  if (r != SHW_OK) return r;
  std::vector<double> sub_tab;
  if (n_sub > 0) {
    r = sodium_tables(cfg, n_wfs, geom, n_sub, dh_m, weight, sub_tab);
    if (r != SHW_OK) return r;
  }
  auto* p = new shw_wfs_plan();
  p->cfg = *cfg;
  p->n_wfs = n_wfs;
  p->npx = cfg->pupil_n / cfg->n_subap;
  p->n_sub = n_sub;
  p->shape = WfsShape{p->npx, cfg->fft_n, cfg->conv_n, cfg->det_n, cfg->lgs, n_sub > 0 ? 1 : 0};
  std::vector<double> illum;
  valid_table(cfg, p->valid, illum);
  p->n_valid = (int32_t)p->valid.size();
  if (p->n_valid == 0) {
    delete p;
    return fail(SHW_E_INVALID, "no valid sub-aperture");
  }
  hipError_t e = hipGetDevice(&p->device);
  if (e != hipSuccess) {
    delete p;
    return hip_fail(e, "hipGetDevice");
  }
  // the valid table, then (shapes with calibration pairs) its inverse: -1 for the other sub-apertures
  std::vector<int32_t> tab = p->valid;
  if (wfs_shape_supported(p->shape) && wfs_modes_supported(p->shape, wfs_default_variant(p->shape, (int64_t)n_wfs * p->n_valid))) {
    tab.resize((size_t)p->n_valid + (size_t)cfg->n_subap * cfg->n_subap, -1);
    for (int32_t i = 0; i < p->n_valid; ++i) tab[(size_t)p->n_valid + p->valid[i]] = i;
  }
  e = hipMalloc(&p->d_valid, sizeof(int32_t) * tab.size());
  if (e == hipSuccess) e = hipMemcpy(p->d_valid, tab.data(), sizeof(int32_t) * tab.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    shw_wfs_plan_destroy(p);
    return hip_fail(e, "plan tables");
  }
  if (tab.size() > (size_t)p->n_valid) p->d_inv = p->d_valid + p->n_valid;
  p->bytes = sizeof(int32_t) * tab.size();
  if (n_sub > 0) {
    e = hipMalloc(&p->d_sub, sizeof(double) * sub_tab.size());
    if (e == hipSuccess)
      e = hipMemcpy(p->d_sub, sub_tab.data(), sizeof(double) * sub_tab.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
      shw_wfs_plan_destroy(p);
      return hip_fail(e, "sub-layer tables");
    }
    p->bytes += sizeof(double) * sub_tab.size();
  }
  p->prec = (int32_t)((cfg->flags >> SHW_PRECISION_SHIFT) & 0xFu);
  if (p->prec != SHW_PREC_FP32) {
    const std::vector<uint16_t> t = mfma_tables(cfg, p->prec);
    e = hipMalloc(&p->d_mfma_tab, t.size() * sizeof(uint16_t));
    if (e == hipSuccess) e = hipMemcpy(p->d_mfma_tab, t.data(), t.size() * sizeof(uint16_t), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
      shw_wfs_plan_destroy(p);
      return hip_fail(e, "MFMA tables");
    }
    p->bytes += t.size() * sizeof(uint16_t);
  }
  bool det_ws = p->prec != SHW_PREC_FP32;
  for (int v = 0; v < wfs_variant_count(p->shape); ++v) det_ws = det_ws || wfs_variant_needs_det_ws(p->shape, v);
  if (det_ws) {
    // the precision form hands its detector values to det_noise_kernel through this workspace too
    // one chunk holds a frame of every sensor, at least 16384 and at most 65536 items
    int64_t items = (int64_t)n_wfs * p->n_valid;
    items = items < 16384 ? 16384 : (items > 65536 ? 65536 : items);
    const size_t nb = sizeof(float) * (size_t)items * cfg->det_n * cfg->det_n;
    e = hipMalloc(&p->d_det_ws, nb);
    if (e != hipSuccess) {
      shw_wfs_plan_destroy(p);
      return hip_fail(e, "detector workspace");
    }
    p->det_ws_items = items;
    p->bytes += nb;
  }
  p->big = p->prec == SHW_PREC_FP32 && !wfs_shape_supported(p->shape);
  if (p->prec == SHW_PREC_FP32 && !p->big) p->variant = wfs_default_variant(p->shape, (int64_t)n_wfs * p->n_valid);
  if (p->big) {
    // about 128 MB of row intermediates per chunk, at least one sensor frame
    const int64_t per_item = (int64_t)p->npx * cfg->fft_n * (int64_t)sizeof(float2);
    int64_t chunk = ((int64_t)128 << 20) / per_item;
    if (chunk < 1) chunk = 1;
    if (chunk > (int64_t)n_wfs * p->n_valid * 16) chunk = (int64_t)n_wfs * p->n_valid * 16;
    p->chunk_items = chunk;
    e = hipMalloc(&p->d_T, (size_t)(chunk * per_item));
    if (e == hipSuccess) e = hipMalloc(&p->d_Jr, sizeof(float) * (size_t)chunk * cfg->det_n * cfg->fft_n);
    if (e != hipSuccess) {
      shw_wfs_plan_destroy(p);
      return hip_fail(e, "large sub-aperture workspace");
    }
    p->bytes += (size_t)(chunk * per_item) + sizeof(float) * (size_t)chunk * cfg->det_n * cfg->fft_n;
  }
  if (cfg->lgs) {
    const int64_t n = (int64_t)n_wfs * p->n_valid;
    const int H = cfg->conv_n / 2 + 1;
    std::vector<double> params((size_t)n * 3);
    for (int w = 0; w < n_wfs; ++w)
      for (int i = 0; i < p->n_valid; ++i) {
        double* q = &params[((size_t)w * p->n_valid + i) * 3];
        elongation(cfg, geom[w], p->valid[i], q);
        if (n_sub > 0) {  // the sub-layers make the elongation: the kernel is the round laser spot
          q[0] = q[1];
          q[2] = 0.0;
        }
      }
    double* d_params = nullptr;
    e = hipMalloc(&d_params, sizeof(double) * params.size());
    if (e == hipSuccess) e = hipMemcpy(d_params, params.data(), sizeof(double) * params.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMalloc(&p->d_khat, sizeof(float) * (size_t)n * H * cfg->conv_n);
    if (e == hipSuccess) e = launch_lgs_spectra(cfg->conv_n, d_params, n, p->d_khat, nullptr);
    // the band-limited variants and the MFMA form read only the in-band part of K^, kept as a compact copy
    const int npx = p->npx;
    const bool band = cfg->fft_n == cfg->conv_n && cfg->conv_n == 4 * npx;
    const size_t band_floats = band ? (size_t)n * npx * (2 * npx - 1) : 0;
    if (e == hipSuccess && band) e = hipMalloc(&p->d_khat_band, sizeof(float) * band_floats);
    if (e == hipSuccess && band) e = launch_khat_band(cfg->conv_n, npx, n, p->d_khat, p->d_khat_band, nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (d_params) (void)hipFree(d_params);
    if (e != hipSuccess) {
      shw_wfs_plan_destroy(p);
      return hip_fail(e, "kernel spectra");
    }
    p->bytes += sizeof(float) * ((size_t)n * H * cfg->conv_n + band_floats);
  }
  *out = p;
  return ok();
}

extern "C" int shw_wfs_plan_create(const shw_wfs_config* cfg, int32_t n_wfs, const shw_lgs_geom* geom,
                                   shw_wfs_plan** out) {
  return plan_create(cfg, n_wfs, geom, 0, nullptr, nullptr, out);
}

extern "C" int shw_wfs_plan_create_sodium(const shw_wfs_config* cfg, int32_t n_wfs, const shw_lgs_geom* geom,
                                          int32_t n_sub, const double* dh_m, const double* weight,
                                          shw_wfs_plan** out) {
  if (n_sub < 1) {
    if (out) *out = nullptr;
    return fail(SHW_E_INVALID, "n_sub %d < 1", n_sub);
  }
  return plan_create(cfg, n_wfs, geom, n_sub, dh_m, weight, out);
}

extern "C" int shw_wfs_plan_info(const shw_wfs_plan* p, int32_t* n_valid, size_t* device_bytes) {
  if (!p) return fail(SHW_E_INVALID, "plan is NULL");
  if (n_valid) *n_valid = p->n_valid;
  if (device_bytes) *device_bytes = p->bytes;
  return ok();
}

extern "C" int shw_wfs_plan_kernel_spectra(const shw_wfs_plan* p, int32_t wfs, float* d_out, void* stream) {
  if (!p || !d_out) return fail(SHW_E_INVALID, "NULL argument");
  if (!p->cfg.lgs) return fail(SHW_E_INVALID, "not an LGS plan");
  if (wfs < 0 || wfs >= p->n_wfs) return fail(SHW_E_INVALID, "wfs %d outside [0, %d)", wfs, p->n_wfs);
  const size_t per = (size_t)p->n_valid * (p->cfg.conv_n / 2 + 1) * p->cfg.conv_n;
  hipError_t e = hipMemcpyAsync(d_out, p->d_khat + per * wfs, per * sizeof(float), hipMemcpyDeviceToDevice,
                                (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "copy spectra");
  return ok();
}

// Fill the kernel arguments of one plan; the caller sets the per-call fields.
static WfsLaunch base_launch(const shw_wfs_plan* p) {
  const shw_wfs_config& c = p->cfg;
  WfsLaunch a{};
  a.valid_idx = p->d_valid;
  a.khat = p->d_khat;
  a.khat_band = p->d_khat_band;
  a.n_valid = p->n_valid;
  a.n_wfs = p->n_wfs;
  a.n_subap = c.n_subap;
  div_magic((uint32_t)(p->n_wfs * p->n_valid), &a.dm_frame_m, &a.dm_frame_s);
  div_magic((uint32_t)p->n_valid, &a.dm_valid_m, &a.dm_valid_s);
  div_magic((uint32_t)c.n_subap, &a.dm_subap_m, &a.dm_subap_s);
  a.inv_lambda = 1.0 / c.wavelength_m;
  const double h = c.pupil_n / 2.0;
  a.r2_outer = (float)(h * h);
  a.r2_inner = (float)((c.obstruction * h) * (c.obstruction * h));
  a.half_n = (float)h;
  a.ph_scale = c.photons_per_subap > 0 ? (float)(c.photons_per_subap / ((double)p->npx * p->npx)) : 0.0f;
  a.ron = (float)c.ron_e;
  a.thr = c.photons_per_subap > 0 ? (float)c.threshold_e : 0.0f;
  a.noise = (c.flags & SHW_FLAG_NOISE) && c.photons_per_subap > 0 ? 1 : 0;
  a.n_sub = p->n_sub;
  a.sub_coef = p->d_sub;
  a.launch_px = p->d_sub ? p->d_sub + 2 * p->n_sub : nullptr;
  a.det_ws = p->d_det_ws;
  a.det_ws_items = p->det_ws_items;
  a.noise_head = p->noise_head;
  return a;
}

// Large-sub-aperture passes for the items of a (chunks of the plan's workspace).
static int launch_big_list(shw_wfs_plan* p, const WfsLaunch& a, void* stream) {
  BigLaunch b{};
  b.opd = a.opd;
  b.row_pitch = a.row_pitch;
  b.wfs_stride = a.wfs_stride;
  b.frame_stride = a.frame_stride;
  b.valid_idx = a.valid_idx;
  b.slopes = a.slopes;
  b.images = a.images;
  b.flags = a.flags;
  b.n_valid = a.n_valid;
  b.n_wfs = a.n_wfs;
  b.n_subap = a.n_subap;
  b.npx = p->npx;
  b.det_n = p->cfg.det_n;
  b.inv_lambda = a.inv_lambda;
  b.r2_outer = a.r2_outer;
  b.r2_inner = a.r2_inner;
  b.half_n = a.half_n;
  b.ph_scale = a.ph_scale;
  b.ron = a.ron;
  b.thr = a.thr;
  b.noise = a.noise;
  b.key0 = a.key0;
  b.key1 = a.key1;
  b.frame0 = a.frame0;
  b.list = a.list;
  for (int64_t i0 = 0; i0 < a.total; i0 += p->chunk_items) {
    const int64_t n = a.total - i0 < p->chunk_items ? a.total - i0 : p->chunk_items;
    hipError_t e = launch_big(b, i0, n, p->d_T, p->d_Jr, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "large sub-aperture launch");
  }
  return ok();
}

// The plan's FP32 kernels for the items of a (images: some item wants its detector image).
static hipError_t launch_plan(const shw_wfs_plan* p, const WfsLaunch& a, bool images, hipStream_t st) {
  if (wfs_moments_supported(p->shape, a)) return launch_wfs_moments(p->shape, a, images, st);
  return launch_wfs_fused(p->shape, p->variant, a, st);
}

static int measure_impl(shw_wfs_plan* p, const float* d_opd_m, int64_t row_pitch, int64_t wfs_stride,
                        int64_t frame_stride, int32_t n_frames, uint64_t seed, uint64_t frame0,
                        const uint64_t* d_frame0, float* d_slopes, float* d_images, uint8_t* d_flags, void* stream,
                        int64_t sub_stride = 0) {
  if (!p) return fail(SHW_E_INVALID, "plan is NULL");
  if (n_frames < 0) return fail(SHW_E_INVALID, "n_frames %d < 0", n_frames);
  if (n_frames == 0) return ok();
  if (!d_opd_m || !d_slopes) return fail(SHW_E_INVALID, "NULL OPD or slope buffer");
  if (row_pitch < p->cfg.pupil_n) return fail(SHW_E_INVALID, "row_pitch %lld < pupil_n", (long long)row_pitch);
  if (wfs_stride < 0 || frame_stride < 0) return fail(SHW_E_INVALID, "negative stride");
  if (!d_frame0 && frame0 + (uint64_t)n_frames > (1ull << 32)) return fail(SHW_E_INVALID, "frame counter exceeds 2^32");
  if (d_frame0 && p->big) return fail(SHW_E_UNSUPPORTED, "device frame counter not available for FFT 512 plans");
  WfsLaunch a = base_launch(p);
  a.opd = d_opd_m;
  a.row_pitch = row_pitch;
  a.wfs_stride = wfs_stride;
  a.frame_stride = frame_stride;
  a.slopes = d_slopes;
  a.images = d_images;
  a.flags = d_flags;
  a.total = (int64_t)n_frames * p->n_wfs * p->n_valid;
  a.key0 = (uint32_t)(seed & 0xFFFFFFFFu);
  a.key1 = (uint32_t)(seed >> 32);
  a.frame0 = (uint32_t)frame0;
  a.frame0_dev = d_frame0;
  a.sub_stride = sub_stride;
  if (p->big) return launch_big_list(p, a, stream);
  if (p->prec != SHW_PREC_FP32) {
    if (d_frame0) return fail(SHW_E_UNSUPPORTED, "device frame counter not available for MFMA plans");
    hipError_t e = launch_wfs_mfma(p->prec, p->cfg.lgs != 0, a, p->d_mfma_tab, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "sh_wfs_measure launch");
    return ok();
  }
  hipError_t e = launch_plan(p, a, d_images != nullptr, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "sh_wfs_measure launch");
  return ok();
}

extern "C" int sh_wfs_measure_batch(const shw_work* items, int32_t n, void* stream) {
  if (n < 0) return fail(SHW_E_INVALID, "n %d < 0", n);
  if (n == 0) return ok();
  if (!items) return fail(SHW_E_INVALID, "items is NULL");
  for (int32_t k = 0; k < n; ++k) {
    const shw_work& w = items[k];
    if (!w.plan || !w.d_opd_m || !w.d_slopes) return fail(SHW_E_INVALID, "item %d has a NULL field", k);
    if (w.row_pitch < w.plan->cfg.pupil_n || w.wfs_stride < 0) return fail(SHW_E_INVALID, "item %d stride", k);
    if (w.frame >= (1ull << 32)) return fail(SHW_E_INVALID, "item %d frame exceeds 2^32", k);
  }
  // one launch per distinct plan, over a device work list of that plan's frames
  std::vector<shw_wfs_plan*> plans;
  for (int32_t k = 0; k < n; ++k) {
    bool seen = false;
    for (auto* q : plans) seen = seen || q == items[k].plan;
    if (!seen) plans.push_back(items[k].plan);
  }
  for (auto* p : plans)
    if (p->prec != SHW_PREC_FP32) return fail(SHW_E_UNSUPPORTED, "work lists need an FP32 plan");
  for (auto* p : plans) {
    std::vector<FrameWork> list;
    for (int32_t k = 0; k < n; ++k) {
      if (items[k].plan != p) continue;
      const shw_work& w = items[k];
      list.push_back(FrameWork{w.d_opd_m, w.row_pitch, w.wfs_stride, w.d_slopes, w.d_images, w.seed, w.frame});
    }
    const int32_t nf = (int32_t)list.size();
    if (nf > p->list_cap) {
      // grow the device list and the host ring: wait for what still uses them first
      hipError_t e = hipStreamSynchronize((hipStream_t)stream);
      for (int k = 0; e == hipSuccess && k < kListRing; ++k)
        if (p->ring_pending[k]) e = hipEventSynchronize(p->ring_ev[k]);
      if (e != hipSuccess) return hip_fail(e, "work list: wait before growing");
      for (int k = 0; k < kListRing; ++k) p->ring_pending[k] = false;
      if (p->d_list) (void)hipFree(p->d_list);
      if (p->h_ring) (void)hipHostFree(p->h_ring);
      p->d_list = nullptr;
      p->h_ring = nullptr;
      p->list_cap = 0;
      const int32_t cap = nf < 256 ? 256 : nf;
      e = hipMalloc(&p->d_list, sizeof(FrameWork) * cap);
      if (e == hipSuccess) e = hipHostMalloc((void**)&p->h_ring, sizeof(FrameWork) * (size_t)cap * kListRing);
      for (int k = 0; e == hipSuccess && k < kListRing; ++k)
        if (!p->ring_ev[k]) e = hipEventCreateWithFlags(&p->ring_ev[k], hipEventDisableTiming);
      if (e != hipSuccess) return hip_fail(e, "work list");
      p->list_cap = cap;
    }
    // stage the list in a pinned ring slot, so that the upload is asynchronous and the caller's
    // thread does not wait for earlier work on the stream; the slot is reused once its previous
    // upload has completed
    const int slot = p->ring_next;
    p->ring_next = (slot + 1) % kListRing;
    if (p->ring_pending[slot]) {
      hipError_t e = hipEventSynchronize(p->ring_ev[slot]);
      if (e != hipSuccess) return hip_fail(e, "work list: wait for a staging slot");
    }
    FrameWork* h = p->h_ring + (size_t)slot * p->list_cap;
    std::memcpy(h, list.data(), sizeof(FrameWork) * nf);
    hipError_t e = hipMemcpyAsync(p->d_list, h, sizeof(FrameWork) * nf, hipMemcpyHostToDevice, (hipStream_t)stream);
    if (e == hipSuccess) e = hipEventRecord(p->ring_ev[slot], (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "work list upload");
    p->ring_pending[slot] = true;
    WfsLaunch a = base_launch(p);
    a.list = p->d_list;
    a.total = (int64_t)nf * p->n_wfs * p->n_valid;
    if (p->big) {
      const int rc = launch_big_list(p, a, stream);
      if (rc != SHW_OK) return rc;
    } else {
      bool images = false;
      for (const FrameWork& w : list) images = images || w.images != nullptr;
      e = launch_plan(p, a, images, (hipStream_t)stream);
      if (e != hipSuccess) return hip_fail(e, "sh_wfs_measure_batch launch");
    }
  }
  return ok();
}

// ---------------------------------------------------------------- science PSF

struct shw_psf_plan {
  int32_t pupil_n = 0;
  int32_t fft_m = 0;
  double dx = 0, obstruction = 0, wavelength = 0;
  int64_t lit = 0;
  int device = 0;
  int32_t chunk = 0;          // frames per row/column pass pair
  float2* d_work = nullptr;   // chunk * pupil_n * fft_m complex
  size_t bytes = 0;
  double* d_ee_ws = nullptr;  // encircled-energy row-group sums
  size_t ee_bytes = 0;
};

extern "C" int shw_psf_plan_destroy(shw_psf_plan* p) {
  if (!p) return ok();
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != p->device) (void)hipSetDevice(p->device);
  if (p->d_work) (void)hipFree(p->d_work);
  if (p->d_ee_ws) (void)hipFree(p->d_ee_ws);
  if (cur != p->device) (void)hipSetDevice(cur);
  delete p;
  return ok();
}

extern "C" int shw_psf_plan_create(int32_t abi_version, int32_t pupil_n, double pupil_dx_m, double obstruction,
                                   int32_t fft_m, double wavelength_m, shw_psf_plan** out) {
  if (!out) return fail(SHW_E_INVALID, "out is NULL");
  *out = nullptr;
  if (abi_version != SHW_ABI_VERSION) return fail(SHW_E_ABI, "abi_version %d, library %d", abi_version, SHW_ABI_VERSION);
  if (pupil_n < 1 || pupil_n > 16384) return fail(SHW_E_INVALID, "pupil_n %d outside [1, 16384]", pupil_n);
  if (fft_m < pupil_n) return fail(SHW_E_INVALID, "fft_m %d < pupil_n %d", fft_m, pupil_n);
  if (!(is_fin(pupil_dx_m) && pupil_dx_m > 0)) return fail(SHW_E_INVALID, "pupil_dx_m must be > 0");
  if (!(is_fin(obstruction) && obstruction >= 0 && obstruction < 1))
    return fail(SHW_E_INVALID, "obstruction must be in [0, 1)");
  if (!(is_fin(wavelength_m) && wavelength_m > 0)) return fail(SHW_E_INVALID, "wavelength_m must be > 0");
  if (!psf_size_supported(fft_m, pupil_n))
    return fail(SHW_E_UNSUPPORTED, "no PSF kernel for fft_m %d with pupil_n %d (fft_m 1600, pupil_n <= 800)", fft_m,
                pupil_n);
  auto* p = new shw_psf_plan();
  p->pupil_n = pupil_n;
  p->fft_m = fft_m;
  p->dx = pupil_dx_m;
  p->obstruction = obstruction;
  p->wavelength = wavelength_m;
  shw_wfs_config c{};
  c.pupil_n = pupil_n;
  c.obstruction = obstruction;
  for (int r = 0; r < pupil_n; ++r)
    for (int col = 0; col < pupil_n; ++col) p->lit += lit(&c, r, col) ? 1 : 0;
  if (p->lit == 0) {
    delete p;
    return fail(SHW_E_INVALID, "pupil has no lit pixel");
  }
  hipError_t e = hipGetDevice(&p->device);
  if (e != hipSuccess) {
    delete p;
    return hip_fail(e, "hipGetDevice");
  }
  p->chunk = 8;
  const size_t work = (size_t)p->chunk * pupil_n * fft_m * sizeof(float2);
  e = hipMalloc(&p->d_work, work);
  if (e != hipSuccess) {
    shw_psf_plan_destroy(p);
    return hip_fail(e, "PSF workspace");
  }
  p->bytes = work;
  *out = p;
  return ok();
}

static int psf_impl(shw_psf_plan* p, const float* d_opd_m, int64_t row_pitch, int64_t frame_stride,
                    int64_t star_stride, int32_t n_frames, int32_t n_stars, float* d_psf_acc, int64_t acc_stride,
                    float* d_strehl, void* stream) {
  if (!p) return fail(SHW_E_INVALID, "plan is NULL");
  if (n_frames < 0 || n_stars < 0) return fail(SHW_E_INVALID, "negative frame or star count");
  if (n_frames == 0 || n_stars == 0) return ok();
  if (!d_opd_m || !d_psf_acc) return fail(SHW_E_INVALID, "NULL OPD or accumulator");
  if (row_pitch < p->pupil_n) return fail(SHW_E_INVALID, "row_pitch %lld < pupil_n", (long long)row_pitch);
  if (frame_stride < 0 || star_stride < 0) return fail(SHW_E_INVALID, "negative stride");
  if (n_stars > 1 && acc_stride < (int64_t)p->fft_m * p->fft_m) return fail(SHW_E_INVALID, "accumulators overlap");
  // grow the intermediate to hold every frame of every star (up to 4 GiB); otherwise run
  // frame chunks of all stars
  const int64_t per_frame = (int64_t)p->pupil_n * p->fft_m * (int64_t)sizeof(float2);
  const int64_t want = (int64_t)n_stars * n_frames;
  if (want > p->chunk && want * per_frame <= ((int64_t)4 << 30)) {
    float2* t = nullptr;
    hipError_t e = hipMalloc(&t, (size_t)(want * per_frame));
    if (e != hipSuccess) return hip_fail(e, "PSF workspace");
    // the old workspace may still be read by queued work on another stream: wait before freeing
    e = hipDeviceSynchronize();
    if (e != hipSuccess) {
      (void)hipFree(t);
      return hip_fail(e, "PSF workspace");
    }
    (void)hipFree(p->d_work);
    p->d_work = t;
    p->chunk = (int32_t)want;
    p->bytes = (size_t)(want * per_frame);
  }
  int32_t k = (int32_t)(p->chunk / n_stars);
  if (k < 1) return fail(SHW_E_NOMEM, "PSF workspace holds %d frames, %d stars", p->chunk, n_stars);
  PsfLaunch a{};
  a.opd = d_opd_m;
  a.row_pitch = row_pitch;
  a.frame_stride = frame_stride;
  a.star_stride = star_stride;
  a.acc_stride = acc_stride;
  a.n_frames = n_frames;
  a.pupil_n = p->pupil_n;
  a.inv_lambda = 1.0 / p->wavelength;
  const double h = p->pupil_n / 2.0;
  a.r2_outer = (float)(h * h);
  a.r2_inner = (float)((p->obstruction * h) * (p->obstruction * h));
  a.half_n = (float)h;
  a.inv_norm = (float)(1.0 / ((double)p->lit * (double)p->lit));
  for (int32_t f0 = 0; f0 < n_frames; f0 += k) {
    const int nf = n_frames - f0 < k ? n_frames - f0 : k;
    hipError_t e = launch_psf_rows(a, n_stars, f0, nf, p->d_work, (hipStream_t)stream);
    if (e == hipSuccess) e = launch_psf_cols(a, n_stars, f0, nf, p->d_work, d_psf_acc, d_strehl, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "psf launch");
  }
  return ok();
}

extern "C" int psf_accumulate(shw_psf_plan* p, const float* d_opd_m, int64_t row_pitch, int64_t frame_stride,
                              int32_t n_frames, float* d_psf_acc, float* d_strehl, void* stream) {
  return psf_impl(p, d_opd_m, row_pitch, frame_stride, 0, n_frames, 1, d_psf_acc, 0, d_strehl, stream);
}

extern "C" int psf_accumulate_stars(shw_psf_plan* p, const float* d_opd_m, int64_t row_pitch, int64_t frame_stride,
                                    int64_t star_stride, int32_t n_frames, int32_t n_stars, float* d_psf_acc,
                                    int64_t acc_stride, float* d_strehl, void* stream) {
  return psf_impl(p, d_opd_m, row_pitch, frame_stride, star_stride, n_frames, n_stars, d_psf_acc, acc_stride, d_strehl,
                  stream);
}

// ---------------------------------------------------------------- deformable mirrors, residual OPD

struct shw_dm_plan {
  int32_t size = 0, pitch = 0, m = 0, patch = 0, n_act = 0;
  double sigma = 0;
  int device = 0;
  std::vector<double> act;   // [n_act][2] (x, y)
  int* d_grid = nullptr;
  float* d_act_xy = nullptr;  // [n_act][2] FP32 device copy (influence-function frames)
};

// Metapupil radius, surface side and actuator grid (host, FP64).
static int dm_geometry(int32_t pupil_n, double dx, double alt_m, int32_t pitch_px, double field_arcsec, double* R,
                       int* size, int* m, std::vector<int>* grid, std::vector<double>* act) {
  if (pupil_n < 2 || pupil_n > 16384 || pupil_n % 2) return fail(SHW_E_INVALID, "pupil_n %d must be even in [2, 16384]", pupil_n);
  if (!(is_fin(dx) && dx > 0)) return fail(SHW_E_INVALID, "pupil_dx_m must be > 0");
  if (!(is_fin(alt_m) && alt_m >= 0)) return fail(SHW_E_INVALID, "alt_m must be >= 0");
  if (pitch_px < 1 || pitch_px > 4096) return fail(SHW_E_INVALID, "pitch_px %d outside [1, 4096]", pitch_px);
  if (!(is_fin(field_arcsec) && field_arcsec >= 0)) return fail(SHW_E_INVALID, "field radius must be >= 0");
  *R = pupil_n / 2.0 + alt_m * field_arcsec * kArcsec / dx;
  *size = 2 * (int)std::ceil(*R - 1e-9);
  if (*size > 65536) return fail(SHW_E_INVALID, "surface too large (%d)", *size);
  *m = (int)std::floor(*R / pitch_px);
  const int G = 2 * *m + 1;
  grid->assign((size_t)G * G, -1);
  act->clear();
  int n = 0;
  for (int gy = -*m; gy <= *m; ++gy)
    for (int gx = -*m; gx <= *m; ++gx) {
      const double x = (double)gx * pitch_px, y = (double)gy * pitch_px;
      if (x * x + y * y <= *R * *R) {
        (*grid)[(size_t)(gy + *m) * G + (gx + *m)] = n++;
        act->push_back(x);
        act->push_back(y);
      }
    }
  return SHW_OK;
}

extern "C" int shw_dm_geometry(int32_t pupil_n, double pupil_dx_m, double alt_m, int32_t pitch_px,
                               double field_radius_arcsec, int32_t* n_act, int32_t* size, double* act_xy) {
  double R;
  int sz, m;
  std::vector<int> grid;
  std::vector<double> act;
  const int r = dm_geometry(pupil_n, pupil_dx_m, alt_m, pitch_px, field_radius_arcsec, &R, &sz, &m, &grid, &act);
  if (r != SHW_OK) return r;
  if (n_act) *n_act = (int32_t)(act.size() / 2);
  if (size) *size = sz;
  if (act_xy)
    for (size_t k = 0; k < act.size(); ++k) act_xy[k] = act[k];
  return ok();
}

extern "C" int shw_dm_plan_destroy(shw_dm_plan* p) {
  if (!p) return ok();
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != p->device) (void)hipSetDevice(p->device);
  if (p->d_grid) (void)hipFree(p->d_grid);
  if (p->d_act_xy) (void)hipFree(p->d_act_xy);
  if (cur != p->device) (void)hipSetDevice(cur);
  delete p;
  return ok();
}

extern "C" int shw_dm_plan_create(int32_t abi_version, int32_t pupil_n, double pupil_dx_m, double alt_m,
                                  int32_t pitch_px, double field_radius_arcsec, double coupling, int32_t patch,
                                  shw_dm_plan** out) {
  if (!out) return fail(SHW_E_INVALID, "out is NULL");
  *out = nullptr;
  if (abi_version != SHW_ABI_VERSION) return fail(SHW_E_ABI, "abi_version %d, library %d", abi_version, SHW_ABI_VERSION);
  if (!(is_fin(coupling) && coupling > 0 && coupling < 1)) return fail(SHW_E_INVALID, "coupling must be in (0, 1)");
  if (patch < 2 || patch > 1024 || patch % 2) return fail(SHW_E_INVALID, "patch %d must be even in [2, 1024]", patch);
  double R;
  int size, m;
  std::vector<int> grid;
  std::vector<double> act;
  const int r = dm_geometry(pupil_n, pupil_dx_m, alt_m, pitch_px, field_radius_arcsec, &R, &size, &m, &grid, &act);
  if (r != SHW_OK) return r;
  auto* p = new shw_dm_plan();
  p->size = size;
  p->pitch = pitch_px;
  p->patch = patch;
  p->m = m;
  p->sigma = pitch_px / std::sqrt(2.0 * std::log(1.0 / coupling));
  p->act = act;
  p->n_act = (int32_t)(act.size() / 2);
  std::vector<float> axy(act.begin(), act.end());
  hipError_t e = hipGetDevice(&p->device);
  if (e == hipSuccess) e = hipMalloc(&p->d_grid, sizeof(int) * grid.size());
  if (e == hipSuccess) e = hipMemcpy(p->d_grid, grid.data(), sizeof(int) * grid.size(), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMalloc(&p->d_act_xy, sizeof(float) * (axy.empty() ? 1 : axy.size()));
  if (e == hipSuccess && !axy.empty())
    e = hipMemcpy(p->d_act_xy, axy.data(), sizeof(float) * axy.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    shw_dm_plan_destroy(p);
    return hip_fail(e, "DM plan tables");
  }
  *out = p;
  return ok();
}

extern "C" int shw_dm_plan_info(const shw_dm_plan* p, int32_t* n_act, int32_t* size, double* act_xy) {
  if (!p) return fail(SHW_E_INVALID, "plan is NULL");
  if (n_act) *n_act = p->n_act;
  if (size) *size = p->size;
  if (act_xy)
    for (size_t k = 0; k < p->act.size(); ++k) act_xy[k] = p->act[k];
  return ok();
}

extern "C" int shw_dm_surface(shw_dm_plan* p, const float* d_coefs, float* d_surface, void* stream) {
  if (!p || !d_coefs || !d_surface) return fail(SHW_E_INVALID, "NULL argument");
  DmLaunch a{};
  a.grid = p->d_grid;
  a.m = p->m;
  a.pitch = p->pitch;
  a.size = p->size;
  a.half_patch = p->patch / 2;
  a.inv_2s2 = (float)(1.0 / (2.0 * p->sigma * p->sigma));
  hipError_t e = launch_dm_surface(a, d_coefs, d_surface, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "shw_dm_surface launch");
  return ok();
}

extern "C" int shw_residual_opd(const float* d_screen, int32_t screen_rows, int32_t screen_cols, int64_t screen_pitch,
                                int32_t n_dm, const float* const* d_surf, const int32_t* surf_size, int32_t pupil_n,
                                int32_t n_out, const int32_t* scr_origin, const int32_t* dm_origin, float* d_out,
                                int64_t out_pitch, int64_t out_stride, void* stream) {
  if (n_out < 0) return fail(SHW_E_INVALID, "n_out < 0");
  if (n_out == 0) return ok();
  if (!d_screen || !d_out || !scr_origin) return fail(SHW_E_INVALID, "NULL argument");
  if (n_dm < 0 || n_dm > kMaxDm) return fail(SHW_E_INVALID, "n_dm %d outside [0, %d]", n_dm, kMaxDm);
  if (n_dm > 0 && (!d_surf || !surf_size || !dm_origin)) return fail(SHW_E_INVALID, "NULL DM argument");
  if (pupil_n < 1 || screen_rows < 1 || screen_cols < 1 || screen_pitch < screen_cols)
    return fail(SHW_E_INVALID, "bad screen or pupil size");
  if (out_pitch < pupil_n || out_stride < 0) return fail(SHW_E_INVALID, "bad output layout");
  for (int d = 0; d < n_dm; ++d)
    if (!d_surf[d] || surf_size[d] < pupil_n) return fail(SHW_E_INVALID, "surface %d missing or smaller than the pupil", d);
  for (int k = 0; k < n_out; ++k) {
    const int r = scr_origin[2 * k], c = scr_origin[2 * k + 1];
    if (r < 0 || c < 0 || r + pupil_n > screen_rows || c + pupil_n > screen_cols)
      return fail(SHW_E_INVALID, "screen window %d at (%d, %d) leaves the screen", k, r, c);
    for (int d = 0; d < n_dm; ++d) {
      const int rr = dm_origin[(k * n_dm + d) * 2], cc = dm_origin[(k * n_dm + d) * 2 + 1];
      if (rr < 0 || cc < 0 || rr + pupil_n > surf_size[d] || cc + pupil_n > surf_size[d])
        return fail(SHW_E_INVALID, "DM %d window %d at (%d, %d) leaves the surface", d, k, rr, cc);
    }
  }
  ResidualLaunch a{};
  a.screen = d_screen;
  a.screen_pitch = screen_pitch;
  a.pupil_n = pupil_n;
  a.out_pitch = out_pitch;
  a.out_stride = out_stride;
  for (int d = 0; d < n_dm; ++d) {
    a.surf[d] = d_surf[d];
    a.surf_size[d] = surf_size[d];
  }
  // outputs with the same mirror windows next to each other (the kernel then reads the mirrors
  // once for a run of them), in groups of a bounded size, so that nothing here throws
  constexpr int kGroup = 1024;
  ResidualOut outs[kGroup];
  for (int64_t g0 = 0; g0 < n_out; g0 += kGroup) {
    const int ng = n_out - g0 < kGroup ? (int)(n_out - g0) : kGroup;
    for (int i = 0; i < ng; ++i) {
      const int64_t k = g0 + i;
      ResidualOut& o = outs[i];
      o = ResidualOut{};
      o.scr_off = (int64_t)scr_origin[2 * k] * screen_pitch + scr_origin[2 * k + 1];
      o.out = k;
      for (int d = 0; d < n_dm; ++d) {
        const int32_t* w = dm_origin + (k * n_dm + d) * 2;
        o.dm_off[d] = (int64_t)w[0] * surf_size[d] + w[1];
      }
    }
    std::stable_sort(outs, outs + ng, [](const ResidualOut& u, const ResidualOut& v) {
      for (int d = 0; d < kMaxDm; ++d)
        if (u.dm_off[d] != v.dm_off[d]) return u.dm_off[d] < v.dm_off[d];
      return false;
    });
    // launches of equal size
    const int launches = (ng + kResidualChunk - 1) / kResidualChunk;
    for (int i = 0; i < launches; ++i) {
      const int k0 = ng * i / launches, k1 = ng * (i + 1) / launches;
      a.n_out = k1 - k0;
      std::copy(outs + k0, outs + k1, a.o);
      hipError_t e = launch_residual(a, n_dm, d_out, (hipStream_t)stream);
      if (e != hipSuccess) return hip_fail(e, "shw_residual_opd launch");
    }
  }
  return ok();
}

extern "C" int sh_wfs_measure(shw_wfs_plan* p, const float* d_opd_m, int64_t row_pitch, int64_t wfs_stride,
                              int64_t frame_stride, int32_t n_frames, uint64_t seed, uint64_t frame0,
                              float* d_slopes, float* d_images, uint8_t* d_flags, void* stream) {
  return measure_impl(p, d_opd_m, row_pitch, wfs_stride, frame_stride, n_frames, seed, frame0, nullptr, d_slopes,
                      d_images, d_flags, stream);
}

extern "C" int sh_wfs_measure_sodium(shw_wfs_plan* p, const float* d_opd_m, int64_t row_pitch, int64_t sub_stride,
                                     int64_t wfs_stride, int64_t frame_stride, int32_t n_frames, uint64_t seed,
                                     uint64_t frame0, float* d_slopes, float* d_images, uint8_t* d_flags,
                                     void* stream) {
  if (!p) return fail(SHW_E_INVALID, "plan is NULL");
  if (p->n_sub < 1) return fail(SHW_E_INVALID, "plan has no sodium sub-layers");
  if (sub_stride < 0) return fail(SHW_E_INVALID, "negative sub-layer stride");
  return measure_impl(p, d_opd_m, row_pitch, wfs_stride, frame_stride, n_frames, seed, frame0, nullptr, d_slopes,
                      d_images, d_flags, stream, sub_stride);
}

extern "C" int sh_wfs_measure_devframe(shw_wfs_plan* p, const float* d_opd_m, int64_t row_pitch, int64_t wfs_stride,
                                       int64_t frame_stride, int32_t n_frames, uint64_t seed, const uint64_t* d_frame0,
                                       float* d_slopes, float* d_images, uint8_t* d_flags, void* stream) {
  if (!d_frame0) return fail(SHW_E_INVALID, "d_frame0 is NULL");
  return measure_impl(p, d_opd_m, row_pitch, wfs_stride, frame_stride, n_frames, seed, 0, d_frame0, d_slopes,
                      d_images, d_flags, stream);
}

extern "C" int sh_wfs_measure_devframe_at(shw_wfs_plan* p, const float* d_opd_m, int64_t row_pitch,
                                          int64_t wfs_stride, int64_t frame_stride, int32_t n_frames, uint64_t seed,
                                          const uint64_t* d_frame0, uint32_t frame_offset, float* d_slopes,
                                          float* d_images, uint8_t* d_flags, void* stream) {
  if (!d_frame0) return fail(SHW_E_INVALID, "d_frame0 is NULL");
  return measure_impl(p, d_opd_m, row_pitch, wfs_stride, frame_stride, n_frames, seed, frame_offset, d_frame0,
                      d_slopes, d_images, d_flags, stream);
}

// ---------------------------------------------------------------- variants, autotuning

extern "C" int shw_wfs_plan_variant_count(const shw_wfs_plan* p, int32_t* n) {
  if (!p || !n) return fail(SHW_E_INVALID, "NULL argument");
  *n = p->big ? 1 : wfs_variant_count(p->shape);
  return ok();
}

extern "C" int shw_wfs_plan_get_variant(const shw_wfs_plan* p, int32_t* variant) {
  if (!p || !variant) return fail(SHW_E_INVALID, "NULL argument");
  *variant = p->variant;
  return ok();
}

extern "C" int shw_wfs_plan_set_variant(shw_wfs_plan* p, int32_t v) {
  if (!p) return fail(SHW_E_INVALID, "plan is NULL");
  const int n = p->big ? 1 : wfs_variant_count(p->shape);
  if (v < 0 || v >= n) return fail(SHW_E_INVALID, "variant %d outside [0, %d)", v, n);
  p->variant = v;
  return ok();
}

extern "C" int shw_wfs_plan_variant_params(const shw_wfs_plan* p, int32_t v, int32_t* params) {
  if (!p || !params) return fail(SHW_E_INVALID, "NULL argument");
  if (p->big || p->prec != SHW_PREC_FP32) return fail(SHW_E_UNSUPPORTED, "no launch variants for this plan");
  if (!wfs_variant_params(p->shape, v, params)) return fail(SHW_E_INVALID, "variant %d out of range", v);
  return ok();
}

extern "C" int shw_wfs_plan_set_noise_head(shw_wfs_plan* p, int32_t head) {
  if (!p) return fail(SHW_E_INVALID, "plan is NULL");
  if (head != 2 && head != 4 && head != 6) return fail(SHW_E_INVALID, "noise head %d not in {2, 4, 6}", head);
  p->noise_head = head;
  return ok();
}

extern "C" int shw_wfs_plan_get_noise_head(const shw_wfs_plan* p, int32_t* head) {
  if (!p || !head) return fail(SHW_E_INVALID, "NULL argument");
  *head = p->noise_head;
  return ok();
}

extern "C" int shw_wfs_plan_autotune(shw_wfs_plan* p, const float* d_opd_m, int64_t row_pitch, int64_t wfs_stride,
                                     int64_t frame_stride, int32_t n_frames, float* d_slopes, int32_t reps,
                                     void* stream, int32_t* best, float* ms) {
  if (!p || !best) return fail(SHW_E_INVALID, "NULL argument");
  if (n_frames < 1 || reps < 1 || reps > 100000) return fail(SHW_E_INVALID, "n_frames >= 1 and reps in [1, 1e5]");
  const int n = p->big ? 1 : wfs_variant_count(p->shape);
  const int32_t keep = p->variant;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  if (e != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    return hip_fail(e, "autotune events");
  }
  float best_ms = 0.0f;
  int32_t best_v = 0;
  const int32_t def_v = p->big ? 0 : wfs_default_variant(p->shape, (int64_t)p->n_wfs * p->n_valid);
  float def_ms = -1.0f;
  int rc = SHW_OK;
  for (int v = 0; v < n && rc == SHW_OK; ++v) {
    p->variant = v;
    for (int k = 0; k < 2 + reps && rc == SHW_OK; ++k) {
      if (k == 2) e = hipEventRecord(e0, (hipStream_t)stream);
      if (e != hipSuccess) break;
      rc = sh_wfs_measure(p, d_opd_m, row_pitch, wfs_stride, frame_stride, n_frames, 0, 0, d_slopes, nullptr,
                          nullptr, stream);
    }
    if (rc != SHW_OK) break;
    if (e == hipSuccess) e = hipEventRecord(e1, (hipStream_t)stream);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float t = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&t, e0, e1);
    if (e != hipSuccess) break;
    t /= (float)reps;
    if (ms) ms[v] = t;
    if (v == def_v) def_ms = t;
    if (v == 0 || t < best_ms) {
      best_ms = t;
      best_v = v;
    }
  }
  // launch times vary by a few per cent from run to run: within 2 % of the fastest the plan's default
  // is kept (for the band-limited shapes the form with the least HBM traffic)
  if (def_ms >= 0.0f && def_ms <= 1.02f * best_ms) best_v = def_v;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != SHW_OK) {
    p->variant = keep;
    return rc;
  }
  if (e != hipSuccess) {
    p->variant = keep;
    return hip_fail(e, "autotune timing");
  }
  p->variant = best_v;
  *best = best_v;
  return ok();
}

extern "C" int shw_wfs_plan_autotune_noise_head(shw_wfs_plan* p, const float* d_opd_m, int64_t row_pitch,
                                                int64_t wfs_stride, int64_t frame_stride, int32_t n_frames,
                                                float* d_slopes, int32_t reps, void* stream, int32_t* best,
                                                float* ms) {
  if (!p || !best) return fail(SHW_E_INVALID, "NULL argument");
  if (n_frames < 1 || reps < 1 || reps > 100000) return fail(SHW_E_INVALID, "n_frames >= 1 and reps in [1, 1e5]");
  static const int32_t kHeads[3] = {2, 4, 6};
  const int32_t keep = p->noise_head;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  hipError_t e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  if (e != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    return hip_fail(e, "autotune events");
  }
  float best_ms = 0.0f;
  int32_t best_h = keep;
  int rc = SHW_OK;
  for (int h = 0; h < 3 && rc == SHW_OK && e == hipSuccess; ++h) {
    p->noise_head = kHeads[h];
    for (int k = 0; k < 2 + reps && rc == SHW_OK; ++k) {
      if (k == 2) e = hipEventRecord(e0, (hipStream_t)stream);
      if (e != hipSuccess) break;
      rc = sh_wfs_measure(p, d_opd_m, row_pitch, wfs_stride, frame_stride, n_frames, 0, 0, d_slopes, nullptr,
                          nullptr, stream);
    }
    if (rc != SHW_OK || e != hipSuccess) break;
    e = hipEventRecord(e1, (hipStream_t)stream);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float t = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&t, e0, e1);
    if (e != hipSuccess) break;
    t /= (float)reps;
    if (ms) ms[h] = t;
    if (h == 0 || t < best_ms) {
      best_ms = t;
      best_h = kHeads[h];
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != SHW_OK) {
    p->noise_head = keep;
    return rc;
  }
  if (e != hipSuccess) {
    p->noise_head = keep;
    return hip_fail(e, "autotune timing");
  }
  p->noise_head = best_h;
  *best = best_h;
  return ok();
}

// ---------------------------------------------------------------- graphs, device counters

struct shw_graph {
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

extern "C" int shw_counter_add(uint64_t* d_counter, uint64_t inc, void* stream) {
  if (!d_counter) return fail(SHW_E_INVALID, "d_counter is NULL");
  hipError_t e = launch_counter_add(d_counter, inc, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "shw_counter_add launch");
  return ok();
}

extern "C" int shw_graph_begin(void* stream) {
  if (!stream) return fail(SHW_E_INVALID, "graph capture needs a non-NULL stream");
  hipError_t e = hipStreamBeginCapture((hipStream_t)stream, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) return hip_fail(e, "hipStreamBeginCapture");
  return ok();
}

extern "C" int shw_graph_end(void* stream, shw_graph** out) {
  if (!stream || !out) return fail(SHW_E_INVALID, "NULL argument");
  *out = nullptr;
  auto* g = new shw_graph();
  hipError_t e = hipStreamEndCapture((hipStream_t)stream, &g->graph);
  if (e == hipSuccess) e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    if (g->graph) (void)hipGraphDestroy(g->graph);
    delete g;
    return hip_fail(e, "graph capture");
  }
  *out = g;
  return ok();
}

extern "C" int shw_graph_launch(shw_graph* g, void* stream) {
  if (!g) return fail(SHW_E_INVALID, "graph is NULL");
  hipError_t e = hipGraphLaunch(g->exec, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "hipGraphLaunch");
  return ok();
}

extern "C" int shw_graph_destroy(shw_graph* g) {
  if (!g) return ok();
  if (g->exec) (void)hipGraphExecDestroy(g->exec);
  if (g->graph) (void)hipGraphDestroy(g->graph);
  delete g;
  return ok();
}

// ---------------------------------------------------------------- push-pull calibration

extern "C" int shw_dm_influence_opd(const shw_dm_plan* p, const int32_t* d_act, const float* d_amp, int32_t n,
                                    int32_t row0, int32_t col0, int32_t pupil_n, float* d_out, int64_t out_pitch,
                                    int64_t out_stride, void* stream) {
  if (!p) return fail(SHW_E_INVALID, "plan is NULL");
  if (n < 0 || n > 65535) return fail(SHW_E_INVALID, "n = %d outside [0, 65535]", n);
  if (n == 0) return ok();
  if (!d_act || !d_amp || !d_out) return fail(SHW_E_INVALID, "NULL argument");
  if (pupil_n < 1 || row0 < 0 || col0 < 0 || row0 + pupil_n > p->size || col0 + pupil_n > p->size)
    return fail(SHW_E_INVALID, "pupil window (%d, %d) + %d leaves the %d-pixel surface", row0, col0, pupil_n, p->size);
  if (out_pitch < pupil_n || out_stride < 0) return fail(SHW_E_INVALID, "bad output layout");
  InfluenceLaunch a{};
  a.act_xy = p->d_act_xy;
  a.act = d_act;
  a.amp = d_amp;
  a.n = n;
  a.n_act = p->n_act;
  a.size = p->size;
  a.half_patch = p->patch / 2;
  a.row0 = row0;
  a.col0 = col0;
  a.pupil_n = pupil_n;
  a.inv_2s2 = (float)(1.0 / (2.0 * p->sigma * p->sigma));
  a.out_pitch = out_pitch;
  a.out_stride = out_stride;
  hipError_t e = launch_influence_opd(a, d_out, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "shw_dm_influence_opd launch");
  return ok();
}

extern "C" int shw_wfs_interaction_matrix(shw_wfs_plan* p, const shw_dm_plan* dm, const int32_t* acts, int32_t n_modes,
                                          float amplitude_m, int32_t row0, int32_t col0, float scale, float* d_im,
                                          int64_t ld_im, void* stream) {
  if (!p || !dm) return fail(SHW_E_INVALID, "plan is NULL");
  if (n_modes < 0) return fail(SHW_E_INVALID, "n_modes %d < 0", n_modes);
  if (n_modes == 0) return ok();
  if (!acts || !d_im) return fail(SHW_E_INVALID, "NULL argument");
  const int32_t n = p->cfg.pupil_n;
  if (row0 < 0 || col0 < 0 || row0 + (int64_t)n > dm->size || col0 + (int64_t)n > dm->size)
    return fail(SHW_E_INVALID, "pupil window (%d, %d) + %d leaves the %d-pixel surface", row0, col0, n, dm->size);
  if (ld_im < n_modes) return fail(SHW_E_INVALID, "ld_im %lld < n_modes %d", (long long)ld_im, n_modes);
  // noise is drawn for every sub-aperture of every frame, so only noise-free pushes leave the
  // untouched ones exactly alike
  if ((p->cfg.flags & SHW_FLAG_NOISE) || p->prec != SHW_PREC_FP32 || p->big || !p->d_inv ||
      !wfs_modes_supported(p->shape, p->variant))
    return fail(SHW_E_UNSUPPORTED, "no calibration kernel for this plan and launch variant");
  const int32_t nb = (dm->patch - 1) / p->npx + 2;
  const int64_t per_mode = (int64_t)p->n_wfs * nb * nb;
  // pairs per launch: 80 lanes each, and a launch has fewer than 2^32
  constexpr int64_t kMaxPairs = (int64_t)1 << 25;
  if (nb >= p->cfg.n_subap || per_mode > kMaxPairs)
    return fail(SHW_E_UNSUPPORTED, "an influence function reaches the whole pupil");
  ModesLaunch q{};
  q.a = base_launch(p);
  q.act_xy = dm->d_act_xy;
  q.inv = p->d_inv;
  q.ld = ld_im;
  q.n_act = dm->n_act;
  q.half = dm->size / 2;
  q.half_patch = dm->patch / 2;
  q.row0 = row0;
  q.col0 = col0;
  q.npx = p->npx;
  q.nb = nb;
  q.shift = (dm->size + dm->patch) / p->npx + 1;
  div_magic((uint32_t)per_mode, &q.dm_mode_m, &q.dm_mode_s);
  div_magic((uint32_t)(nb * nb), &q.dm_cell_m, &q.dm_cell_s);
  div_magic((uint32_t)nb, &q.dm_nb_m, &q.dm_nb_s);
  q.amp = amplitude_m;
  q.inv_2s2 = (float)(1.0 / (2.0 * dm->sigma * dm->sigma));
  q.scale = scale;
  hipStream_t st = (hipStream_t)stream;
  // the difference of equal slopes times the scale (0 for any finite scale)
  hipError_t e = launch_fill_matrix(d_im, (int64_t)p->n_wfs * 2 * p->n_valid, n_modes, ld_im, 0.0f * scale, st);
  const int64_t fit = kMaxPairs / per_mode;
  const int32_t chunk = fit < kModesChunk ? (int32_t)fit : kModesChunk;
  for (int32_t m0 = 0; m0 < n_modes && e == hipSuccess; m0 += chunk) {
    q.n_modes = n_modes - m0 < chunk ? n_modes - m0 : chunk;
    q.a.total = 2 * (int64_t)q.n_modes * per_mode;
    std::copy(acts + m0, acts + m0 + q.n_modes, q.act);
    q.im = d_im + m0;
    e = launch_wfs_modes(p->shape, q, st);
  }
  if (e != hipSuccess) return hip_fail(e, "shw_wfs_interaction_matrix launch");
  return ok();
}

extern "C" int shw_push_pull(const float* d_slopes, int32_t n_modes, int32_t n_slopes, float scale, float* d_im,
                             int64_t ld_im, void* stream) {
  if (n_modes < 0 || n_slopes < 0) return fail(SHW_E_INVALID, "negative size");
  if (n_modes == 0 || n_slopes == 0) return ok();
  if (!d_slopes || !d_im) return fail(SHW_E_INVALID, "NULL argument");
  if (ld_im < n_modes) return fail(SHW_E_INVALID, "ld_im %lld < n_modes %d", (long long)ld_im, n_modes);
  if ((n_modes + 31) / 32 > 65535) return fail(SHW_E_INVALID, "n_modes %d too large", n_modes);
  hipError_t e = launch_push_pull(d_slopes, n_modes, n_slopes, scale, d_im, ld_im, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "shw_push_pull launch");
  return ok();
}

// ---------------------------------------------------------------- closed-loop reconstructor

struct shw_recon_plan {
  int32_t n_modes = 0, n_slopes = 0, n_chunks = 0;
  int device = 0;
  float* d_partial = nullptr;  // [n_chunks][n_modes]
};

extern "C" int shw_recon_plan_create(int32_t n_modes, int32_t n_slopes, shw_recon_plan** out) {
  if (!out) return fail(SHW_E_INVALID, "out is NULL");
  *out = nullptr;
  if (n_modes < 1 || n_modes > (1 << 22)) return fail(SHW_E_INVALID, "n_modes %d outside [1, 2^22]", n_modes);
  if (n_slopes < 1) return fail(SHW_E_INVALID, "n_slopes %d < 1", n_slopes);
  auto* p = new shw_recon_plan();
  p->n_modes = n_modes;
  p->n_slopes = n_slopes;
  p->n_chunks = recon_chunks(n_slopes);
  hipError_t e = hipGetDevice(&p->device);
  if (e == hipSuccess) e = hipMalloc(&p->d_partial, sizeof(float) * (size_t)p->n_chunks * n_modes);
  if (e != hipSuccess) {
    delete p;
    return hip_fail(e, "reconstructor workspace");
  }
  *out = p;
  return ok();
}

extern "C" int shw_recon_step(shw_recon_plan* p, const float* d_cm, int64_t ld_cm, const float* d_slopes, float gain,
                              float* d_coefs, float* d_delta, void* stream) {
  if (!p) return fail(SHW_E_INVALID, "plan is NULL");
  if (!d_cm || !d_slopes || !d_coefs) return fail(SHW_E_INVALID, "NULL argument");
  if (ld_cm < p->n_slopes || ld_cm % 4 != 0)
    return fail(SHW_E_INVALID, "ld_cm %lld must be >= n_slopes %d and a multiple of 4", (long long)ld_cm,
                p->n_slopes);
  if (reinterpret_cast<uintptr_t>(d_cm) % 16 != 0) return fail(SHW_E_INVALID, "d_cm must be 16-byte aligned");
  if (!is_fin(gain)) return fail(SHW_E_INVALID, "gain must be finite");
  hipError_t e = launch_recon_partial(d_cm, ld_cm, p->n_modes, p->n_slopes, d_slopes, p->d_partial,
                                      (hipStream_t)stream);
  if (e == hipSuccess)
    e = launch_recon_integrate(p->d_partial, p->n_chunks, p->n_modes, gain, d_coefs, d_delta, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e, "shw_recon_step launch");
  return ok();
}

extern "C" int shw_recon_plan_destroy(shw_recon_plan* p) {
  if (!p) return ok();
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != p->device) (void)hipSetDevice(p->device);
  if (p->d_partial) (void)hipFree(p->d_partial);
  if (cur != p->device) (void)hipSetDevice(cur);
  delete p;
  return ok();
}

// ---------------------------------------------------------------- open-loop geometry, PSF extras

static int fill_layers(LayerSet& S, int32_t n_layers, const float* const* d_screen, const int32_t* rows,
                       const int32_t* cols, const int64_t* pitch, const double* params) {
  if (n_layers < 1 || n_layers > kMaxLayers) return fail(SHW_E_INVALID, "n_layers %d outside [1, %d]", n_layers, kMaxLayers);
  if (!d_screen || !rows || !cols || !pitch || !params) return fail(SHW_E_INVALID, "NULL layer argument");
  S = LayerSet{};
  S.n_layers = n_layers;
  for (int l = 0; l < n_layers; ++l) {
    const double* q = params + 4 * l;
    if (!d_screen[l]) return fail(SHW_E_INVALID, "layer %d screen is NULL", l);
    if (rows[l] < 2 || cols[l] < 2 || pitch[l] < cols[l]) return fail(SHW_E_INVALID, "layer %d: bad screen size", l);
    if (!(is_fin(q[0]) && q[0] > 0) || !(is_fin(q[1]) && q[1] >= 0) || !is_fin(q[2]) || !is_fin(q[3]))
      return fail(SHW_E_INVALID, "layer %d: pitch must be > 0, altitude >= 0, origin finite", l);
    LayerDesc& L = S.layer[l];
    L.screen = d_screen[l];
    L.rows = rows[l];
    L.cols = cols[l];
    L.pitch = pitch[l];
    L.pitch_m = q[0];
    L.inv_pitch = 1.0 / q[0];
    L.alt_m = q[1];
    L.x0 = q[2];
    L.y0 = q[3];
  }
  return SHW_OK;
}

// True if the screen coordinates of the square [xa, xb] x [ya, yb] (metres, before the layer's
// scale 1/pitch and origin) stay inside layer L's samples.
static bool footprint_inside(const LayerDesc& L, double xa, double xb, double ya, double yb) {
  const double Xa = L.x0 + xa / L.pitch_m, Xb = L.x0 + xb / L.pitch_m;
  const double Ya = L.y0 + ya / L.pitch_m, Yb = L.y0 + yb / L.pitch_m;
  const double lo_x = Xa < Xb ? Xa : Xb, hi_x = Xa < Xb ? Xb : Xa;
  const double lo_y = Ya < Yb ? Ya : Yb, hi_y = Ya < Yb ? Yb : Ya;
  return lo_x >= 0.0 && lo_y >= 0.0 && hi_x <= (double)(L.cols - 1) && hi_y <= (double)(L.rows - 1);
}

extern "C" int shw_project_layers(int32_t n_layers, const float* const* d_screen, const int32_t* screen_rows,
                                  const int32_t* screen_cols, const int64_t* screen_pitch, const double* layer_params,
                                  int32_t pupil_n, double dx_m, int32_t n_targets, const double* target_params,
                                  const double* d_tilt, float* d_out, int64_t out_pitch, int64_t out_stride,
                                  void* stream) {
  LayerSet S;
  int e = fill_layers(S, n_layers, d_screen, screen_rows, screen_cols, screen_pitch, layer_params);
  if (e != SHW_OK) return e;
  if (pupil_n < 1 || pupil_n > 16384) return fail(SHW_E_INVALID, "pupil_n %d outside [1, 16384]", pupil_n);
  if (!(is_fin(dx_m) && dx_m > 0)) return fail(SHW_E_INVALID, "dx_m must be > 0");
  if (n_targets < 0) return fail(SHW_E_INVALID, "n_targets < 0");
  if (n_targets == 0) return ok();
  if (!target_params || !d_out) return fail(SHW_E_INVALID, "NULL argument");
  if (out_pitch < pupil_n) return fail(SHW_E_INVALID, "out_pitch < pupil_n");
  if (n_targets > 1 && out_stride < out_pitch * pupil_n) return fail(SHW_E_INVALID, "targets' outputs overlap");
  const double half = (0.5 * pupil_n - 0.5) * dx_m;  // pupil pixel centres span [-half, half]
  for (int t = 0; t < n_targets; ++t) {
    const double* q = target_params + 3 * t;
    if (!is_fin(q[0]) || !is_fin(q[1]) || !(is_fin(q[2]) && q[2] >= 0))
      return fail(SHW_E_INVALID, "target %d: direction must be finite, altitude >= 0", t);
    for (int l = 0; l < n_layers; ++l) {
      const LayerDesc& L = S.layer[l];
      if (q[2] > 0 && !(q[2] > L.alt_m)) return fail(SHW_E_INVALID, "target %d is not above layer %d", t, l);
      const double s = q[2] > 0 ? 1.0 - L.alt_m / q[2] : 1.0;
      const double cx = L.alt_m * q[0], cy = L.alt_m * q[1];
      if (!footprint_inside(L, cx - s * half, cx + s * half, cy - s * half, cy + s * half))
        return fail(SHW_E_INVALID, "target %d: footprint leaves layer %d", t, l);
    }
  }
  ProjectLaunch a{};
  for (int l = 0; l < n_layers; ++l)
    a.layer[l] = ProjectLayer{S.layer[l].screen, S.layer[l].pitch, S.layer[l].rows, S.layer[l].cols};
  a.n_layers = n_layers;
  a.pupil_n = pupil_n;
  a.dx = dx_m;
  a.out_pitch = out_pitch;
  a.out_stride = out_stride;
  hipStream_t st = (hipStream_t)stream;
  ProjectPlace place[kMaxLayers];
  for (int l = 0; l < n_layers; ++l) {
    const LayerDesc& L = S.layer[l];
    place[l] = ProjectPlace{L.x0, L.y0, L.alt_m, L.alt_m * L.inv_pitch, L.inv_pitch};
  }
  const bool maps = n_targets <= kProjectMaps / n_layers;
  if (!maps) std::copy(place, place + n_layers, a.place);
  for (int t0 = 0; t0 < n_targets; t0 += a.n_t) {
    const int limit = maps ? n_targets : kProjectTargets;
    a.n_t = n_targets - t0 < limit ? n_targets - t0 : limit;
    for (int k = 0; k < a.n_t; ++k) {
      const double* q = target_params + 3 * (t0 + k);
      const ProjectTarget g{q[0], q[1], q[2] > 0 ? 1.0 / q[2] : 0.0};
      if (!maps) a.target[k] = g;
      for (int l = 0; maps && l < n_layers; ++l) a.map[k * n_layers + l] = project_map(place[l], g, dx_m);
    }
    a.tilt = d_tilt ? d_tilt + 2 * t0 : nullptr;
    a.out = d_out + t0 * out_stride;
    hipError_t he = launch_project_layers(a, maps, st);
    if (he != hipSuccess) return hip_fail(he, "project layers");
  }
  return ok();
}

extern "C" int shw_uplink_tilt(int32_t n_layers, const float* const* d_screen, const int32_t* screen_rows,
                               const int32_t* screen_cols, const int64_t* screen_pitch, const double* layer_params,
                               int32_t n_lgs, const double* lgs_params, double llt_diameter_m, int32_t n_samples,
                               double* d_tilt, void* stream) {
  UplinkLaunch a{};
  int e = fill_layers(a.L, n_layers, d_screen, screen_rows, screen_cols, screen_pitch, layer_params);
  if (e != SHW_OK) return e;
  if (n_lgs < 0) return fail(SHW_E_INVALID, "n_lgs < 0");
  if (n_lgs == 0) return ok();
  if (!lgs_params || !d_tilt) return fail(SHW_E_INVALID, "NULL argument");
  if (!(is_fin(llt_diameter_m) && llt_diameter_m > 0)) return fail(SHW_E_INVALID, "llt_diameter_m must be > 0");
  if (n_samples < 2 || n_samples > 256) return fail(SHW_E_INVALID, "n_samples %d outside [2, 256]", n_samples);
  const double half = 0.5 * llt_diameter_m;
  for (int k = 0; k < n_lgs; ++k) {
    const double* q = lgs_params + 5 * k;
    for (int j = 0; j < 4; ++j)
      if (!is_fin(q[j])) return fail(SHW_E_INVALID, "LGS %d: launcher and direction must be finite", k);
    if (!(is_fin(q[4]) && q[4] > 0)) return fail(SHW_E_INVALID, "LGS %d: sodium altitude must be > 0", k);
    for (int l = 0; l < n_layers; ++l) {
      const LayerDesc& L = a.L.layer[l];
      if (!(q[4] > L.alt_m)) return fail(SHW_E_INVALID, "LGS %d is not above layer %d", k, l);
      const double f = L.alt_m / q[4];
      const double cx = q[0] * (1.0 - f) + L.alt_m * q[2], cy = q[1] * (1.0 - f) + L.alt_m * q[3];
      if (!footprint_inside(L, cx - half, cx + half, cy - half, cy + half))
        return fail(SHW_E_INVALID, "LGS %d: beam leaves layer %d", k, l);
    }
  }
  a.n_s = n_samples;
  a.d = llt_diameter_m;
  hipStream_t st = (hipStream_t)stream;
  for (int k0 = 0; k0 < n_lgs; k0 += kUplinkChunk) {
    const int nk = n_lgs - k0 < kUplinkChunk ? n_lgs - k0 : kUplinkChunk;
    a.n = nk;
    for (int k = 0; k < nk; ++k)
      for (int j = 0; j < 5; ++j) a.lgs[k][j] = lgs_params[5 * (k0 + k) + j];
    a.tilt = d_tilt + 2 * k0;
    hipError_t he = launch_uplink_tilt(a, st);
    if (he != hipSuccess) return hip_fail(he, "uplink tilt");
  }
  return ok();
}

// Validation and launch arguments shared by the two encircled-energy entry points.  Returns
// SHW_OK with `a` filled (a.ws left for the caller), or an error; n_psf == 0 is SHW_OK with
// a.n_psf == 0 and nothing to launch.
static int ee_setup(const shw_psf_plan* plan, const float* d_psf, int32_t n_psf, int64_t psf_stride, int32_t n_r,
                    const double* r_px, double* d_ee, EeLaunch& a) {
  a = EeLaunch{};
  if (!plan) return fail(SHW_E_INVALID, "plan is NULL");
  const int M = plan->fft_m;
  if (M > 2048) return fail(SHW_E_UNSUPPORTED, "encircled energy supports fft_m <= 2048");
  if (n_psf < 0) return fail(SHW_E_INVALID, "n_psf < 0");
  if (n_psf == 0) return ok();
  if (!d_psf || !r_px || !d_ee) return fail(SHW_E_INVALID, "NULL argument");
  if (n_psf > 1 && psf_stride < (int64_t)M * M) return fail(SHW_E_INVALID, "psf_stride < fft_m^2");
  if (n_r < 1 || n_r > kMaxRadii) return fail(SHW_E_INVALID, "n_r %d outside [1, %d]", n_r, kMaxRadii);
  for (int k = 0; k < n_r; ++k) {
    if (!(is_fin(r_px[k]) && r_px[k] >= 0)) return fail(SHW_E_INVALID, "radius %d must be finite and >= 0", k);
    a.r2[k] = r_px[k] * r_px[k];
  }
  int cur = 0;
  (void)hipGetDevice(&cur);
  if (cur != plan->device) return fail(SHW_E_INVALID, "the current device is not the plan's device");
  a.psf = d_psf;
  a.psf_stride = psf_stride;
  a.m = M;
  a.n_psf = n_psf;
  a.n_r = n_r;
  a.ee = d_ee;
  return ok();
}

extern "C" int psf_encircled_energy(shw_psf_plan* plan, const float* d_psf, int32_t n_psf, int64_t psf_stride,
                                    int32_t n_r, const double* r_px, double* d_ee, void* stream) {
  EeLaunch a;
  const int rc = ee_setup(plan, d_psf, n_psf, psf_stride, n_r, r_px, d_ee, a);
  if (rc != SHW_OK || n_psf == 0) return rc;
  const size_t need = (size_t)n_psf * kEeGroups * (n_r + 1) * sizeof(double);
  if (need > plan->ee_bytes) {
    hipError_t he = hipDeviceSynchronize();
    if (he != hipSuccess) return hip_fail(he, "synchronise before growing the workspace");
    if (plan->d_ee_ws) (void)hipFree(plan->d_ee_ws);
    plan->d_ee_ws = nullptr;
    plan->ee_bytes = 0;
    he = hipMalloc((void**)&plan->d_ee_ws, need);
    if (he != hipSuccess) return fail(SHW_E_NOMEM, "encircled-energy workspace of %zu bytes", need);
    plan->ee_bytes = need;
  }
  a.ws = plan->d_ee_ws;
  hipError_t he = launch_encircled_energy(a, (hipStream_t)stream);
  if (he != hipSuccess) return hip_fail(he, "encircled energy");
  return ok();
}

extern "C" int psf_encircled_energy_noalloc(const shw_psf_plan* plan, const float* d_psf, int32_t n_psf,
                                            int64_t psf_stride, int32_t n_r, const double* r_px, double* d_ee,
                                            void* stream) {
  EeLaunch a;
  const int rc = ee_setup(plan, d_psf, n_psf, psf_stride, n_r, r_px, d_ee, a);
  if (rc != SHW_OK || n_psf == 0) return rc;
  const size_t need = (size_t)n_psf * kEeGroups * (n_r + 1);
  if (need > kEeScratchDoubles)
    return fail(SHW_E_INVALID, "n_psf * 200 * (n_r + 1) = %zu doubles exceeds the %zu of the static workspace",
                need, kEeScratchDoubles);
  // every workspace entry the final pass reads is written by the first pass of the same call, so
  // nothing is cleared; what an earlier call left there is never read
  hipError_t he = ee_scratch_device(plan->device, &a.ws);
  if (he != hipSuccess) return hip_fail(he, "address of the static encircled-energy workspace");
  he = launch_encircled_energy(a, (hipStream_t)stream);
  if (he != hipSuccess) return hip_fail(he, "encircled energy (static workspace)");
  return ok();
}

extern "C" int psf_resample_accumulate(int32_t fft_m, const float* d_src, double scale, float weight, float* d_dst,
                                       void* stream) {
  if (fft_m < 2 || fft_m > 16384) return fail(SHW_E_INVALID, "fft_m %d outside [2, 16384]", fft_m);
  if (!d_src || !d_dst) return fail(SHW_E_INVALID, "NULL argument");
  if (!(is_fin(scale) && scale > 0) || !std::isfinite(weight)) return fail(SHW_E_INVALID, "scale must be > 0, weight finite");
  const int64_t n = (int64_t)fft_m * fft_m;
  if (d_src < d_dst + n && d_dst < d_src + n) return fail(SHW_E_INVALID, "source and destination overlap");
  hipError_t he = launch_psf_resample(d_src, fft_m, scale, weight, d_dst, (hipStream_t)stream);
  if (he != hipSuccess) return hip_fail(he, "psf resample");
  return ok();
}
