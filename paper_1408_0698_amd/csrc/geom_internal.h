// geom_internal.h - arguments of the LGS geometry kernels (layer projection, uplink tilt) and of
// the PSF extras (encircled energy, resampling), shared by the host library and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace shw {

constexpr int kMaxLayers = 16;
constexpr int kUplinkChunk = 32;   // beams per uplink launch (their parameters travel in the arguments)
constexpr int kMaxRadii = 64;      // encircled-energy radii per call
constexpr int kEeGroups = 200;     // row groups of the encircled-energy pass

// One phase-screen layer: FP32 OPD metres, rows of cols samples pitch apart, sample spacing
// pitch_m metres, altitude alt_m; the point above the telescope axis sits at screen pixel
// coordinates (x0, y0) (pixel centres at integer coordinates).
struct LayerDesc {
  const float* screen;
  int32_t rows, cols;
  int64_t pitch;
  double pitch_m, alt_m, x0, y0;
  double inv_pitch;  // 1 / pitch_m
};

struct LayerSet {
  LayerDesc layer[kMaxLayers];
  int32_t n_layers, pad0;
};

// OPD of target t at pupil pixel (i, j) (centre (j + 1/2 - N/2, i + 1/2 - N/2) dx from the axis):
// sum over layers of the bilinear screen sample at (1 - h/H) r + h theta, H the source altitude
// (0: infinity), plus tilt[t] . r when tilt is set.  In screen samples that point is
// (ax + b (j + 1/2 - N/2), ay + b (i + 1/2 - N/2)), with a map for each target and layer.
// Where a call's maps fit one launch they travel in its arguments; a call of more maps hands over what they are
// made of instead, and the kernel makes them (the same bits).
constexpr int kProjectMaps = 120;    // maps per launch
constexpr int kProjectTargets = 93;  // targets per launch of the second form
struct ProjectLayer {
  const float* screen;
  int64_t pitch;
  int32_t rows, cols;
};
struct ProjectMap {
  double ax, ay, b;
};
struct ProjectPlace {
  double x0, y0;       // origin, screen samples
  double alt_m, h;     // altitude, metres and screen samples
  double inv_pitch;    // 1 / sample spacing
};
struct ProjectTarget {
  double theta_x, theta_y, inv_h;
};
struct ProjectLaunch {
  ProjectLayer layer[kMaxLayers];
  union {
    ProjectMap map[kProjectMaps];  // [n_t][n_layers]
    struct {
      ProjectPlace place[kMaxLayers];
      ProjectTarget target[kProjectTargets];
    };
  };
  int32_t n_layers, n_t, pupil_n, pad0;
  double dx;
  const double* tilt;            // nullable [n_t][2] radians, already offset to the chunk
  float* out;                    // target t at out + t * out_stride
  int64_t out_pitch, out_stride;
};
// The map of a target on a layer, as on the host.
__host__ __device__ inline ProjectMap project_map(const ProjectPlace& L, const ProjectTarget& g, double dx) {
#pragma clang fp contract(off)
  return ProjectMap{L.x0 + L.h * g.theta_x, L.y0 + L.h * g.theta_y, (1.0 - L.alt_m * g.inv_h) * dx * L.inv_pitch};
}
hipError_t launch_project_layers(const ProjectLaunch& a, bool maps, hipStream_t st);

// Uplink tilt of LGS k: least-squares tilt of the summed layer OPD over the launch telescope's
// beam, an n_s x n_s grid of samples inside the disc of diameter d, the beam centred at
// launcher (1 - h/H) + h theta at altitude h.
struct UplinkLaunch {
  LayerSet L;
  double lgs[kUplinkChunk][5];  // launcher x, y (m), theta x, y (rad), sodium altitude (m)
  int32_t n, n_s;
  double d;
  double* tilt;                  // [n][2] radians, already offset to the chunk
};
hipError_t launch_uplink_tilt(const UplinkLaunch& a, hipStream_t st);

// Encircled energy of n_psf M x M PSFs: radii r_k (pixels, k < n_r) around (M/2, M/2).  Pass 1
// writes, per PSF and row group g, the sums over the group's rows of the energy inside each
// radius (ws [n_psf][n_r + 1][kEeGroups], entry n_r the groups' totals); pass 2 adds the
// groups in order and divides by the total.
struct EeLaunch {
  const float* psf;
  int64_t psf_stride;
  int32_t m, n_psf, n_r, pad0;
  double r2[kMaxRadii];
  double* ws;
  double* ee;          // [n_psf][n_r]
};
hipError_t launch_encircled_energy(const EeLaunch& a, hipStream_t st);

// Allocation-free form: the workspace is a file-scope device array of kEeScratchDoubles doubles
// (4 MiB), one per GPU.  ee_scratch_device() returns its address on `device`, which must be the
// current device; the first call per device looks the address up (hipGetSymbolAddress) and keeps it.
constexpr size_t kEeScratchDoubles = (size_t)1 << 19;
constexpr int kMaxDevices = 64;
hipError_t ee_scratch_device(int device, double** out);

// dst[v][u] += w * bilinear(src at (M/2 + (v - M/2) s, M/2 + (u - M/2) s)), zero outside src.
hipError_t launch_psf_resample(const float* src, int32_t m, double s, float w, float* dst, hipStream_t st);

}  // namespace shw
