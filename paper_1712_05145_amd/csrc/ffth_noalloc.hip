// ffth_green_apply_noalloc: the Green operator application of
// ffth_green_apply without a plan or a caller workspace, for callers that
// cannot allocate device memory.  Everything the passes need beyond the input
// and output fields (launch descriptor, gating state and the half spectrum) lives in one file-scope device
// array of fixed size, one copy per GPU, held until the process ends.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>

#include "ffth.h"
#include "ffth_launch.h"
#include "ffth_types.h"

using namespace ffth;

namespace {

constexpr size_t kAlign = 256;
constexpr size_t al(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Regions of the scratch array for the largest grid: descriptor, state and the
// FP64 half spectrum (48 bytes per voxel).
constexpr size_t kVox = FFTH_NOALLOC_MAX_VOXELS;
constexpr size_t kOffDesc = 0;
constexpr size_t kOffState = al(sizeof(Desc));
constexpr size_t kOffSpec = kOffState + al(sizeof(SolverState));
constexpr size_t kBytes = kOffSpec + al(kVox * 6 * sizeof(double));

static_assert(kBytes == FFTH_NOALLOC_SCRATCH_BYTES, "scratch size stated in ffth.h");

static __device__ __align__(256) unsigned char scratch[kBytes];

// Device address of `scratch` per GPU (its name is a host-side stand-in).
constexpr int kMaxDevices = 64;
std::mutex g_mu;
void* g_ptr[kMaxDevices] = {nullptr};

int kchunk_of(int h) {
  int c = h < 16 ? h : 16;
  while (h % c) --c;
  return c;
}

template <typename T>
hipError_t green_passes(const int n[3], hipStream_t st, const Desc& d0, const SolverState& s0, Desc* d) {
  const long rows = (long)n[0] * n[1], nvox = rows * n[2];
  const double scale = 1.0 / (double)nvox;
  const GroupShape g = group_shape(n, sizeof(T) == 8);
  hipError_t e;
  if (g.on) {   // grouped passes, as a plan takes them
    if ((e = GLaunch<T>::field_fwd1(n[2], g, st, d0, s0, d, rows, nvox)) != hipSuccess) return e;
    if ((e = GLaunch<T>::gz(n[0], g, false, 1, st, d, OP_GAMMA, n[1], scale, -1, 0, 0)) != hipSuccess) return e;
    return GLaunch<T>::field_inv(n[2], g, 1, st, d, false, rows, nvox);
  }
  if ((e = Launch<T>::field_fwd1(n[2], st, d0, s0, d, rows, nvox)) != hipSuccess) return e;
  const int h = n[2] / 2, kc = kchunk_of(h);
  if (n[0] == 1) {   // 2-D: one spectral pass
    const int tk = Launch<T>::z_cols(n[1], 0);
    if ((e = Launch<T>::zpass(n[1], 0, false, dim3((kc + tk - 1) / tk * (h / kc), 1), st, d, OP_GAMMA, 1, h, scale,
                              true)) != hipSuccess)
      return e;
    return Launch<T>::field_inv(n[2], 1, st, d, false, rows, nvox);
  }
  const int ncols = kc * 6, nplanes = n[0] * (h / kc);
  const int cw = Launch<T>::y_cols(n[1], 0), ntiles = (ncols + cw - 1) / cw;
  if ((e = Launch<T>::ypass(n[1], 0, false, dim3(nplanes * ntiles, 1), st, d, -1, ncols, ntiles)) != hipSuccess)
    return e;
  const long M = (long)n[1] * kc;
  const int tk = Launch<T>::z_cols(n[0], 0);
  const int nzb = (int)((M + tk - 1) / tk) * (h / kc);
  if ((e = Launch<T>::zpass(n[0], 0, false, dim3(nzb, 1), st, d, OP_GAMMA, n[1], h, scale)) != hipSuccess) return e;
  if ((e = Launch<T>::ypass(n[1], 0, false, dim3(nplanes * ntiles, 1), st, d, +1, ncols, ntiles)) != hipSuccess)
    return e;
  return Launch<T>::field_inv(n[2], 1, st, d, false, rows, nvox);
}

ffth_status fail(ffth_status s, const std::string& msg) {
  set_last_error(msg.c_str());
  return s;
}

}  // namespace

extern "C" {

ffth_status ffth_green_apply_noalloc(const int32_t n[3], double lambda0, double mu0, const double* tau, double* eta,
                                     int32_t precision, void* hip_stream) {
  set_last_error("");
  if (!n || !tau || !eta) return fail(FFTH_ERR_INVALID, "null argument");
  if (precision != FFTH_FP64 && precision != FFTH_FP32) return fail(FFTH_ERR_INVALID, "precision must be FP64 or FP32");
  int nn[3] = {n[0], n[1], n[2]};
  if (!grid_supported(nn)) return fail(FFTH_ERR_INVALID, "unsupported grid");
  const long nvox = (long)nn[0] * nn[1] * nn[2];
  if (nvox > (long)FFTH_NOALLOC_MAX_VOXELS)
    return fail(FFTH_ERR_INVALID, "grid of " + std::to_string(nvox) + " voxels exceeds the " +
                                      std::to_string((long)FFTH_NOALLOC_MAX_VOXELS) +
                                      "-voxel limit of the allocation-free entry point");
  if (!(mu0 != 0.0) || !(lambda0 + 2.0 * mu0 != 0.0) || !std::isfinite(mu0) || !std::isfinite(lambda0))
    return fail(FFTH_ERR_INVALID, "reference medium needs mu0 != 0 and lambda0 + 2 mu0 != 0");
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return fail(FFTH_ERR_DEVICE, "no usable device");
  char* base;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_ptr[dev]) {
      void* p = nullptr;
      const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !p) return fail(FFTH_ERR_DEVICE, std::string("hipGetSymbolAddress: ") + hipGetErrorString(e));
      g_ptr[dev] = p;
    }
    base = (char*)g_ptr[dev];
  }
  hipStream_t st = (hipStream_t)hip_stream;
  Desc d;
  std::memset(&d, 0, sizeof(d));
  d.spec = base + kOffSpec;
  d.st = (SolverState*)(base + kOffState);
  d.io = (void*)tau;
  d.out = eta;
  d.nc = 6;
  d.lam0 = lambda0;
  d.mu0 = mu0;
  d.gam_h = 0.5 / mu0;
  d.gam_r = (lambda0 + mu0) / (lambda0 + 2.0 * mu0);
  d.inv_nvox = 1.0 / (double)nvox;
  d.tau_scale = 1.0;
  d.op_scale = 1.0 / (double)nvox;
  SolverState s;
  std::memset(&s, 0, sizeof(s));
  s.active = 1;
  s.first = 1;
  s.max_iter = 1;
  s.res = 1.0;
  s.dscale = s.idscale = 1.0;
  s.gscale = -1.0;
  Desc* dd = (Desc*)(base + kOffDesc);
  const hipError_t e = precision == FFTH_FP64 ? green_passes<double>(nn, st, d, s, dd)
                                              : green_passes<float>(nn, st, d, s, dd);
  if (e != hipSuccess) return fail(FFTH_ERR_DEVICE, std::string("launch: ") + hipGetErrorString(e));
  return FFTH_OK;
}

}  // extern "C"
