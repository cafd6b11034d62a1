// The full-grid sign map, in a translation unit of its own: its layer loop is
// all there is in the kernel, so the series' coefficients stay in VGPRs
// (MASW_COEFF_POLICY 0; 300 wavelengths x 11,501 velocities over 20 layers:
// 307 us, 319 with all in SGPRs).
#include <hip/hip_runtime.h>

#include "masw_host.hpp"
#include "masw_internal.hpp"
#include "masw_math.hpp"

namespace masw {
namespace {

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Every (wavelength, grid point) of model 0, no early exit: blockIdx.y is
// the wavelength, x covers the grid.
template <typename T>
__global__ __launch_bounds__(256) void sign_map_kernel(SignMapArgs a) {
  const int w = blockIdx.y;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n_c) return;
  const ModelDesc d = a.models[0];
  const double k64 = a.lam_k[w];
  const size_t o = size_t(w) * size_t(a.n_c) + size_t(i);
  if (!(k64 == k64)) {
    a.sigma[o] = int8_t(kNaNSign);
    if (a.logabs) a.logabs[o] = __builtin_nan("");
    return;
  }
  const int N = uniform(d.n_layers);
  const double c = a.c64[d.c_base + i];
  int sg;
  if constexpr (sizeof(T) == 8) {
    const LayerRec64* L = a.layers64 + uniform(d.layer_base);
    if (a.logabs) {
      double la;
      sg = det_sign_logabs<double>(c, k64, L, N, k64 * L[N].aux, &la);
      a.logabs[o] = la;
    } else {
      sg = det_sign<double, false>(c, k64, L, N, nullptr);
    }
  } else {
    const LayerRec32* L = a.layers32 + uniform(d.layer_base);
    const LayerRec64* L64 = a.layers64 + uniform(d.layer_base);
    if (a.logabs) {
      double la;
      sg = det_sign_logabs<float>(float(c), float(k64), L, N, k64 * L64[N].aux, &la);
      a.logabs[o] = la;
    } else {
      sg = det_sign<float, false>(float(c), float(k64), L, N, nullptr);
    }
  }
  a.sigma[o] = int8_t(sg);
}

}  // namespace

hipError_t launch_sign_map(bool fp32, const SignMapArgs& a, hipStream_t s) {
  if (a.n_lam == 0 || a.n_c == 0) return hipSuccess;
  const dim3 grid((a.n_c + 255) / 256, a.n_lam);
  if (fp32)
    hipLaunchKernelGGL(sign_map_kernel<float>, grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(sign_map_kernel<double>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace masw
