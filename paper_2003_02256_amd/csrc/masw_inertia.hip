// The inertia-count search as a launch of its own: the kernels for many
// wavelengths per SIMD, and the choice between them and the lone-wavefront
// variant (masw_inertia_kernel.hpp).
#define MASW_COEFF_POLICY 1
#include "masw_inertia_kernel.hpp"

namespace masw {
namespace {

// Persistent grid: each wavefront claims runs of `chunk` consecutive
// wavelengths from an atomic queue and takes a run model by model.
__global__ __launch_bounds__(64 * kInertiaWaves) __attribute__((amdgpu_waves_per_eu(4)))
void inertia_kernel(SweepArgs a, int chunk) {
  __shared__ unsigned long long s_cnt[kInertiaWaves][7];
  const int lane = threadIdx.x & 63;
  stamp_start(a.tstamp, 1);
  Rounds rounds;
  unsigned long long useful = 0;
  unsigned deferred = 0;
  for (;;) {
    unsigned q = 0;
    if (lane == 0) q = atomicAdd(&a.counters->queue_head, 1u);
    const int64_t first = int64_t(__builtin_amdgcn_readfirstlane(q)) * chunk;
    if (first >= a.n_items) break;
    const int last = int(std::min<int64_t>(first + chunk, a.n_items));
    for (int g = int(first); g < last;) {
      const ModelDesc d = a.models[__builtin_amdgcn_readfirstlane(a.lam_model[g])];
      const int stop = min(last, __builtin_amdgcn_readfirstlane(d.lam_base + d.n_lam));
      run_groups<8>(a, g, stop, d, rounds, useful, deferred);
      g = stop;
    }
  }
  if (__ballot(deferred != 0) != 0ull && lane == 0) atomicAdd(&a.counters->deferred, 1u);
  flush_tally(a, rounds, Tally{}, useful, s_cnt);
  stamp_end(a.tstamp);
}

// The deferred wavelengths, one whole wavefront each.  A wavefront looks
// through every gridDim-th wavelength, so that neighbours, which are often
// deferred together, go to different ones.
__global__ __launch_bounds__(64 * kInertiaWaves) void inertia_deferred_kernel(SweepArgs a) {
  __shared__ unsigned long long s_cnt[kInertiaWaves][7];
  if (a.counters->deferred == 0u) return;
  const int lane = threadIdx.x & 63;
  const int64_t n_waves = int64_t(gridDim.x) * kInertiaWaves;
  Tally t;
  for (int64_t base = int64_t(blockIdx.x) * kInertiaWaves + (threadIdx.x >> 6); base < a.n_items; base += 64 * n_waves) {
    const int64_t mine = base + lane * n_waves;
    unsigned long long todo = __ballot(mine < a.n_items && a.out_idx[mine < a.n_items ? mine : 0] == kDeferredIdx);
    for (; todo != 0ull; todo &= todo - 1)
      run_wavelength(a, int(base + (__ffsll((long long)todo) - 1) * n_waves), t);
  }
  flush_tally(a, Rounds{}, t, 0ull, s_cnt);
  stamp_end(a.tstamp);
}

}  // namespace

hipError_t launch_inertia(const SweepArgs& a, int cus, hipStream_t s, int* blocks_out) {
  *blocks_out = 0;
  if (a.n_items <= 0) return hipSuccess;
  // The lanes per wavelength: 64 or 32 while that leaves two wavefronts per
  // SIMD at most (their rounds overlap; a third would have to wait), 8 in
  // one launch of up to four, and beyond that 8 on a persistent grid, in runs
  // that predict their picks.  Measured on grids of 9,501 points (us a
  // kernel): 1258 wavelengths 68 with 64 lanes and 78 with 32; 2137: 91 with
  // 32 and 115 with 16; 7835: 140 with 8 and 146 with 16; 17,281: 219 with 8
  // at once and 338 on the persistent grid.  Before, with 64 lanes a
  // wavelength throughout: 93, 129, 294 and 693.
  const int64_t simds = int64_t(cus) * 4, n = a.n_items;
  const int S = n <= 2 * simds ? 64 : n <= 4 * simds ? 32 : 8;
  if (n <= 32 * simds) {
    bool deferring = false;
    const hipError_t e = launch_inertia_lone(a, S, s, blocks_out, &deferring);
    if (e != hipSuccess || !deferring) return e;
  } else {
    // Runs of up to 64 wavelengths, 8 of each group, whose predictions take
    // the evaluations per wavelength from 43 to 28; fewer where there are not
    // two runs for every resident wavefront.  One or four runs in that place:
    // 288,503 wavelengths in 1.62 and 1.51 ms against 1.42, 138,879 in 0.93
    // and 0.85 against 0.84.  4096 models, 1.12 M wavelengths: 3.8 ms, and
    // 18.0 with 64 lanes a wavelength.
    const int64_t waves = int64_t(cus) * 16;
    const int chunk = int(std::max<int64_t>(8, std::min<int64_t>(64, int64_t(a.n_items) / (2 * waves) / 8 * 8)));
    const int64_t runs = (int64_t(a.n_items) + chunk - 1) / chunk;
    const int64_t blocks = std::min<int64_t>((runs + kInertiaWaves - 1) / kInertiaWaves, int64_t(cus) * 4);
    *blocks_out = int(blocks);
    if (blocks > a.wg_rows) return hipErrorInvalidValue;
    hipLaunchKernelGGL(inertia_kernel, dim3(unsigned(blocks)), dim3(64 * kInertiaWaves), 0, s, a, chunk);
  }
  SweepArgs b = a;
  b.wg_counts = nullptr;  // the rows are the first launch's
  hipLaunchKernelGGL(inertia_deferred_kernel, 
                     dim3(unsigned(std::min<int64_t>((int64_t(a.n_items) + kInertiaWaves - 1) / kInertiaWaves, cus))),
                     dim3(64 * kInertiaWaves), 0, s, b);
  return hipGetLastError();
}

}  // namespace masw
