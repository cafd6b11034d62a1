// The inertia-count search for launches of few wavefronts per SIMD: 64, 32 or
// 8 lanes per wavelength, every FP64 polynomial coefficient in VGPRs
// (masw_inertia_kernel.hpp).
#define MASW_COEFF_POLICY 2
#include "masw_inertia_kernel.hpp"

namespace masw {
namespace {

// Bound by the latency of its dependent rounds.  With 64 lanes on a grid of
// 115,001 points every wavelength takes four (First, Narrow, Try and one of
// the refinement): 1000 wavelengths over 20 layers in 54 us, where sampling,
// counting and multisecting apart took five and 61 us.
//
// A wavefront takes 64 / S consecutive wavelengths, but only those of the
// first one's model: the others of them, from the start of each further model
// on, are a wavefront's of their own (one for every model, after the first
// a.n_items S / 64), so that none runs two models one after the other.  Where
// there are more models than wavelengths, most have none, and a wavefront looks
// through several.
template <int S>
__global__ __launch_bounds__(64 * kInertiaWaves) void inertia_lone_kernel(SweepArgs a) {
  __shared__ unsigned long long s_cnt[kInertiaWaves][7];
  stamp_start(a.tstamp, 1);
  Tally t;
  Rounds rounds;
  unsigned long long useful = 0;
  unsigned deferred = 0;
  constexpr int kPer = 64 / S;
  const int wave = __builtin_amdgcn_readfirstlane(int(blockIdx.x) * kInertiaWaves + int(threadIdx.x >> 6));
  const int runs = (a.n_items + kPer - 1) / kPer;
  const int extra = int(lone_extra(a.n_items, a.n_models, S));
  for (int m = wave - runs;; m += extra) {
    int begin = a.n_items, model = m;
    if (wave < runs) {
      begin = wave * kPer;
      model = __builtin_amdgcn_readfirstlane(a.lam_model[begin]);
    } else if (wave - runs < extra) {
      begin = __builtin_amdgcn_readfirstlane(a.models[m].lam_base);
      if (begin % kPer == 0) begin = a.n_items;  // the run's own wavefront has it
    }
    if (begin < a.n_items) {
      const ModelDesc d = a.models[model];
      const int stop = min((begin / kPer + 1) * kPer, __builtin_amdgcn_readfirstlane(d.lam_base + d.n_lam));
      run_groups<S>(a, begin, stop, d, rounds, useful, deferred);
    }
    if constexpr (S >= 32) {
      for (unsigned long long left = __ballot(deferred != 0 && (threadIdx.x & (S - 1)) == 0); left != 0ull;
           left &= left - 1)
        run_wavelength(a, begin + (__ffsll((long long)left) - 1) / S, t);
      deferred = 0;
    }
    if (wave < runs || wave - runs >= extra || a.n_models - m <= extra) break;
  }
  if (S < 32 && __ballot(deferred != 0) != 0ull && (threadIdx.x & 63) == 0)
    atomicAdd(&a.counters->deferred, 1u);
  flush_tally(a, rounds, t, useful, s_cnt);
  stamp_end(a.tstamp);
}

}  // namespace

hipError_t launch_inertia_lone(const SweepArgs& a, int S, hipStream_t s, int* blocks_out, bool* deferring) {
  const int64_t blocks = lone_blocks(a.n_items, a.n_models, S);
  if (blocks > a.wg_rows) return hipErrorInvalidValue;
  *blocks_out = int(blocks);
  *deferring = S < 32;
  const dim3 grid(static_cast<unsigned>(blocks)), block(64 * kInertiaWaves);
  switch (S) {
    case 64: hipLaunchKernelGGL(inertia_lone_kernel<64>, grid, block, 0, s, a); break;
    case 32: hipLaunchKernelGGL(inertia_lone_kernel<32>, grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL(inertia_lone_kernel<8>, grid, block, 0, s, a); break;
  }
  return hipGetLastError();
}

}  // namespace masw
