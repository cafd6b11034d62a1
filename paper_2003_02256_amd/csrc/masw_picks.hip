// The walk and the split path on many wavelengths: sweep, then picks.
//
// A sweeping wavefront (masw_sweep.hpp) that checks and refines its own pick
// eliminates K at 64 positions for the split path's check and, twice, at the
// eight points of the refinement with all its 64 lanes.  Over 1.12 M
// wavelengths of 16.5 layers that was 8 of the walk's 160 ms and 13 of the
// split path's 83.  Where there are items enough to keep every SIMD busy
// without the deepest of them deciding the time, the work is three launches
// instead:
//   first_change_kernel: the sweep alone, one wavefront per item of the work
//       order.  Its candidate goes to out_idx.  Without the eliminations it
//       needs few registers (FP32: eight wavefronts per SIMD).
//   pick_kernel: eight lanes per wavelength, eight wavelengths of one model
//       at a time.  Split: FP64 points at the grid's start and from three
//       before the candidate to three after it, seven neighbours.  Where the
//       counts E at the start and at the first of the seven are equal there is
//       no change up to that one (masw_inertia.hpp), and the first of the
//       others where sign(det K) changes is the pick.  Then, and on the walk at
//       once, the refinement by eight points a round (Refine8), whose first
//       round has K's own signs at the pick's two grid points, and their counts.
//   pick_rest_kernel: the others (no change found in FP32, a grid that starts
//       below c_low, a candidate that the eight points do not settle, a pole in
//       the step or several changes of E, a step at or above the half-space's S
//       velocity, a change that the elimination does not confirm), by a whole
//       wavefront each, as the one-launch sweep does them from the candidate on;
//       past a candidate that was none, from the last of the seven points on.
// Between the launches out_idx holds the candidate, or kDeferredIdx with the
// candidate (-1: none) in out_status and, on the split path, in out_ct where to
// go on after it (4 times the position plus the sign before it; 0: nowhere).
// Indices, statuses and roots are those of the one-launch sweep: the same
// eliminations at the same points decide.
// The 1.12 M wavelengths (19,001 velocities): 160 -> 151 ms, split 83 -> 68;
// before the sweeps' sign function, 211 and 98.  What one launch and three take
// differs most on short grids: 124,000 wavelengths x 2,000 velocities 2.82 and
// 2.00 ms (split 2.49 and 1.29), on models of strong contrast, a ninth of whose
// first candidates are a mode and a pole in one grid step, 2.22 and 1.97 (2.11
// and 1.93); 46,500 of the latter 0.87 and 1.02 on the split path, the others
// 0.99 and 0.68.
#define MASW_COEFF_POLICY 1
#include "masw_inertia_kernel.hpp"
#include "masw_sweep.hpp"

namespace masw {
namespace {

// Sweeping wavefronts per SIMD.  Measured on the 4096 models above, the whole
// call (ms): FP64 with 4 to 8 of them 154.1, 152.0, 151.2, 153.4, 153.6; FP32
// 82.3, 74.3, 70.2, 68.3, 69.7 (one launch, 4 and 5: 160.3 and 82.7).
template <int MODE>
constexpr int kSweepWaves = MODE == kModeSplit ? 7 : 6;

// Work claimed one unit at a time from kQueues counters of their own cache
// lines, unit kQueues i + x being the i-th of counter x, and the next counter's
// when one has run out.  Claims of one counter serialise at 12 ns each, which was
// all of the 1441 us of the FP32 sweep of 124,000 wavelengths to 278 velocities
// on average: 509 us with three counters and two items a claim (557 and 605 us
// with four and two items a claim of one counter).
constexpr unsigned kQueues = 1 + sizeof(Counters::more) / sizeof(Counters::Heads);
struct Claims {
  unsigned x, tried;
  // Unit of queue `which` (0: the sweep's items, 1: the last launch's list) of
  // n units, or n when all are taken.
  __device__ __forceinline__ unsigned next(Counters* c, int which, unsigned n) {
    while (tried < kQueues) {
      uint32_t* head = x == 0u ? (which ? &c->rest_head : &c->queue_head) : &c->more[x - 1u].head[which];
      unsigned i = 0;
      if ((threadIdx.x & 63) == 0) i = atomicAdd(head, 1u);
      i = kQueues * unsigned(uniform(int(i))) + x;
      if (i < n) return i;
      ++tried;
      x = x + 1u < kQueues ? x + 1u : 0u;
    }
    return n;
  }
};

// Items a sweeping wavefront takes at a time after its first: two in FP32 on
// grids of up to kShortGrid points with eight items or more for each wavefront,
// where the claims can bound the sweep: 120,000 wavelengths x 2,000 velocities
// 973 us with one, 827 with two.  Else one, whose work ends more evenly: FP32,
// 110,000 x 9,501, 3.83 ms against 3.91; FP64, twice as long an item, 54,000 x
// 8,105 3.66 against 3.83.  (46,500 x 9,501 FP32 1.70 with one, 1.87 with four;
// items dealt out without a claim made large batches 10 to 20% slower.)
constexpr unsigned kItemsForTwo = 8;
constexpr int kShortGrid = 4096;

template <int MODE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kSweepWaves<MODE>)))
void first_change_kernel(SweepArgs a) {
  const int lane = threadIdx.x;
  WorkCount wc;
  stamp_start(a.tstamp, 1);
  Claims claims{blockIdx.x % kQueues, 0u};
  const bool two = MODE == kModeSplit && unsigned(a.n_items) >= kItemsForTwo * gridDim.x &&
                   uniform(a.models[0].n_c) <= kShortGrid;
  const unsigned claim = two ? 2u : 1u;
  for (unsigned it = blockIdx.x, left = 0;;) {
    if (it >= unsigned(a.n_items)) break;
    int g;
    const ItemRef r = item_ref(a, int(it), &g);
    if (int(it) < a.prio_hi) __builtin_amdgcn_s_setprio(2);
    else if (int(it) < a.prio_mid) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
    const ItemOut o = item_out(a, g);
    if (!(r.k64 == r.k64)) {  // invalid model, grid or wavelength
      write_no_pick(o, MASW_STATUS_INVALID, lane == 0);
    } else {
      const int n = MODE == kModeFP64 ? r.n_c : r.n_real;
      const float k32 = float(r.k64);
      int carry = kNoSign, found = -1, sig_f, prev_f;
      // (a grid that starts below c_low is left to the last launch)
      const bool low = MODE == kModeFP64 && r.low;
      for (int base = 0; base < n && !low; base += 64) {
        const int i = base + lane;
        int sg = kNoSign;
        if (i < n) {
          if constexpr (MODE == kModeFP64) sg = sweep_minors64(r.c64[i], r.k64, r.L64, r.N);
          else sg = sweep_code32(r.c32[i], k32, r.L32, r.N);
        }
        const int f = round_first_change<1>(sg, carry, nullptr, &carry, &sig_f, &prev_f);
        wc.sweep += (unsigned long long)min(64, n - base);
        if (f >= 0) {
          found = base + f;
          break;
        }
      }
      if (MODE == kModeFP64 && found < 0 && !low && carry != kNaNSign) {
        write_no_pick(o, MASW_STATUS_NOT_FOUND, lane == 0);
        wc.useful += (unsigned long long)n;
      } else if (lane == 0) {
        *o.idx = found < 0 ? kDeferredIdx : found;
        *o.status = found;
        if (found < 0) *o.ct = 0.0;
      }
    }
    if (left > 0u) {
      ++it;
      --left;
    } else {
      it = gridDim.x + claim * claims.next(a.counters, 0, (unsigned(a.n_items) - gridDim.x + claim - 1u) / claim);
      left = claim - 1u;
    }
  }
  __builtin_amdgcn_s_setprio(0);
  flush_counts(a.counters, a.wg_counts, wc);
  stamp_end(a.tstamp);
}

// The picks of the wavelengths [begin, end) of one model, 64 / 8 at a time,
// each eight lanes a run of consecutive ones.  Per-lane variables are the
// same in a group's lanes.
template <int MODE>
__device__ __forceinline__ void run_picks(const SweepArgs& a, int begin, int end, const ModelDesc& d, WorkCount& wc) {
  const int lane = threadIdx.x & 63, sub = lane & 7, base = lane & ~7;
  const int N = uniform(d.n_layers), n_c = uniform(d.n_c);
  const double* c64 = a.c64 + uniform(d.c_base);
  const LayerRec64* L = a.layers64 + uniform(d.layer_base);
  const int per = (end - begin + 7) / 8;
  int g = begin + (lane >> 3) * per;
  const int g_end = min(g + per, end);
  auto in_group = [&](bool p) -> unsigned { return unsigned(__ballot(p) >> base) & 0xffu; };
  double k = 1.0;
  int at = 0, first = 0;  // candidate, then pick; first of the points of its check
  bool live = false, check = false;
  Refine8<false> r;
  r.init(0.0, 0.0, 0.0);
  for (;;) {
    while (!live && g < g_end) {  // the group's next candidate
      at = a.out_idx[g];
      if (at < 1) {
        ++g;
        continue;
      }
      k = a.lam_k[g];
      live = true;
      check = MODE == kModeSplit;
      if (check) {
        first = max(0, min(at - 3, n_c - 7));
      } else {
        r.init(c64[at - 1], c64[at], a.refine_rel);
      }
    }
    if (__ballot(live) == 0ull) break;
    const bool opens = r.stage == 0 && r.round == 0;  // the refinement's first round
    const double c = check ? c64[sub == 0 ? 0 : min(first + sub - 1, n_c - 1)] : r.point(sub);
    const Point v = eval_point<true>(c, k, L, N, live && (check || (opens && (sub == 0 || sub == 7))));
    const int sg_prev = previous_lane(v.sg);
    const unsigned changes = in_group(sub > 0 && v.sg != sg_prev), nan = in_group(v.sg == kNaNSign);
    wc.check += __popcll(__ballot(live && check));
    wc.refine += __popcll(__ballot(live && !check));
    bool rest = false, done = false;
    int resume = 0;
    if (live && check) {
      // equal counts at the grid's start and at the first of the seven points:
      // no change up to there; the seven are neighbours
      const int E_0 = from_lane<false>(v.E, base), E_1 = from_lane<false>(v.E, base + 1);
      const unsigned later = changes & 0xfcu;
      const int f = later ? __ffs(int(later)) - 1 : 0;
      const double c_lo = from_lane<false>(c, base + max(f - 1, 0)), c_hi = from_lane<false>(c, base + f);
      const bool certain = E_0 == E_1 && E_0 != inertia::kEvent && nan == 0u;
      rest = !certain || f == 0;
      // (no change among the seven: the last launch goes on from the last one)
      resume = certain && f == 0 && first + 7 < n_c ? (first + 7) * 4 + from_lane<false>(v.sg, base + 7) : 0;
      at = rest ? at : first + f - 1;
      r.init(c_lo, c_hi, a.refine_rel);
      check = false;
    } else if (live) {
      // E one larger at the step's upper end, and no pole in it: a single root
      if (opens) {
        const int s_lo = from_lane<false>(v.sg, base), s_hi = from_lane<false>(v.sg, base + 7);
        const int E_lo = from_lane<false>(v.E, base), E_hi = from_lane<false>(v.E, base + 7);
        const int P_lo = from_lane<false>(v.P, base), P_hi = from_lane<false>(v.P, base + 7);
        rest = nan != 0u || s_lo == s_hi || E_hi == inertia::kEvent || E_hi != E_lo + 1 || P_hi != P_lo;
      }
      if (!rest)
        done = r.update(c, v.sg, v.m, v.e, base) || !a.refine;
    }
    if (rest || done) {
      const ItemOut o = item_out(a, g);
      if (sub == 0) {
        *o.idx = rest ? kDeferredIdx : at;
        *o.status = rest ? at : MASW_STATUS_FOUND;
        if (MODE == kModeSplit && rest) *o.ct = double(resume);
        if (done) {
          *o.ct = c64[at];
          if (o.cref) *o.cref = o.refine ? 0.5 * (r.lo + r.hi) : __builtin_nan("");
          wc.useful += (unsigned long long)(at + 1);
        }
      }
      live = false;
      check = false;
      ++g;
    }
  }
}

template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void pick_kernel(SweepArgs a, int chunk) {
  WorkCount wc;
  const int64_t n_waves = int64_t(gridDim.x) * 4;
  for (int64_t run = int64_t(blockIdx.x) * 4 + uniform(threadIdx.x >> 6); run * chunk < a.n_items; run += n_waves) {
    const int begin = int(run * chunk), last = int(std::min<int64_t>((run + 1) * chunk, a.n_items));
    for (int g = begin; g < last;) {
      const ModelDesc d = a.models[uniform(a.lam_model[g])];
      const int stop = min(last, uniform(d.lam_base + d.n_lam));
      run_picks<MODE>(a, g, stop, d, wc);
      g = stop;
    }
    // The run's wavelengths that are left to the last launch, by one atomic:
    // the work order, which the sweep has been through, becomes their list.
    __threadfence();
    const int lane = threadIdx.x & 63;
    const bool left = begin + lane < last && ld_agent(a.out_idx + begin + lane) == kDeferredIdx;
    const unsigned long long all = __ballot(left);
    if (all != 0ull) {
      unsigned at = 0;
      if (lane == 0) at = atomicAdd(&a.counters->deferred, unsigned(__popcll(all)));
      at = unsigned(uniform(int(at))) + unsigned(__popcll(all & ((1ull << lane) - 1ull)));
      if (left) a.order[at] = begin + lane;
    }
  }
  wc.useful = inertia::wave_sum(wc.useful);
  if ((threadIdx.x & 63) == 0) {  // a row of counts for each wavefront
    unsigned long long* row = a.wg_counts + (size_t(blockIdx.x) * 4 + (threadIdx.x >> 6)) * kWgCounts;
    row[0] = row[4] = row[5] = row[6] = row[7] = 0ull;
    row[1] = wc.check;
    row[2] = wc.refine;
    row[3] = wc.useful;
  }
  __syncthreads();  // the stamp is thread 0's: the end of all four wavefronts
  stamp_end(a.tstamp);
}

template <int MODE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void pick_rest_kernel(SweepArgs a) {
  __shared__ SweepShared<1> sh;
  const unsigned n = a.counters->deferred;
  WorkCount wc;
  Claims claims{blockIdx.x % kQueues, 0u};
  bool took = blockIdx.x == 0;
  while (n != 0u) {
    const unsigned i = claims.next(a.counters, 1, n);
    if (i >= n) break;
    took = true;
    const int g = uniform(a.order[i]);
    const ItemRef r = item_of(a, g);
    const ItemOut o = item_out(a, g);
    ItemState st = item_state_init();
    int swept = uniform(*o.status);
    if constexpr (MODE == kModeSplit) {
      const int resume = uniform(int(*o.ct));
      if (resume != 0) {  // past the candidate, with the determinant's sign at seg_start - 1
        st.seg_start = (resume + 1) >> 2;
        st.seg_carry = resume - 4 * st.seg_start;
        st.start = st.seg_start - 1;
        swept = kNotSwept;
      }
    }
    run_item<MODE, 1, kFromRest>(r, st, 0x7fffffff, sh, wc, o, kNoCoop, a.counters, swept);
  }
  flush_counts(a.counters, a.wg_counts, wc);
  // (4096 maxima on one word would take 45 us: of the workgroups without an
  // item, only the first stamps)
  if (took) stamp_end(a.tstamp);
}

// Each launch's rows of work counts follow those of the one before; *rows is
// their number (at most cus (28 + 16 + 16), below the smallest item count).
template <int MODE>
hipError_t launch(int cus, hipStream_t s, const SweepArgs& a, int* blocks_out, int* rows) {
  // wavelengths a wavefront takes at a time: as launch_inertia's runs
  const int chunk = int(std::max<int64_t>(8, std::min<int64_t>(64, int64_t(a.n_items) / (int64_t(cus) * 32) / 8 * 8)));
  const int64_t runs = (int64_t(a.n_items) + chunk - 1) / chunk;
  const int blocks = int(std::min<int64_t>(a.n_items, int64_t(cus) * 4 * kSweepWaves<MODE>));
  const int picking = int(std::min<int64_t>((runs + 3) / 4, int64_t(cus) * 4)), rest = cus * 16;
  *blocks_out = blocks;
  *rows = blocks + 4 * picking + rest;
  if (*rows > a.wg_rows) return hipErrorInvalidValue;
  SweepArgs b = a;
  hipLaunchKernelGGL(first_change_kernel<MODE>, dim3(blocks), dim3(64), 0, s, b);
  b.wg_counts += size_t(blocks) * kWgCounts;
  hipLaunchKernelGGL(pick_kernel<MODE>, dim3(picking), dim3(256), 0, s, b, chunk);
  b.wg_counts += size_t(picking) * 4 * kWgCounts;
  hipLaunchKernelGGL(pick_rest_kernel<MODE>, dim3(rest), dim3(64), 0, s, b);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess || !a.misfit ? e : launch_staged_misfit(a, s);
}

}  // namespace

hipError_t launch_staged_picks(int mode, int cus, hipStream_t s, const SweepArgs& a, int* blocks_out, int* rows) {
  return mode == kModeFP64 ? launch<kModeFP64>(cus, s, a, blocks_out, rows)
                           : launch<kModeSplit>(cus, s, a, blocks_out, rows);
}

}  // namespace masw
