// Pick output shared by the grid sweep and the inertia search: the first
// sign change among a wavefront's lanes, the FP64 refinement of a pick's
// bracket, and the per-wavelength outputs (Algorithm 1's C_t, with the
// refined root that the paper does not compute).
#pragma once
#include <hip/hip_runtime.h>

#include "masw_internal.hpp"
#include "masw_math.hpp"

namespace masw {

// Output slots of one item.
struct ItemOut {
  double* ct;
  int32_t* idx;
  int32_t* status;
  double* cref;  // may be null
  int refine;
  double refine_rel;  // refinement bracket width / c_hi
};

// Outputs of a wavelength without a pick; `writer` is the one thread that
// stores them.
__device__ __forceinline__ void write_no_pick(const ItemOut& o, int status, bool writer) {
  if (writer) {
    *o.idx = -1;
    *o.status = status;
    *o.ct = __builtin_nan("");
    if (o.cref) *o.cref = __builtin_nan("");
  }
}

// First sign change among the 64 lanes of one wavefront, lane l holding
// consecutive position l; lane 0 has no predecessor.  Every wavefront that
// calls it with the same signs gets the same answer, with no LDS or barrier.
// Returns the uniform lane of the first change or -1; *sig_at / *prev_at
// receive the signs at the change and *last the sign of lane 63.
__device__ __forceinline__ int wave_first_change(int sg, int* sig_at, int* prev_at, int* last) {
  const int lane = threadIdx.x & 63;
  const int prev = __shfl_up(sg, 1, 64);
  const bool change = (lane > 0) && (sg != kNoSign) && (prev != kNoSign) && (sg != prev);
  const unsigned long long mask = __ballot(change);
  *last = __shfl(sg, 63, 64);
  if (!mask) return -1;
  const int f = __ffsll((long long)mask) - 1;
  *sig_at = __shfl(sg, f, 64);
  *prev_at = __shfl(prev, f, 64);
  return f;
}

// The value of v in lane l (absolute).  U: l is the same in every lane, and so
// is the result, read into scalar registers; else each lane names its own.
template <bool U>
__device__ __forceinline__ int from_lane(int v, int l) {
  if constexpr (U) return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(l));
  return __shfl(v, l, 64);
}
template <bool U>
__device__ __forceinline__ double from_lane(double v, int l) {
  if constexpr (U) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = uint32_t(from_lane<true>(int(uint32_t(b)), l));
    const uint32_t hi = uint32_t(from_lane<true>(int(uint32_t(b >> 32)), l));
    return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
  }
  return __shfl(v, l, 64);
}

// v of the previous lane (of lane l - 1, in lane l); lane 0 keeps its own.
__device__ __forceinline__ int previous_lane(int v) {
  constexpr int kWaveShr1 = 0x138;  // DPP: a shift by one lane across the wavefront
  return __builtin_amdgcn_update_dpp(v, v, kWaveShr1, 0xf, 0xf, false);
}

// v of the next lane (of lane l + 1, in lane l); lane 63 keeps its own.
__device__ __forceinline__ double next_lane(double v) {
  constexpr int kWaveShl1 = 0x130;  // DPP: a shift by one lane across the wavefront
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const int lo = int(uint32_t(b)), hi = int(uint32_t(b >> 32));
  const uint32_t l = uint32_t(__builtin_amdgcn_update_dpp(lo, lo, kWaveShl1, 0xf, 0xf, false));
  const uint32_t h = uint32_t(__builtin_amdgcn_update_dpp(hi, hi, kWaveShl1, 0xf, 0xf, false));
  return __builtin_bit_cast(double, (uint64_t(h) << 32) | l);
}

// Root estimate between lanes l_b and l_b + 1, where the values m 2^e change
// sign, from the values of the four lanes from l_0 on (among them those two):
// inverse cubic interpolation, or linear interpolation where it leaves the
// interval.  The x of the four lanes rise; lanes are absolute.  Neville's
// scheme at value 0 runs on all lanes at once: after level n lane l holds the
// polynomial through lanes l .. l + n.
// With l_8 >= 0, where the cubic's neighbour among the eight lanes from l_8 on
// is further than tol / 50 from it, the estimate is the polynomial's through all
// eight, unless that is further than 1/16 of the interval from the cubic's
// (values that do not rise or fall throughout).  On grids of 1 m/s the cubic
// alone left one wavelength in 10 to a third round of the refinement, and the
// eight points none in 60; a curve of 12 layers x 1001 velocities, whose time
// is its slowest wavelength's, took 37.3 us and takes 29.7 (40.3 with 64 lanes
// multisecting).
template <bool U>
__device__ __forceinline__ double root_estimate(double x, double m, int e, int l_0, int l_b, int l_8 = -1,
                                                double tol = 0.0) {
  const double x_b = from_lane<U>(x, l_b);
  const double f = __builtin_ldexp(m, max(-1000, min(1000, e - from_lane<U>(e, l_b))));
  double y = x - x_b, f_n = f, r1 = 0.0;
  const double y_c = from_lane<U>(y, l_b + 1);
  auto level = [&] {
    f_n = next_lane(f_n);
    y = (y * f_n - next_lane(y) * f) * special::rcp(f_n - f);
  };
#pragma unroll 1
  for (int n = 1; n < 4; ++n) {
    level();
    if (n == 1) r1 = y;
  }
  double r = from_lane<U>(y, l_0);
  const double near = from_lane<U>(y, l_8 >= 0 && l_0 < l_8 + 4 ? l_0 + 1 : max(l_0 - 1, 0));
  const bool more = l_8 >= 0 && !(__builtin_fabs(near - r) <= 0.02 * tol);
  if (__ballot(more) != 0ull) {
#pragma unroll 1
    for (int n = 4; n < 8; ++n) level();
    const double r8 = from_lane<U>(y, max(l_8, 0));
    if (more && __builtin_fabs(r8 - r) <= 0.0625 * y_c) r = r8;
  }
  if (!(r > 0.0 && r < y_c)) r = from_lane<U>(r1, l_b);
  if (!(r > 0.0 && r < y_c)) r = 0.5 * y_c;
  return x_b + r;
}

// Refinement of a bracket [lo, hi] in which det K changes sign once and no
// layer denominator does, by eight lanes evaluating eight points a round:
//   0. both ends and six equally spaced points between them; the sign change
//      gives the next bracket, and inverse interpolation of det K through the
//      eight points a root estimate (root_estimate);
//   1. points around the estimate: two 0.9 tol apart, which end the
//      refinement when they bracket the root, and three rungs of a widening
//      ladder on either side, so that an estimate that is off still narrows
//      the bracket to a rung, and a new estimate from that round's values;
//   2. eight equally spaced inner points, where a ladder round narrowed the
//      bracket less than eight times or missed the root.
// The two rounds that a pick takes cost 16 evaluations; 64 lanes multisecting
// it 63-fold took 128 for a bracket of the same width, whose middle was 4e5
// times further from the root: the root estimate is good to about 1e-14.
// The outcome depends on the eight points alone, so eight lanes of a
// wavefront (eight wavelengths at once) and a whole wavefront that has them in
// lanes 0..7 (U: every value uniform; the other lanes repeat them, or hold the
// points between them in refine_and_write's first round) give the same bits.
constexpr int kMaxRefineRounds = 48;

template <bool U>
struct Refine8 {
  double lo, hi, tol, est;
  int s_lo, stage, round;

  // U: the state is held in scalar registers between rounds.
  static __device__ __forceinline__ double uni(double v) { return U ? from_lane<U>(v, 0) : v; }

  __device__ __forceinline__ void init(double lo_, double hi_, double refine_rel) {
    lo = uni(lo_);
    hi = uni(hi_);
    tol = uni(refine_rel * hi);
    est = lo;
    s_lo = stage = round = 0;
  }

  // This round's point of lane `sub` of the eight.
  __device__ __forceinline__ double point(int sub) const {
    const double w = hi - lo;
    if (stage == 0) return sub == 7 ? hi : __builtin_fma(w, double(sub) * (1.0 / 7.0), lo);
    if (stage == 2) return __builtin_fma(w, double(sub + 1) * (1.0 / 9.0), lo);
    const int rung = (sub & 4) ? (sub & 3) : 3 - (sub & 3);
    const double off = tol * (rung == 0 ? 0.45 : rung == 1 ? 16.0 : rung == 2 ? 2048.0 : 524288.0);
    return __builtin_fmin(__builtin_fmax((sub & 4) ? est + off : est - off, lo), hi);
  }

  // Takes in the round's signs and values; `base` is the eight lanes' first.
  // True when the bracket is final.
  __device__ __forceinline__ bool update(double c, int sg, double m, int e, int base) {
    if (stage == 0) s_lo = from_lane<U>(sg, base);
    const unsigned diff = unsigned(__ballot(sg != s_lo) >> base) & 0xffu;
    const int f = diff ? __ffs(int(diff)) - 1 : 8;  // first point whose sign differs from lo's
    const int lf = base + min(f, 7), lb = base + max(f - 1, 0);
    if (s_lo == kNaNSign || (f < 8 && from_lane<U>(sg, lf) == kNaNSign)) return true;
    if (stage == 0 && f == 8) return true;
    const double w = hi - lo;
    if (f > 0) lo = from_lane<U>(c, lb);
    if (f < 8) hi = from_lane<U>(c, lf);
    if (hi - lo <= tol || ++round >= kMaxRefineRounds) return true;
    if (stage == 1 && (hi - lo > 0.125 * w || f == 0 || f == 8)) {
      stage = 2;
    } else {
      est = uni(root_estimate<U>(c, m, e, base + min(max(f - 2, 0), 4), base + min(max(f - 1, 0), 6),
                                 stage == 0 ? base : -1, tol));
      stage = 1;
    }
    return false;
  }
};

// Whether the signs of 64 points that rise through lanes 0, 8..15, 1, 16..23,
// 2, ..., 56..63, 7 are those of one change: `differ` has the lanes whose sign
// differs from the first point's.
__device__ __forceinline__ bool one_change(unsigned long long differ) {
  const unsigned long long a = differ & 0xffull, b = differ >> 8;
  const int f = a ? __ffsll((long long)a) - 1 : 8, t = b ? __ffsll((long long)b) - 1 : 56;
  // both rise once, and the first of the 56 lies in the eight's interval f - 1
  return f >= 1 && f < 8 && (a >> f) + 1ull == 1ull << (8 - f) && (b >> t) + 1ull == 1ull << (56 - t) &&
         t >= 8 * (f - 1) && t <= 8 * f;
}

// Status, refined root and outputs of the pick at grid index `found`, whose
// determinant signs are sig_f there and prev_f at found - 1.  Run by one whole
// wavefront, whose lane 0 stores the outputs.  The first round takes 64 equally
// spaced points of the step: the eight of a Refine8 in lanes 0..7 and the 56
// between them, in order, in lanes 8..63.  It yields the layer-denominator sign
// masks at the two grid points (pole flag), and where the masks of all its
// points are the same and the sign changes once, the refinement goes on with
// the eight.  Otherwise (a pole in the step, perhaps with zeros beside it, or
// several zeros) multisection of the whole step takes its place: 64 increasing
// points per round, one per lane, lanes 0 and 63 at the bracket's ends; the new
// bracket is the first sign change.  A uniform round (63 equal parts) is
// followed by at most one window round: linear interpolation of det K (of
// 1/det K at a pole) between the new bracket's ends estimates the root, and
// lanes 1..62 are placed 0.9 tol apart around the estimate.
// Returns the determinant evaluations made (64 in the first round and in those
// of the multisection, else 8).
// With `confirm` the signs are a sweep's (masw_secular.hpp), and the
// determinant's own at the two grid points, which the first round evaluates,
// have the last word: kUnconfirmed is added, and nothing written, where they
// show no change.
constexpr unsigned long long kUnconfirmed = 1ull << 63;
__device__ __forceinline__ unsigned long long refine_and_write(const ItemOut& o, const double* c64, double k64,
                                                               const LayerRec64* L64, int N, int found, int sig_f,
                                                               int prev_f, bool confirm = false) {
  constexpr int kUniform64 = 3, kWindow64 = 4;  // stages of the multisection
  const int lane = threadIdx.x & 63;
  unsigned long long evals = 0;
  int status = MASW_STATUS_FOUND;
  if (!confirm && (sig_f == kNaNSign || prev_f == kNaNSign)) status = MASW_STATUS_NAN;
  double c_ref = __builtin_nan("");
  if (status == MASW_STATUS_FOUND) {
    Refine8<true> r;
    r.init(c64[found - 1], c64[found], o.refine_rel);
    for (int k = 0; k < kMaxRefineRounds; ++k) {
      // (the lane number is opaque to the compiler here: what follows from it
      // would otherwise be held in registers across the loop over layers)
      int lane = threadIdx.x & 63;
      asm volatile("" : "+v"(lane));
      double c;
      if (k == 0) {
        // (n, of 63 equal parts; every ninth is one of the eight, and rounded as it is)
        const int n = lane - 7 + (lane >> 3) - 1;
        c = lane < 8 ? r.point(lane) : __builtin_fma(r.hi - r.lo, double(n) * (1.0 / 63.0), r.lo);
      } else if (r.stage < kUniform64) {
        c = r.point(lane & 7);
      } else if (r.stage == kWindow64) {
        const double step = 0.9 * r.tol;  // window spacing
        const double a = __builtin_fmin(__builtin_fmax(r.est - 30.5 * step, r.lo + 0.5 * step), r.hi - 61.5 * step);
        c = (lane == 0) ? r.lo : (lane == 63) ? r.hi : a + double(lane - 1) * step;
      } else {
        c = (lane == 63) ? r.hi : r.lo + (r.hi - r.lo) * (double(lane) / 63.0);
      }
      uint64_t dm = 0;
      double mant;
      int expo;
      const int sg = det_sign_value(c, k64, L64, N, &dm, &mant, &expo);
      int s_c = 0, p_c = 0, unused;
      if (r.stage < kUniform64) {
        evals += k == 0 ? 64ull : 8ull;
        if (k == 0) {
          if (confirm) {
            const int s_lo = from_lane<true>(sg, 0), s_hi = from_lane<true>(sg, 7);
            if (s_lo == s_hi || s_lo == kNaNSign || s_hi == kNaNSign) return evals + kUnconfirmed;
          }
          const uint64_t dm_lo = (uint64_t(uint32_t(from_lane<true>(int(uint32_t(dm >> 32)), 0))) << 32) |
                                 uint32_t(from_lane<true>(int(uint32_t(dm)), 0));
          const unsigned long long other = __ballot(dm != dm_lo);
          if (other >> 7 & 1ull) status |= MASW_FLAG_POLE;
          if (!o.refine) break;
          const int s_first = from_lane<true>(sg, 0);
          if (other != 0ull || __ballot(sg == kNaNSign) != 0ull || !one_change(__ballot(sg != s_first))) {
            r.stage = kUniform64;
            continue;
          }
        }
        if (r.update(c, sg, mant, expo, 0)) break;
        continue;
      }
      const int f = wave_first_change(sg, &s_c, &p_c, &unused);
      evals += 64ull;
      if (f < 0 || s_c == kNaNSign || p_c == kNaNSign) break;
      const double lo = from_lane<true>(c, f - 1), hi = from_lane<true>(c, f);
      const bool uniform = r.stage == kUniform64;
      r.lo = lo;
      r.hi = hi;
      r.stage = kUniform64;
      if (hi - lo <= r.tol) break;
      if (uniform) {  // an estimate from the values at the new bracket's ends
        const bool pole = (status & MASW_FLAG_POLE) != 0;
        const double ma = from_lane<true>(mant, f - 1), mb = from_lane<true>(mant, f);
        const int ea = from_lane<true>(expo, f - 1), eb = from_lane<true>(expo, f);
        if (ma * mb < 0.0) {  // finite, nonzero, opposite signs
          // q = v_b / v_a for a zero, v_a / v_b for a pole; q < 0 and the
          // estimate is lo + (hi - lo) / (1 - q)
          const int de = max(-1000, min(1000, pole ? ea - eb : eb - ea));
          const double q = __builtin_ldexp(pole ? ma / mb : mb / ma, de);
          const double t = 1.0 / (1.0 - q);
          if (t > 0.0 && t < 1.0) {
            r.est = r.uni(lo + (hi - lo) * t);
            if (62.0 * (0.9 * r.tol) < hi - lo) r.stage = kWindow64;
          }
        }
      }
    }
    if (o.refine) c_ref = 0.5 * (r.lo + r.hi);
  }
  if (lane == 0) {
    *o.idx = found;
    *o.status = status;
    *o.ct = c64[found];
    if (o.cref) *o.cref = c_ref;
  }
  return evals;
}

}  // namespace masw
