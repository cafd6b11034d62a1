// The inertia-count search as a launch of its own (MASW_SEARCH_INERTIA on the
// curve and batch calls): the kernels, compiled by two translation units.
// masw_inertia.hip builds the variant for many wavelengths per SIMD (FP64
// polynomial coefficients materialised in SGPRs where used, four wavefronts
// per SIMD: MASW_COEFF_POLICY 1); masw_inertia_lone.hip builds the variant
// for launches of at most one wavefront per SIMD, with every coefficient in
// VGPRs (MASW_COEFF_POLICY 2), where scalar moves would take issue slots from
// the lone wavefront's vector instructions.
//
// Work split.  S lanes per wavelength, 64 / S wavelengths of one model per
// wavefront at a time, each at its own stage: a round is one elimination of K
// per lane, at the point its wavelength's stage asks for.  With many
// wavelengths S = 8: what counts there is the evaluations per wavelength, and
// eight points narrow a bracket 7 times for 8 evaluations where 64 narrow it
// 63 times for 64.  With at most one wavefront per SIMD the rounds count, and
// S is the largest of 64, 32 and 8 that leaves it about so (launch_inertia).
//
// The usual case is E(c_test[0]) = 0 (no mode and no pole below the grid).  E
// is never negative and never decreases, so E(c) = 0 at a point proves that
// sign(det K) is constant up to it, and it rarely takes sublayers: the pivots
// of K(c) are positive definite and every layer is below its energy bound
// (masw_inertia.hpp).  A wavelength's stages:
//   First:  c_test[0], and S - 1 points: around the pick that the previous
//           wavelengths of the group's run extrapolate to, or spread over the
//           grid.
//   Narrow: S spread points of the bracket [lo, hi], E(lo) = 0, E(hi) != 0.
//   Try:    where the points are at most kTrySpacing grid steps apart, inverse
//           cubic interpolation of det K names the grid step of the change.
//           Round 0 of the refinement (masw_pick.hpp) is evaluated on it (on
//           the S / 8 steps around it): its first and last points are the
//           step's ends, so E = 0 at the one and E = 1 at the other settle the
//           pick, prove that the step holds a single root and no pole, and start
//           its refinement at once.  Otherwise they narrow the bracket.
//   Refine: the further rounds of the refinement, then the outputs.
// So a wavelength whose pick is predicted takes three rounds of eight: 24
// evaluations, where 64 lanes a wavelength took about 65 counts and 128
// evaluations of the refinement.
//
// A wavelength is left to the search of masw_inertia.hpp by a whole wavefront
// where E(c_test[0]) is not 0, the grid step of the change holds a pole or
// several roots, or its upper end is at or above the half-space's S
// velocity.  With S = 64 or 32 the wavefront runs it at once;
// else a second launch does (deferred picks: idx = kDeferredIdx in between),
// so that many of one wavefront's are shared out.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "masw.h"
#include "masw_host.hpp"
#include "masw_inertia.hpp"
#include "masw_internal.hpp"

namespace masw {
namespace {

using inertia::Tally;
using inertia::wave_sum;

constexpr int kDeferredIdx = -0x4d;     // idx of a deferred wavelength between the two launches
constexpr int kTrySpacing = 100;        // grid steps between points, at most, for the Try stage

__device__ __forceinline__ ItemOut item_out(const SweepArgs& a, int g) {
  return ItemOut{a.out_ct + g, a.out_idx + g, a.out_status + g, a.out_cref ? a.out_cref + g : nullptr, a.refine,
                 a.refine_rel};
}

// One wavelength by a whole wavefront: search, refinement and outputs.
__device__ __forceinline__ void run_wavelength(const SweepArgs& a, int g, Tally& t) {
  const int m = __builtin_amdgcn_readfirstlane(a.lam_model[g]);
  const ModelDesc d = a.models[m];
  const ItemOut o = item_out(a, g);
  const double k = a.lam_k[g];
  const int n_c = __builtin_amdgcn_readfirstlane(d.n_c);
  const int N = __builtin_amdgcn_readfirstlane(d.n_layers);
  const double* c64 = a.c64 + __builtin_amdgcn_readfirstlane(d.c_base);
  const LayerRec64* L = a.layers64 + __builtin_amdgcn_readfirstlane(d.layer_base);
  int sig_f = 0, prev_f = 0;
  const int found = inertia::search(c64, n_c, k, L, N, &sig_f, &prev_f, t);
  unsigned long long refined = 0;
  if (found < 0)
    write_no_pick(o, MASW_STATUS_NOT_FOUND, (threadIdx.x & 63) == 0);
  else
    refined = refine_and_write(o, c64, k, L, N, found, sig_f, prev_f);
  t.useful += (unsigned long long)(found < 0 ? n_c : found + 1);
  t.refine += refined;
}

// One grid or refinement point: det_sign's sign and value m 2^e, whether
// E(c) = 0 and, where `ask`, whether E(c) = 1 (inertia::count_E; an event is
// neither).  With COUNT, E(c) itself (kEvent where it has none) and the poles
// counted in it, both only where `ask`.
struct Point {
  double m;
  int e, sg;
  bool zero, one;
  int E, P;
};

template <bool COUNT>
__device__ __forceinline__ Point eval_point(double c, double k, const LayerRec64* __restrict__ L, int N,
                                            bool ask) {
  const double c2 = c * c;
  Block2<double> S{0.0, 0.0, 0.0};
  // (what is tracked over the layers is one mask and otherwise vector registers:
  // masks that do not fit the scalar registers are moved at every layer)
  int odd = 0;             // negative pivot determinants
  bool good = true;        // no pivot with both eigenvalues negative
  int s = 0;               // COUNT: negative eigenvalues
  double x_min = 1.0;      // smallest (k h)^2 (1 - c^2/beta^2)
  Point o;
  double m = 1.0;
  int e = 0;
  auto pivot = [&](double a, double d) {  // (1,1) entry and determinant
    odd += d < 0.0 ? 1 : 0;
    if constexpr (COUNT) s += inertia::neg_eigs(a, d);
    else good = good && (a > 0.0 || d < 0.0);
  };
  LayerRec<double> nxt = load_rec<double>(L, 0);
  for (int j = 0; j < N; ++j) {
    const LayerRec<double> rec = nxt;
    nxt = load_rec<double>(L, j + 1);  // one layer ahead; after the last layer, the half-space
    const double kh = k * rec.h;
    const LayerK<double> K = layer_entries<double>(c2, kh, rec.ia2, rec.ib2, rec.rh, rec.mh);
    const double a = S.s11 + K.k11;
    const double d = schur_layer<double>(S, K);
    pivot(a, d);
    x_min = __builtin_fmin(x_min, kh * kh * (1.0 - c2 * rec.ib2));
    int ex;
    m = __builtin_frexp(m * d, &ex);
    e += ex;
  }
  const LayerRec<double> hs = nxt;
  double re, im, ar;
  halfspace_det<double>(S, c2, hs.ia2, hs.ib2, hs.mh, &re, &im, &ar);
  o.sg = sign_code((odd & 1) != 0, re);
  pivot(ar, re);
  int ex;
  o.m = __builtin_frexp(m * re, &ex);
  o.e = e + ex;
  // (a pivot's determinant that is zero or not finite stays in the product)
  good = good && o.m != 0.0 && __builtin_fabs(o.m) < __builtin_inf() && c2 * hs.ib2 < 1.0;
  // layer_poles' bound k h sqrt(c^2/beta^2 - 1) < pi, with det_sign_inertia's margin
  const bool bounded = x_min > -9.86;
  if constexpr (!COUNT) s = odd;
  // rare: a layer above its energy bound, whose sublayers have to be counted
  int P = 0;
  const bool count = good && !bounded && (COUNT ? ask : s == 0 || (ask && s == 1));
  if (__ballot(count) != 0ull && count) P = inertia::poles_below(c, k, L, N, &good);
  good = good && (bounded || count);
  o.P = P;
  o.E = good ? s + 2 * P : inertia::kEvent;
  o.zero = o.E == 0;
  o.one = o.E == 1;
  return o;
}

enum Stage { kFirst = 0, kNarrow = 1, kTry = 2, kRefine = 3 };

// Work of one wavefront in rounds (uniform): lanes that evaluated a point of
// the search, or of the refinement, and the layers they eliminated.
struct Rounds {
  unsigned long long evals = 0, entries = 0, refine = 0;
};

// Runs the wavelengths [begin, end) of one model, 64 / S at a time, each
// group of S lanes a run of consecutive ones.  Deferred wavelengths are
// marked in out_idx.  Per-lane variables are the same in a group's lanes.
template <int S>
__device__ __forceinline__ void run_groups(const SweepArgs& a, int begin, int end, const ModelDesc& d, Rounds& rounds,
                           unsigned long long& useful, unsigned& deferred) {
  constexpr int kGroups = 64 / S;
  const int lane = threadIdx.x & 63, sub = lane & (S - 1), base = lane & ~(S - 1);
  const int N = __builtin_amdgcn_readfirstlane(d.n_layers), n_c = __builtin_amdgcn_readfirstlane(d.n_c);
  const double* c64 = a.c64 + __builtin_amdgcn_readfirstlane(d.c_base);
  const LayerRec64* L = a.layers64 + __builtin_amdgcn_readfirstlane(d.layer_base);
  const int per = (end - begin + kGroups - 1) / kGroups;
  int g = begin + (lane / S) * per;
  const int g_end = min(g + per, end);
  auto in_group = [&](bool p) -> unsigned long long {  // this group's lanes with p, lane `base` as bit 0
    const unsigned long long b = __ballot(p) >> base;
    return S == 64 ? b : b & ((1ull << (S & 63)) - 1ull);
  };

  double k = 0.0;
  int stage = kFirst, lo = 0, hi = n_c;  // E(lo) = 0; E(hi) != 0, or hi = n_c (not known to change)
  int at = 0;                              // the grid step (at - 1, at] that Try looks at
  int pred = -1, win = 0, p1 = -1, p2 = -1;  // prediction, its window's spacing; the run's last picks
  constexpr bool U = S == 64;  // one wavelength: every value of its stage is uniform
  Refine8<U> r;
  r.init(0.0, 0.0, 0.0);
  bool fresh = true, live = g < g_end;
  while (__ballot(live) != 0ull) {
    if constexpr (U) {  // one wavelength: branches and addresses by scalar values
      stage = __builtin_amdgcn_readfirstlane(stage);
      lo = __builtin_amdgcn_readfirstlane(lo);
      hi = __builtin_amdgcn_readfirstlane(hi);
      at = __builtin_amdgcn_readfirstlane(at);
      g = __builtin_amdgcn_readfirstlane(g);
      fresh = __ballot(fresh) != 0ull;
      live = true;
    }
    if (fresh && live) {
      k = a.lam_k[g];
      stage = kFirst;
      lo = 0;
      hi = n_c;
      pred = -1;
      // two earlier picks: their line; one: its own pick, in a wide window.
      // The spacing follows the last prediction's error, and the window has
      // to fit the grid.
      if (S < 64 && p1 >= 1) {
        win = p2 >= 1 ? max(8, min(96, win)) : 96;
        if ((S - 2) * win < n_c - 1) pred = p2 >= 1 ? 2 * p1 - p2 : p1;
      }
      fresh = false;
    }
    // this round's grid point p (First, Narrow), or, in Try, the grid step
    // (p - 1, p] that these eight lanes look at, `at` among the group's S / 8
    int p = 0;
    bool valid = true;
    if (stage == kFirst && sub > 0) {
      if (S < 64 && pred >= 0)
        p = min(max(pred - (S / 2 - 1) * win, 1), n_c - 1 - (S - 2) * win) + (sub - 1) * win;
      else
        p = inertia::spread(0, n_c - 1, sub, 1, &valid, S);
    } else if (stage == kNarrow) {
      // S spread points from lo to hi, both again (all points, if no more),
      // so that the change is always between two of them
      const int w = min(hi, n_c - 1) - lo;
      valid = w >= S || sub <= w;
      p = w >= S ? lo + int((int64_t(w) * sub) / (S - 1)) : lo + sub;
    }
    if (!valid) p = 0;
    if (stage == kTry) p = min(max(at - (S / 8 - 1) / 2 + (sub >> 3), lo + 1), min(hi, n_c - 1));
    double c;
    if (stage == kRefine) {
      c = r.point(sub & 7);
    } else {
      c = c64[p];
      if (stage == kTry && (sub & 7) != 7) {  // Refine8's round 0
        const double c_b = c64[p - 1];
        c = __builtin_fma(c - c_b, double(sub & 7) * (1.0 / 7.0), c_b);
      }
    }
    const Point v = eval_point<false>(c, k, L, N, live && stage == kTry && (sub & 7) == 7);
    const unsigned n_search = __popcll(__ballot(live && stage < kRefine && valid));
    rounds.evals += n_search;
    rounds.entries += (unsigned long long)n_search * unsigned(N);
    rounds.refine += __popcll(__ballot(live && stage == kRefine && sub < 8));

    // the search stages' outcome: next stage, or a wavelength's end
    int end_as = 0;  // 1: no pick, 2: deferred, 3: picked
    bool located = false;
    int eight = base;  // the first of the eight lanes that refine
    const unsigned long long above = in_group(valid && !v.zero);
    if (live && stage <= kNarrow) {
      const int f = above ? __ffsll((long long)above) - 1 : S;  // first point with E != 0
      const int last = 63 - __clzll((long long)in_group(valid));  // (lane 0 always has a point)
      const int b = min(f - 1, last);                              // the point before it
      const int p_f = from_lane<U>(p, base + min(f, S - 1)), p_b = from_lane<U>(p, base + max(b, 0));
      if (f == 0) end_as = 2;  // E(c_test[0]) is not 0
      if (f < S) hi = p_f;
      lo = p_b;
      bool can_try = f < S && last >= 3 && p_f - p_b <= kTrySpacing;
      // Lone wavefronts, whose time is their rounds': where the points are
      // further apart than 1% of c the cubic often misses the step, and one
      // more Narrow round names it for certain (60 wavelengths x 1901
      // velocities over 25 layers: 86.9 us without this, 74.2 with it).
      if (S >= 32) {
        const double c_f = from_lane<U>(c, base + min(f, S - 1)), c_b = from_lane<U>(c, base + max(b, 0));
        can_try = can_try && c_f - c_b <= 0.01 * c_f;
      }
      double x = 0.0;
      if (__ballot(can_try) != 0ull)
        x = root_estimate<U>(double(p), v.m, v.e, base + max(0, min(f - 2, last - 3)),
                             base + min(max(f - 1, 0), S - 2));
      stage = kNarrow;
      if (hi - lo == 1) {
        if (hi == n_c) end_as = end_as ? end_as : 1;                   // E = 0 at the last grid point
        stage = kTry;
        at = hi;
      } else if (can_try) {
        stage = kTry;
        at = max(lo + 1, min(hi, int(x) + 1));
      }
    } else if (live && stage == kTry) {
      // E rises along the lanes, so the first lane with E != 0 names its step
      const int f = above ? __ffsll((long long)above) - 1 : -1;
      const int first_step = from_lane<U>(p, base), last_step = from_lane<U>(p, base + S - 1);
      if (f == 0) {
        hi = first_step - 1;
      } else if (f < 0) {
        lo = last_step;
      } else {
        const int q = base + (f & ~7);  // its step's eight lanes
        const double c_lo = from_lane<U>(c, q), c_hi = from_lane<U>(c, q + 7);
        hi = from_lane<U>(p, q);
        // E = 0 and E = 1 at the step's ends: a mode lies between them and nothing else
        if ((f & 7) == 0 || (in_group(v.one) >> (f & ~7) & 0x80ull) == 0ull) {
          end_as = 2;
        } else {
          located = true;
          eight = q;
          r.init(c_lo, c_hi, a.refine_rel);
        }
      }
      if (!located && end_as == 0) {
        stage = kNarrow;
        if (hi - lo == 1) {
          if (hi == n_c) end_as = 1;
          stage = kTry;
          at = hi;
        }
      }
    }
    // the refinement's rounds (Try's points are its first)
    if (live && (located || stage == kRefine)) {
      const bool final = r.update(c, v.sg, v.m, v.e, eight);
      stage = kRefine;
      if (final || !a.refine) end_as = 3;
    }
    if (live && !(k == k)) end_as = 4;  // invalid model, grid or wavelength
    if (live && end_as != 0) {
      const ItemOut o = item_out(a, g);
      if (end_as == 3) {
        if (sub == 0) {
          *o.idx = hi;
          *o.status = MASW_STATUS_FOUND;
          *o.ct = c64[hi];
          if (o.cref) *o.cref = o.refine ? 0.5 * (r.lo + r.hi) : __builtin_nan("");
          useful += unsigned(hi + 1);
        }
        p2 = p1;
        p1 = hi;
        if (pred >= 0) win = abs(hi - pred);
      } else {
        if (end_as == 2) {
          if (sub == 0) *o.idx = kDeferredIdx;
          ++deferred;
        } else {
          write_no_pick(o, end_as == 1 ? MASW_STATUS_NOT_FOUND : MASW_STATUS_INVALID, sub == 0);
          if (end_as == 1 && sub == 0) useful += unsigned(n_c);
        }
        p1 = p2 = -1;
      }
      ++g;
      stage = kFirst;  // (a group that has ended goes on evaluating points of the grid)
      fresh = true;
      live = g < g_end;
    }
  }
}

// A wavefront's counts into its workgroup's row of a.wg_counts, or (wg_counts
// null) onto the call's counters.  Called by every wavefront of a workgroup.
__device__ __forceinline__ void flush_tally(const SweepArgs& a, const Rounds& rounds, const Tally& t, unsigned long long useful,
                            unsigned long long (*s_cnt)[7]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned long long evals = wave_sum(t.evals) + rounds.evals,
                           entries = wave_sum(t.entries) + rounds.entries,
                           pivots = wave_sum(t.pivots) + rounds.entries + rounds.evals, use = wave_sum(useful);
  if (lane == 0) {
    s_cnt[wave][0] = evals;
    s_cnt[wave][1] = entries;
    s_cnt[wave][2] = pivots;
    s_cnt[wave][3] = t.scan;
    s_cnt[wave][4] = t.check;
    s_cnt[wave][5] = t.refine + rounds.refine;
    s_cnt[wave][6] = t.useful + use;
  }
  __syncthreads();
  if (threadIdx.x < 8) {
    unsigned long long sum = 0;
    if (threadIdx.x < 7)
      for (int w = 0; w < kInertiaWaves; ++w) sum += s_cnt[w][threadIdx.x];
    constexpr int kCol[8] = {5, 6, 7, 0, 1, 2, 3, 4};  // s_cnt order to the row's
    if (a.wg_counts) {
      a.wg_counts[size_t(blockIdx.x) * kWgCounts + kCol[threadIdx.x]] = sum;
    } else if (sum) {
      Counters* c = a.counters;
      unsigned long long* dst[8] = {&c->inertia_evals, &c->inertia_entries, &c->inertia_pivots, &c->sweep,
                                    &c->check,         &c->refine,          &c->useful,          &c->helper};
      atomicAdd(dst[threadIdx.x], sum);
    }
  }
}

}  // namespace

// The lone-wavefront variant's launch (masw_inertia_lone.hip), S lanes per
// wavelength; *deferring is true where it may leave wavelengths deferred.
hipError_t launch_inertia_lone(const SweepArgs& a, int S, hipStream_t s, int* blocks_out, bool* deferring);

}  // namespace masw
