// Zero/pole classification of determinant sign changes with an independent
// secular function.
//
// sign(det K) of the stiffness formulation (Section 2.1) changes at the zeros
// of the dispersion function and at the poles where some layer denominator
// D_j changes sign.  This kernel evaluates the dispersion function in a
// formulation with no denominators, the Haskell-Thomson propagator of the
// P-SV equations of motion, and shares no arithmetic with the stiffness path.
//
// State and system.  For v = (u_x, -i u_z, tau_xz / (k mu_ref),
// -i tau_zz / (k mu_ref)) and zeta = k z (z down), a layer obeys
// dv/dzeta = A v with a real 4x4 matrix A (entries in `system_matrix` below)
// whose eigenvalues are +-r, +-s (u = r^2 = 1 - c^2/alpha^2,
// w = s^2 = 1 - c^2/beta^2); mu_ref is the half-space's rho beta^2.
//
// Propagator.  A^2 has the two eigenvalues u and w, so every even function of
// A is a first-degree polynomial in A^2 and every odd one is A times such a
// polynomial (Cayley-Hamilton).  With U = t^2 u, W = t^2 w and the divided
// differences of the entire functions cosh(t sqrt(z)) and
// sinh(t sqrt(z)) / sqrt(z) at z = u, w:
//     exp(-A t) = cosh(A t) - sinh(A t) = a0 I + a1 A^2 - b0 A - b1 A^3,
//     a1 = t^2 sum_{n>=1} h_{n-1} / (2n)!,   a0 = 1 - U W sum_{n>=2} h_{n-2} / (2n)!,
//     b1 = t^3 sum_{n>=1} h_{n-1} / (2n+1)!, b0 = t (1 - U W sum_{n>=2} h_{n-2} / (2n+1)!),
// where h_n = sum_{i=0}^{n} U^i W^(n-i) (h_0 = 1, h_n = U h_{n-1} + W^n).
// Nothing here divides by u - w, and every quantity is real for real c on
// either side of alpha and beta.  Steps satisfy t max(|u|, |w|)^(1/2) <= 1,
// so |U|, |W| <= 1 and twelve terms reach the FP64 rounding.
//
// Secular function.  The half-space's solutions decaying with depth (c below
// its beta) are P = (1, r, -2r, g - 2) and SV = (s, 1, g - 2, -2s),
// g = c^2/beta^2.  The pair is carried up across every layer by exp(-A k h)
// in equal steps of at most one unit of k dz max(|r|, |s|), and after each
// step replaced by a nearly orthonormal basis of its span with the same
// orientation (Gram-Schmidt: both columns divided by positive numbers).  At
// the surface F = the determinant of its two traction rows, which vanishes
// exactly at the modes; the positive factors dropped by the
// orthonormalisation leave its sign and zeros unchanged.
//
// Work split.  Eight lanes per wavelength, eight wavelengths per wavefront,
// four wavefronts per workgroup.  The eight lanes evaluate F at eight points
// at once: first at both ends of the bracket and six equally spaced points
// between them (a different sign at the two ends is a mode), then at points
// around the root that the degree-7 polynomial through those values gives,
// two of them 0.9 tol apart, tol = 1e-12 c_test[idx], and six on a widening
// ladder on both sides.  The first point whose sign differs from the lower
// end's gives the next bracket, so a root estimate good to half of tol ends
// the search in two rounds, 16 evaluations, and an estimate off by a rung or
// two narrows the bracket to that rung, with linear interpolation for the
// next round.  A root beyond the ladder, or not reached in kMaxRounds (a grid
// step of many m/s), and a step in which the polynomial has several roots, are
// deferred to a second launch, in which a whole wavefront multisects with 64
// points a round, so that of several roots it finds the first that 64 points
// show.
// For the interpolation F is the analytic dispersion function: the
// orthonormalisations' divisors are multiplied back in, and each layer is cut
// into the same number of steps at every point of a bracket (the larger of
// the two ends' needs).
// Bound by the vector ALU (67% busy; the rest is the end of the launch and
// the latency of three wavefronts a SIMD): what counts is the evaluations
// per pick.  141,745 picks of 512 models (3 to 30 layers, grid 0.05 m/s): 16.0
// evaluations a pick and 0.75 ms, against 320 and 8.9 ms with 64 lanes a pick
// multisecting 63-fold.  Without the divisors multiplied back, 0.4% of the
// picks left the ladder and the second launch alone took 0.38 ms.
// Control flow is uniform across the wavefront but for the layer and step
// loops, where lanes of other models or step counts drop out; finished groups
// go on evaluating until all are done.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "masw.h"
#include "masw_host.hpp"

namespace masw {
namespace {

constexpr int kClassifyWaves = 4;           // wavefronts per workgroup
constexpr int kGroup = 8;                   // lanes per wavelength
constexpr int kGroups = 64 / kGroup;        // wavelengths per wavefront
constexpr int kMaxStepsPerLayer = 1 << 16;  // beyond this a layer is not crossed
constexpr int kMaxRounds = 4;               // of a pick's eight lanes, before it is deferred
constexpr int kMaxWideRounds = 8;           // of a deferred pick's 64 lanes: 63^8 > 2e14
constexpr int kTerms = 12;                  // series terms, |U|, |W| <= 1
constexpr double kRootTol = 1e-12;

// The doubles nearest to 1/m!, m = 0 .. 2 kTerms + 1.
__constant__ double kInvFact[2 * kTerms + 2] = {
    1.0, 1.0, 0.5, 0.16666666666666666, 0.041666666666666664,
    0.008333333333333333, 0.001388888888888889, 0.0001984126984126984, 2.48015873015873e-05, 2.7557319223985893e-06,
    2.755731922398589e-07, 2.505210838544172e-08, 2.08767569878681e-09, 1.6059043836821613e-10, 1.1470745597729725e-11,
    7.647163731819816e-13, 4.779477332387385e-14, 2.8114572543455206e-15, 1.5619206968586225e-16, 8.22063524662433e-18,
    4.110317623312165e-19, 1.9572941063391263e-20, 8.896791392450574e-22, 3.868170170630684e-23, 1.6117375710961184e-24,
    6.446950284384474e-26};

struct ClassifyArgsDev {
  const int32_t* layer_off;
  const double* h;
  const double* alpha;
  const double* beta;
  const double* rho;
  const int32_t* lambda_off;
  const double* lambda;
  const double* c;
  const int32_t* idx;
  int32_t* cls;
  double* c_sec;
  unsigned long long* counters;  // [3]: evaluations, layers crossed, steps
  int64_t n_lam;
  int32_t n_models;
  int32_t n_c;
};

__device__ __forceinline__ bool finite_pos(double v) { return v > 0.0 && v < __builtin_inf(); }

// The six entries of A other than the constants A[0,1] = 1, A[3,2] = -1 (see
// the file comment for the state; every other entry is 0), from the layer's
// M = rho alpha^2, mu = rho beta^2, their reciprocals, rho c^2 and 1/mu_ref.
struct SysMat {
  double a02, a10, a13, a20, a23, a31;
};

__device__ __forceinline__ SysMat system_matrix(double M, double mu, double iM, double imu, double rc2,
                                              double mu_ref, double i_ref) {
  const double lam = M - 2.0 * mu;
  SysMat o;
  o.a02 = mu_ref * imu;
  o.a10 = -lam * iM;
  o.a13 = mu_ref * iM;
  o.a20 = (4.0 * mu * (lam + mu) * iM - rc2) * i_ref;
  o.a23 = lam * iM;
  o.a31 = -rc2 * i_ref;
  return o;
}

// exp(-A t) for one step (file comment), given u = r^2, w = s^2, row-major.
// A couples E = (u_x, tau_zz) only with O = (u_z, tau_xz): in that order
// A = [[0, X], [Y, 0]] with X = [[1, a02], [a31, -1]], Y = [[a10, a13],
// [a20, a23]], so A^2 = diag(XY, YX) and A^3 = [[0, XYX], [YXY, 0]], and
// exp(-A t) = [[a0 I + a1 XY, -(b0 X + b1 XYX)], [-(b0 Y + b1 YXY), a0 I + a1 YX]].
__device__ __forceinline__ void step_propagator(const SysMat& m, double u, double w, double t, double P[16]) {
  const double U = t * t * u, W = t * t * w;
  double sc1 = 0.0, ss1 = 0.0, sc0 = 0.0, ss0 = 0.0;
  double h_prev = 0.0, h_cur = 1.0, Wp = 1.0;  // h_{n-2}, h_{n-1}
#pragma unroll
  for (int n = 1; n <= kTerms; ++n) {
    sc1 = __builtin_fma(h_cur, kInvFact[2 * n], sc1);
    ss1 = __builtin_fma(h_cur, kInvFact[2 * n + 1], ss1);
    if (n >= 2) {
      sc0 = __builtin_fma(h_prev, kInvFact[2 * n], sc0);
      ss0 = __builtin_fma(h_prev, kInvFact[2 * n + 1], ss0);
    }
    Wp *= W;
    const double h_next = __builtin_fma(U, h_cur, Wp);
    h_prev = h_cur;
    h_cur = h_next;
  }
  const double UW = U * W;
  const double a1 = t * t * sc1;
  const double a0 = 1.0 - UW * sc0;
  const double b1 = t * t * t * ss1;
  const double b0 = t * (1.0 - UW * ss0);
  // XY and YX (rows/columns in E and O order)
  const double xy00 = __builtin_fma(m.a02, m.a20, m.a10), xy01 = __builtin_fma(m.a02, m.a23, m.a13);
  const double xy10 = __builtin_fma(m.a31, m.a10, -m.a20), xy11 = __builtin_fma(m.a31, m.a13, -m.a23);
  const double yx00 = __builtin_fma(m.a13, m.a31, m.a10), yx01 = __builtin_fma(m.a10, m.a02, -m.a13);
  const double yx10 = __builtin_fma(m.a23, m.a31, m.a20), yx11 = __builtin_fma(m.a20, m.a02, -m.a23);
  // XYX = (XY) X and YXY = (YX) Y
  const double xyx00 = __builtin_fma(xy01, m.a31, xy00), xyx01 = __builtin_fma(xy00, m.a02, -xy01);
  const double xyx10 = __builtin_fma(xy11, m.a31, xy10), xyx11 = __builtin_fma(xy10, m.a02, -xy11);
  const double yxy00 = __builtin_fma(yx01, m.a20, yx00 * m.a10), yxy01 = __builtin_fma(yx01, m.a23, yx00 * m.a13);
  const double yxy10 = __builtin_fma(yx11, m.a20, yx10 * m.a10), yxy11 = __builtin_fma(yx11, m.a23, yx10 * m.a13);
  // state index of E = (0, 3) and O = (1, 2)
  P[0 * 4 + 0] = __builtin_fma(a1, xy00, a0);
  P[0 * 4 + 3] = a1 * xy01;
  P[3 * 4 + 0] = a1 * xy10;
  P[3 * 4 + 3] = __builtin_fma(a1, xy11, a0);
  P[1 * 4 + 1] = __builtin_fma(a1, yx00, a0);
  P[1 * 4 + 2] = a1 * yx01;
  P[2 * 4 + 1] = a1 * yx10;
  P[2 * 4 + 2] = __builtin_fma(a1, yx11, a0);
  P[0 * 4 + 1] = -__builtin_fma(b1, xyx00, b0);
  P[0 * 4 + 2] = -__builtin_fma(b1, xyx01, b0 * m.a02);
  P[3 * 4 + 1] = -__builtin_fma(b1, xyx10, b0 * m.a31);
  P[3 * 4 + 2] = -__builtin_fma(b1, xyx11, -b0);
  P[1 * 4 + 0] = -__builtin_fma(b1, yxy00, b0 * m.a10);
  P[1 * 4 + 3] = -__builtin_fma(b1, yxy01, b0 * m.a13);
  P[2 * 4 + 0] = -__builtin_fma(b1, yxy10, b0 * m.a20);
  P[2 * 4 + 3] = -__builtin_fma(b1, yxy11, b0 * m.a23);
}

// 1/x: the hardware estimate (within 2^-21 relative) and one third-order step,
// r (1 + e + e^2) with e = 1 - x r.
__device__ __forceinline__ double inv(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, __builtin_fma(e, e, e), r);
}

// 1/sqrt(x): the hardware estimate (within 2^-21 relative) and one Newton step.
__device__ __forceinline__ double inv_sqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  return __builtin_fma(0.5 * y, __builtin_fma(-(x * y), y, 1.0), y);
}

// Replace the columns (x, y) by an orthonormal basis of their span with the
// same orientation: x divided by its norm, then y less its component along x
// and divided by its norm.  Returns the product of the two reciprocal norms
// (positive), by which every 2x2 minor of (x, y) is multiplied.
__device__ __forceinline__ double orthonormalize(double x[4], double y[4]) {
  const double ix = inv_sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3]);
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] *= ix;
  const double d = x[0] * y[0] + x[1] * y[1] + x[2] * y[2] + x[3] * y[3];
#pragma unroll
  for (int i = 0; i < 4; ++i) y[i] = __builtin_fma(-d, x[i], y[i]);
  const double iy = inv_sqrt(y[0] * y[0] + y[1] * y[1] + y[2] * y[2] + y[3] * y[3]);
#pragma unroll
  for (int i = 0; i < 4; ++i) y[i] *= iy;
  return ix * iy;
}

// F(c) for wavenumber k and a model of N layers over a half-space (values at
// index N); c in the bracket [sqrt(c2_lo), sqrt(c2_hi)] below the
// half-space's beta.  Each layer's step count is the larger of the two ends'
// (max(|u|, |w|) is largest at an end: both are linear in c^2).  NaN if a
// layer needs more than kMaxStepsPerLayer steps.
// The value is *mant 2^*expo: the orthonormalisations' divisors are multiplied
// back in (their exponents apart, so nothing overflows), which makes it the
// analytic dispersion function.  Without them F is +-sin of an angle between
// planes, which near a mode of a slow layer turns over within a tiny part of
// a grid step, where interpolation says nothing.
struct Secular {
  double mant;
  int expo;
};
__device__ Secular secular(double c, double c2_lo, double c2_hi, double k, const double* __restrict__ h,
                           const double* __restrict__ al, const double* __restrict__ be,
                           const double* __restrict__ rh, int N, unsigned* steps_taken) {
  const double c2 = c * c;
  const double mu_ref = rh[N] * be[N] * be[N];
  const double i_ref = 1.0 / mu_ref;
  const double g = c2 / (be[N] * be[N]);
  const double r = __builtin_sqrt(1.0 - c2 / (al[N] * al[N]));
  const double s = __builtin_sqrt(1.0 - g);
  double x[4] = {1.0, r, -2.0 * r, g - 2.0};
  double y[4] = {s, 1.0, g - 2.0, -2.0 * s};
  int expo = 0;
  double scale = __builtin_frexp(orthonormalize(x, y), &expo);  // product of reciprocal norms: scale 2^expo
  for (int j = N - 1; j >= 0; --j) {
    const double a = al[j], b = be[j], rho = rh[j];
    const double M = rho * a * a, mu = rho * b * b;
    const double iM = inv(M), imu = inv(mu);
    const double rc2 = rho * c2;
    const double u = 1.0 - rc2 * iM;   // 1 - c^2/alpha^2
    const double w = 1.0 - rc2 * imu;  // 1 - c^2/beta^2
    const double pa = rho * iM, pb = rho * imu;  // 1/alpha^2, 1/beta^2
    const double e_lo = __builtin_fmax(__builtin_fabs(1.0 - c2_lo * pa), __builtin_fabs(1.0 - c2_lo * pb));
    const double e_hi = __builtin_fmax(__builtin_fabs(1.0 - c2_hi * pa), __builtin_fabs(1.0 - c2_hi * pb));
    const double q = __builtin_sqrt(__builtin_fmax(e_lo, e_hi));
    const double kh = k * h[j];
    const double need = __builtin_ceil(kh * q);
    if (!(need <= double(kMaxStepsPerLayer))) return Secular{__builtin_nan(""), 0};
    const int steps = need < 1.0 ? 1 : int(need);
    *steps_taken += unsigned(steps);
    double P[16];
    step_propagator(system_matrix(M, mu, iM, imu, rc2, mu_ref, i_ref), u, w, kh * inv(double(steps)), P);
    for (int st = 0; st < steps; ++st) {
      double nx[4], ny[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        nx[i] = P[i * 4 + 0] * x[0] + P[i * 4 + 1] * x[1] + P[i * 4 + 2] * x[2] + P[i * 4 + 3] * x[3];
        ny[i] = P[i * 4 + 0] * y[0] + P[i * 4 + 1] * y[1] + P[i * 4 + 2] * y[2] + P[i * 4 + 3] * y[3];
      }
      int e;
      scale = __builtin_frexp(scale * orthonormalize(nx, ny), &e);
      expo += e;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[i] = nx[i];
        y[i] = ny[i];
      }
    }
  }
  return Secular{(x[2] * y[3] - y[2] * x[3]) / scale, -expo};
}

__device__ __forceinline__ int sgn(double v) { return int(v > 0.0) - int(v < 0.0); }

// Workgroups are dispatched to the eight XCDs round-robin (block b on XCD
// b mod 8), and each XCD has its own L2.  Within every run of 8 kXcdRun
// dispatched blocks, the blocks are renumbered so that each XCD takes kXcdRun
// consecutive block numbers: neighbouring wavelengths, which share a model's
// records and the output cache lines, stay in one L2, while the runs keep
// every XCD's share of the models mixed.  Blocks past the last whole run keep
// their numbers.  The renumbering is a bijection of [0, nb), so it changes no
// result.
constexpr unsigned kXcds = 8;
constexpr unsigned kXcdRun = 16;

__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned nb) {
  constexpr unsigned span = kXcds * kXcdRun;
  if (b >= nb / span * span) return b;
  const unsigned base = b / span * span, w = b % span;
  return base + (w % kXcds) * kXcdRun + w / kXcds;
}

// The model and bracket that a lane evaluates.
struct LaneWork {
  const double *h, *al, *be, *rh;
  double k, c_lo, c_hi;
  int N;
};

// Wavelength wl with bracket index i as eight lanes (`sub` the lane among them)
// see it: its model, k and bracket, and its class where no evaluation is
// needed, else -1.
__device__ int lane_work(const ClassifyArgsDev& a, int64_t wl, int i, int sub, unsigned long long group, LaneWork* o) {
  // model of wavelength wl: lambda_off[m] <= wl < lambda_off[m + 1]
  int m_lo = 0, m_hi = a.n_models;
  while (m_hi - m_lo > 1) {
    const int mid = (m_lo + m_hi) >> 1;
    if (int64_t(a.lambda_off[mid]) <= wl) m_lo = mid; else m_hi = mid;
  }
  const int m = m_lo;
  const int N = a.layer_off[m + 1] - a.layer_off[m];
  const int64_t r0 = int64_t(a.layer_off[m]) + m;
  o->h = a.h + a.layer_off[m];
  o->al = a.alpha + r0;
  o->be = a.beta + r0;
  o->rh = a.rho + r0;
  o->N = N;
  if (i < 1 || i >= a.n_c) return MASW_PICK_NONE;
  // device validation of the model, the wavelength and the bracket
  bool bad = (N < 0 || N > MASW_MAX_LAYERS);
  for (int j = sub; !bad && j <= N; j += kGroup) {
    const double aj = o->al[j], bj = o->be[j], rj = o->rh[j];
    bool ok = finite_pos(aj) && finite_pos(bj) && finite_pos(rj) && aj > bj;
    if (j < N) ok = ok && finite_pos(o->h[j]);
    bad = !ok;
  }
  const double lam = a.lambda[wl];
  o->c_lo = a.c[i - 1];
  o->c_hi = a.c[i];
  bad = bad || !finite_pos(lam) || !finite_pos(o->c_lo) || !finite_pos(o->c_hi) || !(o->c_hi > o->c_lo);
  o->k = 2.0 * 3.14159265358979323846 / lam;
  // (the eight lanes are converged here: they share wl)
  if ((__ballot(bad) & group) != 0ull) return MASW_PICK_INVALID;
  return o->c_hi >= o->be[N] ? MASW_PICK_LEAKY : -1;
}

// Root, in units of the spacing from the first point, of the polynomial
// through the group's eight values at equally spaced points, between points
// l - 1 and l where the sign changes: forward differences and secant steps
// on Newton's form.  *changes receives the polynomial's sign changes among 64
// equally spaced points (the eight among them): a pair of roots between two of
// the eight points leaves no trace in their signs.
__device__ double poly_root(const Secular& v, int l, int* changes) {
  int top = v.expo;  // the values at one common exponent, the largest
#pragma unroll
  for (int off = kGroup / 2; off >= 1; off >>= 1) top = max(top, __shfl_xor(top, off, kGroup));
  const double F = __builtin_ldexp(v.mant, max(-2000, v.expo - top));
  double d[kGroup];
#pragma unroll
  for (int i = 0; i < kGroup; ++i) d[i] = __shfl(F, i, kGroup);
  double t0 = double(l - 1), t1 = double(l);
  double f0 = __shfl(F, l - 1, kGroup), f1 = __shfl(F, l, kGroup);
#pragma unroll
  for (int n = 1; n < kGroup; ++n)
#pragma unroll
    for (int i = kGroup - 1; i >= n; --i) d[i] -= d[i - 1];
  constexpr double kInv[kGroup] = {1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040};
#pragma unroll
  for (int n = 2; n < kGroup; ++n) d[n] *= kInv[n];
  auto newton_form = [&](double t) {
    double p = d[kGroup - 1];
#pragma unroll
    for (int n = kGroup - 2; n >= 0; --n) p = __builtin_fma(p, t - double(n), d[n]);
    return p;
  };
  int sub = int(threadIdx.x) & (kGroup - 1);
  asm volatile("" : "+v"(sub));  // (the points would otherwise be held in registers over the rounds)
  int n_changes = 0;  // of points 8 sub .. 8 sub + 8 (63 at most) of the 64, spaced 1/9
  bool up = newton_form(double(8 * sub) * (1.0 / 9.0)) > 0.0;
#pragma unroll 1
  for (int i = 1; i <= 8; ++i) {
    const bool next = newton_form(double(min(8 * sub + i, 63)) * (1.0 / 9.0)) > 0.0;
    n_changes += next != up ? 1 : 0;
    up = next;
  }
#pragma unroll
  for (int off = kGroup / 2; off >= 1; off >>= 1) n_changes += __shfl_xor(n_changes, off, kGroup);
  *changes = n_changes;
  const double a = t0, b = t1;
  double t = t0 - f0 * (t1 - t0) / (f1 - f0);
  for (int it = 0; it < 4; ++it) {
    const double p = newton_form(t);
    // secant step from the end of the pair that is nearer in value
    if (__builtin_fabs(f1) < __builtin_fabs(f0)) {
      t0 = t1;
      f0 = f1;
    }
    t1 = t;
    f1 = p;
    const double s = f1 - f0;
    if (!(s != 0.0)) break;
    t = t1 - f1 * (t1 - t0) / s;
    t = __builtin_fmin(__builtin_fmax(t, a), b);
  }
  return t == t ? t : 0.5 * (a + b);
}

// Adds a wavefront's evaluations and this lane's layers and steps to the
// call's counters: summed over the workgroup in LDS, one atomic per counter
// and workgroup (device-scope atomics bypass the L2, so each costs a memory
// write).  Called by every wavefront of the workgroup.
__device__ void add_counts(const ClassifyArgsDev& a, unsigned long long (*s_cnt)[3], unsigned long long n_eval,
                           unsigned long long n_layer, unsigned long long n_step) {
  const int lane = int(threadIdx.x) & 63, wave = int(threadIdx.x) >> 6;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    n_step += __shfl_xor(n_step, off, 64);
    n_layer += __shfl_xor(n_layer, off, 64);
  }
  if (lane == 0) {
    s_cnt[wave][0] = n_eval;
    s_cnt[wave][1] = n_layer;
    s_cnt[wave][2] = n_step;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    unsigned long long sum = 0;
#pragma unroll
    for (int w = 0; w < kClassifyWaves; ++w) sum += s_cnt[w][threadIdx.x];
    if (sum) atomicAdd(&a.counters[threadIdx.x], sum);
  }
}

__global__ __launch_bounds__(64 * kClassifyWaves) __attribute__((amdgpu_waves_per_eu(3))) void classify_kernel(ClassifyArgsDev a) {
  __shared__ unsigned long long s_cnt[kClassifyWaves][3];
  const int lane = int(threadIdx.x) & 63;
  const int wave = int(threadIdx.x) >> 6;
  const int sub = lane & (kGroup - 1);
  const unsigned long long group = 0xffull << (lane & ~(kGroup - 1));
  const unsigned vb = xcd_block(blockIdx.x, gridDim.x);
  const int64_t wl = (int64_t(vb) * kClassifyWaves + wave) * kGroups + (lane / kGroup);
  unsigned rounds = 0, steps = 0;
  LaneWork w{};
  int cls = MASW_PICK_NONE;
  const int idx = wl < a.n_lam ? a.idx[wl] : 0;
  if (wl < a.n_lam) cls = lane_work(a, wl, idx, sub, group, &w);
  double root = __builtin_nan("");
  const unsigned long long todo = __ballot(cls < 0);
  if (todo != 0ull) {
    // lanes without an evaluation of their own mirror the first that has one
    const int src = __ffsll((long long)todo) - 1;
    const int64_t wl_src = __shfl(wl, src, 64);
    const int idx_src = __shfl(idx, src, 64);
    bool done = cls >= 0;
    if (done) {
      LaneWork o{};
      (void)lane_work(a, wl_src, idx_src, sub, group, &o);
      w = o;
    }
    const double tol = kRootTol * w.c_hi;
    const double c2_lo = w.c_lo * w.c_lo, c2_hi = w.c_hi * w.c_hi;
    // the ladder, in units of tol: this lane's offset from the root estimate
    const double rung = (sub & 4) ? 1.0 : -1.0;
    const int step = (sub & 4) ? (sub & 3) : 3 - (sub & 3);
    const double offset = rung * tol * (step == 0 ? 0.45 : step == 1 ? 16.0 : step == 2 ? 2048.0 : 524288.0);
    double lo = w.c_lo, hi = w.c_hi, est = 0.0;
    Secular F_lo{0.0, 0}, F_hi{0.0, 0};
    int s_lo = 0;
    for (int round = 0; round < kMaxRounds; ++round) {
      const double span = hi - lo;
      double cl;
      if (round == 0)
        cl = sub == kGroup - 1 ? hi : __builtin_fma(span, double(sub) * (1.0 / 7.0), lo);
      else
        cl = __builtin_fmin(__builtin_fmax(est + offset, lo), hi);
      const Secular F = secular(cl, c2_lo, c2_hi, w.k, w.h, w.al, w.be, w.rh, w.N, &steps);
      ++rounds;
      const bool nan = !(__builtin_fabs(F.mant) < __builtin_inf());
      const int sg = sgn(F.mant);
      const int s_first = __shfl(sg, 0, kGroup), s_last = __shfl(sg, kGroup - 1, kGroup);
      if (round == 0) s_lo = s_first;
      const unsigned long long nans = __ballot(nan) & group;
      // first point whose sign differs from the lower end's (kGroup: none)
      const unsigned diff = unsigned((__ballot(sg != s_lo) & group) >> (lane & ~(kGroup - 1)));
      const int l = diff ? __ffs(int(diff)) - 1 : kGroup;
      const double c_l = __shfl(cl, l & 7, kGroup), c_b = __shfl(cl, (l - 1) & 7, kGroup);
      const Secular F_l{__shfl(F.mant, l & 7, kGroup), __shfl(F.expo, l & 7, kGroup)};
      const Secular F_b{__shfl(F.mant, (l - 1) & 7, kGroup), __shfl(F.expo, (l - 1) & 7, kGroup)};
      int changes = 1;
      const double t = round == 0 ? poly_root(F, l < 1 || l > 7 ? 1 : l, &changes) : 0.0;
      if (!done) {
        if (nans) {
          cls = MASW_PICK_UNRESOLVED;
          done = true;
        } else if (round == 0 && s_last == s_lo) {
          cls = MASW_PICK_POLE;
          done = true;
        } else if (changes != 1) {  // several roots, perhaps: the first among 64 points, as below
          cls = -idx;
          done = true;
        } else {
          if (l > 0) {
            lo = c_b;
            F_lo = F_b;
          }
          if (l < kGroup) {
            hi = c_l;
            F_hi = F_l;
          }
          if (hi - lo <= tol) {
            cls = MASW_PICK_MODE;
            root = 0.5 * (lo + hi);
            done = true;
          } else if (round == 0) {
            est = __builtin_fma(span, t * (1.0 / 7.0), w.c_lo);
          } else if (l == 0 || l == kGroup || round == kMaxRounds - 1) {
            cls = -idx;  // deferred (idx and pick_class may be one array)
            done = true;
          } else {
            const double q = __builtin_ldexp(F_hi.mant / F_lo.mant, max(-1000, min(1000, F_hi.expo - F_lo.expo)));
            est = lo + (hi - lo) / (1.0 - q);
            if (!(est >= lo && est <= hi)) est = 0.5 * (lo + hi);
          }
        }
      }
      if (__ballot(!done) == 0ull) break;
    }
  }
  if (wl < a.n_lam && sub == 0) {
    a.cls[wl] = cls;
    if (a.c_sec) a.c_sec[wl] = root;
  }
  add_counts(a, s_cnt, 64ull * rounds, rounds * (unsigned long long)unsigned(max(w.N, 0)), steps);
}

// The deferred picks (class -idx), one whole wavefront each: multisection with 64 equally
// spaced points a round, the first whose sign differs from the lower end's
// giving the next bracket, 63 times narrower.  A wavefront looks through
// every gridDim-th pick, so that neighbouring picks, which are often deferred
// together, go to different ones.
__global__ __launch_bounds__(64 * kClassifyWaves) void classify_deferred_kernel(ClassifyArgsDev a) {
  __shared__ unsigned long long s_cnt[kClassifyWaves][3];
  const int lane = int(threadIdx.x) & 63;
  const int64_t n_waves = int64_t(gridDim.x) * kClassifyWaves;
  const int64_t first = int64_t(blockIdx.x) * kClassifyWaves + (threadIdx.x >> 6);
  unsigned long long n_eval = 0, n_layer = 0;
  unsigned steps = 0;
  for (int64_t base = first; base < a.n_lam; base += 64 * n_waves) {
    const int64_t mine = base + lane * n_waves;
    const int marked = mine < a.n_lam ? a.cls[mine] : 0;
    unsigned long long todo = __ballot(marked < 0);
    for (; todo != 0ull; todo &= todo - 1) {
      const int from = __ffsll((long long)todo) - 1;
      const int64_t wl = base + from * n_waves;
      LaneWork w{};
      (void)lane_work(a, wl, -__shfl(marked, from, 64), lane & (kGroup - 1), ~0ull, &w);
      const double tol = kRootTol * w.c_hi;
      const double c2_lo = w.c_lo * w.c_lo, c2_hi = w.c_hi * w.c_hi;
      double lo = w.c_lo, hi = w.c_hi;
      int s_lo = 0, cls = MASW_PICK_MODE;
      for (int round = 0; round < kMaxWideRounds; ++round) {
        const double cl = lane == 63 ? hi : __builtin_fma(hi - lo, double(lane) * (1.0 / 63.0), lo);
        const double F = secular(cl, c2_lo, c2_hi, w.k, w.h, w.al, w.be, w.rh, w.N, &steps).mant;
        n_eval += 64;
        n_layer += unsigned(w.N);
        if (__ballot(!(__builtin_fabs(F) < __builtin_inf())) != 0ull) {
          cls = MASW_PICK_UNRESOLVED;
          break;
        }
        const int sg = sgn(F);
        if (round == 0) s_lo = __shfl(sg, 0, 64);
        // (lane 63's sign differs: it did in the first launch)
        const unsigned long long diff = __ballot(lane >= 1 && sg != s_lo);
        const int l = diff ? __ffsll((long long)diff) - 1 : 63;
        lo = __shfl(cl, l - 1, 64);
        hi = __shfl(cl, l, 64);
        if (hi - lo <= tol) break;
      }
      if (lane == 0) {
        a.cls[wl] = cls;
        if (a.c_sec) a.c_sec[wl] = cls == MASW_PICK_MODE ? 0.5 * (lo + hi) : __builtin_nan("");
      }
    }
  }
  add_counts(a, s_cnt, n_eval, n_layer, steps);
}

__global__ void clear_counters_kernel(unsigned long long* c) {
  if (threadIdx.x < 3) c[threadIdx.x] = 0ull;
}

}  // namespace

hipError_t launch_classify(const ClassifyArgs& in, hipStream_t s) {
  if (in.n_lam <= 0) return hipSuccess;
  if (!in.counters) return hipErrorInvalidValue;
  ClassifyArgsDev a;
  a.layer_off = in.layer_off;
  a.h = in.h;
  a.alpha = in.alpha;
  a.beta = in.beta;
  a.rho = in.rho;
  a.lambda_off = in.lambda_off;
  a.lambda = in.lambda;
  a.c = in.c;
  a.idx = in.idx;
  a.cls = in.cls;
  a.c_sec = in.c_sec;
  a.n_lam = in.n_lam;
  a.n_models = in.n_models;
  a.n_c = in.n_c;
  a.counters = reinterpret_cast<unsigned long long*>(in.counters);
  // a kernel, not a memset, clears the counters, so a caller may capture the call
  hipLaunchKernelGGL(clear_counters_kernel, dim3(1), dim3(64), 0, s, a.counters);
  constexpr int kPerBlock = kClassifyWaves * kGroups;  // wavelengths per workgroup
  const int64_t blocks = (in.n_lam + kPerBlock - 1) / kPerBlock;
  hipLaunchKernelGGL(classify_kernel, dim3(unsigned(blocks)), dim3(64 * kClassifyWaves), 0, s, a);
  // few picks are deferred: a fixed number of wavefronts looks for them
  const int64_t wide = std::min<int64_t>(512, (in.n_lam + kClassifyWaves - 1) / kClassifyWaves);
  hipLaunchKernelGGL(classify_deferred_kernel, dim3(unsigned(wide)), dim3(64 * kClassifyWaves), 0, s, a);
  return hipGetLastError();
}

}  // namespace masw
