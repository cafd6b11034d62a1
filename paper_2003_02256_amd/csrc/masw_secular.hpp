// The sign of det K for the grid sweeps, from the dispersion function in
// minors instead of the block elimination (masw_math.hpp).
//
// det K of the stiffness formulation is the dispersion function F divided by
// the layers' denominators D_j and positive factors, so
//     sign(det K) = sign(F) prod_j sign(D_j),
// and only signs are asked for in a sweep.  F is carried down from the free
// surface as the 2x2 minors of the pair of solutions that satisfy it (the
// delta-matrix or compound-matrix idea, Thomson-Haskell products without
// their cancellation), in the layer's potentials: with zeta = k z, phi the P
// and psi the S potential and ' = d/dzeta, the pair (a, a', b, b') =
// (phi, phi', psi, psi') has horizontal and vertical displacement U = a + b',
// W = a' + b and normal and shear traction (over mu k) (2 - g) a + 2 b' and
// 2 a' + (2 - g) b, g = c^2/beta^2.  With [xy] the minor of rows x and y,
//     z1 = [ab],  z2 = [aa'] = [b'b],  z3 = [b'a'],  p = [ab'],  q = [a'b]
// are all six (a symplectic form makes two of them equal).
//
// Through a layer, phi turns by [[Cr, Sr], [Rr, Cr]] and psi likewise by s
// (C = cosh, S = sinh/r, R = r sinh of k h r, r^2 = 1 - c^2/alpha^2,
// s^2 = 1 - c^2/beta^2): with Z = [[z1, p], [q, -z3]], Z becomes
// [[Cr, Sr], [Rr, Cr]] Z [[Cs, Rs], [Ss, Cs]], and z2 stays.
// At an interface U, W and the tractions are continuous.  In (U, a) the
// symmetric matrix [[z1, z2], [z2, z3]] of the minors between (a, b') and
// (b, a') has the entries z1 + 2 z2 + z3, z1 + z2 and z1; the potentials of
// the next layer are a_next = y U + dr a with y = kap/c^2,
// kap = 2 (mu_next - mu)/rho_next and dr = rho/rho_next, the same for b and W,
// and p and q are multiplied by dr.  Dividing everything by dr > 0:
//     UU = (z1 + 2 z2 + z3)/dr,  Ua = y UU + (z1 + z2),
//     aa = y (Ua + (z1 + z2)) + dr z1,  z1 = aa,  z2 = Ua - aa,  z3 = UU - Ua - z2,
// with p and q as they were.  This order of the sums, with no difference of
// two large products, keeps the sign right to about 1e-15 relative in c around
// a root on the profiles of the workloads (the elimination: 1e-14), and to
// 8e-11 in the worst of 150 random profiles of strong contrasts (4e-12).
//
// At low c UU cancels to the order of (c/beta)^4 and meets y^2, which grows as
// (beta/c)^4: where some layer is much stiffer than c, the sign is rounding
// noise at velocities where the elimination's is exact.  Wrong signs away from
// a root, of 4000 random models (1 to 7 layers, beta 100 to 3500 m/s) and of
// 1500 with any contrast (1 to 30 layers, alpha/beta to 30, layers of 2 mm to
// 300 m): none at velocities above 1/287 of the largest beta, and three above
// 1/100, the highest at 1/52 (the elimination: 1/1083 and 1/229).  So
// velocities below kLowest times the largest beta are swept by the elimination
// (c_low, in the half-space's record).  The elimination has the last word all
// the same: the refinement evaluates it at the two grid points of a pick, and
// where it does not confirm the change the walk is made again by it alone
// (walk_by_k).  Either of the two measures alone loses picks: 1067 of 31,000
// random items of the two kinds, on grids from 0.3 to 50 m/s, without the
// first.  With both, 253 of 196,000 items of the second kind are walked again,
// and 7 picks are one to four grid steps from the elimination's first change,
// which is itself within its rounding of the root there.  The split path checks
// its candidates with the elimination.
//
// In FP32 the noise reaches velocities of interest where a stiff layer lies over
// a much softer one (a pavement: 36% of the signs below the pick were wrong, in
// every profile), and hardly any other (none of 300 profiles of soft layers over
// rock): the relative error is up to 4 eps (beta/c)^4 of the stiff layer.  Every
// wrong sign costs the split path a check of 64 velocities, so a model is walked
// in FP64 where the grid starts below kLowest32 times the largest beta that has
// one of less than 1/kInversion of it below it (ModelDesc::n_real is 0).
// Pavements of 5 to 14 layers, us in FP32 and in FP64 (by the elimination in
// FP32): 100 wavelengths x 2,000 velocities 606 and 71 (221), 600 models x 100 x
// 9,501 32,200 and 6,300 (20,500).
//
// At the surface (free) z1 = 4, z2 = -2 (2 - g), z3 = (2 - g)^2, p = q = 0;
// over the half-space, whose potentials decay as exp(-r zeta), exp(-s zeta),
//     F = r s z1 - z3 + r p + s q,
// divided by 1 - r s where that is complex (at or above its S velocity; the
// real part counts, as in halfspace_det).
//
// D_j is only evaluated where it can be negative: every mode of a layer with
// both faces fixed, that is every sign change of D_j, lies above the energy
// bound k h sqrt(c^2/beta^2 - 1) = pi (masw_inertia.hpp).
//
// With q = sqrt|x|, z = (k h)^2 x for x = r^2 or s^2:
//     |z| <= 4:  the series of cosh and sinh(.)/. in z (FP32) or, in FP64, in
//                w = z/4 and doubled (cosh 2y = 2 cosh^2 y - 1, five operations
//                for four terms of each series);
//     z > 4:     all multiplied by E = exp(-k h q);
//     z < -4:    cos, sin.
// 92% of the potentials of the workloads, and 70% of the wavefronts' (64
// consecutive c), take the series; cos and sin one in 3000.
//
// Per layer in FP64, with both potentials by the series: 84 vector
// instructions (2 for k h, 1 for the energy bound, 25 and 23 for the
// potentials, 16 to turn the minors, 12 for the interface, 1 or 2 for the
// rescaling), against 127 for the entries and the elimination with its two
// reciprocals.  Bound by the vector ALU as before: 4096 models, 1.12 M
// wavelengths, 3.34e9 points: 211.2 -> 160.3 ms in FP64, 98.6 -> 82.7 ms on the
// split path; one model of 20 layers, 1000 wavelengths, 115,001 velocities:
// 1380 -> 1157 us and 808 -> 707 us.
#pragma once
#include <hip/hip_runtime.h>

#include "masw_internal.hpp"
#include "masw_math.hpp"
#include "masw_special.hpp"

namespace masw {
namespace secular {

// The series run in (t q)^2 with t = k h kUnit.
template <typename T>
constexpr T kUnit = sizeof(T) == 8 ? T(0.5) : T(1);
template <typename T>
constexpr T kSeriesEnd = T(4) * kUnit<T> * kUnit<T>;
template <typename T>
constexpr T kBound = T(-9.86) * kUnit<T> * kUnit<T>;  // the energy bound's (t q)^2, inside pi^2

// The lowest velocity swept in minors, over the largest beta (file comment).
constexpr double kLowest = 1.0 / 64.0;

// The largest beta of a layer that has one of less than 1/kInversion of it below
// it (0: none), from 64 consecutive layers, one a lane (`is`: the lane has one);
// *above is the largest beta before them, and then up to their last.  Every
// lane of the wavefront calls it and gets the result.  The maxima go by DPP
// moves: with shuffles the staging took 0.5 us more.
template <int CTRL, int ROWS>
__device__ __forceinline__ float max_with(float v) {
  const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, true);
  return __builtin_fmaxf(v, __builtin_bit_cast(float, o));
}
__device__ __forceinline__ float lane_of(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ float inversion(float beta, bool is, float* above) {
  float top = is ? beta : 0.0f;   // largest up to this layer
  top = max_with<0x111, 0xf>(top);  // shifts by 1, 2, 4 and 8 lanes inside rows of 16
  top = max_with<0x112, 0xf>(top);
  top = max_with<0x114, 0xf>(top);
  top = max_with<0x118, 0xf>(top);
  top = max_with<0x142, 0xa>(top);  // lane 15 of rows 0 and 2 to rows 1 and 3
  top = max_with<0x143, 0xc>(top);  // lane 31 to rows 2 and 3
  top = __builtin_fmaxf(top, *above);
  *above = lane_of(top, 63);
  // (a layer this slow is not the largest itself, and `top` does not fall: the
  // last slow layer's is the result)
  const unsigned long long slow = __ballot(is && top > kInversion * beta);
  return slow ? lane_of(top, 63 - __clzll((long long)slow)) : 0.0f;
}

// Interface constants of layer j over layer j + 1 (or the half-space), as
// they are kept in layer j's record.
struct Interface {
  double dr, idr, kap;
};
__device__ __forceinline__ Interface interface_of(double rho, double beta, double rho_next, double beta_next) {
  return Interface{rho / rho_next, rho_next / rho,
                   2.0 * (rho_next * beta_next * beta_next - rho * beta * beta) / rho_next};
}

template <typename T>
struct Layer {
  T ia2, ib2, h, dr, idr, kap;
};

template <typename T>
__device__ __forceinline__ Layer<T> load_layer(const LayerRec<T>* L, int j) {
  if (__builtin_amdgcn_is_shared((const __attribute__((address_space(0))) void*)(L))) {
    const LayerRec<T>& q = L[j];
    return Layer<T>{q.ia2, q.ib2, q.h, q.aux, q.idr, q.kap};
  }
  ConstRec<T>* q = (ConstRec<T>*)(L) + j;  // scalar loads, as load_rec's
  return Layer<T>{q->ia2, q->ib2, q->h, q->aux, q->idr, q->kap};
}

// C, S and R of one potential (file comment), multiplied by E where z > 4;
// *scale is multiplied by E.  t2 = t^2.
template <typename T>
struct Turn {
  T C, S, R;
};
template <typename T>
__device__ __forceinline__ Turn<T> turn_terms(const special::SeriesCoef<T>& K, T x, T t, T t2, T* scale) {
  Turn<T> o;
  const T w = t2 * x;
  if (__builtin_fabs(w) <= kSeriesEnd<T>) {
    T ch, shc;
    special::cosh_shc(K, w, &ch, &shc);
    if constexpr (sizeof(T) == 8) {
      const T ch2 = ch + ch;
      o.C = fma_(ch2, ch, T(-1));
      o.S = (t * shc) * ch2;
    } else {
      o.C = ch;
      o.S = t * shc;
    }
    o.R = x * o.S;
    return o;
  }
  const T kh = sizeof(T) == 8 ? t + t : t;
  if (x < T(0)) {
    const T iq = special::rsqrt(-x);
    const T q = -x * iq;
    T sn;
    special::sin_cos(kh * q, &sn, &o.C);
    o.S = sn * iq;
    o.R = -q * sn;
  } else {
    const T iq = special::rsqrt(x);
    const T q = x * iq;
    const T E = special::exp_neg(kh * q);
    const T half = T(0.5) * E;
    o.C = fma_(half, E, T(0.5));
    const T sh = fma_(-half, E, T(0.5));
    o.S = sh * iq;
    o.R = sh * q;
    *scale *= E;
  }
  return o;
}

// sign(Re det K(k, c)) in {-1, 0, +1}, or kNaNSign, as det_sign gives it up to
// rounding; *odd receives whether an odd number of the layer denominators are
// negative.
template <typename T>
__device__ __forceinline__ int sign(T c, T k, const LayerRec<T>* __restrict__ L, int N, int* odd) {
  constexpr int kRescale = sizeof(T) == 8 ? 8 : 4;  // layers between rescalings of the minors
  const T ku = kUnit<T> * k;
  const T c2 = c * c;
  const T ic2 = special::rcp(c2);
  const special::SeriesCoef<T> K;
  bool par = false;
  Layer<T> nxt = load_layer<T>(L, 0);
  const T g2 = T(2) - c2 * nxt.ib2;
  T z1 = T(4), z2 = T(-2) * g2, z3 = g2 * g2, p = T(0), q = T(0);
  for (int j = 0; j < N; ++j) {
    const Layer<T> l = nxt;
    nxt = load_layer<T>(L, j + 1);  // one layer ahead; after the last layer, the half-space
    const T xr = T(1) - c2 * l.ia2;
    const T xs = T(1) - c2 * l.ib2;
    const T t = ku * l.h;
    const T t2 = t * t;
    T E = T(1);
    const Turn<T> P = turn_terms(K, xr, t, t2, &E);
    const Turn<T> S = turn_terms(K, xs, t, t2, &E);
    const bool beyond = t2 * xs <= kBound<T>;
    if (__ballot(beyond) != 0ull) {  // (a branch: the compiler would run the rest of it with no lane active)
      const T D = T(2) * (E - P.C * S.C) + P.S * S.S + P.R * S.R;
      par ^= beyond && D < T(0);
    }
    const T a1 = P.C * z1 + P.S * q, a2 = P.C * p - P.S * z3;
    const T b1 = P.R * z1 + P.C * q, b2 = P.R * p - P.C * z3;
    z1 = a1 * S.C + a2 * S.S;
    p = a1 * S.R + a2 * S.C;
    q = b1 * S.C + b2 * S.S;
    z3 = -(b1 * S.R + b2 * S.C);
    z2 *= E;
    const T y = l.kap * ic2;
    const T s = z1 + z2;
    const T UU = (s + (z2 + z3)) * l.idr;
    const T Ua = fma_(y, UU, s);
    const T aa = fma_(y, Ua + s, l.dr * z1);
    z1 = aa;
    z2 = Ua - aa;
    z3 = (UU - Ua) - z2;
    if (((j + 1) & (kRescale - 1)) == 0) {
      const T top = ((__builtin_fabs(z1) + __builtin_fabs(z2)) + (__builtin_fabs(z3) + __builtin_fabs(p))) +
                    __builtin_fabs(q);
      int e;
      (void)frexp_(top, &e);
      z1 = ldexp_(z1, -e);
      z2 = ldexp_(z2, -e);
      z3 = ldexp_(z3, -e);
      p = ldexp_(p, -e);
      q = ldexp_(q, -e);
    }
  }
  const T xr = T(1) - c2 * nxt.ia2;
  const T xs = T(1) - c2 * nxt.ib2;
  T F;
  if (xs > T(0)) {
    const T r = xr * special::rsqrt(xr);
    const T s = xs * special::rsqrt(xs);
    F = (r * s * z1 - z3) + (r * p + s * q);
  } else {
    // s = i |s|, and r real or imaginary: the real part of F conj(1 - r s)
    const T s = sqrt_<T>(-xs);
    const T r = sqrt_<T>(xr < T(0) ? -xr : xr);
    const T rr = xr >= T(0) ? r : T(0), ri = xr >= T(0) ? T(0) : r;
    const T re = (rr * p - z3) - ri * s * z1, im = rr * s * z1 + ri * p + s * q;  // F
    const T dr = T(1) + ri * s, di = -rr * s;                                    // 1 - r s
    F = re * dr + im * di;
  }
  *odd = par ? 1 : 0;
  return sign_code(par, double(F));
}

}  // namespace secular
}  // namespace masw
