// syev3_lane.hpp -- per-lane solver for one 3x3 real symmetric eigenproblem.
//
// One GPU lane owns one matrix and keeps everything in registers: no LDS, no
// cross-lane traffic, no MFMA (the work is a short chain of scalar
// recurrences per matrix, not a contraction).  The method is Borges,
// "Solving the 3x3 Real Symmetric Eigenproblem":
//   Sec. 1    Jacobi rotation in the (1,2)-plane -> ordered arrow
//             (alpha1 >= alpha2, beta1, beta2, gamma)
//   Sec. 1.1  Givens rotation G taking beta1 to zero; h = ||beta||; exact
//             beta- and combo-deflations and the EISPACK-style numerical
//             deflation test on G A G^T (or its simplified form)
//   Sec. 1.2  for an ordered, reduced arrow: mu = lambda1 - alpha1 and
//             nu = alpha2 - lambda3 as rightmost zeros of two fully reduced
//             arrows, lambda2 from the trace identity, eigenvectors u1, u3, u2
//   Sec. 1.4  the zeros: an FP32 start and one FP64 Halley step on the
//             numerator of f, whose bound on what is left is tested; zeros
//             that do not pass it by the Borges-Gragg iteration (rational
//             model w0 x - sigma - w1/x, increment quadratic).  By flag the
//             paper's own iteration (start from +inf, stop when f/f' <
//             2 eps x), or Newton's method from the left.
//
// Choices made here (the paper leaves them open):
//   * every matrix is scaled by a power of two so that max |a_ij| is in
//     [1/2, 1); exact, undone on the eigenvalues at the end;
//   * the Jacobi rotation is the textbook symmetric Schur rotation written
//     with hypot(d, a12), d = (a22 - a11)/2, so it cannot overflow; entries
//     below 2^-500 of the scaled matrix count as zero in it;
//   * h counts as zero when h <= eps (|alpha1| + |alpha2| + |gamma|) (the
//     EISPACK criterion on the other off-diagonal of the tridiagonal
//     G A G^T) unless SYEV3_FLAG_NO_H_GUARD;
//   * the diagonal entries d1, d2 of G A G^T are formed as alpha1 - alpha s^2
//     etc., choosing the form with the smaller correction; algebraically the
//     paper's ratios, and bitwise exact for beta- and combo-deflations;
//   * a Borges-Gragg step that would remove more than half of x_j takes
//     x_{j+1} directly as the zero of the rational model (no cancellation
//     for roots next to the pole at 0);
//   * eigenvalues ascending, eigenvector columns carried along.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace syev3 {

constexpr double kEps64 = 0x1p-52;
constexpr float kEps32 = 0x1p-23f;
constexpr int kMaxIter = 32;     // Borges-Gragg steps per root (FP64)
constexpr int kMaxHalley = 4;    // Halley steps before them, after the first
constexpr int kMaxIter32 = 24;   // FP32 zero-finder evaluations per root

constexpr uint32_t kFlagSimplified = 1u;
constexpr uint32_t kFlagNoHGuard = 2u;
constexpr uint32_t kFlagNewton = 4u;
constexpr uint32_t kFlagPaperBG = 8u;
constexpr uint32_t kFlagRefineConverge = 16u;
constexpr uint32_t kFlagNoScale = 32u;

// Arithmetic forms of the solve, a template argument (equal to the dtype
// codes of the interface): FP64; FP32 storage with the FP64 solve; FP32
// storage with an FP32 zero finder's zeros used as they are (an ablation of
// the refinement).  Each form is compiled on its own, so no form's kernel
// holds another's code.
constexpr int kFormF64 = 0;
constexpr int kFormF32R = 1;
constexpr int kFormF32 = 2;
// FP64 or FP32 storage with the FP64 solve, told apart by the caller's
// loads and stores alone: the serving kernel, which meets both.
constexpr int kFormBoth = 3;

enum Branch : int { kZero = 0, kNonFinite = 1, kDiagonal = 2, kDeflated = 3,
                    kReduced = 4 };

// ---------------------------------------------------------------------------
// Arithmetic primitives.  gfx950's v_rcp_f64, v_rsq_f64 and v_sqrt_f64 are
// accurate to about 2^-24 (measured); Newton-Raphson, Goldschmidt or
// third-order correction steps built from FMAs bring them to the rounding
// level at a fraction of the cost of the IEEE-exact division and square-root
// sequences.  Arguments must be
// normal positive numbers (or, for rcp, any normal non-zero number).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double dabs(double x) { return __builtin_fabs(x); }

// 1/x to ~2^-48 (one Newton-Raphson step).
__device__ __forceinline__ double rcp1(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

// a/b to about one ulp from a ~2^-47 reciprocal rb of b: quotient plus one
// residual correction.
__device__ __forceinline__ double div_r(double a, double b, double rb) {
  const double q = a * rb;
  return __builtin_fma(__builtin_fma(-b, q, a), rb, q);
}

__device__ __forceinline__ double ddiv(double a, double b) { return div_r(a, b, rcp1(b)); }

// 1/sqrt(x) to about one ulp: v_rsq_f64 and one third-order correction.
// With e = 1 - x y^2, 1/sqrt(x) = y (1 - e)^(-1/2) = y (1 + e/2 + 3e^2/8 +
// 5e^3/16 + ...); for |e| ~ 2^-23 the neglected terms are below 2^-66, and
// e itself is formed by one FMA from x y, so the result carries the
// roundings of the last FMA and of e's product, under one ulp together.
__device__ __forceinline__ double rsqrt2(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-(x * y), y, 1.0);
  return __builtin_fma(y, e * __builtin_fma(e, 0.375, 0.5), y);
}

// sqrt(x) to ~2^-47 for normal x > 0: one Goldschmidt step.
__device__ __forceinline__ double sqrt1(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double g = x * y, h = 0.5 * y;
  const double r = __builtin_fma(-g, h, 0.5);
  return __builtin_fma(g, r, g);
}

// sqrt(x) to about one ulp: one Goldschmidt step and a residual correction.
__device__ __forceinline__ double sqrt2(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = __builtin_fma(-g, h, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  return __builtin_fma(__builtin_fma(-g, g, x), h, g);
}

// ---------------------------------------------------------------------------
// 2x2 symmetric eigenproblem [[p, r], [r, q]] by one Jacobi rotation, the
// textbook symmetric Schur rotation written so that it comes out ordered.
// With d = (q - p)/2 and u = r / (|d| + hypot(d, r)) (|u| <= 1, the
// rotation's tangent up to sign), the correction u r = r^2 / (|d| + hypot)
// is >= 0 and
//   l1 = max(p, q) + u r,  l2 = min(p, q) - u r  (l1 >= l2),
// with unit eigenvector (c, u c) of l1 when p >= q, else (u c, c),
// c = 1/sqrt(1 + u^2).  (From 2|d| D + r^2 = D^2, D = |d| + hypot(d, r).)
// The eigenvector of l2 is that of l1 turned by 90 degrees, (-k21, k11), so
// J = [[k11, k12], [k21, k22]] is a rotation with J^T B J = diag(l1, l2);
// choosing the order costs two selects, not six.  Ties p == q keep (c, uc).
// ---------------------------------------------------------------------------
struct Rot2 {
  double l1, l2, k11, k12, k21, k22;
};

__device__ __forceinline__ Rot2 rot2(double p, double r, double q) {
  const double d = 0.5 * (q - p);
  const double ad = dabs(d);
  // 2^-1000 under the root keeps it normal and the quotient's divisor at
  // least 2^-500 (d = r = 0 gives u = 0, and r = 0 gives u = 0 exactly), at
  // no cost in the FMA chain; it moves hypot(d, r) by under half an ulp
  // unless d^2 + r^2 < 2^-946, where the block is below 2^-470 of a matrix
  // scaled to max |a_ij| >= 1/2.
  const double rr = sqrt2(__builtin_fma(d, d, __builtin_fma(r, r, 0x1p-1000)));
  const double u = ddiv(r, ad + rr);
  const double c = rsqrt2(__builtin_fma(u, u, 1.0));
  const double s = u * c;
  const bool keep = p >= q;
  Rot2 o;
  o.l1 = __builtin_fma(u, r, __builtin_fmax(p, q));
  o.l2 = __builtin_fma(-u, r, __builtin_fmin(p, q));
  o.k11 = keep ? c : s;
  o.k21 = keep ? s : c;
  o.k12 = -o.k21;
  o.k22 = o.k11;
  return o;
}

// ---------------------------------------------------------------------------
// Fully reduced arrow [[0, 0, b1], [0, -ab, b2], [b1, b2, gb]] (Sec. 1.4):
// spectral function f(x) = x - gb - b1^2/x - b2^2/(x + ab), its rightmost
// zero.  The structure carries b1^2 and b2^2.
// ---------------------------------------------------------------------------
struct Arrow1 {
  double b1s, b2s, ab, gb;
};

// f and f' at x > 0, with b1^2/x and b2^2/(x + ab) to about one ulp from a
// single reciprocal of x (x + ab).
struct Spec {
  double f, fp, rx, rp, q2;
};

__device__ __forceinline__ Spec spec_eval(const Arrow1& P, double x) {
  const double p = x + P.ab;
  const double r = rcp1(x * p);
  const double rx = p * r, rp = x * r;
  const double q1 = div_r(P.b1s, x, rx);
  const double q2 = div_r(P.b2s, p, rp);
  Spec s;
  s.f = ((x - P.gb) - q1) - q2;
  s.fp = __builtin_fma(q1, rx, __builtin_fma(q2, rp, 1.0));
  s.rx = rx;
  s.rp = rp;
  s.q2 = q2;
  return s;
}

// quad_zero(c, k, a): positive zero of a x^2 - c x - k (a, k > 0), in the
// form without cancellation.
__device__ __forceinline__ double quad_zero(double c, double k, double a) {
  const double c2 = 0.5 * c;
  const double s = dabs(c2) + sqrt1(__builtin_fma(c2, c2, a * k));
  const bool pos = c >= 0.0;
  return (pos ? s : k) * rcp1(pos ? a : s);
}

// FP32 versions (v_rcp_f32 and v_sqrt_f32 are accurate to about one ulp),
// for the start of the FP64 zero finder and for the FP32 zero finder of the
// unrefined FP32 ablation.
__device__ __forceinline__ float quad_zero32(float c, float k, float a) {
  const float c2 = 0.5f * c;
  const float s = __builtin_fabsf(c2) + __builtin_amdgcn_sqrtf(__builtin_fmaf(c2, c2, a * k));
  const bool pos = c >= 0.0f;
  return (pos ? s : k) * __builtin_amdgcn_rcpf(pos ? a : s);
}

// The same for a = 1: positive zero of x^2 - c x - k.
__device__ __forceinline__ float quad_zero32_1(float c, float k) {
  const float c2 = 0.5f * c;
  const float s = __builtin_fabsf(c2) + __builtin_amdgcn_sqrtf(__builtin_fmaf(c2, c2, k));
  return c >= 0.0f ? s : k * __builtin_amdgcn_rcpf(s);
}

// The numerator of f: F(x) = x (x + ab) f(x) = x^3 + A x^2 - K x - C with
//   A = ab - gb,  K = ab gb + b1^2 + b2^2 = ab c0 + b1^2,  C = b1^2 ab.
// F is a shift of the arrow's characteristic polynomial: its zeros are real,
// the one sought the only positive one.  Every term is formed from A, K and
// C once, in FP64: K is where the data cancels (c0 = gb + b2^2/ab is the
// zero's scale next to the pole), and as the start and the step that follows
// take the same rounded K, they agree on the zero to all its digits, however
// little of it the cancellation has left.  (f itself, evaluated term by
// term, moves a zero far below |gb| by its own rounding: FP64 steps on f
// after a start from c0 needed a second trip in 55% of wavefronts of the
// stress mix, steps on F in under 1%.)
struct Cubic {
  double A, K, C;
};

__device__ __forceinline__ Cubic cubic(const Arrow1& P, double hh) {
  return Cubic{P.ab - P.gb, __builtin_fma(P.ab, P.gb, hh), P.b1s * P.ab};
}

// One step of Laguerre's method on F in FP32, x - 3F / (F' + 2 sqrt(F'^2 -
// 3 F F''/2)): third order, and monotone from anywhere right of the zero as
// all zeros of F are real.  No cancellation that the zero does not share:
// the terms of F, taken positive, are at most a few times x F'.
__device__ __forceinline__ float laguerre32(float A, float K, float C, float x) {
  const float q = x + A;
  const float i = __builtin_fmaf(x, q, -K);
  const float F3 = 3.0f * __builtin_fmaf(x, i, -C);
  const float w = x + q;
  const float F1 = __builtin_fmaf(x, w, i);
  const float s = __builtin_amdgcn_sqrtf(__builtin_fmaf(F1, F1, -F3 * (x + w)));
  return __builtin_fmaf(-F3, __builtin_amdgcn_rcpf(__builtin_fmaf(2.0f, s, F1)), x);
}

// Start of the FP64 zero finder, in FP32, where arithmetic costs half as
// much (a multiply, add or FMA 2 cycles per wavefront against 4, measured,
// v_rcp and v_sqrt 8 against 16) and does not lower the clock:
//  * U = x_inf, the zero of x - gb - (b1^2 + b2^2)/x (the first iterate from
//    +infinity, Sec. 1.4.1), an upper bound;
//  * the zero of x - gb - b1^2/x - b2^2 chord(x), chord the chord of the
//    convex 1/(x + ab) over [0, 0.7 U] (over [0, U] it gives an upper bound
//    again; the shorter one is nearer the zero): close whether the zero lies
//    next to the pole at 0 or far from it;
//  * two Laguerre steps.
// In a CPU emulation of this arithmetic its relative error stays below
// 2^-17.5 for all lanes of 100% of wavefronts on N(0,1), uniform and
// chi-square matrices, 99.6% of the stress mix and 98% of condition-1e8 SPD
// matrices; two Borges-Gragg steps instead (70 cycles each against 38) 87%
// on chi-square ones; x_inf and three Laguerre steps as few as none (SPD).
// Nothing is checked here: an arrow that FP32 cannot represent gives some
// useless value (or NaN), which the FP64 step's test rejects.
__device__ __forceinline__ float start_point(const Arrow1& P, const Cubic& Q) {
  const float b1s = (float)P.b1s, b2s = (float)P.b2s, ab = (float)P.ab, gb = (float)P.gb;
  const float K = (float)Q.K;
  const float rab = __builtin_amdgcn_rcpf(ab);
  const float U = quad_zero32_1(gb, b1s + b2s);
  const float k = (b2s * rab) * __builtin_amdgcn_rcpf(__builtin_fmaf(0.7f, U, ab));
  float x = quad_zero32((K - b1s) * rab, b1s, 1.0f + k);
  x = laguerre32(ab - gb, K, b1s * ab, x);
  return laguerre32(ab - gb, K, b1s * ab, x);
}

// One step of Halley's method on F, x - F F' / (F'^2 - F F''/2), in FP64.
//  * done: Newton's correction F/F' at most 2^-17.5 x.  With the other zeros
//    of F at or below 0, |F'/F| is at most 1/d + 2/x at the distance d from
//    the sought one, so d is then that small, whatever x > 0 was given; and
//    the step leaves at most 3 d^3/x^2, that is 2^-51 x, the 2 eps that
//    bg_update's stop test asks for.  NaN, zero, infinite (as the comparison
//    is strict) and, as F' has to be positive, negative x fail it.
//  * The quotient's error, one v_rcp_f64 and one correction (2^-47), is
//    relative to a correction of 2^-17 x.
// 92 cycles per wavefront, against 290 for a Borges-Gragg step with its test.
__device__ __forceinline__ double halley_step(const Cubic& Q, double x, bool& done) {
  const double q = x + Q.A;
  const double i = __builtin_fma(x, q, -Q.K);
  const double F = __builtin_fma(x, i, -Q.C);
  const double w = x + q;
  const double F1 = __builtin_fma(x, w, i);
  const double den = __builtin_fma(F1, F1, -F * (x + w));
  const double r = __builtin_amdgcn_rcp(den);
  const double d0 = (F * F1) * r;
  const double dx = __builtin_fma(d0, __builtin_fma(-den, r, 1.0), d0);
  done = dabs(F) < (0x1.6p-18 * x) * F1 && F1 > 0.0;
  return x - dx;
}

// The start in FP64, for arrows that FP32 cannot represent: its range, not
// its precision, is what a zero needs that is many orders of magnitude below
// the matrix (a nearly isotropic matrix, or tiny betas).
__device__ __forceinline__ double laguerre(const Cubic& Q, double x) {
  const double q = x + Q.A;
  const double i = __builtin_fma(x, q, -Q.K);
  const double F3 = 3.0 * __builtin_fma(x, i, -Q.C);
  const double w = x + q;
  const double F1 = __builtin_fma(x, w, i);
  const double D = __builtin_fmax(0x1p-1000, __builtin_fma(F1, F1, -F3 * (x + w)));
  return __builtin_fma(-F3, rcp1(__builtin_fma(2.0, sqrt1(D), F1)), x);
}

__device__ __forceinline__ double start_point64(const Arrow1& P, const Cubic& Q) {
  const double rab = rcp1(P.ab);
  const double U = quad_zero(P.gb, P.b1s + P.b2s, 1.0);
  const double k = (P.b2s * rab) * rcp1(__builtin_fma(0.7, U, P.ab));
  const double x = quad_zero((Q.K - P.b1s) * rab, P.b1s, 1.0 + k);
  return laguerre(Q, laguerre(Q, x));
}

// FP32 arrow of the unrefined ablation: c0 = gb + b2^2/ab and rab = 1/ab are
// formed in FP64 and rounded.
struct Arrow1f {
  float b1s, b2s, ab, gb, c0, rab;
};

__device__ __forceinline__ Arrow1f to_f32(const Arrow1& P, double rab) {
  return Arrow1f{(float)P.b1s, (float)P.b2s, (float)P.ab, (float)P.gb,
                 (float)__builtin_fma(P.b2s, rab, P.gb), (float)rab};
}

// An upper bound of the zero: x_inf, tightened by chords of 1/(x + ab) over
// [0, U] (see start_point); their constant is c0, which FP32 could not form
// where its terms cancel.
constexpr int kChords = 2;
__device__ __forceinline__ float bg_start32(const Arrow1f& P) {
  float U = quad_zero32(P.gb, P.b1s + P.b2s, 1.0f);
  const float b2r = P.b2s * P.rab;
  const float c = P.c0;
#pragma unroll
  for (int j = 0; j < kChords; ++j) {
    const float k = b2r * __builtin_amdgcn_rcpf(U + P.ab);
    U = __builtin_fminf(U, quad_zero32(c, P.b1s, 1.0f + k));
  }
  return U;
}

// One Borges-Gragg step from x on either side of the zero (Sec. 1.4.1: the
// iteration converges monotonically from any start in (0, inf)).  Sets stop
// when the returned value is final.
//  * The model phi_j = w0 x - sigma - w1/x matches f, f', f'' at x_j, and
//    f - phi_j = -b2^2 ab (x - x_j)^3 / ((x_j + ab)^3 x (x + ab)) (exactly).
//    Since phi_j(x_new) = 0, f(x_new) = -(w0 - 1) D^3 / (x_new (x_new + ab))
//    with D = x_new - x_j: the iterate stays on the side it started from.
//  * Right of the zero (f > 0) the paper's increment D = 2f / (b + sqrt(b^2
//    + 4af)), a = -w0/x, b = f' + f/x > 0.  When it removes more than half
//    of x, x_new is the model zero itself, w0 x^2 - sigma x - w1 = 0, solved
//    without the cancellation of x - D next to the pole.
//  * Left of it (f < 0), a < 0 makes b^2 + 4af exceed b^2, so the increment
//    has no cancellation as 2f / (b + sqrt(b^2 + 4af)) for b >= 0 nor as
//    (sqrt(b^2 + 4af) - b) / (2a) for b < 0 (b is negative where
//    f/x < -f').
//  * Stop right of the zero: the paper's bound x - zero < f(x)/f'(x) at
//    x_new, with f(x_new) from the closed form and f'(x_new) > f'(x_j) (f'
//    decreases): x_new - zero < (w0 - 1)|D|^3 / (x_new (x_new + ab) f'(x_j)),
//    cubic in the step and checked without evaluating f at x_new.  Left of
//    it: zero - x_new < |f(x_new)| / f'(c) <= |f(x_new)| (f' >= 1, the bound
//    of Sec. 1.4.2).  Either is compared with 2 eps x_new.  A step that
//    rounding at the zero leaves in place, or moves by an ulp the wrong way,
//    passes it too.
// D is computed to about 2^-46: near the zero a cubic step's own error must
// stay below the rounding level.
__device__ __forceinline__ double bg_update(const Arrow1& P, double x, const Spec& s,
                                            bool& stop) {
  const bool left = s.f < 0.0;
  const double w0m1 = (s.q2 * P.ab) * (s.rp * s.rp);
  const double b = __builtin_fma(s.f, s.rx, s.fp);
  // 4 a f, with -4 w0 = -4 w0m1 - 4 in one FMA (bitwise the same product)
  const double a4f = (__builtin_fma(w0m1, -4.0, -4.0) * s.rx) * s.f;
  const double disc = __builtin_fmax(0x1p-1000, __builtin_fma(b, b, a4f));
  const double sq = sqrt1(disc);
  double dl = (2.0 * s.f) * rcp1(b + sq);
  if (b < 0.0) {
    // the conjugate form, only far left of the zero (f/x < -f'); in a
    // branch of its own (the empty asm keeps the compiler from evaluating
    // it on every lane and selecting), as no lane takes it after a start
    // close to the zero
    double bb = b, wm = w0m1;
    asm volatile("" : "+v"(bb), "+v"(wm));
    const double a = -(wm + 1.0) * s.rx;
    dl = (sq - bb) * rcp1(2.0 * a);
  }
  double xn;
  if (dl <= 0.5 * x) {
    xn = x - dl;
  } else {
    // right of the zero, a step of more than half of x: the model zero
    double wm = w0m1;
    asm volatile("" : "+v"(wm));
    const double w0 = wm + 1.0;
    const double r = x * s.rp;
    const double w1 = __builtin_fma(P.b2s * r, r * r, P.b1s);
    const double sigma = (w0 * x - w1 * s.rx) - s.f;
    const double sq2 = sqrt2(__builtin_fma(sigma, sigma, 4.0 * w0 * w1));
    xn = sigma >= 0.0 ? ddiv(sigma + sq2, 2.0 * w0) : ddiv(2.0 * w1, sq2 - sigma);
  }
  // Written as "not above", so that a NaN stops the iteration.  A step
  // that rounding at the zero sends the wrong way is below the rounding
  // level and passes the test.
  const double D = dabs(x - xn);
  if (!(w0m1 * (D * D) * D > 2.0 * kEps64 * (xn * xn) * (xn + P.ab) * (left ? 1.0 : s.fp)))
    stop = true;
  return xn;
}

__device__ __forceinline__ double bg_step(const Arrow1& P, double x, bool& stop) {
  return bg_update(P, x, spec_eval(P, x), stop);
}

// Borges-Gragg as the paper states it, for measuring what the start and the
// stop test above save (flag kFlagPaperBG): the start is x_inf, the first
// iterate from +infinity (Sec. 1.4.1); before each step the iteration stops
// when f/f' < 2 eps x (the paper's test with C = 2), when rounding has
// reached the zero (f <= 0), or when the step no longer decreases x.
// Taking f <= 0 as convergence, it needs a start and steps that do not land
// left of the zero by more than rounding, so its arithmetic is rounded to
// about one ulp (ddiv, sqrt2) in the order of the formulas of Sec. 1.4.1.
// The default finder's 2^-46 primitives would not do here (a start 2^-46
// left of the zero would be returned as it is); they do there, since that
// finder iterates from either side and bounds the new iterate.
// quad_zero_ulp: the positive zero of x^2 - c x - k, k > 0.
__device__ __forceinline__ double quad_zero_ulp(double c, double k) {
  const double c2 = 0.5 * c;
  const double s = dabs(c2) + sqrt2(__builtin_fma(c2, c2, k));
  return c >= 0.0 ? s : ddiv(k, s);
}
// One evaluation of the paper's iteration at x: stop (returning x) when f
// <= 0 or f/f' < 2 eps x, else the next iterate; a step that does not
// decrease x stops with x.
__device__ __forceinline__ double paper_step(const Arrow1& P, double x, bool& stop) {
  const double p = x + P.ab;
  const double q1 = ddiv(P.b1s, x), q2 = ddiv(P.b2s, p);
  const double f = ((x - P.gb) - q1) - q2;
  const double fp = (1.0 + ddiv(q1, x)) + ddiv(q2, p);
  if (!(f > 0.0) || ddiv(f, fp) < 2.0 * kEps64 * x) {
    stop = true;
    return x;
  }
  const double w0 = 1.0 + ddiv(ddiv(q2, p) * P.ab, p);
  const double a = -ddiv(w0, x);
  const double b = fp + ddiv(f, x);
  const double F = ddiv(2.0 * f, b);
  const double D = __builtin_fmax(0.0, 1.0 + ddiv(2.0 * a, b) * F);
  const double dl = ddiv(F, 1.0 + sqrt2(D));
  double xn;
  if (dl <= 0.5 * x) {
    xn = x - dl;
  } else {
    // the zero of the model itself (see bg_update)
    const double r = ddiv(x, p);
    const double w1 = P.b1s + P.b2s * r * r * r;
    const double sigma = (w0 * x - ddiv(w1, x)) - f;
    const double sq = sqrt2(sigma * sigma + 4.0 * w0 * w1);
    xn = sigma >= 0.0 ? ddiv(sigma + sq, 2.0 * w0) : ddiv(2.0 * w1, sq - sigma);
  }
  if (!(xn < x)) {
    stop = true;
    return x;
  }
  return xn;
}

// Newton from the left (Sec. 1.4.2): x0 where f meets -b2^2/(x + ab),
// i.e. x0 = gb/2 + sqrt((gb/2)^2 + b1^2); stop when |f| < 2 eps x.
__device__ __forceinline__ double newton_start(const Arrow1& P) {
  const double g2 = 0.5 * P.gb;
  const double disc = sqrt2(__builtin_fma(g2, g2, P.b1s));
  return P.gb >= 0.0 ? g2 + disc : ddiv(P.b1s, disc - g2);
}

__device__ __forceinline__ double newton_step(const Arrow1& P, double x, bool& stop) {
  const Spec s = spec_eval(P, x);
  if (s.f >= 0.0 || -s.f < 2.0 * kEps64 * x) {
    stop = true;
    return x;
  }
  const double xn = x - ddiv(s.f, s.fp);
  if (!(xn > x)) {
    stop = true;
    return x;
  }
  return xn;
}

// The two problems of an ordered, reduced arrow (Sec. 1.2): mu is the
// rightmost zero of A - alpha1 I, nu that of P (alpha2 I - A) P.
// g1 = gamma - alpha1, g2 = alpha2 - gamma.
struct Arrows {
  Arrow1 mu, nu;
};

__device__ __forceinline__ Arrows arrows(double al, double be1, double be2, double g1,
                                         double g2) {
  const double b1s = be1 * be1, b2s = be2 * be2;
  return Arrows{Arrow1{b1s, b2s, al, g1}, Arrow1{b2s, b1s, al, g2}};
}

// Both zeros: their FP32 starts and one Halley step each.  Roots that are
// not done then take more Halley steps, from the start in FP64 where the
// first one moved by more than a quarter of x, and those still not done
// Borges-Gragg steps from x_inf to their stop test (converge: every root,
// from the first Halley step's x where that is done).  x_inf lies right of
// the zero and is formed without cancellation: an arrow whose entries span
// many orders of magnitude may have a start left of the zero (the chord's
// constant is then the rounding error of K), from where Halley's steps run
// to another zero of F, and a Borges-Gragg step back from there, across many
// orders of magnitude at once, loses its digits.  (Entries of
// N(0,1) 10^-U(0,40): 92 of 2^20 matrices were wrong without the return to
// x_inf, by up to infinity; now the worst error of 78 M matrices, with up to
// 300 for the 40, is 7.4 eps in an emulation on the CPU.)  The two
// recurrences are independent, so their latencies overlap.  What follows the
// first steps is a branch of its own, which the empty asm keeps from being
// evaluated on every lane; it forms the arrows again, so that they need not
// be held until there.
__device__ __forceinline__ void zeros_bg(double al, double be1, double be2, double g1,
                                         double g2, double hh, bool converge, double& x1,
                                         double& x2, int& it1, int& it2) {
  const Arrows P = arrows(al, be1, be2, g1, g2);
  const Cubic Q1 = cubic(P.mu, hh), Q2 = cubic(P.nu, hh);
  const double y1 = (double)start_point(P.mu, Q1);
  const double y2 = (double)start_point(P.nu, Q2);
  bool s1, s2;
  x1 = halley_step(Q1, y1, s1);
  x2 = halley_step(Q2, y2, s2);
  it1 = 1;
  it2 = 1;
  const bool near1 = s1, near2 = s2;
  if (converge) {
    asm volatile("");
    s1 = s2 = false;
  }
  if (!(s1 && s2)) {
    asm volatile("" : "+v"(be1), "+v"(be2));
    const Arrows R = arrows(al, be1, be2, g1, g2);
    const Cubic C1 = cubic(R.mu, hh), C2 = cubic(R.nu, hh);
    if (!converge) {
      if (!s1 && !(dabs(x1 - y1) <= 0.25 * y1)) {
        asm volatile("");
        x1 = start_point64(R.mu, C1);
      }
      if (!s2 && !(dabs(x2 - y2) <= 0.25 * y2)) {
        asm volatile("");
        x2 = start_point64(R.nu, C2);
      }
      for (int t = 0; t < kMaxHalley; ++t) {
        if (s1 && s2) break;
        if (!s1) { ++it1; x1 = halley_step(C1, x1, s1); }
        if (!s2) { ++it2; x2 = halley_step(C2, x2, s2); }
      }
    }
    // (an x at the end of the range may pass Halley's test and give NaN)
    if (!(converge ? near1 : s1) || !(x1 > 0.0)) {
      s1 = false;
      x1 = quad_zero(R.mu.gb, hh, 1.0);
    }
    if (!(converge ? near2 : s2) || !(x2 > 0.0)) {
      s2 = false;
      x2 = quad_zero(R.nu.gb, hh, 1.0);
    }
    for (int t = 0; t < kMaxIter; ++t) {
      if (s1 && s2) break;
      if (!s1) { ++it1; x1 = bg_step(R.mu, x1, s1); }
      if (!s2) { ++it2; x2 = bg_step(R.nu, x2, s2); }
    }
  }
}

__device__ __forceinline__ void zeros_bg_paper(const Arrow1& P1, const Arrow1& P2,
                                               double& x1, double& x2, int& it1, int& it2) {
  x1 = quad_zero_ulp(P1.gb, P1.b1s + P1.b2s);
  x2 = quad_zero_ulp(P2.gb, P2.b1s + P2.b2s);
  bool s1 = false, s2 = false;
  it1 = 0;
  it2 = 0;
  for (int k = 0; k < 2 * kMaxIter; ++k) {
    if (s1 && s2) break;
    if (!s1) { ++it1; x1 = paper_step(P1, x1, s1); }
    if (!s2) { ++it2; x2 = paper_step(P2, x2, s2); }
  }
}

__device__ __forceinline__ void zeros_newton(const Arrow1& P1, const Arrow1& P2,
                                             double& x1, double& x2, int& it1, int& it2) {
  x1 = newton_start(P1);
  x2 = newton_start(P2);
  bool s1 = false, s2 = false;
  it1 = 0;
  it2 = 0;
  for (int k = 0; k < 4 * kMaxIter; ++k) {
    if (s1 && s2) break;
    if (!s1) { ++it1; x1 = newton_step(P1, x1, s1); }
    if (!s2) { ++it2; x2 = newton_step(P2, x2, s2); }
  }
}

// ---------------------------------------------------------------------------
// FP32 Borges-Gragg for the unrefined FP32 form (an ablation): the same
// iteration in single precision (v_rcp_f32 and v_sqrt_f32 are accurate to
// about one ulp).
// conv reports a stop by the precision test or at the zero.
// ---------------------------------------------------------------------------
struct Move32 {
  float xn, f, fp, w0m1;
};

__device__ __forceinline__ Move32 bg_move32(const Arrow1f& P, float x) {
  const float p = x + P.ab;
  const float rx = __builtin_amdgcn_rcpf(x);
  const float rp = __builtin_amdgcn_rcpf(p);
  const float q1 = P.b1s * rx;
  const float q2 = P.b2s * rp;
  // For x < ab, f = x - c0 - b1^2/x + b2^2 x / (ab (x + ab)) exactly: with
  // c0 formed in FP64 this keeps a zero that is small next to |gb| (where
  // gb and b2^2/ab nearly cancel) resolvable in FP32.  For x >= ab the
  // usual form has no such cancellation.
  const float f = x < P.ab ? ((x - P.c0) - q1) + q2 * (x * P.rab) : ((x - P.gb) - q1) - q2;
  const float fp = __builtin_fmaf(q1, rx, __builtin_fmaf(q2, rp, 1.0f));
  const float w0m1 = (q2 * P.ab) * (rp * rp);
  const float w0 = w0m1 + 1.0f;
  const float a = -w0 * rx;
  const float b = __builtin_fmaf(f, rx, fp);
  const float disc = __builtin_fmaxf(0.0f, __builtin_fmaf(b, b, 4.0f * a * f));
  const float dl = (2.0f * f) * __builtin_amdgcn_rcpf(b + __builtin_amdgcn_sqrtf(disc));
  float xn;
  if (dl <= 0.5f * x) {
    xn = x - dl;
  } else {
    const float r = x * rp;
    const float w1 = __builtin_fmaf(P.b2s * r, r * r, P.b1s);
    const float sigma = (w0 * x - w1 * rx) - f;
    const float sq = __builtin_amdgcn_sqrtf(__builtin_fmaf(sigma, sigma, 4.0f * w0 * w1));
    xn = sigma >= 0.0f ? (sigma + sq) * __builtin_amdgcn_rcpf(2.0f * w0)
                       : (2.0f * w1) * __builtin_amdgcn_rcpf(sq - sigma);
  }
  return Move32{xn, f, fp, w0m1};
}

// One step of the iteration with its stop tests (the unrefined form).
__device__ __forceinline__ float bg_step32(const Arrow1f& P, float x, bool& stop, bool& conv) {
  const Move32 m = bg_move32(P, x);
  if (m.f <= 0.0f || !(m.xn < x)) {
    // at the zero, or rounding no longer moves x down
    stop = true;
    conv = true;
    return x;
  }
  const float D = x - m.xn;
  if (m.w0m1 * (D * D) * D <= 4.0f * kEps32 * (m.xn * m.xn) * (m.xn + P.ab) * m.fp) {
    stop = true;
    conv = true;
  }
  return m.xn;
}

// ---------------------------------------------------------------------------
// The whole solve.  Input: the 6 unique entries (any doubles).  Output: lam
// ascending, V[3r + c] = row r of eigenvector c.  kFormF32R differs from
// kFormF64 in its storage, its count of evaluations and the flags it knows;
// kFormF32 uses the zeros of an FP32 Borges-Gragg iteration as they are
// (zeros that it cannot give still come from the FP64 finder).
// Returns branch | it_mu << 8 | it_nu << 16.  bad is set for a matrix with
// a NaN or infinite entry: its outputs are then meaningless (the solve runs
// on the non-finite values, every loop bounded) and the caller stores NaN in
// their place, in a branch that costs nothing when no lane of the wavefront
// takes it.
// ---------------------------------------------------------------------------
struct Vec3 {
  double x, y, z;
};

__device__ __forceinline__ double dot(const Vec3& a, const Vec3& b) {
  return __builtin_fma(a.x, b.x, __builtin_fma(a.y, b.y, a.z * b.z));
}

__device__ __forceinline__ Vec3 normalized(Vec3 u) {
  const double r = rsqrt2(dot(u, u));
  return Vec3{u.x * r, u.y * r, u.z * r};
}

// The high word of |x|: sign cleared, exponent in its upper 11 bits.  Among
// finite numbers it orders by exponent, and it is at least 0x7ff00000 for
// infinities and NaNs alone.
__device__ __forceinline__ uint32_t abs_hi(double x) {
  return (uint32_t)(__builtin_bit_cast(uint64_t, x) >> 32) & 0x7fffffffu;
}

template <bool VECS, int FORM>
__device__ __forceinline__ int solve3(const double (&ain)[6], uint32_t flags,
                                      double (&lam)[3], double (&V)[9], bool& bad) {
  double a11 = ain[0], a12 = ain[1], a13 = ain[2], a22 = ain[3], a23 = ain[4],
         a33 = ain[5];
  // Scale by 2^-e so that max |a_ij| is in [1/2, 1); a zero matrix keeps
  // e = 0.  The exponent and the test for NaN and infinity come from the
  // largest high word: six ANDs at 2 cycles per wavefront and three integer
  // maxima, where six v_cmp and five v_max_f64 took 4 each (the maxima of
  // loaded doubles would be canonicalised besides).
  const uint32_t hi = max(max(max(abs_hi(a11), abs_hi(a12)), max(abs_hi(a13), abs_hi(a22))),
                          max(abs_hi(a23), abs_hi(a33)));
  // Kept as a word from here on: left as a condition the compiler re-derives
  // it at the stores, holding its input through the solve.
  uint32_t badw = hi >= 0x7ff00000u ? 1u : 0u;
  asm volatile("" : "+v"(badw));
  bad = badw != 0u;
  int e = (int)(hi >> 20) - 1022;
  bool zero = false;
  if (hi < 0x00100000u) {
    // zero, or every entry subnormal: a branch of its own (the empty asm)
    asm volatile("");
    const double m = __builtin_fmax(
        __builtin_fmax(__builtin_fmax(dabs(a11), dabs(a12)), __builtin_fmax(dabs(a13), dabs(a22))),
        __builtin_fmax(dabs(a23), dabs(a33)));
    e = __builtin_amdgcn_frexp_exp(m);
    zero = m == 0.0;
  }
  // (The flags are the same for every lane: their alternatives are taken in
  // uniform branches, which the empty asm keeps the compiler from turning
  // into per-lane selects that every lane would pay for.)
  if (flags & kFlagNoScale) {
    asm volatile("");
    e = 0;
  }
  a11 = __builtin_amdgcn_ldexp(a11, -e);
  a12 = __builtin_amdgcn_ldexp(a12, -e);
  a13 = __builtin_amdgcn_ldexp(a13, -e);
  a22 = __builtin_amdgcn_ldexp(a22, -e);
  a23 = __builtin_amdgcn_ldexp(a23, -e);
  a33 = __builtin_amdgcn_ldexp(a33, -e);

  // Sec. 1: ordered arrow
  const Rot2 J = rot2(a11, a12, a22);
  const double al1 = J.l1, al2 = J.l2;
  double be1 = __builtin_fma(J.k11, a13, J.k21 * a23);
  double be2 = __builtin_fma(J.k12, a13, J.k22 * a23);
  const double ga = a33;

  // Sec. 1.1: h = ||beta||, the Givens rotation G and the deflation test.
  // The test |e| <= eps (|d1| + |d2|) on G A G^T, whose off-diagonal entry
  // is e = alpha sg cg and whose diagonal is d1 = alpha1 cg^2 + alpha2 sg^2,
  // d2 = alpha1 sg^2 + alpha2 cg^2 (sg = beta1/h, cg = beta2/h), taken
  // times h^2: |alpha beta1 beta2| <= eps (|alpha1 beta2^2 + alpha2 beta1^2|
  // + |alpha1 beta1^2 + alpha2 beta2^2|).  It needs no root or quotient, so
  // G itself is formed only on lanes that deflate.  The exact beta- and
  // combo-deflations (beta1, beta2 or alpha zero) make the left side zero.
  const double b1s = be1 * be1, b2s = be2 * be2;
  double hh = __builtin_fma(be1, be1, b2s);
  double al = al1 - al2, g1 = ga - al1, g2 = al2 - ga;
  const double ee = al * be1 * be2;
  bool diag = false, defl = false;
  double unscale = 1.0;
  // In the scaled matrix |alpha1|, |alpha2| <= 2 and h^2 < 2, so the right
  // side is below 8 eps = 2^-49 and h^2 >= |ee|/2: a left side above 2^-48
  // neither deflates nor has a negligible h, and a wavefront all of whose
  // lanes are there (all N(0,1), uniform and condition-1e8 SPD ones) skips
  // the tests, 44 cycles.  (An unscaled matrix has no such bounds.)
  if (!(dabs(ee) > 0x1p-48) || (flags & kFlagNoScale)) {
    asm volatile("");
    // h <= eps (|alpha1| + |alpha2| + |gamma|) is tested as h^2 <= (eps ...)^2
    const double tol_h = kEps64 * (dabs(al1) + dabs(al2) + dabs(ga));
    if (flags & kFlagNoHGuard) {
      asm volatile("");
      diag = hh == 0.0;
    } else {
      diag = !(hh > tol_h * tol_h);
    }
    double rhs;
    if (flags & kFlagSimplified) {
      asm volatile("");
      rhs = dabs(al1 + al2) * hh;
    } else {
      rhs =
          dabs(__builtin_fma(al1, b2s, al2 * b1s)) + dabs(__builtin_fma(al1, b1s, al2 * b2s));
    }
    defl = !diag && dabs(ee) <= kEps64 * rhs;
    // An arrow far smaller than the matrix it came from (a nearly isotropic
    // one) is scaled up by a power of two, alpha1, alpha2 and gamma through
    // their differences, so that the zero finder's FP32 start can hold the
    // fourth power of its size: isotropic + 1e-12 N(0,1) then takes one
    // Halley step like any other matrix (2^22 eigenvalues 52 us, against 91
    // from the start in FP64).  The vectors do not change by it, and the
    // zeros are scaled back where they are added to alpha1, alpha2 and
    // gamma.  (Where the tests are skipped the arrow's size is at least the
    // cube root of 2^-48.)
    const double size2 = __builtin_fma(g1, g1, __builtin_fma(g2, g2, hh));
    if (!diag && !defl && !(size2 >= 0x1p-30 && size2 <= 0x1p30)) {
      asm volatile("");
      const int k = __builtin_amdgcn_frexp_exp(size2) >> 1;
      al = __builtin_amdgcn_ldexp(al, -k);
      be1 = __builtin_amdgcn_ldexp(be1, -k);
      be2 = __builtin_amdgcn_ldexp(be2, -k);
      g1 = __builtin_amdgcn_ldexp(g1, -k);
      g2 = __builtin_amdgcn_ldexp(g2, -k);
      hh = __builtin_amdgcn_ldexp(hh, -2 * k);
      unscale = __builtin_amdgcn_ldexp(1.0, k);
    }
  }

  double l0, l1, l2;  // ascending
  Vec3 v0, v1, v2;    // their eigenvectors, arrow coordinates
  int branch, it1 = 0, it2 = 0;
  if (diag || defl) {
    // Two pairs known ordered, (lx, ux) >= (ly, uy); (lz, uz) anywhere.
    double lx, ly, lz;
    Vec3 ux, uy, uz;
    if (defl) {
      // accept d1 with G^T e1 = (cg, -sg, 0); solve [[d2, h], [h, gamma]]
      branch = kDeflated;
      const double rh = rsqrt2(hh);
      const double h = hh * rh;
      const double cg = be2 * rh;  // G = [[cg, -sg, 0], [sg, cg, 0], [0, 0, 1]]
      const double sg = be1 * rh;
      // d1, d2 with the smaller correction: bitwise exact for the beta- and
      // combo-deflations (sg or cg zero, or alpha zero)
      const bool small_s = dabs(sg) <= dabs(cg);
      const double s2 = sg * sg, c2 = cg * cg;
      const double d1 = small_s ? __builtin_fma(-al, s2, al1) : __builtin_fma(al, c2, al2);
      const double d2 = small_s ? __builtin_fma(al, s2, al2) : __builtin_fma(-al, c2, al1);
      const Rot2 T = rot2(d2, h, ga);
      lx = T.l1;
      ly = T.l2;
      lz = d1;
      ux = Vec3{sg * T.k11, cg * T.k11, T.k21};  // G^T (0, p, q)
      uy = Vec3{sg * T.k12, cg * T.k12, T.k22};
      uz = Vec3{cg, -sg, 0.0};
    } else {
      // diagonal arrow: (alpha1, e1), (alpha2, e2), (gamma, e3)
      branch = kDiagonal;
      lx = al1;
      ly = al2;
      lz = ga;
      ux = Vec3{1.0, 0.0, 0.0};
      uy = Vec3{0.0, 1.0, 0.0};
      uz = Vec3{0.0, 0.0, 1.0};
    }
    // Ascending, stable in the listing order x, y, z for ties: when
    // lx == ly the two trade vectors first, so equal eigenvalues keep their
    // arrow order (lambda I and 0 give V = I).
    if (lx == ly) {
      const Vec3 tu = ux;
      ux = uy;
      uy = tu;
    }
    if (lz < ly) {
      l0 = lz; l1 = ly; l2 = lx; v0 = uz; v1 = uy; v2 = ux;
    } else if (lz < lx) {
      l0 = ly; l1 = lz; l2 = lx; v0 = uy; v1 = uz; v2 = ux;
    } else {
      l0 = ly; l1 = lx; l2 = lz; v0 = uy; v1 = ux; v2 = uz;
    }
  } else {
    branch = kReduced;
    double mu = 0.0, nu = 0.0;
    if (FORM == kFormF32) {
      const Arrows P = arrows(al, be1, be2, g1, g2);
      const Arrow1 &P1 = P.mu, &P2 = P.nu;
      // The unrefined FP32 ablation: Borges-Gragg in FP32 from the FP32
      // two-chord start, its zeros used as they are.
      const double rab = rcp1(P1.ab);  // both problems share abar
      const Arrow1f Q1 = to_f32(P1, rab), Q2 = to_f32(P2, rab);
      // the FP32 problem must be representable away from the poles
      bool fb = !(Q1.b1s >= 0x1p-100f && Q1.b2s >= 0x1p-100f && Q1.ab >= 0x1p-60f);
      float y1 = bg_start32(Q1), y2 = bg_start32(Q2);
      bool s1 = false, s2 = false, c1 = false, c2 = false;
      for (int k = 0; k < kMaxIter32; ++k) {
        if (s1 && s2) break;
        if (!s1) { ++it1; y1 = bg_step32(Q1, y1, s1, c1); }
        if (!s2) { ++it2; y2 = bg_step32(Q2, y2, s2, c2); }
      }
      fb = fb || !c1 || !c2 || !(y1 > 0x1p-100f) || !(y2 > 0x1p-100f);
      if (fb) {
        // no usable FP32 zero: the FP64 zero finder from its own start
        int j1, j2;
        zeros_bg(al, be1, be2, g1, g2, hh, false, mu, nu, j1, j2);
        it1 += j1;
        it2 += j2;
      } else {
        mu = (double)y1;
        nu = (double)y2;
      }
    } else if (FORM != kFormF32R && (flags & kFlagNewton)) {
      const Arrows P = arrows(al, be1, be2, g1, g2);
      zeros_newton(P.mu, P.nu, mu, nu, it1, it2);
    } else if (FORM != kFormF32R && (flags & kFlagPaperBG)) {
      const Arrows P = arrows(al, be1, be2, g1, g2);
      zeros_bg_paper(P.mu, P.nu, mu, nu, it1, it2);
    } else {
      zeros_bg(al, be1, be2, g1, g2, hh, FORM != kFormF64 && (flags & kFlagRefineConverge), mu,
               nu, it1, it2);
      if (FORM == kFormF32R) {  // and the two FP32 steps of the start
        it1 += 2;
        it2 += 2;
      }
    }
    // lambda3 <= lambda2 <= lambda1; lambda2 by the trace identity
    l2 = __builtin_fma(mu, unscale, al1);
    l0 = __builtin_fma(-nu, unscale, al2);
    l1 = __builtin_fma(nu, unscale, __builtin_fma(-mu, unscale, ga));
    l1 = __builtin_fmin(__builtin_fmax(l1, l0), l2);
    if (VECS) {
      const double mua = mu + al, nua = nu + al;
      const Vec3 u1{be1 * mua, be2 * mu, mu * mua};
      const Vec3 u3{be1 * nu, be2 * nua, -nu * nua};
      v2 = normalized(u1);
      v0 = normalized(u3);
      if (FORM == kFormF32) {
        // the ablation keeps the paper's formula for u2
        const Vec3 u2{-be2 * mu * nua, be1 * nu * mua, be1 * be2 * al};
        v1 = normalized(u2);
      } else {
        // The paper's u2 is (mu + nu + abar) (u1 x u3), a positive multiple
        // of the cross product (expand u1 x u3 and factor), so the middle
        // vector is taken as the cross product of the two unit vectors:
        // orthogonal to both by construction, and 15 operations cheaper
        // than forming and normalising u2.
        v1 = Vec3{__builtin_fma(v2.y, v0.z, -v2.z * v0.y), __builtin_fma(v2.z, v0.x, -v2.x * v0.z),
                  __builtin_fma(v2.x, v0.y, -v2.y * v0.x)};
      }
    }
  }

  lam[0] = __builtin_amdgcn_ldexp(l0, e);
  lam[1] = __builtin_amdgcn_ldexp(l1, e);
  lam[2] = __builtin_amdgcn_ldexp(l2, e);
  if (VECS) {
    // back to A's coordinates: V = diag(J, 1) [v0 v1 v2]
    V[0] = __builtin_fma(J.k11, v0.x, J.k12 * v0.y);
    V[1] = __builtin_fma(J.k11, v1.x, J.k12 * v1.y);
    V[2] = __builtin_fma(J.k11, v2.x, J.k12 * v2.y);
    V[3] = __builtin_fma(J.k21, v0.x, J.k22 * v0.y);
    V[4] = __builtin_fma(J.k21, v1.x, J.k22 * v1.y);
    V[5] = __builtin_fma(J.k21, v2.x, J.k22 * v2.y);
    V[6] = v0.z;
    V[7] = v1.z;
    V[8] = v2.z;
  }
  if (bad) {
    branch = kNonFinite;
  } else if (zero) {
    branch = kZero;
  }
  return branch | (it1 << 8) | (it2 << 16);
}

}  // namespace syev3
