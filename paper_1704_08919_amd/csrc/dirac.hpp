// Per-mode arithmetic of the momentum-space Dirac evolution in 2x2 blocks (Sec. II A of
// arXiv:1704.08919), shared by the evolution kernels and the yield-gradient kernel: the series
// for the exact exponential of a frozen block Hamiltonian, the block states, the rotation
// applied per step, the initial negative-energy state and the projection on the outgoing
// positive-energy state.  Translation units that include it compile with contraction off and
// write every fused multiply-add out, so each mode's arithmetic is one fixed instruction
// sequence.
#pragma once

#include "common.hpp"
#include "cot_fit.hpp"
#include "tan_fit.hpp"

#pragma clang fp contract(off)

namespace po {
namespace {

constexpr int kChunk = kChunkSteps;   // steps staged per LDS buffer

constexpr double factorial(int n) { return n <= 1 ? 1.0 : double(n) * factorial(n - 1); }
// Maclaurin coefficients of cos(sqrt x) and sin(sqrt x)/sqrt x.
constexpr double cos_coef(int k) { return (k % 2 ? -1.0 : 1.0) / factorial(2 * k); }
constexpr double sinc_coef(int k) { return (k % 2 ? -1.0 : 1.0) / factorial(2 * k + 1); }

// Series variants: T(x) = tan(sqrt x)/sqrt x = 1 + x R(x) with R a polynomial fit of degree
// n - 1 (n = 4..11, tan_fit.hpp: Chebyshev interpolation on [0, X_n], |T_fit - T| <= 2^-57 there,
// about two degrees fewer than the Maclaurin series needs for the same range).  Beyond the last
// X_n, index kFineHalving: C and S of degree 7 (first omitted term x^8/16! < 2^-56 for
// x <= 0.3612; both series alternate with decreasing terms) after h angle halvings.
constexpr int kNumFine = kNumFit;
constexpr int kFineHalving = kNumFine;
constexpr double kCosSinXmax = 0.3612;
constexpr int kMaxHalvings = 60;  // x up to 0.3612 * 4^60 ~ 5e35; beyond (or non-finite) the choice stops here
constexpr double kSqrt3Over6 = 0.28867513459481288225;  // sqrt(3)/6, Gauss-Legendre nodes 1/2 -+ sqrt(3)/6

// Horner step k of the C and S series, coefficients forced to compile-time constants.
template <int K>
__device__ __forceinline__ void horner_cs(double x, double& C, double& S) {
  constexpr double cc = cos_coef(K), sc = sinc_coef(K);
  C = fma(C, x, cc);
  S = fma(S, x, sc);
  if constexpr (K > 0) horner_cs<K - 1>(x, C, S);
}

template <int D>
__device__ __forceinline__ void cos_sinc(double x, double& C, double& S) {
  constexpr double cd = cos_coef(D), sd = sinc_coef(D);
  C = cd;
  S = sd;
  horner_cs<D - 1>(x, C, S);
}

// Coefficients of the fit of variant V, put in scalar registers where the caller loads them: the
// empty asm statement per value keeps the compiler from materialising the constants of every
// variant of a kernel at its entry (which exhausts the scalar registers); the values are unchanged.
template <int V>
struct Fit {
  double c[kFitDegree[V]];
};

template <int V>
__device__ __forceinline__ Fit<V> load_fit() {
  Fit<V> f;
#pragma unroll
  for (int k = 0; k < kFitDegree[V]; ++k) {
    f.c[k] = kFitCoef[V][k];
    asm volatile("" : "+s"(f.c[k]));
  }
  return f;
}

// R(x) = (T(x) - 1)/x of variant V (degree kFitDegree[V] - 1), by Horner's rule.
template <int V>
__device__ __forceinline__ double fit_R(double x, const Fit<V>& f) {
  constexpr int n = kFitDegree[V];
  double R = f.c[n - 1];
#pragma unroll
  for (int k = n - 2; k >= 0; --k) R = fma(R, x, f.c[k]);
  return R;
}

// T(x) = tan(sqrt x)/sqrt x of variant V: kFitDegree[V] fused multiply-adds.
template <int V>
__device__ __forceinline__ double tan_ratio(double x, const Fit<V>& f) {
  return fma(fit_R<V>(x, f), x, 1.0);
}

// (a_r, a_i, b_r, b_i) of block s = +1 and (c_r, c_i, d_r, d_i) of block s = -1.
struct State {
  double ar, ai, br, bi, cr, ci, dr, di;
};

// psi <- (C - i S Q_s) psi for both blocks:
//   s = +1:  a' = (C - i sz) a + (-sy - i sx) b ;  b' = (sy - i sx) a + (C + i sz) b,  s_q = S q;
//   s = -1:  the same with sy -> -sy.
__device__ __forceinline__ void rotate(State& v, double C, double S, double qx, double qy, double qz) {
  const double sx = S * qx, sy = S * qy, sz = S * qz;
  const double ar = fma(sx, v.bi, fma(-sy, v.br, fma(sz, v.ai, C * v.ar)));
  const double ai = fma(-sx, v.br, fma(-sy, v.bi, fma(-sz, v.ar, C * v.ai)));
  const double br = fma(-sz, v.bi, fma(C, v.br, fma(sx, v.ai, sy * v.ar)));
  const double bi = fma(sz, v.br, fma(C, v.bi, fma(-sx, v.ar, sy * v.ai)));
  const double cr = fma(sx, v.di, fma(sy, v.dr, fma(sz, v.ci, C * v.cr)));
  const double ci = fma(-sx, v.dr, fma(sy, v.di, fma(-sz, v.cr, C * v.ci)));
  const double dr = fma(-sz, v.di, fma(C, v.dr, fma(sx, v.ci, -sy * v.cr)));
  const double di = fma(sz, v.dr, fma(C, v.di, fma(-sx, v.cr, -sy * v.ci)));
  v = State{ar, ai, br, bi, cr, ci, dr, di};
}

// ---------------------------------------------------------------------------------------------
// Cotangent form of the step.  With everything in units of e = e_perp, q' = (p - A)/e, y = |q'|^2
// and z = (e dt)^2, x = (omega dt)^2 = z (1 + y), the step is a multiple of
//     K' - i (q'_x tau_x + s q'_y tau_y + tau_z),   K' = sqrt(x) cot(sqrt x) / (e dt):
// the tau_z coefficient is exactly 1, so its terms enter the FMA chains as addends and the three
// products T q of the tangent form disappear; and K is smooth up to x = pi^2 (T only up to
// pi^2/4), so its fits are a degree shorter at the same bound and reach x = 2.5 instead of 0.26.
// Per mode-step: 2 FMAs (q'), 2 (y), n (K' as a polynomial in y), 24 (two blocks): 28 + n
// instructions against 31 + n with a larger n.  The state grows by about 1/(e dt) per step and is
// rescaled by an exact power of two every few steps (kGroupLong or kGroupShort).
// ---------------------------------------------------------------------------------------------
constexpr int kCotHalving = kNumCot;  // variant index beyond the fits: the angle-halving path
// Steps between two rescalings.  A step multiplies the norm by sqrt(x)/sin(sqrt x)/(e dt), at most
// 1.6/dt for x <= 2.5: 64 steps stay below 2^960 for dt >= 2^-14, 16 steps for dt >= 2^-59; a
// smaller dt takes the angle-halving path (no halvings needed there, the state does not grow).
constexpr int kGroupLong = 64, kGroupShort = 16;
constexpr double kGroupLongMinDt = 0x1p-14, kGroupShortMinDt = 0x1p-59;

// A mode in the cotangent form: -1/e, p/e and e; per chunk z = (e dt)^2 and 1/(e dt) as hi + lo (the
// rounding of e dt and of the quotient would otherwise act as a fixed relative error of every
// step's angle).
struct CotMode {
  double nie, px, py, e;
};
struct CotStep {
  double z, ih, il;
};

__device__ __forceinline__ CotMode cot_mode(double px, double py, double e) {
  const double ie = 1.0 / e;
  return CotMode{-ie, px * ie, py * ie, e};
}

__device__ __forceinline__ CotStep cot_step_size(double e, double dt) {
  const double qz = e * dt, ih = 1.0 / qz;
  return CotStep{qz * qz, ih, ih * (fma(-ih, qz, 1.0) - ih * fma(e, dt, -qz))};
}

// K' for variant V.  Degrees up to kCotInline: per-lane coefficients of K(z (1 + y))/(e dt) in powers
// of y (the fit's coefficients scaled by powers of z, a Taylor shift by 1, the division by e dt), n
// FMAs per step.  Higher degrees, which large steps take, would need too many registers that way:
// their fit stays in scalar registers and x = z (1 + y) and the division cost three more.
constexpr int kCotInline = 8;

template <int V, bool INLINE = (kCotDegree[V] <= kCotInline)>
struct CotCoef {
  double c[kCotDegree[V] + 1];
};
template <int V>
struct CotCoef<V, false> {
  double r[kCotDegree[V]];
  CotStep s;
};

template <int V>
__device__ __forceinline__ CotCoef<V> cot_coef(const CotStep& m) {
  constexpr int n = kCotDegree[V];
  CotCoef<V> k;
  if constexpr (n <= kCotInline) {
    k.c[0] = 1.0;
    double zp = m.z;
#pragma unroll
    for (int j = 0; j < n; ++j) {
      double r = kCotCoef[V][j];
      asm volatile("" : "+s"(r));  // as load_fit: keeps the constants of other variants out of registers
      k.c[j + 1] = r * zp;
      zp *= m.z;
    }
#pragma unroll
    for (int i = 0; i < n; ++i)
#pragma unroll
      for (int j = n - 1; j >= i; --j) k.c[j] += k.c[j + 1];
    k.c[0] = fma(k.c[0], m.ih, k.c[0] * m.il);
#pragma unroll
    for (int j = 1; j <= n; ++j) k.c[j] *= m.ih;
  } else {
    k.s = m;
#pragma unroll
    for (int j = 0; j < n; ++j) {
      k.r[j] = kCotCoef[V][j];
      asm volatile("" : "+s"(k.r[j]));
    }
  }
  return k;
}

template <int V>
__device__ __forceinline__ double cot_K(double y, const CotCoef<V>& k) {
  constexpr int n = kCotDegree[V];
  if constexpr (n <= kCotInline) {
    double K = k.c[n];
#pragma unroll
    for (int j = n - 1; j >= 0; --j) K = fma(K, y, k.c[j]);
    return K;
  } else {
    const double x = fma(y, k.s.z, k.s.z);
    double R = k.r[n - 1];
#pragma unroll
    for (int j = n - 2; j >= 0; --j) R = fma(R, x, k.r[j]);
    const double K = fma(R, x, 1.0);
    return fma(K, k.s.ih, K * k.s.il);
  }
}

// One step with q'_x, q'_y given and xx = q'_x^2.  K times the component comes last: K is 1/(e dt) times the other
// terms, whose sum is then rounded at their own size, so a component takes one large rounding per step, not three.
template <int V>
__device__ __forceinline__ void step_cot_q(State& v, double qx, double qy, double xx, const CotCoef<V>& k) {
  const double K = cot_K<V>(fma(qy, qy, xx), k);
  const double ar = fma(K, v.ar, fma(qx, v.bi, fma(-qy, v.br, v.ai)));
  const double ai = fma(K, v.ai, fma(-qx, v.br, fma(-qy, v.bi, -v.ar)));
  const double br = fma(K, v.br, fma(qx, v.ai, fma(qy, v.ar, -v.bi)));
  const double bi = fma(K, v.bi, fma(-qx, v.ar, fma(qy, v.ai, v.br)));
  const double cr = fma(K, v.cr, fma(qx, v.di, fma(qy, v.dr, v.ci)));
  const double ci = fma(K, v.ci, fma(-qx, v.dr, fma(qy, v.di, -v.cr)));
  const double dr = fma(K, v.dr, fma(qx, v.ci, fma(-qy, v.cr, -v.di)));
  const double di = fma(K, v.di, fma(-qx, v.cr, fma(-qy, v.ci, v.dr)));
  v = State{ar, ai, br, bi, cr, ci, dr, di};
}

template <int V>
__device__ __forceinline__ void step_cot(State& v, double2 A, const CotMode& m, const CotCoef<V>& k) {
  const double qx = fma(A.x, m.nie, m.px), qy = fma(A.y, m.nie, m.py);
  step_cot_q<V>(v, qx, qy, qx * qx, k);
}

// Rescales both blocks by one exact power of two so that the largest component of the first lies
// in [1/2, 1) (no squares: the components may be near the ends of the exponent range).
__device__ __forceinline__ void rescale(State& v) {
  const double m = fmax(fmax(fabs(v.ar), fabs(v.ai)), fmax(fabs(v.br), fabs(v.bi)));
  const int e = -__builtin_amdgcn_frexp_exp(m);
  v.ar = ldexp(v.ar, e); v.ai = ldexp(v.ai, e); v.br = ldexp(v.br, e); v.bi = ldexp(v.bi, e);
  v.cr = ldexp(v.cr, e); v.ci = ldexp(v.ci, e); v.dr = ldexp(v.dr, e); v.di = ldexp(v.di, e);
}

// psi <- P psi for both blocks, P given by its first column (a multiple of an SU(2) matrix is
// [[a, -conj b], [b, conj a]]).  |P| is in [1/2, 2), so a few products may go by between two rescalings;
// these are exact, so their places do not affect the result.
__device__ __forceinline__ void apply_propagator(State& s, const State& p) {
  const double ar = fma(-p.bi, s.bi, fma(-p.br, s.br, fma(-p.ai, s.ai, p.ar * s.ar)));
  const double ai = fma(p.bi, s.br, fma(-p.br, s.bi, fma(p.ai, s.ar, p.ar * s.ai)));
  const double br = fma(p.ai, s.bi, fma(p.ar, s.br, fma(-p.bi, s.ai, p.br * s.ar)));
  const double bi = fma(-p.ai, s.br, fma(p.ar, s.bi, fma(p.bi, s.ar, p.br * s.ai)));
  const double cr = fma(-p.di, s.di, fma(-p.dr, s.dr, fma(-p.ci, s.ci, p.cr * s.cr)));
  const double ci = fma(p.di, s.dr, fma(-p.dr, s.di, fma(p.ci, s.cr, p.cr * s.ci)));
  const double dr = fma(p.ci, s.di, fma(p.cr, s.dr, fma(-p.di, s.ci, p.dr * s.cr)));
  const double di = fma(-p.ci, s.dr, fma(p.cr, s.di, fma(p.di, s.cr, p.dr * s.ci)));
  s = State{ar, ai, br, bi, cr, ci, dr, di};
}

// C = cos sqrt x, S = sin sqrt x / sqrt x from the degree-7 series at x / 4^h and h double-angle steps.
__device__ __forceinline__ void cos_sinc_halved(double x, int h, double inv4h, double& C, double& S) {
  double xs = x * inv4h;
  cos_sinc<7>(xs, C, S);
  for (int i = 0; i < h; ++i) {
    const double c2 = fma(C, C, -(xs * S) * S);
    S = S * C;
    C = c2;
    xs *= 4.0;
  }
}

// psi <- (C - i s . tau) psi for one block (a, b); the term with C, the largest for small steps, last.
__device__ __forceinline__ void rotate_block(double& ar, double& ai, double& br, double& bi, double C, double sx,
                                             double sy, double sz) {
  const double nar = fma(C, ar, fma(sx, bi, fma(-sy, br, sz * ai)));
  const double nai = fma(C, ai, fma(-sx, br, fma(-sy, bi, -(sz * ar))));
  const double nbr = fma(C, br, fma(-sz, bi, fma(sx, ai, sy * ar)));
  const double nbi = fma(C, bi, fma(sz, br, fma(-sx, ar, sy * ai)));
  ar = nar; ai = nai; br = nbr; bi = nbi;
}

// A lane's state in slot `slot` of a propagator buffer [slot][8 components][256 lanes].
__device__ __forceinline__ void store_state(double* __restrict__ buf, int64_t slot, const State& v) {
  double* p = buf + slot * kSlotDoubles + threadIdx.x;
  p[0] = v.ar; p[kItem] = v.ai; p[2 * kItem] = v.br; p[3 * kItem] = v.bi;
  p[4 * kItem] = v.cr; p[5 * kItem] = v.ci; p[6 * kItem] = v.dr; p[7 * kItem] = v.di;
}

__device__ __forceinline__ State load_state(const double* __restrict__ buf, int64_t slot, int lane) {
  const double* p = buf + slot * kSlotDoubles + lane;
  return State{p[0], p[kItem], p[2 * kItem], p[3 * kItem], p[4 * kItem], p[5 * kItem], p[6 * kItem], p[7 * kItem]};
}

// Applies the n propagators from slot `slot` on to a lane's state, in order; the loads of four are in
// flight together.
constexpr int kApplyBatch = 4;

__device__ __forceinline__ void apply_segments(State& psi, const double* __restrict__ buf, int64_t slot, int n, int lane) {
  for (int s0 = 0; s0 < n; s0 += kApplyBatch) {
    State v[kApplyBatch];
#pragma unroll
    for (int k = 0; k < kApplyBatch; ++k) v[k] = load_state(buf, slot + min(s0 + k, n - 1), lane);
#pragma unroll
    for (int k = 0; k < kApplyBatch; ++k)
      if (s0 + k < n) apply_propagator(psi, v[k]);
    rescale(psi);
  }
}

// Negative-energy eigenvector of h_s(P): (-(P_x - i s P_y), w + e) / sqrt(2 w (w + e)).
__device__ __forceinline__ void init_state(State& v, double Px, double Py, double e) {
  const double w = sqrt(fma(Px, Px, fma(Py, Py, e * e)));
  const double n = 1.0 / sqrt((2.0 * w) * (w + e));
  v.ar = -Px * n; v.ai = Py * n;  v.br = (w + e) * n; v.bi = 0.0;   // s = +1
  v.cr = -Px * n; v.ci = -Py * n; v.dr = (w + e) * n; v.di = 0.0;   // s = -1
}

// f = sum_s |<+_s(P)|psi_s>|^2 / |psi_s|^2 with |+_s> = (w + e, P_x + i s P_y) / sqrt(2 w (w + e)).
__device__ __forceinline__ double project(const State& v, double Px, double Py, double e) {
  const double w = sqrt(fma(Px, Px, fma(Py, Py, e * e)));
  const double we = w + e;
  const double n2 = 1.0 / ((2.0 * w) * we);
  // s = +1: (w+e) a + (P_x - i P_y) b
  const double r1 = fma(Py, v.bi, fma(Px, v.br, we * v.ar));
  const double i1 = fma(-Py, v.br, fma(Px, v.bi, we * v.ai));
  // s = -1: (w+e) c + (P_x + i P_y) d
  const double r2 = fma(-Py, v.di, fma(Px, v.dr, we * v.cr));
  const double i2 = fma(Py, v.dr, fma(Px, v.di, we * v.ci));
  const double m1 = fma(v.bi, v.bi, fma(v.br, v.br, fma(v.ai, v.ai, v.ar * v.ar)));
  const double m2 = fma(v.di, v.di, fma(v.dr, v.dr, fma(v.ci, v.ci, v.cr * v.cr)));
  return (fma(i1, i1, r1 * r1) / m1 + fma(i2, i2, r2 * r2) / m2) * n2;
}
}  // namespace
}  // namespace po
