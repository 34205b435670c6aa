// Gradient of the pair yield J = dV sum_p f(p) with respect to the vector-potential table: the
// exact derivative (discrete adjoint) of the exponential-midpoint Dirac scheme of Sec. II A.  It
// serves the local search of Sec. IV A, which needs the gradient of the objective with respect to
// the field parameters; the paper obtains it from the adjoint of the kinetic equation, here it is
// the adjoint of the Dirac steps that evaluate J.
//
// Per block s and mode, f_s = |alpha_s|^2 with alpha_s = <+_s(P_out)| U_{N-1} ... U_0 |-_s(P_in)>
// and U_n = exp(-i q_n . tau), q_n = dt (P_x, s P_y, e_perp), P = p - A_n.  With the forward
// states psi_n = U_{n-1} ... U_0 |-> and the backward states chi_n = U_n^+ ... U_{N-1}^+ |+>,
//     df_s / dA_n = 2 Re[ conj(alpha_s) <chi_{n+1}| dU_n/dA_n |psi_n> ],
// and, writing U = C - i S q.tau with C = cos|q|, S = sin|q|/|q|, D = (C - S)/|q|^2,
//     dU/dq_j = q_j (-S - i D q.tau) - i S tau_j,   dq_x/dA_x = -dt,  dq_y/dA_y = -s dt.
// The initial and final states depend on A(t_i) and A(t_f) through P_in and P_out (first-order
// perturbation of the block eigenvectors, energies -+ omega):
//     d|->  = -|+><+|dh|->/(2 omega),   d<+|psi> = <+|dh|-><-|psi>/(2 omega),   dP = -dA.
//
// Since f_s is the same with chi_s replaced by alpha_s chi_s, each term is
// 2 Re <chi'_{n+1}| dU/dq_j |psi_n> with chi'_s = alpha_s chi_s, and it depends on the two states
// only through W_s = Im <chi'_s|tau|psi_s>, a real 3-vector that the backward steps rotate.
//
// Three kernels.  The forward sweep is the evolution's own segment kernel: per mode and time segment
// the propagators of the two blocks.  k_grad_join, one lane per mode, applies them to the initial
// state, takes f, the final-state terms and W at t_f, moves W back segment by segment (the
// rotation a propagator induces) and leaves W at the end of each segment in the segment's slot.
// k_grad_back then runs the backward steps of every (256-mode item, segment) at once: each step forms
// the derivative terms and rotates W_{n+1} to W_n, and the terms are summed over the item's modes in a
// fixed order: each lane stores its terms for 8 steps in LDS, the wave reads them back transposed
// (lane (j, p) adds the lanes p, p + 8, ..., p + 56 of step j), pairs up the 8 lanes of a step (DPP), and
// the four waves are added in order.  The results are item partials [item][n][2]; k_grad_reduce
// sums the items of each pulse in order.  So the gradient, like J, does not depend on scheduling.
#include "dirac.hpp"
#include "reduce.hpp"
#include "select.hpp"

#pragma clang fp contract(off)

namespace po {
namespace {

// C = cos sqrt x and S = sin sqrt x / sqrt x by their degree-7 series (x <= 0.3612 keeps both
// remainders below 2^-56), and D = (C - S)/x = C1 - S1, where C = 1 + x C1 and S = 1 + x S1 are the
// last Horner steps (no cancellation: C1 ~ -1/2, S1 ~ -1/6; remainder of D below 2^-54).
template <int K>
__device__ __forceinline__ void horner_cs1(double x, double& C, double& S) {
  constexpr double cc = cos_coef(K), sc = sinc_coef(K);
  C = fma(C, x, cc);
  S = fma(S, x, sc);
  if constexpr (K > 1) horner_cs1<K - 1>(x, C, S);
}

__device__ __forceinline__ void csd_series(double x, double& C, double& S, double& D) {
  constexpr double c7 = cos_coef(7), s7 = sinc_coef(7);
  double C1 = c7, S1 = s7;
  horner_cs1<6>(x, C1, S1);
  D = C1 - S1;
  C = fma(C1, x, 1.0);
  S = fma(S1, x, 1.0);
}

// The same after h halvings of the angle (x / 4^h in the series range, h double-angle steps for C
// and S).  The halving count comes from the block's bound on x, so a single mode-step here can
// have any x >= (e_perp dt)^2; D = (C - S)/x then loses digits to cancellation (C - S ~ -x/3, so
// D carries a relative error of about 3 x 2^-53 / x: 3e-13 at the DE workload's smallest
// x = dt^2 = 2.4e-3), far inside the gradient's error bar.
__device__ __forceinline__ void csd(double x, int h, double inv4h, double& C, double& S, double& D) {
  if (h == 0) {
    csd_series(x, C, S, D);
  } else {
    cos_sinc_halved(x, h, inv4h, C, S);
    D = (C - S) / x;
  }
}

struct Blk {
  double ar, ai, br, bi;
};

// Block s (0: s = +1, 1: s = -1) of a two-block state.
__device__ __forceinline__ Blk block_of(const State& v, int s) {
  return s == 0 ? Blk{v.ar, v.ai, v.br, v.bi} : Blk{v.cr, v.ci, v.dr, v.di};
}

// Unit eigenvectors of h_s(P) = P_x tau_x + s P_y tau_y + e tau_z: |+> = (w + e, P_x + i s P_y)/N,
// |-> = (-(P_x - i s P_y), w + e)/N, N = sqrt(2 w (w + e)).
__device__ __forceinline__ void eig_pm(double Px, double Py, double e, double s, Blk& up, Blk& dn, double& w) {
  w = sqrt(fma(Px, Px, fma(Py, Py, e * e)));
  const double n = 1.0 / sqrt((2.0 * w) * (w + e));
  up = Blk{(w + e) * n, 0.0, Px * n, s * Py * n};
  dn = Blk{-(Px * n), s * Py * n, (w + e) * n, 0.0};
}

// <a|b> for two block vectors.
__device__ __forceinline__ void inner(const Blk& a, const Blk& b, double& r, double& i) {
  r = fma(a.ar, b.ar, fma(a.ai, b.ai, fma(a.br, b.br, a.bi * b.bi)));
  i = fma(a.ar, b.ai, fma(-a.ai, b.ar, fma(a.br, b.bi, -(a.bi * b.br))));
}

// <x|tau_x|y> and <x|s tau_y|y>.
__device__ __forceinline__ void tau_xy(const Blk& x, const Blk& y, double s, double& xr, double& xi, double& yr,
                                       double& yi) {
  // conj(x1) y2 + conj(x2) y1
  const double a_r = fma(x.ar, y.br, x.ai * y.bi), a_i = fma(x.ar, y.bi, -(x.ai * y.br));  // conj(x1) y2
  const double b_r = fma(x.br, y.ar, x.bi * y.ai), b_i = fma(x.br, y.ai, -(x.bi * y.ar));  // conj(x2) y1
  xr = a_r + b_r;
  xi = a_i + b_i;
  // tau_y: -i conj(x1) y2 + i conj(x2) y1
  yr = s * (a_i - b_i);
  yi = s * (b_r - a_r);
}

// The backward sweep carries, per block, the real 3-vector W = Im <chi'|tau|psi> instead of the two
// states.  Moving both states back by one step changes V_k = <chi'|tau_k|psi> by the rotation that
// the step induces on the Pauli vector,
//     U tau_k U^+ = (C^2 - S^2 x) tau_k + 2 S^2 q_k (q.tau) - 2 C S (e_k x q).tau,
// which is real, so W_n = (C^2 - S^2 x) W + 2 S^2 (q.W) q - 2 C S (q x W) with W = W_{n+1}.  And
// since dU/dq_j U^+ = -i [q_j (S^2 + C D) q.tau + C S tau_j - S^2 (e_j x q).tau] has no identity part,
//     Re <chi'_{n+1}| dU/dq_j |psi_n> = Re <chi'_{n+1}| dU/dq_j U^+ |psi_{n+1}>
//                                    = q_j (S^2 + C D)(q.W) + C S W_j - S^2 (q x W)_j.
// Block s = -1 has q = (q_x, -q_y, q_z); its y term enters with the sign s (dq_y/dA_y = -s dt).
struct WPair {
  double ax, ay, az;  // block s = +1
  double bx, by, bz;  // block s = -1
};

// One backward step on W given the step's coefficients: k1 = C^2 - S^2 x, kq = 2 S^2, cb = S^2 + C D,
// cs = C S, and the cross products u x W with u = l q, where the rotation takes -(2 C S / l) (u x W)
// and the terms -(S^2 / l) (u x W).  Returns the two terms summed over the blocks.
__device__ __forceinline__ double2 back_w(WPair& w, double qx, double qy, double qz, double k1, double kq, double cb,
                                          double cs, double l, double rot_c, double term_c) {
  const double ux = l * qx, uy = l * qy, uz = l * qz;
  const double p0 = fma(qz, w.az, fma(qy, w.ay, qx * w.ax));
  const double p1 = fma(qz, w.bz, fma(-qy, w.by, qx * w.bx));
  const double c0x = fma(uy, w.az, -(uz * w.ay)), c0y = fma(uz, w.ax, -(ux * w.az)), c0z = fma(ux, w.ay, -(uy * w.ax));
  const double c1x = fma(-uy, w.bz, -(uz * w.by)), c1y = fma(uz, w.bx, -(ux * w.bz)), c1z = fma(ux, w.by, uy * w.bx);
  const double bp = cb * (p0 + p1);
  const double gx = fma(qx, bp, fma(-term_c, c0x + c1x, cs * (w.ax + w.bx)));
  const double gy = fma(qy, bp, fma(-term_c, c0y - c1y, cs * (w.ay - w.by)));
  const double kp0 = kq * p0, kp1 = kq * p1;
  w.ax = fma(k1, w.ax, fma(kp0, qx, -(rot_c * c0x)));
  w.ay = fma(k1, w.ay, fma(kp0, qy, -(rot_c * c0y)));
  w.az = fma(k1, w.az, fma(kp0, qz, -(rot_c * c0z)));
  w.bx = fma(k1, w.bx, fma(kp1, qx, -(rot_c * c1x)));
  w.by = fma(k1, w.by, fma(-kp1, qy, -(rot_c * c1y)));
  w.bz = fma(k1, w.bz, fma(kp1, qz, -(rot_c * c1z)));
  return make_double2(gx, gy);
}

// Exact C, S form (the angle-halving path): l = 1, the products with 2 C S and S^2 are explicit.
__device__ __forceinline__ double2 back_w_exact(WPair& w, double qx, double qy, double qz, int h, double inv4h) {
  double C, S, D;
  const double x = fma(qx, qx, fma(qy, qy, qz * qz));
  csd(x, h, inv4h, C, S, D);
  const double S2 = S * S, cs = C * S;
  return back_w(w, qx, qy, qz, fma(-S2, x, C * C), S2 + S2, fma(C, D, S2), cs, 1.0, cs + cs, S2);
}

// Within the fits' range.  In units of e_perp (q = e dt q', q'_z = 1, y = |q'|^2 - 1, z = (e dt)^2, x = z (1
// + y)) with v = q' x W, T = tan(sqrt x)/sqrt x, R = (T - 1)/x, k = 2 C S = sin(2 sqrt x)/sqrt x, the rotation is
//     W_n = W - k e dt (v - T e dt q' x v),
// and since dU/dq_j U^+ = -i int_0^1 exp(-i s q.tau) tau_j exp(i s q.tau) ds, a term is the mean of the
// rotating W over the step:
//     2 Re <chi'_{n+1}| dU/dq_j |psi_n> = T (W_n + W_{n+1})_j - 2 R z q'_j (q'.W).
// So beside the two cross products per block a step needs only T and R (one fit), k (a series of its own:
// no cancellation), and the sums of W over the blocks: 48 + n + m FP64 instructions for degrees n and
// m, against 63 + n + m when the terms are formed from C, S and D separately.
// k = sum_j 2 (-4)^j x^j / (2 j + 1)!, alternating with decreasing terms; kFitCos2Degree[v] terms (of the
// series of cos^2, whose terms are larger) keep its remainder below 2^-59 up to the variant's largest x.
constexpr double pow4i(int n) { return n == 0 ? 1.0 : 4.0 * pow4i(n - 1); }
constexpr double sin2_coef(int j) { return (j % 2 ? -2.0 : 2.0) * pow4i(j) / factorial(2 * j + 1); }

// Read from memory where a variant starts: as literals the compiler would set those that several
// variants share at kernel entry.
__constant__ double kSin2Coef[10] = {sin2_coef(0), sin2_coef(1), sin2_coef(2), sin2_coef(3), sin2_coef(4),
                                     sin2_coef(5), sin2_coef(6), sin2_coef(7), sin2_coef(8), sin2_coef(9)};

struct BackMode {
  double nie, px, py, qz, z, z2;  // -1/e, p/e, e dt, (e dt)^2, 2 (e dt)^2
};

template <int MODE>
struct BackFit {
  Fit<MODE> f;
  double k[kFitCos2Degree[MODE] + 1];
};

template <int MODE>
__device__ __forceinline__ BackFit<MODE> load_back_fit() {
  BackFit<MODE> b;
  b.f = load_fit<MODE>();
  const double* k = kSin2Coef;
  asm volatile("" : "+s"(k));
#pragma unroll
  for (int j = 0; j <= kFitCos2Degree[MODE]; ++j) b.k[j] = k[j];
  return b;
}

// One backward step within the fits' range; s holds (ax + bx, ay - by) on entry and exit.  Returns twice
// the terms summed over the blocks.
template <int MODE>
__device__ __forceinline__ double2 back_step(WPair& w, double2& s, double2 A, const BackMode& m, const BackFit<MODE>& f) {
  const double qx = fma(A.x, m.nie, m.px), qy = fma(A.y, m.nie, m.py);
  const double x = fma(fma(qx, qx, qy * qy), m.z, m.z);
  const double R = fit_R<MODE>(x, f.f), T = fma(R, x, 1.0);
  double k = f.k[kFitCos2Degree[MODE]];
#pragma unroll
  for (int j = kFitCos2Degree[MODE] - 1; j >= 0; --j) k = fma(k, x, f.k[j]);
  const double kq = k * m.qz, tz = T * m.qz, tx = tz * qx, ty = tz * qy;
  {
    const double vx = fma(qy, w.az, -w.ay), vy = fma(-qx, w.az, w.ax), vz = fma(qx, w.ay, -(qy * w.ax));
    w.ax = fma(-kq, fma(tz, vy, fma(-ty, vz, vx)), w.ax);
    w.ay = fma(-kq, fma(tx, vz, fma(-tz, vx, vy)), w.ay);
    w.az = fma(-kq, fma(ty, vx, fma(-tx, vy, vz)), w.az);
  }
  {
    const double vx = fma(-qy, w.bz, -w.by), vy = fma(-qx, w.bz, w.bx), vz = fma(qx, w.by, qy * w.bx);
    w.bx = fma(-kq, fma(tz, vy, fma(ty, vz, vx)), w.bx);
    w.by = fma(-kq, fma(tx, vz, fma(-tz, vx, vy)), w.by);
    w.bz = fma(-kq, fma(-ty, vx, fma(-tx, vy, vz)), w.bz);
  }
  const double2 n = make_double2(w.ax + w.bx, w.ay - w.by);
  const double rp = (R * m.z2) * fma(qx, n.x, fma(qy, n.y, w.az + w.bz));
  const double2 g = make_double2(fma(T, s.x + n.x, -(rp * qx)), fma(T, s.y + n.y, -(rp * qy)));
  s = n;
  return g;
}

// Lane-to-lane moves inside rows of 16 (DPP): pairs (l, l^1), (l, l^2), l <-> 7 - l within 8 lanes and
// l <-> 15 - l within 16 lanes.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

template <int CTRL>
__device__ __forceinline__ double dpp_get(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// Sum over each aligned group of L lanes (L = 8 or 16); every lane of a group gets the same value.
template <int L>
__device__ __forceinline__ double group_sum(double v) {
  v += dpp_get<kDppXor1>(v);
  v += dpp_get<kDppXor2>(v);
  v += dpp_get<kDppHalfMirror>(v);
  if constexpr (L == 16) v += dpp_get<kDppMirror>(v);
  return v;
}

// Per-step sums over the 64 lanes of a wave for kGroup steps at once: each lane has written its
// (gx, gy) of step j to buf[j][lane]; lane (j, p) (j = lane / L, p = lane % L, L = 64 / kGroup)
// adds the lanes p, p + L, ... in order, then the L lanes of its step pair up.  Lane p = 0 of step
// j returns the wave's sum of step j.
constexpr int kGroup = 8;
constexpr int kLanesPerStep = 64 / kGroup;

__device__ __forceinline__ double2 group_reduce(const double2 (*buf)[64], int lane) {
  const int j = lane / kLanesPerStep, p = lane % kLanesPerStep;
  double2 v = buf[j][p];
#pragma unroll
  for (int i = 1; i < kGroup; ++i) {
    const double2 u = buf[j][i * kLanesPerStep + p];
    v.x += u.x;
    v.y += u.y;
  }
  return make_double2(group_sum<kLanesPerStep>(v.x), group_sum<kLanesPerStep>(v.y));
}

// Reduces a group of cnt steps (rows 0..cnt-1 of buf, steps top, top - 1, ...) and stores the
// wave's step sums in red[top - j].  The wave reads what its own lanes wrote: the fences complete
// the stores before the loads and the loads before the next group's stores (no other wave uses buf).
__device__ __forceinline__ void group_store(double2 (*buf)[64], double2* red, int lane, int top, int cnt) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  const double2 v = group_reduce(buf, lane);
  const int j = lane / kLanesPerStep;
  if (lane % kLanesPerStep == 0 && j < cnt) red[top - j] = v;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

struct GradArgs {
  const PulseDev* desc;  // of the group's pulses
  int n_pulses;
  int64_t slot0, part0;  // first slot, first partial and first item of the group in the batch
  int item0, items;
  const double* A;
  const double* Aedge;
  const double* ranges;
  double* prop;         // [slots][8][256]: propagators in, W at the segments' ends out (6 components)
  double* part;         // [items of pulse][nt][2] per pulse
  double* epart;        // [items][4 waves][4]: dA(t_i) x, y, dA(t_f) x, y
  double* units;        // 64-mode sums of f
};

constexpr int kWaves = kItem / 64;

// W <- R^T W for the rotation that the propagator (w - i v.tau) / |.| induces (its first column (a, b) of
// a block: a = w - i v_z, b = v_y - i v_x): W + (2 / |.|^2) (v x t - w t) with t = v x W.
__device__ __forceinline__ void rotate_back(double& wx, double& wy, double& wz, double ar, double ai, double br,
                                            double bi) {
  const double w = ar, vx = -bi, vy = br, vz = -ai;
  const double s = 2.0 / fma(bi, bi, fma(br, br, fma(ai, ai, ar * ar)));
  const double tx = fma(vy, wz, -(vz * wy)), ty = fma(vz, wx, -(vx * wz)), tz = fma(vx, wy, -(vy * wx));
  const double dx = fma(vy, tz, fma(-vz, ty, -(w * tx))), dy = fma(vz, tx, fma(-vx, tz, -(w * ty))),
               dz = fma(vx, ty, fma(-vy, tx, -(w * tz)));
  wx = fma(s, dx, wx);
  wy = fma(s, dy, wy);
  wz = fma(s, dz, wz);
}

// One lane per mode, one wave per workgroup (as k_join_segments).
__global__ void __launch_bounds__(64) k_grad_join(GradArgs a) {
  const int rel = blockIdx.x / kWaves, wave = blockIdx.x % kWaves, lane = wave * 64 + threadIdx.x;
  const int pi = find_pulse_item(a.desc, a.n_pulses, a.item0 + rel);
  const PulseDev& d = a.desc[pi];
  const int li = a.item0 + rel - d.item_off;
  const int64_t m = int64_t(li) * kItem + lane, slot = d.slot_off - a.slot0 + int64_t(li) * d.nseg;
  const double2* edge = reinterpret_cast<const double2*>(a.Aedge) + 2 * pi;
  const double2 ain = edge[0], aout = edge[1];
  // modes that stand for a mirror image count twice: everything after t_f is linear in alpha_s^* psi
  const double weight = m >= d.ndist ? 0.0 : mirror_mode(d, m) != m ? 2.0 : 1.0;
  double px, py;
  const double e = lane_mode(d, m, px, py);
  State psi;
  init_state(psi, px - ain.x, py - ain.y, e);
  apply_segments(psi, a.prop, slot, d.nseg, lane);

  // t_f: normalise each block, alpha_s = <+_s(P_out)|psi_s>, final-state terms, and
  // W_s = Im(conj(alpha_s) <+_s|tau|psi_s>), the start of the backward sweep (chi'_s = alpha_s |+_s>)
  WPair w;
  double g_out_x = 0.0, g_out_y = 0.0, f = 0.0;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const double sg = s == 0 ? 1.0 : -1.0;
    Blk up_out, dn_out;
    double w_out;
    eig_pm(px - aout.x, py - aout.y, e, sg, up_out, dn_out, w_out);
    Blk p = block_of(psi, s);
    double nr, ni;
    inner(p, p, nr, ni);
    const double inv = 1.0 / sqrt(nr);
    p = Blk{p.ar * inv, p.ai * inv, p.br * inv, p.bi * inv};
    double al_r, al_i;
    inner(up_out, p, al_r, al_i);
    f += weight * fma(al_r, al_r, al_i * al_i);
    al_r *= weight;
    al_i *= weight;
    // d alpha = <+|dh|-><-|psi>/(2 w), dh = tau_x dP_x + s tau_y dP_y, dP = -dA(t_f)
    double xr, xi, yr, yi, mr, mi;
    tau_xy(up_out, dn_out, sg, xr, xi, yr, yi);
    inner(dn_out, p, mr, mi);
    const double k = -1.0 / (2.0 * w_out);
    // Re[conj(alpha) (t m)]
    const double tmx_r = fma(xr, mr, -(xi * mi)), tmx_i = fma(xr, mi, xi * mr);
    const double tmy_r = fma(yr, mr, -(yi * mi)), tmy_i = fma(yr, mi, yi * mr);
    g_out_x += 2.0 * k * fma(al_r, tmx_r, al_i * tmx_i);
    g_out_y += 2.0 * k * fma(al_r, tmy_r, al_i * tmy_i);
    // <+|tau_x|psi>, <+|tau_y|psi> (tau_y itself: s = 1), <+|tau_z|psi> = conj(u1) p1 - conj(u2) p2
    double vxr, vxi, vyr, vyi;
    tau_xy(up_out, p, 1.0, vxr, vxi, vyr, vyi);
    const double vzr = fma(up_out.ar, p.ar, fma(up_out.ai, p.ai, -fma(up_out.br, p.br, up_out.bi * p.bi)));
    const double vzi = fma(up_out.ar, p.ai, fma(-up_out.ai, p.ar, -fma(up_out.br, p.bi, -(up_out.bi * p.br))));
    const double wx = fma(al_r, vxi, -(al_i * vxr)), wy = fma(al_r, vyi, -(al_i * vyr)),
                 wz = fma(al_r, vzi, -(al_i * vzr));
    if (s == 0) {
      w.ax = wx; w.ay = wy; w.az = wz;
    } else {
      w.bx = wx; w.by = wy; w.bz = wz;
    }
  }

  for (int s1 = d.nseg; s1 > 0; s1 -= kApplyBatch) {
    State v[kApplyBatch];
#pragma unroll
    for (int k = 0; k < kApplyBatch; ++k) v[k] = load_state(a.prop, slot + max(s1 - 1 - k, 0), lane);
#pragma unroll
    for (int k = 0; k < kApplyBatch; ++k)
      if (s1 - 1 - k >= 0) {
        double* o = a.prop + (slot + s1 - 1 - k) * kSlotDoubles + lane;
        o[0] = w.ax; o[kItem] = w.ay; o[2 * kItem] = w.az;
        o[3 * kItem] = w.bx; o[4 * kItem] = w.by; o[5 * kItem] = w.bz;
        rotate_back(w.ax, w.ay, w.az, v[k].ar, v[k].ai, v[k].br, v[k].bi);
        rotate_back(w.bx, w.by, w.bz, v[k].cr, v[k].ci, v[k].dr, v[k].di);
      }
  }

  // t_i: d|-> = -|+><+|dh|->/(2 w), dP = -dA(t_i).  With chi'_0 = a |+> + b |->, the part of W_0
  // across n = (P_x, s P_y, e)/w gives conj(a) <+|tau_k|-> = (n x W_0)_k, so the term of block s is
  // (n x W_0)_x / w for x and s (n x W_0)_y / w for y.
  const double Px = px - ain.x, Py = py - ain.y;
  const double inv_w2 = 1.0 / fma(Px, Px, fma(Py, Py, e * e));
  const double g_in_x = (fma(Py, w.az - w.bz, -(e * (w.ay + w.by)))) * inv_w2;
  const double g_in_y = (fma(e, w.ax - w.bx, -(Px * (w.az - w.bz)))) * inv_w2;
  const double e4[4] = {g_in_x, g_in_y, g_out_x, g_out_y};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double sj = wave_sum(e4[j]);
    if (threadIdx.x == 0) a.epart[(int64_t(rel) * kWaves + wave) * 4 + j] = sj;
  }
  write_unit(d, a.units, m, f);
}

// Backward steps of a piece (len records of tab, last first) in fit variant MODE, kGroup steps at a time
// (a short group first), with the per-wave step sums in red[wave].
template <int MODE, class Momentum>
__device__ __forceinline__ void back_piece(WPair& w, const double2* tab, int len, const BackMode& m, double xb,
                                           double2 (*buf)[64], double2* red, int lane, const Momentum& momentum) {
  int top = len - 1;
  const int r = len % kGroup;
  if constexpr (MODE < kFineHalving) {
    const BackFit<MODE> f = load_back_fit<MODE>();
    double2 s = make_double2(w.ax + w.bx, w.ay - w.by);
    if (r != 0) {
#pragma unroll 1
      for (int j = 0; j < r; ++j) buf[j][lane] = back_step<MODE>(w, s, tab[top - j], m, f);
      group_store(buf, red, lane, top, r);
      top -= r;
    }
    for (; top >= 0; top -= kGroup) {
#pragma unroll
      for (int j = 0; j < kGroup; ++j) buf[j][lane] = back_step<MODE>(w, s, tab[top - j], m, f);
      group_store(buf, red, lane, top, kGroup);
    }
  } else {
    int h = 0;
    for (double x = xb; x > kCosSinXmax && h < kMaxHalvings; x *= 0.25) ++h;
    const double inv4h = ldexp(1.0, -2 * h);
    double px, py, dt;  // q from p - A, as the evolution's angle-halving path
    momentum(px, py, dt);
    for (int n = r != 0 ? r : kGroup; top >= 0; top -= n, n = kGroup) {
#pragma unroll 1
      for (int j = 0; j < n; ++j) {
        const double2 A = tab[top - j];
        const double2 g = back_w_exact(w, (px - A.x) * dt, (py - A.y) * dt, m.qz, h, inv4h);
        buf[j][lane] = make_double2(g.x + g.x, g.y + g.y);
      }
      group_store(buf, red, lane, top, n);
    }
  }
}

// Lowest tangent fit that covers the bound xb, or kFineHalving (compared as in cot_variant).
__device__ __forceinline__ int tan_variant(double xb) {
  const uint32_t hi = __builtin_amdgcn_readfirstlane(__double2hiint(xb));
  int mode = kFineHalving;
#pragma unroll
  for (int k = kNumFine - 1; k >= 0; --k)
    if (hi < high_word(kFitXmax[k])) mode = k;
  return mode;
}

// Backward steps of one (item, segment) slot, one mode per lane; a piece of the segment per 256-step
// chunk, last first, each in its own variant.  Bound by FP64 issue at the clock the power limit
// leaves.  10 pulses of 64x64x16 modes (32768 distinct) at nt = 4096: 3.27 ms here (4.1e11 mode-steps/s,
// about 66 FP64 instructions each with the sums over modes) and 1.61 ms for the segments (8.3e11),
// against 5.6 ms for one kernel that walked both sweeps item by item; 2 pulses of 512 distinct modes
// at nt = 1000: 16 and 11 us against 274 us, which was 4 workgroups doing 2000 steps in a row.
__global__ void __launch_bounds__(kItem) __attribute__((amdgpu_waves_per_eu(3))) k_grad_back(GradArgs a) {
  __shared__ double2 tab[kChunk];
  __shared__ double2 red[kWaves][kChunk];
  __shared__ double2 bufs[kWaves][kGroup][64];
  const int64_t slot = a.slot0 + blockIdx.x;
  const int pi = find_pulse_slot(a.desc, a.n_pulses, slot);
  const PulseDev& d = a.desc[pi];
  const int rel = int(slot - d.slot_off), li = rel / d.nseg, seg = rel - li * d.nseg;
  const double dt = d.dt;
  const double2* A = reinterpret_cast<const double2*>(a.A) + d.tab_off;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double px, py;
  const double e = lane_mode(d, int64_t(li) * kItem + threadIdx.x, px, py);
  BackMode m;
  const double ie = 1.0 / e;
  m.nie = -ie;
  m.px = px * ie;
  m.py = py * ie;
  m.qz = e * dt;
  m.z = m.qz * m.qz;
  m.z2 = m.z + m.z;
  const double* wp = a.prop + int64_t(blockIdx.x) * kSlotDoubles + threadIdx.x;
  WPair w{wp[0], wp[kItem], wp[2 * kItem], wp[3 * kItem], wp[4 * kItem], wp[5 * kItem]};
  const BlockBox bb = uniform_box(d, li * kItem);
  const double* rg = a.ranges + 4 * int64_t(d.chk_off);
  double2* part = reinterpret_cast<double2*>(a.part + (d.part_off - a.part0) + int64_t(li) * d.nt * 2);
  const auto momentum = [&](double& x, double& y, double& step) {
    (void)lane_mode(d, int64_t(li) * kItem + threadIdx.x, x, y);
    step = d.dt;
  };
  const int n0 = seg * d.seg_len;
  for (int n1 = min(n0 + d.seg_len, d.nt); n1 > n0;) {
    const int c = (n1 - 1) / kChunk, beg = max(n0, c * kChunk), len = n1 - beg;
    __syncthreads();
    if (int(threadIdx.x) < len) tab[threadIdx.x] = A[beg + threadIdx.x];
    __syncthreads();
    const double xb = x_bound(bb, rg[4 * c], rg[4 * c + 1], rg[4 * c + 2], rg[4 * c + 3], dt);
    switch (tan_variant(xb)) {
      case 0: back_piece<0>(w, tab, len, m, xb, bufs[wave], red[wave], lane, momentum); break;
      case 1: back_piece<1>(w, tab, len, m, xb, bufs[wave], red[wave], lane, momentum); break;
      case 2: back_piece<2>(w, tab, len, m, xb, bufs[wave], red[wave], lane, momentum); break;
      case 3: back_piece<3>(w, tab, len, m, xb, bufs[wave], red[wave], lane, momentum); break;
      case 4: back_piece<4>(w, tab, len, m, xb, bufs[wave], red[wave], lane, momentum); break;
      case 5: back_piece<5>(w, tab, len, m, xb, bufs[wave], red[wave], lane, momentum); break;
      case 6: back_piece<6>(w, tab, len, m, xb, bufs[wave], red[wave], lane, momentum); break;
      case 7: back_piece<7>(w, tab, len, m, xb, bufs[wave], red[wave], lane, momentum); break;
      default: back_piece<kFineHalving>(w, tab, len, m, xb, bufs[wave], red[wave], lane, momentum); break;
    }
    __syncthreads();
    if (int(threadIdx.x) < len) {
      double2 v = red[0][threadIdx.x];
#pragma unroll
      for (int k = 1; k < kWaves; ++k) {
        v.x += red[k][threadIdx.x].x;
        v.y += red[k][threadIdx.x].y;
      }
      part[beg + threadIdx.x] = v;
    }
    n1 = beg;
  }
}

// dJ/dA[n] = -dt dV sum over the pulse's items (in order) of the partials (the edge partials carry
// their factors); one thread per (n, component).  Of a pulse that goes on in the next group the sums so far are
// kept where the results will be, so they are added in the same order whatever the groups.
__global__ void __launch_bounds__(256) k_grad_reduce(GradArgs a, double* __restrict__ gA, double* __restrict__ gedge) {
  const PulseDev& d = a.desc[blockIdx.y];
  const int first = max(a.item0 - d.item_off, 0), last = min(a.item0 + a.items - d.item_off, d.nitems);
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t per = 2 * int64_t(d.nt);
  if (e < per) {
    const double* p = a.part + (d.part_off - a.part0) + e;
    double* out = gA + 2 * d.tab_off + e;
    double v = first > 0 ? *out : 0.0;
#pragma unroll 8
    for (int i = first; i < last; ++i) v += p[int64_t(i) * per];
    *out = last < d.nitems ? v : v * -d.dt * d.dv;  // dq_x/dA_x = -dt; the partials hold 2 Re[...]
  }
  if (gedge && blockIdx.x == 0 && threadIdx.x < 4) {
    const double* p = a.epart + int64_t(d.item_off - a.item0) * kWaves * 4 + threadIdx.x;
    double* out = gedge + 4 * blockIdx.y + threadIdx.x;
    double v = first > 0 ? *out : 0.0;
    for (int i = first * kWaves; i < last * kWaves; ++i) v += p[int64_t(i) * 4];
    *out = last < d.nitems ? v : v * d.dv;
  }
}

}  // namespace

po_status launch_yield_grad(const PulseDev* d_desc, const GradRange& r, const double* d_A, const double* d_A_edge,
                            const double* d_ranges, double* d_prop, double* d_part, double* d_epart, double* d_units,
                            double* d_gA, double* d_gedge, hipStream_t s) {
  const int n = r.i1 - r.i0;
  const PulseDev* desc = d_desc + r.i0;
  GradArgs a{desc, n, r.slot0, r.part0, r.item0, r.items, d_A, d_A_edge + 4 * int64_t(r.i0), d_ranges, d_prop, d_part,
             d_epart, d_units};
  PO_TRY(launch_segments(desc, n, r.slot0, r.slots, d_A, d_ranges, d_prop, s));
  hipLaunchKernelGGL(k_grad_join, dim3(unsigned(r.items) * kWaves), dim3(64), 0, s, a);
  PO_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_grad_back, dim3(unsigned(r.slots)), dim3(kItem), 0, s, a);
  PO_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_grad_reduce, dim3(unsigned((2 * int64_t(r.max_nt) + 255) / 256), n), dim3(256), 0, s, a, d_gA,
                     d_gedge ? d_gedge + 4 * int64_t(r.i0) : nullptr);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

}  // namespace po
