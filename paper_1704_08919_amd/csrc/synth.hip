// Pulse synthesis on gfx950: B-spline spectra -> field statistics -> scale -> A/E tables.
//
// Sec. III of arXiv:1704.08919: the spectral density and phase of each component are B-spline
// expansions; the field is a Hann-windowed cosine sum over the lines Omega_j = (N_min + j) dw,
// dw = 2 pi / T; A(t) is its antiderivative with A(t_f) = 0.  The global renormalisation of
// Sec. IV B scales E and A by one factor per pulse (peak |E| or energy U).
//
// Time is indexed by half-steps h: t = -T/2 + h dt / 2 (h even: step nodes, h odd: midpoints).
// Every line frequency is an integer multiple k of dw, so the phase Omega_k t equals
// pi k (h - nt) / nt exactly; it is reduced modulo 2 in integers and evaluated with sincospi,
// which keeps all trig arguments in [0, 2) whatever T is.
//
// The window cos^2(pi t/T) = 1/2 + cos(dw t)/2 shifts lines by one, so the windowed field is itself a sum
// over harmonics of dw with coefficients C_k = c_k/2 + (c_{k-1} + c_{k+1})/4 (S_k alike), and
//     A(t) = A_0 - C_0 (t - t_f) - sum_k [P_k sin(k dw t) - Q_k cos(k dw t)],  (P, Q)_k = (C, S)_k / (k dw),
// A_0 = -sum_k (-1)^k Q_k (A(t_f) = 0).  One pass over the harmonics therefore needs, per time and line,
// a rotation of (cos, sin) to the next harmonic (4 operations; exact phase every 16th line) and two
// FMAs per wanted component, E from the raw lines (times the window, so that it vanishes at the ends
// to relative precision) and A from P and Q: 12 operations for E and A, against about 120 when the
// three frequencies of every line are summed separately.  The records are equal for all lanes and come
// through scalar loads, four records in flight.  The tables and the statistics take a point together with
// its images in time (ImageSums), a quarter of that per point.  Bound by FP64 issue on large batches, with
// the exact phases a third of it: 256 pulses x 16384 steps x 128 lines take 0.12 ms for A and E and 0.09 ms for the peak
// (0.36 and 0.27 ms point by point; 2.06 and 0.47 ms when each line's three frequencies and the
// divisions by them were formed per step; 134 MB of tables are 0.03 ms).  A single pulse is a chain of
// rotations and exact phases: 11 and 12 us for 66 harmonics, 72 and 11 us before.
#include "common.hpp"

namespace po {
namespace {

// Fixed-order tree sum of one value per thread over a 256-thread workgroup (every thread gets it).
__device__ __forceinline__ double block_sum(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// Knot w_i of the clamped knot vector (multiplicity k at both ends, equidistant interior knots).
__device__ __forceinline__ double knot(int i, int k, int ns, double wmin, double wmax) {
  if (i < k) return wmin;
  if (i >= ns) return wmax;
  const int nb = ns - k + 2;  // breakpoints
  return wmin + (wmax - wmin) * double(i - k + 1) / double(nb - 1);
}

// All basis values b_i^{(k)}(w), i < ns, by raising the order of the indicator functions
// (Cox-de Boor recursion, 0/0 := 0); the last non-empty span is closed at omega_max.
__device__ void bspline_all(int k, int ns, double wmin, double wmax, double w, double* b /*[ns+k]*/) {
  const int nk = ns + k;
  for (int i = 0; i < nk - 1; ++i) {
    const double a = knot(i, k, ns, wmin, wmax), c = knot(i + 1, k, ns, wmin, wmax);
    b[i] = (a <= w && w < c) ? 1.0 : 0.0;
    if (w == wmax && a < c && c == wmax) b[i] = 1.0;
  }
  for (int r = 2; r <= k; ++r) {
    for (int i = 0; i < nk - r; ++i) {
      const double ti = knot(i, k, ns, wmin, wmax), tir1 = knot(i + r - 1, k, ns, wmin, wmax);
      const double ti1 = knot(i + 1, k, ns, wmin, wmax), tir = knot(i + r, k, ns, wmin, wmax);
      double v = 0.0;
      if (tir1 != ti) v += (w - ti) / (tir1 - ti) * b[i];
      if (tir != ti1) v += (tir - w) / (tir - ti1) * b[i + 1];
      b[i] = v;
    }
  }
}

// First index mu - k + 1 and values N[0..k) of the k basis functions that do not vanish at w, for order
// k <= 4 (de Boor's triangular scheme on the clamped knots; the last span is closed at omega_max).
__device__ __forceinline__ int bspline_local(int k, int ns, double wmin, double wmax, double w, double N[4]) {
  const int nb = ns - k + 2;  // breakpoints
  int mu = k - 1 + min(max(int((w - wmin) / (wmax - wmin) * double(nb - 1)), 0), nb - 2);
  while (mu > k - 1 && w < knot(mu, k, ns, wmin, wmax)) --mu;
  while (mu < ns - 1 && w >= knot(mu + 1, k, ns, wmin, wmax)) ++mu;
  N[0] = 1.0;
#pragma unroll
  for (int j = 1; j < 4; ++j) {
    if (j < k) {
      double saved = 0.0;
#pragma unroll
      for (int r = 0; r < j; ++r) {
        const double right = knot(mu + r + 1, k, ns, wmin, wmax) - w, left = w - knot(mu + 1 - (j - r), k, ns, wmin, wmax);
        const double t = N[r] / (right + left);
        N[r] = saved + right * t;
        saved = left * t;
      }
      N[j] = saved;
    }
  }
  return mu - k + 1;
}

// E and phase Phi of both components at line j, E = sum a b_i, Phi = sum pi (c + 1) b_i.
__device__ void line_spectrum(const PulseDev& d, const double* __restrict__ a, int j, double E[2], double ph[2]) {
  // basis at the line frequency clamped into the band: the end lines sample the end knots
  // whatever the rounding of (N_min + j) dw
  const double w = fmin(fmax(double(d.nmin + j) * d.dw, d.wmin), d.wmax);
  E[0] = E[1] = ph[0] = ph[1] = 0.0;
  if (d.order <= 4) {
    double N[4];
    const int i0 = bspline_local(d.order, d.ns, d.wmin, d.wmax, w, N);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (r < d.order)
        for (int l = 0; l < 2; ++l) {
          E[l] += a[(l * 2 + 0) * d.ns + i0 + r] * N[r];
          ph[l] += M_PI * (a[(l * 2 + 1) * d.ns + i0 + r] + 1.0) * N[r];
        }
  } else {
    double b[2 * kMaxNs + 2];
    bspline_all(d.order, d.ns, d.wmin, d.wmax, w, b);
    for (int i = 0; i < d.ns; ++i)
      for (int l = 0; l < 2; ++l) {
        E[l] += a[(l * 2 + 0) * d.ns + i] * b[i];
        ph[l] += M_PI * (a[(l * 2 + 1) * d.ns + i] + 1.0) * b[i];
      }
  }
}

// Harmonic records of a pulse, kSpecRec doubles each for k = nmin - 1 + i, i = 0..nlines + 1 (padded with
// zero records to a multiple of kSpecPad): the raw line
// (cEx, sEx, cEy, sEy) (cE = E cos Phi, sE = E sin Phi; 0 for the two outer records) and (Px, Qx, Py,
// Qy); then (A_0x, A_0y, C_0x, C_0y).  One workgroup per pulse, in tiles of kSpecTile harmonics.  It also
// empties the chunk ranges that k_tables fills.
constexpr int kSpecTile = 126;

__global__ void __launch_bounds__(128) k_spectra(const PulseDev* __restrict__ desc,
                                                 const double* __restrict__ coeff, double* __restrict__ spec,
                                                 double* __restrict__ ranges) {
  const PulseDev d = desc[blockIdx.x];
  if (ranges)
    for (int i = threadIdx.x; i < 4 * ((d.nt + kChunkSteps - 1) / kChunkSteps); i += 128)
      ranges[4 * int64_t(d.chk_off) + i] = (i & 1) ? -INFINITY : INFINITY;
  const double* a = coeff + d.coeff_off;
  __shared__ double4 raw[128];
  __shared__ double red[4][128];
  __shared__ double c0[2];
  const int t = threadIdx.x, nh = spec_records(d.nlines);
  double* out = spec + d.spec_off;
  // A line's sums over all basis functions hold 0 times every coefficient outside its own few, which line_spectrum
  // leaves out: a coefficient that is not finite spoils its component here, through the first line.
  bool odd = false;
  for (int i = t; i < 4 * d.ns; i += 128) odd = odd || !isfinite(a[i]);
  double a0x = 0.0, a0y = 0.0;
  if (t < 2) c0[t] = 0.0;
  for (int i0 = 0; i0 < nh; i0 += kSpecTile) {
    const int j = i0 + t - 2;  // raw line of this thread; harmonic i0 + t takes lines i0 + t - 2, ..., i0 + t
    double4 q = make_double4(0.0, 0.0, 0.0, 0.0);
    if (j >= 0 && j < d.nlines) {
      double E[2], ph[2], sp, cp;
      line_spectrum(d, a, j, E, ph);
      sincos(ph[0], &sp, &cp);
      q.x = E[0] * cp;
      q.y = E[0] * sp;
      sincos(ph[1], &sp, &cp);
      q.z = E[1] * cp;
      q.w = E[1] * sp;
    }
    if (i0 > 0) {
      __syncthreads();
    } else if (__syncthreads_or(odd) && j == 0) {
      double zero[2] = {0.0, 0.0};
      for (int i = 0; i < 4 * d.ns; ++i) zero[i / (2 * d.ns)] += 0.0 * a[i];
      q = make_double4(q.x + zero[0], q.y + zero[0], q.z + zero[1], q.w + zero[1]);
    }
    raw[t] = q;
    __syncthreads();
    const int i = i0 + t;
    if (t < kSpecTile && i < nh) {
      const int k = d.nmin - 1 + i;
      const double4 l = raw[t], m = raw[t + 1], u = raw[t + 2];
      double4 w = make_double4(0.5 * m.x + 0.25 * (l.x + u.x), 0.5 * m.y + 0.25 * (l.y + u.y),
                               0.5 * m.z + 0.25 * (l.z + u.z), 0.5 * m.w + 0.25 * (l.w + u.w));
      if (k == 1 && d.nmin == 0) {  // cos(-x) = cos x, sin(-x) = -sin x: the side line k = -1 of k = 0 (= l)
        w.x += 0.25 * l.x;
        w.y -= 0.25 * l.y;
        w.z += 0.25 * l.z;
        w.w -= 0.25 * l.w;
      }
      if (k == 0) {
        c0[0] = w.x;
        c0[1] = w.z;
      }
      const double iw = k >= 1 ? 1.0 / (double(k) * d.dw) : 0.0;  // k = 0: the (t - t_f) term; k = -1: folded into 1
      w = make_double4(w.x * iw, w.y * iw, w.z * iw, w.w * iw);
      const double sg = (k & 1) ? 1.0 : -1.0;
      a0x += sg * w.y;
      a0y += sg * w.w;
      double4* o = reinterpret_cast<double4*>(out + int64_t(kSpecRec) * i);
      o[0] = m;
      o[1] = w;
    }
  }
  red[0][t] = a0x;
  red[1][t] = a0y;
  __syncthreads();
  for (int w = 64; w > 0; w >>= 1) {
    if (t < w) {
      red[0][t] += red[0][t + w];
      red[1][t] += red[1][t + w];
    }
    __syncthreads();
  }
  if (t == 0)
    *reinterpret_cast<double4*>(out + int64_t(kSpecRec) * nh) = make_double4(red[0][0], red[1][0], c0[0], c0[1]);
}

// sin and cos of pi (u + lo), lo small.
__device__ __forceinline__ void sincos_turn(double u, double lo, double* s, double* c) {
  double s0, c0;
  sincospi(u, &s0, &c0);
  lo *= M_PI;
  *s = fma(lo, c0, s0);
  *c = fma(-lo, s0, c0);
}

// sin and cos of pi r / n with inv = 1 / n: the rounding of the quotient, the largest error of a phase for n that is no
// power of two (and carried on by every rotation), is put back to first order.
__device__ __forceinline__ void sincos_ratio(double r, double n, double inv, double* s, double* c) {
  const double u = r * inv;
  sincos_turn(u, fma(-u, n, r) * inv, s, c);
}

// Sums over the harmonics of a pulse at phase index hm = h - nt plus a fraction cf (in half-steps): the
// raw field e (without its window), its derivative ed, and sum [P sin - Q cos] in a.  The phase is
// evaluated exactly (sincospi of the reduced index) at every 16th harmonic and carried to the next 15
// by rotating with the step angle (a few ulps).
struct FieldSums {
  double ex, ey, dx, dy, ax, ay;
};

template <bool WE, bool WD, bool WA>
__device__ __forceinline__ FieldSums field_sums(const PulseDev& d, const double* __restrict__ rec, int64_t hm, double cf) {
  const int64_t two_nt = 2 * int64_t(d.nt);
  const double nt = double(d.nt), inv_nt = 1.0 / nt;
  const int nh = spec_records(d.nlines), k0 = d.nmin - 1;
  int64_t r = (int64_t(k0) * hm) % two_nt, r16 = (kSpecPad * hm) % two_nt;
  if (r < 0) r += two_nt;
  if (r16 < 0) r16 += two_nt;
  double sr, cr;  // rotation by one harmonic
  const double ur = (double(hm) + cf) * inv_nt;
  sincos_turn(ur, (fma(-ur, nt, double(hm)) + cf) * inv_nt, &sr, &cr);
  FieldSums o{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int i0 = 0; i0 < nh; i0 += kSpecPad) {
    double s, c, u = double(r) * inv_nt;
    const double lo = fma(-u, nt, double(r)) * inv_nt;
    if (cf != 0.0) {
      u = fma(double(k0 + i0), cf * inv_nt, u);
      u -= 2.0 * floor(0.5 * u);
    }
    sincos_turn(u, lo, &s, &c);
    r += r16;
    if (r >= two_nt) r -= two_nt;
#pragma unroll 4
    for (int i = i0; i < i0 + kSpecPad; ++i) {  // (four records' scalar loads in flight)
      const double* q = rec + int64_t(kSpecRec) * i;
      if (WE || WD) {
        o.ex = fma(q[0], c, fma(q[1], s, o.ex));
        o.ey = fma(q[2], c, fma(q[3], s, o.ey));
      }
      if (WD) {
        const double om = double(k0 + i) * d.dw;
        o.dx = fma(om, fma(q[1], c, -(q[0] * s)), o.dx);
        o.dy = fma(om, fma(q[3], c, -(q[2] * s)), o.dy);
      }
      if (WA) {
        o.ax = fma(q[4], s, fma(-q[5], c, o.ax));
        o.ay = fma(q[6], s, fma(-q[7], c, o.ay));
      }
      const double cn = fma(c, cr, -(s * sr));
      s = fma(s, cr, c * sr);
      c = cn;
    }
  }
  return o;
}

// A(t) from its sums over the harmonics, t - t_f = tmf.
__device__ __forceinline__ double2 potential(const PulseDev& d, const double* __restrict__ rec, double ax, double ay,
                                             double tmf) {
  const double* e = rec + int64_t(kSpecRec) * spec_records(d.nlines);
  return make_double2(e[0] - (e[2] * tmf + ax), e[1] - (e[3] * tmf + ay));
}

// A(t_i) = C_0 T and A(t_f) = 0: all harmonics return to their values at t_f.
__device__ __forceinline__ void write_edges(const PulseDev& d, const double* __restrict__ rec, double s,
                                            double2* __restrict__ edge) {
  const double* e = rec + int64_t(kSpecRec) * spec_records(d.nlines);
  edge[0] = make_double2(s * (e[2] * d.T), s * (e[3] * d.T));
  edge[1] = make_double2(0.0, 0.0);
}

// Times come in images of one another: -theta changes the sign of the sines, theta + pi that of the odd harmonics.  So
// one walk over the harmonics with the sums kept apart by cos or sin and by parity gives the field at theta,
// -theta, theta + pi and -(theta + pi), which are four grid points where nt is even (two where it is odd): a
// quarter of the rotations and products per point.
template <bool WA>
struct ImageSums {
  double c[WA ? 4 : 2][2], s[WA ? 4 : 2][2];  // [E_x, E_y, A_x, A_y][parity of the record]
};

constexpr int kImages = 4;

// First double of every record, one per thread: asks for the pulse's records as a whole, so that the walk's scalar
// loads, four records at a time, find them in its L2 (k_spectra wrote them elsewhere): 12 us instead of 16 for one
// pulse, in the kernel that reads them first.  The value is
// used (keep) after the walk, which does not wait for it.
__device__ __forceinline__ double warm_records(const PulseDev& d, const double* __restrict__ rec) {
  double w = 0.0;
  for (int i = threadIdx.x; i < min(spec_records(d.nlines), 1024); i += 256) w += rec[int64_t(kSpecRec) * i];
  return w;
}
__device__ __forceinline__ void keep(double w) { asm volatile("" ::"v"(w)); }

template <bool WE, bool WA>
__device__ __forceinline__ ImageSums<WA> image_sums(const PulseDev& d, const double* __restrict__ rec, int64_t hm) {
  const int64_t two_nt = 2 * int64_t(d.nt);
  const double nt = double(d.nt), inv_nt = 1.0 / nt;
  const int nh = spec_records(d.nlines), k0 = d.nmin - 1;
  int64_t r = (int64_t(k0) * hm) % two_nt, r16 = (kSpecPad * hm) % two_nt;
  if (r < 0) r += two_nt;
  if (r16 < 0) r16 += two_nt;
  double sr, cr;  // rotation by one harmonic
  sincos_ratio(double(hm), nt, inv_nt, &sr, &cr);
  ImageSums<WA> o{};
  for (int i0 = 0; i0 < nh; i0 += kSpecPad) {
    double s, c;
    sincos_ratio(double(r), nt, inv_nt, &s, &c);
    r += r16;
    if (r >= two_nt) r -= two_nt;
#pragma unroll 2
    for (int i = i0; i < i0 + kSpecPad; i += 2) {  // (four records' scalar loads in flight)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const double* q = rec + int64_t(kSpecRec) * (i + p);
        if (WE) {
          o.c[0][p] = fma(q[0], c, o.c[0][p]);
          o.s[0][p] = fma(q[1], s, o.s[0][p]);
          o.c[1][p] = fma(q[2], c, o.c[1][p]);
          o.s[1][p] = fma(q[3], s, o.s[1][p]);
        }
        if constexpr (WA) {
          o.s[2][p] = fma(q[4], s, o.s[2][p]);
          o.c[2][p] = fma(-q[5], c, o.c[2][p]);
          o.s[3][p] = fma(q[6], s, o.s[3][p]);
          o.c[3][p] = fma(-q[7], c, o.c[3][p]);
        }
        const double cn = fma(c, cr, -(s * sr));
        s = fma(s, cr, c * sr);
        c = cn;
      }
    }
  }
  return o;
}

// Component j at image m (bit 0: -theta, bit 1: + pi).  odd0: whether record 0's harmonic is odd.
template <bool WA>
__device__ __forceinline__ double image_value(const ImageSums<WA>& o, int j, int m, bool odd0) {
  double c = o.c[j][0], s = o.s[j][0], c1 = o.c[j][1], s1 = o.s[j][1];
  if (m & 2) {
    c1 = -c1;
    s1 = -s1;
  }
  c += c1;
  s += s1;
  const double v = (m & 1) ? c - s : c + s;
  return (m & 2) && odd0 ? -v : v;
}

// Points 0..last of a pulse (last = nt - 1 for midpoints, nt for nodes) and their images: point n has
// the images last - n, n + nt/2 and last - nt/2 - n; base points n < image_bases cover them all.
__device__ __forceinline__ int image_point(int n, int m, int nt, int last) {
  const int k = (m & 2) ? n + nt / 2 : n;
  return (m & 1) ? last - k : k;
}

// Per block: max |E| over step nodes (PEAK) or sum |E|^2 over midpoints (ENERGY) -> part[pulse][block].
__global__ void __launch_bounds__(256) k_field_stats(const PulseDev* __restrict__ desc,
                                                     const double* __restrict__ spec, int stride,
                                                     double* __restrict__ part) {
  const PulseDev d = desc[blockIdx.y];
  if (d.norm == PO_NORM_NONE || int(blockIdx.x) >= d.stat_blocks) return;
  __shared__ double red[256];
  const bool peak = d.norm == PO_NORM_PEAK;
  // nodes 0..nt (PEAK) or midpoints 0..nt-1 (ENERGY)
  const int n = blockIdx.x * 256 + threadIdx.x, last = peak ? d.nt : d.nt - 1;
  const double warm = warm_records(d, spec + d.spec_off);
  double v = 0.0;
  if (n < image_bases(d.nt, last)) {
    const int64_t hm = (peak ? 2 * int64_t(n) : 2 * int64_t(n) + 1) - d.nt;
    const ImageSums<false> o = image_sums<true, false>(d, spec + d.spec_off, hm);
    double gs, gc;  // the window's root at the images: |cos(pi t / T)| = gc or gs
    sincos_ratio(double(hm), 2.0 * double(d.nt), 0.5 / double(d.nt), &gs, &gc);
    const bool odd0 = (d.nmin - 1) & 1;
    const int images = d.nt % 2 ? 2 : kImages;
#pragma unroll
    for (int m = 0; m < kImages; ++m) {
      if (m >= images) break;
      bool again = false;  // the same point as an earlier image
#pragma unroll
      for (int q = 0; q < kImages; ++q) again = again || (q < m && image_point(n, q, d.nt, last) == image_point(n, m, d.nt, last));
      if (again) continue;
      const double g = (m & 2) ? gs : gc;
      const double ex = g * g * image_value(o, 0, m, odd0), ey = g * g * image_value(o, 1, m, odd0);
      v = peak ? fmax(v, sqrt(ex * ex + ey * ey)) : v + (ex * ex + ey * ey);
    }
  }
  keep(warm);
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) {
      const double o = red[threadIdx.x + w];
      red[threadIdx.x] = (d.norm == PO_NORM_PEAK) ? fmax(red[threadIdx.x], o) : red[threadIdx.x] + o;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) part[size_t(blockIdx.y) * stride + blockIdx.x] = red[0];
}

// Scale of a pulse from its partials, by a 256-lane workgroup: fixed-order reduction, every lane gets it.
__device__ __forceinline__ double pulse_scale(const PulseDev& d, const double* __restrict__ part, double* red) {
  const bool peak = d.norm == PO_NORM_PEAK;
  double v = 0.0;
  for (int i = threadIdx.x; i < d.stat_blocks; i += 256) v = peak ? fmax(v, part[i]) : v + part[i];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) red[threadIdx.x] = peak ? fmax(red[threadIdx.x], red[threadIdx.x + w])
                                                      : red[threadIdx.x] + red[threadIdx.x + w];
    __syncthreads();
  }
  double s = 1.0;
  if (peak) {
    s = red[0] > 0.0 ? d.norm_value / red[0] : 0.0;
  } else if (d.norm == PO_NORM_ENERGY) {
    const double U = red[0] * d.dt;
    s = U > 0.0 ? sqrt(d.norm_value / U) : 0.0;
  }
  return s;
}

// One block per pulse: the scale.
__global__ void __launch_bounds__(256) k_scale(const PulseDev* __restrict__ desc, const double* __restrict__ part,
                                               int stride, double* __restrict__ scale_ws) {
  __shared__ double red[256];
  const double s = pulse_scale(desc[blockIdx.x], part + size_t(blockIdx.x) * stride, red);
  if (threadIdx.x == 0) scale_ws[blockIdx.x] = s;
}

// The scale in the kernel that applies it: read (FUSED false) or reduced by every workgroup for itself,
// which saves the launch of k_scale where there are few partials (kFusedStats).
constexpr int kFusedStats = 512;

template <bool FUSED>
__device__ __forceinline__ double block_scale(const PulseDev& d, int pulse, const double* __restrict__ part, int stride,
                                              const double* __restrict__ scale_ws, double* red) {
  if constexpr (FUSED) return pulse_scale(d, part + size_t(pulse) * stride, red);
  else return scale_ws[pulse];
}

// Scaled A (and E) at every step midpoint and, where `ranges` is given, the table's range per chunk; workgroup = 256
// base points and their images, each of the four runs contiguous.  A run's part of a chunk is merged into
// the chunk's range (set to (inf, -inf) by k_spectra) by atomic minima and maxima; at most two chunks per
// run.
template <bool FUSED, bool WE>
__global__ void __launch_bounds__(256) k_tables(const PulseDev* __restrict__ desc, const double* __restrict__ spec,
                                                const double* __restrict__ part, int stride,
                                                const double* __restrict__ scale_ws, double* __restrict__ Aout,
                                                double* __restrict__ Eout, double* __restrict__ Aedge,
                                                double* __restrict__ scale_out, double* __restrict__ ranges) {
  static_assert(kChunkSteps == 256, "a run covers at most two chunks");
  const PulseDev d = desc[blockIdx.y];
  const int last = d.nt - 1, bases = image_bases(d.nt, last), n0 = int(blockIdx.x) * 256;
  if (n0 >= bases) return;  // whole workgroup
  __shared__ double red[256];
  __shared__ double2 run[kImages][256];
  const int n = n0 + threadIdx.x;
  const double* rec = spec + d.spec_off;
  const double s = block_scale<FUSED>(d, blockIdx.y, part, stride, scale_ws, red);
  const int images = d.nt % 2 ? 2 : kImages;
  if (n < bases) {
    const int64_t hm = 2 * int64_t(n) + 1 - d.nt;
    const ImageSums<true> o = image_sums<WE, true>(d, rec, hm);
    double gs = 0.0, gc = 0.0;  // the window's root at the images: |cos(pi t / T)| = gc or gs
    if constexpr (WE) sincos_ratio(double(hm), 2.0 * double(d.nt), 0.5 / double(d.nt), &gs, &gc);
    const bool odd0 = (d.nmin - 1) & 1;
#pragma unroll
    for (int m = 0; m < kImages; ++m) {
      if (m >= images) break;
      const int k = image_point(n, m, d.nt, last);
      const double2 A = potential(d, rec, image_value(o, 2, m, odd0), image_value(o, 3, m, odd0),
                                  double(2 * k + 1 - 2 * int64_t(d.nt)) * (0.5 * d.dt));
      const double2 sa = make_double2(s * A.x, s * A.y);
      reinterpret_cast<double2*>(Aout)[d.tab_off + k] = sa;
      run[m][threadIdx.x] = sa;
      if constexpr (WE) {
        const double g = (m & 2) ? gs : gc;
        reinterpret_cast<double2*>(Eout)[d.tab_off + k] =
            make_double2(s * (g * g * image_value(o, 0, m, odd0)), s * (g * g * image_value(o, 1, m, odd0)));
      }
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    write_edges(d, rec, s, reinterpret_cast<double2*>(Aedge) + 2 * blockIdx.y);
    if (scale_out) scale_out[blockIdx.y] = s;
  }
  if (ranges) {
    __syncthreads();
    const int m = threadIdx.x >> 6, lane = threadIdx.x & 63, len = min(256, bases - n0);  // a run per wave
    if (m >= images) return;
    const int ka = image_point(n0, m, d.nt, last), kb = image_point(n0 + len - 1, m, d.nt, last);
    for (int c = min(ka, kb) / kChunkSteps; c <= max(ka, kb) / kChunkSteps; ++c) {
      // NaN entries drop out of the range, as in k_chunk_ranges
      double v[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = lane + 64 * e;
        if (i < len && image_point(n0 + i, m, d.nt, last) / kChunkSteps == c) {
          const double2 a = run[m][i];
          v[0] = fmax(v[0], -a.x);
          v[1] = fmax(v[1], a.x);
          v[2] = fmax(v[2], -a.y);
          v[3] = fmax(v[3], a.y);
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[k] = fmax(v[k], __shfl_xor(v[k], off, 64));
      if (lane < 4) {
        double* p = ranges + 4 * int64_t(d.chk_off + c) + lane;
        const double x = lane < 2 ? (lane ? v[1] : -v[0]) : (lane == 3 ? v[3] : -v[2]);
        if (lane & 1) unsafeAtomicMax(p, x);
        else unsafeAtomicMin(p, x);
      }
    }
  }
}

struct Offsets {
  double c[kMaxSub];
};

// Scaled samples: row r of pulse i is t_i + (r / n_sub + c_{r % n_sub}) dt; with_end adds t_f.  The offset
// part of a phase (below 2 pi k / nt) is added in floating point.
template <bool FUSED, bool WE, bool WD, bool WA>
__global__ void __launch_bounds__(256) k_samples(const PulseDev* __restrict__ desc, const double* __restrict__ spec,
                                                 const double* __restrict__ part, int stride,
                                                 const double* __restrict__ scale_ws, int n_sub, Offsets off,
                                                 int with_end, double* __restrict__ Eout, double* __restrict__ Edout,
                                                 double* __restrict__ Aout, double* __restrict__ Aedge,
                                                 double* __restrict__ scale_out) {
  const PulseDev d = desc[blockIdx.y];
  __shared__ double red[256];
  const int64_t rows = int64_t(d.nt) * n_sub + (with_end ? 1 : 0);
  if (int64_t(blockIdx.x) * 256 >= rows) return;  // whole workgroup
  const int64_t k = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const double* rec = spec + d.spec_off;
  const double s = block_scale<FUSED>(d, blockIdx.y, part, stride, scale_ws, red);
  if (k < rows) {
    const bool end = k == int64_t(d.nt) * n_sub;
    const int64_t n = end ? d.nt : k / n_sub;
    const double c = end ? 0.0 : off.c[k % n_sub];
    const int64_t hm = 2 * n - d.nt;
    const double inv_nt = 1.0 / double(d.nt);
    const FieldSums o = field_sums<WE, WD, WA>(d, rec, hm, 2.0 * c);
    const int64_t row = d.tab_off + k;
    const double arg = (double(hm) + 2.0 * c) * inv_nt;  // 2 t / T
    const double g = cospi(0.5 * arg);                   // cos(pi t / T)
    if constexpr (WE) reinterpret_cast<double2*>(Eout)[row] = make_double2(s * (g * g * o.ex), s * (g * g * o.ey));
    if constexpr (WD) {
      const double g2d = -(M_PI / d.T) * sinpi(arg);  // d cos^2(pi t/T) / dt
      reinterpret_cast<double2*>(Edout)[row] = make_double2(s * (g2d * o.ex + g * g * o.dx), s * (g2d * o.ey + g * g * o.dy));
    }
    if constexpr (WA) {
      const double2 A = potential(d, rec, o.ax, o.ay, (double(n - d.nt) + c) * d.dt);
      reinterpret_cast<double2*>(Aout)[row] = make_double2(s * A.x, s * A.y);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (Aedge) write_edges(d, rec, s, reinterpret_cast<double2*>(Aedge) + 2 * blockIdx.y);
    if (scale_out) scale_out[blockIdx.y] = s;
  }
}

// ------------------------------------------------------------------------------------------
// Adjoint of the synthesis (gradient of J and of the energy U with respect to the coefficients).
// A and the windowed E are linear in the harmonic coefficients C_k, S_k:
//     dJ/dC_k = -sum_n g(t_n) sin(k dw t_n) / (k dw),  dJ/dS_k = sum_n g(t_n) (cos(k dw t_n) - (-1)^k) / (k dw),
//     dJ/dC_0 = -sum_n g(t_n) (t_n - t_f) + g(t_i) T   (A(t_i) = C_0 T; A(t_f) = 0 depends on nothing),
//     dU/dC_k = 2 dt sum_n E(t_n) cos(k dw t_n),  dU/dS_k with sin,
// g = dJ/dA, per component.  The window's adjoint takes them to the lines (half of harmonic k, a quarter of
// its neighbours), and the lines' E and Phi to the coefficients.
// ------------------------------------------------------------------------------------------

// One workgroup per (harmonic, pulse): the eight sums, out[harmonic][8] = d/d(Cx, Sx, Cy, Sy) of J, then of
// U (unscaled field).  A lane takes every 256th midpoint and rotates from one to the next, exact
// phase every 16th.
__global__ void __launch_bounds__(256) k_adjoint_harmonics(const PulseDev* __restrict__ desc,
                                                           const double* __restrict__ gA,
                                                           const double* __restrict__ gedge,
                                                           const double* __restrict__ E,
                                                           const double* __restrict__ scale, double* __restrict__ out) {
  const PulseDev d = desc[blockIdx.y];
  const int i = blockIdx.x;
  if (i >= d.nlines + 2) return;
  const int64_t k = int64_t(d.nmin) - 1 + i, two_nt = 2 * int64_t(d.nt);
  const double nt = double(d.nt), inv_nt = 1.0 / nt, sgn = (k & 1) ? -1.0 : 1.0;
  const double2* g = reinterpret_cast<const double2*>(gA) + d.tab_off;
  const double2* Et = reinterpret_cast<const double2*>(E) + d.tab_off;
  const int64_t r256 = (k * 512) % two_nt;  // phase index step between a lane's midpoints
  double sr, cr;
  sincos_ratio(double(r256), nt, inv_nt, &sr, &cr);
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, s = 0.0, c = 1.0;
  int it = 0;
  for (int64_t n = threadIdx.x; n < d.nt; n += 256, ++it) {
    if ((it & 15) == 0) {
      int64_t r = (k * (2 * n + 1 - d.nt)) % two_nt;
      if (r < 0) r += two_nt;
      sincos_ratio(double(r), nt, inv_nt, &s, &c);
    }
    const double2 gv = g[n], ev = Et[n];
    const double wc = k == 0 ? double(2 * n + 1 - two_nt) * (0.5 * d.dt) : s, ws = c - sgn;
    acc[0] = fma(gv.x, wc, acc[0]);
    acc[1] = fma(gv.x, ws, acc[1]);
    acc[2] = fma(gv.y, wc, acc[2]);
    acc[3] = fma(gv.y, ws, acc[3]);
    acc[4] = fma(ev.x, c, acc[4]);
    acc[5] = fma(ev.x, s, acc[5]);
    acc[6] = fma(ev.y, c, acc[6]);
    acc[7] = fma(ev.y, s, acc[7]);
    const double cn = fma(c, cr, -(s * sr));
    s = fma(s, cr, c * sr);
    c = cn;
  }
  __shared__ double red[4][8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc[q] += __shfl_xor(acc[q], off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q] = acc[q];
  }
  __syncthreads();
  if (threadIdx.x >= 8) return;
  const int q = threadIdx.x;
  double v = ((red[0][q] + red[1][q]) + red[2][q]) + red[3][q];
  if (q < 4) {
    const bool is_c = (q & 1) == 0;
    if (k >= 1) {
      v = (is_c ? -v : v) / (double(k) * d.dw);
    } else if (k == 0 && is_c) {
      v = -v;
      if (gedge) v = fma(gedge[4 * blockIdx.y + q / 2], d.T, v);  // dJ/dA(t_i), components 0 and 1
    } else {
      v = 0.0;
    }
  } else {
    const double sc = scale[blockIdx.y];
    v = k >= 0 && (k > 0 || (q & 1) == 0) && sc != 0.0 ? v * (2.0 * d.dt / sc) : 0.0;
  }
  out[8 * (d.harm_off + i) + q] = v;
}

// One workgroup per pulse.  Fixed-order sums of g.A over the table and of |E|^2 (the energy); per line the
// window's adjoint and the chain through cE = E cos Phi, sE = E sin Phi, values lines[line][q] = d/d(Ex,
// Phix, Ey, Phiy) of J then U, and the basis values at the line; then thread c < 4 n_s sums its line
// contributions in line order.
__global__ void __launch_bounds__(256) k_adjoint_coeff(const PulseDev* __restrict__ desc, const double* __restrict__ coeff,
                                                       const double* __restrict__ harm, double* __restrict__ lines,
                                                       const double* __restrict__ gA, const double* __restrict__ gedge,
                                                       const double* __restrict__ A, const double* __restrict__ Aedge,
                                                       const double* __restrict__ E, const double* __restrict__ scale,
                                                       int stride, double* __restrict__ grad, double* __restrict__ Uout,
                                                       double* __restrict__ gU) {
  const PulseDev d = desc[blockIdx.x];
  __shared__ double red[256];
  const double2* g = reinterpret_cast<const double2*>(gA) + d.tab_off;
  const double2* At = reinterpret_cast<const double2*>(A) + d.tab_off;
  const double2* Et = reinterpret_cast<const double2*>(E) + d.tab_off;
  const double* a = coeff + d.coeff_off;
  double* ln = lines + d.line_off * stride;
  for (int j = threadIdx.x; j < d.nlines; j += 256) {
    const double* h = harm + 8 * (d.harm_off + j);  // harmonic records of k - 1, k, k + 1, k = nmin + j
    const bool zero = d.nmin + j == 0;
    double E2[2], ph[2];
    line_spectrum(d, a, j, E2, ph);
    for (int half = 0; half < 2; ++half)
      for (int l = 0; l < 2; ++l) {
        const int q = 4 * half + 2 * l;
        // k = 0: its lower side line k = -1 is cos(dw t), -sin(dw t)
        const double Gc = 0.5 * h[8 + q] + 0.25 * (h[16 + q] + (zero ? h[16 + q] : h[q]));
        const double Gs = zero ? 0.0 : 0.5 * h[8 + q + 1] + 0.25 * (h[16 + q + 1] + h[q + 1]);
        double sp, cp;
        sincos(ph[l], &sp, &cp);
        ln[int64_t(j) * stride + q] = Gc * cp + Gs * sp;
        ln[int64_t(j) * stride + q + 1] = M_PI * E2[l] * (Gs * cp - Gc * sp);
      }
    double* b = ln + int64_t(j) * stride + 8;
    const double w = fmin(fmax(double(d.nmin + j) * d.dw, d.wmin), d.wmax);
    if (d.order <= 4) {
      double N[4];
      const int i0 = bspline_local(d.order, d.ns, d.wmin, d.wmax, w, N);
      for (int i = 0; i < d.ns; ++i) b[i] = 0.0;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r < d.order) b[i0 + r] = N[r];
    } else {
      double full[2 * kMaxNs + 2];
      bspline_all(d.order, d.ns, d.wmin, d.wmax, w, full);
      for (int i = 0; i < d.ns; ++i) b[i] = full[i];
    }
  }
  double ga = 0.0, uu = 0.0;
  for (int64_t n = threadIdx.x; n < d.nt; n += blockDim.x) {
    const double2 gv = g[n], av = At[n], ev = Et[n];
    ga += gv.x * av.x + gv.y * av.y;
    uu += ev.x * ev.x + ev.y * ev.y;
  }
  if (gedge && threadIdx.x < 2) {
    const double2 gv = reinterpret_cast<const double2*>(gedge)[2 * blockIdx.x + threadIdx.x];
    const double2 av = reinterpret_cast<const double2*>(Aedge)[2 * blockIdx.x + threadIdx.x];
    ga += gv.x * av.x + gv.y * av.y;
  }
  const double gdotA = block_sum(ga, red);
  const double U = block_sum(uu, red) * d.dt;  // energy of the scaled field (midpoint rule)
  const double s = scale[blockIdx.x];
  const bool energy = d.norm == PO_NORM_ENERGY;
  const double Uraw = s != 0.0 ? U / (s * s) : 0.0;
  if (threadIdx.x == 0 && Uout) Uout[blockIdx.x] = U;
  const int t = threadIdx.x;
  if (t >= 4 * d.ns) return;
  const int q = t / d.ns, i = t % d.ns;  // q = 2 component + kind: the column of lines
  double gj = 0.0, gu = 0.0;
#pragma unroll 8
  for (int j = 0; j < d.nlines; ++j) {
    const double* l = ln + int64_t(j) * stride;
    const double b = l[8 + i];
    gj = fma(l[q], b, gj);
    gu = fma(l[4 + q], b, gu);
  }
  // A = s A_raw: NORM_NONE has s = 1; NORM_ENERGY has s = sqrt(U0 / U_raw), so
  // dJ/dc = s dJ_raw/dc - (g.A) / (2 U_raw) dU_raw/dc and the energy stays U0.
  double outv = s * gj;
  if (energy && Uraw > 0.0) outv -= gdotA / (2.0 * Uraw) * gu;
  grad[d.coeff_off + t] = outv;
  if (gU) gU[d.coeff_off + t] = energy ? 0.0 : gu;
}

// Spectra and, where the batch has a normalisation, its partials; the scale kernel unless it is fused.
po_status launch_spectra(const Batch& b, const PulseDev* d_desc, const double* d_coeff, double* d_spec, double* d_part,
                         double* d_scale_ws, double* d_ranges, bool* fused, hipStream_t s) {
  const int P = b.n_pulses;
  hipLaunchKernelGGL(k_spectra, dim3(P), dim3(128), 0, s, d_desc, d_coeff, d_spec, d_ranges);
  PO_HIP(hipGetLastError());
  if (b.max_stat_blocks > 0) {
    hipLaunchKernelGGL(k_field_stats, dim3(b.max_stat_blocks, P), dim3(256), 0, s, d_desc, d_spec,
                       b.max_stat_blocks, d_part);
    PO_HIP(hipGetLastError());
  }
  *fused = b.max_stat_blocks <= kFusedStats;
  if (!*fused) {
    hipLaunchKernelGGL(k_scale, dim3(P), dim3(256), 0, s, d_desc, d_part, b.max_stat_blocks, d_scale_ws);
    PO_HIP(hipGetLastError());
  }
  return PO_OK;
}

template <bool FUSED, bool WE, bool WD, bool WA>
void launch_samples_t(const Batch& b, const PulseDev* d_desc, const double* d_spec, const double* d_part,
                      const double* d_scale_ws, int n_sub, const Offsets& off, int with_end, double* d_E, double* d_Ed,
                      double* d_A, double* d_A_edge, double* d_scale_out, hipStream_t s) {
  const int64_t rows = int64_t(b.max_nt) * n_sub + (with_end ? 1 : 0);
  hipLaunchKernelGGL((k_samples<FUSED, WE, WD, WA>), dim3(unsigned((rows + 255) / 256), b.n_pulses), dim3(256), 0, s,
                     d_desc, d_spec, d_part, b.max_stat_blocks, d_scale_ws, n_sub, off, with_end, d_E, d_Ed, d_A,
                     d_A_edge, d_scale_out);
}

template <bool FUSED, bool... W, class... Args>
void pick_samples(const bool* want, const Args&... args) {
  if constexpr (sizeof...(W) == 3) {
    launch_samples_t<FUSED, W...>(args...);
  } else {
    if (want[sizeof...(W)]) pick_samples<FUSED, W..., true>(want, args...);
    else pick_samples<FUSED, W..., false>(want, args...);
  }
}

}  // namespace

po_status launch_synth(const Batch& b, const PulseDev* d_desc, const double* d_coeff, double* d_spec,
                       double* d_part, double* d_scale_ws, double* d_A, double* d_E, double* d_A_edge,
                       double* d_scale_out, double* d_ranges, hipStream_t s) {
  bool fused = false;
  PO_TRY(launch_spectra(b, d_desc, d_coeff, d_spec, d_part, d_scale_ws, d_ranges, &fused, s));
  const dim3 grid((b.max_bases + 255) / 256, b.n_pulses);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, d_desc, d_spec, d_part, b.max_stat_blocks, d_scale_ws, d_A, d_E,
                       d_A_edge, d_scale_out, d_ranges);
  };
  if (fused && d_E) launch(k_tables<true, true>);
  else if (fused) launch(k_tables<true, false>);
  else if (d_E) launch(k_tables<false, true>);
  else launch(k_tables<false, false>);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

po_status launch_synth_adjoint(const Batch& b, const PulseDev* d_desc, const double* d_coeff, const double* d_gA,
                               const double* d_gedge, const double* d_A, const double* d_A_edge, const double* d_E,
                               const double* d_scale, double* d_harm, double* d_lines, double* d_grad, double* d_U,
                               double* d_gU, hipStream_t s) {
  hipLaunchKernelGGL(k_adjoint_harmonics, dim3(b.max_lines + 2, b.n_pulses), dim3(256), 0, s, d_desc, d_gA, d_gedge,
                     d_E, d_scale, d_harm);
  PO_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_adjoint_coeff, dim3(b.n_pulses), dim3(256), 0, s, d_desc, d_coeff, d_harm, d_lines, d_gA,
                     d_gedge, d_A, d_A_edge, d_E, d_scale, 8 + b.max_ns, d_grad, d_U, d_gU);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

po_status launch_samples(const Batch& b, const PulseDev* d_desc, const double* d_coeff, double* d_spec, double* d_part,
                         double* d_scale_ws, int n_sub, const double* offsets, int with_end, double* d_E,
                         double* d_Ed, double* d_A, double* d_A_edge, double* d_scale_out, hipStream_t s) {
  Offsets off{};
  for (int r = 0; r < n_sub; ++r) off.c[r] = offsets[r];
  bool fused = false;
  PO_TRY(launch_spectra(b, d_desc, d_coeff, d_spec, d_part, d_scale_ws, nullptr, &fused, s));
  const bool want[3] = {d_E != nullptr, d_Ed != nullptr, d_A != nullptr};
  if (fused) pick_samples<true>(want, b, d_desc, d_spec, d_part, d_scale_ws, n_sub, off, with_end, d_E, d_Ed, d_A, d_A_edge, d_scale_out, s);
  else pick_samples<false>(want, b, d_desc, d_spec, d_part, d_scale_ws, n_sub, off, with_end, d_E, d_Ed, d_A, d_A_edge, d_scale_out, s);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

}  // namespace po
