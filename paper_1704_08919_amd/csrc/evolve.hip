// Per-mode evolution of the momentum-space Dirac equation and projection (gfx950, FP64).
//
// Sec. II A of arXiv:1704.08919.  For a field in the x-y plane, p_z is conserved and the 4x4
// Hamiltonian alpha.(p - A) + beta m commutes with an operator K with K^2 = 1, so it splits into
// two 2x2 blocks
//     h_s(P) = P_x tau_x + s P_y tau_y + e_perp tau_z,   s = +1, -1,   e_perp = sqrt(1 + p_z^2),
// each holding one positive- and one negative-energy state of H.  The spin-summed density is
// the sum over the two blocks of |<+_s(P_out)| U_s |-_s(P_in)>|^2, which equals the trace over
// both spinors of the 4x4 form.
//
// One time step is the exact exponential of h frozen at the step midpoint (a second-order,
// unitary scheme): with q = (p - A_{n+1/2}) dt, q_z = e_perp dt, Q_s = q_x tau_x + s q_y tau_y +
// q_z tau_z and x = |q|^2 = (omega dt)^2 (so Q_s^2 = x),
//     U = C(x) 1 - i S(x) Q_s = C(x) [1 - i T(x) Q_s],
//     C(x) = cos sqrt(x),  S(x) = sin sqrt(x) / sqrt(x),  T(x) = tan sqrt(x) / sqrt(x).
// The scalar C is common to both blocks, and f is a ratio of squared norms, so any multiple of U will
// do.  The second-order kernel divides by S e_perp dt instead: with P/e_perp = (P'_x, P'_y),
//     U ~ K' - i (P'_x tau_x + s P'_y tau_y + tau_z),   K' = sqrt(x) cot(sqrt x) / (e_perp dt),
// whose tau_z coefficient is 1 and enters the multiply-add chains as an addend: 24 FMAs for the two
// blocks and no products to form first (the "cotangent form", dirac.hpp).  For any value of K' this
// is a multiple of a unitary matrix, so rounding in K' perturbs only the rotation angle.  K' is a
// polynomial (a fit of (sqrt x cot sqrt x - 1)/x whose error is below 2^-57, re-expanded per mode
// about its smallest x) of the lowest degree that covers the whole range of x of the 512-mode block
// the item belongs to in the 256-step chunk (a box of momenta against the range of the table in the
// chunk); beyond the fits' range (x > 2.48) the large-step path halves the angle and takes C and S
// from truncated Maclaurin series (remainder below 2^-56).  Either is shared by both blocks, because
// omega does not depend on s.
//
// What bounds it: FP64 issue (an FP64 instruction in 0.78-0.81 of the cycles at the 2.4 GHz peak clock; a loop of nothing
// but v_fma_f64 chains issues at 0.78-0.80 at four waves per SIMD and at 0.89-0.91 at eight), so the time
// follows the number of FP64 instructions: 28 + n per mode-step with n = 5.2 on average on the 64-pulse
// 64x64x16 nt = 16384 workload, against 31 + 6.2 for the tangent form that this replaced there: 73.6 ms per
// generation against 80.9 (A/B on one card) when every mode was stepped, 36.8 ms with the distinct modes
// of the mirror-symmetric grid alone.  Five or six waves per SIMD (96 or 80 VGPRs) measured 74.5 and
// 75.5 ms, two or one steps per loop iteration at four waves 74.0 ms and slower (every mode stepped).
//
// Work decomposition: a workgroup of THREADS lanes (64-wide waves) owns an item of
// THREADS x MPL consecutive modes of one pulse, MPL modes per lane.  The pulse's table of A
// is staged through LDS in chunks of 256 steps and every lane reads the same record, an LDS
// broadcast.  The propagators (per block the first column, 2 complex amplitudes per mode) stay in
// VGPRs.  f is summed per 64-mode unit by one
// wave in a fixed butterfly order, and units per pulse in a fixed tree, so J does not depend on
// the launch shape or on scheduling.  Time is cut into segments (a multiple of 64 steps, 8 to 32 of
// them by the pulse's own sizes); each is evolved from the identity and applied to the state.  Three
// launch forms share this code and its results: one workgroup per 256-mode item that walks
// through the segments, persistent workgroups that pull items (longest pulses first) from a device
// queue through an atomic counter, and, for batches too small to fill the chip, one workgroup per
// (item, segment) with a second kernel that applies the segments.
#include <algorithm>

#include "dirac.hpp"
#include "reduce.hpp"
#include "select.hpp"

// Every fused multiply-add below is written out: automatic contraction is off, so each mode's
// arithmetic is the same instruction sequence in every launch shape (threads, modes per lane,
// persistent or not) and f is bitwise independent of the launch.
#pragma clang fp contract(off)

namespace po {
namespace {

// Range (min A_x, max A_x, min A_y, max A_y) of the table over chunk blockIdx.x of pulse blockIdx.y
// (NODES = 2: over both Gauss-node values of every step).
template <int NODES>
__global__ void __launch_bounds__(256) k_chunk_ranges(const PulseDev* __restrict__ desc, const double* __restrict__ A,
                                                      double* __restrict__ ranges) {
  const PulseDev d = desc[blockIdx.y];
  const int c = blockIdx.x;
  const int nchunks = (d.nt + kChunk - 1) / kChunk;
  if (c >= nchunks) return;
  const int n = c * kChunk + int(threadIdx.x);
  double lx = INFINITY, hx = -INFINITY, ly = INFINITY, hy = -INFINITY;
  if (n < d.nt) {
#pragma unroll
    for (int k = 0; k < NODES; ++k) {
      const double2 a = reinterpret_cast<const double2*>(A)[NODES * (d.tab_off + n) + k];
      lx = fmin(lx, a.x); hx = fmax(hx, a.x);
      ly = fmin(ly, a.y); hy = fmax(hy, a.y);
    }
  }
  __shared__ double red[4][256];
  red[0][threadIdx.x] = -lx; red[1][threadIdx.x] = hx; red[2][threadIdx.x] = -ly; red[3][threadIdx.x] = hy;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w)
      for (int k = 0; k < 4; ++k) red[k][threadIdx.x] = fmax(red[k][threadIdx.x], red[k][threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x < 4) {
    const double v = red[threadIdx.x][0];
    ranges[4 * int64_t(d.chk_off + c) + threadIdx.x] = (threadIdx.x % 2 == 0) ? -v : v;
  }
}

constexpr int kCotUnroll = 4;  // steps per iteration of the step loops

struct EvolveArgs {
  const PulseDev* desc;
  int n_pulses;
  const double* A;
  const double* Aedge;
  const double* ranges;  // [total_chunks][4] table range per chunk (k_chunk_ranges)
  double* f;
  double* units;
};

// Fit of sqrt(x) cot(sqrt x) for a bound xb on the squared step angle: the lowest that covers it (compared by the
// upper words, so a bound within 2^-20 of a fit's end takes the next one; NaN and infinity compare above all),
// kCotHalving beyond.
__device__ __forceinline__ int cot_fit(double xb) {
  const uint32_t hi = __builtin_amdgcn_readfirstlane(__double2hiint(xb));
  int mode = kCotHalving;
#pragma unroll
  for (int k = kNumCot - 1; k >= 0; --k)
    if (hi < high_word(kCotXmax[k])) mode = k;
  return mode;
}

// Variant of the cotangent form: kCotHalving also for steps so small that even the short group would
// overflow (dt < 2^-59), which need no halvings there.
__device__ __forceinline__ int cot_variant(double xb, double dt) {
  return dt < kGroupShortMinDt ? kCotHalving : cot_fit(xb);
}

// The steps of one chunk (len table records of buf) for the MPL modes of a lane in fit variant V,
// rescaled every `group` steps.
template <int V, int MPL, bool ROW>
__device__ __forceinline__ void run_cot(State (&v)[MPL], const double2* buf, int len, double dt,
                                        const CotMode (&m)[MPL]) {
  const int group = dt >= kGroupLongMinDt ? kGroupLong : kGroupShort;
  constexpr int kDistinct = ROW ? 1 : MPL;  // ROW: the modes share e and p_x, so K's coefficients, q'_x and its square
  CotCoef<V> k[kDistinct];
#pragma unroll
  for (int j = 0; j < kDistinct; ++j) {
    double e = m[j].e;
    asm volatile("" : "+v"(e));  // keeps this set-up inside the chunk loop, out of long-lived registers
    k[j] = cot_coef<V>(cot_step_size(e, dt));
  }
  for (int n0 = 0; n0 < len; n0 += group) {
    const int end = min(n0 + group, len);
#pragma unroll kCotUnroll
    for (int n = n0; n < end; ++n) {
      const double2 rec = buf[n];
      if constexpr (ROW) {
        const double qx = fma(rec.x, m[0].nie, m[0].px), xx = qx * qx;
#pragma unroll
        for (int j = 0; j < MPL; ++j) step_cot_q<V>(v[j], qx, fma(rec.y, m[0].nie, m[j].py), xx, k[0]);
      } else {
#pragma unroll
        for (int j = 0; j < MPL; ++j) step_cot<V>(v[j], rec, m[j], k[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < MPL; ++j) rescale(v[j]);
  }
}

// Coefficients of the degree-7 series of C and S, read from memory where they are used: as literals
// the compiler sets them at kernel entry and spills them around the other variants' loops.
__constant__ double2 kHalvingCoef[8] = {
    {cos_coef(0), sinc_coef(0)}, {cos_coef(1), sinc_coef(1)}, {cos_coef(2), sinc_coef(2)}, {cos_coef(3), sinc_coef(3)},
    {cos_coef(4), sinc_coef(4)}, {cos_coef(5), sinc_coef(5)}, {cos_coef(6), sinc_coef(6)}, {cos_coef(7), sinc_coef(7)}};

// Halvings that bring the bound xb into the degree-7 series' range (at most kMaxHalvings), uniform.
__device__ __forceinline__ int halvings(double xb) {
  int h = 0;
  for (double x = xb; x > kCosSinXmax && h < kMaxHalvings; x *= 0.25) ++h;
  return __builtin_amdgcn_readfirstlane(h);
}

// C = cos sqrt x, S = sin sqrt x / sqrt x from the series (coefficients cs) at xs = x / 4^h and h doublings.
__device__ __forceinline__ void halved_cos_sinc(double xs, int h, const double2* cs, double& C, double& S) {
  C = cs[7].x;
  S = cs[7].y;
#pragma unroll
  for (int k = 6; k >= 0; --k) {
    C = fma(C, xs, cs[k].x);
    S = fma(S, xs, cs[k].y);
  }
  for (int i = 0; i < h; ++i) {
    const double c2 = fma(C, C, -(xs * S) * S);
    S = S * C;
    C = c2;
    xs *= 4.0;
  }
}

__device__ __forceinline__ const double2* halving_coef() {
  const double2* cs = kHalvingCoef;
  asm volatile("" : "+s"(cs));
  return cs;
}

// The chunk beyond the fits: C and S of degree 7 with angle halvings.  q is formed from p - A: from (p - A) / e its
// relative error would be twice as large, the same in every step, and the angle is large here.  momentum(j, px,
// py) gives the momentum of the lane's mode j, which only these chunks need.
template <int MPL, class Momentum>
__device__ __forceinline__ void run_halving(State (&v)[MPL], const double2* buf, int len, double xb, double dt,
                                            const CotMode (&m)[MPL], const Momentum& momentum) {
  const int h = halvings(xb);
  const double inv4h = ldexp(1.0, -2 * h);
  const double2* cs = halving_coef();
  double px[MPL], py[MPL];
#pragma unroll
  for (int j = 0; j < MPL; ++j) momentum(j, px[j], py[j]);
#pragma unroll 1
  for (int n = 0; n < len; ++n) {
    const double2 rec = buf[n];
#pragma unroll
    for (int j = 0; j < MPL; ++j) {
      const double qz = m[j].e * dt;
      const double qx = (px[j] - rec.x) * dt, qy = (py[j] - rec.y) * dt;
      double C, S;
      halved_cos_sinc(fma(qx, qx, fma(qy, qy, qz * qz)) * inv4h, h, cs, C, S);
      rotate(v[j], C, S, qx, qy, qz);
    }
  }
}

// The steps of one chunk, in the variant that the bound xb on its (omega dt)^2 selects.
template <int MPL, bool ROW, class Momentum>
__device__ __forceinline__ void run_chunk(State (&v)[MPL], const double2* buf, int len, double xb, double dt,
                                          const CotMode (&m)[MPL], const Momentum& momentum) {
  switch (cot_variant(xb, dt)) {
    case 0: run_cot<0, MPL, ROW>(v, buf, len, dt, m); break;
    case 1: run_cot<1, MPL, ROW>(v, buf, len, dt, m); break;
    case 2: run_cot<2, MPL, ROW>(v, buf, len, dt, m); break;
    case 3: run_cot<3, MPL, ROW>(v, buf, len, dt, m); break;
    case 4: run_cot<4, MPL, ROW>(v, buf, len, dt, m); break;
    case 5: run_cot<5, MPL, ROW>(v, buf, len, dt, m); break;
    case 6: run_cot<6, MPL, ROW>(v, buf, len, dt, m); break;
    case 7: run_cot<7, MPL, ROW>(v, buf, len, dt, m); break;
    case 8: run_cot<8, MPL, ROW>(v, buf, len, dt, m); break;
    default: run_halving<MPL>(v, buf, len, xb, dt, m, momentum); break;
  }
}

// Per-item constants of the step loops.
struct ItemTab {
  const double2* tab;  // the pulse's table
  const double* rg;    // its chunk ranges
  BlockBox bb;
  double dt;
};

__device__ __forceinline__ ItemTab item_tab(const EvolveArgs& a, const PulseDev& d, int first) {
  return ItemTab{reinterpret_cast<const double2*>(a.A) + d.tab_off, a.ranges + 4 * int64_t(d.chk_off),
                 uniform_box(d, first), d.dt};
}

// Propagators of steps [n0, n1) for the MPL modes of a lane: the first column per block of a multiple of
// a unitary matrix.  Every lane of the workgroup must call it (barriers).  The table is staged
// through LDS chunk by chunk; the series variant of each piece is chosen from the item's selection
// block (items never straddle blocks) and the chunk's table range, so it depends only on the pulse,
// the block and the chunk, never on the launch.
template <int THREADS, int MPL, bool ROW = false, class Momentum>
__device__ __forceinline__ void propagate(State (&v)[MPL], const ItemTab& t, int n0, int n1, const CotMode (&mode)[MPL],
                                          const Momentum& momentum, double2* lds) {
#pragma unroll
  for (int j = 0; j < MPL; ++j) v[j] = State{1.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0};
  for (int n = n0; n < n1;) {
    const int c = n / kChunk, len = min((c + 1) * kChunk, n1) - n;
    __syncthreads();
    for (int i = threadIdx.x; i < len; i += THREADS) lds[i] = t.tab[n + i];
    __syncthreads();
    const double* rg = t.rg + 4 * c;
    run_chunk<MPL, ROW>(v, lds, len, x_bound(t.bb, rg[0], rg[1], rg[2], rg[3], t.dt), t.dt, mode, momentum);
    n += len;
  }
}

// A lane's states between two segments, in LDS: with them in registers the step loops of a 256-lane workgroup need
// 132 of the 128 registers that four waves per SIMD leave, and the spills of 8192 items were 13 MB of
// memory traffic beside 17 MB of tables and sums (and 0.6% of the time).
template <int THREADS, int MPL>
struct ItemLds {
  double2 tab[kChunk];
  double psi[MPL][8][THREADS];
  double2 mom[MPL][THREADS];  // p_x, p_y of the lane's modes, for chunks beyond the fits
  __device__ __forceinline__ void put(int j, const State& v) {
    double(*p)[THREADS] = psi[j];
    const int t = threadIdx.x;
    p[0][t] = v.ar; p[1][t] = v.ai; p[2][t] = v.br; p[3][t] = v.bi;
    p[4][t] = v.cr; p[5][t] = v.ci; p[6][t] = v.dr; p[7][t] = v.di;
  }
  __device__ __forceinline__ State get(int j) const {
    const double(*p)[THREADS] = psi[j];
    const int t = threadIdx.x;
    return State{p[0][t], p[1][t], p[2][t], p[3][t], p[4][t], p[5][t], p[6][t], p[7][t]};
  }
};

// Evolves the item of THREADS * MPL modes of pulse pi starting at mode `first`, writes f and the
// 64-mode unit sums.  Every lane of the workgroup must call it (it contains barriers).
template <int THREADS, int MPL, bool ROW = false>
__device__ __forceinline__ void process_item(const EvolveArgs& a, int pi, int first, ItemLds<THREADS, MPL>& lds) {
  const PulseDev& d = a.desc[pi];
  const double2* edge = reinterpret_cast<const double2*>(a.Aedge) + 2 * pi;
  const double2 ain = edge[0];
  const ItemTab t = item_tab(a, d, first);

  CotMode mode[MPL];
#pragma unroll
  for (int j = 0; j < MPL; ++j) {
    double px, py;
    const double e = lane_mode(d, int64_t(first) + j * THREADS + threadIdx.x, px, py);
    State psi;
    init_state(psi, px - ain.x, py - ain.y, e);
    lds.put(j, psi);
    lds.mom[j][threadIdx.x] = make_double2(px, py);
    mode[j] = cot_mode(px, py, e);
  }
  const auto momentum = [&](int j, double& px, double& py) {
    const double2 p = lds.mom[j][threadIdx.x];
    px = p.x;
    py = p.y;
  };
  for (int n0 = 0; n0 < d.nt; n0 += d.seg_len) {
    State v[MPL];
    propagate<THREADS, MPL, ROW>(v, t, n0, min(n0 + d.seg_len, d.nt), mode, momentum, lds.tab);
#pragma unroll
    for (int j = 0; j < MPL; ++j) {
      State psi = lds.get(j);
      apply_propagator(psi, v[j]);
      rescale(psi);
      lds.put(j, psi);
    }
  }

  const double2 aout = edge[1];
#pragma unroll
  for (int j = 0; j < MPL; ++j) {
    const int64_t m = int64_t(first) + j * THREADS + threadIdx.x;
    double px, py;
    const double e = lane_mode(d, m, px, py);
    write_density(d, a.f, a.units, m, m < d.ndist ? project(lds.get(j), px - aout.x, py - aout.y, e) : 0.0);
  }
}

// One workgroup per 256-mode item; four waves per SIMD (the register budget of the variant
// switch, met without spills).
__global__ void __launch_bounds__(kItem) __attribute__((amdgpu_waves_per_eu(4))) k_evolve(EvolveArgs a) {
  __shared__ ItemLds<kItem, 1> lds;
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int pi = find_pulse_item(a.desc, a.n_pulses, item);
  process_item<kItem, 1>(a, pi, (item - a.desc[pi].item_off) * kItem, lds);
}

// Two items per workgroup, two modes per lane, where pair_rows says so: the modes m and m + 256 of a lane then lie in
// the same column p_x of the same plane p_z and share q'_x, its square and the coefficients of K: 2 of 66 operations.
// 184 VGPRs, two waves per SIMD (three, with spills around the step loops, measured the same).
__global__ void __launch_bounds__(kItem) __attribute__((amdgpu_waves_per_eu(2))) k_evolve_rows(EvolveArgs a) {
  __shared__ ItemLds<kItem, 2> lds;
  const int item = 2 * xcd_item(blockIdx.x, gridDim.x);
  const int pi = find_pulse_item(a.desc, a.n_pulses, item);
  process_item<kItem, 2, true>(a, pi, (item - a.desc[pi].item_off) * kItem, lds);
}

// Time-split form, first kernel: one workgroup per (item, segment) slot; the segment's propagators go to
// prop[slot][8 components][256 lanes].
__global__ void __launch_bounds__(kItem) __attribute__((amdgpu_waves_per_eu(4)))
k_segments(EvolveArgs a, int64_t slot0, double* __restrict__ prop) {
  __shared__ double2 lds[kChunk];
  const int64_t slot = slot0 + blockIdx.x;
  const int pi = find_pulse_slot(a.desc, a.n_pulses, slot);
  const PulseDev& d = a.desc[pi];
  const int rel = int(slot - d.slot_off), li = rel / d.nseg, seg = rel - li * d.nseg;
  double px, py;
  const double e = lane_mode(d, int64_t(li) * kItem + threadIdx.x, px, py);
  const CotMode mode[1] = {cot_mode(px, py, e)};
  const auto momentum = [&](int, double& x, double& y) { (void)lane_mode(d, int64_t(li) * kItem + threadIdx.x, x, y); };
  State v[1];
  propagate<kItem, 1>(v, item_tab(a, d, li * kItem), seg * d.seg_len, min((seg + 1) * d.seg_len, d.nt), mode, momentum, lds);
  store_state(prop, slot - slot0, v[0]);
}

// Second kernel: one lane per mode applies its segments in order.  Wavefronts of 64 here (one per
// workgroup) spread the few modes over as many CUs.
__global__ void __launch_bounds__(64) k_join_segments(EvolveArgs a, const double* __restrict__ prop) {
  const int item = blockIdx.x / (kItem / 64), lane = (blockIdx.x % (kItem / 64)) * 64 + threadIdx.x;
  const int pi = find_pulse_item(a.desc, a.n_pulses, item);
  const PulseDev& d = a.desc[pi];
  const int li = item - d.item_off;
  const int64_t m = int64_t(li) * kItem + lane, slot = d.slot_off + int64_t(li) * d.nseg;
  const double2* edge = reinterpret_cast<const double2*>(a.Aedge) + 2 * pi;
  const double2 ain = edge[0], aout = edge[1];
  double px, py;
  const double e = lane_mode(d, m, px, py);
  State psi;
  init_state(psi, px - ain.x, py - ain.y, e);
  apply_segments(psi, prop, slot, d.nseg, lane);
  write_density(d, a.f, a.units, m, m < d.ndist ? project(psi, px - aout.x, py - aout.y, e) : 0.0);
}

__global__ void k_reset_counter(int* counter) { *counter = 0; }

// Persistent workgroups: pull {pulse, first mode} items in queue order until the queue is empty.
// Every workgroup reaches the exit: the counter only grows, and each pull returns a new index.
// Register budget: four waves per SIMD with one mode per lane; two with two modes per lane, which
// keep the same number of modes in flight per SIMD without spilling.
template <int THREADS, int MPL>
__global__ void __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(MPL == 1 ? 4 : 2)))
k_evolve_persistent(EvolveArgs a, const int2* __restrict__ queue, int n_items, int* __restrict__ counter) {
  __shared__ ItemLds<THREADS, MPL> lds;
  __shared__ int s_item;
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(counter, 1);
    __syncthreads();
    const int item = s_item;
    __syncthreads();
    if (item >= n_items) break;
    const int2 q = queue[item];
    process_item<THREADS, MPL>(a, q.x, q.y, lds);
  }
}

// Unit sums from a stored f array, in the same butterfly order as the fused reduction (a mirror
// image is added to its mode first: f + f there).
__global__ void __launch_bounds__(256) k_unit_sums(const PulseDev* __restrict__ desc, int n_pulses,
                                                   const double* __restrict__ f, double* __restrict__ units) {
  const int item = blockIdx.x;
  const int pi = find_pulse_item(desc, n_pulses, item);
  const PulseDev& d = desc[pi];
  const int64_t m = int64_t(item - d.item_off) * kItem + threadIdx.x;
  double v = 0.0;
  if (m < d.ndist) {
    const int64_t mm = mirror_mode(d, m);
    v = f[d.mode_off + m];
    if (mm != m) v += f[d.mode_off + mm];
  }
  write_unit(d, units, m, v);
}

// J per pulse: each lane sums units t, t + 256, ... in order, then a fixed tree; times the cell volume.
__global__ void __launch_bounds__(256) k_yield(const PulseDev* __restrict__ desc, const double* __restrict__ units,
                                               double* __restrict__ J) {
  __shared__ double red[256];
  const PulseDev& d = desc[blockIdx.x];
  double v = 0.0;
  for (int t = threadIdx.x; t < d.nunits; t += 256) v += units[d.unit_off + t];
  const double s = block_sum256(v, red);
  if (threadIdx.x == 0) J[blockIdx.x] = s * d.dv;
}

__device__ __forceinline__ int size_class(double xb) {
  int mode = kFineHalving;
  for (int k = kNumFine - 1; k >= 0; --k)
    if (xb <= kFitXmax[k]) mode = k;
  return mode;
}

// Diagnostics: adds modes x steps of every (selection block, chunk) of every pulse to the count
// of its step-size class (the ranges of the tangent fits, kFineHalving beyond: the lower of the block's class over
// the whole table and the chunk's own, but of a block beyond the fits only the last); the blocks here run
// over all modes of the grid, mirror images included.
// One workgroup per pulse, one thread per block.
__global__ void __launch_bounds__(256) k_count_mode_steps(const PulseDev* __restrict__ desc,
                                                          const double* __restrict__ ranges,
                                                          unsigned long long* __restrict__ counts) {
  const PulseDev& d = desc[blockIdx.x];
  const int64_t nmodes = int64_t(d.n[0]) * d.n[1] * d.n[2];
  const int nblk = int((nmodes + kSelBlock - 1) / kSelBlock);
  const int nch = (d.nt + kChunk - 1) / kChunk;
  const double* rg = ranges + 4 * int64_t(d.chk_off);
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) {
    const BlockBox bb = block_box(d, b, nmodes);
    const unsigned long long mb = (unsigned long long)min(int64_t(kSelBlock), nmodes - int64_t(b) * kSelBlock);
    unsigned long long local[kSeriesVariants] = {};
    double lx = rg[0], hx = rg[1], ly = rg[2], hy = rg[3];
    for (int c = 1; c < nch; ++c) {
      lx = fmin(lx, rg[4 * c]); hx = fmax(hx, rg[4 * c + 1]);
      ly = fmin(ly, rg[4 * c + 2]); hy = fmax(hy, rg[4 * c + 3]);
    }
    const int bmode = size_class(x_bound(bb, lx, hx, ly, hy, d.dt));
    for (int c = 0; c < nch; ++c) {
      const int own = size_class(x_bound(bb, rg[4 * c], rg[4 * c + 1], rg[4 * c + 2], rg[4 * c + 3], d.dt));
      const int mode = bmode != kFineHalving ? min(own, bmode) : (own == kFineHalving ? own : kNumFine - 1);
      local[min(max(mode, 0), kSeriesVariants - 1)] += mb * (unsigned long long)min(kChunk, d.nt - c * kChunk);
    }
    for (int k = 0; k < kSeriesVariants; ++k)
      if (local[k]) atomicAdd(&counts[k], local[k]);
  }
}

template <int THREADS, int MPL>
void launch_persistent_t(EvolveArgs a, const int2* q, int n_items, int nwg, int* counter, hipStream_t s) {
  hipLaunchKernelGGL((k_evolve_persistent<THREADS, MPL>), dim3(nwg), dim3(THREADS), 0, s, a, q, n_items, counter);
}

// ---------------------------------------------------------------------------------------------
// Fourth-order Magnus step with two Gauss-Legendre nodes t_n + (1/2 -+ sqrt3/6) dt per step
// (Blanes, Casas, Oteo & Ros, Phys. Rep. 470 (2009) 151): the fourth-order Dirac scheme that
// Sec. V C of the paper leaves for future work.  For the blocks h_s(t) = v_s . tau with
// v_s = (P_x, s P_y, e_perp), [h_2, h_1] = 2i (v_2 x v_1) . tau, so the Magnus exponent of a step
// is -i w_s . tau with
//     w_s = dt (v_1 + v_2)/2 + (sqrt3/6) dt^2 (v_2 x v_1),
// and the step is a multiple of K(|w_s|^2) - i w_s . tau, K = sqrt(x) cot(sqrt x), now with one w_s (and one K)
// per block.  With a_k = (p_x - A_x(t_k)) dt, b_k likewise, e = e_perp dt, abar = (a_1 + a_2)/2 and
// g = (sqrt3/6) (a_1 - a_2, b_1 - b_2):
//     w_s = (abar - s e g_y,  s (bbar + s e g_x),  e + s (abar g_y - bbar g_x)).
// The record staged per step is (-(A_1 + A_2) dt/2, (sqrt3/6)(A_2 - A_1) dt): abar and g cost one
// add each.  The two blocks now rotate by different angles, so each is rescaled on its own.
// ---------------------------------------------------------------------------------------------

struct Magnus4 {
  double Xp, Yp, Zp, Xm, Ym, Zm;  // w_{+1} = (Xp, Yp, Zp); w_{-1} = (Xm, -Ym, Zm)
};

__device__ __forceinline__ Magnus4 magnus4(double4 rec, double pxdt, double pydt, double e) {
  const double ab = pxdt + rec.x, bb = pydt + rec.y;
  const double egx = e * rec.z, egy = e * rec.w;
  const double g = fma(ab, rec.w, -(bb * rec.z));
  return Magnus4{ab - egy, bb + egx, e + g, ab + egy, bb - egx, e - g};
}

// Coefficients of the fit of variant V in scalar registers, read from memory where they are used (the variants share
// some: as literals the compiler keeps them all from the kernel's entry on).
struct CotRows {
  double c[kNumCot][kCotMaxTerms];
};
constexpr CotRows cot_rows() {
  CotRows t{};
  for (int v = 0; v < kNumCot; ++v)
    for (int k = 0; k < kCotMaxTerms; ++k) t.c[v][k] = kCotCoef[v][k];
  return t;
}
__constant__ const CotRows kCotTable = cot_rows();

template <int V>
struct CotFit {
  double r[kCotDegree[V]];
};
template <int V>
__device__ __forceinline__ CotFit<V> load_cot_fit() {
  const double* p = kCotTable.c[V];
  asm volatile("" : "+s"(p));
  CotFit<V> f;
#pragma unroll
  for (int k = 0; k < kCotDegree[V]; ++k) f.r[k] = p[k];
  return f;
}

// K(x) = sqrt(x) cot(sqrt x): kCotDegree[V] fused multiply-adds.
template <int V>
__device__ __forceinline__ double cot_value(double x, const CotFit<V>& f) {
  constexpr int n = kCotDegree[V];
  double R = f.r[n - 1];
#pragma unroll
  for (int k = n - 2; k >= 0; --k) R = fma(R, x, f.r[k]);
  return fma(R, x, 1.0);
}

// Rescales each block by its own exact power of two so that its largest component lies in [1/2, 1).
__device__ __forceinline__ void rescale_blocks(State& v) {
  const int e1 = -__builtin_amdgcn_frexp_exp(fmax(fmax(fabs(v.ar), fabs(v.ai)), fmax(fabs(v.br), fabs(v.bi))));
  const int e2 = -__builtin_amdgcn_frexp_exp(fmax(fmax(fabs(v.cr), fabs(v.ci)), fmax(fabs(v.dr), fabs(v.di))));
  v.ar = ldexp(v.ar, e1); v.ai = ldexp(v.ai, e1); v.br = ldexp(v.br, e1); v.bi = ldexp(v.bi, e1);
  v.cr = ldexp(v.cr, e2); v.ci = ldexp(v.ci, e2); v.dr = ldexp(v.dr, e2); v.di = ldexp(v.di, e2);
}

struct SchemeArgs {
  const PulseDev* desc;
  int n_pulses;
  const double* tab;     // [sum nt][kRec][2] A at the scheme's points of every step
  const double* Aedge;
  const double* ranges;  // [total_chunks][4] range of the table per chunk (k_chunk_ranges<kRec>)
  double* f;
  double* units;
};

// The fourth-order scheme for one lane's mode.  Step s: exp(-i w_s . tau), a multiple of K(|w_s|^2) - i w_s . tau
// with K = sqrt(x) cot(sqrt x): 50 + 2n instructions for the two blocks (56 + 2n in the tangent form, whose
// fits need a larger n and end at x = 0.26; 110 and more beyond).  The norm grows by at most 1.58 per step
// for x <= 2.5, 2^168 over a chunk.  Bound by FP64 issue: 40000 modes x 10000 steps of 0.2 in 1.45 ms (3.2 ms in the
// tangent form with one workgroup per item, which took 157 of 256 CUs).
struct Magnus4Scheme {
  static constexpr int kRec = 2;    // table points per step
  static constexpr int kWaves = 4;  // per SIMD; 3 would take no spills but 4% longer
  const double2* tab;
  double dt, pxdt, pydt, e;
  BlockBox bb;
  __device__ __forceinline__ Magnus4Scheme(const SchemeArgs& a, const PulseDev& d, int first, int lane)
      : tab(reinterpret_cast<const double2*>(a.tab) + 2 * d.tab_off), dt(d.dt), bb(uniform_box(d, first)) {
    double px, py;
    e = lane_mode(d, int64_t(first) + lane, px, py) * dt;
    pxdt = px * dt;
    pydt = py * dt;
  }
  __device__ __forceinline__ void enter(State&) const {}
  __device__ __forceinline__ void leave(State&) const {}
  // the staged record of step n: (-(A_1 + A_2) dt/2, (sqrt3/6)(A_2 - A_1) dt)
  __device__ __forceinline__ void stage(double2* lds, int n) const {
    const double hdt = -0.5 * dt, kdt = kSqrt3Over6 * dt;
    const double2 a1 = tab[2 * int64_t(n)], a2 = tab[2 * int64_t(n) + 1];
    lds[0] = make_double2(hdt * (a1.x + a2.x), hdt * (a1.y + a2.y));
    lds[1] = make_double2(kdt * (a2.x - a1.x), kdt * (a2.y - a1.y));
  }
  // bound on |w_s|^2 over a chunk's table range
  __device__ __forceinline__ double bound(const double* rg) const {
    const double th = sqrt(x_bound(bb, rg[0], rg[1], rg[2], rg[3], dt));
    return (th + kSqrt3Over6 * th * th) * (th + kSqrt3Over6 * th * th) * (1.0 + 1e-6);
  }
  __device__ __forceinline__ Magnus4 angles(const double2* rec, double& xp, double& xm) const {
    const Magnus4 w = magnus4(make_double4(rec[0].x, rec[0].y, rec[1].x, rec[1].y), pxdt, pydt, e);
    xp = fma(w.Xp, w.Xp, fma(w.Yp, w.Yp, w.Zp * w.Zp));
    xm = fma(w.Xm, w.Xm, fma(w.Ym, w.Ym, w.Zm * w.Zm));
    return w;
  }
  template <int V>
  __device__ __forceinline__ void run_fit(State& v, const double2* buf, int len) const {
    const CotFit<V> f = load_cot_fit<V>();
#pragma unroll 2
    for (int k = 0; k < len; ++k) {
      double xp, xm;
      const Magnus4 w = angles(buf + 2 * k, xp, xm);
      const double Kp = cot_value<V>(xp, f), Km = cot_value<V>(xm, f);
      rotate_block(v.ar, v.ai, v.br, v.bi, Kp, w.Xp, w.Yp, w.Zp);
      rotate_block(v.cr, v.ci, v.dr, v.di, Km, w.Xm, -w.Ym, w.Zm);
    }
    rescale_blocks(v);
  }
  __device__ __forceinline__ void run(State& v, const double2* buf, int len, double xb) const {
    switch (cot_fit(xb)) {
      case 0: run_fit<0>(v, buf, len); break;
      case 1: run_fit<1>(v, buf, len); break;
      case 2: run_fit<2>(v, buf, len); break;
      case 3: run_fit<3>(v, buf, len); break;
      case 4: run_fit<4>(v, buf, len); break;
      case 5: run_fit<5>(v, buf, len); break;
      case 6: run_fit<6>(v, buf, len); break;
      case 7: run_fit<7>(v, buf, len); break;
      case 8: run_fit<8>(v, buf, len); break;
      default: {
        const int h = halvings(xb);
        const double inv4h = ldexp(1.0, -2 * h);
        const double2* cs = halving_coef();
#pragma unroll 1
        for (int k = 0; k < len; ++k) {
          double xp, xm, Cp, Sp, Cm, Sm;
          const Magnus4 w = angles(buf + 2 * k, xp, xm);
          halved_cos_sinc(xp * inv4h, h, cs, Cp, Sp);
          halved_cos_sinc(xm * inv4h, h, cs, Cm, Sm);
          rotate_block(v.ar, v.ai, v.br, v.bi, Cp, Sp * w.Xp, Sp * w.Yp, Sp * w.Zp);
          rotate_block(v.cr, v.ci, v.dr, v.di, Cm, Sm * w.Xm, -(Sm * w.Ym), Sm * w.Zm);
        }
      }
    }
  }
};

// ---------------------------------------------------------------------------------------------
// Split-operator steps: the frozen Hamiltonian splits into the part the field does not touch,
// alpha_z p_z + beta m (in each 2x2 block e_perp tau_z), and the field-driven transverse part
// P_x tau_x + s P_y tau_y; Strang's symmetric step with the field at the step midpoint is second
// order (the split-operator scheme Sec. II A names), and the triple-jump composition of three such
// steps of sizes w1 dt, w0 dt, w1 dt (w1 = 1/(2 - 2^(1/3)), w0 = 1 - 2 w1; Yoshida, Phys. Lett. A
// 150 (1990) 262) is fourth order (the splitting Sec. V C leaves for future work).
//
// Per block the constant factor is R(theta) = exp(-i theta tau_z), theta a multiple of e_perp dt,
// and the transverse one K = exp(-i Q_s) with Q_s = q_x tau_x + s q_y tau_y, q = (p - A) w dt.
// Adjacent half steps of R merge, so the whole evolution is
//     R(-theta_0) [prod over steps, substeps i: R(theta_i) K_i] R(theta_0),
// theta_0 = e dt/2 (Strang) or w1 e dt/2, theta_i = e dt (Strang) or ((w1 + w0)/2, (w1 + w0)/2,
// w1) e dt.  In tangent form R(theta) = cos(theta) (1 - i a tau_z), a = tan(theta), and
// K = C (1 - i T Q_s) with T = tan|q| / |q| (polynomial fits, x = |q|^2); the two factors are applied one
// after the other: 30 + n instructions per substep.  (Multiplied out, 34 + n.)  Beyond the tangent
// fits, up to x = 1.6, K is a multiple of |q| cot|q| - i Q_s: 36 + n.  Both are scalar multiples
// of a unitary matrix, of the same norm for both blocks.  Beyond that the exact C, S (angle halving) and
// c = cos(theta), s = sin(theta) give
//     R K = c C - i (S (c q_x - s_b s q_y), S (s_b c q_y + s q_x), s C) . tau,   s_b = +-1.
// ---------------------------------------------------------------------------------------------
constexpr double kTripleW1 = 1.3512071919596576;   // 1 / (2 - 2^(1/3))
constexpr double kTripleW0 = -1.7024143839193153;  // 1 - 2 w1

// psi <- R(phi) psi for both blocks: a <- a e^{-i phi}, b <- b e^{i phi}.
__device__ __forceinline__ void phase_z(State& v, double cp, double sp) {
  double r, i;
  r = fma(v.ai, sp, v.ar * cp); i = fma(-v.ar, sp, v.ai * cp); v.ar = r; v.ai = i;
  r = fma(-v.bi, sp, v.br * cp); i = fma(v.br, sp, v.bi * cp); v.br = r; v.bi = i;
  r = fma(v.ci, sp, v.cr * cp); i = fma(-v.cr, sp, v.ci * cp); v.cr = r; v.ci = i;
  r = fma(-v.di, sp, v.dr * cp); i = fma(v.dr, sp, v.di * cp); v.dr = r; v.di = i;
}

// psi <- (1 - i Q_s) psi for both blocks, Q_s = x tau_x + s y tau_y.
__device__ __forceinline__ void rotate_xy(State& v, double x, double y) {
  const double ar = fma(x, v.bi, fma(-y, v.br, v.ar)), ai = fma(-x, v.br, fma(-y, v.bi, v.ai));
  const double br = fma(x, v.ai, fma(y, v.ar, v.br)), bi = fma(-x, v.ar, fma(y, v.ai, v.bi));
  const double cr = fma(x, v.di, fma(y, v.dr, v.cr)), ci = fma(-x, v.dr, fma(y, v.di, v.ci));
  const double dr = fma(x, v.ci, fma(-y, v.cr, v.dr)), di = fma(-x, v.cr, fma(-y, v.ci, v.di));
  v = State{ar, ai, br, bi, cr, ci, dr, di};
}

// psi <- (k - i Q_s) psi for both blocks.
__device__ __forceinline__ void rotate_xy(State& v, double k, double x, double y) {
  const double ar = fma(k, v.ar, fma(x, v.bi, -(y * v.br))), ai = fma(k, v.ai, fma(-x, v.br, -(y * v.bi)));
  const double br = fma(k, v.br, fma(x, v.ai, y * v.ar)), bi = fma(k, v.bi, fma(-x, v.ar, y * v.ai));
  const double cr = fma(k, v.cr, fma(x, v.di, y * v.dr)), ci = fma(k, v.ci, fma(-x, v.dr, y * v.di));
  const double dr = fma(k, v.dr, fma(x, v.ci, -(y * v.cr))), di = fma(k, v.di, fma(-x, v.cr, -(y * v.ci)));
  v = State{ar, ai, br, bi, cr, ci, dr, di};
}

// psi <- (1 - i a tau_z) psi for both blocks.
__device__ __forceinline__ void tilt_z(State& v, double a) {
  v = State{fma(a, v.ai, v.ar), fma(-a, v.ar, v.ai), fma(-a, v.bi, v.br), fma(a, v.br, v.bi),
            fma(a, v.ci, v.cr), fma(-a, v.cr, v.ci), fma(-a, v.di, v.dr), fma(a, v.dr, v.di)};
}

// The split-operator schemes for one lane's mode.  The series of a chunk bounds |q|^2 <= |p - A|^2
// (w_max dt)^2 through the second-order bound at step w_max dt, which also counts
// (1 + p_z^2)(w_max dt)^2 >= theta_i^2: the tangents a stay below 3.3 for the fits in use (x <= 1.61), and
// the norm below 2^420 over the 64 steps between two rescalings.  Bound by FP64 issue: 40000 modes x 4000 steps of
// 0.2 in 0.46 (Strang) and 1.40 ms (fourth order); 1.06 and 2.69 ms multiplied out, with angle halving
// beyond x = 0.26 and one workgroup per item.
template <int NSUB>
struct SplitScheme {
  static constexpr int kRec = NSUB;
  static constexpr int kWaves = 3;  // 4 would take spills and 2% longer
  static constexpr int kAngles = NSUB == 1 ? 1 : 2;
  static constexpr int kFirstCot = 5, kLastCot = 7;  // cotangent fits in use: x <= 0.35, 0.94, 1.61
  const double2* tab;
  double dt;
  double pxw[kAngles], pyw[kAngles];                  // p w dt for the distinct weights
  double a[kAngles], c[kAngles], s[kAngles];          // tan, cos, sin of theta_i
  double c0, s0;                                      // of theta_0
  BlockBox bb;
  __device__ __forceinline__ static constexpr int weight(int i) { return i == 1 ? 1 : 0; }
  __device__ __forceinline__ static constexpr int angle(int i) { return i == 2 ? 1 : 0; }
  __device__ __forceinline__ static constexpr double step(int i) {
    return NSUB == 1 ? 1.0 : (i == 1 ? kTripleW0 : kTripleW1);
  }
  __device__ __forceinline__ SplitScheme(const SchemeArgs& arg, const PulseDev& d, int first, int lane)
      : tab(reinterpret_cast<const double2*>(arg.tab) + NSUB * d.tab_off), dt(d.dt), bb(uniform_box(d, first)) {
    double px, py;
    const double ep = lane_mode(d, int64_t(first) + lane, px, py);
    double th0;
    if constexpr (NSUB == 1) {
      pxw[0] = px * dt;
      pyw[0] = py * dt;
      sincos(ep * dt, &s[0], &c[0]);
      th0 = 0.5 * ep * dt;
    } else {
      pxw[0] = px * (kTripleW1 * dt); pyw[0] = py * (kTripleW1 * dt);
      pxw[1] = px * (kTripleW0 * dt); pyw[1] = py * (kTripleW0 * dt);
      sincos(0.5 * (kTripleW1 + kTripleW0) * ep * dt, &s[0], &c[0]);
      sincos(kTripleW1 * ep * dt, &s[1], &c[1]);
      th0 = 0.5 * kTripleW1 * ep * dt;
    }
#pragma unroll
    for (int j = 0; j < kAngles; ++j) a[j] = s[j] / c[j];
    sincos(th0, &s0, &c0);
  }
  __device__ __forceinline__ void enter(State& v) const { phase_z(v, c0, s0); }
  __device__ __forceinline__ void leave(State& v) const { phase_z(v, c0, -s0); }
  __device__ __forceinline__ void stage(double2* lds, int n) const {  // -A w_i dt
#pragma unroll
    for (int i = 0; i < NSUB; ++i) {
      const double2 t = tab[NSUB * int64_t(n) + i];
      const double w = -step(i) * dt;
      lds[i] = make_double2(t.x * w, t.y * w);
    }
  }
  __device__ __forceinline__ double bound(const double* rg) const {
    return x_bound(bb, rg[0], rg[1], rg[2], rg[3], NSUB == 1 ? dt : -kTripleW0 * dt);
  }
  // V < kNumFine: tangent fit V; else the cotangent fit V - kNumFine
  template <int V>
  __device__ __forceinline__ void run_fit(State& v, const double2* buf, int len) const {
    constexpr bool kTan = V < kNumFine;
    const auto f = [] {
      if constexpr (kTan) return load_fit<V>();
      else return load_cot_fit<V - kNumFine>();
    }();
    for (int n0 = 0; n0 < len; n0 += kGroupLong) {
      const int end = min(n0 + kGroupLong, len);
#pragma unroll(NSUB == 1 ? 4 : 1)
      for (int n = n0; n < end; ++n)
#pragma unroll
        for (int i = 0; i < NSUB; ++i) {
          const double2 rec = buf[n * NSUB + i];
          const double qx = pxw[weight(i)] + rec.x, qy = pyw[weight(i)] + rec.y;
          const double x = fma(qx, qx, qy * qy);
          if constexpr (kTan) {
            const double T = tan_ratio<V>(x, f);
            rotate_xy(v, T * qx, T * qy);
          } else {
            rotate_xy(v, cot_value<V - kNumFine>(x, f), qx, qy);
          }
          tilt_z(v, a[angle(i)]);
        }
      rescale(v);
    }
  }
  __device__ __forceinline__ void run(State& v, const double2* buf, int len, double xb) const {
    const uint32_t hi = __builtin_amdgcn_readfirstlane(__double2hiint(xb));
    int mode = kNumFine + kCotHalving;
#pragma unroll
    for (int k = kLastCot; k >= kFirstCot; --k)
      if (hi < high_word(kCotXmax[k])) mode = kNumFine + k;
#pragma unroll
    for (int k = kNumFine - 1; k >= 0; --k)
      if (hi < high_word(kFitXmax[k])) mode = k;
    switch (mode) {
      case 0: run_fit<0>(v, buf, len); break;
      case 1: run_fit<1>(v, buf, len); break;
      case 2: run_fit<2>(v, buf, len); break;
      case 3: run_fit<3>(v, buf, len); break;
      case 4: run_fit<4>(v, buf, len); break;
      case 5: run_fit<5>(v, buf, len); break;
      case 6: run_fit<6>(v, buf, len); break;
      case 7: run_fit<7>(v, buf, len); break;
      case kNumFine + 5: run_fit<kNumFine + 5>(v, buf, len); break;
      case kNumFine + 6: run_fit<kNumFine + 6>(v, buf, len); break;
      case kNumFine + 7: run_fit<kNumFine + 7>(v, buf, len); break;
      default: {
        const int h = halvings(xb);
        const double inv4h = ldexp(1.0, -2 * h);
        const double2* cs = halving_coef();
#pragma unroll 1
        for (int n = 0; n < len; ++n)
#pragma unroll
          for (int i = 0; i < NSUB; ++i) {
            const double2 rec = buf[n * NSUB + i];
            const double qx = pxw[weight(i)] + rec.x, qy = pyw[weight(i)] + rec.y;
            const double ci = c[angle(i)], si = s[angle(i)];
            double C, S;
            halved_cos_sinc(fma(qx, qx, qy * qy) * inv4h, h, cs, C, S);
            const double cC = ci * C, sz = si * C;
            const double cx = ci * qx, cy = ci * qy, sx = si * qx, sy = si * qy;
            rotate_block(v.ar, v.ai, v.br, v.bi, cC, S * (cx - sy), S * (cy + sx), sz);
            rotate_block(v.cr, v.ci, v.dr, v.di, cC, S * (cx + sy), S * (sx - cy), sz);
          }
      }
    }
  }
};

// ---------------------------------------------------------------------------------------------
// The same launch forms as the midpoint step's for the schemes above: segments of the pulse's own lengths, each
// evolved from the identity and applied to the state, by one workgroup per item or, where split_in_time
// says so, one per (item, segment) and a second kernel.
// ---------------------------------------------------------------------------------------------
template <class S>
__device__ __forceinline__ State propagate_scheme(const S& sch, const double* rg, int n0, int n1, double2* lds) {
  State v{1.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0};
  for (int n = n0; n < n1;) {
    const int c = n / kChunk, len = min((c + 1) * kChunk, n1) - n;
    __syncthreads();
    for (int i = threadIdx.x; i < len; i += kItem) sch.stage(lds + S::kRec * i, n + i);
    __syncthreads();
    sch.run(v, lds, len, sch.bound(rg + 4 * c));
    n += len;
  }
  rescale_blocks(v);  // the angle-halving path leaves the norm alone
  return v;
}

template <class S>
__global__ void __launch_bounds__(kItem) k_scheme(SchemeArgs a) {
  __shared__ double2 lds[S::kRec * kChunk];
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int pi = find_pulse_item(a.desc, a.n_pulses, item);
  const PulseDev& d = a.desc[pi];
  const int first = (item - d.item_off) * kItem;
  const int64_t m = int64_t(first) + threadIdx.x;
  const double2* edge = reinterpret_cast<const double2*>(a.Aedge) + 2 * pi;
  const double* rg = a.ranges + 4 * int64_t(d.chk_off);
  const double2 ain = edge[0], aout = edge[1];
  const S sch(a, d, first, threadIdx.x);
  double px, py;
  double e = lane_mode(d, m, px, py);
  State psi;
  init_state(psi, px - ain.x, py - ain.y, e);
  sch.enter(psi);
  for (int n0 = 0; n0 < d.nt; n0 += d.seg_len) {
    const State v = propagate_scheme(sch, rg, n0, min(n0 + d.seg_len, d.nt), lds);
    apply_propagator(psi, v);
    rescale(psi);
  }
  sch.leave(psi);
  e = lane_mode(d, m, px, py);
  write_density(d, a.f, a.units, m, m < d.ndist ? project(psi, px - aout.x, py - aout.y, e) : 0.0);
}

template <class S>
__global__ void __launch_bounds__(kItem) __attribute__((amdgpu_waves_per_eu(S::kWaves)))
k_scheme_segments(SchemeArgs a, double* __restrict__ prop) {
  __shared__ double2 lds[S::kRec * kChunk];
  const int64_t slot = blockIdx.x;
  const int pi = find_pulse_slot(a.desc, a.n_pulses, slot);
  const PulseDev& d = a.desc[pi];
  const int rel = int(slot - d.slot_off), li = rel / d.nseg, seg = rel - li * d.nseg;
  const S sch(a, d, li * kItem, threadIdx.x);
  store_state(prop, slot, propagate_scheme(sch, a.ranges + 4 * int64_t(d.chk_off), seg * d.seg_len,
                                           min((seg + 1) * d.seg_len, d.nt), lds));
}

template <class S>
__global__ void __launch_bounds__(64) k_scheme_join(SchemeArgs a, const double* __restrict__ prop) {
  const int item = blockIdx.x / (kItem / 64), lane = (blockIdx.x % (kItem / 64)) * 64 + threadIdx.x;
  const int pi = find_pulse_item(a.desc, a.n_pulses, item);
  const PulseDev& d = a.desc[pi];
  const int li = item - d.item_off;
  const int64_t m = int64_t(li) * kItem + lane;
  const double2* edge = reinterpret_cast<const double2*>(a.Aedge) + 2 * pi;
  const double2 ain = edge[0], aout = edge[1];
  const S sch(a, d, li * kItem, lane);
  double px, py;
  const double e = lane_mode(d, m, px, py);
  State psi;
  init_state(psi, px - ain.x, py - ain.y, e);
  sch.enter(psi);
  apply_segments(psi, prop, d.slot_off + int64_t(li) * d.nseg, d.nseg, lane);
  sch.leave(psi);
  write_density(d, a.f, a.units, m, m < d.ndist ? project(psi, px - aout.x, py - aout.y, e) : 0.0);
}

// d_prop: propagators of the batch's slots, or NULL for the form without.
template <class S>
po_status launch_scheme(const Batch& b, const PulseDev* d_desc, const double* d_tab, const double* d_A_edge,
                        double* d_ranges, double* d_prop, double* d_f, double* d_units, hipStream_t s) {
  const int max_chunks = (b.max_nt + kChunk - 1) / kChunk;
  const SchemeArgs a{d_desc, b.n_pulses, d_tab, d_A_edge, d_ranges, d_f, d_units};
  hipLaunchKernelGGL(k_chunk_ranges<S::kRec>, dim3(max_chunks, b.n_pulses), dim3(256), 0, s, d_desc, d_tab, d_ranges);
  PO_HIP(hipGetLastError());
  if (d_prop) {
    hipLaunchKernelGGL(k_scheme_segments<S>, dim3(unsigned(b.total_slots)), dim3(kItem), 0, s, a, d_prop);
    PO_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_scheme_join<S>, dim3(unsigned(b.total_items) * (kItem / 64)), dim3(64), 0, s, a, d_prop);
  } else {
    hipLaunchKernelGGL(k_scheme<S>, dim3(b.total_items), dim3(kItem), 0, s, a);
  }
  PO_HIP(hipGetLastError());
  return PO_OK;
}

}  // namespace

po_status launch_chunk_ranges(const Batch& b, const PulseDev* d_desc, const double* d_A, double* d_ranges,
                              hipStream_t s) {
  const int max_chunks = (b.max_nt + kChunk - 1) / kChunk;
  hipLaunchKernelGGL(k_chunk_ranges<1>, dim3(max_chunks, b.n_pulses), dim3(256), 0, s, d_desc, d_A, d_ranges);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

// Two items per workgroup where every pulse's grid allows it (row_pairs) and whole rounds of 256 CUs lose no more than
// the 3% that the shared operations save: 2 ceil(items / 512) of its items against ceil(items / 256).
// Measured, 64x64x16 modes at nt = 4096, us per call paired / single: 512 items 804 / 814, 640 items 1202 / 1024,
// 1024 items 1288 / 1323, 1152 items 1756 / 1565, 2048 items 2461 / 2520, 2304 items 2961 / 2811, 3072 items
// 3632 / 3737; and 8192 items at nt = 16384 35.5 / 36.6 ms.  Other grids, nt = 2048: 16x64x128 (512 items) 314 / 321,
// 128x128x32 (2048) 1159 / 1202, 256x256x8 1156 / 1203, 32x32x512 1177 / 1222.
bool pair_rows(const Batch& b) {
  const int64_t single = (int64_t(b.total_items) + 255) / 256, paired = 2 * ((int64_t(b.total_items) + 511) / 512);
  return b.row_pairs && 100 * single >= 97 * paired;
}

po_status launch_evolve_grid(const Batch& b, const PulseDev* d_desc, const double* d_A, const double* d_A_edge,
                             const double* d_ranges, double* d_f, double* d_units, hipStream_t s) {
  EvolveArgs a{d_desc, b.n_pulses, d_A, d_A_edge, d_ranges, d_f, d_units};
  if (pair_rows(b)) hipLaunchKernelGGL(k_evolve_rows, dim3(b.total_items / 2), dim3(kItem), 0, s, a);
  else hipLaunchKernelGGL(k_evolve, dim3(b.total_items), dim3(kItem), 0, s, a);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

// The batch is split in time when its items alone load the CUs thinly or unevenly.  Measured, one
// pulse at nt = 4096, us per call split / not split: 16 items 75 / 357, 128 items 190 / 344, 256 items
// 329 / 352, 320 items 402 / 581 (some CUs then hold two workgroups, the others one), 384 items
// 480 / 594, 512 items 619 / 626 and, at nt = 1024, 194 / 177.  At most 8192 slots (128 MiB of
// propagators).  Short tables pay for the second kernel: at nt = 256, 256 items 48 / 48, 448 items 65 / 59.  The line
// is the same for the schemes, whose steps cost more.  Fourth-order Magnus: nt = 4096, 256 items 541 / 618,
// 384 items 794 / 1049, 448 items 918 / 1069, 512 items 1041 / 1103; nt = 1024, 448 items 259 / 289; nt = 256, 87 / 88.
// Strang, nt = 4096: 448 items 592 / 656, 512 items 671 / 673; nt = 256: 448 items 68 / 62.  Its composition, nt = 4096:
// 448 items 1761 / 2036, 512 items 2003 / 2091; nt = 256: 448 items 140 / 148.
bool split_in_time(const Batch& b) {
  return b.total_items <= 448 && b.total_slots > b.total_items && b.total_slots <= 8192;
}

po_status launch_segments(const PulseDev* d_desc, int n_pulses, int64_t slot0, int64_t slots, const double* d_A,
                          const double* d_ranges, double* d_prop, hipStream_t s) {
  EvolveArgs a{d_desc, n_pulses, d_A, nullptr, d_ranges, nullptr, nullptr};
  hipLaunchKernelGGL(k_segments, dim3(unsigned(slots)), dim3(kItem), 0, s, a, slot0, d_prop);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

po_status launch_evolve_segments(const Batch& b, const PulseDev* d_desc, const double* d_A, const double* d_A_edge,
                                 const double* d_ranges, double* d_prop, double* d_f, double* d_units, hipStream_t s) {
  PO_TRY(launch_segments(d_desc, b.n_pulses, 0, b.total_slots, d_A, d_ranges, d_prop, s));
  EvolveArgs a{d_desc, b.n_pulses, d_A, d_A_edge, d_ranges, d_f, d_units};
  hipLaunchKernelGGL(k_join_segments, dim3(unsigned(b.total_items) * (kItem / 64)), dim3(64), 0, s, a, d_prop);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

template <int THREADS, int MPL>
int resident_persistent_t() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(&k_evolve_persistent<THREADS, MPL>),
                                                   THREADS, 0) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return n;
}

int evolve_workgroups_per_cu(const EvolveConfig& cfg) {
  // workgroups of the instantiated persistent kernel that fit on one CU at its register and LDS
  // use (the runtime's occupancy query); if the query fails, the waves-per-SIMD bound each
  // instantiation is compiled for (4 with one mode per lane, 2 with two), four SIMDs per CU
  int n = 0;
  switch (cfg.threads * 10 + cfg.mpl) {
    case 641: n = resident_persistent_t<64, 1>(); break;
    case 642: n = resident_persistent_t<64, 2>(); break;
    case 1281: n = resident_persistent_t<128, 1>(); break;
    case 1282: n = resident_persistent_t<128, 2>(); break;
    case 2561: n = resident_persistent_t<256, 1>(); break;
    case 2562: n = resident_persistent_t<256, 2>(); break;
    default: break;
  }
  if (n > 0) return n;
  const int waves_per_simd = cfg.mpl == 1 ? 4 : 2;
  return std::max(1, waves_per_simd * 4 / (cfg.threads / 64));
}

po_status launch_evolve_persistent(const EvolveConfig& cfg, int n_pulses, const PulseDev* d_desc, const double* d_A,
                                   const double* d_A_edge, const double* d_ranges, const int2* d_queue, int n_items,
                                   int n_workgroups, int* d_counter, double* d_f, double* d_units, hipStream_t s) {
  EvolveArgs a{d_desc, n_pulses, d_A, d_A_edge, d_ranges, d_f, d_units};
  hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, s, d_counter);
  PO_HIP(hipGetLastError());
  const int key = cfg.threads * 10 + cfg.mpl;
  switch (key) {
    case 641: launch_persistent_t<64, 1>(a, d_queue, n_items, n_workgroups, d_counter, s); break;
    case 642: launch_persistent_t<64, 2>(a, d_queue, n_items, n_workgroups, d_counter, s); break;
    case 1281: launch_persistent_t<128, 1>(a, d_queue, n_items, n_workgroups, d_counter, s); break;
    case 1282: launch_persistent_t<128, 2>(a, d_queue, n_items, n_workgroups, d_counter, s); break;
    case 2561: launch_persistent_t<256, 1>(a, d_queue, n_items, n_workgroups, d_counter, s); break;
    case 2562: launch_persistent_t<256, 2>(a, d_queue, n_items, n_workgroups, d_counter, s); break;
    default: return set_error(PO_ERR_INVALID, "unsupported evolution config threads=%d mpl=%d", cfg.threads, cfg.mpl);
  }
  PO_HIP(hipGetLastError());
  return PO_OK;
}

po_status launch_count_mode_steps(int n_pulses, const PulseDev* d_desc, const double* d_ranges,
                                  unsigned long long* d_counts, hipStream_t s) {
  hipLaunchKernelGGL(k_count_mode_steps, dim3(n_pulses), dim3(256), 0, s, d_desc, d_ranges, d_counts);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

po_status launch_unit_sums_from_f(const Batch& b, const PulseDev* d_desc, const double* d_f, double* d_units,
                                  hipStream_t s) {
  hipLaunchKernelGGL(k_unit_sums, dim3(b.total_items), dim3(256), 0, s, d_desc, b.n_pulses, d_f, d_units);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

po_status launch_yield_from_units(const Batch& b, const PulseDev* d_desc, const double* d_units, double* d_J,
                                  hipStream_t s) {
  hipLaunchKernelGGL(k_yield, dim3(b.n_pulses), dim3(256), 0, s, d_desc, d_units, d_J);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

po_status launch_evolve4(const Batch& b, const PulseDev* d_desc, const double* d_Ag, const double* d_A_edge,
                         double* d_ranges, double* d_prop, double* d_f, double* d_units, hipStream_t s) {
  return launch_scheme<Magnus4Scheme>(b, d_desc, d_Ag, d_A_edge, d_ranges, d_prop, d_f, d_units, s);
}

po_status launch_evolve_split(const Batch& b, int order, const PulseDev* d_desc, const double* d_At,
                              const double* d_A_edge, double* d_ranges, double* d_prop, double* d_f, double* d_units,
                              hipStream_t s) {
  return order == 2 ? launch_scheme<SplitScheme<1>>(b, d_desc, d_At, d_A_edge, d_ranges, d_prop, d_f, d_units, s)
                    : launch_scheme<SplitScheme<3>>(b, d_desc, d_At, d_A_edge, d_ranges, d_prop, d_f, d_units, s);
}

}  // namespace po
