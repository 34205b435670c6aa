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
// omega does not depend on s.  The fourth-order and split-operator kernels below keep the multiple
// 1 - i T Q_s with fits of T.
//
// What bounds it: FP64 issue, at the clock the power limit leaves (a chain of v_fma_f64 on distinct
// registers runs at 1.85-1.95 GHz on this card, 0.73 of the 2.4 GHz peak at four waves per SIMD and
// 0.77 at eight), so the time follows the number of FP64 instructions: 28 + n per mode-step with n =
// 5.2 on average on the 64-pulse 64x64x16 nt = 16384 workload, against 31 + 6.2 for the tangent form
// that this replaced there: 73.6 ms per generation against 80.9 (A/B on one card).  Five or six waves
// per SIMD (96 or 80 VGPRs) measured 74.5 and 75.5 ms, two or one steps per loop iteration at four
// waves 74.0 ms and slower.
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

// NODES = 1: the second-order step's angle.  NODES = 2: the fourth-order step's, from theta^2 the
// bound above over both Gauss nodes, |w_s| <= theta + (sqrt3/6) theta^2.
template <int NODES>
__device__ __forceinline__ int2 choose_variant(const BlockBox& bb, double lx, double hx, double ly, double hy,
                                               double dt) {
  double xb = x_bound(bb, lx, hx, ly, hy, dt);
  if constexpr (NODES == 2) {
    const double th = sqrt(xb);
    xb = (th + kSqrt3Over6 * th * th) * (th + kSqrt3Over6 * th * th) * (1.0 + 1e-6);
  }
  return variant_for_x(xb);
}

// Variant of a block for the whole table (the union of its nchunks chunk ranges rg[c][4]).
template <int NODES = 1>
__device__ __forceinline__ int2 block_variant(const BlockBox& bb, const double* rg, int nchunks, double dt) {
  double lx = rg[0], hx = rg[1], ly = rg[2], hy = rg[3];
  for (int c = 1; c < nchunks; ++c) {
    lx = fmin(lx, rg[4 * c]); hx = fmax(hx, rg[4 * c + 1]);
    ly = fmin(ly, rg[4 * c + 2]); hy = fmax(hy, rg[4 * c + 3]);
  }
  return choose_variant<NODES>(bb, lx, hx, ly, hy, dt);
}

// Variant of chunk c given the block's (bmode).  A block within the T-series range: the lower of
// the block's variant and the one for the chunk's own range (both cover the chunk's steps).  A
// block on the angle-halving path: its chunks take that path with their own number of halvings,
// or, when their own range allows any T fit, the degree-11 one (two code paths only, so the
// loop keeps to its register budget).
template <int NODES = 1>
__device__ __forceinline__ int2 chunk_variant(const BlockBox& bb, const double* rg, int c, int bmode, double dt) {
  const int2 own = choose_variant<NODES>(bb, rg[4 * c], rg[4 * c + 1], rg[4 * c + 2], rg[4 * c + 3], dt);
  if (bmode == kFineHalving) return own.x == kFineHalving ? own : make_int2(kNumFine - 1, 0);
  return make_int2(min(own.x, bmode), 0);
}

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

// Variant of the cotangent form for a bound xb on x = (omega dt)^2: the lowest fit that covers it
// (compared by the upper words, so a bound within 2^-20 of a fit's end takes the next one; NaN and
// infinity compare above all), kCotHalving beyond, and for steps so small that even the short group
// would overflow (dt < 2^-59), which need no halvings there.
__device__ __forceinline__ int cot_variant(double xb, double dt) {
  const uint32_t hi = __builtin_amdgcn_readfirstlane(__double2hiint(xb));
  int mode = kCotHalving;
#pragma unroll
  for (int k = kNumCot - 1; k >= 0; --k)
    if (hi < high_word(kCotXmax[k])) mode = k;
  return dt < kGroupShortMinDt ? kCotHalving : mode;
}

// The steps of one chunk (len table records of buf) for the MPL modes of a lane in fit variant V,
// rescaled every `group` steps.
template <int V, int MPL>
__device__ __forceinline__ void run_cot(State (&v)[MPL], const double2* buf, int len, double dt,
                                        const CotMode (&m)[MPL]) {
  const int group = dt >= kGroupLongMinDt ? kGroupLong : kGroupShort;
  CotCoef<V> k[MPL];
#pragma unroll
  for (int j = 0; j < MPL; ++j) {
    double e = m[j].e;
    asm volatile("" : "+v"(e));  // keeps this set-up inside the chunk loop, out of long-lived registers
    k[j] = cot_coef<V>(cot_step_size(e, dt));
  }
  for (int n0 = 0; n0 < len; n0 += group) {
    const int end = min(n0 + group, len);
#pragma unroll kCotUnroll
    for (int n = n0; n < end; ++n) {
      const double2 rec = buf[n];
#pragma unroll
      for (int j = 0; j < MPL; ++j) step_cot<V>(v[j], rec, m[j], k[j]);
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

// The chunk beyond the fits: C and S of degree 7 with angle halvings.
template <int MPL>
__device__ __forceinline__ void run_halving(State (&v)[MPL], const double2* buf, int len, double xb, double dt,
                                            const CotMode (&m)[MPL]) {
  int h = 0;
  for (double x = xb; x > kCosSinXmax && h < kMaxHalvings; x *= 0.25) ++h;
  h = __builtin_amdgcn_readfirstlane(h);
  const double inv4h = ldexp(1.0, -2 * h);
  const double2* cs = kHalvingCoef;
  asm volatile("" : "+s"(cs));
#pragma unroll 1
  for (int n = 0; n < len; ++n) {
    const double2 rec = buf[n];
#pragma unroll
    for (int j = 0; j < MPL; ++j) {
      // back to units of 1/dt: q = e dt q'
      const double qz = m[j].e * dt;
      const double qx = qz * fma(rec.x, m[j].nie, m[j].px), qy = qz * fma(rec.y, m[j].nie, m[j].py);
      double xs = fma(qx, qx, fma(qy, qy, qz * qz)) * inv4h;
      double C = cs[7].x, S = cs[7].y;
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
      rotate(v[j], C, S, qx, qy, qz);
    }
  }
}

// The steps of one chunk, in the variant that the bound xb on its (omega dt)^2 selects.
template <int MPL>
__device__ __forceinline__ void run_chunk(State (&v)[MPL], const double2* buf, int len, double xb, double dt,
                                          const CotMode (&m)[MPL]) {
  switch (cot_variant(xb, dt)) {
    case 0: run_cot<0, MPL>(v, buf, len, dt, m); break;
    case 1: run_cot<1, MPL>(v, buf, len, dt, m); break;
    case 2: run_cot<2, MPL>(v, buf, len, dt, m); break;
    case 3: run_cot<3, MPL>(v, buf, len, dt, m); break;
    case 4: run_cot<4, MPL>(v, buf, len, dt, m); break;
    case 5: run_cot<5, MPL>(v, buf, len, dt, m); break;
    case 6: run_cot<6, MPL>(v, buf, len, dt, m); break;
    case 7: run_cot<7, MPL>(v, buf, len, dt, m); break;
    case 8: run_cot<8, MPL>(v, buf, len, dt, m); break;
    default: run_halving<MPL>(v, buf, len, xb, dt, m); break;
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
  const BlockBox bb = block_box(d, first / kSelBlock, d.ndist);
  return ItemTab{reinterpret_cast<const double2*>(a.A) + d.tab_off, a.ranges + 4 * int64_t(d.chk_off),
                 BlockBox{uniform(bb.pxl), uniform(bb.pxh), uniform(bb.pyl), uniform(bb.pyh), uniform(bb.pz2)}, d.dt};
}

// Propagators of steps [n0, n1) for the MPL modes of a lane: the first column per block of a multiple of
// a unitary matrix.  Every lane of the workgroup must call it (barriers).  The table is staged
// through LDS chunk by chunk; the series variant of each piece is chosen from the item's selection
// block (items never straddle blocks) and the chunk's table range, so it depends only on the pulse,
// the block and the chunk, never on the launch.
template <int THREADS, int MPL>
__device__ __forceinline__ void propagate(State (&v)[MPL], const ItemTab& t, int n0, int n1, const CotMode (&mode)[MPL],
                                          double2* lds) {
#pragma unroll
  for (int j = 0; j < MPL; ++j) v[j] = State{1.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0};
  for (int n = n0; n < n1;) {
    const int c = n / kChunk, len = min((c + 1) * kChunk, n1) - n;
    __syncthreads();
    for (int i = threadIdx.x; i < len; i += THREADS) lds[i] = t.tab[n + i];
    __syncthreads();
    const double* rg = t.rg + 4 * c;
    run_chunk<MPL>(v, lds, len, x_bound(t.bb, rg[0], rg[1], rg[2], rg[3], t.dt), t.dt, mode);
    n += len;
  }
}

// Evolves the item of THREADS * MPL modes of pulse pi starting at mode `first`, writes f and the
// 64-mode unit sums.  Every lane of the workgroup must call it (it contains barriers).
template <int THREADS, int MPL>
__device__ __forceinline__ void process_item(const EvolveArgs& a, int pi, int first, double2* lds) {
  const PulseDev& d = a.desc[pi];
  const double2* edge = reinterpret_cast<const double2*>(a.Aedge) + 2 * pi;
  const double2 ain = edge[0];
  const ItemTab t = item_tab(a, d, first);

  State psi[MPL];
  CotMode mode[MPL];
#pragma unroll
  for (int j = 0; j < MPL; ++j) {
    double px, py;
    const double e = lane_mode(d, int64_t(first) + j * THREADS + threadIdx.x, px, py);
    init_state(psi[j], px - ain.x, py - ain.y, e);
    mode[j] = cot_mode(px, py, e);
  }
  for (int n0 = 0; n0 < d.nt; n0 += d.seg_len) {
    State v[MPL];
    propagate<THREADS, MPL>(v, t, n0, min(n0 + d.seg_len, d.nt), mode, lds);
#pragma unroll
    for (int j = 0; j < MPL; ++j) {
      apply_propagator(psi[j], v[j]);
      rescale(psi[j]);
    }
  }

  const double2 aout = edge[1];
#pragma unroll
  for (int j = 0; j < MPL; ++j) {
    const int64_t m = int64_t(first) + j * THREADS + threadIdx.x;
    double px, py;
    const double e = lane_mode(d, m, px, py);
    write_density(d, a.f, a.units, m, m < d.ndist ? project(psi[j], px - aout.x, py - aout.y, e) : 0.0);
  }
}

// One workgroup per 256-mode item; four waves per SIMD (the register budget of the variant
// switch, met without spills).
__global__ void __launch_bounds__(kItem) __attribute__((amdgpu_waves_per_eu(4))) k_evolve(EvolveArgs a) {
  __shared__ double2 lds[kChunk];
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int pi = find_pulse_item(a.desc, a.n_pulses, item);
  process_item<kItem, 1>(a, pi, (item - a.desc[pi].item_off) * kItem, lds);
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
  State v[1];
  propagate<kItem, 1>(v, item_tab(a, d, li * kItem), seg * d.seg_len, min((seg + 1) * d.seg_len, d.nt), mode, lds);
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
  __shared__ double2 lds[kChunk];
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

// Diagnostics: adds modes x steps of every (selection block, chunk) of every pulse to the count
// of its step-size class (the ranges of the tangent fits, by block_variant and chunk_variant); the
// blocks here run over all modes of the grid, mirror images included.
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
    const int bmode = block_variant(bb, rg, nch, d.dt).x;
    for (int c = 0; c < nch; ++c) {
      const int mode = chunk_variant(bb, rg, c, bmode, d.dt).x;
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
// and the step is again U = C [1 - i T(|w_s|^2) w_s . tau], now with one w_s (and one T) per
// block.  With a_k = (p_x - A_x(t_k)) dt, b_k likewise, e = e_perp dt, abar = (a_1 + a_2)/2 and
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

template <int V>  // series variant
__device__ __forceinline__ void step4_tan(State& v, double4 rec, double pxdt, double pydt, double e, const Fit<V>& f) {
  const Magnus4 w = magnus4(rec, pxdt, pydt, e);
  const double xp = fma(w.Xp, w.Xp, fma(w.Yp, w.Yp, w.Zp * w.Zp));
  const double xm = fma(w.Xm, w.Xm, fma(w.Ym, w.Ym, w.Zm * w.Zm));
  const double Tp = tan_ratio<V>(xp, f), Tm = tan_ratio<V>(xm, f);
  rotate_block_tan(v.ar, v.ai, v.br, v.bi, Tp * w.Xp, Tp * w.Yp, Tp * w.Zp);
  rotate_block_tan(v.cr, v.ci, v.dr, v.di, Tm * w.Xm, -(Tm * w.Ym), Tm * w.Zm);
}

__device__ __forceinline__ void step4_halving(State& v, double4 rec, double pxdt, double pydt, double e, int h,
                                              double inv4h) {
  const Magnus4 w = magnus4(rec, pxdt, pydt, e);
  const double xp = fma(w.Xp, w.Xp, fma(w.Yp, w.Yp, w.Zp * w.Zp));
  const double xm = fma(w.Xm, w.Xm, fma(w.Ym, w.Ym, w.Zm * w.Zm));
  double Cp, Sp, Cm, Sm;
  cos_sinc_halved(xp, h, inv4h, Cp, Sp);
  cos_sinc_halved(xm, h, inv4h, Cm, Sm);
  rotate_block(v.ar, v.ai, v.br, v.bi, Cp, Sp * w.Xp, Sp * w.Yp, Sp * w.Zp);
  rotate_block(v.cr, v.ci, v.dr, v.di, Cm, Sm * w.Xm, -(Sm * w.Ym), Sm * w.Zm);
}

// Rescales each block by its own exact power of two.
__device__ __forceinline__ void renormalise_blocks(State& v) {
  const double n1 = fma(v.bi, v.bi, fma(v.br, v.br, fma(v.ai, v.ai, v.ar * v.ar)));
  const double n2 = fma(v.di, v.di, fma(v.dr, v.dr, fma(v.ci, v.ci, v.cr * v.cr)));
  const int e1 = -(ilogb(n1) >> 1), e2 = -(ilogb(n2) >> 1);
  v.ar = ldexp(v.ar, e1); v.ai = ldexp(v.ai, e1); v.br = ldexp(v.br, e1); v.bi = ldexp(v.bi, e1);
  v.cr = ldexp(v.cr, e2); v.ci = ldexp(v.ci, e2); v.dr = ldexp(v.dr, e2); v.di = ldexp(v.di, e2);
}

// Steps of one chunk in variant MODE; the tangent form then rescales each block.
template <int MODE>
__device__ __forceinline__ void run_chunk4(State& v, const double4* buf, int len, double pxdt, double pydt, double e,
                                           int h) {
  if constexpr (MODE < kFineHalving) {
    const Fit<MODE> f = load_fit<MODE>();
    if (len == kChunk) {
#pragma unroll 2
      for (int k = 0; k < kChunk; ++k) step4_tan<MODE>(v, buf[k], pxdt, pydt, e, f);
    } else {
      for (int k = 0; k < len; ++k) step4_tan<MODE>(v, buf[k], pxdt, pydt, e, f);
    }
    renormalise_blocks(v);
  } else {
    const double inv4h = ldexp(1.0, -2 * h);
    if (len == kChunk) {
#pragma unroll 2
      for (int k = 0; k < kChunk; ++k) step4_halving(v, buf[k], pxdt, pydt, e, h, inv4h);
    } else {
      for (int k = 0; k < len; ++k) step4_halving(v, buf[k], pxdt, pydt, e, h, inv4h);
    }
  }
}

struct Evolve4Args {
  const PulseDev* desc;
  int n_pulses;
  const double* Ag;  // [sum nt][2 nodes][2] A at the Gauss-Legendre nodes
  const double* Aedge;
  const double* ranges;  // [total_chunks][4] range of the node values per chunk (k_chunk_ranges<2>)
  double* f;
  double* units;
};

// The chunks of a fourth-order item, as chunk_loop: the record staged per step is
// (-(A_1 + A_2) dt/2, (sqrt3/6)(A_2 - A_1) dt); each chunk in its variant (chunk_variant<2>).
template <bool HALVING>
__device__ __forceinline__ void chunk_loop4(State& v, const double4* tab, int nt, double dt, const double* rg,
                                            const BlockBox& bb, int bmode, double pxdt, double pydt, double e,
                                            double4 (*lds)[kChunk]) {
  const double hdt = -0.5 * dt, kdt = kSqrt3Over6 * dt;
  const int nchunks = (nt + kChunk - 1) / kChunk;
  {
    const double4 t = int(threadIdx.x) < nt ? tab[threadIdx.x] : make_double4(0.0, 0.0, 0.0, 0.0);
    lds[0][threadIdx.x] = make_double4(hdt * (t.x + t.z), hdt * (t.y + t.w), kdt * (t.z - t.x), kdt * (t.w - t.y));
  }
  __syncthreads();
  for (int c = 0; c < nchunks; ++c) {
    const int n = (c + 1) * kChunk + threadIdx.x;
    const double4 pre = (c + 1 < nchunks && n < nt) ? tab[n] : make_double4(0.0, 0.0, 0.0, 0.0);
    const double4* buf = lds[c & 1];
    const int len = min(kChunk, nt - c * kChunk);
    const int2 cv = chunk_variant<2>(bb, rg, c, bmode, dt);
    const int mode = __builtin_amdgcn_readfirstlane(cv.x);
    if constexpr (HALVING) {
      if (mode == kFineHalving)
        run_chunk4<kFineHalving>(v, buf, len, pxdt, pydt, e, __builtin_amdgcn_readfirstlane(cv.y));
      else
        run_chunk4<kNumFine - 1>(v, buf, len, pxdt, pydt, e, 0);
    } else {
      switch (mode) {
        case 0: run_chunk4<0>(v, buf, len, pxdt, pydt, e, 0); break;
        case 1: run_chunk4<1>(v, buf, len, pxdt, pydt, e, 0); break;
        case 2: run_chunk4<2>(v, buf, len, pxdt, pydt, e, 0); break;
        case 3: run_chunk4<3>(v, buf, len, pxdt, pydt, e, 0); break;
        case 4: run_chunk4<4>(v, buf, len, pxdt, pydt, e, 0); break;
        case 5: run_chunk4<5>(v, buf, len, pxdt, pydt, e, 0); break;
        case 6: run_chunk4<6>(v, buf, len, pxdt, pydt, e, 0); break;
        default: run_chunk4<7>(v, buf, len, pxdt, pydt, e, 0); break;
      }
    }
    lds[(c + 1) & 1][threadIdx.x] =
        make_double4(hdt * (pre.x + pre.z), hdt * (pre.y + pre.w), kdt * (pre.z - pre.x), kdt * (pre.w - pre.y));
    __syncthreads();
  }
}

// One 256-mode item of pulse pi, one mode per lane; the structure of process_item, with the
// series variant per (selection block, chunk) from the range of both node values.
__device__ __forceinline__ void process_item4(const Evolve4Args& a, int pi, int first, double4 (*lds)[kChunk]) {
  const PulseDev& d = a.desc[pi];
  const int nt = d.nt;
  const double dt = d.dt;
  const double4* tab = reinterpret_cast<const double4*>(a.Ag) + d.tab_off;
  const double2* edge = reinterpret_cast<const double2*>(a.Aedge) + 2 * pi;
  const int64_t m = int64_t(first) + threadIdx.x;
  double px, py, pz;
  mode_momentum(d, m < d.ndist ? m : 0, px, py, pz);
  const double ep = sqrt(fma(pz, pz, 1.0));
  State v;
  const double2 ain = edge[0];
  init_state(v, px - ain.x, py - ain.y, ep);
  const double pxdt = px * dt, pydt = py * dt, e = ep * dt;
  const BlockBox bb = block_box(d, first / kSelBlock, d.ndist);
  const double* rg = a.ranges + 4 * int64_t(d.chk_off);
  const int bmode = __builtin_amdgcn_readfirstlane(block_variant<2>(bb, rg, (nt + kChunk - 1) / kChunk, dt).x);
  if (bmode == kFineHalving)
    chunk_loop4<true>(v, tab, nt, dt, rg, bb, bmode, pxdt, pydt, e, lds);
  else
    chunk_loop4<false>(v, tab, nt, dt, rg, bb, bmode, pxdt, pydt, e, lds);

  const double2 aout = edge[1];
  write_density(d, a.f, a.units, m, m < d.ndist ? project(v, px - aout.x, py - aout.y, ep) : 0.0);
}

__global__ void __launch_bounds__(kItem) __attribute__((amdgpu_waves_per_eu(4))) k_evolve4(Evolve4Args a) {
  __shared__ double4 lds[2][kChunk];
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int pi = find_pulse_item(a.desc, a.n_pulses, item);
  process_item4(a, pi, (item - a.desc[pi].item_off) * kItem, lds);
}

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
// K = C (1 - i T Q_s) with T = tan|q| / |q| (the evolution's polynomial fits, x = |q|^2); since
// tau_z Q_s = i (q_x tau_y - s q_y tau_x), the product is 1 - i w_s . tau with
//     w_s = (u - s a v, s v + a u, a),   u = T q_x, v = T q_y,
// again a scalar multiple of a unitary matrix, of the same norm for both blocks: one rescaling per
// chunk, as in the midpoint step (34 + n VALU instructions per substep against 31 + n).  Beyond
// the fits' range the exact C, S (angle halving) and c = cos(theta), s = sin(theta) give
//     R K = c C - i (S (c q_x - s_b s q_y), S (s_b c q_y + s q_x), s C) . tau,   s_b = +-1.
// ---------------------------------------------------------------------------------------------
constexpr double kTripleW1 = 1.3512071919596576;   // 1 / (2 - 2^(1/3))
constexpr double kTripleW0 = -1.7024143839193153;  // 1 - 2 w1

template <int NSUB>
struct SplitMode {
  double pxw[NSUB == 1 ? 1 : 2], pyw[NSUB == 1 ? 1 : 2];  // p w dt for the distinct weights
  double a[NSUB == 1 ? 1 : 2], c[NSUB == 1 ? 1 : 2], s[NSUB == 1 ? 1 : 2];  // tan, cos, sin of theta_i
};

// Weight index (into pxw, pyw) and angle index (into a, c, s) of substep i.
__device__ __forceinline__ constexpr int split_w(int i) { return i == 1 ? 1 : 0; }
__device__ __forceinline__ constexpr int split_t(int i) { return i == 2 ? 1 : 0; }

// psi <- R(phi) psi for both blocks: a <- a e^{-i phi}, b <- b e^{i phi}.
__device__ __forceinline__ void phase_z(State& v, double cp, double sp) {
  double r, i;
  r = fma(v.ai, sp, v.ar * cp); i = fma(-v.ar, sp, v.ai * cp); v.ar = r; v.ai = i;
  r = fma(-v.bi, sp, v.br * cp); i = fma(v.br, sp, v.bi * cp); v.br = r; v.bi = i;
  r = fma(v.ci, sp, v.cr * cp); i = fma(-v.cr, sp, v.ci * cp); v.cr = r; v.ci = i;
  r = fma(-v.di, sp, v.dr * cp); i = fma(v.dr, sp, v.di * cp); v.dr = r; v.di = i;
}

template <int V>
__device__ __forceinline__ void substep_split_tan(State& v, double2 rec, double pxw, double pyw, double a,
                                                  const Fit<V>& f) {
  const double qx = pxw + rec.x, qy = pyw + rec.y;  // rec = -A w dt
  const double x = fma(qx, qx, qy * qy);
  const double T = tan_ratio<V>(x, f);
  const double u = T * qx, w = T * qy;
  rotate_block_tan(v.ar, v.ai, v.br, v.bi, fma(-a, w, u), fma(a, u, w), a);
  rotate_block_tan(v.cr, v.ci, v.dr, v.di, fma(a, w, u), fma(a, u, -w), a);
}

__device__ __forceinline__ void substep_split_halving(State& v, double2 rec, double pxw, double pyw, double c,
                                                      double s, int h, double inv4h) {
  const double qx = pxw + rec.x, qy = pyw + rec.y;
  const double x = fma(qx, qx, qy * qy);
  double C, S;
  cos_sinc_halved(x, h, inv4h, C, S);
  const double cC = c * C, sz = s * C;
  const double cx = c * qx, cy = c * qy, sx = s * qx, sy = s * qy;
  rotate_block(v.ar, v.ai, v.br, v.bi, cC, S * (cx - sy), S * (cy + sx), sz);
  rotate_block(v.cr, v.ci, v.dr, v.di, cC, S * (cx + sy), S * (sx - cy), sz);
}

template <int NSUB, int MODE>
__device__ __forceinline__ void run_chunk_split(State& v, const double2* buf, int len, const SplitMode<NSUB>& k,
                                                int h) {
  if constexpr (MODE < kFineHalving) {
    const Fit<MODE> f = load_fit<MODE>();
    if (len == kChunk) {
#pragma unroll(NSUB == 1 ? 4 : 1)
      for (int n = 0; n < kChunk; ++n)
#pragma unroll
        for (int i = 0; i < NSUB; ++i)
          substep_split_tan<MODE>(v, buf[n * NSUB + i], k.pxw[split_w(i)], k.pyw[split_w(i)], k.a[split_t(i)], f);
    } else {
      for (int n = 0; n < len; ++n)
#pragma unroll
        for (int i = 0; i < NSUB; ++i)
          substep_split_tan<MODE>(v, buf[n * NSUB + i], k.pxw[split_w(i)], k.pyw[split_w(i)], k.a[split_t(i)], f);
    }
    renormalise(v);
  } else {
    const double inv4h = ldexp(1.0, -2 * h);
    for (int n = 0; n < len; ++n)
#pragma unroll
      for (int i = 0; i < NSUB; ++i)
        substep_split_halving(v, buf[n * NSUB + i], k.pxw[split_w(i)], k.pyw[split_w(i)], k.c[split_t(i)],
                              k.s[split_t(i)], h, inv4h);
  }
}

struct SplitArgs {
  const PulseDev* desc;
  int n_pulses;
  const double* At;  // [sum nt][NSUB][2] A at the substep midpoints
  const double* Aedge;
  const double* ranges;  // [total_chunks][4] range of the table per chunk (k_chunk_ranges<NSUB>)
  double* f;
  double* units;
};

// The chunks of an item: NSUB records per step staged through LDS as -A w_i dt (double-buffered,
// one barrier per chunk), each chunk in its variant for steps of size w_max dt.
template <int NSUB, bool HALVING>
__device__ __forceinline__ void chunk_loop_split(State& v, const double2* tab, int nt, double dt, double dtw,
                                                 const double* rg, const BlockBox& bb, int bmode,
                                                 const SplitMode<NSUB>& k, double2 (*lds)[NSUB * kChunk]) {
  const double wdt[3] = {NSUB == 1 ? -dt : -kTripleW1 * dt, -kTripleW0 * dt, -kTripleW1 * dt};
  const int nchunks = (nt + kChunk - 1) / kChunk;
#pragma unroll
  for (int i = 0; i < NSUB; ++i) {
    const double2 t = int(threadIdx.x) < nt ? tab[NSUB * threadIdx.x + i] : make_double2(0.0, 0.0);
    lds[0][NSUB * threadIdx.x + i] = make_double2(t.x * wdt[i], t.y * wdt[i]);
  }
  __syncthreads();
  for (int c = 0; c < nchunks; ++c) {
    double2 pre[NSUB];
    const int n = (c + 1) * kChunk + threadIdx.x;
#pragma unroll
    for (int i = 0; i < NSUB; ++i) pre[i] = (c + 1 < nchunks && n < nt) ? tab[NSUB * n + i] : make_double2(0.0, 0.0);
    const double2* buf = lds[c & 1];
    const int len = min(kChunk, nt - c * kChunk);
    const int2 cv = chunk_variant<1>(bb, rg, c, bmode, dtw);
    const int mode = __builtin_amdgcn_readfirstlane(cv.x);
    if constexpr (HALVING) {
      if (mode == kFineHalving)
        run_chunk_split<NSUB, kFineHalving>(v, buf, len, k, __builtin_amdgcn_readfirstlane(cv.y));
      else
        run_chunk_split<NSUB, kNumFine - 1>(v, buf, len, k, 0);
    } else {
      switch (mode) {
        case 0: run_chunk_split<NSUB, 0>(v, buf, len, k, 0); break;
        case 1: run_chunk_split<NSUB, 1>(v, buf, len, k, 0); break;
        case 2: run_chunk_split<NSUB, 2>(v, buf, len, k, 0); break;
        case 3: run_chunk_split<NSUB, 3>(v, buf, len, k, 0); break;
        case 4: run_chunk_split<NSUB, 4>(v, buf, len, k, 0); break;
        case 5: run_chunk_split<NSUB, 5>(v, buf, len, k, 0); break;
        case 6: run_chunk_split<NSUB, 6>(v, buf, len, k, 0); break;
        default: run_chunk_split<NSUB, 7>(v, buf, len, k, 0); break;
      }
    }
#pragma unroll
    for (int i = 0; i < NSUB; ++i)
      lds[(c + 1) & 1][NSUB * threadIdx.x + i] = make_double2(pre[i].x * wdt[i], pre[i].y * wdt[i]);
    __syncthreads();
  }
}

// One 256-mode item of pulse pi, one mode per lane, the structure of process_item4.  The series
// variant per (selection block, chunk) bounds |q|^2 <= |p - A|^2 (w_max dt)^2 through the
// second-order bound at step w_max dt (which also counts (1 + p_z^2)(w_max dt)^2: conservative).
template <int NSUB>
__device__ __forceinline__ void process_item_split(const SplitArgs& a, int pi, int first,
                                                   double2 (*lds)[NSUB * kChunk]) {
  const PulseDev& d = a.desc[pi];
  const int nt = d.nt;
  const double dt = d.dt;
  const double dtw = NSUB == 1 ? dt : -kTripleW0 * dt;  // the largest substep
  const double2* tab = reinterpret_cast<const double2*>(a.At) + NSUB * d.tab_off;
  const double2* edge = reinterpret_cast<const double2*>(a.Aedge) + 2 * pi;
  const int64_t m = int64_t(first) + threadIdx.x;
  double px, py, pz;
  mode_momentum(d, m < d.ndist ? m : 0, px, py, pz);
  const double ep = sqrt(fma(pz, pz, 1.0));
  SplitMode<NSUB> k;
  double th0;
  if constexpr (NSUB == 1) {
    k.pxw[0] = px * dt;
    k.pyw[0] = py * dt;
    sincos(ep * dt, &k.s[0], &k.c[0]);
    th0 = 0.5 * ep * dt;
  } else {
    k.pxw[0] = px * (kTripleW1 * dt); k.pyw[0] = py * (kTripleW1 * dt);
    k.pxw[1] = px * (kTripleW0 * dt); k.pyw[1] = py * (kTripleW0 * dt);
    sincos(0.5 * (kTripleW1 + kTripleW0) * ep * dt, &k.s[0], &k.c[0]);
    sincos(kTripleW1 * ep * dt, &k.s[1], &k.c[1]);
    th0 = 0.5 * kTripleW1 * ep * dt;
  }
#pragma unroll
  for (int j = 0; j < (NSUB == 1 ? 1 : 2); ++j) k.a[j] = k.s[j] / k.c[j];
  double s0, c0;
  sincos(th0, &s0, &c0);
  State v;
  const double2 ain = edge[0];
  init_state(v, px - ain.x, py - ain.y, ep);
  phase_z(v, c0, s0);
  const BlockBox bb = block_box(d, first / kSelBlock, d.ndist);
  const double* rg = a.ranges + 4 * int64_t(d.chk_off);
  const int bmode = __builtin_amdgcn_readfirstlane(block_variant<1>(bb, rg, (nt + kChunk - 1) / kChunk, dtw).x);
  if (bmode == kFineHalving)
    chunk_loop_split<NSUB, true>(v, tab, nt, dt, dtw, rg, bb, bmode, k, lds);
  else
    chunk_loop_split<NSUB, false>(v, tab, nt, dt, dtw, rg, bb, bmode, k, lds);
  phase_z(v, c0, -s0);

  const double2 aout = edge[1];
  write_density(d, a.f, a.units, m, m < d.ndist ? project(v, px - aout.x, py - aout.y, ep) : 0.0);
}

template <int NSUB>
__global__ void __launch_bounds__(kItem) k_evolve_split(SplitArgs a) {
  __shared__ double2 lds[2][NSUB * kChunk];
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int pi = find_pulse_item(a.desc, a.n_pulses, item);
  process_item_split<NSUB>(a, pi, (item - a.desc[pi].item_off) * kItem, lds);
}

}  // namespace

po_status launch_chunk_ranges(const Batch& b, const PulseDev* d_desc, const double* d_A, double* d_ranges,
                              hipStream_t s) {
  const int max_chunks = (b.max_nt + kChunk - 1) / kChunk;
  hipLaunchKernelGGL(k_chunk_ranges<1>, dim3(max_chunks, b.n_pulses), dim3(256), 0, s, d_desc, d_A, d_ranges);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

po_status launch_evolve_grid(const Batch& b, const PulseDev* d_desc, const double* d_A, const double* d_A_edge,
                             const double* d_ranges, double* d_f, double* d_units, hipStream_t s) {
  EvolveArgs a{d_desc, b.n_pulses, d_A, d_A_edge, d_ranges, d_f, d_units};
  hipLaunchKernelGGL(k_evolve, dim3(b.total_items), dim3(kItem), 0, s, a);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

// The batch is split in time when its items alone load the CUs thinly or unevenly.  Measured, one
// pulse at nt = 4096, us per call split / not split: 16 items 75 / 357, 128 items 190 / 344, 256 items
// 329 / 352, 320 items 402 / 581 (some CUs then hold two workgroups, the others one), 384 items
// 480 / 594, 512 items 619 / 626 and, at nt = 1024, 194 / 177.  At most 8192 slots (128 MiB of
// propagators).
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

po_status launch_chunk_ranges4(const Batch& b, const PulseDev* d_desc, const double* d_Ag, double* d_ranges,
                               hipStream_t s) {
  const int max_chunks = (b.max_nt + kChunk - 1) / kChunk;
  hipLaunchKernelGGL(k_chunk_ranges<2>, dim3(max_chunks, b.n_pulses), dim3(256), 0, s, d_desc, d_Ag, d_ranges);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

po_status launch_evolve4_grid(const Batch& b, const PulseDev* d_desc, const double* d_Ag, const double* d_A_edge,
                              const double* d_ranges, double* d_f, double* d_units, hipStream_t s) {
  Evolve4Args a{d_desc, b.n_pulses, d_Ag, d_A_edge, d_ranges, d_f, d_units};
  hipLaunchKernelGGL(k_evolve4, dim3(b.total_items), dim3(kItem), 0, s, a);
  PO_HIP(hipGetLastError());
  return PO_OK;
}

po_status launch_evolve_split_grid(const Batch& b, int order, const PulseDev* d_desc, const double* d_At,
                                   const double* d_A_edge, double* d_ranges, double* d_f, double* d_units,
                                   hipStream_t s) {
  const int max_chunks = (b.max_nt + kChunk - 1) / kChunk;
  SplitArgs a{d_desc, b.n_pulses, d_At, d_A_edge, d_ranges, d_f, d_units};
  if (order == 2) {
    hipLaunchKernelGGL(k_chunk_ranges<1>, dim3(max_chunks, b.n_pulses), dim3(256), 0, s, d_desc, d_At, d_ranges);
    PO_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_evolve_split<1>, dim3(b.total_items), dim3(kItem), 0, s, a);
  } else {
    hipLaunchKernelGGL(k_chunk_ranges<3>, dim3(max_chunks, b.n_pulses), dim3(256), 0, s, d_desc, d_At, d_ranges);
    PO_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_evolve_split<3>, dim3(b.total_items), dim3(kItem), 0, s, a);
  }
  PO_HIP(hipGetLastError());
  return PO_OK;
}

}  // namespace po
