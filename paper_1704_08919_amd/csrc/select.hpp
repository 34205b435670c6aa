// Choice of the step's series from bounds on the step angle, and the lane's mode: shared by the
// evolution and yield-gradient kernels.
#pragma once

#include "dirac.hpp"
#include "reduce.hpp"

#pragma clang fp contract(off)

namespace po {
namespace {

// Box of cell-centred momenta of selection block b (kSelBlock consecutive modes of the first nmodes)
// of a pulse: [pxl, pxh] x [pyl, pyh] and the largest p_z^2.
struct BlockBox {
  double pxl, pxh, pyl, pyh, pz2;
};

__device__ __forceinline__ BlockBox block_box(const PulseDev& d, int b, int64_t nmodes) {
  const int nx = d.n[0], ny = d.n[1];
  const int64_t m0 = int64_t(b) * kSelBlock, m1 = min(m0 + kSelBlock, nmodes) - 1;
  const int64_t r0 = m0 / nx, r1 = m1 / nx;  // rows (iy, iz)
  const int64_t z0 = r0 / ny, z1 = r1 / ny;
  const int ix0 = r0 == r1 ? int(m0 % nx) : 0, ix1 = r0 == r1 ? int(m1 % nx) : nx - 1;
  const int iy0 = z0 == z1 ? int(r0 % ny) : 0, iy1 = z0 == z1 ? int(r1 % ny) : ny - 1;
  const double px0 = d.lo[0] + (ix0 + 0.5) * d.dp[0], px1 = d.lo[0] + (ix1 + 0.5) * d.dp[0];
  const double py0 = d.lo[1] + (iy0 + 0.5) * d.dp[1], py1 = d.lo[1] + (iy1 + 0.5) * d.dp[1];
  const double pz0 = d.lo[2] + (z0 + 0.5) * d.dp[2], pz1 = d.lo[2] + (z1 + 0.5) * d.dp[2];
  return BlockBox{fmin(px0, px1), fmax(px0, px1), fmin(py0, py1), fmax(py0, py1), fmax(pz0 * pz0, pz1 * pz1)};
}

// Bound on x = (omega dt)^2 for a block box against a range [lx, hx] x [ly, hy] of table values, with the largest
// |p - A| per component: dt^2 [ max|p_x - A_x|^2 + max|p_y - A_y|^2 + 1 + max p_z^2 ].
__device__ __forceinline__ double x_bound(const BlockBox& bb, double lx, double hx, double ly, double hy, double dt) {
  const double X = fmax(fmax(bb.pxh - lx, hx - bb.pxl), 0.0);
  const double Y = fmax(fmax(bb.pyh - ly, hy - bb.pyl), 0.0);
  return (X * X + Y * Y + 1.0 + bb.pz2) * dt * dt * (1.0 + 1e-6);
}

// A value that is equal in all lanes, in scalar registers.
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// Box of the selection block that distinct mode `first` (the same in all lanes) lies in, in scalar registers.
__device__ __forceinline__ BlockBox uniform_box(const PulseDev& d, int first) {
  const BlockBox bb = block_box(d, first / kSelBlock, d.ndist);
  return BlockBox{uniform(bb.pxl), uniform(bb.pxh), uniform(bb.pyl), uniform(bb.pyh), uniform(bb.pz2)};
}

// Upper 32 bits of a positive double (ordered as the doubles are).
constexpr uint32_t high_word(double v) { return uint32_t(__builtin_bit_cast(uint64_t, v) >> 32); }

// Momentum of distinct mode m, its e_perp; lanes beyond the last one take the last one's, which lies in the box their
// block's series is chosen for (another mode's step angle may be far outside the fit's range, where the
// state overflows).
__device__ __forceinline__ double lane_mode(const PulseDev& d, int64_t m, double& px, double& py) {
  double pz;
  mode_momentum(d, min(m, d.ndist - 1), px, py, pz);
  return sqrt(fma(pz, pz, 1.0));
}

}  // namespace
}  // namespace po
