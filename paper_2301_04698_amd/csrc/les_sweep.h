// Point update of a weighted-Jacobi / Chebyshev sweep and the lane shifts of
// its x neighbours, shared by every sweep kernel so that their iterates are
// bitwise equal:
//   r   = rhs - (N(phi) - D phi)     N: off-diagonal neighbour sum, FP64
//   J   = phi - omega_j r / D         (weighted Jacobi)
//   out = J, or Chebyshev: prev + omega_c (J - prev)
// formed in FP64 from the stored values with explicit FMAs (no other
// contraction) and rounded once to the storage type.  An FP32 update
// written as (N - rhs)/D - phi cancels catastrophically; its rounding error
// is the same from sweep to sweep and accumulates in the slow modes.
#pragma once

#include "les_device.h"

namespace lesmi {

struct SweepCoef {
  double ix2, iy2, iz2, diag;
  double step;  // -omega_j / D, as the product of omega_j and the rounded 1 / D
};

inline SweepCoef sweep_coef(const Grid &g, double omega_j) {
  SweepCoef k;
  k.ix2 = 1.0 / (g.dx * g.dx);
  k.iy2 = 1.0 / (g.dy * g.dy);
  k.iz2 = 1.0 / (g.dz * g.dz);
  k.diag = 2.0 * (k.ix2 + k.iy2 + k.iz2);
  k.step = -omega_j * (1.0 / k.diag);
  return k;
}

__device__ __forceinline__ double point_residual(const SweepCoef &k, double c0, double hx,
                                                 double hy, double hz, double rhs) {
#pragma clang fp contract(off)
  const double lap = fma(hx, k.ix2, fma(hy, k.iy2, fma(hz, k.iz2, -k.diag * c0)));
  return rhs - lap;
}

__device__ __forceinline__ double point_update(const SweepCoef &k, double c0, double res,
                                               bool cheb, double pv, double wc) {
#pragma clang fp contract(off)
  const double jac = fma(k.step, res, c0);
  return cheb ? fma(wc, jac - pv, pv) : jac;
}

// Value of v in the next (+1) or previous (-1) lane of the 64-wide
// wavefront by DPP wave shifts; the lane without a source gets `edge`.  A
// double moves as two 32-bit halves.
template <int DIR>
__device__ __forceinline__ int lane_shift_word(int edge, int x) {
  return __builtin_amdgcn_update_dpp(edge, x, DIR > 0 ? 0x130 : 0x138, 0xF, 0xF, false);
}
template <int DIR>
__device__ __forceinline__ float lane_shift(float v, float edge) {
  return __int_as_float(lane_shift_word<DIR>(__float_as_int(edge), __float_as_int(v)));
}
template <int DIR>
__device__ __forceinline__ double lane_shift(double v, double edge) {
  return __hiloint2double(lane_shift_word<DIR>(__double2hiint(edge), __double2hiint(v)),
                          lane_shift_word<DIR>(__double2loint(edge), __double2loint(v)));
}
// As above; a lane without a source keeps its own value (the caller
// replaces the end lanes).
template <int DIR, typename T>
__device__ __forceinline__ T lane_shift(T v) {
  return lane_shift<DIR>(v, v);
}

}  // namespace lesmi
