// Small dense algebra in fp64 inside one workgroup (gfx950): symmetric positive definite systems
// of up to 64 x 64 elements as 16 x 16 tiles in registers, eliminated with 4 x 4 pivot blocks, a
// rank-4 update of a tile being one v_mfma_f64_16x16x4.  fp64 instructions issue at the rate of
// unpacked fp32 ones here, so the wider type costs registers and LDS but hardly any time.  Used by
// the prefill factorisation and by the decode-time factor update.
#pragma once

#include "lrqk_device.h"

namespace lrqk {
namespace alg64 {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// D(16x16) = A(16x4) B(4x16) + C; lane i + 16 h supplies A[i][h] and B[h][i]; register v of
// lane l holds D[4 v + l / 16][l % 16]
__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

using dev::lds_barrier;

// 1 / x: the hardware estimate and three Newton steps (an IEEE division would lengthen the chain
// of every elimination step by half; the last bit does not matter here).
__device__ __forceinline__ double recip(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
  y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
  return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
}

// Element (i, k) of the factor N by which a step of Gauss-Jordan elimination multiplies the pivot
// rows before it adds them to every row: -C D^-1, and D^-1 - I for the pivot rows themselves.
// C: the pivot columns, [rows][4] in LDS; the pivots are rows p0 .. p0 + 3, D = C[p0 ..].
__device__ __forceinline__ double pivot_factor(const double* C, int p0, int i, int k) {
  const double* D = C + p0 * 4;
  const double d00 = D[0], d01 = D[1], d02 = D[2], d03 = D[3], d11 = D[5], d12 = D[6],
               d13 = D[7], d22 = D[10], d23 = D[11], d33 = D[15];
  // D = [E F; F^T L] in 2 x 2 blocks, W = E^-1 F, T = (L - F^T W)^-1
  const double ie = recip(d00 * d11 - d01 * d01);
  const double e00 = d11 * ie, e01 = -d01 * ie, e11 = d00 * ie;
  const double w00 = e00 * d02 + e01 * d12, w01 = e00 * d03 + e01 * d13;
  const double w10 = e01 * d02 + e11 * d12, w11 = e01 * d03 + e11 * d13;
  const double l00 = d22 - (d02 * w00 + d12 * w10), l01 = d23 - (d02 * w01 + d12 * w11);
  const double l11 = d33 - (d03 * w01 + d13 * w11);
  const double il = recip(l00 * l11 - l01 * l01);
  const double t00 = l11 * il, t01 = -l01 * il, t11 = l00 * il;
  const double u00 = w00 * t00 + w01 * t01, u01 = w00 * t01 + w01 * t11;  // W T
  const double u10 = w10 * t00 + w11 * t01, u11 = w10 * t01 + w11 * t11;
  // column k of D^-1 = [E^-1 + W T W^T, -W T; -T W^T, T].  (Every entry is computed before the
  // selection: with the arithmetic inside the branches of a chain of ifs on k, this compiler
  // gave the lanes of the last branch an unset register.)
  const double f00 = e00 + (u00 * w00 + u01 * w01), f01 = e01 + (u00 * w10 + u01 * w11);
  const double f11 = e11 + (u10 * w10 + u11 * w11);
  const bool odd = k & 1, low = k < 2;
  const double x0 = low ? (odd ? f01 : f00) : -(odd ? u01 : u00);
  const double x1 = low ? (odd ? f11 : f01) : -(odd ? u11 : u10);
  const double x2 = low ? -(odd ? u10 : u00) : (odd ? t01 : t00);
  const double x3 = low ? -(odd ? u11 : u01) : (odd ? t11 : t01);
  const double* c = C + i * 4;
  const double n = -(c[0] * x0 + c[1] * x1 + (c[2] * x2 + c[3] * x3));
  const int m = i - p0;
  const double own = (m == 0 ? x0 : m == 1 ? x1 : m == 2 ? x2 : x3) - (m == k ? 1.0 : 0.0);
  return m >= 0 && m < 4 ? own : n;
}

// Sum over the 16 lanes of a DPP row, the same in every lane of it.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double lane_value_f64(double v, int lane) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wave_sum_f64(double v) {
  v += dpp_f64<0x128>(v);  // row_ror:8
  v += dpp_f64<0x124>(v);  // row_ror:4
  v += dpp_f64<0x122>(v);  // row_ror:2
  v += dpp_f64<0x121>(v);  // row_ror:1
  return (lane_value_f64(v, 0) + lane_value_f64(v, 16)) +
         (lane_value_f64(v, 32) + lane_value_f64(v, 48));
}

}  // namespace alg64
}  // namespace lrqk
