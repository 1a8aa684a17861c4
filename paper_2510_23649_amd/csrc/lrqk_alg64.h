// Small dense algebra in fp64 inside one workgroup (gfx950): symmetric positive definite systems
// of up to 64 x 64 elements as 16 x 16 tiles in registers, eliminated tile by tile, a product of two
// tiles being four v_mfma_f64_16x16x4.  fp64 instructions issue at the rate of
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

// 1 / x: the hardware estimate and two Newton steps, to the last bit or two (an IEEE division would
// lengthen the chain of every elimination step).
__device__ __forceinline__ double recip(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
  return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
}

// Element (i, k) of the factor N by which a step of Gauss-Jordan elimination inside a tile
// multiplies the four pivot rows before it adds them to every row: -C D^-1, and D^-1 for the pivot
// rows themselves, which start again from zero.  (With D^-1 - I for them, added to what they held, the
// rows lose as many digits as D is larger than 1.)  In LDS, [4][16] each: D, the pivot rows from the
// pivot columns on, and C, -C^T with the columns of the pivot rows replaced by those of the identity.
__device__ __forceinline__ double pivot_factor(const double* D, const double* C, int i, int k) {
  const double d00 = D[0], d01 = D[1], d02 = D[2], d03 = D[3], d11 = D[17], d12 = D[18],
               d13 = D[19], d22 = D[34], d23 = D[35], d33 = D[51];
  const double c0 = C[i], c1 = C[16 + i], c2 = C[32 + i], c3 = C[48 + i];
  // D = [E F; F^T L] in 2 x 2 blocks, W = E^-1 F, T = (L - F^T W)^-1
  const double ie = recip(d00 * d11 - d01 * d01);
  const double e00 = d11 * ie, e01 = -d01 * ie, e11 = d00 * ie;
  const double w00 = e00 * d02 + e01 * d12, w01 = e00 * d03 + e01 * d13;
  const double w10 = e01 * d02 + e11 * d12, w11 = e01 * d03 + e11 * d13;
  const double l00 = d22 - (d02 * w00 + d12 * w10), l01 = d23 - (d02 * w01 + d12 * w11);
  const double l11 = d33 - (d03 * w01 + d13 * w11);
  const double il = recip(l00 * l11 - l01 * l01);
  // y = D^-1 c: y_b = T (c_b - W^T c_a), y_a = E^-1 c_a - W y_b.  (A lane wants one of the four; y_a in
  // the way of y_b, with the halves exchanged, would be shorter, but two halves that do not come
  // from one elimination cost 3 digits and more on an ill-conditioned tile.)
  const double g0 = (c2 - (w00 * c0 + w10 * c1)) * il, g1 = (c3 - (w01 * c0 + w11 * c1)) * il;
  const double y2 = l11 * g0 - l01 * g1, y3 = l00 * g1 - l01 * g0;
  const double y0 = (e00 * c0 + e01 * c1) - (w00 * y2 + w01 * y3);
  const double y1 = (e01 * c0 + e11 * c1) - (w10 * y2 + w11 * y3);
  const double lo = k & 1 ? y1 : y0, hi = k & 1 ? y3 : y2;
  return k & 2 ? hi : lo;
}

// One step of in-place Gauss-Jordan elimination inside a 16 x 16 tile by one wavefront, the pivots rows
// 4 q .. 4 q + 3 (a step's pivot columns start again as columns of the identity); returns the operand N_q by
// which the pivot rows are multiplied.  The rows and columns up to the last pivot are symmetric positive
// definite to begin with: the pivot columns are taken from the pivot rows, with the sign turned for rows
// that have been pivots before.  P: 128 doubles of LDS that no other wavefront touches meanwhile; the LDS
// operations of a wavefront keep their order, so nothing is waited for but the data.
__device__ __forceinline__ double pivot_step(f64x4& d, int q, double* P, int lane) {
  const int k = lane >> 4, c16 = lane & 15, cq = c16 >> 2;
  const double x = cq == q ? (k == (lane & 3) ? 1.0 : 0.0) : d[q];
  P[lane] = d[q];
  P[64 + lane] = cq > q ? -x : x;
  __builtin_amdgcn_wave_barrier();
  const double n = pivot_factor(P + 4 * q, P + 64, c16, k);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int v = 0; v < 4; ++v) d[v] = v == q || cq == q ? 0.0 : d[v];
  d = mfma_f64(n, x, d);
  return n;
}
// The operands of all four steps.
__device__ __forceinline__ f64x4 pivot_tile(f64x4 d, double* P, int lane) {
  f64x4 n;
#pragma unroll
  for (int q = 0; q < 4; ++q) n[q] = pivot_step(d, q, P, lane);
  return n;
}

// [A | Y] -> [A^-1 | A^-1 Y] in place by Gauss-Jordan elimination with 4 x 4 pivot blocks, A of RT x RT
// tiles, symmetric positive definite (no pivoting needed), Y of RT x (NT - RT) tiles; a wavefront owns
// tiles of tile row tr (tr >= RT: none, it only passes the barriers), those of A that lie in columns tc0,
// tc0 + STEP, ... < RT first and then those of Y in columns RT + tc0, RT + tc0 + STEP, ...  Where INV is
// false A's tiles are left undefined.
// The four pivot blocks of a tile are taken together: its owner finds the four operands N_q and leaves them
// in LDS; the owners of that row's tiles take the four steps, P_q = rows 4 q .. 4 q + 3 of a tile before step
// q being a register of theirs, and W_q = D_q^-1 P_q the same register after it, and leave both in LDS;
// every other row i then adds N_iq P_q, N_iq = -C_iq D_q^-1, where C_iq, the pivot column, is P_q^T of tile
// i of the pivot row, with the sign turned if i has been the pivot before: register W_q of that tile is,
// but for the sign, the operand N_iq as it stands.  The next pivot tile comes first there, so that its
// operands are found during the other products.
// What a step of 16 pivots waits for are four 4 x 4 inversions in one wavefront (2260 cycles), the MFMAs
// of a tile row (64 cycles each, four a tile) and two barriers.  With an exchange and a barrier for every
// 4 pivots all wavefronts made the 4 x 4 inverse, 0.5 us for 4 pivots at r = 32, 0.8 us at r = 64, most
// of it the issue of those fp64 operations.  (The inverse of the whole pivot tile times the others would be
// shorter still, but on ill-conditioned systems it loses two to three digits against 4 x 4 blocks: 3e-6
// instead of 6e-9 for random systems of condition 1e8 at r = 32.)
// The tile row is a template parameter, and what depends on the column is a selection: with branches
// around the products the compiler copies every tile at every join.
// LDS: sweep_doubles<RT, NT>() at `lds`, free from the next barrier on.
template <int RT, int NT>
constexpr int sweep_doubles() {
  return (NT + RT + 1) * 256 + 128;
}
template <int RT, int STEP>
__device__ __forceinline__ int tile_column(int tc0, int u) {
  constexpr int kSys = (RT + STEP - 1) / STEP;  // tiles of A (what lies beyond RT does not exist)
  return u < kSys ? tc0 + STEP * u : RT + tc0 + STEP * (u - kSys);
}
template <int TR, int RT, int NT, int TPW, int STEP, bool INV>
__device__ __forceinline__ void sweep_row(f64x4 (&d)[TPW], int tc0, double* lds, int lane) {
  double* const P = lds + lane;       // [NT][4][64]
  double* const W = P + NT * 256;     // [RT][4][64]
  double* const N = W + RT * 256;     // [4][64]
  const int cq = (lane & 15) >> 2;
  const double unit = lane >> 4 == (lane & 3) ? 1.0 : 0.0;
  // the operands of pivot tile TR, in d[kOwn] of the wavefront with tc0 == own0
  constexpr int kSys = NT == RT ? TPW : (RT + STEP - 1) / STEP;
  constexpr int kOwn = NT == RT ? TR % TPW : TR / STEP, own0 = TR - STEP * kOwn;
  auto find_operands = [&]() {
    if (tc0 == own0) {
      const f64x4 n = pivot_tile(d[kOwn], lds + (NT + RT + 1) * 256, lane);
#pragma unroll
      for (int q = 0; q < 4; ++q) N[q * 64] = n[q];
    }
  };
  if (TR == 0) find_operands();
#pragma unroll
  for (int pt = 0; pt < RT; ++pt) {
    f64x4 n;
    lds_barrier();
    if (TR == pt) {
#pragma unroll
      for (int q = 0; q < 4; ++q) n[q] = N[q * 64];
#pragma unroll
      for (int q = 0; q <= 4; ++q)
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
          if (!INV && RT == 1 && u < kSys) continue;
          const int tc = NT == RT ? tc0 + u : tile_column<RT, STEP>(tc0, u);
          const bool exists = u >= kSys || tc < RT;
          // (W a step later than its product, so that nothing waits for one)
          if (RT > 1 && u < kSys && q > 0 && exists) W[(tc * 4 + q - 1) * 64] = d[u][q - 1];
          if (q == 4) continue;
          double x = d[u][q], p = x;
          d[u][q] = 0.0;
          if (u < kSys && STEP * u <= pt) {  // may be the pivot tile
            const bool pivot = tc == pt, columns = pivot && cq == q;
            x = columns ? unit : x;
            p = pivot && cq > q ? 0.0 : x;  // columns that are pivots only later
#pragma unroll
            for (int v = 0; v < 4; ++v) d[u][v] = columns ? 0.0 : d[u][v];
          }
          if (RT > 1 && exists) P[(tc * 4 + q) * 64] = p;
          d[u] = mfma_f64(n[q], x, d[u]);
        }
    }
    if (RT == 1) break;
    lds_barrier();
    if (TR != pt) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double w = W[(TR * 4 + q) * 64];
        n[q] = TR < pt ? w : -w;
      }
      auto add = [&](int u) {
        const int tc = NT == RT ? tc0 + u : tile_column<RT, STEP>(tc0, u);
        if (u < kSys && STEP * u <= pt) {
#pragma unroll
          for (int v = 0; v < 4; ++v) d[u][v] = tc == pt ? 0.0 : d[u][v];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          d[u] = mfma_f64(n[q], P[(tc * 4 + q) * 64], d[u]);  // (tc < NT)
      };
      if (TR == pt + 1) {
        add(kOwn);
        find_operands();
      }
#pragma unroll
      for (int u = 0; u < TPW; ++u) {
        if (TR == pt + 1 && u == kOwn) continue;
        if (!INV && TR < pt && u < kSys) continue;  // nothing reads it any more
        add(u);
      }
    }
  }
}
template <int RT, int NT, int TPW, int STEP, bool INV>
__device__ __forceinline__ void sweep_tiles(f64x4 (&d)[TPW], int tr, int tc0, double* lds, int lane) {
  if (tr == 0) {
    sweep_row<0, RT, NT, TPW, STEP, INV>(d, tc0, lds, lane);
  } else if (RT > 1 && tr == 1) {
    sweep_row<1, RT, NT, TPW, STEP, INV>(d, tc0, lds, lane);
  } else if (RT > 2 && tr == 2) {
    sweep_row<2, RT, NT, TPW, STEP, INV>(d, tc0, lds, lane);
  } else if (RT > 2 && tr == 3) {
    sweep_row<3, RT, NT, TPW, STEP, INV>(d, tc0, lds, lane);
  } else {
    for (int i = 0; i < 2 * RT; ++i) lds_barrier();
  }
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
