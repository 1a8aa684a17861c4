// p1 -- prefill factorisation (Alg. 1; Sec. 4.1 "Prefill": the four update rules; App. A.1).
//
// With X = Y M (Y = Q or K of a head, M the d x r operand of an update), the sums that the next
// update needs are  X^T Y = M^T (Y^T Y)  and  X^T X = M^T (Y^T Y) M:  once the d x d matrix
// G = Y^T Y of a head is known, every round but for its last products is r x d algebra.  So Q
// and K are read twice, whatever the number of rounds:
//
//   1. prefill_reduce_kernel   G = Y^T Y,  S = A0^T Y,  H = A0^T A0  of every head (A0 = the
//                              initial A_Q, A_K), one partial per chunk of rows
//   2. prefill_sum_kernel      adds the chunk partials in order, in fp64
//   3. n_iter times            B_K = H_K^-1 S_K, M_K, and S_K, H_K of A_K = K M_K
//      (prefill_round_k)       and, in other workgroups, B_Q = H_Q^-1 S_Q;
//      (prefill_round_q)       M_Q, and S_Q, H_Q of A_Q = Q M_Q unless it is the last round
//      (prefill_group_kernel   before them at r = 64: sums over the query heads of a KV group)
//   4. prefill_apply_kernel    A_K = K M_K, A_Q = Q M_Q
//
// (With a pass over Q and K in every update, X^T Y and X^T X from the fp32 matrix cores and the
// solves in fp32, the whole took 2.35 ms at 32 + 8 heads, l = 131072, r = 32, bf16, two rounds;
// now 0.94 ms.)
//
// Precision.  The long products run on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16) with
// every fp32 operand split into three bf16 terms, x = x0 + x1 + x2, 8 bits of significand each, and
// the products x_i y_j with i + j <= 2, accumulated in fp32: what is left out is at most about 2^-24
// of a product, 2^-27 in the mean square.  bf16 rows are one term.  G is better than that (below).
// The r x d algebra is fp64.  Distance from the factors computed in 64 bits, |.|_2, worst of the four,
// on near-rank-r data, in brackets with sums over A_Q and A_K in fp32: 7e-6 (3e-4) at l = 131072,
// r = 32; 2.4e-6 (1.2e-4) at l = 4096, r = 16; 5e-6 (1.5e-4) at l = 30011, r = 64.
#include <type_traits>
#include <utility>

#include "lrqk_alg64.h"
#include "lrqk_internal.h"

namespace lrqk {
namespace {

using namespace alg64;

using dev::bf16x8;
using dev::f32x16;
using dev::mfma_bf16;
using dev::mfma_row;
using dev::pack_bf16;
using dev::split3;
using dev::u32x4;

// split3 for bf16 numbers, which two terms give exactly
__device__ __forceinline__ void split2(float x0, float x1, float grid, uint32_t& hi, uint32_t& lo) {
  const float g0 = (x0 + grid) - grid, g1 = (x1 + grid) - grid;
  hi = pack_bf16(g0, g1);
  lo = pack_bf16(x0 - g0, x1 - g1);
}

constexpr int kPfThreads = 256;

template <int R>
struct PfShape {
  static constexpr int RB = (R + 31) / 32;  // 32-wide blocks of the rank dimension
  static constexpr int RP = 32 * RB;        // rank padded to the MFMA block
  // 32 x 32 blocks of a chunk's partial, each as 16 registers x 64 lanes: 10 of G (the upper
  // ones) in fp64, then 4 RB of S and HB of H in fp32
  static constexpr int GB = 10, HB = RB == 1 ? 4 : 8;
  static constexpr int HB0 = 4 * RB, FB = HB0 + HB;                         // fp32 blocks
  static constexpr size_t part_bytes = (size_t)(GB * 8 + FB * 4) * 1024;
  static constexpr size_t mpack_units = (size_t)3 * RB * 8 * 64;  // 16-byte units of M per head
};

// ------------------------------------------------------------------------------------------
// Reduce.  A workgroup (8 wavefronts) walks a chunk of rows in tiles of 64, two in LDS in turn.
//
// G has to be better than fp32.  H of the next X is M^T G M and where Y is strong in directions that
// M suppresses, the rounding of G enters as |M|^2 |Y|^2 while H itself is only |X|^2 large (a sum over
// X proper, which a pass over Y per update would give, loses |M| |Y| |X|).  So every element is split
// on a grid of its column: y = y0 + y1 (+ y2 for fp32 rows), y0 the nearest multiple of a power of
// two q, about 2^-5 of the column's typical size, y1 and y2 the rest.  Products y0 y0' are whole
// multiples of q q' of some 12 bits, so that fp32 accumulators add up 512 rows of them WITHOUT
// rounding; what is rounded are the products with y1, a hundred times smaller.  (Where a column's
// sizes vary too much for that, the sums round as any fp32 sum: nothing depends on the grid but the
// last bits.)  bf16 rows: y1 is exact, and y0 y1' + y1 y' with the whole y' makes three products;
// fp32 rows: all but y2 y2'.  Every 512 rows the accumulators go to fp64.
// One fp32 accumulation of y y' instead left the factors 2 to 20 times further from their 64-bit
// values than sums over X in fp32, for keys with a mean of 30 sigma or queries and keys whose
// spectra lie 1000 : 1 apart; now they are nearer (tests: test_prefill_strong_directions).
//
// The products contract over the rows while the rows are what is contiguous in memory: a thread
// takes eight rows of two columns, which makes whole operands (8 rows of a column, 16 bytes).
// Wavefront c < 4 owns the blocks (c, c), (c, c + 1) of G (indices modulo 4); wavefront 4 + c
// column block c of S and, c < 2, block (c, c + 2) of G.  With A0 = a0 + a1 + a2,
// H = D + U + U^T, D = a0^T a0 + a1^T a1, U = a0^T a1 + a0^T a2: r <= 32: wavefront 6 does D, 7 U;
// r = 64: wavefronts 4, 5 the diagonal blocks of U, 6, 7 those of D and block (0, 1) of H.
// a1^T a1 has accumulators of its own: its diagonal is a sum of squares 2^-18 the size of the
// main term's, and each addend would round away against that sum (H 2e-6 too small after 11000
// rows).
// 2.0 GB in 0.58 ms at 32 + 8 heads, l = 131072, r = 32 (0.43 ms with y y' alone), 0.29 ms (0.22) at
// 2 x (28 + 4) heads, l = 30011, r = 64: 48 MFMAs of 32 cycles per SIMD and tile are 0.26 ms at the
// 1.9 GHz that this load runs at, everything but the loads 0.46 ms.  Operands read with
// ds_read_b64_tr_b16 from row-major tiles, two tiles of loads in flight, or products reordered
// measured the same.  256 registers a wavefront hold one workgroup on a CU: the LDS takes two tiles.
constexpr int kRedThreads = 512;
constexpr int kBufferFlags = 0x00027000;  // raw 32-bit buffer
constexpr int kNt = 2;                    // non-temporal: A0 is read once, and leaves the caches to Y
constexpr int kFlushRows = 256;  // of S and H; twice as many of G
constexpr int kScaleRows = 32;   // rows from which the grids of a head's columns are taken
template <int R, int NS>
struct PfReduce {
  static constexpr int NP = 3;              // planes of Y: y0, y1 and y (bf16 rows) or y2
  static constexpr int TR = 64;             // rows per tile
  static constexpr int kRows = 2 * TR;      // ... and pass of the loop
  static constexpr int kYPlane = TR * 256;  // bytes
  static constexpr int kAPlane = TR * 2 * PfShape<R>::RP;
  static constexpr int kTile = NP * kYPlane + 3 * kAPlane;
  static constexpr size_t lds_bytes = 2 * (size_t)kTile;
  static constexpr int kFlushTiles = kFlushRows / TR;
  // S and H beyond kFlushRows rows in fp64, not fp32: where there are registers for it (r = 8 and 16 would
  // spill 38 of them, 446 -> 471 us for the whole call at l = 65536, r = 16; r = 64 spills as it is).
  static constexpr bool kWideSums = R == 32;
};

template <int R, int NS>
__global__ __launch_bounds__(kRedThreads, 2) void prefill_reduce_kernel(
    const void* __restrict__ Q, const void* __restrict__ K, const float* __restrict__ A_Q,
    const float* __restrict__ A_K, void* __restrict__ part, int BHq, int l, int lk, int nchunk,
    int units_per_chunk) {
  using S = PfShape<R>;
  using T = PfReduce<R, NS>;
  constexpr int RB = S::RB, TR = T::TR, NP = T::NP;
  constexpr int YB = NS == 1 ? 256 : 512;                           // bytes of a row of Y
  constexpr int NA = (TR / 4 * R + kRedThreads - 1) / kRedThreads;  // pieces of A0 per thread
  extern __shared__ __align__(16) unsigned char pf_lds[];
  __shared__ uint32_t exps[kD];

  const int bh = blockIdx.x / nchunk, chunk = blockIdx.x - bh * nchunk;  // Q heads, then K heads
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int cb = w & 3;        // column block
  const bool sums = w >= 4;    // S and what shares its wavefronts, or G
  const bool isq = bh < BHq;
  const size_t head = isq ? bh : bh - BHq;
  const char* __restrict__ Yh = static_cast<const char*>(isq ? Q : K) + head * (size_t)l * YB;
  const float* __restrict__ Ah = isq ? A_Q + head * (size_t)l * R : A_K + head * (size_t)lk * R;
  const int row_begin = chunk * T::kRows * units_per_chunk;
  const int row_end = min(l, row_begin + T::kRows * units_per_chunk);

  if (S::RP > R) {  // padding columns of A0 stay zero
    for (int i = t; i < 2 * 3 * T::kAPlane / 16; i += kRedThreads)
      reinterpret_cast<uint4*>(pf_lds + NP * T::kYPlane +
                               (i < 3 * T::kAPlane / 16 ? 0 : NP * T::kYPlane))[i] =
          make_uint4(0u, 0u, 0u, 0u);
  }

  // On its way through registers: rows 8 w .. 8 w + 7 of the thread's two columns of Y, and rows
  // 4 g .. 4 g + 3 of a column of A0, g = q / R, q = t + 512 j.  A tile is contiguous in memory; rows
  // past the end of the chunk are outside the buffers that the loads go through and come as zeros.
  struct Pieces {
    uint32_t y[8][NS == 1 ? 1 : 2];
    uint32_t a[NA][4];
  };
  Pieces next;
  auto fetch = [&](int row0) {
    Pieces& p = next;
    const int rows = __builtin_amdgcn_readfirstlane(max(0, min(TR, row_end - row0)));
    const auto yb = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(Yh + (size_t)row0 * YB), 0, rows * YB, kBufferFlags);
    const auto ab = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float*>(Ah + (size_t)row0 * R), 0, rows * R * 4, kBufferFlags);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if constexpr (NS == 1) {
        p.y[i][0] = __builtin_amdgcn_raw_buffer_load_b32(yb, (8 * w + i) * YB + 4 * lane, 0, 0);
      } else {
        const uint2 v = __builtin_bit_cast(
            uint2, __builtin_amdgcn_raw_buffer_load_b64(yb, (8 * w + i) * YB + 8 * lane, 0, 0));
        p.y[i][0] = v.x;
        p.y[i][NS == 1 ? 0 : 1] = v.y;
      }
    }
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q = t + kRedThreads * j;
        p.a[j][i] = __builtin_amdgcn_raw_buffer_load_b32(ab, (q / R * 4 + i) * R * 4 + q % R * 4, 0, kNt);
      }
  };
  // The grids of this thread's columns: q = 2^-5 times the mean binary exponent of kScaleRows rows
  // spread over the head.  (y + grid) - grid is y rounded to a multiple of q.
  float grid[2];
  {
    uint32_t sc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const char* row = Yh + (size_t)((long)l * (4 * w + i) / kScaleRows) * YB;
      if constexpr (NS == 1) {
        const uint32_t v = reinterpret_cast<const uint32_t*>(row)[lane];
        sc[i][0] = v << 16;
        sc[i][1] = v;
      } else {
        const uint2 v = reinterpret_cast<const uint2*>(row)[lane];
        sc[i][0] = v.x;
        sc[i][1] = v.y;
      }
    }
    fetch(row_begin);
    if (t < kD) exps[t] = 0u;
    lds_barrier();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      uint32_t sum = 0u;  // of the exponents of numbers that are not zero, and 2^16 times how many
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t e = (sc[i][c] >> 23) & 255u;
        sum += e > 0u ? 0x10000u + e : 0u;
      }
      atomicAdd(&exps[2 * lane + c], sum);
    }
    lds_barrier();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int sum = exps[2 * lane + c] & 0xffff, n = exps[2 * lane + c] >> 16;
      const int e = n > 0 ? (sum + n / 2) / n - 5 + 23 : 0;
      grid[c] = n > 0 ? __uint_as_float((uint32_t)min(e, 254) << 23 | 0x400000u) : 0.0f;
    }
  }

  // A tile in LDS, plane by plane: unit (8 rows r, column c) of 16 bytes is one lane's part of an
  // operand, the columns of a block of 32 in the order 0, 2 .. 30, 1, 3 .. 31 (column_of), so that
  // both the stores and the reads of a wavefront are contiguous.
  const unsigned char* const yl = pf_lds + ((lane >> 5) * kD + (lane & 31)) * 16;
  const unsigned char* const al = pf_lds + NP * T::kYPlane + ((lane >> 5) * S::RP + (lane & 31)) * 16;
  auto y_op = [&](int half, int plane, int ks, int c) {
    return *reinterpret_cast<const bf16x8*>(yl + half * T::kTile + plane * T::kYPlane +
                                            ks * (2 * kD * 16) + c * 512);
  };
  auto a_op = [&](int half, int plane, int ks, int rb) {
    return *reinterpret_cast<const bf16x8*>(al + half * T::kTile + plane * T::kAPlane +
                                            ks * (2 * S::RP * 16) + rb * 512);
  };
  auto put_y = [&](int half, int c) {  // column c of the thread's two
    const Pieces& p = next;
    uint32_t s[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (NS == 1) {
        const uint32_t v0 = p.y[2 * i][0], v1 = p.y[2 * i + 1][0];
        s[2][i] = c == 0 ? (v0 & 0xffffu) | (v1 << 16) : (v0 >> 16) | (v1 & 0xffff0000u);
        const float x0 = __uint_as_float(c == 0 ? v0 << 16 : v0 & 0xffff0000u);
        const float x1 = __uint_as_float(c == 0 ? v1 << 16 : v1 & 0xffff0000u);
        split2(x0, x1, grid[c], s[0][i], s[1][i]);
      } else {
        uint32_t x[3];
        split3(__uint_as_float(p.y[2 * i][NS == 1 ? 0 : c]),
               __uint_as_float(p.y[2 * i + 1][NS == 1 ? 0 : c]), x, grid[c]);
#pragma unroll
        for (int k = 0; k < 3; ++k) s[k][i] = x[k];
      }
    }
    unsigned char* const to =
        pf_lds + half * T::kTile + (w * kD + 32 * (lane >> 4) + (lane & 15) + 16 * c) * 16;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      *reinterpret_cast<uint4*>(to + k * T::kYPlane) = make_uint4(s[k][0], s[k][1], s[k][2], s[k][3]);
  };
  auto put_a = [&](int half, int j) {
    const Pieces& p = next;
    const int q = t + kRedThreads * j, g = q / R;
    if (TR / 4 * R % kRedThreads != 0 && q >= TR / 4 * R) return;
    uint32_t s0[3], s1[3];
    split3(__uint_as_float(p.a[j][0]), __uint_as_float(p.a[j][1]), s0);
    split3(__uint_as_float(p.a[j][2]), __uint_as_float(p.a[j][3]), s1);
    unsigned char* const to =
        pf_lds + half * T::kTile + NP * T::kYPlane + ((g >> 1) * S::RP + q % R) * 16 + 8 * (g & 1);
#pragma unroll
    for (int k = 0; k < 3; ++k)
      *reinterpret_cast<uint2*>(to + k * T::kAPlane) = make_uint2(s0[k], s1[k]);
  };
  put_y(0, 0);
  put_y(0, 1);
#pragma unroll
  for (int j = 0; j < NA; ++j) put_a(0, j);
  fetch(row_begin + TR);
  lds_barrier();

  // One barrier per tile: a wavefront that stores a tile while others still read the one before
  // writes the other half of the LDS.  The walk is compiled once for each role of a
  // wavefront (0: G; 1, 2, 3: S with what column blocks 0 and 1, 2, 3 add to it): with the roles
  // as branches around the products the accumulators were copied at every step (0.76 ms instead
  // of 0.40 ms at l = 131072, r = 32, 32 + 8 heads).  Every role passes the same barriers.
  auto walk = [&](auto role) {
    constexpr int ROLE = decltype(role)::value;
    constexpr int NG = ROLE == 0 ? 2 : ROLE == 1 ? 1 : 0;   // blocks of G
    constexpr int NACC = ROLE == 0 ? 0 : ROLE == 1 ? RB + RB - 1 : RB + 1 + RB;  // S, parts of H
    constexpr int NFL = ROLE == 0 ? 0 : ROLE == 1 ? NACC : 2 * RB;               // flushed ones
    double g[NG + 1][16];
    f32x16 ghi[NG + 1], glo[NG + 1], acc[NACC + 1];
    std::conditional_t<T::kWideSums, double, float> acc2[NFL + 1][16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        g[i][v] = 0.0;
        ghi[i][v] = glo[i][v] = 0.0f;
      }
#pragma unroll
      for (int i = 0; i < NACC; ++i) acc[i][v] = 0.0f;
#pragma unroll
      for (int i = 0; i < NFL; ++i) acc2[i][v] = 0;
    }
    // From time to time the accumulators of G go to fp64 ones, those of S, D and the off-diagonal
    // products of H to second ones, of fp32 or fp64 (kWideSums): rounding errors follow the size of the sum that they are
    // made in, however many rows a chunk has, and the second round's factors amplify those of S.
    // (The second-order parts of H and, at r <= 32, a0^T a2 may stay: they are 2^-17 of it.)
    auto flush_sums = [&]() {
#pragma unroll
      for (int i = 0; i < NFL; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          acc2[i][v] += acc[i][v];
          acc[i][v] = 0.0f;
        }
    };
    auto flush_gram = [&]() {
#pragma unroll
      for (int i = 0; i < NG; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          g[i][v] += (double)ghi[i][v] + (double)glo[i][v];
          ghi[i][v] = glo[i][v] = 0.0f;
        }
    };

    // The operands of 16 rows, and their products.
    struct Ops {
      bf16x8 y[NP], z[NP], a[RB][3];
    };
    auto load = [&](int half, int ks) {
      Ops o;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        if (ROLE <= 1 || NS > 1 || p == 2) o.y[p] = y_op(half, p, ks, cb);
        if (ROLE <= 1) o.z[p] = y_op(half, p, ks, (cb + (ROLE == 0 ? 1 : 2)) & 3);
        if (ROLE > 0) {
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) o.a[rb][p] = a_op(half, p, ks, rb);
        }
      }
      return o;
    };
    auto multiply = [&](const Ops& o) {
      if constexpr (ROLE <= 1) {  // blocks of G: the leading products, and the small ones
        if constexpr (ROLE == 0) ghi[0] = mfma_bf16(o.y[0], o.y[0], ghi[0]);
        ghi[NG - 1] = mfma_bf16(o.y[0], o.z[0], ghi[NG - 1]);
#pragma unroll
        for (int i = 0; i < NP; ++i)
#pragma unroll
          for (int j = 0; j < NP; ++j)
            if (NS == 1 ? (i == 0 && j == 1) || (i == 1 && j == 2) : i + j > 0 && i + j < 4) {
              if constexpr (ROLE == 0) glo[0] = mfma_bf16(o.y[i], o.y[j], glo[0]);
              glo[NG - 1] = mfma_bf16(o.y[i], o.z[j], glo[NG - 1]);
            }
      }
      if constexpr (ROLE > 0) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int j = 0; j < NP; ++j)
            if (NS == 1 ? j == 2 : i + j < 3) {
#pragma unroll
              for (int rb = 0; rb < RB; ++rb) acc[rb] = mfma_bf16(o.a[rb][i], o.y[j], acc[rb]);
            }
        f32x16& e0 = acc[RB];
        f32x16& e1 = acc[RB == 1 ? NACC - 1 : RB + 1];
        f32x16& e2 = acc[NACC - 1];
        if constexpr (ROLE == 1) {
          if constexpr (RB > 1) {  // U of diagonal block cb
            const auto& b = o.a[0];
            const auto& c = o.a[RB - 1];
            const bf16x8 b0 = cb == 0 ? b[0] : c[0];
            e0 = mfma_bf16(b0, cb == 0 ? b[1] : c[1], e0);
            e0 = mfma_bf16(b0, cb == 0 ? b[2] : c[2], e0);
          }
        } else if constexpr (ROLE == 2) {
          e0 = mfma_bf16(o.a[0][0], o.a[0][0], e0);
          e2 = mfma_bf16(o.a[0][1], o.a[0][1], e2);
          if constexpr (RB > 1) e1 = mfma_bf16(o.a[0][0], o.a[RB - 1][0], e1);
        } else if constexpr (RB == 1) {
          e0 = mfma_bf16(o.a[0][0], o.a[0][1], e0);
          e1 = mfma_bf16(o.a[0][0], o.a[0][2], e1);
        } else {
          constexpr int B1 = RB - 1;
          e1 = mfma_bf16(o.a[0][0], o.a[B1][1], e1);
          e0 = mfma_bf16(o.a[B1][0], o.a[B1][0], e0);
          e1 = mfma_bf16(o.a[0][1], o.a[B1][0], e1);
          e2 = mfma_bf16(o.a[B1][1], o.a[B1][1], e2);
          e1 = mfma_bf16(o.a[0][0], o.a[B1][2], e1);
          e1 = mfma_bf16(o.a[0][2], o.a[B1][0], e1);
          e1 = mfma_bf16(o.a[0][1], o.a[B1][1], e1);
        }
      }
    };
    // One tile's products.  The next tile goes to the other half of the LDS between them, and its
    // registers take the loads of the one after.  r <= 32: a step's operands are read during the
    // step before; the barrier stands before the last step, whose operands every wavefront has by
    // then, so that the next tile's first ones are read behind it.
    constexpr bool kAhead = RB == 1;
    constexpr int kSteps = TR / 16;
    Ops ops;
    if (kAhead) ops = load(0, 0);
    auto body = [&](int row0, int cur) {
#pragma unroll
      for (int ks = 0; ks < kSteps; ++ks) {
        const bool last = ks == kSteps - 1;
        if (kAhead && last) {
          fetch(row0 + 2 * TR);
          lds_barrier();
        }
        const Ops o = kAhead && !last ? load(cur, ks + 1) : kAhead ? load(cur ^ 1, 0) : load(cur, ks);
        if (ks < 2) put_y(cur ^ 1, ks);
        if (ks >= 2 && ks - 2 < NA) put_a(cur ^ 1, ks - 2);
        multiply(kAhead ? ops : o);
        if (kAhead) ops = o;
      }
      if (!kAhead) {
        fetch(row0 + 2 * TR);
        lds_barrier();
      }
    };
    // (the second of a pass's two tiles is empty where the rows have run out)
    for (int row0 = row_begin, tile = 0; row0 < row_end; row0 += 2 * TR, tile += 2) {
      if (tile % T::kFlushTiles == 0) flush_sums();
      if (tile % (2 * T::kFlushTiles) == 0) flush_gram();
      body(row0, 0);
      body(row0 + TR, 1);
    }

    flush_sums();
    flush_gram();
    double* const gout =
        reinterpret_cast<double*>(reinterpret_cast<char*>(part) + blockIdx.x * S::part_bytes) + lane;
    float* const out = reinterpret_cast<float*>(gout - lane + S::GB * 1024) + lane;
    auto put_g = [&](int block, const double (&x)[16]) {
#pragma unroll
      for (int v = 0; v < 16; ++v) gout[block * 1024 + v * 64] = x[v];
    };
    auto put = [&](int block, const auto& x) {
#pragma unroll
      for (int v = 0; v < 16; ++v) out[block * 1024 + v * 64] = (float)x[v];
    };
    if constexpr (ROLE == 0) {
      put_g(cb, g[0]);
      put_g(4 + cb, g[1]);
    } else {
      if constexpr (ROLE == 1) put_g(8 + cb, g[0]);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) put(4 * rb + cb, acc2[rb]);
      if constexpr (ROLE == 1) {
        if constexpr (RB > 1) put(S::HB0 + 2 + cb, acc2[RB]);
      } else {
        put(S::HB0 + cb - 2, acc2[RB]);
        if constexpr (RB > 1) put(S::HB0 + 2 + cb, acc2[RB + 1]);
        put(S::FB - 4 + cb, acc[NACC - 1]);
      }
    }
  };
  if (!sums)
    walk(std::integral_constant<int, 0>{});
  else if (cb < 2)
    walk(std::integral_constant<int, 1>{});
  else if (cb == 2)
    walk(std::integral_constant<int, 2>{});
  else
    walk(std::integral_constant<int, 3>{});
}

// The column of Y that stands at place i of a block of 32.
__device__ __forceinline__ int column_of(int i) { return 2 * (i & 15) + (i >> 4); }

// Place of element (i, j) of a 32 x 32 block among its 16 x 64 accumulator values.
__device__ __forceinline__ int acc_index(int i, int j) {
  return (4 * (i >> 3) + (i & 3)) * 64 + 32 * ((i >> 2) & 1) + j;
}

// The chunk partials of a head added in chunk order, in fp64: G [d][d], S [r][d], H [r][r] (the first of ADD
// addends, the others zero).
template <int R, int ADD>
__global__ __launch_bounds__(256) void prefill_sum_kernel(const void* __restrict__ part,
                                                          double* __restrict__ G,
                                                          double* __restrict__ Sm,
                                                          double* __restrict__ H, int nchunk) {
  using S = PfShape<R>;
  constexpr int kBlocks = ((S::GB + S::HB0) * 1024 + R * R + 255) / 256;  // workgroups per head
  // A head's sum and its solves on one die: what one launch writes the next reads from that die's L2
  // (the whole call, 32 + 8 heads, bf16: 79.6 -> 77.4 us at l = 4096, r = 16; 177.9 -> 175.4 at
  // l = 16384, r = 32; 2 x (28 + 4) heads, l = 30011, r = 64: 593.9 -> 589.9).  With the chunks' partials
  // on it as well nothing more is gained (77.6, 174.5, 594.0): they come from every die's share of Q and K.
  int at, block;
  dev::place(blockIdx.x, gridDim.x / kBlocks, kBlocks, at, block);
  const size_t head = at;
  int e = block * 256 + threadIdx.x;
  const char* p = static_cast<const char*>(part) + head * nchunk * S::part_bytes;
  auto total = [&](const auto* q) {  // q: the element in the first chunk's partial
    double acc = 0.0;
    constexpr size_t stride = S::part_bytes / sizeof(*q);
    for (int c0 = 0; c0 < nchunk; c0 += 8) {  // (eight loads in flight, those past the end unused)
      std::remove_cv_t<std::remove_reference_t<decltype(*q)>> v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = q[(size_t)min(c0 + j, nchunk - 1) * stride];
#pragma unroll
      for (int j = 0; j < 8; ++j) acc += c0 + j < nchunk ? (double)v[j] : 0.0;
    }
    return acc;
  };
  auto place = [](int e, int& row, int& col) {
    row = mfma_row((e >> 6) & 15, e & 63);
    col = column_of(e & 31);
  };
  int row, col;
  if (e < S::GB * 1024) {
    place(e, row, col);
    row = column_of(row);
    const int bi = (e >> 10) & 3, bj = (bi + (e >> 12)) & 3;
    // The diagonal blocks are symmetric but for the rounding of the small products, 1e-9 of them, which
    // the solves, for which a system is symmetric, would not see in the same way as the products
    // with G (B_Q 20 times further off at l = 20000, r = 32): their upper halves count.
    if (bi == bj && row > col) return;
    const double x = total(reinterpret_cast<const double*>(p) + e);
    double* Gh = G + head * kD * kD;
    Gh[(32 * bi + row) * kD + 32 * bj + col] = x;
    Gh[(32 * bj + col) * kD + 32 * bi + row] = x;
    return;
  }
  const float* f = reinterpret_cast<const float*>(p + (size_t)S::GB * 8 * 1024);
  e -= S::GB * 1024;
  if (e < S::HB0 * 1024) {
    place(e, row, col);
    const int i = 32 * (e >> 12) + row, j = 32 * ((e >> 10) & 3) + col;
    if (i < R) Sm[(head * R + i) * kD + j] = total(f + e);
    return;
  }
  const int h = e - S::HB0 * 1024;
  if (h >= R * R) return;
  int i = h / R, j = h % R;
  double x = 0.0;
  auto add = [&](int block, int i, int j) { x += total(f + (S::HB0 + block) * 1024 + acc_index(i, j)); };
  if (S::RB == 1) {
    add(0, i, j);  // D, U, second-order parts of D and U
    add(2, i, j);
    for (int block = 1; block < 4; block += 2) {
      add(block, i, j);
      add(block, j, i);
    }
  } else if (i / 32 == j / 32) {
    const int d = i / 32;  // D, U, second-order part of D
    i &= 31;
    j &= 31;
    add(d, i, j);
    add(6 + d, i, j);
    add(2 + d, i, j);
    add(2 + d, j, i);
  } else {
    const int lo = i < j ? i : j, hi = i < j ? j : i;
    add(4, lo, hi - 32);
    add(5, lo, hi - 32);
  }
  H[head * ADD * R * R + h] = x;
#pragma unroll
  for (int c = 1; c < ADD; ++c) H[(head * ADD + c) * R * R + h] = 0.0;
}

// ------------------------------------------------------------------------------------------
// The r x d algebra of one head in fp64, by a workgroup of 8 wavefronts.
constexpr int kAlgThreads = 512;
constexpr int kLdx = kD + 2;  // LDS row stride: 16 rows x 2 columns fall on 32 different bank pairs

template <int R>
struct PfAlg {
  static constexpr int RT = (R + 15) / 16;  // 16 x 16 tiles: RT x RT of the system,
  static constexpr int NT = RT + kD / 16;   // RT x 8 of the right-hand sides
  static constexpr int WPR = 8 / RT;        // wavefronts per tile row
  static constexpr int SYS = (RT + WPR - 1) / WPR;  // tiles of a wavefront: of the system (some do not
  static constexpr int TPW = SYS + 8 / WPR;         // exist), all of them (tile_column)
  static constexpr int kX = 16 * RT * kLdx;         // doubles of an r x d matrix in LDS
  // Where the chip has compute units to spare four workgroups share the sums S = X G, H = S X^T of a head:
  // RS stretches of tile rows times CS of columns.  H comes in CS addends then, kept side by side.
  static constexpr int RS = RT > 1 ? 2 : 1, CS = 4 / RS;
  static constexpr int kH = CS * R * R;
  static constexpr int kRaw = 4 * (TPW + SYS * (CS - 1));  // doubles of a wavefront's tiles in memory
  // another one, and in its place during a solve the tiles that are exchanged
  static constexpr int kY = sweep_doubles<RT, NT>() > kX ? sweep_doubles<RT, NT>() : kX;
  static constexpr size_t lds_bytes = ((size_t)kX + kY) * sizeof(double);
};

// [A | Y] -> [. | A^-1 Y]; lds: Z::kY doubles, free again when every wavefront has returned.
template <int R>
__device__ __forceinline__ void solve_tiles(f64x4 (&d)[PfAlg<R>::TPW], double* lds, int w, int lane) {
  using Z = PfAlg<R>;
  sweep_tiles<Z::RT, Z::NT, Z::TPW, Z::WPR, false>(d, w / Z::WPR, w % Z::WPR, lds, lane);
}

// The tiles of [H | S] of this wavefront, H [ADD][r][r] and S [r][d] in memory: register v of tile u, for
// the system's tiles of every addend.  Nothing is waited for; rows that do not exist read ones that do.
template <int R, int ADD = PfAlg<R>::CS>
__device__ __forceinline__ void fetch_tiles(double (&x)[PfAlg<R>::kRaw], int w, int lane,
                                            const double* __restrict__ H, const double* __restrict__ S) {
  using Z = PfAlg<R>;
  const int tr = w / Z::WPR, tc0 = w % Z::WPR;
  int n = 0;
#pragma unroll
  for (int u = 0; u < Z::TPW; ++u) {
    const int tc = tile_column<Z::RT, Z::WPR>(tc0, u), j = 16 * tc + (lane & 15);
#pragma unroll
    for (int c = 0; c < (u < Z::SYS ? ADD : 1); ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = min(16 * tr + 4 * v + (lane >> 4), R - 1);
        if (u < Z::SYS)
          x[n++] = tc < Z::RT ? H[c * R * R + i * R + min(j, R - 1)] : 0.0;
        else
          x[n++] = S[i * kD + j - 16 * Z::RT];
      }
  }
}
// d = them, or d += them; `use` false: zeros in their place.
template <int R, int ADD = PfAlg<R>::CS>
__device__ __forceinline__ void take_tiles(f64x4 (&d)[PfAlg<R>::TPW], const double (&x)[PfAlg<R>::kRaw],
                                           bool add, bool use) {
  using Z = PfAlg<R>;
  int n = 0;
#pragma unroll
  for (int u = 0; u < Z::TPW; ++u)
#pragma unroll
    for (int c = 0; c < (u < Z::SYS ? ADD : 1); ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double y = use ? x[n] : 0.0;
        d[u][v] = add || c > 0 ? d[u][v] + y : y;
        ++n;
      }
}
// The padding of a system is the identity, that of its right-hand sides zero.
template <int R>
__device__ __forceinline__ void pad_tiles(f64x4 (&d)[PfAlg<R>::TPW], int w, int lane) {
  using Z = PfAlg<R>;
  if (R % 16 == 0) return;
  const int tr = w / Z::WPR, tc0 = w % Z::WPR;
#pragma unroll
  for (int u = 0; u < Z::TPW; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * tr + 4 * v + (lane >> 4);
      const int j = 16 * tile_column<Z::RT, Z::WPR>(tc0, u) + (lane & 15);
      if (i >= R || (u < Z::SYS && j >= R)) d[u][v] = (u < Z::SYS && i == j) ? 1.0 : 0.0;
    }
}
template <int R>
__device__ __forceinline__ void load_tiles(f64x4 (&d)[PfAlg<R>::TPW], int w, int lane,
                                           const double* __restrict__ H,
                                           const double* __restrict__ S) {
  using Z = PfAlg<R>;
  double x[Z::kRaw];
  fetch_tiles<R>(x, w, lane, H, S);
  take_tiles<R>(d, x, false, true);
  pad_tiles<R>(d, w, lane);
}

// Right-hand-side tiles += lam X, X [r][d] in LDS.
template <int R>
__device__ __forceinline__ void add_rhs(f64x4 (&d)[PfAlg<R>::TPW], const double* X, double lam,
                                        int w, int lane) {
  using Z = PfAlg<R>;
  const int tr = w / Z::WPR, tc0 = w % Z::WPR;
#pragma unroll
  for (int u = Z::SYS; u < Z::TPW; ++u) {
    const int tc = tile_column<Z::RT, Z::WPR>(tc0, u);
#pragma unroll
    for (int v = 0; v < 4; ++v)
      d[u][v] = __builtin_fma(lam, X[(16 * tr + 4 * v + (lane >> 4)) * kLdx + 16 * (tc - Z::RT) +
                                     (lane & 15)], d[u][v]);
  }
}

// The solution part of the tiles: put(i, j, value) for i < r, j < d.
template <int R, typename F>
__device__ __forceinline__ void store_solution(const f64x4 (&d)[PfAlg<R>::TPW], int w, int lane,
                                               F put) {
  using Z = PfAlg<R>;
  const int tr = w / Z::WPR, tc0 = w % Z::WPR;
#pragma unroll
  for (int u = Z::SYS; u < Z::TPW; ++u) {
    const int tc = tile_column<Z::RT, Z::WPR>(tc0, u);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 16 * tr + 4 * v + (lane >> 4);
      if (i < R) put(i, 16 * (tc - Z::RT) + (lane & 15), d[u][v]);
    }
  }
}

// One wavefront's share of A B^T over d, A and B the 16 rows at `a` and `b` in LDS: one of `shares`
// stretches of the sum.
template <int SHARES>
__device__ __forceinline__ f64x4 tile_product(const double* a, const double* b, int share, int lane) {
  constexpr int kLen = kD / SHARES;
  const int at = (lane & 15) * kLdx + (lane >> 4) + share * kLen;
  f64x4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
  for (int s = 0; s < kLen; s += 4) x = mfma_f64(a[at + s], b[at + s], x);
  return x;
}

// System tiles += lam X X^T, X [r][d] in LDS (rows up to the tile size are zero).  Y: LDS scratch.  At
// r <= 32 there are more wavefronts than tiles: several share a tile (a chain of 32 MFMAs of 64 cycles by
// its owner alone would be the longest part of a round at r = 16 after the solves).
template <int R>
__device__ __forceinline__ void add_gram(f64x4 (&d)[PfAlg<R>::TPW], const double* X, double* Y,
                                         double lam, int w, int lane) {
  using Z = PfAlg<R>;
  constexpr int kTiles = Z::RT * Z::RT, kShares = kTiles < 8 ? 8 / kTiles : 1;
  const int tr = w / Z::WPR, tc0 = w % Z::WPR;
  if (kShares > 1) {
    const int tile = w / kShares;
    const f64x4 x = tile_product<kShares>(X + 16 * (tile / Z::RT) * kLdx, X + 16 * (tile % Z::RT) * kLdx,
                                          w % kShares, lane);
#pragma unroll
    for (int v = 0; v < 4; ++v) Y[w * 256 + v * 64 + lane] = x[v];
    lds_barrier();
  }
#pragma unroll
  for (int u = 0; u < Z::SYS; ++u) {
    const int tc = tc0 + Z::WPR * u;
    if (tc >= Z::RT) continue;
    f64x4 x = {0.0, 0.0, 0.0, 0.0};
    if (kShares > 1) {
#pragma unroll
      for (int i = 0; i < kShares; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] += Y[((tr * Z::RT + tc) * kShares + i) * 256 + v * 64 + lane];
    } else {
      x = tile_product<1>(X + 16 * tr * kLdx, X + 16 * tc * kLdx, 0, lane);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) d[u][v] = __builtin_fma(lam, x[v], d[u][v]);
  }
}

// The share of a workgroup in the sums of a head, and of a wavefront in it: columns 16 col .. 16 col + 15
// (with WC wavefronts side by side) and, of the sum over d, steps of 4 from step0 on, 32 / KS of them.
// SHARED: four workgroups, RS x CS; otherwise one.
template <int R, bool SHARED>
struct PfPart {
  using Z = PfAlg<R>;
  static constexpr bool kShared = SHARED;
  static constexpr int RS = SHARED ? Z::RS : 1, CS = SHARED ? Z::CS : 1;
  static constexpr int WC = 8 / CS, KS = CS, kSteps = 32 / KS;
  int row, addend, col, ks;
  __device__ PfPart(int part, int w)
      : row(part % RS), addend(part / RS), col(addend * WC + w % WC), ks(w / WC) {}
};

// Whether these operands (32 doubles a lane in the unshared form) are read after the solve before them
// instead of under it: at r = 64 the solve's tiles leave no registers for them, 88 and 14 of which went to
// memory (8 x (28 + 4) heads, the whole call at l = 2048: 397 -> 395 us, at l = 500: 302.6 -> 299.7).
template <int R, bool SHARED>
constexpr bool kGramLate = R > 32 && !SHARED;
// This wavefront's operands of X G, G [d][d] in memory.
template <class Q>
__device__ __forceinline__ void load_gram(double (&g)[Q::kSteps], const double* __restrict__ G,
                                          const Q& p, int lane) {
  const auto buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(G), 0, kD * kD * 8, kBufferFlags);
  const int first = ((4 * Q::kSteps * p.ks + (lane >> 4)) * kD + 16 * p.col + (lane & 15)) * 8;
#pragma unroll
  for (int s = 0; s < Q::kSteps; ++s)
    g[s] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(buf, first, 4 * s * kD * 8, 0));
}

// This workgroup's part of S = X G and H = S X^T, X [r][d] in LDS: rows and columns of S, and of H the
// addend that these columns make, in these rows.  Ys [r][d]: LDS scratch.
template <int R, class Q>
__device__ __forceinline__ void sums_of(const double* X, double* Ys, const double (&g)[Q::kSteps],
                                        const Q& p, double* __restrict__ Sm,
                                        double* __restrict__ H, int w, int lane) {
  using Z = PfAlg<R>;
  const int c16 = lane & 15, k = lane >> 4, t = w * 64 + lane;
  constexpr int kRows = Z::RT / Q::RS;  // tile rows
#pragma unroll 1
  for (int rr = 0; rr < kRows; ++rr) {
    const double* x = X + (16 * (p.row * kRows + rr) + c16) * kLdx + 4 * Q::kSteps * p.ks + k;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < Q::kSteps; ++s) acc = mfma_f64(x[4 * s], g[s], acc);
    // (stretch ks of the sum in columns 16 WC ks .. of the row)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      Ys[(16 * rr + 4 * v + k) * kLdx + 16 * (Q::WC * p.ks + w % Q::WC) + c16] = acc[v];
  }
  lds_barrier();
  constexpr int kCols = 16 * Q::WC;
  for (int e = t; e < 16 * kRows * kCols; e += kAlgThreads) {
    const int i = e / kCols, j = e % kCols, row = 16 * p.row * kRows + i;
    double x = Ys[i * kLdx + j];
#pragma unroll
    for (int ks = 1; ks < Q::KS; ++ks) x += Ys[i * kLdx + kCols * ks + j];
    if (Q::KS > 1) Ys[i * kLdx + j] = x;
    if (row < R) Sm[row * kD + kCols * p.addend + j] = x;
  }
  if (Q::KS > 1) lds_barrier();
  // H: kRows x RT tiles, each a sum over kCols; where there are fewer tiles than wavefronts several share one
  constexpr int kTiles = kRows * Z::RT, kShares = kTiles < 8 ? 8 / kTiles : 1, kLen = kCols / kShares;
  static_assert(kLen % 4 == 0, "whole steps");
  H += p.addend * R * R;
  f64x4 h[kTiles > 8 ? kTiles / 8 : 1];
#pragma unroll
  for (int n = 0; n < (kTiles > 8 ? kTiles / 8 : 1); ++n) {
    const int tile = w / kShares + 8 * n, share = w % kShares;
    const double* y = Ys + (16 * (tile / Z::RT) + c16) * kLdx + k + kLen * share;
    const double* x = X + (16 * (tile % Z::RT) + c16) * kLdx + kCols * p.addend + k + kLen * share;
    h[n] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int s = 0; s < kLen; s += 4) h[n] = mfma_f64(y[s], x[s], h[n]);
  }
  auto put = [&](int tile, int v, int l, double x) {
    const int i = 16 * (p.row * kRows + tile / Z::RT) + 4 * v + (l >> 4), j = 16 * (tile % Z::RT) + (l & 15);
    if (i >= R || j >= R) return;
    H[i * R + j] = x;
    if (!Q::kShared) {
#pragma unroll
      for (int c = 1; c < Z::CS; ++c) H[c * R * R + i * R + j] = 0.0;
    }
  };
  if (kShares > 1) {
    lds_barrier();  // Ys has been read
#pragma unroll
    for (int v = 0; v < 4; ++v) Ys[w * 256 + v * 64 + lane] = h[0][v];
    lds_barrier();
    for (int e = t; e < kTiles * 256; e += kAlgThreads) {
      double x = 0.0;
#pragma unroll
      for (int i = 0; i < kShares; ++i) x += Ys[((e >> 8) * kShares + i) * 256 + (e & 255)];
      put(e >> 8, (e >> 6) & 3, e & 63, x);
    }
  } else {
#pragma unroll
    for (int n = 0; n < (kTiles > 8 ? kTiles / 8 : 1); ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) put(w + 8 * n, v, lane, h[n][v]);
  }
}

// M (its transpose [r][d] in LDS) as the apply kernel's operands: unit (term, rank block, k step,
// lane) holds M[16 step + 8 (lane / 32) ..][32 block + lane % 32], one of three bf16 terms.
template <int R>
__device__ __forceinline__ void pack_operand(const double* Xt, uint4* __restrict__ pack, int t) {
  constexpr int RB = PfShape<R>::RB;
  for (int e = t; e < RB * 8 * 64; e += kAlgThreads) {
    const int rank = 32 * (e >> 9) + (e & 31), k0 = 16 * ((e >> 6) & 7) + 8 * ((e >> 5) & 1);
    uint32_t s[4][3];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      split3(rank < R ? (float)Xt[rank * kLdx + k0 + 2 * j] : 0.0f,
             rank < R ? (float)Xt[rank * kLdx + k0 + 2 * j + 1] : 0.0f, s[j]);
#pragma unroll
    for (int p = 0; p < 3; ++p)
      pack[p * (RB * 512) + e] = make_uint4(s[0][p], s[1][p], s[2][p], s[3][p]);
  }
}

struct PfState {
  const double* G;             // [BHq + BHkv][d][d]
  double *S, *H;               // [BHq][r][d], [BHq][CS][r][r]: sums of A_Q
  const double *SK, *HK;       // [BHkv][r][d], [BHkv][CS][r][r]: sums of A_K before the round
  double *SK_new, *HK_new;     // ... and after its first half
  double* group;               // [BHkv][r][r + d] (kGroupSums)
  double* BQ;                  // [BHq][r][d]
  uint4* M;                    // [BHq + BHkv] packed operands
  float* B_Q;                  // results
  float* B_K;
  int Hq, Hkv, BHq, BHkv;
  double lam_pQ, lam_pK;
  bool last;  // last round: M is needed, the sums of the new A_Q are not
};

// At r = 64 the sums of a group's query heads, 0.7 to 0.9 MB at G = 7, are added up beforehand by all the
// chip: [H | S] of the group, [r][r] and then [r][d].  One compute unit takes 17 us to read them, this
// launch 4 us; at r = 32 (0.2 MB at G = 4) most of the reading lies under the first solve.
template <int R>
constexpr bool kGroupSums = R > 32;
template <int R>
__global__ __launch_bounds__(256) void prefill_group_kernel(const PfState a) {
  using Z = PfAlg<R>;
  constexpr int kSize = R * (R + kD), kBlocks = kSize / 256;
  static_assert(kSize % 256 == 0 && R * R % 256 == 0, "whole workgroups");
  const int bkv = blockIdx.x / kBlocks, e = (int)(blockIdx.x % kBlocks) * 256 + (int)threadIdx.x;
  const int b = bkv / a.Hkv, G = a.Hq / a.Hkv;
  const size_t q0 = (size_t)b * a.Hq + (size_t)(bkv - b * a.Hkv) * G;
  double x = 0.0;
  if (e < R * R) {
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int c = 0; c < Z::CS; ++c) x += a.H[(q0 + g) * Z::kH + c * R * R + e];
  } else {
#pragma unroll 4
    for (int g = 0; g < G; ++g) x += a.S[(q0 + g) * R * kD + e - R * R];
  }
  a.group[(size_t)bkv * kSize + e] = x;
}

// First half of a round.  Workgroups [0, B Hkv) (4 B Hkv if SHARED), a KV head each:
//   B_K = H_K^-1 S_K,
//   M_K = (sum_g S_Q,g^T + lambda_pK B_K^T)(sum_g H_Q,g + lambda_pK B_K B_K^T)^-1,
//   S_K, H_K of A_K = K M_K.
// The others, a query head each: B_Q = H_Q^-1 S_Q (the next launch reads it).
// SHARED: the workgroups of a head all solve for the same M and share the sums.  G alone is 128 KB, 2 us
// for one compute unit, and its products take a chain of MFMAs nearly as long as a solve at r = 16.
template <int R, bool SHARED>
__global__ __launch_bounds__(kAlgThreads) void prefill_round_k_kernel(const PfState a) {
  using Z = PfAlg<R>;
  extern __shared__ __align__(16) double pf_alg[];
  double* const X = pf_alg;
  double* const Ys = X + Z::kX;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  constexpr int kParts = SHARED ? 4 : 1;
  const bool iskv = (int)blockIdx.x < a.BHkv * kParts;
  int kv_at, kv_part;
  dev::place(blockIdx.x, a.BHkv, kParts, kv_at, kv_part);
  const size_t own = iskv ? kv_at : (int)blockIdx.x - a.BHkv * kParts;
  const int b = (int)own / a.Hkv, kvh = (int)own - b * a.Hkv, G = a.Hq / a.Hkv;
  const size_t q0 = (size_t)b * a.Hq + (size_t)kvh * G;  // a KV head's query heads
  f64x4 d[Z::TPW];
  load_tiles<R>(d, w, lane, (iskv ? a.HK : a.H) + own * Z::kH, (iskv ? a.SK : a.S) + own * R * kD);
  // On its way during the first solve: the sums of the first query heads; during the second: G.
  constexpr int kPre = R <= 16 ? 3 : R <= 32 ? 2 : 1;
  using Part = PfPart<R, SHARED>;
  const int part = iskv ? kv_part : 0;
  const Part share(part, w);
  double pre[kPre][Z::kRaw], gram[Part::kSteps];
  if constexpr (kGroupSums<R>) {
    const double* group = a.group + (iskv ? own : 0) * R * (R + kD);
    fetch_tiles<R, 1>(pre[0], w, lane, group, group + R * R);
  } else {
#pragma unroll
    for (int g = 0; g < kPre; ++g) {
      const size_t head = iskv ? q0 + min(g, G - 1) : own;
      fetch_tiles<R>(pre[g], w, lane, a.H + head * Z::kH, a.S + head * R * kD);
    }
  }
  solve_tiles<R>(d, Ys, w, lane);
  if (!iskv) {
    double* BQ = a.BQ + own * R * kD;
    float* B_Q = a.B_Q + own * R * kD;
    store_solution<R>(d, w, lane, [&](int i, int j, double x) {
      BQ[i * kD + j] = x;
      if (a.last) B_Q[i * kD + j] = (float)x;
    });
    return;
  }
  if (16 * Z::RT > R)
    for (int e = t; e < (16 * Z::RT - R) * kLdx; e += kAlgThreads) X[R * kLdx + e] = 0.0;
  {
    float* B_K = a.B_K + own * R * kD;
    const bool keep = a.last && part == 0;
    store_solution<R>(d, w, lane, [&](int i, int j, double x) {
      X[i * kLdx + j] = x;
      if (keep) B_K[i * kD + j] = (float)x;
    });
  }
  // (the padding of the system is the identity, to which padding of X adds nothing)
  if constexpr (kGroupSums<R>) {
    take_tiles<R, 1>(d, pre[0], false, true);
  } else {
#pragma unroll
    for (int g = 0; g < kPre; ++g) take_tiles<R>(d, pre[g], g > 0, g < G);
#pragma unroll 2
    for (int g = kPre; g < G; ++g) {
      double x[Z::kRaw];
      fetch_tiles<R>(x, w, lane, a.H + (q0 + g) * Z::kH, a.S + (q0 + g) * R * kD);
      take_tiles<R>(d, x, true, true);
    }
  }
  pad_tiles<R>(d, w, lane);
  const double* const Gm = a.G + (a.BHq + own) * kD * kD;
  if (!kGramLate<R, SHARED>) load_gram(gram, Gm, share, lane);
  lds_barrier();
  add_rhs<R>(d, X, a.lam_pK, w, lane);
  add_gram<R>(d, X, Ys, a.lam_pK, w, lane);
  lds_barrier();  // X has been read
  solve_tiles<R>(d, Ys, w, lane);
  if (kGramLate<R, SHARED>) load_gram(gram, Gm, share, lane);
  store_solution<R>(d, w, lane, [&](int i, int j, double x) { X[i * kLdx + j] = x; });
  lds_barrier();
  if (a.last && part == 0) pack_operand<R>(X, a.M + (a.BHq + own) * PfShape<R>::mpack_units, t);
  sums_of<R>(X, Ys, gram, share, a.SK_new + own * R * kD, a.HK_new + own * Z::kH, w, lane);
}

// Second half, a query head per workgroup (SHARED: per four): with the sums of the new A_K,
//   M_Q = (S_K^T + lambda_pQ B_Q^T)(H_K + lambda_pQ B_Q B_Q^T)^-1,  and S_Q, H_Q of A_Q = Q M_Q.
template <int R, bool SHARED>
__global__ __launch_bounds__(kAlgThreads) void prefill_round_q_kernel(const PfState a) {
  using Z = PfAlg<R>;
  extern __shared__ __align__(16) double pf_alg[];
  double* const X = pf_alg;
  double* const Ys = X + Z::kX;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  constexpr int kParts = SHARED ? 4 : 1;
  int bh, part;
  dev::place(blockIdx.x, a.BHq, kParts, bh, part);
  using Part = PfPart<R, SHARED>;
  const Part share(part, w);
  const int b = bh / a.Hq, kvh = (bh - b * a.Hq) / (a.Hq / a.Hkv);
  const size_t kv = (size_t)b * a.Hkv + kvh;
  const double* BQ = a.BQ + (size_t)bh * R * kD;
  f64x4 d[Z::TPW];
  load_tiles<R>(d, w, lane, a.HK_new + kv * Z::kH, a.SK_new + kv * R * kD);
#pragma unroll 8
  for (int e = t; e < R * kD; e += kAlgThreads) X[(e / kD) * kLdx + e % kD] = BQ[e];
  if (16 * Z::RT > R)
    for (int e = t; e < (16 * Z::RT - R) * kLdx; e += kAlgThreads) X[R * kLdx + e] = 0.0;
  double gram[Part::kSteps];
  const double* const Gm = a.G + (size_t)bh * kD * kD;
  if (!kGramLate<R, SHARED> && !a.last) load_gram(gram, Gm, share, lane);
  lds_barrier();
  add_rhs<R>(d, X, a.lam_pQ, w, lane);
  add_gram<R>(d, X, Ys, a.lam_pQ, w, lane);
  lds_barrier();  // X has been read
  solve_tiles<R>(d, Ys, w, lane);
  if (kGramLate<R, SHARED> && !a.last) load_gram(gram, Gm, share, lane);
  store_solution<R>(d, w, lane, [&](int i, int j, double x) { X[i * kLdx + j] = x; });
  lds_barrier();
  if (a.last)
    pack_operand<R>(X, a.M + (size_t)bh * PfShape<R>::mpack_units, t);
  else
    sums_of<R>(X, Ys, gram, share, a.S + (size_t)bh * R * kD, a.H + (size_t)bh * Z::kH, w, lane);
}

// ------------------------------------------------------------------------------------------
// Apply: X = Y M, a wavefront per 32 rows.  The rows pass through 8 KB of LDS of the wavefront's
// own (256 bytes a row: bf16 rows at once, fp32 rows in two halves), from coalesced loads to
// "lane = row"; 16-byte piece c of row i is kept at c ^ (i % 16), so that 16 rows' reads of one
// piece lie in different banks.  The next rows' loads are in flight during the products.  M is
// the same for a whole head: in registers at r <= 32 (96 of them), in LDS at r = 64.
// Bound by HBM (Y in, X out): 2.0 GB in 0.32 ms at 32 + 8 heads, l = 131072, r = 32.  The rows go from the
// last to the first: the last that the reduction read are still in the Infinity Cache (1018 -> 1006 us for
// the whole call at that shape).
template <int R>
constexpr size_t apply_lds_bytes() {
  return 4 * 8192 + (R > 32 ? PfShape<R>::mpack_units * 16 : 0);
}

template <int R, int NS, bool NT_LOAD, bool NT_STORE>
__global__ __launch_bounds__(kPfThreads, 2) void prefill_apply_kernel(
    const void* __restrict__ Q, const void* __restrict__ K, const uint4* __restrict__ M,
    float* __restrict__ A_Q, float* __restrict__ A_K, int BHq, int l, int lk, int units,
    int blocks_per_head) {
  using S = PfShape<R>;
  constexpr int RB = S::RB;
  constexpr int ROW16 = NS == 1 ? 16 : 32;
  constexpr int NPH = ROW16 / 16;            // 256-byte phases of a row
  constexpr int STEPS = 8 / NPH;             // k steps of 16 per phase
  extern __shared__ __align__(16) unsigned char pf_lds[];
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  u32x4* const Yl = reinterpret_cast<u32x4*>(pf_lds) + w * 512;
  u32x4* const Ml = reinterpret_cast<u32x4*>(pf_lds) + 4 * 512;
  const int at = gridDim.x - 1 - blockIdx.x;  // from the last rows on: see above
  const int bh = at / blocks_per_head, block = at - bh * blocks_per_head;
  const bool isq = bh < BHq;
  const size_t head = isq ? bh : bh - BHq;
  const u32x4* __restrict__ Yh = static_cast<const u32x4*>(isq ? Q : K) + head * (size_t)l * ROW16;
  float* __restrict__ Xh = isq ? A_Q + head * (size_t)l * R : A_K + head * (size_t)lk * R;
  const u32x4* __restrict__ Mh = reinterpret_cast<const u32x4*>(M) + bh * S::mpack_units;

  u32x4 mreg[RB == 1 ? 24 : 1];
  if (RB == 1) {
#pragma unroll
    for (int i = 0; i < 24; ++i) mreg[RB == 1 ? i : 0] = Mh[i * 64 + lane];
  } else {
    for (int i = t; i < (int)S::mpack_units; i += kPfThreads) Ml[i] = Mh[i];
    __syncthreads();
  }
  auto m_op = [&](int p, int rb, int step) {
    const u32x4 u = RB == 1 ? mreg[RB == 1 ? p * 8 + step : 0] : Ml[((p * RB + rb) * 8 + step) * 64 + lane];
    return __builtin_bit_cast(bf16x8, u);
  };

  const int first = (block * 4 + w) * units * 32;
  const int last = min(l, first + units * 32);
  u32x4 pre[8];
  auto prefetch = [&](int row0, int ph) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int row = min(row0 + 4 * j + (lane >> 4), last - 1);  // (results past the end are dropped)
      const u32x4* at = Yh + (size_t)row * ROW16 + 16 * ph + (lane & 15);
      pre[j] = NT_LOAD ? __builtin_nontemporal_load(at) : *at;
    }
  };
  if (first >= last) return;  // (no barrier follows)
  prefetch(first, 0);
  const int i = lane & 31, kh = lane >> 5;
  for (int row0 = first; row0 < last; row0 += 32) {
    f32x16 acc[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[rb][v] = 0.0f;
#pragma unroll
    for (int ph = 0; ph < NPH; ++ph) {
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int row = 4 * j + (lane >> 4);
        Yl[row * 16 + ((lane & 15) ^ (row & 15))] = pre[j];
      }
      __builtin_amdgcn_wave_barrier();
      if (ph + 1 < NPH)
        prefetch(row0, ph + 1);
      else if (row0 + 32 < last)
        prefetch(row0 + 32, 0);
#pragma unroll
      for (int st = 0; st < STEPS; ++st) {
        const int step = ph * STEPS + st;
        bf16x8 y[NS];
        if (NS == 1) {
          y[0] = __builtin_bit_cast(bf16x8, Yl[i * 16 + ((2 * st + kh) ^ (i & 15))]);
        } else {
          uint32_t s[4][3];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const u32x4 u = Yl[i * 16 + ((4 * st + 2 * kh + h) ^ (i & 15))];
            split3(__uint_as_float(u.x), __uint_as_float(u.y), s[2 * h]);
            split3(__uint_as_float(u.z), __uint_as_float(u.w), s[2 * h + 1]);
          }
#pragma unroll
          for (int p = 0; p < NS; ++p)
            y[p] = __builtin_bit_cast(bf16x8, (u32x4{s[0][p], s[1][p], s[2][p], s[3][p]}));
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            const bf16x8 m = m_op(j, rb, step);
#pragma unroll
            for (int p = 0; p < NS && p + j < 3; ++p) acc[rb] = mfma_bf16(y[p], m, acc[rb]);
          }
      }
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int j = 32 * rb + i;
      if (j < R) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int row = row0 + mfma_row(v, lane);
          if (row >= last) continue;
          if (NT_STORE)
            __builtin_nontemporal_store(acc[rb][v], Xh + (size_t)row * R + j);
          else
            Xh[(size_t)row * R + j] = acc[rb][v];
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// Chunks of rows per head: the fewest workgroup rounds (one workgroup per CU) times the passes
// of a workgroup, a partial costing about as much as four passes.  At most kPfSlots partials
// unless there are more heads than that.
// `wide`: the sums of a chunk are as good however long it is (kWideSums), and a partial also costs its
// traffic, written and read, a 64th of a round: 6 chunks instead of 19 at 32 + 8 heads, l = 131072, r = 32,
// 956 -> 944 us for the whole call.  Not where S and H are in fp32 over a chunk and in fp64 only beyond it:
// three times as many fp32 additions in a row round three times as far off (test_prefill_long_sums, 6.3e-7
// instead of 2.0e-7).
constexpr int kPfSlots = 1024;
int reduce_chunks(int heads, int l, int rows, bool wide) {
  const int tiles = ceil_div(l, rows);
  const int most = heads >= kPfSlots ? 1 : min(tiles, kPfSlots / heads);
  int best = 1;
  long best_cost = 0;
  for (int n = 1; n <= most; ++n) {
    const int per = ceil_div(tiles, n);
    const long cost = 64 * (long)ceil_div(heads * ceil_div(tiles, per), 256) * (per + 4) +
                      (wide ? (long)heads * n : 0);
    if (n == 1 || cost < best_cost) {
      best = n;
      best_cost = cost;
    }
  }
  return best;
}

struct PrefillWs {
  void* part;
  double *G, *S, *H, *SK2, *HK2, *BQ, *group;  // (S and H: query heads, then KV heads)
  uint4* M;
  size_t bytes;
};
template <int R>
PrefillWs carve_prefill(void* base, const lrqk_shape& s) {
  using S = PfShape<R>;
  const size_t BHq = (size_t)s.B * s.Hq, heads = BHq + (size_t)s.B * s.Hkv;
  // room for the partials of any shape that is no larger than this one
  const size_t tiles = (size_t)ceil_div(s.l, PfReduce<R, 1>::kRows);
  const size_t most = heads > kPfSlots ? heads : (size_t)kPfSlots;
  const size_t parts = heads * tiles < most ? heads * tiles : most;
  PrefillWs w;
  size_t off = 0;
  auto take = [&](size_t n) {
    char* p = base ? static_cast<char*>(base) + off : nullptr;
    off += round_up(n, 256);
    return static_cast<void*>(p);
  };
  w.part = take(parts * S::part_bytes);
  w.G = static_cast<double*>(take(heads * kD * kD * sizeof(double)));
  w.S = static_cast<double*>(take(heads * R * kD * sizeof(double)));
  w.H = static_cast<double*>(take(heads * PfAlg<R>::kH * sizeof(double)));
  w.SK2 = static_cast<double*>(take((heads - BHq) * R * kD * sizeof(double)));
  w.HK2 = static_cast<double*>(take((heads - BHq) * PfAlg<R>::kH * sizeof(double)));
  w.BQ = static_cast<double*>(take(BHq * R * kD * sizeof(double)));
  w.group = static_cast<double*>(take(kGroupSums<R> ? (heads - BHq) * R * (R + kD) * sizeof(double) : 0));
  w.M = static_cast<uint4*>(take(heads * S::mpack_units * sizeof(uint4)));
  w.bytes = off;
  return w;
}

// A kernel's dynamic-LDS ceiling is raised once per device and instantiation.
template <int R, int NS>
struct PfKernels {
  static hipError_t allow() {
    static std::atomic<uint64_t> reduce{0}, rk[2], rq[2], apply[3];
    constexpr size_t lds = PfAlg<R>::lds_bytes;
    hipError_t e = raise_dynamic_lds_once(prefill_reduce_kernel<R, NS>, PfReduce<R, NS>::lds_bytes, reduce);
    if (e == hipSuccess) e = raise_dynamic_lds_once(prefill_round_k_kernel<R, false>, lds, rk[0]);
    if (e == hipSuccess) e = raise_dynamic_lds_once(prefill_round_k_kernel<R, true>, lds, rk[1]);
    if (e == hipSuccess) e = raise_dynamic_lds_once(prefill_round_q_kernel<R, false>, lds, rq[0]);
    if (e == hipSuccess) e = raise_dynamic_lds_once(prefill_round_q_kernel<R, true>, lds, rq[1]);
    constexpr size_t al = apply_lds_bytes<R>();
    if (e == hipSuccess) e = raise_dynamic_lds_once(prefill_apply_kernel<R, NS, false, false>, al, apply[0]);
    if (e == hipSuccess) e = raise_dynamic_lds_once(prefill_apply_kernel<R, NS, false, true>, al, apply[1]);
    if (e == hipSuccess) e = raise_dynamic_lds_once(prefill_apply_kernel<R, NS, true, true>, al, apply[2]);
    return e;
  }
};

template <int R, int NS>
hipError_t run_prefill(const lrqk_shape& s, const void* Q, const void* K, float* A_Q, float* A_K,
                       float* B_Q, float* B_K, float lam_pQ, float lam_pK, int n_iter, void* ws,
                       hipStream_t st) {
  using S = PfShape<R>;
  const PrefillWs w = carve_prefill<R>(ws, s);
  const int BHq = s.B * s.Hq, BHkv = s.B * s.Hkv, heads = BHq + BHkv, l = s.l, lk = row_cap(s);
  hipError_t e = PfKernels<R, NS>::allow();
  if (e != hipSuccess) return e;
  constexpr int kRows = PfReduce<R, NS>::kRows;
  const int per_chunk = ceil_div(ceil_div(l, kRows), reduce_chunks(heads, l, kRows, PfReduce<R, NS>::kWideSums));
  const int nchunk = ceil_div(ceil_div(l, kRows), per_chunk);
  hipLaunchKernelGGL((prefill_reduce_kernel<R, NS>), dim3(nchunk * heads), dim3(kRedThreads),
                     (PfReduce<R, NS>::lds_bytes), st, Q, K, A_Q, A_K, w.part, BHq, l, lk, nchunk,
                     per_chunk);
  hipLaunchKernelGGL((prefill_sum_kernel<R, PfAlg<R>::CS>),
                     dim3(ceil_div((S::GB + S::HB0) * 1024 + R * R, 256) * heads),
                     dim3(256), 0, st, w.part, w.G, w.S, w.H, nchunk);
  PfState a;
  a.G = w.G; a.S = w.S; a.H = w.H; a.BQ = w.BQ; a.M = w.M; a.group = w.group; a.B_Q = B_Q;
  a.B_K = B_K;
  a.Hq = s.Hq; a.Hkv = s.Hkv; a.BHq = BHq; a.BHkv = BHkv; a.lam_pQ = lam_pQ; a.lam_pK = lam_pK;
  // four workgroups per head while there is a compute unit for every one
  const bool share_k = 4 * BHkv + BHq <= 256, share_q = 4 * BHq <= 256;
  double *SK = w.S + (size_t)BHq * R * kD, *HK = w.H + (size_t)BHq * PfAlg<R>::kH;
  double *SK_new = w.SK2, *HK_new = w.HK2;
  constexpr size_t lds = PfAlg<R>::lds_bytes;
  for (int it = 0; it < n_iter; ++it) {
    a.last = it + 1 == n_iter;
    a.SK = SK; a.HK = HK; a.SK_new = SK_new; a.HK_new = HK_new;
    if constexpr (kGroupSums<R>)
      hipLaunchKernelGGL((prefill_group_kernel<R>), dim3(BHkv * (R * (R + kD) / 256)), dim3(256), 0, st, a);
    if (share_k)
      hipLaunchKernelGGL((prefill_round_k_kernel<R, true>), dim3(4 * BHkv + BHq), dim3(kAlgThreads), lds, st, a);
    else
      hipLaunchKernelGGL((prefill_round_k_kernel<R, false>), dim3(BHkv + BHq), dim3(kAlgThreads), lds, st, a);
    if (share_q && !a.last)
      hipLaunchKernelGGL((prefill_round_q_kernel<R, true>), dim3(4 * BHq), dim3(kAlgThreads), lds, st, a);
    else
      hipLaunchKernelGGL((prefill_round_q_kernel<R, false>), dim3(BHq), dim3(kAlgThreads), lds, st, a);
    std::swap(SK, SK_new);
    std::swap(HK, HK_new);
  }
  // 32-row units per wavefront: enough workgroups to fill the chip a few times over
  // (the whole call at l = 131072, r = 32, 32 + 8 heads, with at most 16 or 8 of them: 26 and 2 us more)
  const int row_units = ceil_div(l, 32);
  int units = 1;
  while (units < 4 && (long)ceil_div(row_units, 8 * units) * heads >= 2048) units *= 2;
  const int blocks = ceil_div(row_units, 4 * units);
  // Non-temporal stores where A_Q and A_K exceed the L2s (32 MB), loads where Q and K exceed the
  // Infinity Cache (256 MB).  Whole call, 32 + 8 heads, bf16, in us with neither, stores, both: l = 131072,
  // r = 32: 1013, 980, 967; l = 16384: 185, 180, 187; l = 4096, r = 16: 78.9, 79.5, 82.0; 4 x (16 + 2) heads,
  // l = 8192, r = 8 (19 MB out): 134, 137, 145.
  const bool nt_load = (size_t)heads * l * kD * (NS == 1 ? 2 : 4) > (size_t)256 << 20;
  const bool nt_store = nt_load || (size_t)heads * l * R * 4 > (size_t)32 << 20;
  auto apply = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks * heads), dim3(kPfThreads), apply_lds_bytes<R>(), st, Q, K,
                       w.M, A_Q, A_K, BHq, l, lk, units, blocks);
  };
  if (nt_load)
    apply(prefill_apply_kernel<R, NS, true, true>);
  else if (nt_store)
    apply(prefill_apply_kernel<R, NS, false, true>);
  else
    apply(prefill_apply_kernel<R, NS, false, false>);
  return hipGetLastError();
}

template <int R>
hipError_t run_prefill_dtype(const lrqk_shape& s, const void* Q, const void* K, float* A_Q,
                             float* A_K, float* B_Q, float* B_K, float lam_pQ, float lam_pK,
                             int n_iter, void* ws, hipStream_t st) {
  return s.kv_dtype == LRQK_KV_BF16
             ? run_prefill<R, 1>(s, Q, K, A_Q, A_K, B_Q, B_K, lam_pQ, lam_pK, n_iter, ws, st)
             : run_prefill<R, 3>(s, Q, K, A_Q, A_K, B_Q, B_K, lam_pQ, lam_pK, n_iter, ws, st);
}

}  // namespace

bool prefill_supported(const lrqk_shape& s) {
  return s.r == 8 || s.r == 16 || s.r == 32 || s.r == 64;
}

size_t prefill_ws_bytes(const lrqk_shape& s) {
  switch (s.r) {
    case 8: return carve_prefill<8>(nullptr, s).bytes;
    case 16: return carve_prefill<16>(nullptr, s).bytes;
    case 32: return carve_prefill<32>(nullptr, s).bytes;
    case 64: return carve_prefill<64>(nullptr, s).bytes;
    default: return 0;
  }
}

hipError_t launch_prefill(const lrqk_shape& s, const void* Q, const void* K, float* A_Q,
                          float* A_K, float* B_Q, float* B_K, float lam_pQ, float lam_pK,
                          int n_iter, float* ws, hipStream_t st) {
  switch (s.r) {
    case 8:
      return run_prefill_dtype<8>(s, Q, K, A_Q, A_K, B_Q, B_K, lam_pQ, lam_pK, n_iter, ws, st);
    case 16:
      return run_prefill_dtype<16>(s, Q, K, A_Q, A_K, B_Q, B_K, lam_pQ, lam_pK, n_iter, ws, st);
    case 32:
      return run_prefill_dtype<32>(s, Q, K, A_Q, A_K, B_Q, B_K, lam_pQ, lam_pK, n_iter, ws, st);
    case 64:
      return run_prefill_dtype<64>(s, Q, K, A_Q, A_K, B_Q, B_K, lam_pQ, lam_pK, n_iter, ws, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lrqk
