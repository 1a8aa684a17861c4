// u1 — decode-time update of the factors (Alg. 2 from the initial guess of k_hat to the
// two gradient steps; Sec. 4.2 update rules for q_hat_t, k_hat_t, B_Q, B_K; App. A.2 optimal
// step lengths).
//
// Three launches at r = 32 and 64 (r = 8 and 16: factor_update_small.hip, which says why).
//
//  1. factor_gram_kernel: the sums over the rows of Omega of a query head (the k rows selected at
//     the previous step, read from their cache slots, and the w lite rows):  S = sum_i a_i^T a_i
//     (r x r) and g = sum_i u_i a_i (r), a_i = row of A_K, u_i = q . K_i.  The row list of a head is
//     cut into chunks of at most 144 rows, one workgroup each, so that batch-1 steps still use
//     hundreds of CUs; K rows are read by 16 lanes each exactly as the attention kernel reads
//     them (update_gram.h).  Partial sums per chunk go to the workspace: no atomics, the result does
//     not depend on scheduling.
//  2. factor_inverse_kernel: P^-1 and N^-1 (what changes between rounds is a low-rank correction
//     of these two), a workgroup per matrix.
//  3. factor_rounds_kernel: the n_iter rounds and the line-search gradient steps on B_Q and B_K in
//     place, workgroups per (batch, KV head).
// Times in us at k = 2048, w = 64, 32 + 8 heads, r = 32: 10.5 + 9.2 + 9.5; at 8 x (28 + 4) heads, k = 1024, r = 64:
// 37 + 22 + 19.5 (launches on four sets of inputs in turn; on one set, whose rows the caches then hold, launch 1
// takes 8.6 and 32, and the calls that the comments below give times of 25.8 and 69.8 instead of 27.9 and 77).
// (Factorising in fp32 with a row per lane, P once and the k_hat system in every
// round, all in one wavefront per head, launches 2 and 3 took 30 and 114 us.)  What is left is
// latency: the loads at the start of each launch (2 us; 5 to 9 us at the second shape, where every
// compute unit reads 130 and 265 KB), the eliminations (3.5 and 9 us) and the rounds (2 and 4 us each).
//
// Sums over rows are fp32 (App. B.1 runs these updates in fp32; at r = 64 made of products of the bf16 terms
// that add up to the fp32 numbers), the rest fp64.
#include <algorithm>

#include "lrqk_alg64.h"
#include "lrqk_device.h"
#include "lrqk_internal.h"
#include "update_gram.h"

namespace lrqk {
namespace {

using namespace alg64;
using dev::place;

// (r = 64, bf16 rows: as many workgroups on a compute unit as its LDS holds, four, 79.6 -> 77.6 us for the call at
// 8 x (28 + 4) heads; left alone the registers allow one fewer.  fp32 rows keep twice as many in flight: three)
template <int R, bool BF16>
__global__ __launch_bounds__(kGramThreads, R > 32 ? BF16 ? 4 : 3 : 1) void factor_gram_kernel(GramRows a,
                                                                                           int BHkv,
                                                                                           bool by_die) {
  __shared__ GramLds<R> s;
  const int t = threadIdx.x, G = a.Hq / a.Hkv;
  int bkv, part;
  place(blockIdx.x, BHkv, G * a.nchunk, bkv, part, by_die);
  const int job = part % a.nchunk;
  const int bh = bkv / a.Hkv * a.Hq + bkv % a.Hkv * G + part / a.nchunk;
  GramAcc<R> acc;
  float gpart;
  gram_chunk<R, BF16>(a, s, bh, bkv, job, acc, gpart, t);
  gram_store<R>(s, acc, gpart, a.gram_om + ((size_t)bh * a.nchunk + job) * (R * R + R), t);
}

struct SolveArgs {
  const float* gram_om;  // [B*Hq][nchunk][r*r + r]
  double* inv;           // [B*Hq + B*Hkv][r*r + r]: P^-1 and c of a query head, N^-1 and nb of a KV head
  const float* q;        // [B,Hq,d]
  const void* k_new;     // [B,Hkv,d]
  float* B_Q;            // [B,Hq,r,d]   updated in place
  float* B_K;            // [B,Hkv,r,d]  updated in place
  float* q_hat;          // [B,Hq,r]
  float* k_hat;          // [B,Hkv,r]
  int Hq, Hkv, BHq, BHkv, nchunk, n_iter;
  int parts;             // workgroups per KV head in the rounds
  float lam1, lam2;
};

// ---- 2. the inverses --------------------------------------------------------------------------
// One workgroup of 8 wavefronts per matrix, all in fp64:
//   query head:  P = B_Q B_Q^T + lambda_d2 A_Om^T A_Om,  c = q B_Q^T + lambda_d2 q K_Om^T A_Om
//   KV head:     N = B_K B_K^T,                          nb = k B_K^T
// The chunk partials of launch 1 are added in chunk order.  The matrix lies in 16 x 16 tiles in
// the wavefronts' registers and is inverted in place by Gauss-Jordan elimination, a pivot tile at a
// time (lrqk_alg64.h).  Latency bound: r / 16 steps, each four inversions of 4 x 4 blocks in one
// wavefront, an exchange through LDS with two barriers, and the MFMAs.
constexpr int kInvThreads = 512;
constexpr int kLdb = kD + 2;  // LDS row stride: 16 rows x 2 columns fall on 32 different bank pairs
template <int R>
struct InvShape {
  static_assert(R % 32 == 0, "no padding");
  static constexpr int RT = R / 16;                           // RT x RT tiles
  static constexpr int TPW = RT * RT > 8 ? RT * RT / 8 : 1;   // tiles of a wavefront, one tile row
  static constexpr int kX = 16 * RT * kLdb;
  static_assert(sweep_doubles<RT, RT>() <= kX, "the elimination works in the memory of B");
  static constexpr size_t lds_bytes = ((size_t)kX + kD) * sizeof(double);
};

template <int R, bool BF16>
__global__ __launch_bounds__(kInvThreads) void factor_inverse_kernel(SolveArgs a) {
  using Z = InvShape<R>;
  constexpr int kEntries = R * R;
  constexpr size_t ROWB = kD * (BF16 ? 2 : 4);
  extern __shared__ __align__(16) double inv_lds[];
  double* const X = inv_lds;            // [16 RT][kLdb]  B
  double* const xs = X + Z::kX;         // [d]  q or k
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int G = a.Hq / a.Hkv;
  int bkv, job;
  place(blockIdx.x, a.BHkv, G + 1, bkv, job);
  const bool isq = job < G;
  const size_t head = isq ? (size_t)(bkv / a.Hkv) * a.Hq + (size_t)(bkv % a.Hkv) * G + job : bkv;
  const size_t m = isq ? head : a.BHq + head;
  const float* __restrict__ Bm = (isq ? a.B_Q : a.B_K) + head * R * kD;
  const float* __restrict__ part = a.gram_om + (isq ? head : 0) * a.nchunk * (size_t)(kEntries + R);
  const int tr = w * Z::TPW / Z::RT, tc0 = w * Z::TPW % Z::RT;
  const bool own = tr < Z::RT;          // (r <= 32: the other wavefronts own no tile)
  const int k = lane >> 4, c16 = lane & 15;

  constexpr int NB4 = R * kD / 4, NB = (NB4 + kInvThreads - 1) / kInvThreads;
  float4 bv[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
    bv[j] = reinterpret_cast<const float4*>(Bm)[min(t + kInvThreads * j, NB4 - 1)];
  // (q and k both, of which one is wanted: a load inside a branch is waited for before the next is issued)
  const float q_t = a.q[(isq ? head : 0) * kD + (t & (kD - 1))];
  const float k_t = kv_load<BF16>(static_cast<const char*>(a.k_new) + (size_t)bkv * ROWB, t & (kD - 1));
  // The chunk partials are on their way while B B^T is made: of the matrix, of the first SB chunks; of c,
  // row t / 8 and every eighth chunk, of the first 16.  (A KV head reads a query head's and drops them.)
  // Issued earlier, beside the loads of B, they make those wait: at r = 64 all compute units together read
  // 30 MB.  The whole call so, with the load of q or k in no branch, 77.5 -> 76.5 us there, 26.3 -> 25.9 at
  // 32 + 8 heads, r = 32, k = 2048.
  constexpr int SB = 16 / Z::TPW;
  float x[SB][Z::TPW][4];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int sc = 0; sc < SB; ++sc)
#pragma unroll
      for (int u = 0; u < Z::TPW; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          x[sc][u][v] = part[(size_t)min(s0 + sc, a.nchunk - 1) * (kEntries + R) +
                             (16 * min(tr, Z::RT - 1) + 4 * v + k) * R + 16 * (tc0 + u) + c16];
  };
  const int row = t >> 3, part8 = t & 7;
  auto g_at = [&](int s) {
    return part[(size_t)min(s, a.nchunk - 1) * (kEntries + R) + kEntries + min(row, R - 1)];
  };
  if (t < kD) xs[t] = isq ? q_t : k_t;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int e = 4 * (t + kInvThreads * j);
    if (e < R * kD) {
      double* b = X + e / kD * kLdb + e % kD;
      b[0] = bv[j].x; b[1] = bv[j].y; b[2] = bv[j].z; b[3] = bv[j].w;
    }
  }
  lds_barrier();
  const float g0 = g_at(part8), g1 = g_at(part8 + 8);
  fetch(0);
  __builtin_amdgcn_sched_barrier(0);
  // B B^T
  f64x4 d[Z::TPW];
#pragma unroll
  for (int u = 0; u < Z::TPW; ++u) {
    d[u] = f64x4{0.0, 0.0, 0.0, 0.0};
    const double* xa = X + (16 * tr + c16) * kLdb + k;
    const double* xb = X + (16 * (tc0 + u) + c16) * kLdb + k;
    if (own) {
#pragma unroll 8
      for (int s = 0; s < kD; s += 4) d[u] = mfma_f64(xa[s], xb[s], d[u]);
    }
  }
  // c (or nb): 8 lanes a row
  double* const out = a.inv + m * (kEntries + R);
  const double lam2 = isq ? (double)a.lam2 : 0.0;
  {
    double c = 0.0;
    if (row < R) {
      const double* b = X + row * kLdb + part8;
#pragma unroll
      for (int j = 0; j < kD; j += 8) c = __builtin_fma(b[j], xs[j + part8], c);
    }
    if (isq) {
      if (part8 < a.nchunk) c = __builtin_fma(lam2, (double)g0, c);
      if (part8 + 8 < a.nchunk) c = __builtin_fma(lam2, (double)g1, c);
      for (int s = part8 + 16; s < a.nchunk; s += 8) c = __builtin_fma(lam2, (double)g_at(s), c);
    }
    c += dpp_f64<0xB1>(c);   // quad_perm [1,0,3,2]
    c += dpp_f64<0x4E>(c);   // quad_perm [2,3,0,1]
    c += dpp_f64<0x141>(c);  // row_half_mirror
    if (row < R && part8 == 0) out[kEntries + row] = c;
  }
  // += lambda_d2 A_Om^T A_Om, in chunk order.  (At r = 64 an entry of the sums and its mirror image may differ in
  // their last bits, and the elimination takes pivot columns from pivot rows: with such sums of condition 10 to 1e6
  // emulated on the CPU the solutions are as far off as with the upper half mirrored, to three digits.)
  if (isq && own) {
    f64x4 sum[Z::TPW] = {};
    for (int s0 = 0; s0 < a.nchunk; s0 += SB) {
      if (s0 > 0) fetch(s0);
#pragma unroll
      for (int sc = 0; sc < SB; ++sc)
#pragma unroll
        for (int u = 0; u < Z::TPW; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v) sum[u][v] += s0 + sc < a.nchunk ? (double)x[sc][u][v] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < Z::TPW; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) d[u][v] = __builtin_fma(lam2, sum[u][v], d[u][v]);
  }
  lds_barrier();  // X has been read: the exchanged tiles take its place
  sweep_tiles<Z::RT, Z::RT, Z::TPW, 1, true>(d, tr, tc0, X, lane);
  if (own) {
#pragma unroll
    for (int u = 0; u < Z::TPW; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 16 * tr + 4 * v + k, j = 16 * (tc0 + u) + c16;
        out[i * R + j] = d[u][v];
      }
  }
}

// ---- 3. the rounds ------------------------------------------------------------------------------
// A wavefront per query head of a group, two at r = 64; lane i holds element i of a vector.  With P^-1
// and N^-1 at hand a round is products of r x r matrices with vectors (P^-1 in registers, symmetric: lane i
// holds 32 elements of column i, 64 being more than fit beside the rest; the vector's elements as LDS
// broadcasts; N^-1 in LDS, its products by MFMA):
//   q_hat = m_lq M_rq^-1, M_rq = P + lambda_d1 k_hat^T k_hat a rank-one change of P:
//     z = k_hat P^-1,  v = m_lq P^-1 = y0 + lambda_d1 (q.k) z  (y0 = c P^-1),
//     q_hat = v - z * lambda_d1 (k_hat . v) / (1 + lambda_d1 (k_hat . z))
//   k_hat = rhs M^-1, M = N + lambda_d1 Q^T Q (Q: the group's q_hat as rows) a rank-G change of N:
//     W = Q N^-1,  u = rhs N^-1 = nb N^-1 + lambda_d1 sum_g (q_g.k) w_g,
//     k_hat = u - lambda_d1 s W  with  (I + lambda_d1 W Q^T) s = Q u,
//   a G x G system that the first wavefront sets up in one tile, W Q^T and Q u from one chain of MFMAs,
//   and solves with one or two pivot steps (shuffles between lanes, in every wavefront, took 2 us a round).
// fp64 throughout, so that the corrections lose nothing.
// Then one gradient step on 1/2 |x_hat B - x|^2 for every B_Q of the group and B_K (App. A.2): with
// e = x_hat B - x the gradient is x_hat^T e and x_hat times it |x_hat|^2 e, so the step length
// <e, |x_hat|^2 e> / | |x_hat|^2 e |^2 is 1 / |x_hat|^2 and a column of B needs nothing from the
// others: eight rows of a column per thread.  (e = 0 or x_hat = 0: B stays.)
// Those steps read and write G + 1 matrices, 256 KB at r = 64 and G = 7, which took one compute unit
// 8 us.  So the matrices of a group are dealt out over `parts` workgroups, all of which go through the
// rounds (on compute units that would be idle) and whose first matrix is on its way meanwhile.  The whole
// call, 8 x (28 + 4) heads, r = 64, with 1, 2, 4, 8 of them: 106.6, 95.9, 90.9, 88.7 us; 32 + 8 heads, r = 32,
// with 1 and 5: 31.0, 28.5; but 8 x (32 + 8) heads with 4 and 5, that is 256 and 320: 36.1, 43.8.
template <int R>
struct RoundShape {
  static constexpr int kPerHead = R / 32;  // wavefronts per query head
  static constexpr int kWaves = kMaxG * kPerHead, kThreads = 64 * kWaves;
  static constexpr int kAcross = kThreads / kD;  // threads per column of B
  static constexpr int kRows = R / kAcross;      // rows of a column per thread
  static constexpr int LDV = R + 2;  // LDS row stride of the exchanged vectors: 8 rows, 8 bank groups
  // q_hat (padded to a tile); q_hat N^-1, u (padded); a vector per wavefront; parts of z
  static constexpr int kVectors = 16 + 16 + kWaves + kWaves;
  // The first matrix of the gradient steps waits in LDS at r = 64, where P^-1 takes half of the registers:
  // kept in others, each of its loads was waited for and spilled (so, with kAside, the kernel took 23.6 us
  // instead of 25.7 at 8 x (28 + 4) heads, the call 73.4 instead of 76.5).
  static constexpr bool kStash = R > 32;
  // and so do kAside of the 32 elements of P^-1 that a lane holds
  static constexpr int kAside = R > 32 ? 4 : 0;
  static constexpr size_t doubles =
      (size_t)R * R + kVectors * LDV + 128 + kAcross * kD + 3 * kMaxG + 1 + kAside * kThreads;
  static constexpr size_t lds_bytes = doubles * sizeof(double) + (kStash ? (size_t)R * kD * sizeof(float) : 0);
};

template <int R, bool BF16>
__global__ __launch_bounds__(RoundShape<R>::kThreads) void factor_rounds_kernel(SolveArgs a) {
  using Z = RoundShape<R>;
  constexpr int kEntries = R * R, LDV = Z::LDV;
  constexpr int kRoundThreads = Z::kThreads;
  constexpr size_t ROWB = kD * (BF16 ? 2 : 4);
  extern __shared__ __align__(16) double rnd_lds[];
  double* const n_s = rnd_lds;                  // [r][r]  N^-1
  double* const qh_s = n_s + kEntries;          // [16][LDV]  q_hat of the group
  double* const wv_s = qh_s + 16 * LDV;         // [16][LDV]  q_hat N^-1; row 8: u
  double* const vec_s = wv_s + 16 * LDV;        // [kWaves][LDV]  one vector per wavefront
  double* const z_s = vec_s + Z::kWaves * LDV;  // [kWaves][LDV]  part of a product with P^-1
  double* const piv_s = z_s + Z::kWaves * LDV;  // [128]
  double* const part_s = piv_s + 128;           // [kAcross][d]
  double* const s_s = part_s + Z::kAcross * kD; // [8]  lambda_d1 s
  double* const qk_s = s_s + kMaxG;             // [8]  lambda_d1 q.k
  double* const inv_norm_s = qk_s + kMaxG;      // [9]  1 / |x_hat|^2 of the group's q_hat, of k_hat
  double* const aside = inv_norm_s + kMaxG + 1 + threadIdx.x;                         // [kAside][threads]
  float* const stash = reinterpret_cast<float*>(rnd_lds + Z::doubles) + threadIdx.x;  // [kRows][threads]
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int g = w % kMaxG, h = w / kMaxG;  // head, and which rows of P^-1
  const int G = a.Hq / a.Hkv;
  int bkv, part;
  place(blockIdx.x, a.BHkv, a.parts, bkv, part);
  const int b = bkv / a.Hkv, kvh = bkv - b * a.Hkv;
  const size_t q0 = (size_t)b * a.Hq + (size_t)kvh * G;
  const bool act = g < G;
  const size_t bh = q0 + (act ? g : 0);
  const bool row = lane < R;
  const int li = row ? lane : 0;  // keeps the loads of idle lanes in bounds
  const double* __restrict__ inv_q = a.inv + bh * (kEntries + R);
  const double* __restrict__ inv_k = a.inv + (size_t)(a.BHq + bkv) * (kEntries + R);
  const float* qp = a.q + bh * kD;
  const char* kp = static_cast<const char*>(a.k_new) + (size_t)bkv * ROWB;
  // the gradient steps: rows kRows sub .. of column col of a matrix
  const int col = t & (kD - 1), sub = t / kD;
  auto matrix = [&](int job) {
    return (job < G ? a.B_Q + (q0 + job) * R * kD : a.B_K + (size_t)bkv * R * kD) +
           sub * Z::kRows * kD + col;
  };

  float bv[Z::kRows];
#pragma unroll
  for (int i = 0; i < Z::kRows; ++i) bv[i] = matrix(part)[i * kD];
  constexpr int kN = kEntries / 2 / kRoundThreads;
  static_assert(kN * kRoundThreads * 2 == kEntries, "whole pieces");
  double2 nv[kN];
#pragma unroll
  for (int j = 0; j < kN; ++j) nv[j] = reinterpret_cast<const double2*>(inv_k)[t + j * kRoundThreads];
  double pinv[32];
#pragma unroll
  for (int c = 0; c < 32; ++c) pinv[c] = inv_q[(32 * h + c) * R + li];
  const double cvec = inv_q[kEntries + li], nb = inv_k[kEntries + li];
#pragma unroll
  for (int i = 0; i < Z::kRows; ++i)
    if (Z::kStash) stash[i * kRoundThreads] = bv[i];
#pragma unroll
  for (int j = 0; j < kN; ++j) reinterpret_cast<double2*>(n_s)[t + j * kRoundThreads] = nv[j];
#pragma unroll
  for (int c = 0; c < Z::kAside; ++c) aside[c * kRoundThreads] = pinv[c];
  for (int e = t; e < 32 * LDV; e += kRoundThreads) qh_s[e] = 0.0;  // and wv_s
  const double qk = wave_sum_f64((double)qp[lane] * kv_load<BF16>(kp, lane) +
                                 (double)qp[lane + 64] * kv_load<BF16>(kp, lane + 64));
  const double lam1 = a.lam1;
  if (lane == 0) qk_s[g] = act ? lam1 * qk : 0.0;
  double* const vec = vec_s + w * LDV;
  // x M of the vector x that lane i holds element i of
  auto put = [&](double x) {
    __builtin_amdgcn_wave_barrier();
    if (row) vec[lane] = x;
    __builtin_amdgcn_wave_barrier();
  };
  auto times_pinv = [&](double x, int ln) {  // (a barrier at r = 64); ln: the lane
    __builtin_amdgcn_wave_barrier();
    if (row) vec[ln] = x;
    __builtin_amdgcn_wave_barrier();
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int c = 0; c < 32; c += 2) {
      const double2 v = *reinterpret_cast<const double2*>(vec + 32 * h + c);
      s0 = __builtin_fma(c < Z::kAside ? aside[c * kRoundThreads] : pinv[c], v.x, s0);
      s1 = __builtin_fma(c < Z::kAside ? aside[(c + 1) * kRoundThreads] : pinv[c + 1], v.y, s1);
    }
    s0 += s1;
    if (Z::kPerHead > 1) {
      if (row) z_s[w * LDV + ln] = s0;
      lds_barrier();
      s0 = z_s[g * LDV + ln] + z_s[(g + kMaxG) * LDV + ln];
    }
    return row ? s0 : 0.0;
  };
  const double y0 = times_pinv(cvec, lane);
  __syncthreads();  // n_s, qk_s; qh_s and wv_s are zero
  // k0 = nb N^-1, also the initial guess (lambda_d1 = 0): every wavefront its share of the sum
  {
    constexpr int kShare = R / Z::kWaves;
    put(nb);
    double s0 = 0.0;
#pragma unroll
    for (int c = 0; c < kShare; ++c)
      s0 = __builtin_fma(n_s[(w * kShare + c) * R + li], vec[w * kShare + c], s0);
    put(s0);
  }
  lds_barrier();
  double k0 = 0.0;
#pragma unroll
  for (int ww = 0; ww < Z::kWaves; ++ww) k0 += vec_s[ww * LDV + li];
  if (!row) k0 = 0.0;
  lds_barrier();
  double k_hat = k0, q_hat = 0.0;
#pragma unroll 1
  for (int it = 0; it < a.n_iter; ++it) {
    // r = 64: addresses are made anew in every round; kept across them they were spilled, as P^-1 was for
    // their sake (24 -> 20.5 us for the kernel at 8 x (28 + 4) heads, 73.4 -> 69.8 for the call).  At r = 32
    // there are registers for them (25.8 us for the call at 32 + 8 heads, 26.0 without them).
    int ln = lane;
    if (R > 32) asm volatile("" : "+v"(ln));
    const int c16 = ln & 15, k4 = ln >> 4, li = row ? ln : 0;
    const double z = times_pinv(k_hat, ln);
    const double v = __builtin_fma(lam1 * qk, z, y0);
    const double kv_ = wave_sum_f64(k_hat * v), kz = wave_sum_f64(k_hat * z);
    q_hat = __builtin_fma(-z, lam1 * kv_ / __builtin_fma(lam1, kz, 1.0), v);
    if (act && row && h == 0) qh_s[g * LDV + ln] = q_hat;
    lds_barrier();
    const double* qa = qh_s + c16 * LDV + k4;
    if (w < R / 16) {  // W, 16 columns a wavefront
      f64x4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
      for (int c = 0; c < R; c += 4) x = mfma_f64(qa[c], n_s[(c + k4) * R + 16 * w + c16], x);
#pragma unroll
      for (int e = 0; e < 2; ++e) wv_s[(4 * e + k4) * LDV + 16 * w + c16] = x[e];
    }
    lds_barrier();
    if (w == 0) {
      double u = k0;
#pragma unroll
      for (int gg = 0; gg < kMaxG; ++gg) u = __builtin_fma(qk_s[gg], wv_s[gg * LDV + li], u);
      __builtin_amdgcn_wave_barrier();
      if (row) wv_s[8 * LDV + ln] = u;
      __builtin_amdgcn_wave_barrier();
      // element (a, b) is q_hat_a . w_b, and (a, 8) is q_hat_a . u
      const double* wb = wv_s + c16 * LDV + k4;
      f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
      for (int c = 0; c < R; c += 4) d = mfma_f64(qa[c], wb[c], d);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c16 != 8) d[e] = __builtin_fma(lam1, d[e], 4 * e + k4 == c16 ? 1.0 : 0.0);
      pivot_step(d, 0, piv_s, ln);
      if (G > 4) pivot_step(d, 1, piv_s, ln);
      if (c16 == 8) {
        s_s[k4] = lam1 * d[0];
        s_s[4 + k4] = G > 4 ? lam1 * d[1] : 0.0;
      }
    }
    lds_barrier();
    k_hat = wv_s[8 * LDV + li];
#pragma unroll
    for (int gg = 0; gg < kMaxG; ++gg) k_hat = __builtin_fma(-s_s[gg], wv_s[gg * LDV + li], k_hat);
    if (!row) k_hat = 0.0;
  }

  // gradient steps
  const double nq = wave_sum_f64(q_hat * q_hat), nk = wave_sum_f64(k_hat * k_hat);
  if (lane == 0 && h == 0) {
    inv_norm_s[g] = nq > 0.0 ? 1.0 / nq : 0.0;
    if (g == 0) inv_norm_s[kMaxG] = nk > 0.0 ? 1.0 / nk : 0.0;
  }
  if (w == 0) put(k_hat);  // vec_s[0]
  if (act && row && h == 0 && g % a.parts == part) a.q_hat[bh * R + lane] = (float)q_hat;
  if (w == 0 && row && G % a.parts == part) a.k_hat[(size_t)bkv * R + lane] = (float)k_hat;
  lds_barrier();
#pragma unroll 1
  for (int job = part; job <= G; job += a.parts) {
    const bool isq = job < G;
    float* Bm = matrix(job);
    if (job != part || Z::kStash) {
#pragma unroll
      for (int i = 0; i < Z::kRows; ++i) bv[i] = job != part ? Bm[i * kD] : stash[i * kRoundThreads];
    }
    const double* xh = (isq ? qh_s + job * LDV : vec_s) + sub * Z::kRows;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int i = 0; i < Z::kRows; i += 2) {
      s0 = __builtin_fma(xh[i], (double)bv[i], s0);
      s1 = __builtin_fma(xh[i + 1], (double)bv[i + 1], s1);
    }
    part_s[sub * kD + col] = s0 + s1;
    lds_barrier();
    double e = -(double)(isq ? a.q[(q0 + job) * kD + col] : kv_load<BF16>(kp, col));
#pragma unroll
    for (int i = 0; i < Z::kAcross; ++i) e += part_s[i * kD + col];
    const double step = e * inv_norm_s[isq ? job : kMaxG];
#pragma unroll
    for (int i = 0; i < Z::kRows; ++i)
      Bm[i * kD] = (float)__builtin_fma(-xh[i], step, (double)bv[i]);
    lds_barrier();  // part_s has been read
  }
}

template <int R, bool BF16>
hipError_t launch_update_r(const lrqk_shape& s, const GramRows& ga, const SolveArgs& sa,
                           hipStream_t st) {
  static std::atomic<uint64_t> inv{0}, rounds{0};  // devices on which the LDS ceilings are up
  hipError_t e = raise_dynamic_lds_once(factor_inverse_kernel<R, BF16>, InvShape<R>::lds_bytes, inv);
  if (e == hipSuccess)
    e = raise_dynamic_lds_once(factor_rounds_kernel<R, BF16>, RoundShape<R>::lds_bytes, rounds);
  if (e != hipSuccess) return e;
  // The partials to the die of their inverse as long as they fit its L2 (4 MB) with room to spare: 28.8 ->
  // 28.5 us for the call at 32 + 8 heads, r = 32 (2 MB in all); 88.7 -> 89.9 at 8 x (28 + 4) heads, r = 64 (30).
  const size_t partials = (size_t)s.B * s.Hq * ga.nchunk * (R * R + R) * sizeof(float);
  hipLaunchKernelGGL((factor_gram_kernel<R, BF16>), dim3(ga.nchunk * s.B * s.Hq), dim3(kGramThreads), 0,
                     st, ga, s.B * s.Hkv, partials <= (size_t)16 << 20);
  hipLaunchKernelGGL((factor_inverse_kernel<R, BF16>), dim3(s.B * (s.Hq + s.Hkv)),
                     dim3(kInvThreads), InvShape<R>::lds_bytes, st, sa);
  hipLaunchKernelGGL((factor_rounds_kernel<R, BF16>), dim3(s.B * s.Hkv * sa.parts), dim3(RoundShape<R>::kThreads),
                     RoundShape<R>::lds_bytes, st, sa);
  return hipGetLastError();
}

template <int R>
hipError_t launch_update_dtype(bool bf16, const lrqk_shape& s, const GramRows& ga,
                               const SolveArgs& sa, hipStream_t st) {
  return bf16 ? launch_update_r<R, true>(s, ga, sa, st) : launch_update_r<R, false>(s, ga, sa, st);
}

}  // namespace

bool factor_update_supported(const lrqk_shape& s) {
  return s.r == 8 || s.r == 16 || s.r == 32 || s.r == 64;
}

UpdateGeom update_geometry(const lrqk_shape& s) {
  UpdateGeom g;
  // as few chunks of at most one LDS batch as cover the k + w rows, evenly sized
  g.nchunk = ceil_div(s.k + s.w, kGramBatch);
  g.chunk_rows = ceil_div(ceil_div(s.k + s.w, g.nchunk), 16) * 16;
  g.per_gram = (size_t)s.r * s.r + s.r;
  return g;
}

size_t update_ws_bytes(const lrqk_shape& s) {
  if (s.r <= 16) return update_small_ws_bytes(s);
  const UpdateGeom g = update_geometry(s);
  const size_t BHq = (size_t)s.B * s.Hq, BHkv = (size_t)s.B * s.Hkv;
  return round_up(BHq * g.nchunk * g.per_gram * sizeof(float), 256) +
         round_up((BHq + BHkv) * g.per_gram * sizeof(double), 256);
}

hipError_t launch_factor_update(const lrqk_shape& s, const float* A_K, const void* cacheK,
                                const void* liteK, const int32_t* sel_idx_prev,
                                const int32_t* sel_slot_prev, const float* q, const void* k_new,
                                float* B_Q, float* B_K, float lam1, float lam2, int n_iter,
                                float* q_hat, float* k_hat, float* ws, hipStream_t st) {
  if (s.r <= 16)
    return launch_factor_update_small(s, A_K, cacheK, liteK, sel_idx_prev, sel_slot_prev, q, k_new,
                                      B_Q, B_K, lam1, lam2, n_iter, q_hat, k_hat, ws, st);
  const UpdateGeom g = update_geometry(s);
  const size_t BHq = (size_t)s.B * s.Hq;
  GramRows ga;
  ga.A_K = A_K; ga.cacheK = cacheK; ga.liteK = liteK;
  ga.sel_idx_prev = sel_idx_prev; ga.sel_slot_prev = sel_slot_prev;
  ga.q = q; ga.gram_om = ws;
  ga.Hq = s.Hq; ga.Hkv = s.Hkv; ga.l = s.l; ga.l_rows = row_cap(s); ga.k = s.k; ga.w = s.w; ga.C = s.C;
  ga.nchunk = g.nchunk; ga.chunk_rows = g.chunk_rows;
  SolveArgs sa;
  sa.gram_om = ga.gram_om;
  sa.inv = reinterpret_cast<double*>(
      reinterpret_cast<char*>(ws) + round_up(BHq * g.nchunk * g.per_gram * sizeof(float), 256));
  sa.q = q; sa.k_new = k_new; sa.B_Q = B_Q; sa.B_K = B_K; sa.q_hat = q_hat; sa.k_hat = k_hat;
  sa.Hq = s.Hq; sa.Hkv = s.Hkv; sa.BHq = (int)BHq; sa.nchunk = g.nchunk; sa.n_iter = n_iter;
  sa.BHkv = s.B * s.Hkv;
  // as many as there are compute units for (one workgroup on each), at most one per matrix
  sa.parts = std::max(1, std::min(s.Hq / s.Hkv + 1, 256 / sa.BHkv));
  sa.lam1 = lam1; sa.lam2 = lam2;
  const bool bf16 = s.kv_dtype == LRQK_KV_BF16;
  switch (s.r) {
    case 32: return launch_update_dtype<32>(bf16, s, ga, sa, st);
    case 64: return launch_update_dtype<64>(bf16, s, ga, sa, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lrqk
