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
//     place, a workgroup per (batch, KV head).
// Times in us at k = 2048, w = 64, 32 + 8 heads, r = 32: 11 + 10 + 13; at 8 x (28 + 4) heads, k = 1024, r = 64:
// 38 + 28 + 31.  (Factorising in fp32 with a row per lane, P once and the k_hat system in every
// round, all in one wavefront per head, launches 2 and 3 took 30 and 114 us.)  What is left is
// latency: the loads at the start of each launch, a chain of r / 4 elimination steps (0.5 us each
// at r = 32, 0.8 us at r = 64).
//
// Sums over rows are fp32 (App. B.1 runs these updates in fp32), the rest fp64.
#include "lrqk_alg64.h"
#include "lrqk_device.h"
#include "lrqk_internal.h"
#include "update_gram.h"

namespace lrqk {
namespace {

using namespace alg64;

template <int R, bool BF16>
__global__ __launch_bounds__(kGramThreads) void factor_gram_kernel(GramRows a) {
  __shared__ GramLds<R> s;
  const int bh = blockIdx.y, job = blockIdx.x, t = threadIdx.x;
  const int b = bh / a.Hq, h = bh - b * a.Hq;
  const int bkv = b * a.Hkv + h / (a.Hq / a.Hkv);
  f32x16 sacc;
#pragma unroll
  for (int v = 0; v < 16; ++v) sacc[v] = 0.0f;
  float gpart = 0.0f;
  gram_chunk<R, BF16>(a, s, bh, bkv, job, sacc, gpart, t);
  gram_store<R>(s, sacc, gpart, a.gram_om + ((size_t)bh * a.nchunk + job) * (R * R + R), t);
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
  int Hq, Hkv, BHq, nchunk, n_iter;
  float lam1, lam2;
};

// ---- 2. the inverses --------------------------------------------------------------------------
// One workgroup of 8 wavefronts per matrix, all in fp64:
//   query head:  P = B_Q B_Q^T + lambda_d2 A_Om^T A_Om,  c = q B_Q^T + lambda_d2 q K_Om^T A_Om
//   KV head:     N = B_K B_K^T,                          nb = k B_K^T
// The chunk partials of launch 1 are added in chunk order.  The matrix lies in 16 x 16 tiles in
// the wavefronts' registers and is inverted in place by Gauss-Jordan elimination with 4 x 4 pivot
// blocks, one MFMA per tile and step (lrqk_alg64.h).  Latency bound: r / 4 steps, each an exchange
// through LDS, two reciprocals and the MFMAs.
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
  const int m = blockIdx.x;
  const bool isq = m < a.BHq;
  const size_t head = isq ? m : m - a.BHq;
  const float* __restrict__ Bm = (isq ? a.B_Q : a.B_K) + head * R * kD;
  const float* __restrict__ part = a.gram_om + head * a.nchunk * (size_t)(kEntries + R);
  const int tr = w * Z::TPW / Z::RT, tc0 = w * Z::TPW % Z::RT;
  const bool own = tr < Z::RT;          // (r <= 32: the other wavefronts own no tile)
  const int k = lane >> 4, c16 = lane & 15;

  constexpr int NB4 = R * kD / 4, NB = (NB4 + kInvThreads - 1) / kInvThreads;
  float4 bv[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
    bv[j] = reinterpret_cast<const float4*>(Bm)[min(t + kInvThreads * j, NB4 - 1)];
  double xv = 0.0;
  if (t < kD)
    xv = isq ? a.q[head * kD + t]
             : kv_load<BF16>(static_cast<const char*>(a.k_new) + head * ROWB, t);
  f64x4 d[Z::TPW];
#pragma unroll
  for (int u = 0; u < Z::TPW; ++u) d[u] = f64x4{0.0, 0.0, 0.0, 0.0};
  if (isq && own) {
    constexpr int SB = 16 / Z::TPW;  // chunks whose loads are in flight together
    for (int s0 = 0; s0 < a.nchunk; s0 += SB) {
      float x[SB][Z::TPW][4];
#pragma unroll
      for (int sc = 0; sc < SB; ++sc)
#pragma unroll
        for (int u = 0; u < Z::TPW; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            x[sc][u][v] = part[(size_t)min(s0 + sc, a.nchunk - 1) * (kEntries + R) +
                               (16 * tr + 4 * v + k) * R + 16 * (tc0 + u) + c16];
#pragma unroll
      for (int sc = 0; sc < SB; ++sc)
#pragma unroll
        for (int u = 0; u < Z::TPW; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v) d[u][v] += s0 + sc < a.nchunk ? (double)x[sc][u][v] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < Z::TPW; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) d[u][v] *= (double)a.lam2;
  }
  if (t < kD) xs[t] = xv;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int e = 4 * (t + kInvThreads * j);
    if (e < R * kD) {
      double* x = X + e / kD * kLdb + e % kD;
      x[0] = bv[j].x; x[1] = bv[j].y; x[2] = bv[j].z; x[3] = bv[j].w;
    }
  }
  lds_barrier();
  // c (or nb): 8 lanes a row
  double* const out = a.inv + (size_t)m * (kEntries + R);
  {
    const int row = t >> 3, part8 = t & 7;
    double c = 0.0;
    if (row < R) {
      const double* x = X + row * kLdb + part8;
#pragma unroll
      for (int j = 0; j < kD; j += 8) c = __builtin_fma(x[j], xs[j + part8], c);
      if (isq)
        for (int s = part8; s < a.nchunk; s += 8)
          c = __builtin_fma((double)a.lam2, (double)part[(size_t)s * (kEntries + R) + kEntries + row], c);
    }
    c += dpp_f64<0xB1>(c);   // quad_perm [1,0,3,2]
    c += dpp_f64<0x4E>(c);   // quad_perm [2,3,0,1]
    c += dpp_f64<0x141>(c);  // row_half_mirror
    if (row < R && part8 == 0) out[kEntries + row] = c;
  }
  // += B B^T
  if (own) {
#pragma unroll
    for (int u = 0; u < Z::TPW; ++u) {
      const double* xa = X + (16 * tr + c16) * kLdb + k;
      const double* xb = X + (16 * (tc0 + u) + c16) * kLdb + k;
#pragma unroll 8
      for (int s = 0; s < kD; s += 4) d[u] = mfma_f64(xa[s], xb[s], d[u]);
    }
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
// One workgroup per (batch, KV head), wavefront g < G per query head of the group; lane i holds
// element i of a vector.  With P^-1 and N^-1 at hand a round is products of an r x r matrix with a
// vector (the vector's elements as LDS broadcasts, the matrix symmetric: lane i reads column i):
//   q_hat = m_lq M_rq^-1, M_rq = P + lambda_d1 k_hat^T k_hat a rank-one change of P:
//     z = k_hat P^-1,  v = m_lq P^-1 = y0 + lambda_d1 (q.k) z  (y0 = c P^-1),
//     q_hat = v - z * lambda_d1 (k_hat . v) / (1 + lambda_d1 (k_hat . z))
//   k_hat = rhs M^-1, M = N + lambda_d1 Q^T Q (Q: the group's q_hat as rows) a rank-G change of N:
//     W = Q N^-1,  u = rhs N^-1 = nb N^-1 + lambda_d1 sum_g (q_g.k) w_g,
//     k_hat = u - lambda_d1 s W  with  (I + lambda_d1 W Q^T) s = Q u,
//   a G x G system that every wavefront solves for itself, lane 8 a + b holding element (a, b).
// fp64 throughout, so that the corrections lose nothing.
// Then one gradient step on 1/2 |x_hat B - x|^2 for every B_Q of the group and B_K (App. A.2): with
// e = x_hat B - x the gradient is x_hat^T e and x_hat times it |x_hat|^2 e, so the step length
// <e, |x_hat|^2 e> / | |x_hat|^2 e |^2 is 1 / |x_hat|^2 and a column of B needs nothing from the
// others: a thread per column.  (e = 0 or x_hat = 0: B stays.)
constexpr int kRoundThreads = kMaxG * 64;
template <int R>
struct RoundShape {
  static constexpr int LDV = R + 2;  // LDS row stride of the exchanged vectors: 8 rows, 8 bank groups
  static constexpr size_t lds_bytes =
      ((size_t)R * R + 3 * kMaxG * LDV + kMaxG + kMaxG + 1) * sizeof(double);
};

template <int R, bool BF16>
__global__ __launch_bounds__(kRoundThreads) void factor_rounds_kernel(SolveArgs a) {
  using Z = RoundShape<R>;
  constexpr int kEntries = R * R, LDV = Z::LDV;
  constexpr size_t ROWB = kD * (BF16 ? 2 : 4);
  extern __shared__ __align__(16) double rnd_lds[];
  double* const n_s = rnd_lds;                  // [r][r]  N^-1
  double* const qh_s = n_s + kEntries;          // [8][LDV]  q_hat of the group
  double* const wv_s = qh_s + kMaxG * LDV;      // [8][LDV]  q_hat N^-1
  double* const vec_s = wv_s + kMaxG * LDV;     // [8][LDV]  one vector per wavefront
  double* const qk_s = vec_s + kMaxG * LDV;     // [8]
  double* const inv_norm_s = qk_s + kMaxG;      // [9]  1 / |x_hat|^2 of the group's q_hat, of k_hat
  const int t = threadIdx.x, lane = t & 63, g = __builtin_amdgcn_readfirstlane(t >> 6);
  const int G = a.Hq / a.Hkv;
  const int bkv = blockIdx.x, b = bkv / a.Hkv, kvh = bkv - b * a.Hkv;
  const bool act = g < G;
  const int bh = b * a.Hq + kvh * G + (act ? g : 0);
  const bool row = lane < R;
  const int li = row ? lane : 0;  // keeps the loads of idle lanes in bounds
  const double* __restrict__ inv_q = a.inv + (size_t)bh * (kEntries + R);
  const double* __restrict__ inv_k = a.inv + (size_t)(a.BHq + bkv) * (kEntries + R);
  const float* qp = a.q + (size_t)bh * kD;
  const char* kp = static_cast<const char*>(a.k_new) + (size_t)bkv * ROWB;

  double pinv[R];
#pragma unroll
  for (int c = 0; c < R; ++c) pinv[c] = inv_q[c * R + li];
  const double cvec = inv_q[kEntries + li], nb = inv_k[kEntries + li];
  for (int e = t; e < kEntries / 2; e += kRoundThreads)
    reinterpret_cast<double2*>(n_s)[e] = reinterpret_cast<const double2*>(inv_k)[e];
  for (int e = t; e < 2 * kMaxG * LDV; e += kRoundThreads) qh_s[e] = 0.0;  // and wv_s
  const double qk = wave_sum_f64((double)qp[lane] * kv_load<BF16>(kp, lane) +
                                 (double)qp[lane + 64] * kv_load<BF16>(kp, lane + 64));
  if (lane == 0) qk_s[g] = act ? qk : 0.0;
  double* const vec = vec_s + g * LDV;
  const double lam1 = a.lam1;
  // x M of the vector x that lane i holds element i of
  auto put = [&](double x) {
    __builtin_amdgcn_wave_barrier();
    if (row) vec[lane] = x;
    __builtin_amdgcn_wave_barrier();
  };
  auto times_pinv = [&](double x) {
    put(x);
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int c = 0; c < R; c += 2) {
      const double2 v = *reinterpret_cast<const double2*>(vec + c);
      s0 = __builtin_fma(pinv[c], v.x, s0);
      s1 = __builtin_fma(pinv[c + 1], v.y, s1);
    }
    return row ? s0 + s1 : 0.0;
  };
  auto times_ninv = [&](double x) {
    put(x);
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 16
    for (int c = 0; c < R; c += 2) {
      const double2 v = *reinterpret_cast<const double2*>(vec + c);
      s0 = __builtin_fma(n_s[c * R + li], v.x, s0);
      s1 = __builtin_fma(n_s[(c + 1) * R + li], v.y, s1);
    }
    return row ? s0 + s1 : 0.0;
  };
  const double y0 = times_pinv(cvec);
  __syncthreads();  // n_s, qk_s; qh_s and wv_s are zero
  // k0 = nb N^-1, also the initial guess (lambda_d1 = 0): every wavefront an eighth of the sum
  {
    put(nb);
    double s0 = 0.0;
#pragma unroll
    for (int c = 0; c < R / 8; ++c)
      s0 = __builtin_fma(n_s[(g * (R / 8) + c) * R + li], vec[g * (R / 8) + c], s0);
    put(s0);
  }
  lds_barrier();
  double k0 = 0.0;
#pragma unroll
  for (int gg = 0; gg < kMaxG; ++gg) k0 += vec_s[gg * LDV + li];
  if (!row) k0 = 0.0;
  lds_barrier();
  double k_hat = k0, q_hat = 0.0;
  for (int it = 0; it < a.n_iter; ++it) {
    const double z = times_pinv(k_hat);
    const double v = __builtin_fma(lam1 * qk, z, y0);
    const double kv_ = wave_sum_f64(k_hat * v), kz = wave_sum_f64(k_hat * z);
    q_hat = __builtin_fma(-z, lam1 * kv_ / __builtin_fma(lam1, kz, 1.0), v);
    const double wv = times_ninv(q_hat);
    if (it > 0) lds_barrier();  // the previous round's vectors have been read
    if (act && row) {
      qh_s[g * LDV + lane] = q_hat;
      wv_s[g * LDV + lane] = wv;
    }
    lds_barrier();
    double u = k0;
#pragma unroll
    for (int gg = 0; gg < kMaxG; ++gg)
      u = __builtin_fma(lam1 * qk_s[gg], wv_s[gg * LDV + li], u);
    if (!row) u = 0.0;
    put(u);
    const int ra = lane >> 3, cb = lane & 7;
    double kab = 0.0, ta = 0.0;
#pragma unroll 8
    for (int c = 0; c < R; c += 2) {
      const double2 x = *reinterpret_cast<const double2*>(qh_s + ra * LDV + c);
      const double2 y = *reinterpret_cast<const double2*>(wv_s + cb * LDV + c);
      kab = __builtin_fma(x.x, y.x, __builtin_fma(x.y, y.y, kab));
    }
#pragma unroll
    for (int c = 0; c < R; c += 8) ta = __builtin_fma(qh_s[ra * LDV + c + cb], vec[c + cb], ta);
    ta += dpp_f64<0xB1>(ta);
    ta += dpp_f64<0x4E>(ta);
    ta += dpp_f64<0x141>(ta);
    kab = __builtin_fma(lam1, kab, ra == cb ? 1.0 : 0.0);
    // Gauss-Jordan over lanes (rows and columns beyond G are those of the identity, with ta = 0)
    for (int p = 0; p < G; ++p) {
      const double ap = __shfl(kab, ra * 8 + p), pb = __shfl(kab, p * 8 + cb);
      const double tp = __shfl(ta, p * 8), pp = lane_value_f64(kab, p * 9);
      const double f = ra == p ? 0.0 : ap * recip(pp);
      kab = __builtin_fma(-f, pb, kab);
      ta = __builtin_fma(-f, tp, ta);
    }
    const double sa = ta * recip(__shfl(kab, ra * 9));
    k_hat = u;
#pragma unroll
    for (int gg = 0; gg < kMaxG; ++gg)
      k_hat = __builtin_fma(-lam1 * lane_value_f64(sa, 8 * gg), wv_s[gg * LDV + li], k_hat);
    if (!row) k_hat = 0.0;
  }
  if (act && row) a.q_hat[(size_t)bh * R + lane] = (float)q_hat;
  if (g == 0 && row) a.k_hat[(size_t)bkv * R + lane] = (float)k_hat;

  // gradient steps
  const double nq = wave_sum_f64(q_hat * q_hat), nk = wave_sum_f64(k_hat * k_hat);
  if (lane == 0) {
    inv_norm_s[g] = nq > 0.0 ? 1.0 / nq : 0.0;
    if (g == 0) inv_norm_s[kMaxG] = nk > 0.0 ? 1.0 / nk : 0.0;
  }
  if (g == 0) put(k_hat);  // vec_s[0]
  lds_barrier();
  for (int c = t; c < (G + 1) * kD; c += kRoundThreads) {
    const int job = c / kD, col = c % kD;
    const bool isq = job < G;
    const size_t head = isq ? (size_t)b * a.Hq + (size_t)kvh * G + job : bkv;
    float* Bm = (isq ? a.B_Q : a.B_K) + head * R * kD + col;
    const double* xh = isq ? qh_s + job * LDV : vec_s;
    double s0 = -(double)(isq ? a.q[head * kD + col] : kv_load<BF16>(kp, col)), s1 = 0.0;
    // (the column stays in registers between the two uses up to r = 32; at r = 64 it would push
    // P^-1 out of them: 35 us instead of 31)
    constexpr int U = R <= 32 ? R : 16;
    float bv[U];
#pragma unroll 1
    for (int i0 = 0; i0 < R; i0 += U) {
#pragma unroll
      for (int i = 0; i < U; ++i) bv[i] = Bm[(i0 + i) * kD];
#pragma unroll
      for (int i = 0; i < U; i += 2) {
        s0 = __builtin_fma(xh[i0 + i], (double)bv[i], s0);
        s1 = __builtin_fma(xh[i0 + i + 1], (double)bv[i + 1], s1);
      }
    }
    const double step = (s0 + s1) * inv_norm_s[isq ? job : kMaxG];
#pragma unroll 1
    for (int i0 = 0; i0 < R; i0 += U) {
      if (U < R) {
#pragma unroll
        for (int i = 0; i < U; ++i) bv[i] = Bm[(i0 + i) * kD];
      }
#pragma unroll
      for (int i = 0; i < U; ++i)
        Bm[(i0 + i) * kD] = (float)__builtin_fma(-xh[i0 + i], step, (double)bv[i]);
    }
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
  hipLaunchKernelGGL((factor_gram_kernel<R, BF16>), dim3(ga.nchunk, s.B * s.Hq),
                     dim3(kGramThreads), 0, st, ga);
  hipLaunchKernelGGL((factor_inverse_kernel<R, BF16>), dim3(s.B * (s.Hq + s.Hkv)),
                     dim3(kInvThreads), InvShape<R>::lds_bytes, st, sa);
  hipLaunchKernelGGL((factor_rounds_kernel<R, BF16>), dim3(s.B * s.Hkv), dim3(kRoundThreads),
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
  sa.lam1 = lam1; sa.lam2 = lam2;
  const bool bf16 = s.kv_dtype == LRQK_KV_BF16;
  switch (s.r) {
    case 32: return launch_update_dtype<32>(bf16, s, ga, sa, st);
    case 64: return launch_update_dtype<64>(bf16, s, ga, sa, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lrqk
