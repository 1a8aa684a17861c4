// u1 — decode-time update of the factors (Alg. 2 from the initial guess of k_hat to the
// two gradient steps; Sec. 4.2 update rules for q_hat_t, k_hat_t, B_Q, B_K; App. A.2 optimal
// step lengths), r = 8 and 16.
//
// Two launches.
//
//  1. factor_gram_kernel: everything that is a sum over many rows.  For a list of rows a_i
//     (r floats each) with weights u_i it produces  S = sum_i a_i^T a_i  (r x r)  and
//     g = sum_i u_i a_i  (r).  Three kinds of jobs share the code:
//       * Omega of a query head (the k rows selected at the previous step, read from their
//         cache slots, and the w lite rows): a_i = row of A_K, u_i = q . K_i.  This gives
//         A_Om^T A_Om and q K_Om^T A_Om.  The row list of a head is cut into chunks of at most
//         144 rows, one workgroup each, so that batch-1 steps still use hundreds of CUs; K rows
//         are read by 16 lanes each exactly as the attention kernel reads them;
//       * B_Q of a query head, read column-wise: a_i = column i of B_Q, u_i = q_i, which
//         gives B_Q B_Q^T and q B_Q^T;
//       * B_K of a KV head with u = k_t: B_K B_K^T and k B_K^T.
//     The chunk's rows are staged in LDS and summed on the matrix cores (update_gram.h); partial
//     sums per chunk go to the workspace and are added up, in chunk order, by the second kernel:
//     no atomics, the result does not depend on scheduling.
//
//  2. factor_solve_kernel: one workgroup per (batch, KV head), one wavefront per query
//     head of the group.  The r x r systems are solved inside a wavefront: lane i
//     holds row i of the matrix in registers, a right-looking Cholesky factorisation takes
//     column j from lane registers with v_readlane (all register indices are compile-time
//     constants), the two triangular solves follow the same pattern, with one transpose of
//     the factor through LDS in between.  Only what changes between rounds is factorised
//     again: M_rq = P + lambda_d1 k_hat^T k_hat differs from the fixed
//     P = B_Q B_Q^T + lambda_d2 A_Om^T A_Om by a rank-one term, so P is factorised once and
//     each q_hat costs one pair of triangular solves (Sherman-Morrison); the k_hat system
//     changes by a rank-G term and is factorised anew each round.  The alternating updates
//     of q_hat (per query head) and k_hat (per KV head, summed over the group's heads)
//     exchange q_hat through LDS; every wavefront solves the k_hat system redundantly, which
//     is cheaper than a second exchange.  The same kernel then applies the two rank-one
//     gradient steps to B_Q and B_K in place.
//
// All arithmetic is fp32 (App. B.1 runs these updates in fp32).
//
// For r <= 16.  There the chain of a factorisation is short and what counts is the number of
// launches and exchanges: these two launches take 14.4 us at r = 8 and 17.2 us at r = 16 (32 + 8
// heads, k = 256), inverses in fp64 inside the rounds' launch 20.5 and 24.7 us (in a launch of
// their own: 20.3 where these take 16.2).  From r = 32 on it is the other way round (28.4 against
// 25.9 us at 16 + 8 heads, k = 200;
// 44.0 against 29.6 us at 28 + 4 heads, k = 600; r = 64: 118 against 59 us): factor_update.hip.
#include "lrqk_device.h"
#include "lrqk_internal.h"
#include "lrqk_linalg.h"
#include "update_gram.h"

namespace lrqk {
namespace {

using namespace linalg;

__device__ __forceinline__ float wave_sum(float v) {
  v = row16_sum(v);
  // the four 16-lane rows of the wavefront
  const float a = __shfl(v, 0), b = __shfl(v, 16), c = __shfl(v, 32), e = __shfl(v, 48);
  return (a + b) + (c + e);
}

struct GramArgs : GramRows {
  const void* k_new;  // [B,Hkv,d]
  const float* B_Q;   // [B,Hq,r,d]
  const float* B_K;   // [B,Hkv,r,d]
  float* gram_q;      // [B*Hq][r*r + r]
  float* gram_k;      // [B*Hkv][r*r + r]
};

template <int R, bool BF16>
__global__ __launch_bounds__(kGramThreads) void factor_gram_kernel(GramArgs a) {
  constexpr int kEntries = R * R, LDA = GramLds<R>::LDA;
  constexpr size_t ROWB = kD * (BF16 ? 2 : 4);
  __shared__ GramLds<R> s;
  const int bh = blockIdx.y, job = blockIdx.x, t = threadIdx.x;
  const int b = bh / a.Hq, h = bh - b * a.Hq;
  const int G = a.Hq / a.Hkv;
  const int kvh = h / G;
  const int bkv = b * a.Hkv + kvh;
  if (job == a.nchunk + 1 && h != kvh * G) return;  // the B_K job runs once per KV head

  GramAcc<R> acc;
  float gpart;

  float* out;
  if (job < a.nchunk) {
    out = a.gram_om + ((size_t)bh * a.nchunk + job) * (kEntries + R);
    gram_chunk<R, BF16>(a, s, bh, bkv, job, acc, gpart, t);
  } else {
    // ---- B_Q of this query head, or B_K of this KV head, read column by column ------------
    const bool isq = job == a.nchunk;
    out = isq ? a.gram_q + (size_t)bh * (kEntries + R) : a.gram_k + (size_t)bkv * (kEntries + R);
    const float* __restrict__ Bm =
        isq ? a.B_Q + (size_t)bh * R * kD : a.B_K + (size_t)bkv * R * kD;
    static_assert(kD <= kGramBatch, "one batch");
    if (t < kGramBatch) {
      float u = 0.0f;
      if (t < kD)
        u = isq ? a.q[(size_t)bh * kD + t]
                : kv_load<BF16>(static_cast<const char*>(a.k_new) + (size_t)bkv * ROWB, t);
      s.u[t] = u;
    }
    // every load is issued before the first is waited for (addresses clamped, the values
    // past the end zeroed)
    constexpr int kBPieces = (kGramBatch * R + kGramThreads - 1) / kGramThreads;
    float bv[kBPieces];
#pragma unroll
    for (int u = 0; u < kBPieces; ++u) {
      const int idx = t + u * kGramThreads;
      const int c = min(idx / kGramBatch, R - 1), ii = idx % kGramBatch;
      bv[u] = Bm[(size_t)c * kD + min(ii, kD - 1)];
      if (ii >= kD) bv[u] = 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kBPieces; ++u) {
      const int idx = t + u * kGramThreads;
      if (idx < kGramBatch * R) s.a[idx % kGramBatch * LDA + idx / kGramBatch] = bv[u];
    }
    __syncthreads();
    gram_accumulate<R>(s.a, s.u, acc, gpart, t);
  }
  gram_store<R>(s, acc, gpart, out, t);
}

struct SolveArgs {
  const float* gram_om;  // [B*Hq][nchunk][r*r + r]
  const float* gram_q;   // [B*Hq][r*r + r]
  const float* gram_k;   // [B*Hkv][r*r + r]
  const float* q;        // [B,Hq,d]
  const void* k_new;     // [B,Hkv,d]
  float* B_Q;            // [B,Hq,r,d]   updated in place
  float* B_K;            // [B,Hkv,r,d]  updated in place
  float* q_hat;          // [B,Hq,r]
  float* k_hat;          // [B,Hkv,r]
  int Hq, Hkv, nchunk, n_iter;
  float lam1, lam2;
};

// One exact line-search gradient step on 1/2 |x_hat B - x|^2 (App. A.2), by one wavefront:
//   resid = x_hat B - x,  grad = x_hat^T resid,  eta = <resid, x_hat grad> / |x_hat grad|^2,
//   B <- B - eta grad.  Lane i (< R) holds x_hat_i; x(j) returns element j of the target.
template <int R, typename XF>
__device__ __forceinline__ void line_search_step(float xh, float* __restrict__ Bm, XF x, int lane) {
  const float xhz = lane < R ? xh : 0.0f;
  const float nrm2 = wave_sum(xhz * xhz);
  // this lane's two columns of the residual
  float e0 = -x(lane), e1 = -x(lane + 64);
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const float xi = lane_value(xh, i);
    e0 = __builtin_fmaf(xi, Bm[(size_t)i * kD + lane], e0);
    e1 = __builtin_fmaf(xi, Bm[(size_t)i * kD + lane + 64], e1);
  }
  // x_hat grad = |x_hat|^2 resid
  const float v0 = nrm2 * e0, v1 = nrm2 * e1;
  const float num = wave_sum(e0 * v0 + e1 * v1);
  const float den = wave_sum(v0 * v0 + v1 * v1);
  const float eta = den > 0.0f ? num / den : 0.0f;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const float s = eta * lane_value(xh, i);
    Bm[(size_t)i * kD + lane] = __builtin_fmaf(-s, e0, Bm[(size_t)i * kD + lane]);
    Bm[(size_t)i * kD + lane + 64] = __builtin_fmaf(-s, e1, Bm[(size_t)i * kD + lane + 64]);
  }
}

template <int R, bool BF16>
__global__ __launch_bounds__(kMaxG * 64) void factor_solve_kernel(SolveArgs a) {
  constexpr int kEntries = R * R;
  constexpr size_t ROWB = kD * (BF16 ? 2 : 4);
  extern __shared__ __align__(16) float lds[];
  const int G = a.Hq / a.Hkv;
  constexpr int NLD = R + 4;  // padded row of the LDS copy of N
  // [G][R*(R+1)] transpose space | [R][NLD] N = B_K B_K^T | [G][R] q_hat exchange | [G] q.k
  float* const lt = lds + (size_t)(threadIdx.x >> 6) * R * (R + 1);
  float* const n_s = lds + ((size_t)G * R * (R + 1) + 3) / 4 * 4;
  float* const qhat_s = n_s + R * NLD;
  float* const qk_s = qhat_s + G * R;

  const int bkv = blockIdx.x;
  const int b = bkv / a.Hkv, kvh = bkv - b * a.Hkv;
  const int g = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int bh = b * a.Hq + kvh * G + g;
  const bool row = lane < R;
  const int li = row ? lane : 0;  // keeps the loads of idle lanes in bounds
  const float* qp = a.q + (size_t)bh * kD;
  const char* kp = static_cast<const char*>(a.k_new) + (size_t)bkv * ROWB;
  const float qk_part = qp[lane] * kv_load<BF16>(kp, lane) +
                        qp[lane + 64] * kv_load<BF16>(kp, lane + 64);
  // P = B_Q B_Q^T + lambda_d2 A_Om^T A_Om,  cvec = q B_Q^T + lambda_d2 q K_Om^T A_Om;
  // N = B_K B_K^T,  nb = k B_K^T.  The chunk partials are added in chunk order.  They are
  // read with consecutive lanes on consecutive 16-byte pieces and turned into "lane = row"
  // through LDS.
  float p[R], pt[R], m[R];
  float cvec, nb;
  {
    constexpr int U = (kEntries / 4 + 63) / 64;  // 16-byte pieces of an r x r matrix per lane
    const float* gq = a.gram_q + (size_t)bh * (kEntries + R);
    const float* gk = a.gram_k + (size_t)bkv * (kEntries + R);
    constexpr bool kHoist = U <= 4;  // large r: too many registers to hold them that long
    float4 acc[U], vq[U], vk[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      const int e4 = lane + 64 * u;  // issued first: these loads overlap the first round below
      const bool on = kHoist && e4 < kEntries / 4;
      vq[u] = on ? reinterpret_cast<const float4*>(gq)[e4] : acc[u];
      vk[u] = (on && g == 0) ? reinterpret_cast<const float4*>(gk)[e4] : acc[u];
    }
    const float cq = gq[kEntries + li];
    nb = gk[kEntries + li];
    float gsum = 0.0f;
    // chunks whose loads are in flight together (the partials were written by the previous
    // kernel and come from memory, so each round of loads costs a full memory latency)
    constexpr int SB = U >= 16 ? 2 : (U >= 4 ? 8 : 16);
    const float* go0 = a.gram_om + (size_t)bh * a.nchunk * (kEntries + R);
    for (int s0 = 0; s0 < a.nchunk; s0 += SB) {
      float4 v[SB][U];
      float gv[SB];
#pragma unroll
      for (int j = 0; j < SB; ++j) {
        const bool on = s0 + j < a.nchunk;
        const float* go = go0 + (size_t)(on ? s0 + j : s0) * (kEntries + R);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int e4 = lane + 64 * u;
          v[j][u] = (on && e4 < kEntries / 4) ? reinterpret_cast<const float4*>(go)[e4]
                                              : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        gv[j] = on ? go[kEntries + li] : 0.0f;
      }
#pragma unroll
      for (int j = 0; j < SB; ++j) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          acc[u].x += v[j][u].x; acc[u].y += v[j][u].y;
          acc[u].z += v[j][u].z; acc[u].w += v[j][u].w;
        }
        gsum += gv[j];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e4 = lane + 64 * u;
      if (e4 < kEntries / 4) {
        if (!kHoist) {
          vq[u] = reinterpret_cast<const float4*>(gq)[e4];
          if (g == 0) vk[u] = reinterpret_cast<const float4*>(gk)[e4];
        }
        const int e = 4 * e4, rr = e / R, cc = e % R;
        lt[rr * (R + 1) + cc + 0] = __builtin_fmaf(a.lam2, acc[u].x, vq[u].x);
        lt[rr * (R + 1) + cc + 1] = __builtin_fmaf(a.lam2, acc[u].y, vq[u].y);
        lt[rr * (R + 1) + cc + 2] = __builtin_fmaf(a.lam2, acc[u].z, vq[u].z);
        lt[rr * (R + 1) + cc + 3] = __builtin_fmaf(a.lam2, acc[u].w, vq[u].w);
        if (g == 0) *reinterpret_cast<float4*>(&n_s[rr * NLD + cc]) = vk[u];
      }
    }
    cvec = __builtin_fmaf(a.lam2, gsum, cq);
    __syncthreads();  // n_s (and, within the wavefront, lt) is complete
#pragma unroll
    for (int c = 0; c < R; ++c) p[c] = lt[li * (R + 1) + c];
#pragma unroll
    for (int c4 = 0; c4 < R / 4; ++c4) {
      const float4 vk = *reinterpret_cast<const float4*>(&n_s[li * NLD + 4 * c4]);
      m[4 * c4 + 0] = vk.x; m[4 * c4 + 1] = vk.y; m[4 * c4 + 2] = vk.z; m[4 * c4 + 3] = vk.w;
    }
  }

  // q . k of this query head
  const float qk = wave_sum(qk_part);
  if (lane == 0) qk_s[g] = qk;
  // Factorise N (for the initial guess) and P (kept for every round) together.
  float dN, dP;
  chol_factor2<R>(m, p, dN, dP, lane);
  // initial guess (lambda_d1 = 0): k_hat = k B_K^T (B_K B_K^T)^-1
  float k_hat = tri_forward<R>(m, dN, nb, lane);
  transpose_rows<R>(m, m, lt, lane);
  k_hat = tri_backward<R>(m, dN, k_hat, lane);
  // y0 = cvec P^-1
  transpose_rows<R>(p, pt, lt, lane);
  const float y0 = tri_backward<R>(pt, dP, tri_forward<R>(p, dP, cvec, lane), lane);
  float q_hat = 0.0f;
  for (int it = 0; it < a.n_iter; ++it) {
    // q_hat = m_lq M_rq^-1 with M_rq = P + lambda_d1 k_hat^T k_hat a rank-one change of P:
    //   z = k_hat P^-1,  v = m_lq P^-1 = y0 + lambda_d1 (q.k) z,
    //   q_hat = v - z * lambda_d1 (k_hat . v) / (1 + lambda_d1 (k_hat . z))
    const float z = tri_backward<R>(pt, dP, tri_forward<R>(p, dP, k_hat, lane), lane);
    const float v = __builtin_fmaf(a.lam1 * qk, z, y0);
    const float kv_ = wave_sum(row ? k_hat * v : 0.0f);
    const float kz = wave_sum(row ? k_hat * z : 0.0f);
    q_hat = __builtin_fmaf(-z, a.lam1 * kv_ / __builtin_fmaf(a.lam1, kz, 1.0f), v);
    __syncthreads();  // the previous round's q_hat has been read by every wavefront
    if (row) qhat_s[g * R + lane] = q_hat;
    __syncthreads();
    // k_hat = (k B_K^T + lambda_d1 sum_g (q_g.k) q_hat_g)
    //         (B_K B_K^T + lambda_d1 sum_g q_hat_g^T q_hat_g)^-1
    float rhs = nb;
#pragma unroll
    for (int c4 = 0; c4 < R / 4; ++c4) {
      const float4 vk = *reinterpret_cast<const float4*>(&n_s[li * NLD + 4 * c4]);
      m[4 * c4 + 0] = vk.x; m[4 * c4 + 1] = vk.y; m[4 * c4 + 2] = vk.z; m[4 * c4 + 3] = vk.w;
    }
    for (int gg = 0; gg < G; ++gg) {
      const float qi = qhat_s[gg * R + li];
      rhs = __builtin_fmaf(a.lam1 * qk_s[gg], qi, rhs);
#pragma unroll
      for (int c = 0; c < R; ++c) m[c] = __builtin_fmaf(a.lam1 * qi, qhat_s[gg * R + c], m[c]);
    }
    const float dM = chol_factor<R>(m, lane);
    k_hat = tri_forward<R>(m, dM, rhs, lane);
    transpose_rows<R>(m, m, lt, lane);
    k_hat = tri_backward<R>(m, dM, k_hat, lane);
  }
  if (row) a.q_hat[(size_t)bh * R + lane] = q_hat;
  if (row && g == 0) a.k_hat[(size_t)bkv * R + lane] = k_hat;

  // gradient steps on B_Q (every wavefront its head) and B_K (the first wavefront)
  line_search_step<R>(q_hat, a.B_Q + (size_t)bh * R * kD, [&](int j) { return qp[j]; }, lane);
  if (g == 0)
    line_search_step<R>(k_hat, a.B_K + (size_t)bkv * R * kD,
                        [&](int j) { return kv_load<BF16>(kp, j); }, lane);
}

template <int R, bool BF16>
hipError_t launch_update_r(const lrqk_shape& s, const GramArgs& ga, const SolveArgs& sa,
                           hipStream_t st) {
  const int G = s.Hq / s.Hkv;
  hipLaunchKernelGGL((factor_gram_kernel<R, BF16>), dim3(ga.nchunk + 2, s.B * s.Hq),
                     dim3(kGramThreads), 0, st, ga);
  const size_t lds =
      (((size_t)G * R * (R + 1) + 3) / 4 * 4 + (size_t)R * (R + 4) + (size_t)G * R + G) *
      sizeof(float);
  hipLaunchKernelGGL((factor_solve_kernel<R, BF16>), dim3(s.B * s.Hkv), dim3(G * 64), lds, st,
                     sa);
  return hipGetLastError();
}

template <int R>
hipError_t launch_update_dtype(bool bf16, const lrqk_shape& s, const GramArgs& ga,
                               const SolveArgs& sa, hipStream_t st) {
  return bf16 ? launch_update_r<R, true>(s, ga, sa, st) : launch_update_r<R, false>(s, ga, sa, st);
}

}  // namespace

size_t update_small_ws_bytes(const lrqk_shape& s) {
  const UpdateGeom g = update_geometry(s);
  const size_t BHq = (size_t)s.B * s.Hq, BHkv = (size_t)s.B * s.Hkv;
  return round_up((BHq * g.nchunk + BHq + BHkv) * g.per_gram * sizeof(float), 256);
}

hipError_t launch_factor_update_small(const lrqk_shape& s, const float* A_K, const void* cacheK,
                                const void* liteK, const int32_t* sel_idx_prev,
                                const int32_t* sel_slot_prev, const float* q, const void* k_new,
                                float* B_Q, float* B_K, float lam1, float lam2, int n_iter,
                                float* q_hat, float* k_hat, float* ws, hipStream_t st) {
  const UpdateGeom g = update_geometry(s);
  const size_t BHq = (size_t)s.B * s.Hq;
  GramArgs ga;
  ga.A_K = A_K; ga.cacheK = cacheK; ga.liteK = liteK;
  ga.sel_idx_prev = sel_idx_prev; ga.sel_slot_prev = sel_slot_prev;
  ga.q = q; ga.k_new = k_new; ga.B_Q = B_Q; ga.B_K = B_K;
  ga.gram_om = ws;
  ga.gram_q = ws + BHq * g.nchunk * g.per_gram;
  ga.gram_k = ga.gram_q + BHq * g.per_gram;
  ga.Hq = s.Hq; ga.Hkv = s.Hkv; ga.l = s.l; ga.l_rows = row_cap(s); ga.k = s.k; ga.w = s.w; ga.C = s.C;
  ga.nchunk = g.nchunk; ga.chunk_rows = g.chunk_rows;
  SolveArgs sa;
  sa.gram_om = ga.gram_om; sa.gram_q = ga.gram_q; sa.gram_k = ga.gram_k;
  sa.q = q; sa.k_new = k_new; sa.B_Q = B_Q; sa.B_K = B_K; sa.q_hat = q_hat; sa.k_hat = k_hat;
  sa.Hq = s.Hq; sa.Hkv = s.Hkv; sa.nchunk = g.nchunk; sa.n_iter = n_iter;
  sa.lam1 = lam1; sa.lam2 = lam2;
  const bool bf16 = s.kv_dtype == LRQK_KV_BF16;
  switch (s.r) {
    case 8: return launch_update_dtype<8>(bf16, s, ga, sa, st);
    case 16: return launch_update_dtype<16>(bf16, s, ga, sa, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lrqk
