// Sums over the rows of Omega of a query head, shared by the two forms of the factor update
// (factor_update.hip, factor_update_small.hip):  S = sum_i a_i^T a_i  (r x r)  and  g = sum_i u_i a_i
// (r), a_i = row of A_K, u_i = q . K_i, by workgroups of 256 threads, a chunk of the row list each.
#pragma once

#include "lrqk_device.h"
#include "lrqk_internal.h"

namespace lrqk {
namespace {

constexpr int kGramThreads = 256;
constexpr int kGramBatch = 144;  // rows staged in LDS at a time (a multiple of 16)

template <int CTRL>
__device__ __forceinline__ float fu_dpp(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row16_sum(float v) {
  v += fu_dpp<0x128>(v);  // row_ror:8
  v += fu_dpp<0x124>(v);  // row_ror:4
  v += fu_dpp<0x122>(v);  // row_ror:2
  v += fu_dpp<0x121>(v);  // row_ror:1
  return v;
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __uint_as_float((uint32_t)h << 16);
}
template <bool BF16>
__device__ __forceinline__ float kv_load(const void* row, int j) {
  if (BF16) return bf16_to_f32(static_cast<const uint16_t*>(row)[j]);
  return static_cast<const float*>(row)[j];
}

// q . K_row for the 16 lanes that share a row; lane c of the 16 takes elements 8c .. 8c+7.
// The load and the arithmetic are separate so that a batch of loads can be issued together.
template <bool BF16>
struct RowPiece {
  uint4 lo, hi;  // bf16: lo only
};
template <bool BF16>
__device__ __forceinline__ RowPiece<BF16> load_piece(const void* row, int c) {
  RowPiece<BF16> p;
  if (BF16) {
    p.lo = static_cast<const uint4*>(row)[c];
    p.hi = p.lo;
  } else {
    p.lo = static_cast<const uint4*>(row)[2 * c];
    p.hi = static_cast<const uint4*>(row)[2 * c + 1];
  }
  return p;
}
template <bool BF16>
__device__ __forceinline__ float dot_piece(const RowPiece<BF16>& p, const float (&qv)[8]) {
  float x[8];
  if (BF16) {
    const uint4 u = p.lo;
    x[0] = __uint_as_float(u.x << 16); x[1] = __uint_as_float(u.x & 0xffff0000u);
    x[2] = __uint_as_float(u.y << 16); x[3] = __uint_as_float(u.y & 0xffff0000u);
    x[4] = __uint_as_float(u.z << 16); x[5] = __uint_as_float(u.z & 0xffff0000u);
    x[6] = __uint_as_float(u.w << 16); x[7] = __uint_as_float(u.w & 0xffff0000u);
  } else {
    x[0] = __uint_as_float(p.lo.x); x[1] = __uint_as_float(p.lo.y);
    x[2] = __uint_as_float(p.lo.z); x[3] = __uint_as_float(p.lo.w);
    x[4] = __uint_as_float(p.hi.x); x[5] = __uint_as_float(p.hi.y);
    x[6] = __uint_as_float(p.hi.z); x[7] = __uint_as_float(p.hi.w);
  }
  float acc = 0.0f;
#pragma unroll
  for (int j = 0; j < 8; ++j) acc = __builtin_fmaf(x[j], qv[j], acc);
  return acc;
}

// S += sum_i a_i^T a_i and g += sum_i u_i a_i over the kGramBatch rows staged in LDS (a_s: row
// stride LDA floats, rows past the end are zero), by the 256 threads of a workgroup.
// S is a dense contraction over the rows and goes through v_mfma_f32_32x32x2_f32, whose two
// operands are here the same numbers: lane i + 32 kk supplies A[i][kk] = B[kk][i] = element i
// of row kk of the pair.  r <= 32: one 32 x 32 block (columns >= r read as zero), each
// wavefront sums a quarter of the rows; r = 64: wavefront (bi, bj) owns block (bi, bj) of S
// and sums all the rows.  g: thread t sums column t % r over every (256 / r)-th row.
typedef float f32x16 __attribute__((ext_vector_type(16)));
template <int R>
__device__ __forceinline__ void gram_accumulate(const float* a_s, const float* u_s, f32x16& sacc,
                                                float& gpart, int t) {
  constexpr int LDA = R + 4;
  const int wave = t >> 6, lane = t & 63, li = lane & 31, lk = lane >> 5;
  if constexpr (R <= 32) {
    constexpr int kRows = kGramBatch / 4;  // rows per wavefront
    static_assert(kRows % 2 == 0, "rows are consumed in pairs");
#pragma unroll 6
    for (int i = 0; i < kRows; i += 2) {
      const float x = li < R ? a_s[(wave * kRows + i + lk) * LDA + li] : 0.0f;
      sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(x, x, sacc, 0, 0, 0);
    }
  } else {
    const int bi = wave >> 1, bj = wave & 1;
#pragma unroll 6
    for (int i = 0; i < kGramBatch; i += 2) {
      const float xa = a_s[(i + lk) * LDA + 32 * bi + li];
      const float xb = a_s[(i + lk) * LDA + 32 * bj + li];
      sacc = __builtin_amdgcn_mfma_f32_32x32x2f32(xa, xb, sacc, 0, 0, 0);
    }
  }
  constexpr int kSub = kGramThreads / R;
  const int gc = t % R;
#pragma unroll 4
  for (int i = t / R; i < kGramBatch; i += kSub) gpart = __builtin_fmaf(u_s[i], a_s[i * LDA + gc], gpart);
}

template <int R>
struct GramLds {
  static constexpr int LDA = R + 4;  // padded LDS row, keeps 16-byte alignment
  alignas(16) float a[kGramBatch * LDA];
  // r <= 32: the partial blocks of wavefronts 1..3; then the partial sums of g
  float red[R <= 32 ? 3 * 1024 : kGramThreads];
  float u[kGramBatch];
  int pos[kGramBatch];
  const char* krow[kGramBatch];
};

// The rows of Omega.
struct GramRows {
  const float* A_K;              // [B,Hkv,l_rows,r]
  const void* cacheK;            // [B,Hq,C,d]
  const void* liteK;             // [B,Hkv,w,d], row j holds the position p of [l-w,l), p % w == j
  const int32_t* sel_idx_prev;   // [B,Hq,k]
  const int32_t* sel_slot_prev;  // [B,Hq,k]
  const float* q;                // [B,Hq,d]
  float* gram_om;                // [B*Hq][nchunk][r*r + r]
  int Hq, Hkv, l, l_rows, k, w, C, nchunk, chunk_rows;
};

// Chunk `job` of query head bh, KV head bkv.
template <int R, bool BF16>
__device__ __forceinline__ void gram_chunk(const GramRows& a, GramLds<R>& s, int bh, int bkv, int job,
                                           f32x16& sacc, float& gpart, int t) {
  constexpr int LDA = GramLds<R>::LDA;
  constexpr size_t ROWB = kD * (BF16 ? 2 : 4);
  const int n_om = a.k + a.w;
  const int i_begin = job * a.chunk_rows;
  const int i_end = min(n_om, i_begin + a.chunk_rows);
  const float* __restrict__ Ahead = a.A_K + (size_t)bkv * (size_t)a.l_rows * R;
  const char* Kc = static_cast<const char*>(a.cacheK) + (size_t)bh * a.C * ROWB;
  const char* Kl = static_cast<const char*>(a.liteK) + (size_t)bkv * a.w * ROWB;
  const int c16 = t & 15, rsub = t >> 4;
  float qv[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) qv[j] = a.q[(size_t)bh * kD + c16 * 8 + j];
  const char* qrow = reinterpret_cast<const char*>(a.q + (size_t)bh * kD);
  const int lite0 = a.l - a.w;  // first position of the lite window
  for (int i0 = i_begin; i0 < i_end; i0 += kGramBatch) {
    __syncthreads();  // the previous batch has been consumed
    if (t < kGramBatch) {
      const int i = i0 + t;
      int pos = -1;
      const char* krow = nullptr;
      if (i < i_end) {
        if (i < a.k) {
          const int tok = a.sel_idx_prev[(size_t)bh * a.k + i];
          const int slot = a.sel_slot_prev[(size_t)bh * a.k + i];
          if (tok >= 0 && tok < a.l && slot >= 0 && slot < a.C) {
            pos = tok;
            krow = Kc + (size_t)slot * ROWB;
          }
        } else {
          const int j = i - a.k;  // row of the lite ring
          // the position in [l-w, l) that is congruent to j modulo w
          int off = (j - lite0) % a.w;
          if (off < 0) off += a.w;
          pos = lite0 + off;
          krow = Kl + (size_t)j * ROWB;
        }
      }
      s.pos[t] = pos;
      s.krow[t] = krow;
    }
    __syncthreads();
    // All the loads of the batch are issued before anything waits for one of them; rows
    // that do not exist read memory that does (the head's q, which is at least as long as
    // a K row; row 0 of A_K) and are zeroed afterwards.
    // u_i = q . K_i: 16 lanes per row, 16 rows per pass
    constexpr int kPasses = kGramBatch / 16;
    RowPiece<BF16> piece[kPasses];
#pragma unroll
    for (int pass = 0; pass < kPasses; ++pass) {
      const char* krow = s.krow[pass * 16 + rsub];
      piece[pass] = load_piece<BF16>(krow ? krow : qrow, c16);
    }
    // a_i = A_K[pos_i, :]
    constexpr int kAPieces = (kGramBatch * (R / 4) + kGramThreads - 1) / kGramThreads;
    float4 av[kAPieces];
#pragma unroll
    for (int u = 0; u < kAPieces; ++u) {
      const int idx = t + u * kGramThreads;
      const int rr = min(idx / (R / 4), kGramBatch - 1), c4 = idx % (R / 4);
      const int pos = s.pos[rr];
      av[u] = reinterpret_cast<const float4*>(Ahead + (size_t)max(pos, 0) * R)[c4];
      if (pos < 0) av[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int pass = 0; pass < kPasses; ++pass) {
      const int rr = pass * 16 + rsub;
      float dot = s.krow[rr] ? dot_piece<BF16>(piece[pass], qv) : 0.0f;
      dot = row16_sum(dot);
      if (c16 == 0) s.u[rr] = dot;
    }
#pragma unroll
    for (int u = 0; u < kAPieces; ++u) {
      const int idx = t + u * kGramThreads;
      if (idx < kGramBatch * (R / 4))
        *reinterpret_cast<float4*>(&s.a[idx / (R / 4) * LDA + 4 * (idx % (R / 4))]) = av[u];
    }
    __syncthreads();
    gram_accumulate<R>(s.a, s.u, sacc, gpart, t);
  }
}

// The sums of the workgroup's wavefronts added up and written to out [r*r + r].
template <int R>
__device__ __forceinline__ void gram_store(GramLds<R>& s, const f32x16& sacc, float gpart, float* out,
                                           int t) {
  constexpr int kEntries = R * R;
  // Register v of lane l of an accumulator holds element [8 (v / 4) + 4 (l / 32) + v % 4][l % 32]
  // of its block.
  const int wave = t >> 6, lane = t & 63;
  if constexpr (R <= 32) {
    __syncthreads();
    if (wave > 0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) s.red[(wave - 1) * 1024 + v * 64 + lane] = sacc[v];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float sum = ((sacc[v] + s.red[v * 64 + lane]) + s.red[1024 + v * 64 + lane]) +
                          s.red[2048 + v * 64 + lane];
        const int pr = 8 * (v / 4) + 4 * (lane >> 5) + v % 4, qc = lane & 31;
        if (pr < R && qc < R) out[pr * R + qc] = sum;
      }
    }
  } else {
    const int bi = wave >> 1, bj = wave & 1;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int pr = 32 * bi + 8 * (v / 4) + 4 * (lane >> 5) + v % 4, qc = 32 * bj + (lane & 31);
      out[pr * R + qc] = sacc[v];
    }
  }
  __syncthreads();
  s.red[t] = gpart;
  __syncthreads();
  if (t < R) {
    float g = 0.0f;
    for (int sub = 0; sub < kGramThreads / R; ++sub) g += s.red[sub * R + t];
    out[kEntries + t] = g;
  }
}

}  // namespace
}  // namespace lrqk
