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

// S = sum_i a_i^T a_i and g = sum_i u_i a_i over the kGramBatch rows staged in LDS (a_s: row
// stride LDA floats, rows past the end are zero), by the 256 threads of a workgroup.
// S is a dense contraction over the rows.  r <= 32: one 32 x 32 block (columns >= r read as zero) by
// v_mfma_f32_32x32x2_f32, whose two operands are here the same numbers: lane i + 32 kk supplies
// A[i][kk] = B[kk][i] = element i of row kk of the pair; each wavefront sums a quarter of the rows.
// r = 64: blocks (0, 0), (0, 1) and (1, 1) by v_mfma_f32_32x32x16_bf16, every number as three bf16 terms
// and the six products of terms down to 2^-16 of the leading one (what is left out is 2^-24 of a product
// and smaller, as the rounding of an fp32 sum), the small ones first; a wavefront sums every fourth 16 rows.
// 18 MFMAs of 32 cycles for 16 rows instead of 32 of 64 cycles in fp32, and fewer roundings: at 8 x (28 + 4)
// heads, k = 1024 the kernel takes 31 us instead of 38 (24 would be its bytes; calls back to back on the same
// inputs, 37 on four sets of inputs in turn), and the update's results are 1.2e-7 instead of 1.7e-7 from those in
// 64 bits.  (Of an entry of a diagonal block and its mirror image two products swap places, so that the two may
// differ in their last bits.)
// g: thread t sums column t % r over every (256 / r)-th row.
using dev::bf16x8;
using dev::f32x16;
template <int R>
struct GramAcc {
  f32x16 s[R <= 32 ? 1 : 3];
};
template <int R>
struct GramRow {
  static constexpr int LDA = R <= 32 ? R + 4 : R;  // floats of an LDS row; 16-byte aligned
};
template <int R>
__device__ __forceinline__ void gram_accumulate(const float* a_s, const float* u_s, GramAcc<R>& acc,
                                                float& gpart, int t) {
  constexpr int LDA = GramRow<R>::LDA;
  const int wave = t >> 6, lane = t & 63, li = lane & 31, lk = lane >> 5;
  acc = {};
  gpart = 0.0f;
  if constexpr (R <= 32) {
    constexpr int kRows = kGramBatch / 4;  // rows per wavefront
    static_assert(kRows % 2 == 0, "rows are consumed in pairs");
#pragma unroll 6
    for (int i = 0; i < kRows; i += 2) {
      const float x = li < R ? a_s[(wave * kRows + i + lk) * LDA + li] : 0.0f;
      acc.s[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, x, acc.s[0], 0, 0, 0);
    }
  } else {
    static_assert(kGramBatch % 16 == 0, "whole steps");
#pragma unroll 1
    for (int row0 = 16 * wave; row0 < kGramBatch; row0 += 64) {
      bf16x8 x[2][3];  // lane i + 32 h: rows row0 + 8 h .. of column i of a block, three terms
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const float* p = a_s + (row0 + 8 * lk) * LDA + 32 * b + li;
        uint32_t w[4][3];
#pragma unroll
        for (int j = 0; j < 4; ++j) dev::split3(p[2 * j * LDA], p[(2 * j + 1) * LDA], w[j]);
#pragma unroll
        for (int k = 0; k < 3; ++k)
          x[b][k] = __builtin_bit_cast(bf16x8, (dev::u32x4{w[0][k], w[1][k], w[2][k], w[3][k]}));
      }
      constexpr int kI[6] = {2, 0, 1, 1, 0, 0}, kJ[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int n = 0; n < 6; ++n) {
        acc.s[0] = dev::mfma_bf16(x[0][kI[n]], x[0][kJ[n]], acc.s[0]);
        acc.s[1] = dev::mfma_bf16(x[0][kI[n]], x[1][kJ[n]], acc.s[1]);
        acc.s[2] = dev::mfma_bf16(x[1][kI[n]], x[1][kJ[n]], acc.s[2]);
      }
    }
  }
  constexpr int kSub = kGramThreads / R;
  const int gc = t % R;
#pragma unroll 4
  for (int i = t / R; i < kGramBatch; i += kSub) gpart = __builtin_fmaf(u_s[i], a_s[i * LDA + gc], gpart);
}

template <int R>
struct GramLds {
  static constexpr int LDA = GramRow<R>::LDA;
  alignas(16) float a[kGramBatch * LDA];  // r = 64: then nine blocks of the wavefronts' sums
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
                                           GramAcc<R>& acc, float& gpart, int t) {
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
  // (a chunk is one batch at most)
  if (t < kGramBatch) {
    const int i = i_begin + t;
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
  gram_accumulate<R>(s.a, s.u, acc, gpart, t);
}

// The sums of the workgroup's wavefronts added up and written to out [r*r + r].
template <int R>
__device__ __forceinline__ void gram_store(GramLds<R>& s, GramAcc<R>& acc, float gpart, float* out,
                                           int t) {
  constexpr int kEntries = R * R;
  // Register v of lane l of an accumulator holds element [8 (v / 4) + 4 (l / 32) + v % 4][l % 32]
  // of its block.
  const int wave = t >> 6, lane = t & 63;
  if constexpr (R <= 32) {
    __syncthreads();
    if (wave > 0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) s.red[(wave - 1) * 1024 + v * 64 + lane] = acc.s[0][v];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float sum = ((acc.s[0][v] + s.red[v * 64 + lane]) + s.red[1024 + v * 64 + lane]) +
                          s.red[2048 + v * 64 + lane];
        const int pr = 8 * (v / 4) + 4 * (lane >> 5) + v % 4, qc = lane & 31;
        if (pr < R && qc < R) out[pr * R + qc] = sum;
      }
    }
  } else {
    // Wavefront b < 3 adds up block b of the four; the last one writes block (1, 0), the transpose of (0, 1).
    static_assert(kGramBatch * R >= 9 * 1024, "the blocks that change hands");
    auto block = [&](int w, int b) { return s.a + (2 * w + (w < 3 && b > w ? b - 1 : b)) * 1024 + lane; };
    __syncthreads();  // a has been read
#pragma unroll
    for (int b = 0; b < 3; ++b)
      if (wave != b) {
#pragma unroll
        for (int v = 0; v < 16; ++v) block(wave, b)[v * 64] = acc.s[b][v];
      }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 3; ++b)
      if (wave == b) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          float sum = acc.s[b][v];
#pragma unroll
          for (int w = 0; w < 4; ++w)
            if (w != b) sum += block(w, b)[v * 64];
          acc.s[b][v] = sum;
          out[(32 * (b >> 1) + dev::mfma_row(v, lane)) * R + 32 * (b > 0) + (lane & 31)] = sum;
        }
      }
    // (in place of the first wavefront's block (0, 1), which only this one reads; a column a row, piece p of
    // row q at p ^ q, so that neither side meets a bank twice)
    float* const turned = s.a;
    const int c = lane & 31;
    if (wave == 1) {
      __builtin_amdgcn_wave_barrier();  // other lanes of the wavefront have read what is overwritten
#pragma unroll
      for (int v = 0; v < 16; ++v) turned[c * 32 + (dev::mfma_row(v, lane) ^ c)] = acc.s[1][v];
    }
    __syncthreads();
    if (wave == 3) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int q = 2 * i + (lane >> 5);
        out[(32 + q) * R + c] = turned[q * 32 + (c ^ q)];
      }
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
