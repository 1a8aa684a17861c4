// a5 — exact softmax attention of one query over the k + w selected rows
// (Sec. 4.3: Attention(q_t, K_Omega, V_Omega) with the original q, K, V).
//
// One query row per head and 2*d flops per K/V element pair: the step is bound by
// the HBM reads of the selected rows (a random gather of d-element rows from the
// cache plus the contiguous lite rows).  Layout of the work:
//   * the k + w rows of a head are split over `nsplit` workgroups so that batch-1
//     steps still fill the chip; a workgroup of 4 wavefronts handles a contiguous
//     range of the row list;
//   * a row is read by 16 lanes, each taking one 16-byte (bf16) or 32-byte (fp32)
//     chunk of the K row and the same chunk of the V row, so a wavefront reads 4
//     rows per load instruction in full 256/512-byte segments; four such groups
//     of loads are issued before any is consumed;
//   * q.K is finished with a 16-lane rotate-and-add; every 16-lane group keeps its
//     own running (max, sum, acc[8 per lane]) so no cross-group traffic is needed
//     until the end, where the 4 groups and then the 4 wavefronts are merged;
//   * each workgroup writes one partial (m, s, acc[128]); a second small kernel
//     merges the partials of a head.
// Arithmetic is fp32 throughout; exp is exp2 on log2(e)-scaled logits.
//
// A small launch is bound by the chain index -> row -> result, not by its bytes: the body is
// compiled per mode and loads a row's slot, hit flag and token together and without a branch,
// so that the chain is two loads long.  Whole decode step, before -> after (bf16, 32 + 8 heads): 4K
// context, one layer, 25.3 -> 24.6 us; two layers at 32K 120.1 -> 118.3, at 128K 237.7 -> 235.3.  A
// batch of eight at 64K, bound by the host link and A_K, takes 306 to 309 us either way.
#include <type_traits>

#include "lrqk_device.h"
#include "lrqk_internal.h"

namespace lrqk {
namespace {

constexpr int kAttThreads = 256;
constexpr int kRowsPerPass = 16;  // 4 wavefronts x 4 row groups
// passes whose loads are in flight together; with 16 rows a pass, a workgroup's minimal share is
// 32 rows (measured on rows that no cache holds: 32 rows a workgroup 11.7 us, 64 rows 13.2 us,
// 128 rows 16.4 us for the 33.8 MB of the 128K-context shape: many small workgroups win)
constexpr int kUnroll = 2;
constexpr float kLog2e = 1.4426950408889634f;

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// sum over the 16 lanes of a DPP row; every lane of the row ends with the total
__device__ __forceinline__ float row16_allreduce_sum(float v) {
  v += dpp_f32<0x128>(v);  // row_ror:8
  v += dpp_f32<0x124>(v);  // row_ror:4
  v += dpp_f32<0x122>(v);  // row_ror:2
  v += dpp_f32<0x121>(v);  // row_ror:1
  return v;
}

struct Chunk8 {
  float v[8];
};

__device__ __forceinline__ Chunk8 unpack_bf16x8(const uint4 u) {
  Chunk8 c;
  c.v[0] = __uint_as_float(u.x << 16);
  c.v[1] = __uint_as_float(u.x & 0xffff0000u);
  c.v[2] = __uint_as_float(u.y << 16);
  c.v[3] = __uint_as_float(u.y & 0xffff0000u);
  c.v[4] = __uint_as_float(u.z << 16);
  c.v[5] = __uint_as_float(u.z & 0xffff0000u);
  c.v[6] = __uint_as_float(u.w << 16);
  c.v[7] = __uint_as_float(u.w & 0xffff0000u);
  return c;
}

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Loads the lane's 8-element chunk of a row.  BF16: 16 bytes; F32: 32 bytes.
template <bool BF16>
struct RowChunk;
template <>
struct RowChunk<true> {
  uint4 raw;
  __device__ __forceinline__ void load(const void* row, int c) {
    // a selected row is read once per step: streaming load
    const v4u x = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(row) + c);
    raw = make_uint4(x.x, x.y, x.z, x.w);
  }
  __device__ __forceinline__ void store(void* row, int c) const {
    reinterpret_cast<uint4*>(row)[c] = raw;
  }
  __device__ __forceinline__ Chunk8 get() const { return unpack_bf16x8(raw); }
};
template <>
struct RowChunk<false> {
  float4 a, b;
  __device__ __forceinline__ void load(const void* row, int c) {
    const v4f x = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(row) + 2 * c);
    const v4f y = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(row) + 2 * c + 1);
    a = make_float4(x.x, x.y, x.z, x.w);
    b = make_float4(y.x, y.y, y.z, y.w);
  }
  __device__ __forceinline__ void store(void* row, int c) const {
    reinterpret_cast<float4*>(row)[2 * c] = a;
    reinterpret_cast<float4*>(row)[2 * c + 1] = b;
  }
  __device__ __forceinline__ Chunk8 get() const {
    Chunk8 o;
    o.v[0] = a.x; o.v[1] = a.y; o.v[2] = a.z; o.v[3] = a.w;
    o.v[4] = b.x; o.v[5] = b.y; o.v[6] = b.z; o.v[7] = b.w;
    return o;
  }
};

// kAttendAllFetch: rows that missed the cache are read straight from the pinned host store
// (device-visible host memory), used, and written into their cache slot on the way: the
// fetch leg and the attention become one kernel, so the host-link reads of the few missing
// rows overlap with the HBM reads of all the others.
struct FetchSrc {
  const char* K_host;       // [B,Hkv,lrows,d] rows
  const char* V_host;
  const int32_t* sel_idx;   // [B,Hq,k] position of each selected row
  int l;                    // context length
  int lrows;                // rows allocated per (batch, KV head)
};

struct AttendArgs {
  FetchSrc fs;
  const float* q;
  const void* cacheK;
  const void* cacheV;
  const int32_t* sel_slot;
  const uint8_t* hit;
  const int32_t* miss_slot;
  const int32_t* n_miss;
  const void* liteK;
  const void* liteV;
  float* partials;
  int B, Hq, Hkv, C, k, w, rows_per_block, parts_per_head, part_offset;
  int blocks;  // workgroups per head
  bool by_die; // one-dimensional grid, dealt out by place_head; otherwise (blocks, heads)
  float scale;
};

// One workgroup's share of a head's row list: block bx of head bh.
template <bool BF16, int MODE>
__device__ __forceinline__ void attend_partial_body(const AttendArgs& a, int bx, int bh) {
  const FetchSrc fs = a.fs;
  const float* __restrict__ q = a.q;
  const void* cacheK = a.cacheK;
  const void* cacheV = a.cacheV;
  const int32_t* __restrict__ n_miss = a.n_miss;
  const int Hq = a.Hq, Hkv = a.Hkv, C = a.C, k = a.k, w = a.w;
  const int rows_per_block = a.rows_per_block, parts_per_head = a.parts_per_head;
  const int part_offset = a.part_offset;
  const float scale = a.scale;
  constexpr size_t ROWB = kD * (BF16 ? 2 : 4);
  __shared__ float wm[4], wsum[4];
  __shared__ float wacc[4][kD];

  const int b = bh / Hq, h = bh - b * Hq;
  const int kvh = h / (Hq / Hkv);
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int grp = lane >> 4, c = lane & 15;

  char* const Kc = const_cast<char*>(static_cast<const char*>(cacheK)) + (size_t)bh * C * ROWB;
  char* const Vc = const_cast<char*>(static_cast<const char*>(cacheV)) + (size_t)bh * C * ROWB;
  const size_t kv_row0 = ((size_t)b * Hkv + kvh) * (size_t)fs.lrows;
  const char* const Kh = MODE == kAttendAllFetch ? fs.K_host + kv_row0 * ROWB : nullptr;
  const char* const Vh = MODE == kAttendAllFetch ? fs.V_host + kv_row0 * ROWB : nullptr;
  const int32_t* __restrict__ toks = MODE == kAttendAllFetch ? fs.sel_idx + (size_t)bh * k : nullptr;
  const char* const Kl = static_cast<const char*>(a.liteK) + ((size_t)b * Hkv + kvh) * (size_t)w * ROWB;
  const char* const Vl = static_cast<const char*>(a.liteV) + ((size_t)b * Hkv + kvh) * (size_t)w * ROWB;
  const int32_t* __restrict__ slots = (MODE == kAttendMisses ? a.miss_slot : a.sel_slot) + (size_t)bh * k;
  constexpr bool kUsesHit = MODE == kAttendHitsAndLite || MODE == kAttendAllFetch;
  const uint8_t* __restrict__ hits = kUsesHit ? a.hit + (size_t)bh * k : nullptr;

  int n_rows;  // length of this head's row list
  if (MODE == kAttendMisses) {
    const int nm = n_miss[bh];
    n_rows = nm < 0 ? 0 : min(nm, k);
  } else {
    n_rows = k + w;
  }

  float qv[8];
  {
    const float4 q0 = reinterpret_cast<const float4*>(q + (size_t)bh * kD)[2 * c];
    const float4 q1 = reinterpret_cast<const float4*>(q + (size_t)bh * kD)[2 * c + 1];
    const float f = scale * kLog2e;  // logits are kept in log2 units
    qv[0] = q0.x * f; qv[1] = q0.y * f; qv[2] = q0.z * f; qv[3] = q0.w * f;
    qv[4] = q1.x * f; qv[5] = q1.y * f; qv[6] = q1.z * f; qv[7] = q1.w * f;
  }

  float m = -INFINITY, ssum = 0.0f;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  const int row_begin = bx * rows_per_block;
  const int row_end = min(n_rows, row_begin + rows_per_block);
  for (int base = row_begin; base < row_end; base += kRowsPerPass * kUnroll) {
    // Everything a row's address depends on is loaded at once, then the rows: no load sits in a
    // branch (it would be waited for before the next is issued) or behind another one's value
    // that it does not need; entries that do not exist read ones that do.
    int32_t slot[kUnroll], tok[kUnroll];
    uint8_t was_hit[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int jc = min(base + u * kRowsPerPass + wv * 4 + grp, k - 1);
      slot[u] = slots[jc];
      was_hit[u] = kUsesHit ? hits[jc] : (uint8_t)1;
      tok[u] = MODE == kAttendAllFetch ? toks[jc] : 0;
    }
    bool ok[kUnroll], fetch[kUnroll];
    size_t dst[kUnroll];  // cache slot to fill when the row comes from the host store
    RowChunk<BF16> kc[kUnroll], vc[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int j = base + u * kRowsPerPass + wv * 4 + grp;
      const bool lite = MODE != kAttendMisses && j >= k;
      const bool usable = slot[u] >= 0 && slot[u] < C &&
                          !(MODE == kAttendHitsAndLite && was_hit[u] == 0);
      ok[u] = j < row_end && (lite || usable);
      fetch[u] = MODE == kAttendAllFetch && ok[u] && !lite && was_hit[u] == 0 && tok[u] >= 0 &&
                 tok[u] < fs.l;
      dst[u] = (size_t)(usable ? slot[u] : 0) * ROWB;
      const size_t off = fetch[u] ? (size_t)tok[u] * ROWB
                                  : (ok[u] && lite) ? (size_t)(j - k) * ROWB : dst[u];
      // (the rows that the launch beside this one fetches are left alone: a tenth of the list)
      if (MODE != kAttendHitsAndLite || ok[u]) {
        kc[u].load((fetch[u] ? Kh : (ok[u] && lite) ? Kl : Kc) + off, c);
        vc[u].load((fetch[u] ? Vh : (ok[u] && lite) ? Vl : Vc) + off, c);
      }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (fetch[u]) {
        kc[u].store(Kc + dst[u], c);
        vc[u].store(Vc + dst[u], c);
      }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      float part = 0.0f;
      Chunk8 kk = kc[u].get();
#pragma unroll
      for (int i = 0; i < 8; ++i) part = __builtin_fmaf(qv[i], ok[u] ? kk.v[i] : 0.0f, part);
      const float logit = row16_allreduce_sum(part);  // all lanes take part in the DPP ops
      if (ok[u]) {
        const float m_new = fmaxf(m, logit);
        const float corr = exp2f(m - m_new);  // m = -inf on the first row gives 0
        const float p = exp2f(logit - m_new);
        ssum = ssum * corr + p;
        Chunk8 vv = vc[u].get();
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = __builtin_fmaf(p, vv.v[i], acc[i] * corr);
        m = m_new;
      }
    }
  }

  // merge the 4 row groups of the wavefront (lanes c, c+16, c+32, c+48)
  float mw = fmaxf(m, __shfl_xor(m, 16));
  mw = fmaxf(mw, __shfl_xor(mw, 32));
  const float f = (m == -INFINITY) ? 0.0f : exp2f(m - mw);
  ssum *= f;
  ssum += __shfl_xor(ssum, 16);
  ssum += __shfl_xor(ssum, 32);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float a = acc[i] * f;
    a += __shfl_xor(a, 16);
    a += __shfl_xor(a, 32);
    acc[i] = a;
  }
  if (lane < 16) {
#pragma unroll
    for (int i = 0; i < 8; ++i) wacc[wv][8 * c + i] = acc[i];
    if (lane == 0) {
      wm[wv] = mw;
      wsum[wv] = ssum;
    }
  }
  __syncthreads();
  // merge the 4 wavefronts; thread j < 128 owns output dimension j
  if (t < kD) {
    const float M = fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]));
    float a0 = 0.0f, s0 = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float g = (wm[i] == -INFINITY) ? 0.0f : exp2f(wm[i] - M);
      a0 += wacc[i][t] * g;
      s0 += wsum[i] * g;
    }
    float* __restrict__ P =
        a.partials + ((size_t)bh * parts_per_head + part_offset + bx) * kPartialStride;
    P[4 + t] = a0;
    if (t == 0) {
      P[0] = M;
      P[1] = s0;
    }
  }
}

template <bool BF16, int MODE>
__global__ __launch_bounds__(kAttThreads) void attend_partial_kernel(const AttendArgs a) {
  int bh = blockIdx.y, block = blockIdx.x;
  if (a.by_die) dev::place_head(blockIdx.x, a.B, a.Hq, a.Hkv, a.blocks, bh, block);
  attend_partial_body<BF16, MODE>(a, block, bh);
}

// Fetch shared by the query heads of a KV group (K and V exist once per KV head, Sec. 4
// preliminaries; Alg. 2 "Fetch missing", "merge"): the missing rows of head bh, 16 lanes a row.
// A position that several heads of the group miss is read from the host store once, by the
// lowest of those heads, and written into the slot each of them gave it; the other heads skip
// it.  The heads' miss lists are ascending, so "does head g2 miss this position, and where" is
// a binary search, run by lane g2 of the 16-lane group for its head.
struct GroupFetchArgs {
  FetchSrc fs;          // sel_idx unused
  void* cacheK;
  void* cacheV;
  const int32_t* miss_tok;
  const int32_t* miss_slot;
  const int32_t* n_miss;
  int32_t* link_rows;   // [B,Hkv] rows read from the host store, or null (not counted)
  int Hq, Hkv, C, k;
};
template <bool BF16>
__device__ __forceinline__ void group_fetch_body(const GroupFetchArgs& a, int fx, int nfx, int bh) {
  constexpr size_t ROWB = kD * (BF16 ? 2 : 4);
  const int Hq = a.Hq, Hkv = a.Hkv, C = a.C, k = a.k;
  const int G = Hq / Hkv;
  const int b = bh / Hq, h = bh - b * Hq, kvh = h / G, g = h - kvh * G;
  const int bh0 = bh - g;  // first head of the group
  const int t = threadIdx.x, lane = t & 63, sub = t & 15, rgrp = t >> 4;
  const int nm = max(0, min(a.n_miss[bh], k));
  const int32_t* __restrict__ mt = a.miss_tok + (size_t)bh * k;
  const int32_t* __restrict__ ms = a.miss_slot + (size_t)bh * k;
  const char* __restrict__ Kh = a.fs.K_host + ((size_t)b * Hkv + kvh) * (size_t)a.fs.lrows * ROWB;
  const char* __restrict__ Vh = a.fs.V_host + ((size_t)b * Hkv + kvh) * (size_t)a.fs.lrows * ROWB;
  // lane `sub` < G looks positions up in the list of head bh0 + sub
  const int32_t* __restrict__ ot = a.miss_tok + (size_t)(bh0 + min(sub, G - 1)) * k;
  const int32_t* __restrict__ os = a.miss_slot + (size_t)(bh0 + min(sub, G - 1)) * k;
  const int onm = sub < G ? max(0, min(a.n_miss[bh0 + sub], k)) : 0;
  for (int j0 = fx * 16; j0 < nm; j0 += nfx * 16) {  // uniform trip count over the wavefront
    const int j = j0 + rgrp;
    const bool have = j < nm;
    const int32_t tok = have ? mt[j] : -1;
    const int32_t slot = have ? ms[j] : -1;
    const bool ok = tok >= 0 && tok < a.fs.l && slot >= 0 && slot < C;
    // where, if anywhere, head bh0 + sub lists this position
    int32_t oslot = -1;
    if (ok && sub < G && sub != g) {
      int lo = 0, hi = onm;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ot[mid] < tok) lo = mid + 1; else hi = mid;
      }
      if (lo < onm && ot[lo] == tok) {
        const int32_t s2 = os[lo];
        oslot = (s2 >= 0 && s2 < C) ? s2 : -2;  // -2: listed, but with an unusable slot
      }
    }
    // the lowest head that lists the position fetches it
    const unsigned long long listed = __ballot(oslot != -1);
    const unsigned mine16 = (unsigned)(listed >> (lane & 48)) & 0xffffu;
    const bool owner = ok && (mine16 & ((1u << g) - 1u)) == 0u;
    RowChunk<BF16> kc, vc;
    if (owner) {
      kc.load(Kh + (size_t)tok * ROWB, sub);
      vc.load(Vh + (size_t)tok * ROWB, sub);
      kc.store(static_cast<char*>(a.cacheK) + ((size_t)bh * C + slot) * ROWB, sub);
      vc.store(static_cast<char*>(a.cacheV) + ((size_t)bh * C + slot) * ROWB, sub);
      if (sub == 0 && a.link_rows) atomicAdd(&a.link_rows[b * Hkv + kvh], 1);
    }
    for (int g2 = g + 1; g2 < G; ++g2) {  // uniform
      const int32_t s2 = __shfl(oslot, (lane & 48) + g2);
      if (owner && s2 >= 0) {
        kc.store(static_cast<char*>(a.cacheK) + ((size_t)(bh0 + g2) * C + s2) * ROWB, sub);
        vc.store(static_cast<char*>(a.cacheV) + ((size_t)(bh0 + g2) * C + s2) * ROWB, sub);
      }
    }
  }
}

template <bool BF16>
__global__ __launch_bounds__(kAttThreads) void group_fetch_kernel(const GroupFetchArgs a) {
  group_fetch_body<BF16>(a, blockIdx.x, gridDim.x, blockIdx.y);
}

// The attention over the rows that hit and the lite rows (blocks [0, n_attend) of a head) and
// the group's shared fetch (the remaining blocks) in one launch: the two do not depend on each
// other, so the host-link reads run beside the HBM reads.
template <bool BF16>
__global__ __launch_bounds__(kAttThreads) void attend_hits_group_fetch_kernel(
    const AttendArgs a, const GroupFetchArgs f) {
  if ((int)blockIdx.x < a.blocks)
    attend_partial_body<BF16, kAttendHitsAndLite>(a, blockIdx.x, blockIdx.y);
  else
    group_fetch_body<BF16>(f, blockIdx.x - a.blocks, gridDim.x - a.blocks, blockIdx.y);
}

constexpr int kCombThreads = 512;
constexpr int kCombMaxParts = 1024;

// Merge the partial softmax states of one head.  The per-part weights are computed
// once in LDS; four groups of 128 threads then walk the parts with independent,
// coalesced loads (thread = output dimension) and are summed through LDS.
__global__ __launch_bounds__(kCombThreads) void attend_combine_kernel(
    const float* __restrict__ partials, int parts_per_head, int nparts,
    float* __restrict__ out, int B, int Hq, int Hkv, bool by_die) {
  __shared__ float wgt[kCombMaxParts];
  __shared__ float red[kCombThreads / 64];
  __shared__ float accs[kCombThreads / kD][kD];
  __shared__ float sh_M, sh_S;
  int bh = blockIdx.x, block;
  if (by_die) dev::place_head(blockIdx.x, B, Hq, Hkv, 1, bh, block);
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const float* __restrict__ P = partials + (size_t)bh * parts_per_head * kPartialStride;
  // block max of the part maxima
  float m = -INFINITY;
  for (int p = t; p < nparts; p += kCombThreads) m = fmaxf(m, P[(size_t)p * kPartialStride]);
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d));
  if (lane == 0) red[wv] = m;
  __syncthreads();
  if (t == 0) {
    float M = red[0];
    for (int i = 1; i < kCombThreads / 64; ++i) M = fmaxf(M, red[i]);
    sh_M = M;
  }
  __syncthreads();
  const float M = sh_M;
  float ssum = 0.0f;
  for (int p = t; p < nparts; p += kCombThreads) {
    const float mp = P[(size_t)p * kPartialStride];
    const float g = (mp == -INFINITY) ? 0.0f : exp2f(mp - M);
    wgt[p] = g;
    ssum += P[(size_t)p * kPartialStride + 1] * g;
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) ssum += __shfl_xor(ssum, d);
  __syncthreads();
  if (lane == 0) red[wv] = ssum;
  __syncthreads();
  if (t == 0) {
    float S = 0.0f;
    for (int i = 0; i < kCombThreads / 64; ++i) S += red[i];
    sh_S = S;
  }
  const int dim = t & (kD - 1), grp = t / kD;
  float a = 0.0f;
#pragma unroll 8
  for (int p = grp; p < nparts; p += kCombThreads / kD)
    a = __builtin_fmaf(P[(size_t)p * kPartialStride + 4 + dim], wgt[p], a);
  accs[grp][dim] = a;
  __syncthreads();
  if (t < kD) {
    float tot = 0.0f;
#pragma unroll
    for (int g = 0; g < kCombThreads / kD; ++g) tot += accs[g][t];
    const float S = sh_S;
    out[(size_t)bh * kD + t] = S > 0.0f ? tot / S : 0.0f;
  }
}

}  // namespace

AttendGeom attend_geometry(int BHq, int k, int w) {
  const int rows = k + w;
  AttendGeom g;
  g.rows_per_block = kRowsPerPass * kUnroll;
  // fewer, larger workgroups once there are plenty of them
  while (g.rows_per_block < 512 && (long)ceil_div(rows, g.rows_per_block * 2) * BHq >= 2048)
    g.rows_per_block *= 2;
  g.nsplit = ceil_div(rows, g.rows_per_block);
  return g;
}

size_t attend_ws_bytes(int BHq, int k, int w, int phases) {
  const AttendGeom g = attend_geometry(BHq, k, w);
  const int parts = g.nsplit + (phases > 1 ? ceil_div(k, g.rows_per_block) : 0);
  return round_up((size_t)BHq * parts * kPartialStride * sizeof(float), 256);
}

// The workgroups of a head on the die of its selection and of its merge, where they are few: a step with
// direct fetch at 32 + 8 heads with 9 workgroups a head (4K context) 21.9 -> 21.1 us, with 17 (8K) 37.4 -> 36.3,
// with 26 (16K) 47.3 -> 45.8, two layers with 34 (32K) 116.5 -> 115.2.  Beyond it nothing: two layers with 66
// (128K) 233.3 -> 233.0, one of 224 heads 306.3 -> 306.2 (there the link and A_K set the time).  The
// stand-alone attention, whose rows another launch has fetched, gains nothing either (the chain of calls at
// 50K 87.2, 87.4 us, at 20K, 16 + 2 heads, 51.3, 51.8).  Where heads are not placed the grid is (workgroups,
// heads), without the divisions that take a one-dimensional one apart.
bool attend_by_die(const lrqk_shape& s, int nblocks) { return s.B * s.Hq * nblocks <= 1536; }

static AttendArgs make_attend_args(const lrqk_shape& s, const float* q,
                                   const void* cacheK, const void* cacheV,
                                   const int32_t* sel_slot, const uint8_t* hit,
                                   const int32_t* miss_slot, const int32_t* n_miss,
                                   const void* liteK, const void* liteV, float* partials,
                                   int nblocks, int rows_per_block, int parts_per_head,
                                   int part_offset, bool by_die, const void* K_host,
                                   const void* V_host, const int32_t* sel_idx) {
  AttendArgs a;
  a.fs = FetchSrc{static_cast<const char*>(K_host), static_cast<const char*>(V_host), sel_idx,
                  s.l, row_cap(s)};
  a.q = q;
  a.cacheK = cacheK;
  a.cacheV = cacheV;
  a.sel_slot = sel_slot;
  a.hit = hit;
  a.miss_slot = miss_slot;
  a.n_miss = n_miss;
  a.liteK = liteK;
  a.liteV = liteV;
  a.partials = partials;
  a.B = s.B;
  a.Hq = s.Hq;
  a.Hkv = s.Hkv;
  a.C = s.C;
  a.k = s.k;
  a.w = s.w;
  a.rows_per_block = rows_per_block;
  a.parts_per_head = parts_per_head;
  a.part_offset = part_offset;
  a.blocks = nblocks;
  a.by_die = by_die;
  a.scale = s.scale;
  return a;
}

// workgroups per head that the shared fetch is spread over (16 rows per pass each)
static int group_fetch_blocks(const lrqk_shape& s) { return min(ceil_div(s.k, 16), 32); }

static GroupFetchArgs make_group_fetch_args(const lrqk_shape& s, const void* K_host,
                                            const void* V_host, const int32_t* miss_tok,
                                            const int32_t* miss_slot, const int32_t* n_miss,
                                            void* cacheK, void* cacheV, int32_t* link_rows) {
  GroupFetchArgs f;
  f.fs = FetchSrc{static_cast<const char*>(K_host), static_cast<const char*>(V_host), nullptr,
                  s.l, row_cap(s)};
  f.cacheK = cacheK;
  f.cacheV = cacheV;
  f.miss_tok = miss_tok;
  f.miss_slot = miss_slot;
  f.n_miss = n_miss;
  f.link_rows = link_rows;
  f.Hq = s.Hq;
  f.Hkv = s.Hkv;
  f.C = s.C;
  f.k = s.k;
  return f;
}

hipError_t launch_attend_partial(const lrqk_shape& s, int mode, const float* q, const void* cacheK,
                                 const void* cacheV, const int32_t* sel_slot, const uint8_t* hit,
                                 const int32_t* miss_slot, const int32_t* n_miss,
                                 const void* liteK, const void* liteV, float* partials,
                                 int nblocks, int rows_per_block, int parts_per_head,
                                 int part_offset, hipStream_t st, const void* K_host,
                                 const void* V_host, const int32_t* sel_idx, bool by_die) {
  if (nblocks <= 0) return hipSuccess;
  if (mode == kAttendAllFetch && (!K_host || !V_host || !sel_idx || !hit))
    return hipErrorInvalidValue;
  const AttendArgs a = make_attend_args(s, q, cacheK, cacheV, sel_slot, hit, miss_slot,
                                        n_miss, liteK, liteV, partials, nblocks, rows_per_block,
                                        parts_per_head, part_offset, by_die, K_host, V_host, sel_idx);
  const dim3 grid = by_die ? dim3(nblocks * s.B * s.Hq) : dim3(nblocks, s.B * s.Hq);
  auto run = [&](auto m) {
    constexpr int MODE = decltype(m)::value;
    if (s.kv_dtype == LRQK_KV_BF16)
      LRQK_LAUNCH((attend_partial_kernel<true, MODE>), grid, dim3(kAttThreads), 0, st, a);
    else
      LRQK_LAUNCH((attend_partial_kernel<false, MODE>), grid, dim3(kAttThreads), 0, st, a);
  };
  switch (mode) {
    case kAttendAll: run(std::integral_constant<int, kAttendAll>{}); break;
    case kAttendHitsAndLite: run(std::integral_constant<int, kAttendHitsAndLite>{}); break;
    case kAttendMisses: run(std::integral_constant<int, kAttendMisses>{}); break;
    case kAttendAllFetch: run(std::integral_constant<int, kAttendAllFetch>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_group_fetch(const lrqk_shape& s, const void* K_host, const void* V_host,
                              const int32_t* miss_tok, const int32_t* miss_slot,
                              const int32_t* n_miss, void* cacheK, void* cacheV,
                              int32_t* link_rows, hipStream_t st) {
  const GroupFetchArgs f = make_group_fetch_args(s, K_host, V_host, miss_tok, miss_slot, n_miss,
                                                 cacheK, cacheV, link_rows);
  const dim3 grid(group_fetch_blocks(s), s.B * s.Hq);
  if (s.kv_dtype == LRQK_KV_BF16)
    LRQK_LAUNCH((group_fetch_kernel<true>), grid, dim3(kAttThreads), 0, st, f);
  else
    LRQK_LAUNCH((group_fetch_kernel<false>), grid, dim3(kAttThreads), 0, st, f);
  return hipGetLastError();
}

hipError_t launch_attend_hits_group_fetch(const lrqk_shape& s, const float* q, void* cacheK,
                                          void* cacheV, const int32_t* sel_slot,
                                          const uint8_t* hit, const void* liteK,
                                          const void* liteV, float* partials, int nblocks,
                                          int rows_per_block, int parts_per_head,
                                          const void* K_host, const void* V_host,
                                          const int32_t* miss_tok, const int32_t* miss_slot,
                                          const int32_t* n_miss, int32_t* link_rows,
                                          hipStream_t st) {
  const AttendArgs a = make_attend_args(s, q, cacheK, cacheV, sel_slot, hit,
                                        nullptr, nullptr, liteK, liteV, partials, nblocks,
                                        rows_per_block, parts_per_head, 0, false, nullptr, nullptr,
                                        nullptr);
  const GroupFetchArgs f = make_group_fetch_args(s, K_host, V_host, miss_tok, miss_slot, n_miss,
                                                 cacheK, cacheV, link_rows);
  const dim3 grid(nblocks + group_fetch_blocks(s), s.B * s.Hq);
  if (s.kv_dtype == LRQK_KV_BF16)
    LRQK_LAUNCH((attend_hits_group_fetch_kernel<true>), grid, dim3(kAttThreads), 0, st, a, f);
  else
    LRQK_LAUNCH((attend_hits_group_fetch_kernel<false>), grid, dim3(kAttThreads), 0, st, a, f);
  return hipGetLastError();
}

hipError_t launch_attend_combine(const lrqk_shape& s, const float* partials, int parts_per_head,
                                 int nparts, float* out, hipStream_t st, bool by_die) {
  if (nparts > kCombMaxParts) return hipErrorInvalidValue;
  LRQK_LAUNCH(attend_combine_kernel, dim3(s.B * s.Hq), dim3(kCombThreads), 0, st,
                     partials, parts_per_head, nparts, out, s.B, s.Hq, s.Hkv,
                     by_die);
  return hipGetLastError();
}

}  // namespace lrqk
