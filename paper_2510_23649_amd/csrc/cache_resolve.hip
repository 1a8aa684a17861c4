// a3 — hit/miss resolution against the GPU-resident KV cache (Sec. 4.1: a token
// already in the GPU cache is a hit, only missing tokens are fetched; Sec. 5.3:
// miss rate = fetched rows / selected rows).
//
// The paper does this indexing on the CPU and names it as its bottleneck
// (Limitations); here it is one workgroup per (batch, query head), entirely in
// LDS.  Replacement rule for C >= k slots: least recently selected, ties by lower
// slot; the j-th miss in ascending position takes the j-th victim.
// Usual sizes: cache_resolve_kernel, the resolution of the fused step (assign_victims: a histogram
// of the slots' ages, victims ranked class by class).  Caches so large that its lists do not fit
// the LDS: cache_resolve_sort_kernel,
//   1. every selected token looks up slot_of: hits refresh last_used, misses get
//      their rank by a prefix count in position order;
//   2. the slots not used in this step are the victim candidates; their keys
//      (last_used + 1) << 32 | slot are sorted in LDS (all other slots sort last);
//   3. miss j takes sorted[j]: evict its token, install the new one.
// All of it is integer work with a fixed order, so the result is deterministic.
#include "lrqk_device.h"
#include "lrqk_internal.h"
#include "select_common.h"

namespace lrqk {
namespace {

using dev::bitonic_sort_lds;

constexpr int kResThreads = 1024;

__global__ __launch_bounds__(256) void fill_i32_kernel(int32_t* p, size_t n, int32_t v) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}

// LDS of cache_resolve_kernel: last_used, token_of [C]; miss positions, their output indices,
// victims [k]; age histogram; the sort of the rare cases (8 bytes a slot).
__host__ __device__ inline size_t round256(size_t x) { return (x + 255) / 256 * 256; }
struct ResolveArena {
  size_t st_b, k_b, hist, sort, total;
};
__host__ __device__ inline ResolveArena resolve_arena(int k, int C) {
  ResolveArena a;
  a.st_b = round256((size_t)C * 4);
  a.k_b = round256((size_t)k * 4);
  a.hist = 2 * a.st_b + 3 * a.k_b;
  a.sort = a.hist + (size_t)kAgeBins * 4;
  int Cpad = 2;
  while (Cpad < C) Cpad <<= 1;
  a.total = a.sort + (size_t)Cpad * 8;
  return a;
}
constexpr size_t kResolveLdsLimit = 150 * 1024;

// Thread t owns k / 1024 consecutive entries of the selection (at most 4) and C / 1024 consecutive
// slots (at most SPT).  A chain of short phases: 6 us at k = 1000, C = 2000 (24 us with a sort of
// every slot).
template <int SPT>
__global__ __launch_bounds__(kT) void cache_resolve_kernel(
    const int32_t* __restrict__ sel_idx, int32_t step, int l, int lrows, int C, int k,
    int32_t* __restrict__ slot_of, int32_t* __restrict__ token_of,
    int32_t* __restrict__ last_used, int32_t* __restrict__ sel_slot, uint8_t* __restrict__ hit,
    int32_t* __restrict__ miss_tok, int32_t* __restrict__ miss_slot,
    int32_t* __restrict__ n_miss) {
  constexpr int PER = kMaxK / kT;
  extern __shared__ __align__(16) unsigned char res_lds[];
  __shared__ uint32_t wave_tot[4 * 2 * kWaves];  // four areas of 32 words, used in rotation
  __shared__ uint32_t sh_bad, sh_ncls, sh_clip;
  __shared__ uint32_t cls_age[kMaxCls], cls_base[kMaxCls];
  const int bh = blockIdx.x, t = threadIdx.x;
  const ResolveArena az = resolve_arena(k, C);
  int32_t* const lu_s = reinterpret_cast<int32_t*>(res_lds);
  int32_t* const to_s = reinterpret_cast<int32_t*>(res_lds + az.st_b);
  int32_t* const mt_s = reinterpret_cast<int32_t*>(res_lds + 2 * az.st_b);
  int32_t* const mj_s = reinterpret_cast<int32_t*>(res_lds + 2 * az.st_b + az.k_b);
  int32_t* const vsorted = reinterpret_cast<int32_t*>(res_lds + 2 * az.st_b + 2 * az.k_b);
  uint32_t* const ahist = reinterpret_cast<uint32_t*>(res_lds + az.hist);
  const int32_t* __restrict__ sel = sel_idx + (size_t)bh * k;
  int32_t* so = slot_of + (size_t)bh * lrows;
  int32_t* to = token_of + (size_t)bh * C;
  int32_t* lu = last_used + (size_t)bh * C;
  int32_t* ss = sel_slot + (size_t)bh * k;
  uint8_t* __restrict__ ht = hit + (size_t)bh * k;
  int32_t* __restrict__ mt = miss_tok + (size_t)bh * k;
  int32_t* ms = miss_slot + (size_t)bh * k;

  // every load that does not depend on another, then the slot_of look-ups; entries that do not
  // exist read ones that do
  const int per = (k + kT - 1) / kT, spt = (C + kT - 1) / kT;
  const int j0 = t * per;
  int32_t tok[PER], slot[PER], lu_r[SPT], to_r[SPT];
#pragma unroll
  for (int i = 0; i < PER; ++i) tok[i] = sel[min(j0 + i, k - 1)];
#pragma unroll
  for (int u = 0; u < SPT; ++u) {
    const int sl = min(u * kT + t, C - 1);
    lu_r[u] = lu[sl];
    to_r[u] = to[sl];
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) slot[i] = so[min(max(tok[i], 0), l - 1)];
  for (int i = t; i < kAgeBins; i += kT) ahist[i] = 0u;
  if (t == 0) {
    sh_bad = 0u;
    sh_ncls = 0u;
    sh_clip = 0u;
  }
#pragma unroll
  for (int u = 0; u < SPT; ++u)
    if (u * kT + t < C) {
      lu_s[u * kT + t] = lu_r[u];
      to_s[u * kT + t] = to_r[u];
    }
  uint32_t nmiss = 0;
  bool valid[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const bool on = i < per && j0 + i < k;
    valid[i] = on && tok[i] >= 0 && tok[i] < l;
    if (slot[i] >= C) slot[i] = -1;  // corrupt map entry: treat as absent
    nmiss += (valid[i] && slot[i] < 0) ? 1u : 0u;
  }
  uint32_t tot;
  uint32_t rank = scan1(nmiss, wave_tot + 2 * 2 * kWaves, &tot);  // (orders the LDS writes above)
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int j = j0 + i;
    if (i >= per || j >= k) continue;
    const bool is_hit = valid[i] && slot[i] >= 0;
    ht[j] = is_hit ? 1 : 0;
    if (is_hit) {
      ss[j] = slot[i];
      lu[slot[i]] = step;
      lu_s[slot[i]] = step;  // used in this step: never a victim
    } else if (valid[i]) {
      mt[rank] = tok[i];
      mt_s[rank] = tok[i];
      mj_s[rank] = j;
      ++rank;
    } else {
      atomicOr(&sh_bad, 1u);
      ss[j] = -1;
    }
  }
  lds_barrier();
  const int nm = (int)tot;
  if (nm > 0) {
    VictimWork v;
    v.lu_s = lu_s;
    v.to_s = to_s;
    v.mt_s = mt_s;
    v.mj_s = mj_s;
    v.vsorted = vsorted;
    v.ahist = ahist;
    v.cls_age = cls_age;
    v.cls_base = cls_base;
    v.sh_ncls = &sh_ncls;
    v.sh_clip = &sh_clip;
    v.sh_bad = &sh_bad;
    v.scan_areas = wave_tot;
    v.sort_area = res_lds + az.sort;
    v.so = so;
    v.to = to;
    v.lu = lu;
    v.ms = ms;
    v.ss = ss;
    v.step = step;
    v.C = C;
    v.l = l;
    v.spt = spt;
    assign_victims<SPT>(v, nm);
  }
  lds_barrier();
  if (t == 0) n_miss[bh] = sh_bad ? -1 : nm;
}

// dynamic LDS: uint64 keys[Cpad]
__global__ __launch_bounds__(kResThreads) void cache_resolve_sort_kernel(
    const int32_t* __restrict__ sel_idx, int32_t step, int l, int lrows, int C, int Cpad, int k,
    int32_t* __restrict__ slot_of, int32_t* __restrict__ token_of,
    int32_t* __restrict__ last_used, int32_t* __restrict__ sel_slot, uint8_t* __restrict__ hit,
    int32_t* __restrict__ miss_tok, int32_t* __restrict__ miss_slot,
    int32_t* __restrict__ n_miss) {
  extern __shared__ uint64_t keys[];
  __shared__ uint32_t wave_counts[kResThreads / 64];
  __shared__ uint32_t sh_nmiss, sh_bad;
  const int bh = blockIdx.x, t = threadIdx.x;
  const int lane = t & 63, wv = t >> 6;
  const int32_t* __restrict__ sel = sel_idx + (size_t)bh * k;
  int32_t* __restrict__ so = slot_of + (size_t)bh * lrows;
  int32_t* __restrict__ to = token_of + (size_t)bh * C;
  int32_t* __restrict__ lu = last_used + (size_t)bh * C;
  int32_t* __restrict__ ss = sel_slot + (size_t)bh * k;
  uint8_t* __restrict__ ht = hit + (size_t)bh * k;
  int32_t* __restrict__ mt = miss_tok + (size_t)bh * k;
  int32_t* __restrict__ ms = miss_slot + (size_t)bh * k;

  if (t == 0) {
    sh_nmiss = 0u;
    sh_bad = 0u;
  }
  // victim keys from the state before this step; slots hit below are taken out afterwards
  for (int s = t; s < Cpad; s += kResThreads)
    keys[s] = s < C ? (((uint64_t)(uint32_t)(lu[s] + 1)) << 32) | (uint32_t)s : ~0ull;
  __syncthreads();

  // pass over the selected tokens in position order, kResThreads at a time
  for (int j0 = 0; j0 < k; j0 += kResThreads) {
    const int j = j0 + t;
    int32_t tok = -1, slot = -1;
    bool valid = false, miss = false;
    if (j < k) {
      tok = sel[j];
      valid = tok >= 0 && tok < l;
      if (valid) slot = so[tok];
      if (valid && slot >= C) slot = -1;  // corrupt map entry: treat as absent
      miss = valid && slot < 0;
      if (!valid) {
        atomicOr(&sh_bad, 1u);
        ss[j] = -1;
        ht[j] = 0;
      } else if (!miss) {
        ss[j] = slot;
        ht[j] = 1;
        lu[slot] = step;
        keys[slot] = ~0ull;  // used in this step: never a victim
      } else {
        ht[j] = 0;
      }
    }
    // rank of this miss among all misses, in position order
    const unsigned long long m = __ballot(miss);
    if (lane == 0) wave_counts[wv] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t before = sh_nmiss, tot = 0;
    for (int i = 0; i < kResThreads / 64; ++i) {
      const uint32_t c = wave_counts[i];
      before += i < wv ? c : 0u;
      tot += c;
    }
    const uint32_t rank = before + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
    if (miss) {
      mt[rank] = tok;
      ss[j] = -(int32_t)rank - 2;  // remember the rank; replaced by the slot below
    }
    __syncthreads();
    if (t == 0) sh_nmiss += tot;
    __syncthreads();
  }
  const int nm = (int)sh_nmiss;
  if (nm > 0) {
    // a slot whose last_used already equals `step` (step reused by the caller) is protected too
    for (int s = t; s < C; s += kResThreads)
      if (keys[s] != ~0ull && (int32_t)(keys[s] >> 32) - 1 == step) keys[s] = ~0ull;
    bitonic_sort_lds(keys, Cpad);
    for (int j = t; j < nm; j += kResThreads) {
      const uint64_t key = keys[j];
      const int32_t tok = mt[j];
      if (key == ~0ull) {  // ran out of victims
        atomicOr(&sh_bad, 1u);
        ms[j] = -1;
        continue;
      }
      const int32_t s = (int32_t)(uint32_t)key;
      const int32_t old = to[s];
      if (old >= 0 && old < l) so[old] = -1;
      to[s] = tok;
      so[tok] = s;
      lu[s] = step;
      ms[j] = s;
    }
    __syncthreads();
    // translate remembered ranks into slots
    for (int j = t; j < k; j += kResThreads) {
      const int32_t v = ss[j];
      if (v <= -2) ss[j] = ms[-(v + 2)];
    }
  }
  __syncthreads();
  if (t == 0) n_miss[bh] = sh_bad ? -1 : nm;
}

}  // namespace

hipError_t launch_fill_i32(int32_t* p, size_t n, int32_t v, hipStream_t st) {
  if (n == 0) return hipSuccess;
  LRQK_LAUNCH(fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

hipError_t launch_cache_init(const lrqk_shape& s, int32_t* slot_of, int32_t* token_of,
                             int32_t* last_used, hipStream_t st) {
  const size_t BHq = (size_t)s.B * s.Hq;
  const size_t n1 = BHq * row_cap(s), n2 = BHq * s.C;
  LRQK_LAUNCH(fill_i32_kernel, dim3((unsigned)((n1 + 255) / 256)), dim3(256), 0, st,
                     slot_of, n1, -1);
  LRQK_LAUNCH(fill_i32_kernel, dim3((unsigned)((n2 + 255) / 256)), dim3(256), 0, st,
                     token_of, n2, -1);
  LRQK_LAUNCH(fill_i32_kernel, dim3((unsigned)((n2 + 255) / 256)), dim3(256), 0, st,
                     last_used, n2, -1);
  return hipGetLastError();
}

hipError_t launch_cache_resolve(const lrqk_shape& s, const int32_t* sel_idx, int32_t step,
                                int32_t* slot_of, int32_t* token_of, int32_t* last_used,
                                int32_t* sel_slot, uint8_t* hit, int32_t* miss_tok,
                                int32_t* miss_slot, int32_t* n_miss, hipStream_t st) {
  const size_t lds = resolve_arena(s.k, s.C).total;
  if (lds <= kResolveLdsLimit) {
    auto run = [&](auto kernel, std::atomic<uint64_t>& raised) {
      const hipError_t e = raise_dynamic_lds_once(kernel, kResolveLdsLimit, raised);
      if (e != hipSuccess) return e;
      LRQK_LAUNCH(kernel, dim3(s.B * s.Hq), dim3(kT), lds, st, sel_idx, step, s.l, row_cap(s),
                  s.C, s.k, slot_of, token_of, last_used, sel_slot, hit, miss_tok, miss_slot,
                  n_miss);
      return hipGetLastError();
    };
    static std::atomic<uint64_t> raised2{0}, raised4{0}, raised8{0};
    if (s.C <= 2 * kT) return run(cache_resolve_kernel<2>, raised2);
    if (s.C <= 4 * kT) return run(cache_resolve_kernel<4>, raised4);
    return run(cache_resolve_kernel<8>, raised8);
  }
  const int Cpad = next_pow2(s.C < 2 ? 2 : s.C);
  const size_t sort_lds = (size_t)Cpad * sizeof(uint64_t);
  if (sort_lds > 48 * 1024) {  // large caches need the dynamic-LDS ceiling raised once
    static std::atomic<uint64_t> raised{0};
    const hipError_t e = raise_dynamic_lds_once(cache_resolve_sort_kernel, 64 * 1024, raised);
    if (e != hipSuccess) return e;
  }
  LRQK_LAUNCH(cache_resolve_sort_kernel, dim3(s.B * s.Hq), dim3(kResThreads), sort_lds, st, sel_idx,
                     step, s.l, row_cap(s), s.C, Cpad, s.k, slot_of, token_of, last_used, sel_slot, hit,
                     miss_tok, miss_slot, n_miss);
  return hipGetLastError();
}

}  // namespace lrqk
