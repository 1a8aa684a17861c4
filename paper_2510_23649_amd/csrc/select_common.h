// Pieces shared by the one-workgroup-per-head selection kernels (1024 threads): score
// loading, the proxy score of a single row, and the exact selection of a head from its
// materialised scores (the route taken when a candidate estimate turns out unusable).
#pragma once

#include "lrqk_device.h"
#include "lrqk_internal.h"

namespace lrqk {
namespace {

using namespace dev;

constexpr int kT = 1024;  // threads per workgroup
constexpr int kWaves = kT / 64;
constexpr int kIter = kT * 4;  // scores per workgroup iteration (one float4 per lane)
constexpr int kBatch = 8;      // iterations whose loads are issued together
constexpr int kAgeBins = 2048;
constexpr int kSampleStride = 8;

constexpr int kMaxCls = 16;   // victim age classes numbered by the fast resolution

// Prefix sum over the 16 wave totals held in wt[0..16): returns the sum of the totals of the
// wavefronts before this one, and the grand total.  Lanes 0..15 of every wavefront read one
// total each and scan them with DPP row shifts (one LDS read instead of sixteen per thread).
__device__ __forceinline__ uint32_t waves_before(const uint32_t* wt, uint32_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t v = wt[lane & 15];
  uint32_t incl = v;
  incl += dpp_zero_fill<0x111, 0xf>(incl);  // row_shr:1
  incl += dpp_zero_fill<0x112, 0xf>(incl);  // row_shr:2
  incl += dpp_zero_fill<0x114, 0xf>(incl);  // row_shr:4
  incl += dpp_zero_fill<0x118, 0xf>(incl);  // row_shr:8
  *total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 15);
  return (uint32_t)__builtin_amdgcn_readlane((int)(incl - v), wv);
}

// Exclusive prefix sum over the 1024 threads and the total, with ONE LDS-only barrier.
// wt: 16 words of LDS that no thread may still be reading from an earlier scan: consecutive
// scans take different areas (scan_area), and an area comes round again only after two
// other barriers.
__device__ __forceinline__ uint32_t scan1(uint32_t v, uint32_t* wt, uint32_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_scan(v);
  if (lane == 63) wt[wv] = incl;
  lds_barrier();
  return waves_before(wt, total) + incl - v;
}
// The same for two values at once.  wt: 32 words of LDS, as above.
__device__ __forceinline__ void scan2(uint32_t v0, uint32_t v1, uint32_t* wt, uint32_t* ex0,
                                      uint32_t* ex1, uint32_t* tot0, uint32_t* tot1) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t i0 = wave_inclusive_scan(v0), i1 = wave_inclusive_scan(v1);
  if (lane == 63) {
    wt[wv] = i0;
    wt[16 + wv] = i1;
  }
  lds_barrier();
  *ex0 = waves_before(wt, tot0) + i0 - v0;
  *ex1 = waves_before(wt + 16, tot1) + i1 - v1;
}

// (key, position) of a candidate as one number: larger = better (higher key, or equal key and lower position)
__device__ __forceinline__ uint64_t value_of(uint32_t key, int p) {
  return ((uint64_t)key << 32) | (uint32_t)~(uint32_t)p;
}
__device__ __forceinline__ int position_of(uint64_t v) { return (int)~(uint32_t)v; }

constexpr int kSmall = 64;  // candidates of the threshold bin that one wavefront ranks directly

// Scan of a 2048-bin histogram from the top (thread t owns bins 2t, 2t+1) for two ranks at
// once: res[0] = the bin d that holds the want_a-th entry from the top, res[1] = the entries
// above d, res[3] = the bin that holds the want_b-th entry (0xffffffff where there are fewer
// entries than that).  Returns the number of entries.  LDS-only barriers.
__device__ __forceinline__ uint32_t find_two_from_top(const uint32_t* hist, uint32_t want_a,
                                                      uint32_t want_b, uint32_t* wt,
                                                      uint32_t* res) {
  const int t = threadIdx.x;
  const uint32_t c0 = hist[2 * t], c1 = hist[2 * t + 1];
  if (t == 0) {
    res[0] = 0xffffffffu;
    res[3] = 0xffffffffu;
  }
  uint32_t total;
  const uint32_t below = scan1(c0 + c1, wt, &total);  // its barriers order the writes of res
  const uint32_t above1 = total - below - c0 - c1;
  const uint32_t above0 = above1 + c1;
  if (above1 < want_a && want_a <= above1 + c1) {
    res[0] = 2 * t + 1;
    res[1] = above1;
  } else if (above0 < want_a && want_a <= above0 + c0) {
    res[0] = 2 * t;
    res[1] = above0;
  }
  if (above1 < want_b && want_b <= above1 + c1) {
    res[3] = 2 * t + 1;
  } else if (above0 < want_b && want_b <= above0 + c0) {
    res[3] = 2 * t;
  }
  lds_barrier();
  return total;
}

// The value of the k-th largest of a head's candidates, whose keys are all >= thr_key, at least k of them,
// in position order over the threads: entry e < E of a thread in val[e], 0: none.  Entries below the bin
// that holds it are zeroed before `meanwhile` is called, whose loads then run under the rest.  *shift: the
// width of a bin; *d_next: the bin of rank `rank_next` (0xffffffff: fewer entries than that).
struct CutWork {
  uint32_t* hist0;       // [2048], zero; taken
  uint32_t* hist1;       // [2048], zero; zero again afterwards
  uint64_t* small;       // [kSmall]
  uint32_t* sh_small_n;  // zero
  uint64_t* sh_cut;
  uint32_t* wave_tot;    // four areas of 32 words; area 0 may still be in use
  uint32_t* res;         // [4]
};
template <int MAXE, class F>
__device__ __forceinline__ uint64_t cut_of_entries(uint64_t (&val)[MAXE], uint32_t E, uint32_t thr_key,
                                                   uint32_t k, uint32_t rank_next, const CutWork& w,
                                                   F meanwhile, int* shift, uint32_t* d_next) {
  const int t = threadIdx.x, lane = t & 63;
  auto scan_area = [&](int i) { return w.wave_tot + (i & 3) * 2 * kWaves; };
  // Bin of a key: (key - thr_key) >> s, the top bin taking everything beyond.  For a positive
  // threshold s = 12 spreads the scores between the threshold and twice the threshold over the 2048 bins.
  int s = (thr_key > 0x80800000u && thr_key < 0xff800000u) ? 12 : 21;
  auto bin_of = [&](uint64_t v) { return min(((uint32_t)(v >> 32) - thr_key) >> s, 2047u); };
  auto for_each = [&](auto&& f) {
#pragma unroll
    for (int e = 0; e < MAXE; ++e) {
      if ((uint32_t)e >= E) break;  // uniform
      if (val[e] != 0ull) f(val[e]);
    }
  };
  for_each([&](uint64_t v) { atomicAdd(&w.hist0[bin_of(v)], 1u); });
  lds_barrier();
  find_two_from_top(w.hist0, k, rank_next, scan_area(1), w.res);
  uint32_t d0 = w.res[0], above0 = w.res[1];
  *d_next = w.res[3];
  if (__builtin_expect(d0 == 2047u && s != 21, 0)) {
    // the k-th largest lies beyond twice the threshold: bin the whole key range instead
    s = 21;
    lds_barrier();  // res has been read
    for (int i = t; i < 2048; i += kT) w.hist0[i] = 0u;
    lds_barrier();
    for_each([&](uint64_t v) { atomicAdd(&w.hist0[bin_of(v)], 1u); });
    lds_barrier();
    find_two_from_top(w.hist0, k, rank_next, scan_area(2), w.res);
    d0 = w.res[0];
    above0 = w.res[1];
    *d_next = w.res[3];
  }
  *shift = s;
#pragma unroll
  for (int e = 0; e < MAXE; ++e)
    if (val[e] != 0ull && bin_of(val[e]) < d0) val[e] = 0ull;  // not selected
  meanwhile();
  const uint32_t c0 = w.hist0[d0];
  const uint32_t want1 = k - above0;  // how many of bin d0 are selected
  if (__builtin_expect(c0 <= (uint32_t)kSmall, 1)) {
    // the few candidates of bin d0 are ranked on (key, position); the want1-th of them is
    // the cut
    for_each([&](uint64_t v) {
      if (bin_of(v) == d0) w.small[atomicAdd(w.sh_small_n, 1u)] = v;
    });
    lds_barrier();
    // every wavefront ranks the bin for itself (no second barrier to hand the cut over)
    const uint64_t mine = lane < (int)c0 ? w.small[lane] : 0ull;
    uint32_t larger = 0;
#pragma unroll 8
    for (uint32_t jj = 0; jj < c0; ++jj) larger += w.small[jj] > mine ? 1u : 0u;
    const unsigned long long is_cut = __ballot(lane < (int)c0 && larger == want1 - 1u);
    const int src = __builtin_ctzll(is_cut);  // exactly one entry has that rank
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), src);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, src);
    return ((uint64_t)hi << 32) | lo;
  }
  // many candidates in the bin (ties): further histogram levels over the low s bits give
  // the exact key tau of the k-th largest; of the candidates with that key the first
  // need_eq in position order are selected, so the cut is the need_eq-th of them
  uint32_t known = d0, want = want1;
  int rem = s;
  while (rem > 0) {
    const int bits = rem < 11 ? rem : 11;
    const int nsh = rem - bits;
    for_each([&](uint64_t v) {
      const uint32_t rel = (uint32_t)(v >> 32) - thr_key;
      if ((rel >> rem) == known) atomicAdd(&w.hist1[(rel >> nsh) & ((1u << bits) - 1u)], 1u);
    });
    __syncthreads();
    find_from_top(w.hist1, want, w.wave_tot, w.res);
    const uint32_t dd = w.res[0], ab = w.res[1];
    known = (known << bits) | dd;
    want -= ab;
    rem = nsh;
    __syncthreads();  // res and hist1 have been read
    for (int i = t; i < 2048; i += kT) w.hist1[i] = 0u;
    __syncthreads();
  }
  // (bin d0 is never the catch-all top bin here, so rel >> s == d0 identifies it)
  const uint32_t tau = thr_key + known, need_eq = want;
  uint32_t neq = 0;
  for_each([&](uint64_t v) { neq += (uint32_t)(v >> 32) == tau ? 1u : 0u; });
  uint32_t tot;
  uint32_t eq_rank = block_exclusive_scan(neq, w.wave_tot, &tot);
  for_each([&](uint64_t v) {  // (in position order)
    if ((uint32_t)(v >> 32) == tau && ++eq_rank == need_eq) *w.sh_cut = v;
  });
  __syncthreads();
  return *w.sh_cut;
}

struct Keys4 {
  uint32_t k[4];
  bool ok[4];
};
struct Raw4 {
  float v[4];
};
// Four consecutive scores starting at element e of the n of a head; entries past the end repeat
// the last one.  `whole`: (uniform) e + 3 < n for every thread, one 16-byte load.  Heads start at
// multiples of 4 bytes only (l need not be a multiple of 4), which such a load allows.  No load is
// in a branch of its own: it would be waited for before the next one is issued (at l = 50001 the
// two passes over the scores took 14 us each that way).
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ Raw4 load_raw4(const float* __restrict__ s, int e, int n, bool whole) {
  Raw4 r;
  if (whole) {
    const f32x4_u x = *reinterpret_cast<const f32x4_u*>(s + e);
    r.v[0] = x.x; r.v[1] = x.y; r.v[2] = x.z; r.v[3] = x.w;
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) r.v[c] = s[min(e + c, n - 1)];
  }
  return r;
}
// kBatch iterations' scores of a thread from iteration it0 on, `step` iterations apart
__device__ __forceinline__ void load_batch(Raw4 (&raw)[kBatch], const float* __restrict__ s,
                                           int it0, int step, int n) {
  const int t = threadIdx.x;
  if ((it0 + (kBatch - 1) * step + 1) * kIter <= n) {  // uniform over a wavefront
#pragma unroll
    for (int u = 0; u < kBatch; ++u) raw[u] = load_raw4(s, (it0 + u * step) * kIter + 4 * t, n, true);
  } else {
#pragma unroll
    for (int u = 0; u < kBatch; ++u) raw[u] = load_raw4(s, (it0 + u * step) * kIter + 4 * t, n, false);
  }
}
__device__ __forceinline__ Keys4 keys_of(const Raw4& r, int e, int n) {
  Keys4 q;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    q.ok[c] = e + c < n;
    q.k[c] = q.ok[c] ? order_key(r.v[c]) : 0u;
  }
  return q;
}

// Proxy score of one row of a head's key factor: the same fused-multiply-add chain (j
// ascending from 0.0f) as the proxy-score kernels, so the bits agree with theirs.
__device__ __forceinline__ float proxy_score_of_row(const float* __restrict__ Arow,
                                                    const float* __restrict__ qh, int r, int row) {
  const float4* __restrict__ a4 = reinterpret_cast<const float4*>(Arow + (size_t)row * r);
  const int V4 = r / 4;
  float acc = 0.0f;
  for (int c0 = 0; c0 < V4; c0 += 8) {  // 128 bytes of the row in flight (past its end: its last piece)
    float4 a[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] = a4[min(c0 + u, V4 - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = c0 + u;
      if (c >= V4) break;
      acc = __builtin_fmaf(a[u].x, qh[4 * c + 0], acc);
      acc = __builtin_fmaf(a[u].y, qh[4 * c + 1], acc);
      acc = __builtin_fmaf(a[u].z, qh[4 * c + 2], acc);
      acc = __builtin_fmaf(a[u].w, qh[4 * c + 3], acc);
    }
  }
  return acc;
}

// Exact selection of one head from its n materialised scores s: the k positions with the
// largest keys, equal keys by lower position, written to sel[0..k) in ascending position.
// A complete histogram of the top 12 key bits, two 10-bit refinements of the threshold over
// the scores, one pass that sets a bitmap of the selection (positions with the threshold
// key counted in position order) and a prefix count over the bitmap.
// LDS: hist [kBins], bitmap [(n + 31) / 32], sel [k], wave_tot [kWaves], res [4].
// *bin_of_rank receives the 12-bit key prefix of the bin that holds the `rank`-th largest
// score (0 if the head has fewer scores than that).
// With MAKE_LIST false the function stops at the bitmap of the selection (bit e % 32 of word
// e / 32 for position e; complete for every thread on return) and sel is not touched.
template <bool MAKE_LIST>
__device__ __forceinline__ void exact_select_from_scores(const float* s, int n, int k,
                                                         uint32_t rank, uint32_t* hist,
                                                         uint32_t* bitmap, int32_t* sel,
                                                         uint32_t* wave_tot, uint32_t* res,
                                                         uint32_t* bin_of_rank) {
  const int t = threadIdx.x, lane = t & 63;
  const int n_iter = (n + kIter - 1) / kIter;
  const int words = (n + 31) / 32;
  const int wpt = (words + kT - 1) / kT;
  uint32_t bin, above;
  for (int i = t; i < kBins; i += kT) hist[i] = 0u;
  __syncthreads();
  for (int it0 = 0; it0 < n_iter; it0 += kBatch) {
    Raw4 raw[kBatch];
    load_batch(raw, s, it0, 1, n);
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const Keys4 q = keys_of(raw[u], (it0 + u) * kIter + 4 * t, n);
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (q.ok[c]) atomicAdd(&hist[q.k[c] >> kBinShift], 1u);
    }
  }
  __syncthreads();
  {
    uint32_t above_unused;
    find_from_top_4096(hist, rank, wave_tot, res, bin_of_rank, &above_unused);
  }
  find_from_top_4096(hist, (uint32_t)k, wave_tot, res, &bin, &above);
  // refine the threshold inside the bin: two 10-bit levels over the low 20 key bits
  uint32_t prefix = bin, remaining = (uint32_t)k - above;
  int shift = kBinShift;
  for (int level = 0; level < 2; ++level) {
    for (int i = t; i < 2048; i += kT) hist[i] = 0u;
    __syncthreads();
    const int nshift = shift - 10;
    for (int it0 = 0; it0 < n_iter; it0 += kBatch) {
      Raw4 raw[kBatch];
      load_batch(raw, s, it0, 1, n);
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const Keys4 q = keys_of(raw[u], (it0 + u) * kIter + 4 * t, n);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (q.ok[c] && (q.k[c] >> shift) == prefix)
            atomicAdd(&hist[(q.k[c] >> nshift) & 1023u], 1u);
      }
    }
    __syncthreads();
    find_from_top(hist, remaining, wave_tot, res);
    prefix = (prefix << 10) | res[0];
    remaining -= res[1];
    shift = nshift;
    __syncthreads();
  }
  const uint32_t tau = prefix, need_eq = remaining;
  // bitmap of the selection; positions with key == tau are counted in position order
  uint32_t taken = 0;
  for (int it = 0; it < n_iter; ++it) {
    const int e = it * kIter + 4 * t;
    const Keys4 q = keys_of(load_raw4(s, e, n, (it + 1) * kIter <= n), e, n);
    uint32_t cnt = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) cnt += (q.ok[c] && q.k[c] == tau) ? 1u : 0u;
    uint32_t tot;
    uint32_t rk = taken + block_exclusive_scan(cnt, wave_tot, &tot);
    uint32_t nib = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (!q.ok[c]) continue;
      if (q.k[c] > tau) nib |= 1u << c;
      if (q.k[c] == tau) {
        if (rk < need_eq) nib |= 1u << c;
        ++rk;
      }
    }
    taken += tot;
    const uint32_t word = or_reduce8(nib << (4 * (lane & 7)));
    const int wi = e >> 5;
    if ((lane & 7) == 0 && wi < words) bitmap[wi] = word;
  }
  __syncthreads();
  if (!MAKE_LIST) return;
  uint32_t cnt = 0;
  for (int j = 0; j < wpt; ++j)
    if (t * wpt + j < words) cnt += (uint32_t)__popc(bitmap[t * wpt + j]);
  uint32_t tot;
  uint32_t off = block_exclusive_scan(cnt, wave_tot, &tot);
  for (int j = 0; j < wpt; ++j) {
    if (t * wpt + j >= words) break;
    uint32_t wbits = bitmap[t * wpt + j];
    while (wbits) {
      const int bpos = __ffs((int)wbits) - 1;
      wbits &= wbits - 1;
      if (off < (uint32_t)k) sel[off] = (t * wpt + j) * 32 + bpos;
      ++off;
    }
  }
}

// Victim slots for the nm missing positions of a head (Sec. 4.1 hit-and-miss cache; replacement
// by least recent selection: victims in (last_used, slot) order, the j-th miss taking the j-th
// victim), then eviction and installation in the maps.  Called by all 1024 threads.
struct VictimWork {
  // LDS
  int32_t* lu_s;          // [C] last_used, already `step` where used in this step
  const int32_t* to_s;    // [C] token_of before the step
  const int32_t* mt_s;    // [nm] missing positions, ascending
  const int32_t* mj_s;    // [nm] their indices in the outputs
  int32_t* vsorted;       // [nm] receives the victims in rank order
  uint32_t* ahist;        // [kAgeBins], zero
  uint32_t* cls_age;      // [kMaxCls]
  uint32_t* cls_base;     // [kMaxCls]
  uint32_t* sh_ncls;      // zero
  uint32_t* sh_clip;      // zero
  uint32_t* sh_bad;
  uint32_t* scan_areas;   // four areas of 32 words for the prefix counts
  unsigned char* sort_area;  // 8 bytes per slot (C rounded up to a power of two): rare cases only
  // this head's maps and outputs (global)
  int32_t* so;
  int32_t* to;
  int32_t* lu;
  int32_t* ms;
  int32_t* ss;
  int32_t step;
  int C, l, spt;
};
template <int SPT>
__device__ __forceinline__ void assign_victims(const VictimWork& v, int nm) {
  const int t = threadIdx.x;
  const int C = v.C, l = v.l, spt = v.spt;
  const int32_t step = v.step;
  auto scan_area = [&](int i) { return v.scan_areas + (i & 3) * 2 * kWaves; };
  // ages of the slots not used in this step; thread t owns slots [s0, s1)
  const int s0 = min(C, t * spt), s1 = min(C, s0 + spt);
  uint32_t age[SPT];
#pragma unroll
  for (int u = 0; u < SPT; ++u) {
    age[u] = 0xffffffffu;  // not eligible
    if (u < spt && s0 + u < s1) {
      const int32_t lv = v.lu_s[s0 + u];
      if (lv > step) atomicOr(v.sh_clip, 2u);  // (not allowed; ordered by the sort below all the same)
      if (lv != step) {
        age[u] = min((uint32_t)(step - 1 - lv), (uint32_t)(kAgeBins - 1));
        atomicAdd(&v.ahist[age[u]], 1u);
      }
    }
  }
  lds_barrier();
  // scan the age classes from the oldest: eligible slots above each class, and the number of
  // non-empty classes above it.  A non-empty class with fewer than nm slots above it holds
  // victims; its number among those classes is its index in cls_age / cls_base.
  uint32_t n_elig;
  {
    const uint32_t c0b = v.ahist[2 * t], c1b = v.ahist[2 * t + 1];
    const uint32_t e0 = c0b ? 1u : 0u, e1 = c1b ? 1u : 0u;
    uint32_t bc, be, ne;
    scan2(c0b + c1b, e0 + e1, scan_area(3), &bc, &be, &n_elig, &ne);
    const uint32_t above1 = n_elig - bc - c0b - c1b, ne_above1 = ne - be - e0 - e1;
    const uint32_t above0 = above1 + c1b, ne_above0 = ne_above1 + e1;
    if (c1b && above1 < (uint32_t)nm) {
      if (ne_above1 < (uint32_t)kMaxCls) {
        v.cls_age[ne_above1] = 2 * t + 1;
        v.cls_base[ne_above1] = above1;
      }
      atomicMax(v.sh_ncls, ne_above1 + 1);
      if (2 * t + 1 == kAgeBins - 1) atomicOr(v.sh_clip, 1u);
    }
    if (c0b && above0 < (uint32_t)nm) {
      if (ne_above0 < (uint32_t)kMaxCls) {
        v.cls_age[ne_above0] = 2 * t;
        v.cls_base[ne_above0] = above0;
      }
      atomicMax(v.sh_ncls, ne_above0 + 1);
    }
    lds_barrier();
  }
  const int ncls = (int)*v.sh_ncls;
  // ages beyond the histogram's range share its last class, which then does not order them
  const bool clipped = (*v.sh_clip & 2u) != 0u || (*v.sh_clip != 0u && step > kAgeBins - 1);
  int nv = nm;  // number of victims found (< nm only if the caller reused `step`)
  if (n_elig >= (uint32_t)nm && ncls <= kMaxCls && !clipped) {
    // rank of a victim = slots in older classes + its index in its class, in slot order: two
    // classes per prefix count (16-bit fields; there are mostly one to three).  Selection and
    // resolution at 32K with 100 misses in 1, 4, 8, 15 classes: 11.6, 12.0, 13.1, 14.8 us; with four
    // classes per count of two words 12.7, 12.8, 13.8, 15.4.
    for (int c2 = 0; c2 < ncls; c2 += 2) {
      const uint32_t ca0 = v.cls_age[c2], cb0 = v.cls_base[c2];
      const bool two = c2 + 1 < ncls;
      const uint32_t ca1 = two ? v.cls_age[c2 + 1] : 0xfffffffeu, cb1 = two ? v.cls_base[c2 + 1] : 0u;
      uint32_t n01 = 0;
#pragma unroll
      for (int u = 0; u < SPT; ++u) n01 += (age[u] == ca0 ? 1u : 0u) + (age[u] == ca1 ? 1u << 16 : 0u);
      uint32_t tot;
      const uint32_t ex = scan1(n01, scan_area(c2 >> 1), &tot);
      uint32_t before0 = cb0 + (ex & 0xffffu), before1 = cb1 + (ex >> 16);
      if (n01 != 0u) {
#pragma unroll
        for (int u = 0; u < SPT; ++u) {
          const bool is0 = age[u] == ca0, is1 = age[u] == ca1;
          const uint32_t rk = is0 ? before0 : before1;
          if ((is0 || is1) && rk < (uint32_t)nm) v.vsorted[rk] = s0 + u;
          before0 += is0 ? 1u : 0u;
          before1 += is1 ? 1u : 0u;
        }
      }
    }
    lds_barrier();
  } else {
    // out of victims, too many classes, or ages beyond the histogram's range: sort every
    // slot's (last_used, slot) key
    uint64_t* const vlist = reinterpret_cast<uint64_t*>(v.sort_area);
    int Cpad = 2;
    while (Cpad < C) Cpad <<= 1;
    for (int i = t; i < Cpad; i += kT) {
      uint64_t key64 = ~0ull;
      if (i < C && v.lu_s[i] != step)
        key64 = (((uint64_t)(uint32_t)(v.lu_s[i] + 1)) << 32) | (uint32_t)i;
      vlist[i] = key64;
    }
    bitonic_sort_lds(vlist, Cpad);
    nv = (int)min((uint32_t)nm, n_elig);
    for (int jj = t; jj < nv; jj += kT) v.vsorted[jj] = (int32_t)(uint32_t)vlist[jj];
    __syncthreads();
  }
  for (int jj = t; jj < nm; jj += kT) {
    if (jj >= nv) {  // ran out of victims (the caller reused `step`)
      atomicOr(v.sh_bad, 1u);
      v.ms[jj] = -1;
      v.ss[v.mj_s[jj]] = -1;
      continue;
    }
    const int32_t slot = v.vsorted[jj];
    const int32_t tok = v.mt_s[jj];
    const int32_t old = v.to_s[slot];
    if (old >= 0 && old < l) v.so[old] = -1;
    v.to[slot] = tok;
    v.so[tok] = slot;
    v.lu[slot] = step;
    v.ms[jj] = slot;
    v.ss[v.mj_s[jj]] = slot;
  }
}

}  // namespace
}  // namespace lrqk
