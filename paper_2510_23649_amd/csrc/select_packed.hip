// a2 + a3 of the fused step, one workgroup of 1024 threads per (batch, query head), working
// straight from what the proxy-score pass left behind: the candidate bitmap (one 64-bit word
// per group of 64 positions) and the candidates' scores packed 8 per group
// (Alg. 2, top(., k); Sec. 4.1 active / lite tokens and the hit-and-miss cache).
//
// What costs time here is not memory but a chain of short phases, and in them the instructions that a
// wavefront issues for lanes that have nothing to do: candidates are few and unevenly spread over the
// groups.  So they are listed once, in LDS and in position order, and dealt out evenly from then on:
//   * one round of coalesced loads brings a thread's bitmap words and packed scores in (GPT
//     consecutive groups; with what the resolution will need from the cache state: last_used and
//     token_of go to LDS).  A prefix count over the candidates gives each its place in the list, an
//     entry being (key, ~position) as one number, larger = better; candidates beyond the packed ones of
//     a group get their score computed again from A_K and q_hat with the proxy pass's fma chain, dealt
//     out over all threads;
//   * thread t takes entries t E .. t E + E - 1 (E = entries / 1024, mostly 2 to 4) into registers: thread
//     order is position order, and every prefix count over the threads is one in position order;
//   * ONE histogram over (key - threshold key) >> s, 2048 bins (the candidates are the tail
//     of the score distribution above the threshold, so they spread over the bins instead
//     of piling into the two or three bins that fixed key bits would give), is scanned from
//     the top: it gives the bin that holds the k-th largest.  The few candidates of that bin
//     are ranked on (key, position) -- every wavefront does it for itself -- and the one
//     with the right rank is the cut: the selection is every candidate at or above it.  A
//     bin with many candidates (ties) goes through further 11-bit histogram levels and an
//     ordered cut instead;
//   * whether a position is in the cache, and where, is for slot_of to say (a caller that cuts its context
//     back and goes on leaves slots whose token_of names a removed token; tests:
//     test_context_cut_back_and_continued).  It is looked up for the entries from the bin of the cut on,
//     while the cut is found: k cache lines, 4 cycles each at the least.  Looked up before the histogram,
//     for all 1.5 k entries, a step at 4K context takes 0.25 us less and two layers at 128K 0.5 us more.
//     (Every cache slot looking its token_of up in a map of the selection needs no such loads, 0.5 us more
//     at 4K, 3.4 us less at 128K, but answers from the wrong array.)  One prefix count over (selected, missing)
//     gives every entry its place in the outputs;
//   * the same histogram yields the key at rank 1.5 k, which (divided by |q_hat|) is handed
//     to the next step of the layer as its candidate threshold, so that steps after the
//     first need no threshold estimate of their own.
// (Before, a thread kept the candidates of its own groups in registers, 8 a group, from the first load to
// the last store: every phase then had 8 to 16 predicated steps of which most lanes skipped most.  A whole
// step at 4K context, where one wavefront owned all the groups: 23.9 -> 21.0 us.)
// Cycles at 2.3 GHz, one head at 32K: first loads 6200, list 3000, histogram 2000, scan 1900, victims 6500.
// More candidates than the list holds (8192; a threshold carried into a step whose scores it is far too
// low for): a histogram of all of them gives a higher threshold, about that of the 1.5 k largest, and the
// list takes those.  A head with fewer than k candidates, with scores to be
// computed again for more than half of its positions, or with more equal scores than the list holds,
// computes all its scores into the workspace and selects exactly from them (exact_select_from_scores):
// slower, same result.  A whole step at 32 + 8 heads with 4, 6, 12 times k candidates, in us, in
// brackets with all scores computed: 32K, k = 1024: 36, 47, 70 (224); 128K, k = 2048: 65, 73, 147 (743); 34
// and 57 with the usual 1.5.  (With 8 a group in registers and 2048 more in LDS it was 40, 254, 255
// and 62, 69, 821.)
// What is rare is out of the way of the instructions (__builtin_expect): a step at 4K 21.2 -> 20.9 us, two
// layers at 128K 233.3 -> 231.4.
//
// Resolution (Sec. 4.1; least recently selected victims in (last_used, slot) order): a
// histogram of the ages of the slots not used in this step is scanned from the oldest; the
// age classes that hold the n_miss oldest slots are numbered, and a victim's rank is the
// number of slots in older classes plus its index inside its class in slot order -- one
// more prefix count, whatever the number of victims.  Cache state is read from LDS: but for
// candidates beyond the packed ones, the slot_of look-ups are the only dependent global round trip.
//
// All decisions are integer comparisons: the result is exact and independent of scheduling.
#include "lrqk_device.h"
#include "lrqk_internal.h"
#include "select_common.h"

namespace lrqk {
namespace {

constexpr int kPackedMaxK = 4 * kT;             // k
constexpr int kMaxE = 8;                  // list entries per thread
constexpr int kListCap = kMaxE * kT;      // candidates of a head
constexpr int kMaxSpt = 8;    // cache slots per thread (C <= 8192)
constexpr size_t kPackedLdsLimit = 150 * 1024;

__host__ __device__ inline size_t up256(size_t x) { return (x + 255) / 256 * 256; }

// LDS: last_used and token_of [C] each; age and key histograms; the threshold bin's entries; then, in one
// area, one after the other,
//   the list of candidates, or the exact route's histogram and bitmap;
//   [k] miss positions, their output indices, victims in rank order; from 3 k_b on the selection in output
//   order, its positions and slots [k] each, and after them the all-slots sort of the rare resolution cases.
struct PackedArena {
  size_t st_b, k_b, fixed, total;
};
__host__ __device__ inline PackedArena packed_arena(int k, int n, int C) {
  PackedArena a;
  a.st_b = up256((size_t)C * 4);
  a.k_b = up256((size_t)k * 4);
  a.fixed = 2 * a.st_b + (kAgeBins + 2048) * 4 + up256((kSmall + 1) * 8);
  const size_t exact = (size_t)kBins * 4 + up256(((size_t)n + 31) / 32 * 4);
  int Cpad = 2;
  while (Cpad < C) Cpad <<= 1;
  const size_t sort_b = (size_t)Cpad * 8;
  const size_t out = 3 * a.k_b + (2 * a.k_b > sort_b ? 2 * a.k_b : sort_b);
  size_t z = out > exact ? out : exact;
  // (one workgroup is on a compute unit in any case, for its registers: the list has its full size)
  if (z < (size_t)kListCap * 8) z = (size_t)kListCap * 8;
  a.total = a.fixed + z;
  return a;
}

struct PackedArgs {
  const unsigned long long* bitmap;  // [BHq][words64]
  const float* cand_scores;          // [BHq][words64][cand_per_group]
  const uint32_t* thr_used;          // [BHq] key the proxy pass filtered with
  const float* A_K;
  const float* q_hat;
  float* scores_w;  // [BHq][l] scratch of a head that takes the exact route
  float* sel_thr;   // [BHq] threshold / |q_hat| handed to the layer's next step (may be null)
  int words64, r, B, Hq, Hkv, l, lrows, n, k, C;
  int32_t step;
  int32_t* sel_idx;
  int32_t* slot_of;
  int32_t* token_of;
  int32_t* last_used;
  int32_t* sel_slot;
  uint8_t* hit;
  int32_t* miss_tok;
  int32_t* miss_slot;
  int32_t* n_miss;
};

template <int GPT, int SPT, int CPG>
__global__ __launch_bounds__(kT) void select_packed_kernel(const PackedArgs a) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  __shared__ uint32_t wave_tot[4 * 2 * kWaves];  // four areas of 32 words, used in rotation
  auto scan_area = [&](int i) { return wave_tot + (i & 3) * 2 * kWaves; };
  __shared__ uint32_t res[4];
  __shared__ uint32_t sh_again, sh_small_n, sh_bad, sh_ncls, sh_clip;
  __shared__ uint64_t sh_cut;
  __shared__ __align__(16) float qh[128];
  __shared__ uint32_t cls_age[kMaxCls], cls_base[kMaxCls];

  int bh, block;
  place_head(blockIdx.x, a.B, a.Hq, a.Hkv, 1, bh, block);
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int n = a.n, k = a.k, C = a.C, l = a.l, r = a.r;
  const PackedArena az = packed_arena(k, n, C);
  int32_t* const lu_s = reinterpret_cast<int32_t*>(lds_raw);
  int32_t* const to_s = reinterpret_cast<int32_t*>(lds_raw + az.st_b);
  uint32_t* const ahist = reinterpret_cast<uint32_t*>(lds_raw + 2 * az.st_b);
  uint32_t* const hist0 = ahist + kAgeBins;
  uint64_t* const small = reinterpret_cast<uint64_t*>(hist0 + 2048);
  unsigned char* const Z = lds_raw + az.fixed;
  uint64_t* const list = reinterpret_cast<uint64_t*>(Z);
  // (in place of the list, once every thread holds its entries in registers)
  int32_t* const mt_s = reinterpret_cast<int32_t*>(Z);                     // [k] miss positions
  int32_t* const mj_s = reinterpret_cast<int32_t*>(Z + az.k_b);            // their j
  int32_t* const vsorted = reinterpret_cast<int32_t*>(Z + 2 * az.k_b);
  unsigned char* const X = Z + 3 * az.k_b;
  int32_t* const sel_o = reinterpret_cast<int32_t*>(X);                    // [k]
  int32_t* const slot_o = reinterpret_cast<int32_t*>(X + az.k_b);          // [k]

  const int b = bh / a.Hq, h = bh - b * a.Hq, kvh = h / (a.Hq / a.Hkv);
  const float* __restrict__ Arow = a.A_K + ((size_t)b * a.Hkv + kvh) * (size_t)a.lrows * r;
  int32_t* __restrict__ so = a.slot_of + (size_t)bh * a.lrows;
  int32_t* __restrict__ to = a.token_of + (size_t)bh * C;
  int32_t* __restrict__ lu = a.last_used + (size_t)bh * C;
  const int32_t step = a.step;
  // ---- 0. every load that does not depend on the selection -----------------------------------
  // (from clamped addresses and without a branch: a load inside one is waited for before the
  // next is issued.  Whole step at 4K context 24.4 -> 23.9 us, of two layers at 128K 235.3 -> 234.8.)
  const int ngroups = (n + 63) >> 6;
  const unsigned long long* __restrict__ bm = a.bitmap + (size_t)bh * a.words64;
  const float4* __restrict__ cs4 =
      reinterpret_cast<const float4*>(a.cand_scores + (size_t)bh * a.words64 * CPG);
  unsigned long long mask[GPT];
  float4 sc[GPT][CPG / 4];
#pragma unroll
  for (int g = 0; g < GPT; ++g) {
    const int gi = min(t * GPT + g, ngroups - 1);
    mask[g] = bm[gi];
    // a group without candidates holds stale scores; they are never interpreted
#pragma unroll
    for (int i = 0; i < CPG / 4; ++i) sc[g][i] = cs4[CPG / 4 * gi + i];
  }
  // cache state: coalesced loads (slot i by thread i mod 1024), handed over through LDS to
  // the threads that own contiguous runs of slots below
  const int spt = (C + kT - 1) / kT;  // cache slots per thread, <= SPT
  int32_t lu_r[SPT], to_r[SPT];
#pragma unroll
  for (int u = 0; u < SPT; ++u) {
    const int sl = min(u * kT + t, C - 1);
    lu_r[u] = lu[sl];
    to_r[u] = to[sl];
  }
  uint32_t thr_key = a.thr_used[bh];
  const float q_r = a.q_hat[(size_t)bh * r + min(t, r - 1)];  // to LDS (r <= 128)
#pragma unroll
  for (int g = 0; g < GPT; ++g)
    if (t * GPT + g >= ngroups) mask[g] = 0ull;

  for (int i = t; i < 2048 + kAgeBins; i += kT) ahist[i] = 0u;  // ahist and hist0
  if (t == 0) {
    sh_again = 0u;
    sh_small_n = 0u;
    sh_bad = 0u;
    sh_ncls = 0u;
    sh_clip = 0u;
  }

  // ---- 1. the list of candidates -------------------------------------------------------------------
  uint32_t own = 0;
#pragma unroll
  for (int g = 0; g < GPT; ++g) own += (uint32_t)__popcll(mask[g]);
  uint32_t m;
  uint32_t at = scan1(own, scan_area(0), &m);
  float* const sw = a.scores_w + (size_t)bh * l;
  constexpr uint32_t cap = kListCap;
  bool listed = m >= (uint32_t)k && m <= cap;  // uniform
  if (__builtin_expect(listed, 1)) {
#pragma unroll
    for (int g = 0; g < GPT; ++g) {
      unsigned long long mb = mask[g];
      const int base = (t * GPT + g) * 64;
#pragma unroll
      for (int i = 0; i < CPG; ++i)
        if (mb) {
          const float4 q = sc[g][i / 4];
          const float v = i % 4 == 0 ? q.x : i % 4 == 1 ? q.y : i % 4 == 2 ? q.z : q.w;
          list[at++] = value_of(order_key(v), base + __builtin_ctzll(mb));
          mb &= mb - 1ull;
        }
      if (mb) {
        sh_again = 1u;
        while (mb) {  // more candidates than the proxy pass packed: no key yet (no score's key is 0)
          list[at++] = value_of(0u, base + __builtin_ctzll(mb));
          mb &= mb - 1ull;
        }
      }
    }
  } else if (__builtin_expect(m > cap, 0)) {
    // more than the list holds: those from a higher threshold on
    if (t < r) qh[t] = q_r;
    uint32_t beyond = 0, all_beyond;  // candidates without a packed score
#pragma unroll
    for (int g = 0; g < GPT; ++g) beyond += (uint32_t)max((int)__popcll(mask[g]) - CPG, 0);
    const uint32_t ofs = scan1(beyond, scan_area(1), &all_beyond);
    if (2u * all_beyond <= (uint32_t)n) {  // (with more, to compute every score is no dearer)
      // the scores that are missing, into the workspace: listed and dealt out over all threads
      uint32_t* const todo = reinterpret_cast<uint32_t*>(Z);
      for (uint32_t b0 = 0; b0 < all_beyond; b0 += 2u * cap) {
        const uint32_t b1 = min(b0 + 2u * cap, all_beyond);
        uint32_t i = ofs;
#pragma unroll
        for (int g = 0; g < GPT; ++g) {
          unsigned long long mb = mask[g];
#pragma unroll
          for (int c = 0; c < CPG; ++c) mb &= mb - 1ull;
          for (; mb; mb &= mb - 1ull, ++i)
            if (i >= b0 && i < b1) todo[i - b0] = (uint32_t)((t * GPT + g) * 64 + __builtin_ctzll(mb));
        }
        __syncthreads();
        for (uint32_t u = b0 + t; u < b1; u += kT)
          sw[todo[u - b0]] = proxy_score_of_row(Arow, qh, r, (int)todo[u - b0]);
        __threadfence_block();
        __syncthreads();
      }
      // the thread's candidates in position order
      auto for_own = [&](auto&& f) {
#pragma unroll
        for (int g = 0; g < GPT; ++g) {
          unsigned long long mb = mask[g];
          const int base = (t * GPT + g) * 64;
#pragma unroll
          for (int i = 0; i < CPG; ++i)
            if (mb) {
              const float4 q = sc[g][i / 4];
              f(order_key(i % 4 == 0 ? q.x : i % 4 == 1 ? q.y : i % 4 == 2 ? q.z : q.w),
                base + __builtin_ctzll(mb));
              mb &= mb - 1ull;
            }
          for (; mb; mb &= mb - 1ull) {
            const int p = base + __builtin_ctzll(mb);
            f(order_key(sw[p]), p);
          }
        }
      };
      // The lower edge of the bin that holds rank 1.5 k: bins of 2^-7 of a binade above a positive
      // threshold, otherwise (and if the top bin, which takes everything beyond, is reached) of all keys;
      // inside a bin with too many entries once more.
      uint32_t base = thr_key, want = (uint32_t)k + (uint32_t)(k >> 1), above = 0, width = 0;
      int s = thr_key > 0x80800000u && thr_key < 0xff800000u ? 16 : 21;
      for (int level = 0;; ++level) {
        for_own([&](uint32_t kk, int) {
          if (kk >= base && (width == 0u || kk - base < width))
            atomicAdd(&hist0[min((kk - base) >> s, 2047u)], 1u);
        });
        lds_barrier();
        find_two_from_top(hist0, want, want, scan_area(2 + (level & 1)), res);
        const uint32_t d = res[0], ab = res[1], c = hist0[d];
        lds_barrier();  // res and hist0 have been read
        for (int i = t; i < 2048; i += kT) hist0[i] = 0u;
        lds_barrier();
        if (width == 0u && d == 2047u && s == 16) {
          s = 21;
          continue;
        }
        base += d << s;
        above += ab;
        if (above + c <= cap || s == 0) break;
        want -= ab;
        width = 1u << s;
        s = s > 11 ? s - 11 : 0;
      }
      own = 0;
      for_own([&](uint32_t kk, int) { own += kk >= base ? 1u : 0u; });
      at = scan1(own, scan_area(0), &m);
      listed = m <= cap;
      if (listed) {
        for_own([&](uint32_t kk, int p) {
          if (kk >= base) list[at++] = value_of(kk, p);
        });
        thr_key = base;  // what the rest takes for the threshold
      }
    }
  }
  // q_hat and the cache state go to LDS beside it
  if (t < r) qh[t] = q_r;
#pragma unroll
  for (int u = 0; u < SPT; ++u)
    if (u < spt && u * kT + t < C) {
      lu_s[u * kT + t] = lu_r[u];
      to_s[u * kT + t] = to_r[u];
    }
  lds_barrier();
  if (__builtin_expect(sh_again != 0u, 0)) {  // uniform
    for (uint32_t i = t; i < m; i += kT) {
      const uint64_t v = list[i];
      if ((uint32_t)(v >> 32) != 0u) continue;
      const int p = position_of(v);
      list[i] = value_of(order_key(proxy_score_of_row(Arow, qh, r, p)), p);
    }
    lds_barrier();
  }

  const uint32_t rank_next = (uint32_t)k + (uint32_t)(k >> 1);  // candidates wanted next step
  float thr_next;
  uint64_t cut;
  uint64_t val[kMaxE];  // the thread's entries; 0: none
  uint32_t E = 0;
  auto take_entries = [&](uint32_t n_entries) {
    E = (n_entries + kT - 1) / kT;
#pragma unroll
    for (int e = 0; e < kMaxE; ++e) {
      const uint32_t i = (uint32_t)t * E + e;
      val[e] = 0ull;
      if ((uint32_t)e < E && i < n_entries) val[e] = list[i];
    }
  };
  // slot_of of the entries that may be selected (from clamped addresses, as above)
  int32_t slot[kMaxE];
#pragma unroll
  for (int e = 0; e < kMaxE; ++e) slot[e] = -1;
  auto look_up = [&]() {
    auto load = [&](int e) { slot[e] = so[min(max(position_of(val[e]), 0), n - 1)]; };
    load(0);
    load(1);
    if (E > 2u) {
      load(2);
      load(3);
    }
    if (E > 4u) {
#pragma unroll
      for (int e = 4; e < kMaxE; ++e) load(e);
    }
  };
  if (__builtin_expect(listed, 1)) {
    take_entries(m);
    // ---- 2. the cut: histogram of the keys --------------------------------------------------------
    CutWork cw;
    cw.hist0 = hist0;
    cw.hist1 = ahist;
    cw.small = small;
    cw.sh_small_n = &sh_small_n;
    cw.sh_cut = &sh_cut;
    cw.wave_tot = wave_tot;
    cw.res = res;
    int s;
    uint32_t d_next;
    cut = cut_of_entries(val, E, thr_key, (uint32_t)k, rank_next, cw, look_up, &s, &d_next);
    // threshold for the layer's next step: the lower edge of the bin that holds rank 1.5 k, or,
    // with fewer candidates than that, an extrapolation along an exponential tail through
    // (threshold used, m) and (the k-th largest, k)
    if (d_next != 0xffffffffu) {
      thr_next = key_to_float(thr_key + (d_next << s));
    } else {
      const float tau_f = key_to_float((uint32_t)(cut >> 32)), used_f = key_to_float(thr_key);
      float ratio = 8.0f;
      if (m > (uint32_t)k) {
        ratio = __logf(1.5f) / __logf((float)m / (float)k);
        ratio = fminf(fmaxf(ratio, 1.0f), 8.0f);
      }
      thr_next = tau_f - fmaxf(tau_f - used_f, 0.0f) * ratio;
    }
  } else {
    // ---- exact route: all scores of this head, then selection from them ------------------------------
    for (int row = t; row < n; row += kT) sw[row] = proxy_score_of_row(Arow, qh, r, row);
    __threadfence_block();
    __syncthreads();
    uint32_t* const hist = reinterpret_cast<uint32_t*>(Z);
    uint32_t* const bitmap_l = hist + kBins;
    uint32_t bin_next;
    exact_select_from_scores<false>(sw, n, k, rank_next, hist, bitmap_l, nullptr,
                                    wave_tot, res, &bin_next);
    // the selection, listed: every entry is at or above the cut
#pragma unroll
    for (int g = 0; g < GPT; ++g) {
      const int gi = t * GPT + g;
      mask[g] = 0ull;
      if (gi < ngroups) {
        const uint32_t lo = bitmap_l[2 * gi];
        const uint32_t hi = (2 * gi + 1) * 32 < n ? bitmap_l[2 * gi + 1] : 0u;
        mask[g] = ((unsigned long long)hi << 32) | lo;
      }
    }
    own = 0;
#pragma unroll
    for (int g = 0; g < GPT; ++g) own += (uint32_t)__popcll(mask[g]);
    uint32_t tot;
    at = block_exclusive_scan(own, wave_tot, &tot);  // (its barriers: the bitmap has been read)
#pragma unroll
    for (int g = 0; g < GPT; ++g) {
      unsigned long long mb = mask[g];
      while (mb) {
        if (at < (uint32_t)k) list[at] = value_of(1u, (t * GPT + g) * 64 + __builtin_ctzll(mb));
        ++at;
        mb &= mb - 1ull;
      }
    }
    __syncthreads();
    take_entries((uint32_t)k);
    look_up();
    __syncthreads();
    cut = 1ull;
    thr_next = key_to_float(bin_next << kBinShift);  // lower edge of that 12-bit bin
  }
  // ---- 3. places in the outputs: one prefix count over (selected, missing) ---------------------------
  uint32_t nsel = 0, nmiss = 0;
#pragma unroll
  for (int e = 0; e < kMaxE; ++e) {
    if (val[e] < cut) val[e] = 0ull;
    if (slot[e] >= C) slot[e] = -1;  // corrupt map entry: treat as absent
    nsel += val[e] != 0ull ? 1u : 0u;
    nmiss += val[e] != 0ull && slot[e] < 0 ? 1u : 0u;
  }
  uint32_t j, mrank, tot_sel, tot_miss;
  scan2(nsel, nmiss, scan_area(3), &j, &mrank, &tot_sel, &tot_miss);
  const int nm = (int)tot_miss;
#pragma unroll
  for (int e = 0; e < kMaxE; ++e) {
    if ((uint32_t)e >= E) break;  // uniform
    if (val[e] == 0ull || j >= (uint32_t)k) continue;  // (exactly k positions are selected)
    const int p = position_of(val[e]);
    sel_o[j] = p;
    if (slot[e] >= 0) {
      slot_o[j] = slot[e];
    } else {
      slot_o[j] = -1 - (int32_t)mrank;
      mt_s[mrank] = p;
      mj_s[mrank] = (int32_t)j;
      ++mrank;
    }
    ++j;
  }
  lds_barrier();
  // the outputs, coalesced
  int32_t* __restrict__ out = a.sel_idx + (size_t)bh * k;
  int32_t* __restrict__ ss = a.sel_slot + (size_t)bh * k;
  uint8_t* __restrict__ ht = a.hit + (size_t)bh * k;
  int32_t* __restrict__ mt = a.miss_tok + (size_t)bh * k;
  int32_t* __restrict__ ms = a.miss_slot + (size_t)bh * k;
  for (int jj = t; jj < k; jj += kT) {
    const int p = sel_o[jj];
    const int32_t sl = slot_o[jj];
    out[jj] = p;
    ht[jj] = sl >= 0 ? 1 : 0;
    if (sl >= 0) {
      ss[jj] = sl;
      lu[sl] = step;
      lu_s[sl] = step;  // used in this step: never a victim
    } else {
      mt[-1 - sl] = p;
    }
  }
  if (wv == kWaves - 1) {
    // |q_hat|: the next step multiplies by its own
    float q2 = lane < r ? qh[lane] * qh[lane] : 0.0f;
    if (lane + 64 < r) q2 = __builtin_fmaf(qh[lane + 64], qh[lane + 64], q2);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) q2 += __shfl_xor(q2, d);
    if (lane == 0 && a.sel_thr) {
      const float nrm = sqrtf(q2);
      const float v = thr_next / nrm;
      a.sel_thr[bh] = (nrm > 0.0f && isfinite(v)) ? v : __uint_as_float(0x7fc00000u);
    }
  }

  lds_barrier();

  // ---- 4. victims ------------------------------------------------------------------------------------
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
    v.sort_area = X;
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
  if (t == 0) a.n_miss[bh] = sh_bad ? -1 : nm;
}

template <int GPT, int SPT, int CPG>
hipError_t launch_inst(const PackedArgs& a, int BHq, size_t lds, hipStream_t st) {
  static std::atomic<uint64_t> raised{0};  // devices on which this instantiation's ceiling is up
  const hipError_t e =
      raise_dynamic_lds_once(select_packed_kernel<GPT, SPT, CPG>,
                             kPackedLdsLimit, raised);
  if (e != hipSuccess) return e;
  LRQK_LAUNCH((select_packed_kernel<GPT, SPT, CPG>), dim3(BHq), dim3(kT), lds, st, a);
  return hipGetLastError();
}
template <int GPT, int CPG>
hipError_t launch_gpt(const PackedArgs& a, int BHq, size_t lds, hipStream_t st) {
  if (a.C <= 2 * kT) return launch_inst<GPT, 2, CPG>(a, BHq, lds, st);
  if (a.C <= 4 * kT) return launch_inst<GPT, 4, CPG>(a, BHq, lds, st);
  return launch_inst<GPT, 8, CPG>(a, BHq, lds, st);
}

}  // namespace

int cand_per_group(const lrqk_shape& s) {
  const int groups = filter_words64(s.l - s.w);
  return groups <= kT && 3L * s.k > 5L * groups && select_packed_fits(s) ? 2 * kCandPerGroup
                                                                         : kCandPerGroup;
}

bool select_packed_fits(const lrqk_shape& s) {
  const int n = s.l - s.w;
  if (((n + 63) >> 6) > 4 * kT) return false;  // at most 4 groups of 64 positions per thread
  if (s.C > kMaxSpt * kT || s.k > kPackedMaxK) return false;
  // Dense selections (k a sizeable fraction of the context) put many candidates into most groups;
  // of the 1.5 k that the threshold aims at, few may be left for their scores to be computed again
  if ((long)s.k + s.k / 2 - (long)kCandPerGroup * ((n + 63) >> 6) > 1024) return false;
  return packed_arena(s.k, n, s.C).total <= kPackedLdsLimit;
}

hipError_t launch_select_packed(const lrqk_shape& s, const unsigned long long* bitmap,
                                const float* cand_scores, const uint32_t* thr_used,
                                const float* A_K, const float* q_hat, float* scores_w,
                                float* sel_thr, int32_t* sel_idx, int32_t step, int32_t* slot_of,
                                int32_t* token_of, int32_t* last_used, int32_t* sel_slot,
                                uint8_t* hit, int32_t* miss_tok, int32_t* miss_slot,
                                int32_t* n_miss, hipStream_t st) {
  const int n = s.l - s.w;
  PackedArgs a;
  a.bitmap = bitmap;
  a.cand_scores = cand_scores;
  a.thr_used = thr_used;
  a.A_K = A_K;
  a.q_hat = q_hat;
  a.scores_w = scores_w;
  a.sel_thr = sel_thr;
  a.words64 = filter_words64(n);
  a.r = s.r;
  a.B = s.B;
  a.Hq = s.Hq;
  a.Hkv = s.Hkv;
  a.l = s.l;
  a.lrows = row_cap(s);
  a.n = n;
  a.k = s.k;
  a.C = s.C;
  a.step = step;
  a.sel_idx = sel_idx;
  a.slot_of = slot_of;
  a.token_of = token_of;
  a.last_used = last_used;
  a.sel_slot = sel_slot;
  a.hit = hit;
  a.miss_tok = miss_tok;
  a.miss_slot = miss_slot;
  a.n_miss = n_miss;
  const size_t lds = packed_arena(s.k, n, s.C).total;
  const int groups = (n + 63) >> 6;
  const int BHq = s.B * s.Hq;
  if (cand_per_group(s) > kCandPerGroup) return launch_gpt<1, 2 * kCandPerGroup>(a, BHq, lds, st);
  if (groups <= kT) return launch_gpt<1, kCandPerGroup>(a, BHq, lds, st);
  if (groups <= 2 * kT) return launch_gpt<2, kCandPerGroup>(a, BHq, lds, st);
  if (groups <= 3 * kT) return launch_gpt<3, kCandPerGroup>(a, BHq, lds, st);
  return launch_gpt<4, kCandPerGroup>(a, BHq, lds, st);
}

}  // namespace lrqk
