// a2 from materialised scores, contexts of up to 65536 rankable positions: the k positions of [0, n) with
// the largest scores, equal ones by lower position, ascending (Alg. 2, top(., k)).  One workgroup of 1024
// threads per (batch, query head).
//
// A chain of short phases in one workgroup, as in the fused step's selection (select_packed.hip), from the
// score array instead of the proxy pass's bitmap and packed scores:
//   * the head's scores come into registers in ONE round of loads (four in a row per thread and 4096
//     positions), so that what follows reads memory only for the candidates;
//   * a histogram of the top 12 key bits over one position in eight (all of them in short contexts) gives a
//     bin at or below the one of the k-th largest, with a margin;
//   * the positions from that bin on go to a bitmap in LDS, and from it, by one prefix count, to an ascending
//     list of candidates, whose scores are read back (one round trip, from the L2 that has just
//     delivered them); thread t takes entries t E .. t E + E - 1 of it;
//   * one histogram over their own key range, the few in the bin of the k-th largest ranked directly
//     (cut_of_entries), one prefix count for their places.
// A head with fewer than k candidates or more than the list holds (a sample that misleads, massive ties)
// goes through exact_select_from_scores, which reads the scores as often as it needs.
// At 32 heads, l = 50001, k = 1000 the kernel takes 10.9 us, 20.0 with two passes over the scores in batches of
// eight loads and a three-level radix select over fixed key bits (select_resolve.hip, which still takes
// longer contexts: more than 64 scores a thread would not stay in registers); the chain of stand-alone calls
// 77.7 instead of 87.2.  Cycles at 2.3 GHz: loads 4500, sample 4600, scan 1200, bitmap 5500, list and read-back
// 2300, cut 5500, places 1300.
#include "lrqk_device.h"
#include "lrqk_internal.h"
#include "select_common.h"

namespace lrqk {
namespace {

constexpr int kMaxE = 8;              // list entries per thread
constexpr int kListCap = kMaxE * kT;  // candidates of a head
constexpr int kMaxNV = 16;            // groups of four scores per thread

template <int NV>
__global__ __launch_bounds__(kT) void select_scores_kernel(const float* __restrict__ scores, int l, int n,
                                                           int k, int32_t* __restrict__ sel_idx) {
  static_assert(2 * 2048 == kBins, "the first histogram's memory holds the two of the cut");
  __shared__ __align__(16) uint32_t hist[kBins];
  __shared__ __align__(16) uint32_t bitmap[kMaxNV * kIter / 32];
  __shared__ int32_t clist[kListCap];
  __shared__ uint64_t small[kSmall];
  __shared__ uint32_t wave_tot[4 * 2 * kWaves];  // four areas of 32 words, used in rotation
  __shared__ uint32_t res[4];
  __shared__ uint32_t sh_small_n;
  __shared__ uint64_t sh_cut;
  auto scan_area = [&](int i) { return wave_tot + (i & 3) * 2 * kWaves; };
  const int bh = blockIdx.x, t = threadIdx.x, lane = t & 63;
  const float* __restrict__ s = scores + (size_t)bh * l;

  Raw4 raw[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) raw[j] = load_raw4(s, j * kIter + 4 * t, n, (j + 1) * kIter <= n);
  reinterpret_cast<uint4*>(hist)[t] = make_uint4(0u, 0u, 0u, 0u);
  if (t == 0) {
    res[0] = 0u;
    sh_small_n = 0u;
  }
  lds_barrier();
  // ---- 1. a bin at or below that of the k-th largest ------------------------------------------------
  // (One in eight: of every other thread's four scores one, another one in the next 4096 positions; the rank
  // taken lies 5.5, 5.0 and 5.0 standard deviations beyond the k-th at k = 128, 256 and 512.  At n = 20000 and
  // 60000, 32 heads, the kernel takes 8.0 and 11.4 us with the sample at k = 512, 9.6 and 17.0 counting all
  // at k = 511; sampled from k = 128 on it would take 7.8 and 11.2 there.  The line is that of the kernel for
  // longer contexts, select_resolve.hip.)
  const bool sampled = n >= 16384 && k >= 512;
  auto count = [&](float v) { atomicAdd(&hist[order_key(v) >> kBinShift], 1u); };
  if (sampled) {
#pragma unroll
    for (int j = 0; j < NV; ++j)
      if (((t ^ j) & 1) == 0 && ((j + 1) * kIter <= n || j * kIter + 4 * t + (j & 3) < n)) count(raw[j].v[j & 3]);
  } else {
#pragma unroll
    for (int j = 0; j < NV; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if ((j + 1) * kIter <= n || j * kIter + 4 * t + c < n) count(raw[j].v[c]);
  }
  lds_barrier();
  {
    const uint32_t ks = (uint32_t)(k + 7) / 8;
    const uint32_t want = sampled ? ks + (ks * 3) / 8 + 16 : (uint32_t)k;
    const uint4 h = reinterpret_cast<const uint4*>(hist)[t];
    const uint32_t own = (h.x + h.y) + (h.z + h.w);
    uint32_t total;
    const uint32_t below = scan1(own, scan_area(0), &total);
    uint32_t above = total - below - own;  // (in the bins of the threads after this one)
    const uint32_t cnt[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
    for (int c = 3; c >= 0; --c) {
      if (above < want && want <= above + cnt[c]) res[0] = 4 * t + c;
      above += cnt[c];
    }
  }
  lds_barrier();
  const uint32_t b_lo = res[0];
  // ---- 2. the candidates, in position order -----------------------------------------------------------
  reinterpret_cast<uint4*>(hist)[t] = make_uint4(0u, 0u, 0u, 0u);
  // (what takes time here are the instructions for every score; where the bin's lower edge is a positive number
  // its bits compare with a score's as signed integers as their keys do, and no key is needed: this phase
  // 10300 -> 5500 cycles at n = 49941)
  auto mark = [&](auto at_or_above) {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int e = j * kIter + 4 * t;
      uint32_t nib = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) nib |= at_or_above(raw[j].v[c]) ? 1u << c : 0u;
      if ((j + 1) * kIter > n) nib &= (1u << min(max(n - e, 0), 4)) - 1u;  // (scores that exist)
      const uint32_t word = or_reduce8(nib << (4 * (lane & 7)));
      if ((lane & 7) == 0) bitmap[e >> 5] = word;
    }
  };
  if (__builtin_expect(b_lo > 0x800u, 1)) {
    const int edge = (int)((b_lo << kBinShift) & 0x7fffffffu);
    mark([&](float v) { return __float_as_int(v) >= edge; });
  } else {
    mark([&](float v) { return (order_key(v) >> kBinShift) >= b_lo; });
  }
  lds_barrier();
  constexpr int kWords = NV * kIter / 32, kWpt = (kWords + kT - 1) / kT;
  uint32_t bits[kWpt], own = 0, m;
#pragma unroll
  for (int j = 0; j < kWpt; ++j) {
    const int w = t * kWpt + j;
    bits[j] = w < kWords ? bitmap[min(w, kWords - 1)] : 0u;
    own += (uint32_t)__popc(bits[j]);
  }
  uint32_t at = scan1(own, scan_area(1), &m);
  if (__builtin_expect(m < (uint32_t)k || m > (uint32_t)kListCap, 0)) {  // uniform
    uint32_t bin_unused;
    exact_select_from_scores<true>(s, n, k, (uint32_t)k, hist, bitmap, clist, wave_tot, res, &bin_unused);
    __syncthreads();
    for (int i = t; i < k; i += kT) sel_idx[(size_t)bh * k + i] = clist[i];
    return;
  }
#pragma unroll
  for (int j = 0; j < kWpt; ++j)
    for (uint32_t b = bits[j]; b; b &= b - 1u) clist[at++] = (t * kWpt + j) * 32 + __builtin_ctz(b);
  lds_barrier();
  const uint32_t E = (m + kT - 1) / kT;
  int pos[kMaxE];
  float v[kMaxE];
#pragma unroll
  for (int e = 0; e < kMaxE; ++e) {
    pos[e] = clist[min((uint32_t)t * E + min((uint32_t)e, E - 1u), m - 1u)];
    v[e] = 0.0f;
  }
  v[0] = s[pos[0]];
  v[1] = s[pos[1]];
  if (E > 2u) {  // uniform
    v[2] = s[pos[2]];
    v[3] = s[pos[3]];
  }
  if (E > 4u) {
#pragma unroll
    for (int e = 4; e < kMaxE; ++e) v[e] = s[pos[e]];
  }
  uint64_t val[kMaxE];  // the thread's entries; 0: none
#pragma unroll
  for (int e = 0; e < kMaxE; ++e)
    val[e] = (uint32_t)e < E && (uint32_t)t * E + e < m ? value_of(order_key(v[e]), pos[e]) : 0ull;
  // ---- 3. the cut, and the places of what is at or above it --------------------------------------------
  CutWork cw;
  cw.hist0 = hist;
  cw.hist1 = hist + 2048;
  cw.small = small;
  cw.sh_small_n = &sh_small_n;
  cw.sh_cut = &sh_cut;
  cw.wave_tot = scan_area(0);
  cw.res = res;
  int shift;
  uint32_t d_unused;
  const uint64_t cut =
      cut_of_entries(val, E, b_lo << kBinShift, (uint32_t)k, (uint32_t)k, cw, [] {}, &shift, &d_unused);
  uint32_t nsel = 0, tot;
#pragma unroll
  for (int e = 0; e < kMaxE; ++e) nsel += val[e] != 0ull && val[e] >= cut ? 1u : 0u;
  uint32_t j = scan1(nsel, scan_area(3), &tot);
#pragma unroll
  for (int e = 0; e < kMaxE; ++e)
    if (val[e] != 0ull && val[e] >= cut && j < (uint32_t)k)  // (exactly k positions are selected)
      sel_idx[(size_t)bh * k + j++] = position_of(val[e]);
}

}  // namespace

bool select_scores_fits(const lrqk_shape& s) { return s.l - s.w <= kMaxNV * kIter; }

hipError_t launch_select_scores(const lrqk_shape& s, const float* scores, int32_t* sel_idx, hipStream_t st) {
  const int n = s.l - s.w, nv = ceil_div(n, kIter);
  auto run = [&](auto kernel) {
    LRQK_LAUNCH(kernel, dim3(s.B * s.Hq), dim3(kT), 0, st, scores, s.l, n, s.k, sel_idx);
    return hipGetLastError();
  };
  // A kernel goes over its NV groups of 4096 scores whether they exist or not, 0.4 us a group at 32 heads (7.0 us for
  // two, 11.3 for 16); with these eight at most two groups are gone over for nothing.
  if (nv <= 1) return run(select_scores_kernel<1>);
  if (nv <= 2) return run(select_scores_kernel<2>);
  if (nv <= 4) return run(select_scores_kernel<4>);
  if (nv <= 6) return run(select_scores_kernel<6>);
  if (nv <= 8) return run(select_scores_kernel<8>);
  if (nv <= 10) return run(select_scores_kernel<10>);
  if (nv <= 13) return run(select_scores_kernel<13>);
  return run(select_scores_kernel<kMaxNV>);
}

}  // namespace lrqk
