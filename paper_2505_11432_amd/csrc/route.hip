// Gating and row map (Section 2.1: top-k gate; Section 3.2 "Efficient operators": the mapping from
// input rows to output rows is computed once from the routing result; Section 4.2: rows ordered by
// expert, then by source).  The paper lists the "multitude of small operators" of the gate as a
// launch-latency straggler (Section 7); here the whole step is two or three launches and no host read-back:
//   1. route_topk_kernel   per token: k-fold arg-max under the total order (logit desc, id asc) by DPP exchanges
//                          inside groups of <= 16 lanes (4+ tokens per wave at a time), softmax over the
//                          selected logits, per-chunk expert histogram
//   2. route_scan_kernel   one wave per expert: exclusive scan of its per-chunk counts (left out while the
//                          histogram is small enough for every workgroup of 3. to sum it itself)
//   3. route_rank_kernel   offsets = scan of the counts; stable rank of every assignment inside its
//                          expert: equal-expert lanes found with one ballot per bit of the expert id
// All three are bound by latency (dependent steps, launches), not by bytes.  Kernel times before (shuffles, four
// rounds of tokens per workgroup, one wave ranking a chunk 64 at a time) and now, E = 64, k = 8: T = 257 1. 23.8 -> 6.7 us,
// 2. 5.1 -> none, 3. 9.2 -> 4.9; T = 4096 20.5 -> 7.0, 4.6 -> none, 6.5 -> 4.2; T = 16384 24.8 -> 8.2, 5.1 -> none,
// 10.0 -> 7.4.
// No atomics decide an order, so perm / inv_perm are unique and reproducible bit for bit.
#include "lane_groups.h"
#include "moe_common.h"

namespace moe {
namespace {

// The total order of the gate: a logit's bits mapped to an unsigned order, -0 as +0, a NaN of either sign below -inf (1: it is
// selected only when nothing else is left, and read back as a NaN).  0 is no logit.  Between lanes the complement of the
// expert id follows as low word: larger = first, equal logits in ascending order of their ids.
__device__ __forceinline__ unsigned order_key(float z) {
  const unsigned b = __float_as_uint(z + 0.0f);
  return z != z ? 1u : b ^ ((unsigned)((int)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float key_logit(unsigned u) { return __uint_as_float((u >> 31) ? (u & 0x7fffffffu) : ~u); }

// G lanes (G <= 16) cooperate on one token; lane `sub` of a group holds the VPL experts sub, sub+G, sub+2G, ...  64 groups
// per workgroup: a chunk of 64 tokens is one round.  hist strides: he per expert, hc per chunk.  Many tokens of many experts
// are bound by the vector ALU: a lane picks its best on 32-bit keys, and only that one is exchanged together with its id (64-bit
// keys throughout: whole route of T = 262144, E = 256, k = 1 141 us, now 57, T = 65536 38.5, now 27.9).
template <int G, int VPL>
__global__ void __launch_bounds__(64 * G) route_topk_kernel(const float* __restrict__ logits, int T, int E, int k,
                                                            int renorm, int chunk_tokens, int he, int hc,
                                                            int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                            int32_t* __restrict__ chunk_hist,
                                                            float* __restrict__ score) {
  __shared__ int hist[MOE_MAX_EXPERTS];
  for (int e = threadIdx.x; e < MOE_MAX_EXPERTS; e += blockDim.x) hist[e] = 0;
  __syncthreads();

  const int sub = threadIdx.x % G;
  const int grp = threadIdx.x / G;
  constexpr int ngroups = 64;
  const int t_begin = blockIdx.x * chunk_tokens;
  const int t_end = min(t_begin + chunk_tokens, T);

  // all groups of a wave run the same number of rounds (the exchanges need every lane active; a group past
  // the end of the chunk works on the last token again and skips the stores)
  const int rounds = (t_end - t_begin + ngroups - 1) / ngroups;
  for (int it = 0; it < rounds; ++it) {
    const int t_raw = t_begin + it * ngroups + grp;
    const bool live = t_raw < t_end;
    const int t = live ? t_raw : t_end - 1;
    float v[VPL];
    unsigned key[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int e = sub + i * G;
      v[i] = e < E ? logits[(long)t * E + e] : -INFINITY;
      key[i] = e < E ? order_key(v[i]) : 0u;
    }
    unsigned long long mine = 0;
    float top_z = 0.f;
    for (int j = 0; j < k; ++j) {
      unsigned top = key[0];
      int at = 0;
#pragma unroll
      for (int i = 1; i < VPL; ++i) {                // a lane's ids ascend: the first of equal keys stays
        at = key[i] > top ? i : at;
        top = key[i] > top ? key[i] : top;
      }
      unsigned long long best = ((unsigned long long)top << 32) | (unsigned)~(sub + at * G);
      best = group_reduce<G>(best, [](unsigned long long a, unsigned long long b) { return a > b ? a : b; });
      const int won = (int)~(unsigned)best - sub;    // the owner retires the winner
#pragma unroll
      for (int i = 0; i < VPL; ++i) key[i] = won == i * G ? 0u : key[i];
      if (sub == j) mine = best;                     // lane j keeps slot j (k <= min(E, 16) <= G)
      if (j == 0) top_z = key_logit((unsigned)(best >> 32));
    }
    const int my_e = (int)~(unsigned)mine;
    // weights: softmax over the selected logits (renorm) or over all logits read at the selected ones
    const bool holds_slot = sub < k;
    const float ex = holds_slot ? expf(key_logit((unsigned)(mine >> 32)) - top_z) : 0.f;
    float den_all = 0.f;
    if (!renorm || score != nullptr) {
#pragma unroll
      for (int i = 0; i < VPL; ++i)
        if (sub + i * G < E) den_all += expf(v[i] - top_z);
      den_all = group_sum<G>(den_all);
    }
    const float den = renorm ? group_sum<G>(ex) : den_all;
    if (live && holds_slot) {
      topk_idx[(long)t * k + sub] = my_e;
      topk_w[(long)t * k + sub] = ex / den;
      if (score != nullptr) score[(long)t * k + sub] = ex / den_all;     // affinity: softmax over all experts
      atomicAdd(&hist[my_e], 1);     // integer count: the sum does not depend on the order
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += blockDim.x) chunk_hist[(long)e * he + (long)blockIdx.x * hc] = hist[e];
}

// One wave per expert: exclusive prefix of that expert's per-chunk counts, in place; counts[e] = total.
__global__ void __launch_bounds__(64) route_scan_kernel(int32_t* __restrict__ chunk_hist, int nchunks,
                                                        int32_t* __restrict__ counts) {
  const int e = blockIdx.x, lane = threadIdx.x;
  int32_t* row = chunk_hist + (long)e * nchunks;
  const int per_lane = (nchunks + 63) / 64;          // nchunks <= 1024 -> at most 16
  const int c0 = lane * per_lane;
  int vals[16];
  int sum = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    vals[i] = (i < per_lane && c0 + i < nchunks) ? row[c0 + i] : 0;
    sum += vals[i];
  }
  int incl = sum;                                    // inclusive scan of the lane sums across the wave
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  int run = incl - sum;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (i < per_lane && c0 + i < nchunks) row[c0 + i] = run;
    run += vals[i];
  }
  if (lane == 63) counts[e] = incl;
}

// A workgroup per chunk ranks its assignments 512 at a time, one wave per 64 in order.  Lanes with the same expert are
// found with one ballot per bit of the expert id; a wave's highest lane of each expert publishes the wave's count, the
// counts of the eight waves are added up per expert, and a lane's row is its wave's start plus the lower equal lanes.
// Only experts in [e_lo, e_hi) get rows (one GPU's expert-parallel share: the local scatter of Section 3.2);
// assignments to other experts get inv_perm = -1.  offsets has e_hi - e_lo + 1 entries.
// SUMS: chunk_hist holds the raw counts [nchunks][E]; every workgroup adds them up itself and workgroup 0 writes counts.
// Otherwise chunk_hist holds the scanned ones [E][nchunks], and counts was written by route_scan_kernel.
constexpr int kRankWaves = 8;
template <bool SUMS>
__global__ void __launch_bounds__(64 * kRankWaves) route_rank_kernel(const int32_t* __restrict__ topk_idx, int T, int E, int k,
                                                                     int e_lo, int e_hi, int chunk_tokens, int nchunks,
                                                                     const int32_t* __restrict__ chunk_hist,
                                                                     int32_t* __restrict__ counts,
                                                                     int32_t* __restrict__ offsets,
                                                                     int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
                                                                     const uint8_t* __restrict__ keep) {
  __shared__ int next_row[MOE_MAX_EXPERTS];                    // first: assignments of earlier chunks
  __shared__ int total[MOE_MAX_EXPERTS];
  __shared__ int expert_off[MOE_MAX_EXPERTS + 1];
  __shared__ int wave_cnt[kRankWaves][MOE_MAX_EXPERTS];
  constexpr int kThreads = 64 * kRankWaves;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long a_begin = (long)blockIdx.x * chunk_tokens * k;
  const long a_end = min((long)(blockIdx.x + 1) * chunk_tokens, (long)T) * k;
  const long a_first = a_begin + threadIdx.x;
  int e_next = a_first < a_end ? topk_idx[a_first] : -1;        // in flight while the tables are built
  for (int i = threadIdx.x; i < kRankWaves * MOE_MAX_EXPERTS; i += kThreads) (&wave_cnt[0][0])[i] = 0;
  if constexpr (SUMS) {
    for (int e = threadIdx.x; e < E; e += kThreads) { next_row[e] = 0; total[e] = 0; }
    __syncthreads();
    int width = 1;                                              // threads side by side over the experts
    while (width < E) width <<= 1;
    const int e = threadIdx.x & (width - 1), step = kThreads / width;
    if (e < E) {
      int all = 0, before = 0;
#pragma unroll 8
      for (int c = threadIdx.x / width; c < nchunks; c += step) {
        const int h = chunk_hist[(long)c * E + e];
        all += h;
        before += c < (int)blockIdx.x ? h : 0;
      }
      atomicAdd(&total[e], all);                                // (LDS; integer sums do not depend on the order)
      atomicAdd(&next_row[e], before);
    }
  } else {
    for (int e = threadIdx.x; e < E; e += kThreads) {
      total[e] = counts[e];
      next_row[e] = chunk_hist[(long)e * nchunks + blockIdx.x];
    }
  }
  __syncthreads();
  // offsets = exclusive scan of the counts (every workgroup recomputes it; workgroup 0 publishes it)
  if (wave == 0) {
    int run = 0;
    for (int e0 = 0; e0 < E; e0 += 64) {
      const int e = e0 + lane;
      const int c = (e >= e_lo && e < e_hi) ? total[e] : 0;
      int incl = c;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
      }
      if (e < E) expert_off[e] = run + incl - c;
      run += __builtin_amdgcn_readlane(incl, 63);
    }
    if (lane == 0) expert_off[E] = run;
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int e = e_lo + threadIdx.x; e <= e_hi; e += kThreads) offsets[e - e_lo] = expert_off[e];
    if constexpr (SUMS)
      for (int e = threadIdx.x; e < E; e += kThreads) counts[e] = total[e];
  }
  for (int e = threadIdx.x; e < E; e += kThreads) next_row[e] += expert_off[e];

  int ebits = 0;
  while ((1 << ebits) < E) ++ebits;
  const unsigned long long lt_mask = (1ull << lane) - 1ull;
  for (long base = a_begin; base < a_end; base += kThreads) {
    const long a = base + threadIdx.x;
    const bool valid = a < a_end;
    const int e = valid ? e_next : 0;
    if (a + kThreads < a_end) e_next = topk_idx[a + kThreads];
    const bool gets_row = valid && e >= e_lo && e < e_hi && (keep == nullptr || keep[a] != 0);
    unsigned long long same = __ballot(gets_row);
    for (int b = 0; b < ebits; ++b) {
      const unsigned long long mb = __ballot((e >> b) & 1);
      same &= ((e >> b) & 1) ? mb : ~mb;
    }
    if (gets_row && (same >> lane) >> 1 == 0) wave_cnt[wave][e] = __popcll(same);    // the group's highest lane
    __syncthreads();
    for (int x = threadIdx.x; x < E; x += kThreads) {
      int run = next_row[x];
#pragma unroll
      for (int w = 0; w < kRankWaves; ++w) {
        const int c = wave_cnt[w][x];
        wave_cnt[w][x] = run;
        run += c;
      }
      next_row[x] = run;
    }
    __syncthreads();
    if (gets_row) {
      const int r = wave_cnt[wave][e] + __popcll(same & lt_mask);
      inv_perm[a] = r;
      perm[r] = (int)a;
    } else if (valid) {
      inv_perm[a] = -1;
    }
    if (base + kThreads < a_end) {
      __syncthreads();
      for (int i = threadIdx.x; i < kRankWaves * MOE_MAX_EXPERTS; i += kThreads) (&wave_cnt[0][0])[i] = 0;
      __syncthreads();
    }
  }
}

// d_logits of 256 / G tokens per workgroup, G lanes per token as in route_topk_kernel: the token's softmax (renorm = 0) and
// the sum over its slots once, the row assembled in LDS (zeros or -p * inner, then the k selected entries) and written whole.
// Bound by writing [T,E]; with renorm = 0 a thread per (token, expert) that redoes the softmax needs E times the
// exponentials (moe_route + moe_route_bwd, T = 16384, E = 160: 302 -> 29 us; renorm = 1, T = 16384, E = 64, this kernel: 12.2 -> 5.2 us).
template <int G, int VPL>
__global__ void __launch_bounds__(256) route_bwd_kernel(const float* __restrict__ logits,
                                                        const int32_t* __restrict__ topk_idx,
                                                        const float* __restrict__ topk_w,
                                                        const float* __restrict__ d_topk_w, int T, int E, int k,
                                                        int renorm, float* __restrict__ d_logits) {
  constexpr int TOKENS = 256 / G;
  __shared__ float rows[TOKENS * G * VPL];                      // [TOKENS][E], E <= G * VPL
  const int sub = threadIdx.x % G, grp = threadIdx.x / G;
  const int t0 = blockIdx.x * TOKENS, t = min(t0 + grp, T - 1);
  int e_j = -1;
  float w = 0.f, dw = 0.f;
  if (sub < k) {
    e_j = topk_idx[(long)t * k + sub];
    w = topk_w[(long)t * k + sub];
    dw = d_topk_w[(long)t * k + sub];
  }
  const float inner = group_sum<G>(w * dw);
  float p[VPL];
#pragma unroll
  for (int i = 0; i < VPL; ++i) p[i] = 0.f;
  if (!renorm) {
    float m = -INFINITY, den = 0.f;
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      p[i] = sub + i * G < E ? logits[(long)t * E + sub + i * G] : -INFINITY;
      m = fmaxf(m, p[i]);
    }
    m = group_max<G>(m);
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      p[i] = sub + i * G < E ? expf(p[i] - m) : 0.f;
      den += p[i];
    }
    den = group_sum<G>(den);
#pragma unroll
    for (int i = 0; i < VPL; ++i) p[i] = p[i] / den;
  }
#pragma unroll
  for (int i = 0; i < VPL; ++i)
    if (sub + i * G < E) rows[grp * E + sub + i * G] = 0.f - p[i] * inner;      // (no -0 for an expert without a share)
  __syncthreads();
  if ((unsigned)e_j < (unsigned)E) rows[grp * E + e_j] += renorm ? w * dw - w * inner : w * dw;
  __syncthreads();
  const int n = min(TOKENS, T - t0) * E;
  for (int i = threadIdx.x; i < n; i += 256) d_logits[(long)t0 * E + i] = rows[i];
}


// ---- device-level token dropping (Section 3.2 "Load balance": capacity per device, the experts of one GPU form
// a group, as in DeepSeek-V2: when a device gets more than `capacity` assignments the ones with the lowest
// affinity are dropped) -------------------------------------------------------------------------------------
// Order of an assignment inside its device: key = affinity bits (positive floats order like integers) in the
// high word, ~assignment id in the low word, so larger key = kept first and equal affinities keep the lower id.
// The capacity-th largest key of every device is found by a most-significant-digit radix select, 8 bits per
// pass: one kernel counts the digit of every key that still matches the device's prefix (integer atomics: the
// counts do not depend on the order), one small kernel picks the digit and narrows the prefix.
struct SelectState {
  unsigned long long prefix[MOE_MAX_EXPERTS];     // high bits of the threshold found so far, per device
  int remaining[MOE_MAX_EXPERTS];                 // rank of the threshold among the keys that match the prefix
  int all_kept[MOE_MAX_EXPERTS];                  // device has no more than `capacity` assignments
  int hist[MOE_MAX_EXPERTS][256];
};

__device__ __forceinline__ unsigned long long drop_key(float score, long a) {
  return ((unsigned long long)__float_as_uint(score) << 32) | (unsigned long long)(0xffffffffu - (unsigned)a);
}

__global__ void __launch_bounds__(256) select_init_kernel(SelectState* st, int n_groups, int capacity) {
  for (int i = threadIdx.x; i < MOE_MAX_EXPERTS * 256; i += blockDim.x) (&st->hist[0][0])[i] = 0;
  for (int g = threadIdx.x; g < n_groups; g += blockDim.x) {
    st->prefix[g] = 0ull;
    st->remaining[g] = capacity;
    st->all_kept[g] = 0;
  }
}

// LDS_GROUPS > 0: the block counts into LDS first (up to 16 devices) and adds its totals once; otherwise straight
// into the global histogram.
template <int LDS_GROUPS>
__global__ void __launch_bounds__(256) select_count_kernel(const int32_t* __restrict__ topk_idx,
                                                           const float* __restrict__ score, long M, int per_group,
                                                           int n_groups, int pass, SelectState* st) {
  __shared__ int h[LDS_GROUPS > 0 ? LDS_GROUPS : 1][256];
  if constexpr (LDS_GROUPS > 0) {
    for (int i = threadIdx.x; i < LDS_GROUPS * 256; i += blockDim.x) (&h[0][0])[i] = 0;
    __syncthreads();
  }
  const int shift = 56 - 8 * pass;
  for (long a = blockIdx.x * (long)blockDim.x + threadIdx.x; a < M; a += (long)gridDim.x * blockDim.x) {
    const int g = topk_idx[a] / per_group;
    if (st->all_kept[g]) continue;
    const unsigned long long key = drop_key(score[a], a);
    const bool match = pass == 0 || (key >> (shift + 8)) == st->prefix[g];
    if (match) {
      const int digit = (int)((key >> shift) & 0xffull);
      if constexpr (LDS_GROUPS > 0) atomicAdd(&h[g][digit], 1);
      else atomicAdd(&st->hist[g][digit], 1);
    }
  }
  if constexpr (LDS_GROUPS > 0) {
    __syncthreads();
    for (int i = threadIdx.x; i < n_groups * 256; i += blockDim.x) {
      const int v = (&h[0][0])[i];
      if (v) atomicAdd(&st->hist[i / 256][i % 256], v);
    }
  }
}

// One wave per device: lane l holds the counts of digits 4l .. 4l+3; the digit that contains the threshold is the
// highest d with (keys in digits above d) + hist[d] >= remaining.
__global__ void __launch_bounds__(256) select_pick_kernel(SelectState* st, int n_groups, int pass) {
  const int lane = threadIdx.x % 64;
  const int g = blockIdx.x * 4 + threadIdx.x / 64;
  if (g >= n_groups || st->all_kept[g]) return;            // wave-uniform
  int c[4];
  int mine = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    c[i] = st->hist[g][4 * lane + i];
    st->hist[g][4 * lane + i] = 0;
    mine += c[i];
  }
  int incl = mine;                                          // inclusive suffix sum over lanes (lane 63 first)
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_down(incl, off);
    if (lane + off < 64) incl += o;
  }
  const int total = __shfl(incl, 0);
  const int remaining = st->remaining[g];
  if (pass == 0 && total <= remaining) {
    if (lane == 0) { st->all_kept[g] = 1; st->prefix[g] = 0ull; }   // threshold 0: every key passes
    return;
  }
  int cum = incl - mine;                                    // keys in digits above this lane's four
  int hit = -1, cum_at_hit = 0;
#pragma unroll
  for (int i = 3; i >= 0; --i) {
    if (hit < 0 && cum + c[i] >= remaining) { hit = 4 * lane + i; cum_at_hit = cum; }
    cum += c[i];
  }
  const unsigned long long hits = __ballot(hit >= 0);
  // remaining <= total here, so some lane hits; remaining = 0 (capacity 0) hits in lane 63 at digit 255
  const int winner = 63 - __builtin_clzll(hits);
  if (lane == winner) {
    st->prefix[g] = (st->prefix[g] << 8) | (unsigned long long)hit;
    st->remaining[g] = remaining - cum_at_hit;
  }
}

// The same selection in one launch for up to 1024 * KPT assignments: a workgroup per device holds its keys in registers and
// walks the digits with the histogram in LDS, until all keys left under the prefix are kept.  The launches above are 17
// times a few microseconds whatever the size: 4593 assignments, 8 devices: 71 us; this: 7.  A training step with 24000
// assignments: 373 -> 279 us.
template <int KPT>
__global__ void __launch_bounds__(1024) select_small_kernel(const int32_t* __restrict__ topk_idx, const float* __restrict__ score,
                                                            int M, int per_group, int capacity, SelectState* st) {
  __shared__ int hist[256];
  __shared__ unsigned long long prefix_s;
  __shared__ int remaining_s, state_s;                    // state: 0 next digit, 1 all kept, 2 threshold found
  const int g = blockIdx.x, lane = threadIdx.x & 63;
  unsigned long long key[KPT];                            // 0: no key (a key's low word is never 0)
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const int a = threadIdx.x + i * 1024;
    key[i] = a < M && topk_idx[a] / per_group == g ? drop_key(score[a], a) : 0ull;
  }
  unsigned long long prefix = 0;
  int remaining = capacity, state = 0;
  for (int pass = 0; pass < 8 && state == 0; ++pass) {
    const int shift = 56 - 8 * pass;
    if (threadIdx.x < 256) hist[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KPT; ++i)
      if (key[i] != 0 && (pass == 0 || (key[i] >> (shift + 8)) == prefix)) atomicAdd(&hist[(int)((key[i] >> shift) & 0xffull)], 1);
    __syncthreads();
    if (threadIdx.x < 64) {                               // lane l: digits 4l .. 4l+3, as in select_pick_kernel
      int c[4], mine = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) { c[i] = hist[4 * lane + i]; mine += c[i]; }
      int incl = mine;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_down(incl, off);
        if (lane + off < 64) incl += o;
      }
      const int total = __builtin_amdgcn_readfirstlane(incl);
      int cum = incl - mine, hit = -1, cum_at_hit = 0, count = 0;
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        if (hit < 0 && cum + c[i] >= remaining) { hit = 4 * lane + i; cum_at_hit = cum; count = c[i]; }
        cum += c[i];
      }
      const unsigned long long hits = __ballot(hit >= 0);
      if (pass == 0 && total <= remaining) {
        if (lane == 0) { prefix_s = 0; remaining_s = 0; state_s = 1; }
      } else if (lane == 63 - __builtin_clzll(hits)) {
        prefix_s = (prefix << 8) | (unsigned long long)hit;
        remaining_s = remaining - cum_at_hit;
        state_s = count == remaining - cum_at_hit ? 2 : 0;      // every key under this prefix is kept
      }
    }
    __syncthreads();
    prefix = prefix_s;
    remaining = remaining_s;
    state = state_s;
    if (state == 2) prefix <<= shift;
  }
  if (threadIdx.x == 0) {
    st->prefix[g] = prefix;
    st->all_kept[g] = state == 1;
  }
}

// keep[a] and the per-chunk expert histogram of the kept assignments (same layout as route_topk_kernel's)
__global__ void __launch_bounds__(256) keep_hist_kernel(const int32_t* __restrict__ topk_idx,
                                                        const float* __restrict__ score, int T, int E, int k,
                                                        int per_group, int chunk_tokens, int he, int hc,
                                                        const SelectState* __restrict__ st,
                                                        uint8_t* __restrict__ keep, int32_t* __restrict__ chunk_hist) {
  __shared__ int hist[MOE_MAX_EXPERTS];
  for (int e = threadIdx.x; e < MOE_MAX_EXPERTS; e += blockDim.x) hist[e] = 0;
  __syncthreads();
  const long a_begin = (long)blockIdx.x * chunk_tokens * k;
  const long a_end = min((long)(blockIdx.x + 1) * chunk_tokens, (long)T) * k;
  for (long a = a_begin + threadIdx.x; a < a_end; a += blockDim.x) {
    const int e = topk_idx[a];
    const int g = e / per_group;
    const bool kp = st->all_kept[g] || drop_key(score[a], a) >= st->prefix[g];
    keep[a] = kp ? 1 : 0;
    if (kp) atomicAdd(&hist[e], 1);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += blockDim.x) chunk_hist[(long)e * he + (long)blockIdx.x * hc] = hist[e];
}

}  // namespace

size_t route_ws_bytes(int T, int E) {
  const int tb = route_chunk_tokens(T);
  return align_up((size_t)cdiv(T, tb) * E * sizeof(int32_t), 256);
}

size_t route_capacity_ws_bytes(int T, int E, int k) {
  return route_ws_bytes(T, E) + align_up(sizeof(SelectState), 256) + align_up((size_t)T * k, 256);
}

// n_groups = 0: no dropping.  Otherwise `score` [T,k] must be given and ws holds route_capacity_ws_bytes.
int launch_route(const float* logits, int T, int E, int k, int renorm, int e_lo, int e_hi, int n_groups, int capacity,
                 int32_t* idx, float* w, float* score, int32_t* counts, int32_t* offsets, int32_t* perm,
                 int32_t* inv_perm, void* ws, hipStream_t s) {
  const int tb = route_chunk_tokens(T);
  const int nchunks = cdiv(T, tb);
  int32_t* hist = static_cast<int32_t*>(ws);
  // Up to 16384 counts every workgroup of the rank kernel adds them up itself (at most 64 KB from L2, 32 loads per thread when E is
  // a power of two, up to twice as many otherwise, in batches of 8), which spares a launch and its latency; beyond that the scan
  // kernel does it once.
  const bool sums = (long)nchunks * E <= 16384;
  const int he = sums ? 1 : nchunks, hc = sums ? E : 1;
  const int rc = with_group(E, [&](auto g, auto v) -> int {
    route_topk_kernel<g.value, v.value><<<nchunks, 64 * g.value, 0, s>>>(logits, T, E, k, renorm, tb, he, hc, idx, w, hist, score);
    MOE_LAUNCH_CHECK();
    return MOE_OK;
  });
  if (rc != MOE_OK) return rc;
  const uint8_t* keep = nullptr;
  if (n_groups > 0) {
    char* base = static_cast<char*>(ws) + route_ws_bytes(T, E);
    SelectState* st = reinterpret_cast<SelectState*>(base);
    uint8_t* keep_w = reinterpret_cast<uint8_t*>(base + align_up(sizeof(SelectState), 256));
    const long M = (long)T * k;
    const int per_group = E / n_groups;
    if (M <= 1024 * 8) {
      select_small_kernel<8><<<n_groups, 1024, 0, s>>>(idx, score, (int)M, per_group, capacity, st);
      MOE_LAUNCH_CHECK();
    } else if (M <= 1024 * 32) {
      select_small_kernel<32><<<n_groups, 1024, 0, s>>>(idx, score, (int)M, per_group, capacity, st);
      MOE_LAUNCH_CHECK();
    } else {
      long blocks = (M + 1023) / 1024;
      if (blocks > 512) blocks = 512;
      select_init_kernel<<<1, 256, 0, s>>>(st, n_groups, capacity);
      MOE_LAUNCH_CHECK();
      for (int pass = 0; pass < 8; ++pass) {
        if (n_groups <= 16) select_count_kernel<16><<<(int)blocks, 256, 0, s>>>(idx, score, M, per_group, n_groups, pass, st);
        else select_count_kernel<0><<<(int)blocks, 256, 0, s>>>(idx, score, M, per_group, n_groups, pass, st);
        MOE_LAUNCH_CHECK();
        select_pick_kernel<<<cdiv(n_groups, 4), 256, 0, s>>>(st, n_groups, pass);
        MOE_LAUNCH_CHECK();
      }
    }
    keep_hist_kernel<<<nchunks, 256, 0, s>>>(idx, score, T, E, k, per_group, tb, he, hc, st, keep_w, hist);
    MOE_LAUNCH_CHECK();
    keep = keep_w;
  }
  if (sums) {
    route_rank_kernel<true><<<nchunks, 64 * kRankWaves, 0, s>>>(idx, T, E, k, e_lo, e_hi, tb, nchunks, hist, counts, offsets, perm,
                                                                inv_perm, keep);
  } else {
    route_scan_kernel<<<E, 64, 0, s>>>(hist, nchunks, counts);
    MOE_LAUNCH_CHECK();
    route_rank_kernel<false><<<nchunks, 64 * kRankWaves, 0, s>>>(idx, T, E, k, e_lo, e_hi, tb, nchunks, hist, counts, offsets, perm,
                                                                 inv_perm, keep);
  }
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

int launch_route_bwd(const float* logits, const int32_t* idx, const float* w, const float* dw, int T, int E, int k,
                     int renorm, float* d_logits, hipStream_t s) {
  return with_group(E, [&](auto g, auto v) -> int {
    constexpr int kMaxTokens = 1 << 27;        // per launch, which holds less than 2^32 threads (up to 16 of them per token)
    for (long t = 0; t < T; t += kMaxTokens) {
      const int n = T - t < kMaxTokens ? (int)(T - t) : kMaxTokens;
      route_bwd_kernel<g.value, v.value><<<cdiv(n, 256 / g.value), 256, 0, s>>>(logits ? logits + t * E : nullptr, idx + t * k, w + t * k,
                                                                                dw + t * k, n, E, k, renorm, d_logits + t * E);
      MOE_LAUNCH_CHECK();
    }
    return MOE_OK;
  });
}

}  // namespace moe
