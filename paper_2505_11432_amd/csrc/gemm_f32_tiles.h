// Which output tile of a grouped fp32 GEMM a workgroup works on (gemm_f32.hip, gemm_f32_split.hip).
#pragma once
#include "moe_common.h"

namespace moe {

constexpr int kF32GroupN = 8;         // n-tiles per group: neighbouring workgroups of an XCD form a compact block of tiles
constexpr int kF32Xcds = 8, kF32Window = 32;

// Expert segment that holds running tile index l when every segment of n rows has cdiv(n, bm) * tiles_n tiles.  A wave
// looks at 64 segments at a time (a lane each, prefix sum by shuffles).
__device__ __forceinline__ bool find_segment(const int32_t* __restrict__ offsets, int E, int bm, int tiles_n, int l, int& e,
                                             int& lo, int& hi, int& l_in) {
  const int lane = threadIdx.x & 63;
  int base = 0;
  for (int e0 = 0; e0 < E; e0 += 64) {
    const int ei = min(e0 + lane, E - 1);
    const int o0 = offsets[ei], o1 = offsets[ei + 1];
    const int n = e0 + lane < E ? (o1 - o0 + bm - 1) / bm * tiles_n : 0;
    int incl = n;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    const unsigned long long hit = __ballot(base + incl > l);
    if (hit != 0) {
      const int src = __builtin_ctzll(hit);
      e = e0 + src;
      lo = __builtin_amdgcn_readlane(o0, src);
      hi = __builtin_amdgcn_readlane(o1, src);
      l_in = l - base - (__builtin_amdgcn_readlane(incl, src) - __builtin_amdgcn_readlane(n, src));
      return true;
    }
    base += __builtin_amdgcn_readlane(incl, 63);
  }
  return false;
}

struct F32Tile {
  int e, m0, m_end, n0;         // expert, first row, end of its rows, first column
  int k0, k_end;                // the contraction
};

// The tile of workgroup `block` of `blocks`; false where the grid, which is sized for any segments, has one too many.
template <int BM, int BN>
__device__ __forceinline__ bool f32_tile(const GemmProblem& p, int tiles_n, int tiles_m_fixed, int block, int blocks, F32Tile& t) {
  // runs of kF32Window consecutive tiles go to one XCD (workgroup b runs on XCD b % 8) so that its L2 serves their panels
  int l = block;
  const int span = kF32Xcds * kF32Window, first = l / span * span;
  if (first + span <= blocks) l = first + (l % kF32Xcds) * kF32Window + (l - first) / kF32Xcds;
  int m_lo = 0, mt_e = tiles_m_fixed;
  t.e = 0;
  t.k0 = 0;
  t.k_end = p.K;
  t.m_end = p.M;
  if (p.mode == 0) {
    int hi, l_in;
    if (!find_segment(p.offsets, p.E, BM, tiles_n, l, t.e, m_lo, hi, l_in)) return false;
    l = l_in;
    t.m_end = hi;
    mt_e = (hi - m_lo + BM - 1) / BM;
  } else if (p.mode == 1) {
    t.e = l / (mt_e * tiles_n);
    l -= t.e * mt_e * tiles_n;
    t.k0 = p.offsets[t.e];
    t.k_end = p.offsets[t.e + 1];
  }
  const int ng = l / (mt_e * kF32GroupN), rest = l - ng * mt_e * kF32GroupN;
  const int gw = min(kF32GroupN, tiles_n - ng * kF32GroupN);
  const int mt = rest / gw;
  t.m0 = m_lo + mt * BM;
  t.n0 = (ng * kF32GroupN + (rest - mt * gw)) * BN;
  // the same in every lane, and known to be: what follows from it stays in scalar registers
  t.e = __builtin_amdgcn_readfirstlane(t.e);
  t.m0 = __builtin_amdgcn_readfirstlane(t.m0);
  t.m_end = __builtin_amdgcn_readfirstlane(t.m_end);
  t.n0 = __builtin_amdgcn_readfirstlane(t.n0);
  t.k0 = __builtin_amdgcn_readfirstlane(t.k0);
  t.k_end = __builtin_amdgcn_readfirstlane(t.k_end);
  return true;
}

// Workgroups of a launch with BM x BN tiles: an upper bound over any segment lengths.
inline long f32_blocks(const GemmProblem& p, int bm, int bn) {
  const long tiles_n = cdiv(p.N, bn), tiles_m = cdiv(p.M, bm);
  return p.mode == 0 ? tiles_n * (tiles_m + p.E) : p.mode == 1 ? tiles_n * tiles_m * p.E : tiles_n * tiles_m;
}

// gemm_f32_split.hip: whether it is the faster way for this problem; its launch
bool gemm_f32_splits(const GemmProblem& p);
int launch_gemm_f32_split(const GemmProblem& p, hipStream_t s);

}  // namespace moe
