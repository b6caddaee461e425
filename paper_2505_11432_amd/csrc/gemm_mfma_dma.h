// Grouped bf16 GEMM on the gfx950 matrix cores with an asynchronous global->LDS pipeline.
//
// Same contract and tile geometry as gemm_mfma.h (the paper's GroupedGEMM operator, Section 4.1, in
// its three contraction layouts), but operand tiles travel global -> LDS directly
// (global_load_lds_dwordx4) into an NSTAGE-deep ring, so loads for k-step s+NSTAGE-1 are in flight
// while k-step s is on the matrix cores, no VGPRs stage the tiles and no ds_write phase exists.
// One s_barrier per k-step: after it every wave's loads for the step have landed and every wave has
// left the previous step, whose buffer the new loads may overwrite.
//
// The products run on the 16x16 matrix instructions (16x16x32 bf16, 16x16x128 e4m3), which do the same products for less power, and power
// sets the clock: register-only loops of eight waves per CU on N(0,1) bf16 operands reach 2.07 PFLOP/s against 1.78 with the 32x32
// ones, fed from LDS 1.67 against 1.54, with this kernel's load traffic, waits and barriers beside them 1.48 against 1.41 (random
// e4m3 codes 4.13 against 3.75).  8 experts, 16384 rows, 4096 x 14336, bf16 (us): FC1 3261 -> 3064, FC2 1547 -> 1449, dgrad1 3041 -> 2880,
// dgrad2 2096 -> 2020, weight gradients 1892 -> 1843 and 3628 -> 3585.  FC1, FC2 and dgrad1 take 1.06 to 1.14 of what their products
// take in the last of these loops, dgrad2 and the weight gradients 1.3 to 1.5, with their epilogues and stores in between.
//
// The kernel is persistent: one workgroup per CU (two where they fit its LDS) walks a static list of tiles.  When the last k-step of
// a tile is done the ring is free, so the first stages of the NEXT tile are put in flight before the
// current tile's epilogue runs; workgroup launch, tile lookup, pointer set-up and the cold first loads
// all disappear behind the epilogue's stores.
//
// A direct-to-LDS load deposits the wave's 64 x 16 bytes contiguously, so the LDS swizzles are applied
// on the global side: the lane that owns physical chunk pc of a row fetches logical chunk pc ^ swz(row).
//   K-major tile [rows][BKT]:  swz = (row / rows_per_256B) mod chunks_per_row  -> ds_read_b128 conflict-free
//   M/N-major tile [BKT][cols]: swz = 4 * (k mod 4) ^ 2 * (k / 8 mod 2)        -> ds_read_b64_tr_b16 conflict-free
// Loads that fall outside the contraction range fetch from a 16-byte zero block instead, which gives
// the exact zero fill that ragged expert segments (wgrad) and K tails need.
#pragma once
#include <type_traits>

#include "gemm_mfma.h"
#include "row_plan.h"

namespace moe {
namespace mfma {

static __device__ __attribute__((aligned(16))) const unsigned int g_zero_block[4] = {0u, 0u, 0u, 0u};

// One wave-wide direct-to-LDS load: lane i's 16 bytes land at lds_addr + 16*i.  lds_addr is wave-uniform.
__device__ __forceinline__ void dma16(const void* gptr, unsigned lds_addr) {
  // No "memory" clobber: the LDS write is asynchronous anyway and is ordered by wait_vmcnt + s_barrier, and
  // without it the compiler stays free to hoist LDS fragment reads of the current stage across the load.
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr), "s"(lds_addr) : "m0");
}

// The same load with the address split into a wave-uniform 64-bit base (scalar registers) and a 32-bit per-lane
// byte offset: the per-k-step address update is then scalar arithmetic, and issuing the load needs no vector ALU
// slot (those are what the SIMD partner's MFMAs compete for).
__device__ __forceinline__ void dma16s(const char* sbase, unsigned voff, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_addr) : "m0");
}

// One wave-wide 4-byte direct-to-LDS load whose data nobody reads (it lands in a dump area): its only effect is to
// bring the 64 lines it touches into this XCD's L2 ahead of the tile loads that need them.
__device__ __forceinline__ void touch4s(const char* sbase, unsigned voff, unsigned lds_dump) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dword %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_dump) : "m0");
}

// Sixteen of those loads in one block: eight from sbase_a, then eight from sbase_b, into LDS slots that lie a fixed
// 4 KiB apart from lds_first on (a 32 KiB A tile followed by the B tile, four loader waves).  M0 is stepped with
// scalar adds inside the block, so the sixteen slot addresses need no registers of their own (kept as sixteen
// loop-invariant scalars they were spilled to vector lanes and read back with v_readlane before every load).
__device__ __forceinline__ void dma16s_x16(const char* sbase_a, const char* sbase_b, const unsigned (&va)[8],
                                           const unsigned (&vb)[8], unsigned lds_first) {
  asm volatile(
      "s_mov_b32 m0, %18\n\t"
      "global_load_lds_dwordx4 %0, %16\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %1, %16\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %2, %16\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %3, %16\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %4, %16\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %5, %16\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %6, %16\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %7, %16\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %8, %17\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %9, %17\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %10, %17\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %11, %17\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %12, %17\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %13, %17\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %14, %17\n\ts_add_u32 m0, m0, 0x1000\n\t"
      "global_load_lds_dwordx4 %15, %17"
      ::"v"(va[0]), "v"(va[1]), "v"(va[2]), "v"(va[3]), "v"(va[4]), "v"(va[5]), "v"(va[6]), "v"(va[7]),
        "v"(vb[0]), "v"(vb[1]), "v"(vb[2]), "v"(vb[3]), "v"(vb[4]), "v"(vb[5]), "v"(vb[6]), "v"(vb[7]),
        "s"(sbase_a), "s"(sbase_b), "s"(lds_first)
      : "m0", "scc");
}

__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return reinterpret_cast<const char*>(((unsigned long long)hi << 32) | lo);
}

template <int N> __device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  // gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] at [15:14]; other counters left open
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

__device__ __forceinline__ void wait_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (3 << 14)); }

template <int ROWS, int BKT, int ESZ = 2> struct KTile {        // K-major [ROWS][BKT] of ESZ-byte elements
  static constexpr int ROW_BYTES = BKT * ESZ, CPR = ROW_BYTES / 16, RPL = 256 / ROW_BYTES;
  static constexpr int BYTES = ROWS * ROW_BYTES;
  static constexpr int ROWS_PER_DMA = 1024 / ROW_BYTES;
  __device__ static __forceinline__ int swz(int row) { return (row / RPL) % CPR; }
  __device__ static __forceinline__ int offset(int row, int chunk) { return row * ROW_BYTES + ((chunk ^ swz(row)) << 4); }
};
template <int COLS, int BKT> struct MNTile {       // M/N-major [BKT][COLS] bf16
  static constexpr int ROW_BYTES = COLS * 2, CPR = ROW_BYTES / 16;
  static constexpr int BYTES = BKT * ROW_BYTES;
  static constexpr int ROWS_PER_DMA = 1024 / ROW_BYTES;
  static_assert(ROW_BYTES <= 1024 && CPR >= 16, "M/N-major tiles are 128..512 columns wide");
  __device__ static __forceinline__ int swz(int krow) { return ((krow & 3) << 2) ^ ((krow >> 2) & 2); }
};

template <Layout L, int EXTENT, int BKT, int ESZ = 2> struct DmaTileBytes;
template <int EXTENT, int BKT, int ESZ> struct DmaTileBytes<KMAJOR, EXTENT, BKT, ESZ> { static constexpr int value = KTile<EXTENT, BKT, ESZ>::BYTES; };
template <int EXTENT, int BKT, int ESZ> struct DmaTileBytes<MNMAJOR, EXTENT, BKT, ESZ> {
  static_assert(ESZ == 2, "M/N-major tiles exist for bf16 only");
  static constexpr int value = MNTile<EXTENT, BKT>::BYTES;
};

// Fragment of the 16x16x32 bf16 MFMA: lane l holds k = 8 * (l / 16) + 0..7 of row (or column) l % 16.  `origin` is what
// frag_origin gives for the wave's first row, moved to the tile; fragment i lies 16 rows (columns) on, sub-step kk 32 of k.
// In M/N-major tiles fragment i is the origin with i at bits 5..7 flipped: the caller hides the origin from the optimiser
// once per phase, so that one exclusive-or makes an address where it is used instead of eight of them filling registers.
template <Layout L, int EXTENT, int BKT, int ESZ = 2>
__device__ __forceinline__ unsigned frag_origin(int base, int lane) {
  const int i = lane & 15, g = lane >> 4;
  if constexpr (L == KMAJOR) {
    return (unsigned)KTile<EXTENT, BKT, ESZ>::offset(base + i, g);
  } else {
    using TL = MNTile<EXTENT, BKT>;
    const int krow = (g << 3) + (i >> 2), col = base + ((i & 3) << 2);
    return (unsigned)(krow * TL::ROW_BYTES + (((col >> 3) ^ TL::swz(krow)) << 4) + ((col & 7) << 1));
  }
}
template <Layout L, int EXTENT, int BKT>
__device__ __forceinline__ bf16x8 read_frag_dma(unsigned origin, int i, int kk) {
  if constexpr (L == KMAJOR) {
    using TL = KTile<EXTENT, BKT>;
    return lds_read_b128((origin ^ (unsigned)(kk << 6)) + (unsigned)(i * 16 * TL::ROW_BYTES));
  } else {
    using TL = MNTile<EXTENT, BKT>;
    const unsigned p = (origin ^ (unsigned)(i << 5)) + (unsigned)(kk * 32 * TL::ROW_BYTES);
    const bf16x4 lo = lds_read_tr(p);
    const bf16x4 hi = lds_read_tr(p + 4 * TL::ROW_BYTES);             // krow + 4 has the same swizzle
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
}
// e4m3 fragment of the 16x16x128 f8f6f4 MFMA (32 bytes per lane, K-major tiles).  Lane l takes chunks l / 16 and 4 + l / 16 of
// its row's 128 bytes: the same order of k in both operands, and no two of the lanes served together meet in a bank.
template <int EXTENT, int BKT>
__device__ __forceinline__ i32x8 read_frag_fp8(unsigned origin, int i, int kk) {
  typedef __attribute__((ext_vector_type(4))) int i32x4;
  using TL = KTile<EXTENT, BKT, 1>;
  const unsigned step = (unsigned)(i * 16 * TL::ROW_BYTES);
  const i32x4 lo = __builtin_bit_cast(i32x4, lds_read_b128((origin ^ (unsigned)(kk << 7)) + step));
  const i32x4 hi = __builtin_bit_cast(i32x4, lds_read_b128((origin ^ (unsigned)(kk << 7) ^ 64u) + step));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}


// ---- epilogue staging --------------------------------------------------------------------------------
// After the MFMA (weight fragment first) a lane holds row lane % 16 and columns 4*(lane/16) + 0..3 of each 16x16
// tile; the epilogues work on blocks of 2x2 of them, 32x32, in which group q = 0..3 of a lane's values is row
// 16*(q/2) + lane%16, columns 16*(q%2) + 4*(lane/16) + 0..3.  A direct store would touch 16 rows with 16 bytes each
// quarter.  Each wave therefore owns a small LDS patch of 32 rows x 64 bytes; blocks pass through it so that
// global memory sees 16-byte lanes forming 64-byte row segments (4 lanes per row, 16 rows per instruction).
constexpr int STG_STRIDE = 80;                  // bytes per staged row (64 payload + 16 pad)
constexpr int STG_BYTES = 32 * STG_STRIDE;      // per wave
__device__ __forceinline__ int patch_row(int q, int lane) { return ((q >> 1) << 4) + (lane & 15); }
__device__ __forceinline__ int patch_col(int q, int lane) { return ((q & 1) << 4) + ((lane >> 4) << 2); }
struct Block { f32x4 q[4]; };                   // a lane's values of one 32x32 block

// Global accesses of the epilogues are raw buffer instructions on a descriptor that starts at the block's origin
// (wave-uniform): a lane outside the valid rows or columns gets an offset past the end of the buffer, which the
// hardware answers with zeros (loads) or drops (stores).  No lane-dependent branch surrounds a memory instruction, so
// every wave issues the same, known number of them and the compiler's s_waitcnt vmcnt(n) stay exact: with stores
// inside `if (valid)` blocks it has to assume that none was issued and waits for vmcnt(0), i.e. for every store of
// the previous block, before each read.
typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));
constexpr unsigned BUF_SPAN = 0x40000000u;      // 1 GiB from the block origin; a 32-row block spans far less
constexpr unsigned BUF_OOB = 0x80000000u;       // offset of a masked lane
__device__ __forceinline__ __amdgpu_buffer_rsrc_t block_rsrc(const void* origin) {
  char* base = const_cast<char*>(uniform_ptr(static_cast<const char*>(origin)));
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)BUF_SPAN, 0x00020000);   // raw buffer, 32-bit data format
}
__device__ __forceinline__ unsigned block_offset(int r, int c, long ld, int esz, int rows_valid, int cols_valid) {
  return (r < rows_valid && c < cols_valid) ? (unsigned)(((long)r * ld + c) * esz) : BUF_OOB;
}

// 32 rows x 32 bf16 columns from registers to global memory (row-major, leading dimension ld elements).
__device__ __forceinline__ void stage_store_bf16(char* stg, const bf16x4 (&v)[4], bf16* g, long ld, int rows_valid,
                                                 int cols_valid, int lane) {
#pragma unroll
  for (int q = 0; q < 4; ++q) *reinterpret_cast<bf16x4*>(stg + patch_row(q, lane) * STG_STRIDE + patch_col(q, lane) * 2) = v[q];
  const __amdgpu_buffer_rsrc_t rs = block_rsrc(g);
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int r = pass * 16 + (lane >> 2), c = (lane & 3) * 8;
    const u32x4v val = *reinterpret_cast<const u32x4v*>(stg + r * STG_STRIDE + c * 2);
    __builtin_amdgcn_raw_buffer_store_b128(val, rs, block_offset(r, c, ld, 2, rows_valid, cols_valid), 0, 0);
  }
}

// 32 rows x 32 bf16 columns from global memory into registers (same lane layout as the accumulators).
__device__ __forceinline__ void stage_load_bf16(char* stg, bf16x4 (&v)[4], const bf16* g, long ld, int rows_valid,
                                                int cols_valid, int lane) {
  const __amdgpu_buffer_rsrc_t rs = block_rsrc(g);
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int r = pass * 16 + (lane >> 2), c = (lane & 3) * 8;
    const u32x4v val = __builtin_amdgcn_raw_buffer_load_b128(rs, block_offset(r, c, ld, 2, rows_valid, cols_valid), 0, 0);
    *reinterpret_cast<u32x4v*>(stg + r * STG_STRIDE + c * 2) = val;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const bf16x4*>(stg + patch_row(q, lane) * STG_STRIDE + patch_col(q, lane) * 2);
}

// The same load in two phases, so that the global reads of the next 32x32 block can be in flight while the
// current block is processed: fetch (global -> registers, zero where masked) and unpack (registers -> LDS patch ->
// accumulator lane layout).
struct StageFetch { u32x4v v[2]; };
__device__ __forceinline__ StageFetch stage_fetch_bf16(const bf16* g, long ld, int rows_valid, int cols_valid, int lane) {
  StageFetch f;
  const __amdgpu_buffer_rsrc_t rs = block_rsrc(g);
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int r = pass * 16 + (lane >> 2), c = (lane & 3) * 8;
    f.v[pass] = __builtin_amdgcn_raw_buffer_load_b128(rs, block_offset(r, c, ld, 2, rows_valid, cols_valid), 0, 0);
  }
  return f;
}
__device__ __forceinline__ void stage_unpack_bf16(char* stg, const StageFetch& f, bf16x4 (&v)[4], int lane) {
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int r = pass * 16 + (lane >> 2), c = (lane & 3) * 8;
    *reinterpret_cast<u32x4v*>(stg + r * STG_STRIDE + c * 2) = f.v[pass];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const bf16x4*>(stg + patch_row(q, lane) * STG_STRIDE + patch_col(q, lane) * 2);
}

// 32 rows x 32 fp32 columns, as two halves of 16 columns; optional read-modify-write accumulation.
__device__ __forceinline__ void stage_store_f32(char* stg, const Block& acc, float* g, long ld, int rows_valid,
                                                int cols_valid, bool accumulate, int lane) {
  const __amdgpu_buffer_rsrc_t rs = block_rsrc(g);
#pragma unroll
  for (int half = 0; half < 2; ++half) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      *reinterpret_cast<f32x4*>(stg + patch_row(2 * i, lane) * STG_STRIDE + patch_col(2 * i, lane) * 4) = acc.q[2 * i + half];
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      const int r = pass * 16 + (lane >> 2), c = half * 16 + (lane & 3) * 4;
      f32x4 val = *reinterpret_cast<const f32x4*>(stg + r * STG_STRIDE + (lane & 3) * 16);
      const unsigned off = block_offset(r, c, ld, 4, rows_valid, cols_valid);
      if (accumulate) val += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));   // (uniform)
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4v, val), rs, off, 0, 0);
    }
  }
}

// Work list with the last round split along K: tiles [0, full_tiles) are whole; each of the remaining
// total_tiles - full_tiles tiles becomes `split` items of at least two k-steps.  No split unless it at least halves the
// last round.
__host__ __device__ __forceinline__ void splitk_plan(int total_tiles, int workgroups, int steps, int& full_tiles, int& split, int& total_items) {
  full_tiles = total_tiles / workgroups * workgroups;
  const int rem = total_tiles - full_tiles;
  split = 1;
  if (rem > 0) {
    split = workgroups / rem;
    split = split < 8 ? split : 8;                     // (the fix-up reads every part)
    split = split < steps / 2 ? split : steps / 2;
  }
  if (split <= 1) { split = 1; full_tiles = total_tiles; }
  total_items = full_tiles + (total_tiles - full_tiles) * split;
}

// cum[e] = number of BM-row tiles of the experts before e, by the first wave (64 experts at a time).
template <int BM>
__device__ __forceinline__ void tile_table(const int32_t* __restrict__ offsets, int E, int* cum) {
  const int lane = threadIdx.x;
  if (lane >= 64) return;
  if (lane == 0) cum[0] = 0;
  int base = 0;
  for (int e0 = 0; e0 < E; e0 += 64) {
    const int e = e0 + lane;
    int incl = e < E ? (offsets[e + 1] - offsets[e] + BM - 1) / BM : 0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    if (e < E) cum[e + 1] = base + incl;
    base += __builtin_amdgcn_readlane(incl, 63);
  }
}

// Adds the K parts of every split tile and writes the bf16 result with the tile's row / column masks.  16 workgroups per
// split tile while they last (four per GEMM workgroup are launched), else 8; the tile list is rebuilt exactly as in the GEMM kernel (same grouping constants).
template <int BM, int BN>
__global__ void __launch_bounds__(256) splitk_fixup_kernel(const float* __restrict__ parts, const int32_t* __restrict__ offsets,
                                                           int E, int N, int steps, int gemm_workgroups, bf16* __restrict__ C, long ldc) {
  constexpr int GN = 8;
  __shared__ int cum_tiles[MOE_MAX_EXPERTS + 1];
  tile_table<BM>(offsets, E, cum_tiles);
  __syncthreads();
  const int tiles_n = (N + BN - 1) / BN;
  const int total_tiles = cum_tiles[E] * tiles_n;
  int full_tiles, split, total_items;
  splitk_plan(total_tiles, gemm_workgroups, steps, full_tiles, split, total_items);
  const int n_split = total_tiles - full_tiles;      // at most half of the GEMM workgroups
  const int slices = n_split * 16 <= (int)gridDim.x ? 16 : 8;      // workgroups per split tile, BM / slices rows each
  const int r_tile = blockIdx.x / slices, slice = blockIdx.x % slices;
  if (split == 1 || r_tile >= n_split) return;
  int l = full_tiles + r_tile;
  int lo = 0, hi = E;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cum_tiles[mid] * tiles_n <= l) lo = mid; else hi = mid;
  }
  const int e = lo;
  const int mt_e = cum_tiles[e + 1] - cum_tiles[e];
  l -= cum_tiles[e] * tiles_n;
  const int ng = l / (mt_e * GN);
  const int r = l - ng * mt_e * GN;
  const int gw = min(GN, tiles_n - ng * GN);
  const int mt = r / gw;
  const int nt = ng * GN + (r - mt * gw);
  const int m0 = offsets[e] + mt * BM, m_end = offsets[e + 1], n0 = nt * BN;
  const float* base = parts + (long)r_tile * split * (BM * BN);
  const int rows = BM / slices;
  for (int i = threadIdx.x; i < rows * BN / 8; i += blockDim.x) {
    const int row = slice * rows + i / (BN / 8), col = (i % (BN / 8)) * 8;
    if (m0 + row >= m_end || n0 + col >= N) continue;          // N is a multiple of 8
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = 0.f;
    for (int s = 0; s < split; ++s) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(base + (long)s * (BM * BN) + row * BN + col);
      const f32x4 b = *reinterpret_cast<const f32x4*>(base + (long)s * (BM * BN) + row * BN + col + 4);
#pragma unroll
      for (int q = 0; q < 4; ++q) { v[q] += a[q]; v[4 + q] += b[q]; }
    }
    bf16x8 o;
#pragma unroll
    for (int q = 0; q < 8; ++q) o[q] = static_cast<bf16>(v[q]);
    *reinterpret_cast<bf16x8*>(C + (long)(m0 + row) * ldc + n0 + col) = o;
  }
}

template <int BM, int BN, int BKT, int NSTAGE, int NW, Layout LA, Layout LB, int ESZ = 2>
constexpr int dma_smem_bytes() {
  // the ring, the per-expert tile table and one epilogue patch per wave
  return NSTAGE * (DmaTileBytes<LA, BM, BKT, ESZ>::value + DmaTileBytes<LB, BN, BKT, ESZ>::value) + (MOE_MAX_EXPERTS + 8) * 4 +
         NW * STG_BYTES + 256 + 1024;       // + the dump area of the L2 touches + the block-scale ring
}

// Two workgroups of such a kernel share a CU's LDS; the launch makes twice the workgroups.
template <int BM, int BN, int BKT, int NSTAGE, int NW, Layout LA, Layout LB, int ESZ = 2>
constexpr bool dma_in_pairs() { return 2 * dma_smem_bytes<BM, BN, BKT, NSTAGE, NW, LA, LB, ESZ>() <= 160 * 1024; }

template <int BM, int BN, int BKT, int NSTAGE, int WM, int WN, Layout LA, Layout LB, Mode MODE, Epi EPI, typename TC,
          typename TIN = bf16>   // TIN = uint8_t: e4m3 codes, K-major operands only
__global__ void __launch_bounds__(WM * WN * 64, 2) grouped_gemm_dma_kernel(Args p) {
  constexpr int NW = WM * WN;
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int FM = WTM / 16, FN = WTN / 16;         // fragments of a wave along each side
  constexpr int TM = WTM / 32, TN = WTN / 32;         // 32x32 blocks of its epilogue
  constexpr int ESZ = sizeof(TIN);
  constexpr bool FP8 = ESZ == 1;
  constexpr int CHUNK = 16 / ESZ;                     // elements per 16-byte chunk
  static_assert(!FP8 || (LA == KMAJOR && LB == KMAJOR), "e4m3 operands are K-major");
  constexpr bool PAIR = dma_in_pairs<BM, BN, BKT, NSTAGE, NW, LA, LB, ESZ>();
  constexpr bool BSCALE = FP8 && MODE == KSEG;        // block-scaled contraction over tokens (weight gradients)
  static_assert(!BSCALE || (BKT == 128 && NSTAGE == 2), "one 128-token scale group per k-step; scale loads rely on the vmcnt(0) wait");
  constexpr int A_BYTES = DmaTileBytes<LA, BM, BKT, ESZ>::value, B_BYTES = DmaTileBytes<LB, BN, BKT, ESZ>::value;
  constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  constexpr int RING_BYTES = NSTAGE * STAGE_BYTES;
  // With 8 waves (two per SIMD; waves w and w + 4 share one) only the lower four issue loads: a wave stalls while
  // the texture-address queue is full (64 loads take ~1100 clocks), and this way its SIMD partner runs MFMAs
  // meanwhile.  Smaller workgroups (one wave per SIMD) let every wave load.
  constexpr bool SPLIT = (NW == 8);
  constexpr int NL = SPLIT ? NW / 2 : NW;                                      // loader waves
  constexpr int A_DMA = A_BYTES / 1024 / NL, B_DMA = B_BYTES / 1024 / NL;     // loads per loader wave per stage
  constexpr int LOADS = A_DMA + B_DMA;
  constexpr int KK = FP8 ? BKT / 128 : BKT / 32;   // MFMA sub-steps per k-step
  constexpr bool SWI = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_W;              // FC1 + SwiGLU epilogue
  constexpr bool FOLD = EPI == EPI_SWIGLU_W || EPI == EPI_SWIGLU_BWD_W;       // gate weight folded in (Section 4.1)
  constexpr bool GATHER_A = EPI == EPI_SWIGLU_W;                              // A rows selected by index map (Section 4.2)
  static_assert(!FOLD || (!FP8 && MODE == ROWSEG && LA == KMAJOR), "the folded order exists for the bf16 row-segmented kernels");
  constexpr int BN_OUT = SWI ? BN / 2 : BN;
  // Store instructions a wave issues in the epilogue of a full tile (branch-free buffer stores, bf16 kernels): two
  // per 32x32 bf16 block, four per fp32 block; 0 = not known at compile time.
  constexpr int EPI_STORES_RAW = EPI == EPI_STORE ? TM * TN * (sizeof(TC) == 4 ? 4 : 2)
                                 : SWI ? TM * TN * 3
                                 : EPI == EPI_SWIGLU_BWD ? TM * TN * 6
                                 : EPI == EPI_SWIGLU_BWD_W ? TM * TN * 6 + TM
                                 : 0;
  constexpr int EPI_STORES = (NSTAGE - 2) * LOADS + EPI_STORES_RAW <= 63 ? EPI_STORES_RAW : 0;   // vmcnt is a 6-bit field
  // what this wave's epilogue of the previous tile put into the memory queue (wave-uniform): exactly EPI_STORES stores,
  // nothing, or an unknown number
  enum { EPI_UNKNOWN = 0, EPI_ALL = 1, EPI_NONE = 2 };
  int epi_state = EPI_NONE;
  constexpr int GN = 8, XCDS = 8;   // GN n-tiles per group: a window of 32 tiles is 4 m-tiles x 8 n-tiles (measured against 8 x 4, 16 x 2, 2 x 16)
  static_assert(A_BYTES % (1024 * NL) == 0 && B_BYTES % (1024 * NL) == 0, "tile does not split over the loader waves");
  static_assert(NSTAGE >= 2 && (NSTAGE - 2) * LOADS < 64, "pipeline depth exceeds the vmcnt range");
  static_assert(!SWI || TN % 2 == 0, "SwiGLU pairs gate/up MFMA tiles inside a wave");
  static_assert(NW <= 8, "LDS is budgeted for at most 8 epilogue patches");

  // Fragments, chunks and sub-steps are told apart by flipping bits below 256 of an address (read_frag_dma, read_frag_fp8), so tiles
  // begin at multiples of 256 bytes.
  extern __shared__ __attribute__((aligned(256))) char smem[];
  static_assert(A_BYTES % 256 == 0 && STAGE_BYTES % 256 == 0, "every tile of the ring begins at a multiple of 256 bytes");
  const unsigned smem_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  int* cum_tiles = reinterpret_cast<int*>(smem + RING_BYTES);          // [E+1] running count of m-tiles (ROWSEG)
  constexpr int TABLE_BYTES = (MOE_MAX_EXPERTS + 8) * 4;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Waves w and w + 4 of eight share a SIMD.  In FC1 they lie in opposite halves of the tile along both sides, elsewhere along one.  Of 8
  // experts, 16384 rows, 4096 x 14336 (us, one side and both): FC1 3093, 3078, dgrad1 2920, 2955; of 4, 24576 rows 4415, 4385 and 4257,
  // 4281; of 64, 131072 rows, 2048 x 1408 1384, 1376 and 1216, 1220; the others the same.
  const int wm = wave / WN, wn = wave % WN ^ (SPLIT && SWI && wave >= NL ? WN / 2 : 0);
  const char* zero = reinterpret_cast<const char*>(g_zero_block);
  char* stg = smem + RING_BYTES + TABLE_BYTES + wave * STG_BYTES;      // this wave's epilogue patch
  // where this lane's fragments of the wave's first rows lie in a ring slot
  const unsigned fo_a = frag_origin<LA, BM, BKT, ESZ>(wm * WTM, lane);
  const unsigned fo_b = (unsigned)A_BYTES + frag_origin<LB, BN, BKT, ESZ>(wn * WTN, lane);

  // ---- the tile list ------------------------------------------------------------------------------
  // Workgroup b runs on XCD b % 8 and each XCD has its own L2.  The logical tile order is cut into windows
  // of W = G/8 consecutive tiles (one per CU of an XCD); a window is a compact block of one expert -- GN
  // adjacent n-tiles for a run of m-tiles -- whose tiles stream the same A and B panels at the same k, so
  // most of their loads hit in L2.  Windows are dealt round-robin to the XCDs: at any moment the eight
  // XCDs work on eight neighbouring windows, mostly the next m-tiles of the same n-tiles, i.e. the same B
  // panels (shared through the Infinity Cache) and disjoint A panels.
  const int tiles_n = (p.N + BN_OUT - 1) / BN_OUT;
  const int tiles_m_fixed = (p.M + BM - 1) / BM;              // KSEG / PLAIN
  int total_tiles;
  if constexpr (MODE == ROWSEG) {
    tile_table<BM>(p.offsets, p.E, cum_tiles);
    __syncthreads();
    total_tiles = __builtin_amdgcn_readfirstlane(cum_tiles[p.E]) * tiles_n;
  } else if constexpr (MODE == KSEG) {
    total_tiles = p.E * tiles_m_fixed * tiles_n;
  } else {
    total_tiles = tiles_m_fixed * tiles_n;
  }
  // split-K plan for the partly filled last round (see Args::splitk_ws); identical arithmetic in splitk_fixup_kernel
  constexpr bool SPLITK = MODE == ROWSEG && EPI == EPI_STORE && sizeof(TC) == 2;
  int full_tiles = total_tiles, split = 1, total_items = total_tiles;
  if constexpr (SPLITK) {
    if (p.splitk_ws != nullptr) splitk_plan(total_tiles, (int)gridDim.x, (p.K + BKT - 1) / BKT, full_tiles, split, total_items);
  }
  const int xcd = blockIdx.x % XCDS;
  const int window = gridDim.x / XCDS;           // tiles per window = CUs per XCD
  const int in_window = blockIdx.x / XCDS;
  int slot = 0;                                  // this XCD's window counter
  // All workgroups walk tiles of one length, so without more their epilogues coincide, and 256 epilogues at once write at what the
  // memory takes: 256 KB per workgroup in 12 us (5.6 TB/s), where 64 of them need 3 us (probe of the store pattern: 8, 32, 64, 128, 256
  // workgroups 2.2, 2.3, 3.0, 5.9, 12.1 us; 32 of one XCD alone 6.6).  The workgroups of an XCD therefore start in groups, each `lag`
  // k-steps of time after the one before, and walk the contraction from as many k-steps further on, wrapping around: at any moment
  // all of them are at the same k and go on sharing panels in their L2.  (Late starts without the rotation bring nothing: the late ones
  // find their panels in L2, run faster and catch up.)  Sizes and figures: Stagger in row_plan.h.
  // Only for e4m3: the walk decides the order in which a tile's products are added.  In bf16 equal rows and weights get equal bits whichever
  // workgroup has the tile, and whole layers gained no more than 1 % by it.
  constexpr bool STAGGER = FP8 && (MODE == KSEG || SWI) && BM == 256 && BN == 256;
  const int lag = STAGGER ? __builtin_amdgcn_readfirstlane(in_window * p.stagger.groups / window * p.stagger.lag) : 0;

  // tile state
  int e = 0, m0 = 0, m_end = 0, n0 = 0, klen = 0, nk = 0;
  int k_start = 0;                  // k-step this workgroup's walk begins at (see issue)
  int part_slot = -1;               // >= 0: this work item is one K part of a split tile; index of its partial tile
  const bool is_loader = !SPLIT || wave < NL;            // wave-uniform; the lower waves win issue arbitration
  const int lw = wave & (NL - 1);                        // loader index
  const char* a_base = zero;        // wave-uniform: operand origin of the open tile at its first k
  const char* b_base = zero;
  unsigned a_off[A_DMA], b_off[B_DMA];   // this lane's byte offset from the base, fixed over the k loop
  // k coordinate (relative to the k-step start) at which this lane's chunk of load slot 0 begins, and how far the following
  // slots lie on: K-major slots are whole swizzle periods apart
  constexpr int A_KSTEP = LA == KMAJOR ? 0 : A_BYTES / A_DMA / (BM * 2), B_KSTEP = LB == KMAJOR ? 0 : B_BYTES / B_DMA / (BN * 2);
  static_assert(LA != KMAJOR || NL * 1024 % (16 * BKT * ESZ) == 0, "a loader's K-major slots have different chunk orders");
  static_assert(LB != KMAJOR || NL * 1024 % (16 * BKT * ESZ) == 0, "a loader's K-major slots have different chunk orders");
  int a_k0 = 0, b_k0 = 0;
  // L2 touches (bf16 kernels).  The workgroups of a window stream the same A and B panels at the same k, so every
  // new line is requested by several of them at once and all of them wait for the one fill.  At the end of k-step kt
  // the first wave that does not load (wave NL) touches this workgroup's quarter of the A-panel lines that the
  // loader waves request next (the n-tiles of a group share the A panel; quarter = position in the group mod 4).
  // Measured: touches at the start of a step queue behind the tile loads in the texture-address unit (kernel 16 %
  // slower); at the end of the step they gain 1.2 to 3 %; one or two steps further ahead: no change; touching the B
  // panel as well, or half of A, or from two waves: slower again (each touch instruction costs the address unit as
  // much as a 1 KB tile load).  Not for e4m3 operands: half the time per k-step for the same loads, touches cost 2 %.
  constexpr bool TOUCH = MODE == ROWSEG && NSTAGE == 2 && SPLIT && !FP8;
  // the same for the bf16 weight-gradient kernel (four stages of 32 k-rows): two k-steps per touch, every other step
  constexpr bool TOUCH_K = MODE == KSEG && !FP8 && SPLIT && LA == MNMAJOR && LB == MNMAJOR && NSTAGE == 4;
  constexpr bool TOUCH_K2 = MODE == KSEG && !FP8 && SPLIT && LA == MNMAJOR && LB == MNMAJOR && NSTAGE == 2 && BKT == 64;
  const bool is_toucher = (TOUCH || TOUCH_K || TOUCH_K2) && wave == NL;
  const unsigned lds_dump = smem_lds + RING_BYTES + TABLE_BYTES + NW * STG_BYTES;
  const unsigned scale_lds = lds_dump + 256;                                   // block-scale ring: 2 stages x (256 + 256) bytes
  const char* scale_smem = smem + RING_BYTES + TABLE_BYTES + NW * STG_BYTES + 256;
  unsigned ta_off = 0;
  // rotation of this workgroup's load order within the A / B tile (see open_tile); only where it pays: the e4m3
  // row-segmented kernels (in the others the extra scalar state pushes tile offsets out of registers)
  constexpr bool ROT = FP8 && MODE == ROWSEG;
  int rot_a = 0, rot_b = 0;
  // block scales of the current and the next k-step for this lane's fragment rows (byte 0 of each register)
  // Block scales (e4m3 weight gradients): the 256 + 256 E8M0 bytes of a k-step travel global -> LDS with the tiles
  // (two 4-byte direct-to-LDS loads by loader wave 0, into a two-stage ring of 512 bytes) and every wave reads its
  // rows' bytes from there.  Fetching them per lane from global memory took six more vector-memory instructions per
  // wave and k-step, 48 per workgroup next to the 64 tile loads, and the address unit is what the load issue is
  // bound by: the k-step was 0.4 us longer.
  static_assert(!BSCALE || (BM == 256 && BN == 256), "one 4-byte load per lane covers the 256 channels of a tile side");
  int sa_cur[FM], sb_cur[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) sa_cur[i] = 127;
#pragma unroll
  for (int j = 0; j < FN; ++j) sb_cur[j] = 127;
  const char* sa_base = nullptr;        // scale row of the tile's first k-step (wave-uniform)
  const char* sb_base = nullptr;
  unsigned sa_voff = 0, sb_voff = 0;    // this lane's four channels
  const long a_step = (LA == KMAJOR) ? (long)BKT * ESZ : (long)BKT * p.lda * ESZ;   // bytes per k-step
  const long b_step = (LB == KMAJOR) ? (long)BKT * ESZ : (long)BKT * p.ldb * ESZ;

  // Decode slot -> tile and set up this lane's source pointers.  Returns false when the list is exhausted.
  auto open_tile = [&](int sl) __attribute__((always_inline)) -> bool {
    const int first = sl * XCDS * window;
    const int w = tiles_per_xcd(total_items, total_items - first, window, PAIR);
    int l = first + xcd * w + in_window;
    if (in_window >= w || l >= total_items) return false;
    int part = 0;
    part_slot = -1;
    if (l >= full_tiles) {           // only with SPLITK: parts of one tile are neighbours in the list
      part_slot = l - full_tiles;
      part = part_slot % split;
      l = full_tiles + part_slot / split;
    }
    int mt_e, m_lo, m_hi;
    if constexpr (MODE == ROWSEG) {
      // binary search: largest ex with cum_tiles[ex] * tiles_n <= l
      int lo = 0, hi = p.E;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cum_tiles[mid] * tiles_n <= l) lo = mid; else hi = mid;
      }
      // everything about the tile is wave-uniform: keep it in scalar registers
      e = __builtin_amdgcn_readfirstlane(lo);
      mt_e = __builtin_amdgcn_readfirstlane(cum_tiles[e + 1] - cum_tiles[e]);
      l = __builtin_amdgcn_readfirstlane(l - cum_tiles[e] * tiles_n);
      m_lo = p.offsets[e]; m_hi = p.offsets[e + 1];
    } else {
      mt_e = tiles_m_fixed;
      e = l / (mt_e * tiles_n);          // always 0 in PLAIN mode
      l -= e * mt_e * tiles_n;
      m_lo = 0; m_hi = p.M;
    }
    const int ng = l / (mt_e * GN);
    const int r = l - ng * mt_e * GN;
    const int gw = min(GN, tiles_n - ng * GN);
    const int mt = r / gw;
    const int nt = ng * GN + (r - mt * gw);
    m0 = m_lo + mt * BM; m_end = m_hi; n0 = nt * BN_OUT;
    // Sharers of a panel start their loads at different quarters of it (the n-tiles of a group share A, the m-tiles
    // of a window share B), so that the first request for each new line, the one that starts its L2 fill, is spread
    // over the sharers and over the step instead of all of them queueing on the same line in the same order.
    if constexpr (ROT) {
      rot_a = __builtin_amdgcn_readfirstlane(((r - mt * gw) & 3) * A_DMA / 4);
      rot_b = __builtin_amdgcn_readfirstlane((mt & 3) * B_DMA / 4);
    }
    int k_begin, k_end;
    if constexpr (MODE == KSEG) { k_begin = p.offsets[e]; k_end = p.offsets[e + 1]; }
    else { k_begin = 0; k_end = p.K; }
    klen = k_end - k_begin;
    nk = (klen + BKT - 1) / BKT;
    if (part_slot >= 0) {            // this item covers k-steps [s0, s1) of the tile
      const int s0 = part * nk / split, s1 = (part + 1) * nk / split;
      k_begin += s0 * BKT;
      klen = min(klen, s1 * BKT) - s0 * BKT;
      nk = s1 - s0;
    }
    if constexpr (STAGGER) k_start = nk > 0 ? lag % nk : 0;
    else k_start = (xcd * 2 + in_window * 2 / window) * nk / (2 * XCDS);
    const char* Ag = static_cast<const char*>(p.A);
    const char* Bg = static_cast<const char*>(p.B) + (long)e * p.b_es * ESZ;
    // Base of each operand at the tile's first k (wave-uniform) and this lane's fixed byte offset from it.
    // Load j of loader wave lw fills DMA slot q = lw + j*NL of the tile (1 KiB of LDS each).
    if constexpr (GATHER_A) a_base = uniform_ptr(Ag + (long)k_begin * ESZ);          // row offsets are absolute
    else if constexpr (LA == KMAJOR) a_base = uniform_ptr(Ag + ((long)m0 * p.lda + k_begin) * ESZ);
    else a_base = uniform_ptr(Ag + (long)k_begin * p.lda * ESZ);
    if constexpr (LB == KMAJOR) b_base = uniform_ptr(Bg + (long)k_begin * ESZ);
    else b_base = uniform_ptr(Bg + (long)k_begin * p.ldb * ESZ);
#pragma unroll
    for (int j = 0; j < A_DMA; ++j) {
      const int q = lw + ((j + rot_a) % A_DMA) * NL;
      if constexpr (LA == KMAJOR) {
        using TL = KTile<BM, BKT, ESZ>;
        const int row = q * TL::ROWS_PER_DMA + lane / TL::CPR;
        const int lc = (lane % TL::CPR) ^ TL::swz(lw * TL::ROWS_PER_DMA + lane / TL::CPR);
        int rel = min(row, p.M - 1 - m0);                             // rows past the end of A repeat its last row
        if constexpr (GATHER_A) rel = p.a_rowmap[m0 + rel];           // < a_phys_rows: the launcher's contract
        a_off[j] = (unsigned)rel * (unsigned)(p.lda * ESZ) + (unsigned)(lc * 16);
        a_k0 = lc * CHUNK;
      } else {
        using TL = MNTile<BM, BKT>;
        const int krow = q * TL::ROWS_PER_DMA + lane / TL::CPR;
        const int lc = (lane % TL::CPR) ^ TL::swz(krow);
        const int col = min(m0 + lc * 8, p.M - 8);
        a_off[j] = (unsigned)krow * (unsigned)(p.lda * ESZ) + (unsigned)(col * ESZ);
        a_k0 = lw * TL::ROWS_PER_DMA + lane / TL::CPR;
      }
    }
#pragma unroll
    for (int j = 0; j < B_DMA; ++j) {
      const int q = lw + ((j + rot_b) % B_DMA) * NL;
      if constexpr (LB == KMAJOR) {
        using TL = KTile<BN, BKT, ESZ>;
        const int row = q * TL::ROWS_PER_DMA + lane / TL::CPR;
        const int lc = (lane % TL::CPR) ^ TL::swz(lw * TL::ROWS_PER_DMA + lane / TL::CPR);
        int gr;
        if constexpr (SWI) {
          const int qq = row >> 5;
          const int n = min(n0 + (qq >> 1) * 32 + (row & 31), p.f - 1);
          gr = (qq & 1) ? p.f + n : n;
        } else {
          gr = min(n0 + row, p.N - 1);
        }
        b_off[j] = (unsigned)gr * (unsigned)(p.ldb * ESZ) + (unsigned)(lc * 16);     // < 4 GiB: checked by the launcher
        b_k0 = lc * CHUNK;
      } else {
        using TL = MNTile<BN, BKT>;
        const int krow = q * TL::ROWS_PER_DMA + lane / TL::CPR;
        const int lc = (lane % TL::CPR) ^ TL::swz(krow);
        const int col = min(n0 + lc * 8, p.N - 8);
        b_off[j] = (unsigned)krow * (unsigned)(p.ldb * ESZ) + (unsigned)(col * ESZ);
        b_k0 = lw * TL::ROWS_PER_DMA + lane / TL::CPR;
      }
    }
    if constexpr (TOUCH) {
      // the gw n-tiles of a group share the A panel: quarter (position in the group mod 4) of its 256 rows, one line per lane
      const int qa = (r - mt * gw) & 3;
      int arow = min(qa * 64 + lane, p.M - 1 - m0);
      if constexpr (GATHER_A) arow = p.a_rowmap[m0 + arow];
      ta_off = (unsigned)arow * (unsigned)(p.lda * ESZ);
    }
    if constexpr (TOUCH_K2) {
      // weight gradient, 64-deep steps: this workgroup's quarter (16 k-rows x 4 lines) of the A tile of one k-step
      const int qa = (r - mt * gw) & 3;
      ta_off = (unsigned)(qa * 16 + (lane >> 2)) * (unsigned)(p.lda * ESZ) + (unsigned)(min(m0 + (lane & 3) * 64, p.M - 8) * ESZ);
    }
    if constexpr (TOUCH_K) {
      // weight gradient, 32-deep steps: lanes 0..31 take this workgroup's quarter (8 k-rows x 4 lines) of the A tile of one k-step,
      // lanes 32..63 the same quarter of the following k-step
      const int qa = (r - mt * gw) & 3;
      const int kr = (lane >> 5) * BKT + (((lane & 31) >> 2));
      ta_off = (unsigned)(kr + qa * 8) * (unsigned)(p.lda * ESZ) + (unsigned)(min(m0 + (lane & 3) * 64, p.M - 8) * ESZ);
    }
    if constexpr (BSCALE) {
      const long g0 = k_begin / BKT;
      sa_base = uniform_ptr(reinterpret_cast<const char*>(p.a_e8m0) + g0 * p.a_e8_ld);
      sb_base = uniform_ptr(reinterpret_cast<const char*>(p.b_e8m0) + g0 * p.b_e8_ld);
      // channels past the end repeat the last four (their rows and columns are masked when the tile is stored)
      sa_voff = (unsigned)min(m0 + 4 * lane, p.M - 4);
      sb_voff = (unsigned)min(n0 + 4 * lane, p.N - 4);
    }
    return true;
  };
  // The small tiles stream the weights, and with every workgroup at the same columns of its rows the requests of a moment
  // crowd on few memory channels (row strides are multiples of kilobytes).  Each XCD starts its walk over the contraction an
  // eighth further on and wraps around, and the second half of its workgroups (other n-tiles, mostly of the same expert) a
  // sixteenth after that.  Measured on the 64-row tile (us; one start, one per XCD, this): 8 experts, 4 rows, FC1 of 4096 x
  // 14336 334, 303, 304, FC2 180, 168, 155; 64 experts, 32 rows, FC1 of 2048 x 1408 164, 143, 143; 8 experts, 8 rows, FC1 of
  // 2048 x 8192 116, 96, 97.  A start of its own for every workgroup of an XCD: 362, 159, 141, 106.
  constexpr bool KROT = (MODE == ROWSEG && BM <= 128) || STAGGER;
  // Issue the loads of k-step `ks` of the open tile into ring slot ks % NSTAGE.  Only the last step can be ragged.
  auto issue = [&](int ks) __attribute__((always_inline)) {
    if (!is_loader) return;
    const int ring = ks % NSTAGE;
    const unsigned stage = smem_lds + (unsigned)ring * STAGE_BYTES;
    if constexpr (KROT) {
      ks += k_start;
      if (ks >= nk) ks -= nk;
    }
    const int k_left = klen - ks * BKT;          // valid k in this step
    const char* ab = a_base + (long)ks * a_step;     // scalar arithmetic
    const char* bb = b_base + (long)ks * b_step;
    if constexpr (BSCALE) {
      if (lw == 0) {
        const unsigned dst = scale_lds + (unsigned)ring * 512u;
        touch4s(sa_base + (long)ks * p.a_e8_ld, sa_voff, dst);
        touch4s(sb_base + (long)ks * p.b_e8_ld, sb_voff, dst + 256u);
      }
    }
    if (k_left >= BKT) {
      // the e4m3 weight-gradient kernel asks for the B tile first, the others for the A tile: measured
      constexpr bool B_FIRST = FP8 && MODE == KSEG;
      if constexpr (A_DMA == 8 && B_DMA == 8 && NL == 4 && A_BYTES == 8 * 4096 && !ROT && !B_FIRST) {
        dma16s_x16(ab, bb, a_off, b_off, stage + (unsigned)lw * 1024u);
      } else {
        if constexpr (B_FIRST) {
#pragma unroll
          for (int j = 0; j < B_DMA; ++j) dma16s(bb, b_off[j], stage + A_BYTES + (unsigned)(lw + ((j + rot_b) % B_DMA) * NL) * 1024u);
        }
#pragma unroll
        for (int j = 0; j < A_DMA; ++j) dma16s(ab, a_off[j], stage + (unsigned)(lw + ((j + rot_a) % A_DMA) * NL) * 1024u);
        if constexpr (!B_FIRST) {
#pragma unroll
          for (int j = 0; j < B_DMA; ++j) dma16s(bb, b_off[j], stage + A_BYTES + (unsigned)(lw + ((j + rot_b) % B_DMA) * NL) * 1024u);
        }
      }
    } else {
      // ragged last step: chunks past the end of the contraction come from the zero block.  The offsets pass
      // through an empty asm so that their 64-bit extensions are made here, in the cold path, instead of being
      // kept in register pairs across the whole k loop.
#pragma unroll
      for (int j = 0; j < A_DMA; ++j) {
        unsigned off = a_off[j];
        asm volatile("" : "+v"(off));
        dma16(a_k0 + ((j + rot_a) % A_DMA) * A_KSTEP >= k_left ? zero : ab + off, stage + (unsigned)(lw + ((j + rot_a) % A_DMA) * NL) * 1024u);
      }
#pragma unroll
      for (int j = 0; j < B_DMA; ++j) {
        unsigned off = b_off[j];
        asm volatile("" : "+v"(off));
        dma16(b_k0 + ((j + rot_b) % B_DMA) * B_KSTEP >= k_left ? zero : bb + off, stage + A_BYTES + (unsigned)(lw + ((j + rot_b) % B_DMA) * NL) * 1024u);
      }
    }
  };
  auto issue_prologue = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < NSTAGE - 1; ++s)
      if (s < nk) issue(s);
  };

  if (!open_tile(slot)) return;
  if constexpr (STAGGER) {
    // (a k-step takes 1.5 us; the counter runs at 100 MHz)
    const unsigned long long until = __builtin_amdgcn_s_memrealtime() + (unsigned)lag * 150u;
    while ((long long)(__builtin_amdgcn_s_memrealtime() - until) < 0) __builtin_amdgcn_s_sleep(8);
  }
  issue_prologue();

  for (;;) {
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Wait until this wave's loads for step s have landed.  vmcnt counts loads and stores together, in issue order, so
    // the wait names how many younger operations may still be outstanding: the loads of the (NSTAGE - 2) following
    // steps, and, in the first NSTAGE - 1 steps of a tile (whose loads were issued before the previous tile's
    // epilogue), that epilogue's stores when their number is known (unknown: wait for everything).  With few rows per
    // expert no tile is full, but a wave still issues all of its (masked) stores or none: waiting for everything at each
    // tile's start would drain the ring there.
    auto wait_step = [&](int s) __attribute__((always_inline)) {
      if (s + NSTAGE - 2 < nk) {
        if constexpr (EPI_STORES > 0) {
          if (s < NSTAGE - 1 && epi_state == EPI_ALL) { wait_vmcnt<(NSTAGE - 2) * LOADS + EPI_STORES>(); return; }
        }
        if (s > 0 || epi_state == EPI_NONE) { wait_vmcnt<(NSTAGE - 2) * LOADS>(); return; }
      }
      wait_vmcnt<0>();
    };
    // ---- k loop ------------------------------------------------------------------------------------
    // Fragments are read one phase ahead (see below), also across the step barrier.  The barrier that opens step s+1 sits
    // before the last phase's products of step s (whose fragments are in registers by then), so the first fragment reads of
    // a step, which all eight waves issue at once, overlap products instead of leaving the matrix cores idle at every step
    // start: -1.6 to -2.2 % on the bf16 forward kernels and dgrad1, -4 to -6 % on the weight-gradient kernel with 64-deep
    // steps (with 32-deep steps it gains nothing), -6 % on the e4m3 FC2 and dgrad1, -2 % on the e4m3 FC1.  The dgrad2 kernels
    // gain from it once their epilogue ends with an explicit vmcnt wait (see there).
    constexpr bool XPIPE = MODE != KSEG || NSTAGE == 2;
    if constexpr (XPIPE) {
      // A sub-step is cut into phases: the wave's fragments of its shorter side are held for the whole sub-step, those of
      // the longer side pass through PC at a time.  Phase p multiplies while the fragments of phase p + 1 are read.
      constexpr bool HOLD_A = FM <= FN;
      constexpr int FH = HOLD_A ? FM : FN, FS = HOLD_A ? FN : FM;
      constexpr int PC = !FP8 && FS % 4 == 0 ? 4 : 2, NPH = FS / PC;
      constexpr int PHASES = KK * NPH;
      // One sub-step per step (e4m3): the held fragments have no second set.  In the last phase each is read again, from the
      // next step, as soon as its last product is issued.
      constexpr int HSETS = KK % 2 == 0 ? 2 : 1;
      static_assert((HSETS == 2 || KK == 1) && PHASES % 2 == 0 && FS % PC == 0, "fragment sets alternate by sub-step and by phase parity");
      static_assert(!BSCALE || (KK == 1 && HOLD_A), "group scales are read with the held fragments' order");
      // opens step s: its loads have landed (at most the younger steps' loads are outstanding; the first step of a
      // tile also drains the previous tile's epilogue stores), every wave is done with step s-1, whose stage is
      // refilled right away
      auto open_step = [&](int s) __attribute__((always_inline)) {
        if (!is_toucher) {                  // (the touching wave has no tile loads of its own to wait for)
          wait_step(s);
        }
        __syncthreads();
        if (s + NSTAGE - 1 < nk) issue(s + NSTAGE - 1);
      };
      // A wave whose rows all lie past the last one (of the expert, or of the gradient), or whose columns all lie past the width, has nothing
      // to multiply (wave-uniform; it still issues its loads and takes part in the barriers).  In a nearly empty last tile only one or two
      // waves per CU then use the matrix cores, and the k-step shrinks to what the loads need.
      // Eight waves, columns and gradient rows as well (us): 64 experts, 131072 rows, 2048 x 1408 d_w2 766 -> 749, dgrad1 1260 -> 1250, d_w1 1443 ->
      // 1427; 8 experts, 16384 rows, 1040 x 1424 d_w2 61 -> 58, dgrad1 127 -> 122, d_w1 119 -> 111.  (Four waves have no partner on their SIMD.)
      const bool wave_active = SPLIT ? m0 + wm * WTM < m_end && n0 + wn * (SWI ? WTN / 2 : WTN) < (SWI ? p.f : p.N)
                                     : MODE != ROWSEG || m0 + wm * WTM < m_end;
      if (!wave_active) {
        for (int s = 0; s < nk; ++s) open_step(s);
      } else if (nk > 0) {
        using Frag = std::conditional_t<FP8, i32x8, bf16x8>;
        Frag held[HSETS][FH], strm[2][PC];
        auto read_a = [&](unsigned ao, int i, int kk) __attribute__((always_inline)) -> Frag {
          if constexpr (FP8) return read_frag_fp8<BM, BKT>(ao, i, kk); else return read_frag_dma<LA, BM, BKT>(ao, i, kk);
        };
        auto read_b = [&](unsigned bo, int j, int kk) __attribute__((always_inline)) -> Frag {
          if constexpr (FP8) return read_frag_fp8<BN, BKT>(bo, j, kk); else return read_frag_dma<LB, BN, BKT>(bo, j, kk);
        };
        auto origins = [&](unsigned slot_lds, unsigned& ao, unsigned& bo) __attribute__((always_inline)) {
          ao = fo_a + slot_lds;
          bo = fo_b + slot_lds;
          if constexpr (LA == MNMAJOR) asm volatile("" : "+v"(ao));
          if constexpr (LB == MNMAJOR) asm volatile("" : "+v"(bo));
        };
        // held fragment h of sub-step kk; the streamed fragments of phase p; the group scales of a step's A and B rows
        auto read_held = [&](unsigned ao, unsigned bo, int h, int kk) __attribute__((always_inline)) {
          held[kk % HSETS][h] = HOLD_A ? read_a(ao, h, kk) : read_b(bo, h, kk);
        };
        auto read_strm = [&](unsigned ao, unsigned bo, int p) __attribute__((always_inline)) {
          const int kk = p / NPH, ph = p % NPH;
#pragma unroll
          for (int c = 0; c < PC; ++c) strm[p & 1][c] = HOLD_A ? read_b(bo, ph * PC + c, kk) : read_a(ao, ph * PC + c, kk);
        };
        auto scale_a = [&](int step, int i) __attribute__((always_inline)) {
          sa_cur[i] = reinterpret_cast<const unsigned char*>(scale_smem)[(step % NSTAGE) * 512 + wm * WTM + i * 16 + (lane & 15)];
        };
        auto scale_b = [&](int step, int j) __attribute__((always_inline)) {
          sb_cur[j] = reinterpret_cast<const unsigned char*>(scale_smem)[(step % NSTAGE) * 512 + 256 + wn * WTN + j * 16 + (lane & 15)];
        };
        open_step(0);
        {
          unsigned ao, bo;
          origins(smem_lds, ao, bo);
#pragma unroll
          for (int h = 0; h < FH; ++h) read_held(ao, bo, h, 0);
          read_strm(ao, bo, 0);
          if constexpr (BSCALE) {
#pragma unroll
            for (int i = 0; i < FM; ++i) scale_a(0, i);
#pragma unroll
            for (int j = 0; j < FN; ++j) scale_b(0, j);
          }
        }
        for (int kt = 0; kt < nk; ++kt) {
          const unsigned at = smem_lds + (unsigned)(kt % NSTAGE) * STAGE_BYTES;
#pragma unroll
          for (int p = 0; p < PHASES; ++p) {
            constexpr int TOUCH_AT = PHASES >= 2 ? PHASES - 2 : 0;      // one phase ahead of the refill it runs before (later: slower)
            if constexpr (TOUCH || TOUCH_K2) {
              if (p == TOUCH_AT && is_toucher && (kt + NSTAGE + 1) * BKT <= klen) {   // whole k-steps only: every touched address exists
                touch4s(a_base + (long)(kt + NSTAGE) * a_step, ta_off, lds_dump);
              }
            }
            const bool last = p + 1 == PHASES;
            const int pn = (p + 1) % PHASES, kn = pn / NPH;
            unsigned ao, bo;
            auto read_next = [&](unsigned slot_lds) __attribute__((always_inline)) {
              origins(slot_lds, ao, bo);
              if (HSETS == 2 && pn % NPH == 0) {
#pragma unroll
                for (int h = 0; h < FH; ++h) read_held(ao, bo, h, kn);
              }
              read_strm(ao, bo, pn);
            };
            if (!last) {
              read_next(at);
            } else {
              if constexpr (HSETS == 1) {
                // the products issued so far stay in front of the barrier: moved behind it, as the compiler would, they
                // keep every streamed fragment of the step in registers
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                  for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(acc[i][j]));
              }
              // This phase's fragments are waited for on the way to both paths (the barrier needs that anyway): left to where the
              // paths meet, the wait would also hold up this phase's products behind the reads just issued on one of them.
              wait_lgkmcnt0();
              if (kt + 1 < nk) {
                open_step(kt + 1);
                read_next(smem_lds + (unsigned)((kt + 1) % NSTAGE) * STAGE_BYTES);
              } else {
                if constexpr (HSETS == 1) origins(at, ao, bo);      // the last step reads its own held fragments again
              }
            }
            const int kk = p / NPH, ph = p % NPH;
            auto product = [&](int h, int c) __attribute__((always_inline)) {
              const Frag fa = HOLD_A ? held[kk % HSETS][h] : strm[p & 1][c], fb = HOLD_A ? strm[p & 1][c] : held[kk % HSETS][h];
              const int i = HOLD_A ? h : ph * PC + c, j = HOLD_A ? ph * PC + c : h;
              // e4m3 x e4m3 (format selectors 0, 0); block scales 2^0 (E8M0 code 127) unless the operands are scaled by group
              if constexpr (FP8)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fb, fa, acc[i][j], 0, 0, 0, BSCALE ? sb_cur[j] : 127, 0, BSCALE ? sa_cur[i] : 127);
              else
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb, fa, acc[i][j], 0, 0, 0);
            };
            if (HSETS == 1 && last) {
              if constexpr (BSCALE) {
#pragma unroll
                for (int j = 0; j < FN - PC; ++j) scale_b(kt + 1 < nk ? kt + 1 : kt, j);
              }
#pragma unroll
              for (int h = 0; h < FH; ++h) {
#pragma unroll
                for (int c = 0; c < PC; ++c) product(h, c);
                read_held(ao, bo, h, 0);
                if constexpr (BSCALE) scale_a(kt + 1 < nk ? kt + 1 : kt, h);
                __builtin_amdgcn_sched_barrier(0);
              }
              if constexpr (BSCALE) {
#pragma unroll
                for (int j = FN - PC; j < FN; ++j) scale_b(kt + 1 < nk ? kt + 1 : kt, j);
              }
            } else {
#pragma unroll
              for (int c = 0; c < PC; ++c)
#pragma unroll
                for (int h = 0; h < FH; ++h) product(h, c);
            }
            if constexpr (HSETS == 1) __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    } else
    for (int kt = 0; kt < nk; ++kt) {
      static_assert(XPIPE || !FP8, "reads bf16 fragments");
      // my loads for step kt have landed once at most the younger steps' loads are outstanding; the first
      // step of a tile also drains the previous tile's epilogue stores, which share the counter
      if (!is_toucher) {                    // (the touching wave has no tile loads of its own to wait for)
        wait_step(kt);
      }
      __syncthreads();
      if (kt + NSTAGE - 1 < nk) issue(kt + NSTAGE - 1);

      const unsigned at = smem_lds + (unsigned)(kt % NSTAGE) * STAGE_BYTES;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        if constexpr (TOUCH_K) {
          // late in the step, when the tile loads of this step have left the texture-address queue
          if (kk == KK - 1 && is_toucher && (kt & 1) == 0 && (kt + NSTAGE + 2) * BKT <= klen) {
            touch4s(a_base + (long)(kt + NSTAGE) * a_step, ta_off, lds_dump);
          }
        }
        {
          bf16x8 af[FM], bfr[FN];
#pragma unroll
          for (int i = 0; i < FM; ++i) af[i] = read_frag_dma<LA, BM, BKT>(fo_a + at, i, kk);
#pragma unroll
          for (int j = 0; j < FN; ++j) bfr[j] = read_frag_dma<LB, BN, BKT>(fo_b + at, j, kk);
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
        }
      }
    }

    if constexpr (TOUCH || TOUCH_K || TOUCH_K2) {
      if (is_toucher) wait_vmcnt<0>();      // no touch may still be on its way into LDS when the patches are used
    }
    // ---- hand the ring to the next tile, then write this one out -------------------------------------
    const int ep_e = e, ep_m0 = m0, ep_m_end = m_end, ep_n0 = n0, ep_part_slot = part_slot;
    // a full tile that is no split-K part and does not read-modify-write issues every store of its epilogue; a wave of
    // one 32-row block does so if it has a valid row, and issues none otherwise
    epi_state = EPI_UNKNOWN;
    if (EPI_STORES > 0 && part_slot < 0 && !p.accumulate && n0 + BN_OUT <= (SWI ? p.f : p.N)) {
      if (m0 + BM <= m_end || (TM == 1 && m0 + wm * WTM < m_end)) epi_state = EPI_ALL;
      else if (TM == 1) epi_state = EPI_NONE;
    }
    // SwiGLU' (bf16): the saved G and U of the wave's first block are asked for before the hand-over, ahead of the
    // next tile's first loads in the memory queue
    constexpr bool EARLY_GU = EPI == EPI_SWIGLU_BWD || EPI == EPI_SWIGLU_BWD_W;
    StageFetch fg_first, fu_first;
    if constexpr (EARLY_GU) {
      const int mb = m0 + wm * WTM, nb = n0 + wn * WTN;
      const bf16* hrow = p.H + (long)mb * 2 * p.N + nb;
      fg_first = stage_fetch_bf16(hrow, 2L * p.N, m_end - mb, p.N - nb, lane);
      fu_first = stage_fetch_bf16(hrow + p.N, 2L * p.N, m_end - mb, p.N - nb, lane);
    }
    slot += 1;
    __syncthreads();                      // every wave has read its last fragments: the ring is free
    const bool has_next = open_tile(slot);
    if (has_next) {
      issue_prologue();
    }
    {
      const int e = ep_e, m0 = ep_m0, m_end = ep_m_end, n0 = ep_n0;
      (void)e;
      // e4m3 operands with per-row / per-output-channel scales: output = acc * scale of the row (token) * scale of
      // the output channel, applied block by block right before a block is written, so that only one block's 16
      // channel scales are live at a time
      auto block = [&](int i, int j) __attribute__((always_inline)) -> Block {
        Block b = {{acc[2 * i][2 * j], acc[2 * i][2 * j + 1], acc[2 * i + 1][2 * j], acc[2 * i + 1][2 * j + 1]}};
        if constexpr (FP8 && !BSCALE) {
          float rs[2] = {1.f, 1.f};
          f32x4 cs[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            if (p.row_scale) rs[h] = p.row_scale[min(m0 + wm * WTM + i * 32 + patch_row(2 * h, lane), p.M - 1)];
            int n;
            if constexpr (SWI) {
              const int nn = min(n0 + ((wn * WTN + (j & ~1) * 32) >> 1) + patch_col(h, lane), p.f - 4);
              n = (j & 1) ? p.f + nn : nn;
            } else {
              n = min(n0 + wn * WTN + j * 32 + patch_col(h, lane), p.N - 4);
            }
            cs[h] = f32x4{1.f, 1.f, 1.f, 1.f};
            if (p.col_scale) cs[h] = *reinterpret_cast<const f32x4*>(p.col_scale + (long)e * p.cs_es + n);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) b.q[q][t] *= rs[q >> 1] * cs[q & 1][t];
        }
        return b;
      };
      // every 32x32 block goes through the wave's LDS patch (see stage_store_* above)
      if (SPLITK && ep_part_slot >= 0) {
        // one K part of a split tile: the whole fp32 tile goes to the partial buffer, no masks
        float* part_tile = p.splitk_ws + (long)ep_part_slot * (BM * BN);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            stage_store_f32(stg, block(i, j), part_tile + (long)(wm * WTM + i * 32) * BN + wn * WTN + j * 32, BN, 32, 32, false, lane);
          }
      } else if constexpr (EPI == EPI_STORE) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int mb = m0 + wm * WTM + i * 32;
          const int rows_valid = m_end - mb;
          if (rows_valid <= 0) continue;
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const int nb = n0 + wn * WTN + j * 32;
            const int cols_valid = p.N - nb;
            if (cols_valid <= 0) continue;
            const Block b = block(i, j);
            if constexpr (sizeof(TC) == 4) {
              float* g = static_cast<float*>(p.C) + (long)e * p.c_es + (long)mb * p.ldc + nb;
              stage_store_f32(stg, b, g, p.ldc, rows_valid, cols_valid, p.accumulate != 0, lane);
            } else {
              bf16* g = static_cast<bf16*>(p.C) + (long)e * p.c_es + (long)mb * p.ldc + nb;
              bf16x4 v[4];
              if (p.accumulate) {
                bf16x4 old[4];
                stage_load_bf16(stg, old, g, p.ldc, rows_valid, cols_valid, lane);
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                  for (int t = 0; t < 4; ++t)
                    v[q][t] = static_cast<bf16>(b.q[q][t] + static_cast<float>(old[q][t]));
              } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                  for (int t = 0; t < 4; ++t) v[q][t] = static_cast<bf16>(b.q[q][t]);
              }
              stage_store_bf16(stg, v, g, p.ldc, rows_valid, cols_valid, lane);
            }
          }
        }
      } else if constexpr (EPI == EPI_BIAS_F32) {
        float* __restrict__ Cg = static_cast<float*>(p.C);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const int m = m0 + wm * WTM + i * 16 + (lane & 15);
          if (m >= m_end) continue;
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int n = n0 + wn * WTN + j * 16 + ((lane >> 4) << 2) + r;
              if (n < p.N) Cg[(long)m * p.ldc + n] = acc[i][j][r] + (p.bias ? p.bias[n] : 0.f);
            }
        }
      } else if constexpr (SWI) {
        // block 2j holds G and block 2j+1 holds U for the same 32 output columns
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int mb = m0 + wm * WTM + i * 32;
          const int rows_valid = m_end - mb;
          if (rows_valid <= 0) continue;
          float w_row[2] = {1.0f, 1.0f};                        // of this lane's two rows of the block
          if constexpr (FOLD) {
#pragma unroll
            for (int h = 0; h < 2; ++h) w_row[h] = p.row_w[min(mb + patch_row(2 * h, lane), p.M - 1)];
          }
#pragma unroll
          for (int j = 0; j < TN; j += 2) {
            const int nb = n0 + ((wn * WTN + j * 32) >> 1);
            const int cols_valid = p.f - nb;
            if (cols_valid <= 0) continue;
            const Block bg = block(i, j), bu = block(i, j + 1);
            bf16x4 g[4], u[4], a[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                g[q][t] = static_cast<bf16>(bg.q[q][t]);
                u[q][t] = static_cast<bf16>(bu.q[q][t]);
                const float gf = static_cast<float>(g[q][t]);
                a[q][t] = static_cast<bf16>(w_row[q >> 1] * (gf * sigmoid_f32(gf) * static_cast<float>(u[q][t])));
              }
            bf16* hrow = p.H + (long)mb * 2 * p.f + nb;
            stage_store_bf16(stg, g, hrow, 2L * p.f, rows_valid, cols_valid, lane);
            stage_store_bf16(stg, u, hrow + p.f, 2L * p.f, rows_valid, cols_valid, lane);
            stage_store_bf16(stg, a, p.A_out + (long)mb * p.f + nb, p.f, rows_valid, cols_valid, lane);
          }
        }
      } else {
        // acc = dA; read G|U, write dG|dU and the recomputed SwiGLU output.  Folded order (Section 4.1): acc is dA', the
        // gradient w.r.t. A' = w_r * A.  dG|dU are written for dA' as it is (the row's weight is applied downstream:
        // once per row in the combine of d_xp and in the rows handed to wgrad1, not per element here), the stored
        // FC2 input is A', and <dA'[r,:], A[r,:]> over this wave's columns goes to dw_part as one partial sum of the
        // gate-weight gradient of row r.
        auto swiglu_bwd_block = [&](const Block& dacc, const bf16x4 (&g)[4], const bf16x4 (&u)[4], int mb, int nb,
                                    int rows_valid, int cols_valid, const float (&w_row)[2], float (&dw_sum)[2]) __attribute__((always_inline)) {
          bf16x4 dg[4], du[4], a[4];
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const float gf = static_cast<float>(g[q][t]), uf = static_cast<float>(u[q][t]);
              float d = static_cast<float>(static_cast<bf16>(dacc.q[q][t]));
              const float sg = sigmoid_f32(gf);
              const float av = gf * sg * uf;
              if constexpr (FOLD) dw_sum[q >> 1] += d * av;      // masked G, U are zero: columns past N and rows past the segment add 0
              dg[q][t] = static_cast<bf16>(d * uf * sg * (1.0f + gf * (1.0f - sg)));
              du[q][t] = static_cast<bf16>(d * gf * sg);
              a[q][t] = static_cast<bf16>(FOLD ? w_row[q >> 1] * av : av);
            }
          bf16* drow = p.dH + (long)mb * 2 * p.N + nb;
          stage_store_bf16(stg, dg, drow, 2L * p.N, rows_valid, cols_valid, lane);
          stage_store_bf16(stg, du, drow + p.N, 2L * p.N, rows_valid, cols_valid, lane);
          stage_store_bf16(stg, a, p.A_out + (long)mb * p.N + nb, p.N, p.A_out ? rows_valid : 0, cols_valid, lane);   // no A_out: all lanes masked
        };
        // the four lanes with the same lane % 16 hold a row's columns.  Every row of the expert's segment gets exactly one
        // partial per (n-tile, wave along n); blocks past N contribute zero.
        auto row_weight = [&](int i, float (&w)[2]) __attribute__((always_inline)) {
          if constexpr (FOLD) {
#pragma unroll
            for (int h = 0; h < 2; ++h) w[h] = p.row_w[min(m0 + wm * WTM + i * 32 + patch_row(2 * h, lane), p.M - 1)];
          }
        };
        auto write_dw = [&](int i, const float (&dw_sum)[2]) __attribute__((always_inline)) {
          if constexpr (FOLD) {
            float tot[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              tot[h] = dw_sum[h] + __shfl_xor(dw_sum[h], 16);
              tot[h] += __shfl_xor(tot[h], 32);
            }
            const int mb = m0 + wm * WTM + i * 32;
            const __amdgpu_buffer_rsrc_t rs = block_rsrc(p.dw_part + (long)((n0 / BN) * WN + wn) * p.M + mb);
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, lane < 16 ? tot[0] : tot[1]), rs,
                                                  (lane < 32 && mb + lane < m_end) ? (unsigned)lane * 4u : BUF_OOB, 0, 0);
          }
        };
        float w_row[2] = {1.0f, 1.0f}, dw_sum[2] = {0.f, 0.f};
        {
          // The G and U reads of block b+1 are issued as soon as block b has been unpacked from the fetch registers,
          // so they are in flight while block b is computed and stored (one set of fetch registers: a second set
          // makes the compiler spill the loaders' tile offsets and reload them inside the k loop).
          constexpr int NB = TM * TN;
          auto block_geom = [&](int b, int& mb, int& nb, int& rows_valid, int& cols_valid) __attribute__((always_inline)) {
            const int i = b / TN, j = b % TN;
            mb = m0 + wm * WTM + i * 32;
            nb = n0 + wn * WTN + j * 32;
            rows_valid = m_end - mb;
            cols_valid = p.N - nb;
          };
          auto fetch_block = [&](int b, StageFetch& fg, StageFetch& fu) __attribute__((always_inline)) {
            int mb, nb, rows_valid, cols_valid;
            block_geom(b, mb, nb, rows_valid, cols_valid);
            const bf16* hrow = p.H + (long)mb * 2 * p.N + nb;
            fg = stage_fetch_bf16(hrow, 2L * p.N, rows_valid, cols_valid, lane);
            fu = stage_fetch_bf16(hrow + p.N, 2L * p.N, rows_valid, cols_valid, lane);
          };
          // Every block runs whether or not it has valid rows or columns (the masks live in the buffer offsets): a
          // uniform skip of single blocks would again make the number of stores in flight unknown to the compiler.
          // A wave without any valid row skips all of it.
          StageFetch fg = fg_first, fu = fu_first;
          if (m0 + wm * WTM < m_end)
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            if (b % TN == 0) { row_weight(b / TN, w_row); dw_sum[0] = dw_sum[1] = 0.f; }
            int mb, nb, rows_valid, cols_valid;
            block_geom(b, mb, nb, rows_valid, cols_valid);
            bf16x4 g[4], u[4];
            stage_unpack_bf16(stg, fg, g, lane);
            stage_unpack_bf16(stg, fu, u, lane);
            if (b + 1 < NB) fetch_block(b + 1, fg, fu);
            __builtin_amdgcn_sched_barrier(0);      // the read-ahead stays ahead of this block's arithmetic and stores
            swiglu_bwd_block(block(b / TN, b % TN), g, u, mb, nb, rows_valid, cols_valid, w_row, dw_sum);
            if (b % TN == TN - 1) write_dw(b / TN, dw_sum);
          }
          // Every wave leaves this epilogue with none of its vector memory operations in flight.  The first step of
          // the next tile would wait for them anyway (more stores than vmcnt can name), so this costs nothing; but
          // it has to be said here, once, on a path every wave takes.  The k loop has a path without any vmcnt wait
          // (the touching wave's), and when the compiler cannot rule out that the read-ahead loads of G and U above
          // are still writing their registers on that path, it guards the registers where they are reused: if the
          // allocation gives them to the fragments, that is a vmcnt wait in front of the fragment reads of every step
          // on every wave, which there also waits for the tile loads issued a moment before (seen: dgrad2 +20 % after
          // a change to the epilogue's arithmetic that moved the allocation).
          wait_vmcnt<0>();
        }
      }
    }
    if (!has_next) break;
  }
}

}  // namespace mfma
}  // namespace moe
