// Grouped GEMM on fp32 data with the bf16 matrix instructions: every operand element is the exact sum of three bf16 numbers.
//
// x = hi + mid + lo with hi = bf16(x), mid = bf16(x - hi) and lo = x - hi - mid: 24 significant bits in three times 8, nothing is lost.
// Of the nine products of two such sums the six largest are added; the three left out are together below 2^-24 of the product, of
// either sign and 2^-27 on average.  hi * hi has accumulators of its own, which round once per 32 products (the fp32 instruction once
// per 2), so the sums are closer to float64 than with it.  Error of a layer's results, forward and backward, fp32 instruction and this:
// 8 experts, 2000 rows, d = 1024, f = 2816 1.2e-6, 5.8e-7; 512 rows, d = 128, f = 256 2.8e-7, 2.0e-7 (with all sums in one accumulator
// 1.4e-6, 4.2e-7; parts cut off instead of rounded 6.0e-7, 2.8e-7).  (The splitting is that of Henry, Tang and Heinecke, "Leveraging the
// bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", 2019.)  It does not hold for sums of one term: kFewTerms.
// In a longer contraction that holds a single product other than zero, of two full 24-bit numbers, 4 % of the results are not the nearest
// number (up to 1.5 units of 2^-24 off instead of 1); products by powers of two and other numbers of up to 8 bits are exact.
//
// Bound: six bf16 products take 0.4 of the time of one fp32 product on the matrix cores, but two elements also cost thirteen vector
// instructions to scale and split, and the three parts pass through LDS.  Products, split and LDS take about as long each, and a SIMD issues
// either a matrix or a vector instruction; what they overlap comes back in part as a lower clock (2.0 GHz).
// Each operand element is split once per tile by the thread that loads it, so larger tiles split less often.  Measured (us, operands from
// memory; the fp32 instruction, then the split as it is now; 8 experts, 2000 rows, d = 1024, f = 2816): FC1 238, 218; FC2 137, 111; dgrad2 115, 106;
// wgrad2 117, 105; dgrad1 271, 189; wgrad1 229, 188.  128 x 128 tiles by eight waves of 32 x 64 with two stages in LDS, one workgroup per CU, on
// the same box: 229, 137, 121, 115, 286, 207 (4400 rows 353, 199, 205, 182, 423, 335, now 325, 199, 171, 166, 322, 305).  They stay for a single round (f32_split_in_eight).
// Not faster (FC1, 2000 rows, against 195): the two workgroups as one, taking turns by barriers (191, weight gradients 15 % slower); 32 x 32
// instructions with the split between their products, the parts written behind the barrier (200; loads of whole lines by four k per lane
// changed nothing); a higher wave priority while multiplying (180 to 225, dgrad1 15 % slower).  64 x 64 tiles: one wave per SIMD,
// fragments read ahead across the step barrier, products and split interleaved by scheduling barriers changed nothing or lost.
#include <atomic>

#include "gemm_f32_tiles.h"
#include "row_plan.h"

namespace moe {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

constexpr int kStep = kF32SplitStep;     // contraction per step
// Contractions of so few terms (weight gradients of one or two rows) are left to the fp32 instruction: the three products left out and
// the sum of two accumulators round more than it does on them.  Against float64 in units of 2^-24, the fp32 instruction and the split: one term
// rms 0.43, 0.44, largest 1.0, 1.56; two 0.52, 0.44, 1.88, 2.26; three 0.60, 0.44, 2.55, 2.36; four 0.66, 0.45, 2.86, 2.25; 1024 4.9, 3.1.
constexpr int kFewTerms = 2;
constexpr unsigned kSpan = 0x40000000u;  // bytes that a tile's rows span at most

// Elements are scaled by this on the way in and sums by its square on the way out, exactly: the parts of every element other than zero, the
// smallest subnormal number among them, are then normal numbers, and so is every part product that can reach a result other than zero.  What
// leaves the range at its other end (elements from 2^104 on, sums from 2^80 on, infinities and NaN) is seen in the sums.
// (Left as they are, elements below 2^-103 and sums below 2^-80 had to be found and their tiles made again: two vector instructions per element
// instead of one, and FC1 as above 488 us instead of 184 with one such element per tile, as gates below -72 give.)
constexpr float kScale = 0x1p24f, kUnscale = 0x1p-48f;

// LDS image of one part of one operand tile: EXT rows (or columns) of 32 bf16, 64 bytes.  A 16-byte read serves lanes 0-3, 12-15, 20-27 and
// 4-11, 16-19, 28-31 together, so quads of rows meet others at the neighbouring chunk: quad q of 16 rows is turned by 0, 2, 3, 1 (by q
// itself, reads took twice as long: FC1 as above 203 -> 184 us).
template <int EXT> struct Part {
  static constexpr int BYTES = EXT * 64;
  __device__ static __forceinline__ int offset(int row, int chunk) {
    const int q = (row >> 2) & 3;
    return (row << 6) + ((chunk ^ (((q << 1) ^ (q & 2) ^ (q >> 1)) & 3)) << 4);
  }
};

// This thread's share of an operand tile: eight consecutive k of one row.  Loads are raw buffer instructions on a descriptor at the tile's
// origin at the step's k, which moves on by scalar arithmetic; what lies past the end of the contraction is out of the
// descriptor's range and reads as zero.
template <bool KFAST, int EXT> struct Share {
  __device__ static __forceinline__ int row() { return KFAST ? threadIdx.x >> 2 : threadIdx.x % EXT; }
  __device__ static __forceinline__ int chunk() { return KFAST ? threadIdx.x & 3 : threadIdx.x / EXT; }

  const char* base;             // row (column) ext0 at the first k
  long step;                    // bytes per step
  int ld4, left0;               // bytes from one row of the buffer to the next; across k: bytes of a row in front of the tile
  unsigned off[KFAST ? 1 : 8];

  // ext_n: valid rows of the tile; rows past them repeat the last one (they only reach outputs that are not stored)
  __device__ __forceinline__ void open(const float* p, long ld, int ext0, int ext_n, int k0) {
    ld4 = (int)ld * 4;
    left0 = ext0 * 4;
    step = KFAST ? kStep * 4 : (long)kStep * ld4;
    base = reinterpret_cast<const char*>(p + (KFAST ? (long)ext0 * ld + k0 : (long)k0 * ld + ext0));
    const unsigned r = min(row(), ext_n - 1);
    if constexpr (KFAST) {
      off[0] = r * (unsigned)ld4 + (unsigned)chunk() * 32u;
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) off[i] = (unsigned)(chunk() * 8 + i) * (unsigned)ld4 + r * 4u;
    }
  }
  // k_left: contraction left from step s on (not positive: nothing)
  __device__ __forceinline__ void load(float (&v)[8], int s, int k_left) const {
    const char* at = base + s * step;
    const int span = KFAST ? (int)kSpan : max(min(k_left, kStep) * ld4 - left0, 0);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(at), 0, span, 0x00020000);
    if constexpr (KFAST) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const unsigned o = chunk() * 8 + 4 * q < k_left ? off[0] + 16u * q : kSpan;
        const f32x4 t = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) v[4 * q + i] = t[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off[i], 0, 0));
    }
  }

  // The split in four units of two elements: unit u, whose parts gather in `part` and go to lds with the last one.
  __device__ static __forceinline__ void split(const float (&v)[8], int u, u32x4 (&part)[3], char* lds) {
    float r0 = v[2 * u] * kScale, r1 = v[2 * u + 1] * kScale;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const unsigned two = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{r0, r1}), bf16x2));
      part[p][u] = two;
      r0 -= __builtin_bit_cast(float, two << 16);
      r1 -= __builtin_bit_cast(float, two & 0xffff0000u);
    }
    if (u == 3)
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4*>(lds + p * Part<EXT>::BYTES + Part<EXT>::offset(row(), chunk())) = part[p];
  }

  // as fp32 rows of 32 k at a stride of 36
  __device__ static __forceinline__ void stash(const float (&v)[8], float* lds) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
      *reinterpret_cast<f32x4*>(lds + row() * 36 + chunk() * 8 + 4 * q) = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
  }
};

// Products of row segments may be cut along K (gridDim.y parts): the whole steps of this workgroup's part.
__device__ __forceinline__ void part_of_tile(F32Tile& t) {
  if (gridDim.y == 1) return;
  const int steps = (t.k_end - t.k0 + kStep - 1) / kStep, q = blockIdx.y, n = gridDim.y, k0 = t.k0;
  t.k0 = k0 + q * steps / n * kStep;
  t.k_end = min(t.k_end, k0 + (q + 1) * steps / n * kStep);
}

// WM x WN waves.  While the products of step s run from one LDS buffer the operands of step s + 1 are split into the other, and those of
// steps s + 2 and s + 3 are on their way into registers.
template <int BM, int BN, int WM, int WN, bool AK, bool BKF>
__global__ void __launch_bounds__(WM * WN * 64, 2) gemm_f32_split_kernel(GemmProblem p, int tiles_n, int tiles_m_fixed, int blocks) {
  constexpr int THREADS = WM * WN * 64, WTM = BM / WM, WTN = BN / WN, FM = WTM / 16, FN = WTN / 16;
  constexpr int A_BYTES = 3 * Part<BM>::BYTES, STAGE = A_BYTES + 3 * Part<BN>::BYTES;
  static_assert(BM * 4 == THREADS && BN * 4 == THREADS, "one chunk of each operand per thread");
  static_assert((BM + BN) * 36 * 4 <= STAGE, "the fp32 rows of a step fit");
  extern __shared__ __attribute__((aligned(16))) char lds[];        // two stages
  __shared__ int redo;
  F32Tile t;
  if (!f32_tile<BM, BN>(p, tiles_n, tiles_m_fixed, blockIdx.x, blocks, t)) return;
  part_of_tile(t);
  const int m0 = t.m0, m_end = t.m_end, n0 = t.n0, klen = t.k_end - t.k0;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int i16 = lane & 15, g = lane >> 4;

  Share<AK, BM> a;
  Share<BKF, BN> b;
  a.open(static_cast<const float*>(p.A), AK ? p.a_rs : p.a_cs, m0, m_end - m0, t.k0);
  b.open(static_cast<const float*>(p.B) + (long)t.e * p.b_es, BKF ? p.b_cs : p.b_rs, n0, p.N - n0, t.k0);
  float va[2][8], vb[2][8];
  auto load = [&](int set, int s) __attribute__((always_inline)) {
    a.load(va[set], s, klen - s * kStep);
    b.load(vb[set], s, klen - s * kStep);
  };
  constexpr int UNITS = 8;
  u32x4 part[3];
  auto split = [&](int set, int buf, int u) __attribute__((always_inline)) {
    if (u < 4) a.split(va[set], u, part, lds + buf * STAGE);
    else b.split(vb[set], u - 4, part, lds + buf * STAGE + A_BYTES);
  };
  f32x4 acc[FM][FN], low[FM][FN];        // the products of the first parts, the smaller ones
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = low[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // The products of a step, and between them the split of the next one.  Blocks of FM x 2 outputs go through the six terms together, so that
  // an accumulator is used again only after 2 * FM products.
  auto advance = [&](int buf, int set) __attribute__((always_inline)) {
    constexpr int PRODUCTS = 6 * FM * FN, EACH = PRODUCTS / UNITS;
    static_assert(PRODUCTS % UNITS == 0 && FN % 2 == 0, "every unit of the split gets as many products");
    constexpr int TB[6] = {2, 1, 0, 1, 0, 0}, TA[6] = {0, 1, 2, 0, 1, 0};        // parts of B and A, the smallest terms first
    const char* at = lds + buf * STAGE;
    bf16x8 fa[FM][3], fb[2][2][3];
    auto read_a = [&](int q) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
        fa[i][q] = *reinterpret_cast<const bf16x8*>(at + q * Part<BM>::BYTES + Part<BM>::offset(wm * WTM + i * 16 + i16, g));
    };
    auto read_b = [&](int jp, int q) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
        fb[jp & 1][j][q] =
            *reinterpret_cast<const bf16x8*>(at + A_BYTES + q * Part<BN>::BYTES + Part<BN>::offset(wn * WTN + (2 * jp + j) * 16 + i16, g));
    };
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      read_a(q);
      read_b(0, 2 - q);
    }
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
#pragma unroll
      for (int c = 0; c < EACH; ++c) {
        const int m = u * EACH + c, i = m % FM, j = m / FM % 2, term = m / (2 * FM) % 6, jp = m / (12 * FM);
        if (m % (12 * FM) == 0 && jp + 1 < FN / 2)
#pragma unroll
          for (int q = 0; q < 3; ++q) read_b(jp + 1, 2 - q);
        f32x4& sum = term == 5 ? acc[i][2 * jp + j] : low[i][2 * jp + j];
        sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[jp & 1][j][TB[term]], fa[i][TA[term]], sum, 0, 0, 0);
      }
      split(set, buf ^ 1, u);
    }
  };
  clear();
  const int steps = (klen + kStep - 1) / kStep;
  const bool few = klen <= kFewTerms;
  if (threadIdx.x == 0) redo = few;
  if (!few) {
    load(0, 0);
    load(1, 1);
#pragma unroll
    for (int u = 0; u < UNITS; ++u) split(0, 0, u);
    load(0, 2);
    __syncthreads();
    int s = 0;
    for (; s + 2 <= steps; s += 2) {
      advance(0, 1);
      load(1, s + 3);
      __syncthreads();
      advance(1, 0);
      load(0, s + 4);
      __syncthreads();
    }
    if (s < steps) advance(0, 1);
  }
  __syncthreads();
  // Parts or sums that overflowed (they give infinities or NaN in every output they reach): the tile is made again with the fp32 instruction.
  // With such an element in every tile FC1 as above takes 417 us, dgrad1 503 (488 and 557 with loads not ahead; gemm_f32.hip 252 and 268).
  bool bad = false;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float sum = acc[i][j][r] + low[i][j][r];
        bad |= (__builtin_bit_cast(unsigned, sum) & 0x7f800000u) == 0x7f800000u;
        acc[i][j][r] = sum * kUnscale;
      }
  if (bad) redo = 1;
  __syncthreads();
  if (redo) {
    // as the split: step s in one buffer, steps s + 1 and s + 2 on their way into registers
    clear();
    auto exact = [&](int set, int s) __attribute__((always_inline)) {
      float* at = reinterpret_cast<float*>(lds + set * STAGE);
      float* bt = at + BM * 36;
      a.stash(va[set], at);
      b.stash(vb[set], bt);
      load(set, s + 2);
      __syncthreads();
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const f32x4 fb = *reinterpret_cast<const f32x4*>(bt + (wn * WTN + j * 16 + i16) * 36 + h * 16 + g * 4);
#pragma unroll
          for (int i = 0; i < FM; ++i) {
            const f32x4 fa = *reinterpret_cast<const f32x4*>(at + (wm * WTM + i * 16 + i16) * 36 + h * 16 + g * 4);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[r], fa[r], acc[i][j], 0, 0, 0);
          }
        }
    };
    load(0, 0);
    load(1, 1);
    for (int s = 0; s < steps; s += 2) {
      exact(0, s);
      if (s + 1 < steps) exact(1, s + 1);
    }
  }
  // a lane holds row lane % 16 and columns 4 * (lane / 16) + 0..3 of every 16 x 16 block
  float* __restrict__ C = static_cast<float*>(p.C) + (long)t.e * p.c_es + (long)blockIdx.y * p.part_stride;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int m = m0 + wm * WTM + i * 16 + i16;
    if (m >= m_end) continue;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = n0 + wn * WTN + j * 16 + g * 4;
      if (n >= p.N) continue;
      f32x4* dst = reinterpret_cast<f32x4*>(C + (long)m * p.ldc + n);
      *dst = p.accumulate ? acc[i][j] + *dst : acc[i][j];
    }
  }
}

// The same with CH chunks of eight k per thread.
template <bool KFAST, int EXT, int THREADS> struct Shares {
  static constexpr int CH = EXT * 4 / THREADS;
  static_assert(EXT * 4 % THREADS == 0 && (KFAST || THREADS % EXT == 0), "whole chunks per thread");
  __device__ static __forceinline__ int row(int c) { return KFAST ? (threadIdx.x >> 2) + c * (THREADS / 4) : threadIdx.x % EXT; }
  __device__ static __forceinline__ int chunk(int c) { return KFAST ? threadIdx.x & 3 : threadIdx.x / EXT + c * (THREADS / EXT); }

  const char* base;             // row (column) ext0 at the first k
  long step;                    // bytes per step
  int ld4, left0;               // bytes from one row of the buffer to the next; across k: bytes of a row in front of the tile
  unsigned off[KFAST ? CH : 8];

  // ext_n: valid rows of the tile; rows past them repeat the last one (they only reach outputs that are not stored)
  __device__ __forceinline__ void open(const float* p, long ld, int ext0, int ext_n, int k0) {
    ld4 = (int)ld * 4;
    left0 = ext0 * 4;
    step = KFAST ? kStep * 4 : (long)kStep * ld4;
    base = reinterpret_cast<const char*>(p + (KFAST ? (long)ext0 * ld + k0 : (long)k0 * ld + ext0));
    if constexpr (KFAST) {
#pragma unroll
      for (int c = 0; c < CH; ++c) off[c] = (unsigned)min(row(c), ext_n - 1) * (unsigned)ld4 + (unsigned)chunk(c) * 32u;
    } else {
      const unsigned r = min(row(0), ext_n - 1);
#pragma unroll
      for (int i = 0; i < 8; ++i) off[i] = (unsigned)(chunk(0) * 8 + i) * (unsigned)ld4 + r * 4u;
    }
  }
  // k_left: contraction left from step s on (not positive: nothing)
  __device__ __forceinline__ void load(float (&v)[8], int c, int s, int k_left) const {
    const char* at = base + s * step;
    if constexpr (KFAST) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(at), 0, (int)kSpan, 0x00020000);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const unsigned o = chunk(c) * 8 + 4 * q < k_left ? off[c] + 16u * q : kSpan;
        const f32x4 t = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, o, 0, 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) v[4 * q + i] = t[i];
      }
    } else {
      const int k0 = c * (THREADS / EXT) * 8;        // chunks of one thread lie so far apart
      const int span = max(min(k_left - k0, kStep - k0) * ld4 - left0, 0);
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(at + (long)k0 * ld4), 0, span, 0x00020000);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off[i], 0, 0));
    }
  }

  // The split in four units of two elements: unit u, whose parts gather in `part` and go to lds with the last one.
  __device__ static __forceinline__ void split(const float (&v)[8], int c, int u, u32x4 (&part)[3], char* lds) {
    float r0 = v[2 * u] * kScale, r1 = v[2 * u + 1] * kScale;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const unsigned two = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{r0, r1}), bf16x2));
      part[p][u] = two;
      r0 -= __builtin_bit_cast(float, two << 16);
      r1 -= __builtin_bit_cast(float, two & 0xffff0000u);
    }
    if (u == 3)
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4*>(lds + p * Part<EXT>::BYTES + Part<EXT>::offset(row(c), chunk(c))) = part[p];
  }

  // as fp32 rows of 32 k at a stride of 36
  __device__ static __forceinline__ void stash(const float (&v)[8], int c, float* lds) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
      *reinterpret_cast<f32x4*>(lds + row(c) * 36 + chunk(c) * 8 + 4 * q) = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
  }
};

// 128 x 128 outputs by four waves of 64 x 64.  With one stage in LDS and 256 registers two workgroups share a CU, and while one splits and writes
// the other multiplies; a wave of 64 x 64 reads two thirds of what two of 64 x 32 read, and an element is split half as often as in tiles of
// 64 x 64.
template <bool AK, bool BKF>
__global__ void __launch_bounds__(256, 2) gemm_f32_split128_kernel(GemmProblem p, int tiles_n, int tiles_m_fixed, int blocks) {
  constexpr int BM = 128, BN = 128, WM = 2, WN = 2, THREADS = 256, WTM = BM / WM, WTN = BN / WN, FM = WTM / 16, FN = WTN / 16;
  constexpr int A_BYTES = 3 * Part<BM>::BYTES, STAGE = A_BYTES + 3 * Part<BN>::BYTES;
  typedef Shares<AK, BM, THREADS> ShareA;
  typedef Shares<BKF, BN, THREADS> ShareB;
  constexpr int CA = ShareA::CH, CB = ShareB::CH;
  static_assert((BM + BN) * 36 * 4 <= STAGE, "the fp32 rows of a step fit");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __shared__ int redo;
  F32Tile t;
  if (!f32_tile<BM, BN>(p, tiles_n, tiles_m_fixed, blockIdx.x, blocks, t)) return;
  part_of_tile(t);
  const int m0 = t.m0, m_end = t.m_end, n0 = t.n0, klen = t.k_end - t.k0;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int i16 = lane & 15, g = lane >> 4;

  ShareA a;
  ShareB b;
  a.open(static_cast<const float*>(p.A), AK ? p.a_rs : p.a_cs, m0, m_end - m0, t.k0);
  b.open(static_cast<const float*>(p.B) + (long)t.e * p.b_es, BKF ? p.b_cs : p.b_rs, n0, p.N - n0, t.k0);
  float va[CA][8], vb[CB][8];
  auto load_a = [&](int c, int s) __attribute__((always_inline)) { a.load(va[c], c, s, klen - s * kStep); };
  auto load_b = [&](int c, int s) __attribute__((always_inline)) { b.load(vb[c], c, s, klen - s * kStep); };
  auto load = [&](int s) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < CA; ++c) load_a(c, s);
#pragma unroll
    for (int c = 0; c < CB; ++c) load_b(c, s);
  };
  constexpr int UNITS = 4 * (CA + CB);
  u32x4 part[3];
  auto split = [&](int u) __attribute__((always_inline)) {
    if (u < 4 * CA) a.split(va[u / 4], u / 4, u % 4, part, lds);
    else b.split(vb[u / 4 - CA], u / 4 - CA, u % 4, part, lds + A_BYTES);
  };
  f32x4 acc[FM][FN], low[FM][FN];        // the products of the first parts, the smaller ones
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = low[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // The products of a step: column by column through the six terms, so that an accumulator is used again only after FM products.
  auto multiply = [&]() __attribute__((always_inline)) {
    constexpr int TB[6] = {2, 1, 0, 1, 0, 0}, TA[6] = {0, 1, 2, 0, 1, 0};        // parts of B and A, the smallest terms first
    bf16x8 fa[FM][3], fb[2][3];
    auto read_a = [&](int q) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
        fa[i][q] = *reinterpret_cast<const bf16x8*>(lds + q * Part<BM>::BYTES + Part<BM>::offset(wm * WTM + i * 16 + i16, g));
    };
    auto read_b = [&](int j, int q) __attribute__((always_inline)) {
      fb[j & 1][q] = *reinterpret_cast<const bf16x8*>(lds + A_BYTES + q * Part<BN>::BYTES + Part<BN>::offset(wn * WTN + j * 16 + i16, g));
    };
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      read_a(q);
      read_b(0, 2 - q);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      if (j + 1 < FN)
#pragma unroll
        for (int q = 0; q < 3; ++q) read_b(j + 1, 2 - q);
#pragma unroll
      for (int term = 0; term < 6; ++term)
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          f32x4& sum = term == 5 ? acc[i][j] : low[i][j];
          sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j & 1][TB[term]], fa[i][TA[term]], sum, 0, 0, 0);
        }
    }
  };
  clear();
  const int steps = (klen + kStep - 1) / kStep;
  const bool few = klen <= kFewTerms;
  if (threadIdx.x == 0) redo = few;
  if (!few) {
    load(0);
    for (int s = 0; s < steps; ++s) {
      // a chunk's registers take the next step's as soon as it is split
#pragma unroll
      for (int u = 0; u < UNITS; ++u) {
        split(u);
        if (u % 4 == 3) {
          if (u < 4 * CA) load_a(u / 4, s + 1);
          else load_b(u / 4 - CA, s + 1);
        }
      }
      __syncthreads();
      multiply();
      __syncthreads();
    }
  }
  __syncthreads();
  // as above: what overflowed is made again with the fp32 instruction
  bool bad = false;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float sum = acc[i][j][r] + low[i][j][r];
        bad |= (__builtin_bit_cast(unsigned, sum) & 0x7f800000u) == 0x7f800000u;
        acc[i][j][r] = sum * kUnscale;
      }
  if (bad) redo = 1;
  __syncthreads();
  if (redo) {
    clear();
    float* at = reinterpret_cast<float*>(lds);
    float* bt = at + BM * 36;
    load(0);
    for (int s = 0; s < steps; ++s) {
#pragma unroll
      for (int c = 0; c < CA; ++c) a.stash(va[c], c, at);
#pragma unroll
      for (int c = 0; c < CB; ++c) b.stash(vb[c], c, bt);
      load(s + 1);
      __syncthreads();
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const f32x4 fb = *reinterpret_cast<const f32x4*>(bt + (wn * WTN + j * 16 + i16) * 36 + h * 16 + g * 4);
#pragma unroll
          for (int i = 0; i < FM; ++i) {
            const f32x4 fa = *reinterpret_cast<const f32x4*>(at + (wm * WTM + i * 16 + i16) * 36 + h * 16 + g * 4);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[r], fa[r], acc[i][j], 0, 0, 0);
          }
        }
      __syncthreads();
    }
  }
  // a lane holds row lane % 16 and columns 4 * (lane / 16) + 0..3 of every 16 x 16 block
  float* __restrict__ C = static_cast<float*>(p.C) + (long)t.e * p.c_es + (long)blockIdx.y * p.part_stride;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int m = m0 + wm * WTM + i * 16 + i16;
    if (m >= m_end) continue;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = n0 + wn * WTN + j * 16 + g * 4;
      if (n >= p.N) continue;
      f32x4* dst = reinterpret_cast<f32x4*>(C + (long)m * p.ldc + n);
      *dst = p.accumulate ? acc[i][j] + *dst : acc[i][j];
    }
  }
}

// C = the sum of the K parts of a product, in their order; rows outside the segments are left as they are
__global__ void __launch_bounds__(256) f32_add_parts_kernel(const float* __restrict__ parts, long stride, int n, const int32_t* __restrict__ offsets,
                                                            int E, int M, int N, float* __restrict__ C, long ldc) {
  const int per_row = N / 4, first = offsets[0], rows = min(offsets[E], M) - first;
  const long total = (long)rows * per_row;
  for (long i = blockIdx.x * 256L + threadIdx.x; i < total; i += gridDim.x * 256L) {
    const long r = first + i / per_row;
    const int c = (int)(i % per_row) * 4;
    const float* src = parts + r * N + c;
    f32x4 sum = *reinterpret_cast<const f32x4*>(src);
    for (int q = 1; q < n; ++q) sum += *reinterpret_cast<const f32x4*>(src + q * stride);
    *reinterpret_cast<f32x4*>(C + r * ldc + c) = sum;
  }
}

constexpr int kLds = 12 * Part<64>::BYTES, kLdsEight = 12 * Part<128>::BYTES;      // two stages
static_assert(kLds == 6 * Part<128>::BYTES, "one stage of 128 x 128");

template <bool AK, bool BKF> int launch_as(const GemmProblem& p, F32Plan plan, hipStream_t s) {
  const int b = plan.tile == F32_64 ? 64 : 128;
  const int blocks = (int)f32_blocks(p, b, b), tiles_n = cdiv(p.N, b), tiles_m = cdiv(p.M, b);
  const dim3 grid((unsigned)blocks, (unsigned)plan.parts);
  if (plan.tile == F32_128_EIGHT) gemm_f32_split_kernel<128, 128, 4, 2, AK, BKF><<<grid, dim3(512), kLdsEight, s>>>(p, tiles_n, tiles_m, blocks);
  else if (plan.tile == F32_128) gemm_f32_split128_kernel<AK, BKF><<<grid, dim3(256), kLds, s>>>(p, tiles_n, tiles_m, blocks);
  else gemm_f32_split_kernel<64, 64, 2, 2, AK, BKF><<<grid, dim3(256), kLds, s>>>(p, tiles_n, tiles_m, blocks);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}
int launch(const GemmProblem& p, F32Plan plan, hipStream_t s) {
  const bool a_kfast = p.a_cs == 1, b_kfast = p.b_rs == 1;
  if (a_kfast && b_kfast) return launch_as<true, true>(p, plan, s);
  return a_kfast ? launch_as<true, false>(p, plan, s) : launch_as<false, false>(p, plan, s);
}

}  // namespace

// Operands that the kernel can take, where it is the faster way.
bool gemm_f32_splits(const GemmProblem& p) {
  if (p.mode == 2 || p.bias || !aligned16(p.C) || p.N % 4 || p.ldc % 4 || p.c_es % 4) return false;
  const long lda = p.a_cs == 1 ? p.a_rs : p.a_cs, ldb = p.b_rs == 1 ? p.b_cs : p.b_rs;
  if (lda >= 1 << 20 || ldb >= 1 << 20) return false;                   // 128 rows of a tile span less than kSpan
  if (f32_blocks(p, 64, 64) * 256 >= 1L << 31) return false;            // a launch holds less than 2^32 threads
  return f32_split_pays({p.mode == 0, p.M, p.N, p.K, p.E});
}

int launch_gemm_f32_split(const GemmProblem& p, hipStream_t s) {
  const size_t one = (size_t)p.M * p.N;
  const F32Plan plan = f32_plan({p.mode == 0, p.M, p.N, p.K, p.E}, p.scratch && !p.accumulate ? (long)(p.scratch_floats / one) : 0);
  if (plan.tile == F32_128_EIGHT)
    if (const int rc = gemm_f32_split_configure()) return rc;
  GemmProblem q = p;
  if (plan.parts > 1) {
    q.C = p.scratch; q.ldc = p.N; q.part_stride = (long)one;
  }
  const int rc = launch(q, plan, s);
  if (rc != MOE_OK || plan.parts == 1) return rc;
  const long quads = (long)(one / 4);
  f32_add_parts_kernel<<<dim3((unsigned)(quads < 256 * 2048 ? (quads + 255) / 256 : 2048)), dim3(256), 0, s>>>(
      p.scratch, q.part_stride, plan.parts, p.offsets, p.E, p.M, p.N, static_cast<float*>(p.C), p.ldc);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

// The tiles of eight waves need their dynamic-LDS limit raised once per device; moe_init does it ahead of a graph capture.  The
// values are the same on every call, the bit only saves work.
int gemm_f32_split_configure() {
  static std::atomic<unsigned long long> done{0};
  int dev = 0;
  MOE_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return MOE_ERR_UNSUPPORTED;
  if (done.load(std::memory_order_acquire) >> dev & 1) return MOE_OK;
  for (const void* k : {(const void*)gemm_f32_split_kernel<128, 128, 4, 2, true, true>, (const void*)gemm_f32_split_kernel<128, 128, 4, 2, true, false>,
                        (const void*)gemm_f32_split_kernel<128, 128, 4, 2, false, false>})
    MOE_HIP_TRY(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsEight));
  done.fetch_or(1ull << dev, std::memory_order_release);
  return MOE_OK;
}

}  // namespace moe
