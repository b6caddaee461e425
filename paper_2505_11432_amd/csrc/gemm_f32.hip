// Grouped GEMM on fp32 data with the fp32 matrix instruction (v_mfma_f32_32x32x2_f32), for operands whose rows or columns
// can be read in whole 16-byte pieces: the expert products (widths are multiples of 16, buffers 16-byte aligned) and
// router logits of such rows.  Expert products of 192 and more 64 x 64 tiles are faster on the bf16 instructions
// (gemm_f32_split.hip); here stay the router, small problems, weight gradients of few rows per expert and very wide rows.
//
// Bound: the fp32 matrix rate, 256 FLOP per clock and CU, twice what unpacked fp32 FMAs give.  One instruction takes 64
// clocks for 4 KFLOP, so the operands are cheap to feed and small tiles are affordable; what matters is that loads are
// in flight early and that the tile count fills 256 CUs.  Three shapes of four waves, 32 x 32 outputs per wave; where
// waves share outputs each takes its part of every k-step and the sums are added through LDS at the end:
//   64 x 64, k-steps of 32;  64 x 32, two waves per output, k-steps of 32;  32 x 32, four per output, k-steps of 64.
// All keep two k-steps of global loads in registers ahead of the LDS stage that is being multiplied; several workgroups
// share a CU and hide each other's latency.
// A small layer (256 tokens, d = 128, f = 256, 8 experts) is launches, not arithmetic: its backward's last three products share one (80.8 ->
// 71.0 us, forward and backward), and the SwiGLU passes go into the products beside them (71.0 -> 65.2).
// Measured (a vector-ALU kernel of 64 x 64 x 16 first): router logits of 1000 tokens 182 -> 13 us.
#include "gemm_f32_tiles.h"

namespace moe {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;

// LDS image of one operand tile of EXT rows (or columns) x BK.  K-fast: [ext][BK + 4], a lane reads four consecutive k with
// one b128 (16 lanes then cover the 64 banks once).  MN-fast: [BK][EXT + 8], a lane reads its row at one k with a b32;
// the two lane halves read k rows four apart, 4 * (EXT + 8) = 32 mod 64 banks apart.
template <bool KFAST, int EXT, int BK> struct Tile {
  static constexpr int LD = KFAST ? BK + 4 : EXT + 8;
  static constexpr int FLOATS = (KFAST ? EXT : BK) * LD;
  static constexpr int VECS = EXT * BK / 4 / kThreads;      // 16-byte pieces per thread and k-step
  static constexpr int PER_ROW = (KFAST ? BK : EXT) / 4;
  static_assert(EXT * BK % (4 * kThreads) == 0, "a k-step splits evenly over the threads");
  // piece v of this thread: row and column (elements) inside the stored tile
  __device__ static __forceinline__ int row(int v) { return (v * kThreads + (int)threadIdx.x) / PER_ROW; }
  __device__ static __forceinline__ int col(int v) { return (v * kThreads + (int)threadIdx.x) % PER_ROW * 4; }
};

// Operand piece -> registers.  ext0 / ext_n: first row (column) of the tile and the number of valid ones; k is absolute,
// k_end its end.  Rows past the end repeat the last valid one (they only reach outputs that are not stored); pieces past
// the end of the contraction are zero.
template <bool KFAST, int EXT, int BK>
__device__ __forceinline__ void fetch(const float* __restrict__ base, long ld, int ext0, int ext_n, int k, int k_end,
                                      f32x4 (&out)[Tile<KFAST, EXT, BK>::VECS]) {
  using TL = Tile<KFAST, EXT, BK>;
#pragma unroll
  for (int v = 0; v < TL::VECS; ++v) {
    const int r = TL::row(v), c = TL::col(v);
    const int kk = k + (KFAST ? c : r);
    const int x = KFAST ? min(r, ext_n - 1) : min(c, ext_n - 4);
    const float* p = base + (KFAST ? (long)(ext0 + x) * ld + kk : (long)kk * ld + ext0 + x);
    f32x4 t = {0.f, 0.f, 0.f, 0.f};
    if (kk < k_end) t = *reinterpret_cast<const f32x4*>(p);
    out[v] = t;
  }
}
template <bool KFAST, int EXT, int BK>
__device__ __forceinline__ void stash(float* lds, const f32x4 (&in)[Tile<KFAST, EXT, BK>::VECS]) {
  using TL = Tile<KFAST, EXT, BK>;
#pragma unroll
  for (int v = 0; v < TL::VECS; ++v) *reinterpret_cast<f32x4*>(lds + TL::row(v) * TL::LD + TL::col(v)) = in[v];
}
// The four k values 4 * (lane / 32) + 0..3 of an 8-deep group, for tile row x.
template <bool KFAST, int EXT, int BK>
__device__ __forceinline__ f32x4 frag(const float* lds, int x, int k8, int half) {
  using TL = Tile<KFAST, EXT, BK>;
  if constexpr (KFAST) {
    return *reinterpret_cast<const f32x4*>(lds + x * TL::LD + k8 + 4 * half);
  } else {
    f32x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = lds[(k8 + 4 * half + j) * TL::LD + x];
    return r;
  }
}

// Floats of LDS of a workgroup: two stages
template <int BM, int BN, int BK, bool AK, bool BKF> constexpr int kLdsFloats = 2 * (Tile<AK, BM, BK>::FLOATS + Tile<BKF, BN, BK>::FLOATS);

// What a small layer's products take over from the SwiGLU passes: FC2 makes its A operand from H = [G|U] on the way to LDS; dgrad2 turns the dA
// it has summed into dH and, where A_out is given, the SwiGLU output.
enum Fuse { PLAIN, FROM_H, TO_DH };
struct SwigluArgs { const float* H; float* dH; float* A_out; };

// The tile of workgroup `block` of `blocks`
template <int BM, int BN, int BK, int WM, int WN, int WK, bool AK, bool BKF, Fuse FUSE = PLAIN>
__device__ __forceinline__ void gemm_f32_tile(const GemmProblem& p, int tiles_n, int tiles_m_fixed, int block, int blocks, float* lds_floats,
                                              const SwigluArgs& sw = SwigluArgs{}) {
  static_assert(WM * WN * WK == 4 && BM == 32 * WM && BN == 32 * WN && BK % (8 * WK) == 0, "four waves of 32 x 32");
  using TA = Tile<AK, BM, BK>;
  using TB = Tile<BKF, BN, BK>;
  constexpr int STAGE = TA::FLOATS + TB::FLOATS;
  static_assert(2 * STAGE >= (WK - 1) * WM * WN * 32 * 32, "the sums that change waves fit");

  F32Tile t;
  if (!f32_tile<BM, BN>(p, tiles_n, tiles_m_fixed, block, blocks, t)) return;
  const int e = t.e, m0 = t.m0, m_end = t.m_end, n0 = t.n0, k0 = t.k0, k_end = t.k_end;
  const float* __restrict__ A = static_cast<const float*>(p.A);
  const float* __restrict__ B = static_cast<const float*>(p.B) + (long)e * p.b_es;
  const long lda = AK ? p.a_rs : p.a_cs, ldb = BKF ? p.b_cs : p.b_rs;

  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave % WK, wm = wave / WK % WM, wn = wave / WK / WM;
  const int row = wm * 32 + (lane & 31), colr = wn * 32 + (lane & 31);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;

  f32x4 ra[2][TA::VECS], rb[2][TB::VECS];
  f32x4 up_in[2][FUSE == FROM_H ? TA::VECS : 1];         // U beside the G in ra
  auto load = [&](int set, int k) __attribute__((always_inline)) {
    fetch<AK, BM, BK>(A, lda, m0, m_end - m0, k, k_end, ra[set]);
    if constexpr (FUSE == FROM_H) fetch<AK, BM, BK>(A + p.K, lda, m0, m_end - m0, k, k_end, up_in[set]);
    fetch<BKF, BN, BK>(B, ldb, n0, p.N - n0, k, k_end, rb[set]);
  };
  auto put = [&](int set, int buf) __attribute__((always_inline)) {
    if constexpr (FUSE == FROM_H)
#pragma unroll
      for (int v = 0; v < TA::VECS; ++v)
#pragma unroll
        for (int j = 0; j < 4; ++j) ra[set][v][j] = ra[set][v][j] * sigmoid_f32(ra[set][v][j]) * up_in[set][v][j];
    stash<AK, BM, BK>(lds_floats + buf * STAGE, ra[set]);
    stash<BKF, BN, BK>(lds_floats + buf * STAGE + TA::FLOATS, rb[set]);
  };
  auto multiply = [&](int buf) __attribute__((always_inline)) {
    const float* at = lds_floats + buf * STAGE;
    const float* bt = at + TA::FLOATS;
#pragma unroll
    for (int g = 0; g < BK / 8 / WK; ++g) {
      const int k8 = (wk * (BK / 8 / WK) + g) * 8;
      const f32x4 a = frag<AK, BM, BK>(at, row, k8, half);
      const f32x4 b = frag<BKF, BN, BK>(bt, colr, k8, half);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b[j], acc, 0, 0, 0);
    }
  };
  // step s sits in LDS buffer s & 1; the registers hold steps s + 1 and s + 2 while step s is multiplied.  A buffer is
  // overwritten one barrier after its last read.
  const int steps = (k_end - k0 + BK - 1) / BK;
  if (steps > 0) {
    load(0, k0);
    if (steps > 1) load(1, k0 + BK);
    put(0, 0);
    if (steps > 2) load(0, k0 + 2 * BK);
    __syncthreads();
    for (int s = 0; s < steps; s += 2) {
      multiply(0);
      if (s + 1 < steps) put(1, 1);
      if (s + 3 < steps) load(1, k0 + (s + 3) * BK);
      __syncthreads();
      if (s + 1 >= steps) break;
      multiply(1);
      if (s + 2 < steps) put(0, 0);
      if (s + 4 < steps) load(0, k0 + (s + 4) * BK);
      __syncthreads();
    }
  }
  if constexpr (FUSE == TO_DH) {
    // every wave takes a quarter of the rows (a lane's values r = 4 * wk + i), summed in the order of the waves
    static_assert(BM == 32 && BN == 32 && WK == 4, "one output of 32 x 32");
    static_assert(2 * STAGE >= 4 * 1024, "the sums of all waves fit");
    const int n = n0 + (lane & 31), f = p.N, mb = m0 + wk * 8 + half * 4;
    float gate[4], up[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* h = sw.H + (long)min(mb + i, m_end - 1) * 2 * f + min(n, f - 1);
      gate[i] = h[0];
      up[i] = h[f];
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) lds_floats[(wk * 16 + r) * 64 + lane] = acc[r];
    __syncthreads();
    if (n >= f) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (mb + i >= m_end) continue;
      float d = lds_floats[(wk * 4 + i) * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; ++w) d += lds_floats[(w * 16 + wk * 4 + i) * 64 + lane];
      const float g = gate[i], u = up[i], s = sigmoid_f32(g);
      float* dh = sw.dH + (long)(mb + i) * 2 * f + n;
      dh[0] = d * u * s * (1.0f + g * (1.0f - s));
      dh[f] = d * g * s;
      if (sw.A_out) sw.A_out[(long)(mb + i) * f + n] = g * s * u;
    }
    return;
  }
  if constexpr (WK > 1) {
    // (the loop ended with a barrier, or never started) the other waves of an output hand their sums to its first one,
    // which adds them in wave order
    float* part = lds_floats + (wm * WN + wn) * (WK - 1) * 1024;
    if (wk > 0)
#pragma unroll
      for (int r = 0; r < 16; ++r) part[((wk - 1) * 16 + r) * 64 + lane] = acc[r];
    __syncthreads();
    if (wk > 0) return;
#pragma unroll
    for (int w = 0; w < WK - 1; ++w)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] += part[(w * 16 + r) * 64 + lane];
  }
  // a lane holds column lane % 32 and rows 8q + 4 * (lane / 32) + 0..3: a store writes two rows of 128 bytes
  float* __restrict__ C = static_cast<float*>(p.C) + (long)e * p.c_es;
  const int n = n0 + colr;
  if (n >= p.N) return;
  const float bias = p.bias ? p.bias[n] : 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int m = m0 + wm * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
    if (m >= m_end) continue;
    float* dst = C + (long)m * p.ldc + n;
    float v = acc[r] + bias;
    if (p.accumulate) v += *dst;
    *dst = v;
  }
}

template <int BM, int BN, int BK, int WM, int WN, int WK, bool AK, bool BKF>
__global__ void __launch_bounds__(kThreads) gemm_f32_kernel(GemmProblem p, int tiles_n, int tiles_m_fixed, int blocks) {
  __shared__ __attribute__((aligned(16))) float lds[kLdsFloats<BM, BN, BK, AK, BKF>];
  gemm_f32_tile<BM, BN, BK, WM, WN, WK, AK, BKF>(p, tiles_n, tiles_m_fixed, blockIdx.x, blocks, lds);
}

constexpr int kSmall = 32, kSmallK = 64;
template <bool BKF, Fuse FUSE>
__global__ void __launch_bounds__(kThreads) gemm_f32_swiglu_kernel(GemmProblem p, int tiles_n, int blocks, SwigluArgs sw) {
  __shared__ __attribute__((aligned(16))) float lds[kLdsFloats<kSmall, kSmall, kSmallK, true, BKF>];
  gemm_f32_tile<kSmall, kSmall, kSmallK, 1, 1, 4, true, BKF, FUSE>(p, tiles_n, 0, blockIdx.x, blocks, lds, sw);
}

// The three products at the end of a backward, d_w2, d_xp and d_w1, in one launch where each is small: none needs another, and alone each leaves
// most of the chip idle behind a chain of dependent loads.
struct SmallTrio { GemmProblem p[3]; int tiles_n[3], tiles_m[3], blocks[3]; };
__global__ void __launch_bounds__(kThreads) gemm_f32_trio_kernel(SmallTrio t) {
  constexpr int kWgrad = kLdsFloats<kSmall, kSmall, kSmallK, false, false>, kDgrad = kLdsFloats<kSmall, kSmall, kSmallK, true, false>;
  __shared__ __attribute__((aligned(16))) float lds[kWgrad > kDgrad ? kWgrad : kDgrad];
  int b = blockIdx.x;
  if (b < t.blocks[0]) {
    gemm_f32_tile<kSmall, kSmall, kSmallK, 1, 1, 4, false, false>(t.p[0], t.tiles_n[0], t.tiles_m[0], b, t.blocks[0], lds);
    return;
  }
  b -= t.blocks[0];
  if (b < t.blocks[1]) {
    gemm_f32_tile<kSmall, kSmall, kSmallK, 1, 1, 4, true, false>(t.p[1], t.tiles_n[1], t.tiles_m[1], b, t.blocks[1], lds);
    return;
  }
  gemm_f32_tile<kSmall, kSmall, kSmallK, 1, 1, 4, false, false>(t.p[2], t.tiles_n[2], t.tiles_m[2], b - t.blocks[1], t.blocks[2], lds);
}

template <int BM, int BN, int BK, int WM, int WN, int WK>
int launch(const GemmProblem& p, bool a_kfast, bool b_kfast, hipStream_t s) {
  const int tiles_n = cdiv(p.N, BN), tiles_m_fixed = cdiv(p.M, BM);
  const long blocks = f32_blocks(p, BM, BN);
  if (blocks > 0x7fffffffL) return MOE_ERR_UNSUPPORTED;
  const dim3 grid((unsigned)blocks), block(kThreads);
  if (a_kfast && b_kfast) gemm_f32_kernel<BM, BN, BK, WM, WN, WK, true, true><<<grid, block, 0, s>>>(p, tiles_n, tiles_m_fixed, (int)blocks);
  else if (a_kfast) gemm_f32_kernel<BM, BN, BK, WM, WN, WK, true, false><<<grid, block, 0, s>>>(p, tiles_n, tiles_m_fixed, (int)blocks);
  else gemm_f32_kernel<BM, BN, BK, WM, WN, WK, false, false><<<grid, block, 0, s>>>(p, tiles_n, tiles_m_fixed, (int)blocks);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

}  // namespace

// True when the operands can be read in whole 16-byte pieces along their fast dimension.
bool gemm_f32_covers(const GemmProblem& p) {
  const bool a_kfast = p.a_cs == 1, b_kfast = p.b_rs == 1;
  if (!aligned16(p.A) || !aligned16(p.B) || p.N <= 0 || p.M <= 0) return false;
  if (!a_kfast && (p.a_rs != 1 || b_kfast)) return false;
  if (!b_kfast && p.b_cs != 1) return false;
  if ((a_kfast ? p.a_rs : p.a_cs) % 4 || (b_kfast ? p.b_cs : p.b_rs) % 4 || p.b_es % 4) return false;
  if (!a_kfast && p.M % 4) return false;
  if (!b_kfast && p.N % 4) return false;
  // a piece that lies along k must not straddle the end of the contraction: K a multiple of 4, segments of any length no
  if ((a_kfast || b_kfast) && (p.mode == 1 || p.K % 4)) return false;
  return true;
}

// Which shape: smaller tiles read more per FLOP but spread a problem over more workgroups and shorten its serial chain of
// k-steps.  Fewer 64 x 64 tiles than CUs: 32 x 32 (512 rows of 8 experts, N = 512, K = 1408: 21 us against 26 with 64 x 32 and 36 with
// 64 x 64; router logits of 4000 tokens, 64 experts, d = 1024 14.5, 19.6, 25.8; of 15000 29.6, 29.9, 29.1).  Beyond that come router
// logits (20000 tokens 38.7, 37.6, 41.9; 66000 111, 99, 98; 120000 201, 180, 168) and weight gradients of up to 32 rows per expert (8
// experts, 20 rows, 256 x 512 6.9, 5.8, 4.5; 4 experts, 7 rows, 1024 x 1024 21.4, 12.5, 8.7; 8 experts, 25 rows, 512 x 1408 29, 16, 11): 64 x 32 for
// the logits and up to four 64 x 64 tiles per CU, where two waves share an output and each sums half as long a chain (the average
// segment is short, the longest may not be), 64 x 64 for longer lists of weight gradients and for what a launch of 64 x 32 could not hold
// (less than 2^32 threads).  Other expert products of so many tiles come only with rows of 2^20 elements and at the limit of a launch.
static long tiles64(const GemmProblem& p) {
  const long tiles_m = (long)cdiv(p.M, 64) + (p.mode == 0 ? p.E / 2 : 0);      // segments end inside a tile
  return (long)cdiv(p.N, 64) * tiles_m * (p.mode == 1 ? p.E : 1);
}
int launch_gemm_f32(const GemmProblem& p, hipStream_t s) {
  if (p.M <= 0 || p.N <= 0) return MOE_OK;
  if (gemm_f32_splits(p)) return launch_gemm_f32_split(p, s);
  const bool a_kfast = p.a_cs == 1, b_kfast = p.b_rs == 1;
  const long tiles = tiles64(p);
  if (tiles < 256) return launch<32, 32, 64, 1, 1, 4>(p, a_kfast, b_kfast, s);
  const long narrow = (long)cdiv(p.N, 32) * (cdiv(p.M, 64) + (p.mode == 0 ? (long)p.E : 0)) * (p.mode == 1 ? p.E : 1);      // 64 x 32 workgroups
  if (tiles < 1024 || (b_kfast && narrow * kThreads < 1L << 32)) return launch<64, 32, 32, 2, 1, 2>(p, a_kfast, b_kfast, s);
  return launch<64, 64, 32, 2, 2, 1>(p, a_kfast, b_kfast, s);
}

// True for a product that goes to 32 x 32 tiles.
static bool small(const GemmProblem& p) { return p.M > 0 && p.N > 0 && !gemm_f32_splits(p) && tiles64(p) < 256; }

// H -> yp: SwiGLU into A and FC2 (fc2, which reads A), or both in one launch of small tiles.  Every column of tiles makes A again, at 0.1 us per
// k-step of 64, which costs more than a launch where a CU has a long contraction or several tiles; and yp may be written over H, which a column
// of tiles must not do before the others have read it.  Whole forwards back to back, SwiGLU and FC2, one launch (us; 32 x 32 tiles on a CU times
// K): 256 16.0, 14.5; 17.1, 15.7; 336 24.0, 22.8; 512 19.2, 18.7; 22.7, 22.3; 20.6, 18.9; 640 22.8, 22.4; 768 22.5, 22.6; 1024 28.1, 28.8; 31.2, 31.9;
// 1280 28.3, 29.8; 1536 31.2, 34.1; 2000 40.2, 43.6.
int launch_gemm_f32_fc2(const GemmProblem& fc2, const void* H, void* A, hipStream_t s) {
  const long blocks32 = f32_blocks(fc2, kSmall, kSmall);
  if (small(fc2) && (blocks32 + 255) / 256 * fc2.K <= 640 && apart(H, 8 * (size_t)fc2.M * fc2.K, fc2.C, 4 * (size_t)fc2.M * fc2.ldc)) {
    GemmProblem p = fc2;
    p.A = H;
    p.a_rs = 2L * fc2.K;
    const int blocks = (int)blocks32;
    gemm_f32_swiglu_kernel<true, FROM_H><<<dim3((unsigned)blocks), dim3(kThreads), 0, s>>>(p, cdiv(p.N, kSmall), blocks, SwigluArgs{});
    MOE_LAUNCH_CHECK();
    return MOE_OK;
  }
  const int rc = launch_swiglu_fwd(H, A, fc2.M, fc2.K, fc2.offsets + fc2.E, MOE_F32, s);
  return rc != MOE_OK ? rc : launch_gemm_f32(fc2, s);
}
// d_yp -> dH and, unless A is NULL, the FC2 input again: dgrad2 (which writes dA) and SwiGLU', or both in one launch of small tiles.
int launch_gemm_f32_dgrad2(const GemmProblem& dgrad2, const void* H, void* dH, void* A, hipStream_t s) {
  if (small(dgrad2)) {
    const int blocks = (int)f32_blocks(dgrad2, kSmall, kSmall);
    gemm_f32_swiglu_kernel<false, TO_DH><<<dim3((unsigned)blocks), dim3(kThreads), 0, s>>>(
        dgrad2, cdiv(dgrad2.N, kSmall), blocks, SwigluArgs{static_cast<const float*>(H), static_cast<float*>(dH), static_cast<float*>(A)});
    MOE_LAUNCH_CHECK();
    return MOE_OK;
  }
  const int rc = launch_gemm_f32(dgrad2, s);
  return rc != MOE_OK ? rc : launch_swiglu_bwd(H, dgrad2.C, dH, A, dgrad2.M, dgrad2.N, dgrad2.offsets + dgrad2.E, MOE_F32, s);
}

// Whether `q` may run beside `p`: what it writes is neither read nor written by `p` (operands dense, rows or segments up to their bound).
static bool writes_apart(const GemmProblem& q, const GemmProblem& p) {
  auto c_floats = [](const GemmProblem& g) { return (size_t)(g.mode == 1 ? g.E * g.c_es : g.M * g.ldc); };
  const size_t a = (size_t)(p.mode == 1 ? p.K * p.a_cs : p.M * p.a_rs), b = (size_t)(p.mode == 1 ? p.K * p.b_rs : p.E * p.b_es);
  const size_t out = c_floats(q) * 4;
  return apart(q.C, out, p.A, a * 4) && apart(q.C, out, p.B, b * 4) && apart(q.C, out, p.C, c_floats(p) * 4);
}

// d_w2, d_xp and d_w1 of a backward: one launch where each would go to 32 x 32 tiles, else one by one in this order.  A caller may
// write d_xp over d_yp or a_override, or d_w1 over w1, which d_w2 and d_xp read before: those go one by one.
int launch_gemm_f32_trio(const GemmProblem& dw2, const GemmProblem& dxp, const GemmProblem& dw1, hipStream_t s) {
  const GemmProblem* p[3] = {&dw2, &dxp, &dw1};
  SmallTrio t{};
  long all = 0;
  bool joint = true;
  for (int i = 0; i < 3; ++i) {
    const bool a_kfast = p[i]->a_cs == 1, b_kfast = p[i]->b_rs == 1;
    joint = joint && small(*p[i]) && a_kfast == (i == 1) && !b_kfast;
    for (int j = 0; j < 3; ++j) joint = joint && (i == j || writes_apart(*p[i], *p[j]));
    const long blocks = f32_blocks(*p[i], kSmall, kSmall);
    t.p[i] = *p[i];
    t.tiles_n[i] = cdiv(p[i]->N, kSmall);
    t.tiles_m[i] = cdiv(p[i]->M, kSmall);
    t.blocks[i] = (int)blocks;
    all += blocks;
  }
  if (joint && all <= 0x7fffff) {
    gemm_f32_trio_kernel<<<dim3((unsigned)all), dim3(kThreads), 0, s>>>(t);
    MOE_LAUNCH_CHECK();
    return MOE_OK;
  }
  for (int i = 0; i < 3; ++i) {
    const int rc = launch_gemm_f32(*p[i], s);
    if (rc != MOE_OK) return rc;
  }
  return MOE_OK;
}

}  // namespace moe
