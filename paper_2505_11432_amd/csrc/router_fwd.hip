// Router matmul when the chip is not filled by it: logits[T,E] = x[T,d] * w_r[E,d]^T (+ bias) on bf16 data, fp32 result.
//
// Bound: the latency of a serial walk over d, and with more tokens the reading of x.  So no LDS ring and no long k loop: a
// workgroup owns 16 tokens x 16 experts, its eight waves take every eighth 64-column block of the rows straight from
// global memory into 16x16x32 MFMA operands (16 loads in flight per lane), and their fp32 sums meet in LDS in wave order,
// which also rounds less than one long chain.
// Measured against the direct-to-LDS GEMM with 64-token tiles (us): T = 16, d = 4096, E = 8: 19.5 -> 7.9; T = 1, d = 4096,
// E = 64: 25.2 -> 6.8; T = 257, d = 2048, E = 64: 19.3 -> 6.5; T = 4096, d = 4096, E = 16: 21.8 -> 11.2; T = 8192,
// d = 4096, E = 8: 22.9 -> 19.1.  Beyond 512 tiles x is read once per 16 experts too often, or the deeper ring streams it
// faster (T = 65536, E = 8: 112 against 122; T = 16384, E = 64: 26 against 69): the GEMM keeps those.
#include "gemm_mfma.h"

namespace moe {
namespace {

using namespace mfma;
constexpr int kWaves = 8, kBlock = 64, kAhead = 4;      // kAhead: 64-column blocks a wave loads before it multiplies

__global__ void __launch_bounds__(kWaves * 64) router_fwd_kernel(const bf16* __restrict__ x, const bf16* __restrict__ w_r,
                                                                 const float* __restrict__ bias, int T, int d, int E,
                                                                 float* __restrict__ logits) {
  __shared__ f32x4 sums[kWaves][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, q = lane >> 4;
  const int t0 = blockIdx.x * 16, e0 = blockIdx.y * 16;
  const bf16* xrow = x + (long)min(t0 + r, T - 1) * d;             // rows past the end are not stored
  const bf16* wrow = w_r + (long)min(e0 + r, E - 1) * d;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int b0 = wave; b0 * kBlock < d; b0 += kAhead * kWaves) {
    bf16x8 xv[kAhead][2], wv[kAhead][2];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if ((b0 + u * kWaves) * kBlock >= d) break;                      // (wave-uniform) nothing is loaded for what a short row lacks
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int k = (b0 + u * kWaves) * kBlock + c * 32 + q * 8;     // d is a multiple of 8: a piece is in or out
        const bool in = k < d;
        const int kk = in ? k : 0;
        const bf16x8 zero = {};
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(xrow + kk), b = *reinterpret_cast<const bf16x8*>(wrow + kk);
        xv[u][c] = in ? a : zero;
        wv[u][c] = in ? b : zero;
      }
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if ((b0 + u * kWaves) * kBlock >= d) break;
#pragma unroll
      for (int c = 0; c < 2; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[u][c], xv[u][c], acc, 0, 0, 0);
    }
  }
  sums[wave][lane] = acc;
  __syncthreads();
  if (wave != 0) return;
  f32x4 s = sums[0][lane];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) s += sums[w][lane];
  // a lane of the 16 x 16 result holds token lane % 16 and experts 4 * (lane / 16) + 0..3
  const int t = t0 + r, e = e0 + q * 4;
  if (t >= T) return;
#pragma unroll
  for (int v = 0; v < 4; ++v)
    if (e + v < E) logits[(long)t * E + e + v] = s[v] + (bias ? bias[e + v] : 0.f);
}

}  // namespace

bool router_fwd_small(int T, int E) { return (long)cdiv(T, 16) * cdiv(E, 16) <= 512; }

// d a multiple of 8, x and w_r 16-byte aligned.
int launch_router_fwd_small(const void* x, const void* w_r, const float* bias, int T, int d, int E, float* logits, hipStream_t s) {
  router_fwd_kernel<<<dim3((unsigned)cdiv(T, 16), (unsigned)cdiv(E, 16)), kWaves * 64, 0, s>>>(
      static_cast<const bf16*>(x), static_cast<const bf16*>(w_r), bias, T, d, E, logits);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

}  // namespace moe
