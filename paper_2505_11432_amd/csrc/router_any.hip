// Router matmul on the vector ALU (fp32 FMA, LDS-tiled 64x64x16): logits[T,E] = x[T,d] * w_r[E,d]^T (+ bias) for rows of any
// length and alignment.  Rows that can be read in 16-byte pieces go to the matrix cores (router_fwd.hip, gemm_mfma.hip,
// gemm_f32.hip); here every element is a load of its own, which is what bounds it.
#include "moe_common.h"

namespace moe {
namespace {

constexpr int BM = 64, BN = 64, BK = 16, NT = 256;

template <typename T>
__global__ void __launch_bounds__(NT) router_any_kernel(const T* __restrict__ x, const T* __restrict__ w_r, const float* __restrict__ bias,
                                                        int rows, int d, int E, int tiles_n, float* __restrict__ logits) {
  __shared__ float As[BK][BM + 4];
  __shared__ float Bs[BK][BN + 4];
  const int tid = threadIdx.x;
  const int n0 = blockIdx.x % tiles_n * BN, m0 = blockIdx.x / tiles_n * BM;

  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  const int ty = tid / 16, tx = tid % 16;
  for (int kb = 0; kb < d; kb += BK) {
#pragma unroll
    for (int i = 0; i < (BM * BK) / NT; ++i) {
      const int idx = tid + i * NT;
      const int r = idx / BK, k = idx % BK;
      const bool in = kb + k < d;
      As[k][r] = in && m0 + r < rows ? to_f32(x[(long)(m0 + r) * d + kb + k]) : 0.f;
      Bs[k][r] = in && n0 + r < E ? to_f32(w_r[(long)(n0 + r) * d + kb + k]) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }

#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= rows) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n < E) logits[(long)m * E + n] = acc[i][j] + (bias ? bias[n] : 0.f);
    }
  }
}

}  // namespace

int launch_router_any(const void* x, const void* w_r, const float* bias, moe_dtype dt, int T, int d, int E, float* logits, hipStream_t s) {
  const int tiles_n = cdiv(E, BN);
  const long blocks = (long)tiles_n * cdiv(T, BM);
  if (blocks > 0x7fffffffL) return MOE_ERR_UNSUPPORTED;
  const dim3 grid((unsigned)blocks), block(NT);
  if (dt == MOE_F32)
    router_any_kernel<float><<<grid, block, 0, s>>>((const float*)x, (const float*)w_r, bias, T, d, E, tiles_n, logits);
  else
    router_any_kernel<bf16><<<grid, block, 0, s>>>((const bf16*)x, (const bf16*)w_r, bias, T, d, E, tiles_n, logits);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

}  // namespace moe
