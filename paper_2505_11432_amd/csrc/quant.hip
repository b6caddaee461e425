// E4M3 cast of activations and gradients (Section 5 "Communication compression for FP8 training":
// E4M3 for all tensors, per-token quantisation forward, per-channel quantisation in groups of 128
// tokens backward; Section 7 "FP8 training": per-token 1 x h scales).
//
// Scale rule (the paper gives none): amax = max|v| of the group; amax == 0 -> scale 1, codes 0;
// else inv = 448/amax and scale = amax/448 (one fp32 division each), code = nearest-even e4m3 of
// clamp(fp32(v)*inv, -448, 448).  The clamp comes first because the gfx950 converter turns
// magnitudes of 465 and more into NaN instead of saturating.
#include "moe_common.h"

namespace moe {
namespace {

constexpr float kE4M3Max = 448.0f;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float clamp448(float p) { return fminf(fmaxf(p, -kE4M3Max), kE4M3Max); }

// Four floats -> four packed codes (byte i = element i).
__device__ __forceinline__ unsigned pack4_e4m3(float a, float b, float c, float d) {
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(a), clamp448(b), 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(clamp448(c), clamp448(d), w, true);
  return (unsigned)w;
}

// The codes of one 16-byte vector of T: V bytes, V-byte aligned, one store.
template <typename T> __device__ __forceinline__ void store_codes(const Vec16<T>& v, float inv, uint8_t* dst) {
  constexpr int V = 16 / sizeof(T);
  unsigned out[V / 4];
#pragma unroll
  for (int i = 0; i < V / 4; ++i)
    out[i] = pack4_e4m3(to_f32(v.v[4 * i]) * inv, to_f32(v.v[4 * i + 1]) * inv, to_f32(v.v[4 * i + 2]) * inv,
                        to_f32(v.v[4 * i + 3]) * inv);
  if constexpr (V == 8) { const u32x2 o = {out[0], out[1]}; __builtin_nontemporal_store(o, reinterpret_cast<u32x2*>(dst)); }
  else __builtin_nontemporal_store(out[0], reinterpret_cast<unsigned*>(dst));
}

template <int THREADS>
__device__ __forceinline__ float block_max(float v, float* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = v;
  __syncthreads();
  v = red[0];
#pragma unroll
  for (int w = 1; w < THREADS / 64; ++w) v = fmaxf(v, red[w]);
  __syncthreads();
  return v;
}

// One block per row.  A row of up to THREADS x 8 vectors stays in registers between the amax pass and the
// convert pass, so HBM sees each element once (256 threads: 16384 bf16 columns; 1024 threads, used for wider
// rows: 65536); longer rows are read a second time (from L2).
template <typename T, int THREADS, int kHold = 8>
__global__ void __launch_bounds__(THREADS) quant_rows_kernel(const T* __restrict__ src, int rows, int cols,
                                                             uint8_t* __restrict__ codes, float* __restrict__ scales) {
  __shared__ float red[THREADS / 64];
  constexpr int V = 16 / sizeof(T);
  const int nvec = cols / V;
  const bool in_regs = nvec <= THREADS * kHold;
  for (int r = blockIdx.x; r < rows; r += gridDim.x) {
    const T* row = src + (long)r * cols;
    Vec16<T> hold[kHold];
    float amax = 0.f;
    if (in_regs) {
      // every load is issued before the first value is used; vectors past the row's end re-read its last vector
      // (same maximum, never stored), which keeps the loads unconditional
#pragma unroll
      for (int h = 0; h < kHold; ++h) {
        const int c = min((int)threadIdx.x + h * THREADS, nvec - 1);
        // streamed once: non-temporal
        hold[h] = __builtin_bit_cast(Vec16<T>, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(row + (long)c * V)));
      }
#pragma unroll
      for (int h = 0; h < kHold; ++h)
#pragma unroll
        for (int i = 0; i < V; ++i) amax = fmaxf(amax, fabsf(to_f32(hold[h].v[i])));
    } else {
      for (int c = threadIdx.x; c < nvec; c += THREADS) {
        const Vec16<T> v = *reinterpret_cast<const Vec16<T>*>(row + (long)c * V);
#pragma unroll
        for (int i = 0; i < V; ++i) amax = fmaxf(amax, fabsf(to_f32(v.v[i])));
      }
    }
    amax = block_max<THREADS>(amax, red);
    const float inv = amax > 0.f ? kE4M3Max / amax : 1.0f;
    if (threadIdx.x == 0) scales[r] = amax > 0.f ? amax / kE4M3Max : 1.0f;
    auto convert = [&](const Vec16<T>& v, int c) { store_codes(v, inv, codes + (long)r * cols + (long)c * V); };
    if (in_regs) {
#pragma unroll
      for (int h = 0; h < kHold; ++h) {
        const int c = threadIdx.x + h * THREADS;
        {
          // keep the row as the 16 raw bytes per vector between the two passes: without this the compiler holds
          // the fp32 values it made for the amax pass (4x the registers)
          u32x4 raw = __builtin_bit_cast(u32x4, hold[h]);
          asm volatile("" : "+v"(raw));
          hold[h] = __builtin_bit_cast(Vec16<T>, raw);
        }
        if (c < nvec) convert(hold[h], c);
      }
    } else {
      for (int c = threadIdx.x; c < nvec; c += THREADS) convert(*reinterpret_cast<const Vec16<T>*>(row + (long)c * V), c);
    }
  }
}

// One wave per row, for rows of at most 64 x kHold vectors: no barrier, and four rows per block in flight.  Holding eight
// vectors per thread of a 256-thread block for rows that fill two of them cost six more loads per thread: rows of 4096
// bf16 columns, 8192 of them, 22.8 -> 18.0 us.
template <typename T, int kHold>
__global__ void __launch_bounds__(256) quant_rows_wave_kernel(const T* __restrict__ src, int rows, int cols,
                                                              uint8_t* __restrict__ codes, float* __restrict__ scales) {
  constexpr int V = 16 / sizeof(T);
  const int lane = threadIdx.x & 63, nvec = cols / V;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const T* row = src + (long)r * cols;
  u32x4 raw[kHold];
#pragma unroll
  for (int h = 0; h < kHold; ++h)      // vectors past the row's end re-read its last one (same maximum, never stored)
    raw[h] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(row + (long)min(lane + h * 64, nvec - 1) * V));
  float amax = 0.f;
#pragma unroll
  for (int h = 0; h < kHold; ++h) {
    const Vec16<T> v = __builtin_bit_cast(Vec16<T>, raw[h]);
#pragma unroll
    for (int i = 0; i < V; ++i) amax = fmaxf(amax, fabsf(to_f32(v.v[i])));
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
  const float inv = amax > 0.f ? kE4M3Max / amax : 1.0f;
  if (lane == 0) scales[r] = amax > 0.f ? amax / kE4M3Max : 1.0f;
#pragma unroll
  for (int h = 0; h < kHold; ++h) {
    asm volatile("" : "+v"(raw[h]));            // the raw vectors are what lives on, not their fp32 values
    const int c = lane + h * 64;
    if (c < nvec) store_codes(__builtin_bit_cast(Vec16<T>, raw[h]), inv, codes + (long)r * cols + (long)c * V);
  }
}

// Column of load l of thread cq of CQ in a slab, V elements a load: the CQ threads of a row take neighbouring 16 bytes, so that
// a load reads whole lines whatever the type (fp32: a thread's eight columns are two runs of four).
template <int V, int CQ = 16> __device__ __forceinline__ constexpr int slab_col(int cq, int l) { return l * CQ * V + cq * V; }

// One block per (128-row group, slab of CQ * 8 columns): thread (rg, cq) holds R rows rg, rg + 128 / R, ... of eight columns, 16
// bytes (fp32: two times 16) per row with all loads in flight together; the column maxima are reduced over a wave's row
// groups with shuffles and over the waves through LDS.  (Four columns per thread, read one by one, 16 maxima per column read
// back from LDS: 8192 x 4096 bf16 from memory 28.8 us, from the last-level cache 20.5, fp32 37 and 28.7; this kernel 19.5,
// 19.5, 35 and 27.  Eight columns per thread as one run, also of fp32: 23, 22, - and 40.)
template <typename T, int CQ, bool NT>
__global__ void __launch_bounds__(256) quant_colgroup_kernel(const T* __restrict__ src, int rows, int cols,
                                                             uint8_t* __restrict__ codes,
                                                             float* __restrict__ scales, int slabs) {
  constexpr int V = 16 / sizeof(T), L = 8 / V;      // loads per row
  constexpr int GROUPS = 256 / CQ, R = 128 / GROUPS, WAVES = 4, SLAB = CQ * 8;
  __shared__ __attribute__((aligned(16))) float cmax[WAVES][SLAB];
  const int g = blockIdx.x / slabs;
  const int cq = threadIdx.x % CQ, rg = threadIdx.x / CQ;
  const int c0 = (blockIdx.x % slabs) * SLAB;
  const int r0 = g * 128;
  u32x4 raw[R][L];
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const int c = c0 + slab_col<V, CQ>(cq, l);
#pragma unroll
    for (int i = 0; i < R; ++i) raw[i][l] = u32x4{0, 0, 0, 0};
    if (c < cols) {                                 // cols is a multiple of 16: all V columns or none
#pragma unroll
      for (int i = 0; i < R; ++i) {
        // rows past the end repeat the last row: the same column maxima, never stored
        const u32x4* p = reinterpret_cast<const u32x4*>(src + (long)min(r0 + rg + GROUPS * i, rows - 1) * cols + c);
        raw[i][l] = NT ? __builtin_nontemporal_load(p) : *p;
      }
    }
  }
  float v[R][8];
  float amax[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) amax[j] = 0.f;
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const Vec16<T> w = __builtin_bit_cast(Vec16<T>, raw[i][l]);
#pragma unroll
      for (int j = 0; j < V; ++j) {
        v[i][l * V + j] = to_f32(w.v[j]);
        amax[l * V + j] = fmaxf(amax[l * V + j], fabsf(v[i][l * V + j]));
      }
    }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
#pragma unroll
    for (int off = CQ; off < 64; off <<= 1) amax[j] = fmaxf(amax[j], __shfl_xor(amax[j], off));
  }
  if ((threadIdx.x & 63) < CQ) {
#pragma unroll
    for (int j = 0; j < 8; ++j) cmax[threadIdx.x >> 6][slab_col<V, CQ>(cq, j / V) + j % V] = amax[j];
  }
  __syncthreads();
  float inv[8];
#pragma unroll
  for (int j4 = 0; j4 < 8; j4 += 4) {
    const int cs = slab_col<V, CQ>(cq, j4 / V) + j4 % V;
    float m[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < WAVES; ++q) {
      const float4 t = *reinterpret_cast<const float4*>(&cmax[q][cs]);
      m[0] = fmaxf(m[0], t.x); m[1] = fmaxf(m[1], t.y); m[2] = fmaxf(m[2], t.z); m[3] = fmaxf(m[3], t.w);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      inv[j4 + j] = m[j] > 0.f ? kE4M3Max / m[j] : 1.0f;
      if (rg == 0 && c0 + cs < cols) scales[(long)g * cols + c0 + cs + j] = m[j] > 0.f ? m[j] / kE4M3Max : 1.0f;
    }
  }
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int r = r0 + rg + GROUPS * i;
    if (r >= rows) break;
    const unsigned lo = pack4_e4m3(v[i][0] * inv[0], v[i][1] * inv[1], v[i][2] * inv[2], v[i][3] * inv[3]);
    const unsigned hi = pack4_e4m3(v[i][4] * inv[4], v[i][5] * inv[5], v[i][6] * inv[6], v[i][7] * inv[7]);
    uint8_t* dst = codes + (long)r * cols + c0;
    if constexpr (V == 8) {
      if (c0 + cq * 8 < cols) *reinterpret_cast<u32x2*>(dst + cq * 8) = u32x2{lo, hi};
    } else {
      if (c0 + cq * 4 < cols) *reinterpret_cast<unsigned*>(dst + cq * 4) = lo;
      if (c0 + slab_col<V, CQ>(cq, 1) < cols) *reinterpret_cast<unsigned*>(dst + slab_col<V, CQ>(cq, 1)) = hi;
    }
  }
}


// ---- backward-orientation cast for the weight-gradient GEMMs ---------------------------------------------
// Section 7 "FP8 training": per-channel quantisation within 128-token groups for the backward pass.  The
// contraction index of a weight-gradient GEMM is the token, so the codes are written transposed ([channel]
// [token], K-major for the matrix cores) and every expert's segment is padded with zero codes to a multiple
// of 128 tokens: a group never spans two experts, every k-step of the GEMM is one whole group, and the group
// scale is a power of two (E8M0 byte), which the block-scaled MFMA applies inside the contraction.
// Scale rule: k = smallest integer with amax * 2^-k <= 448 (448 = 1.75 * 2^8), k = 0 for amax = 0,
// clamped to [-126, 127]; byte = k + 127; code = nearest-even e4m3 of clamp(v * 2^-k, +-448).

// pad_offsets[e] = first padded token column of expert e (a multiple of 128); pad_offsets[E] = total.
__global__ void tgroup_offsets_kernel(const int32_t* __restrict__ offsets, int E, int32_t* __restrict__ pad_offsets) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    int run = 0;
    pad_offsets[0] = 0;
    for (int e = 0; e < E; ++e) {
      run += (offsets[e + 1] - offsets[e] + 127) / 128 * 128;
      pad_offsets[e + 1] = run;
    }
  }
}

// One block per (padded 128-token group, 128-channel slab).  Thread (rgrp, cq) holds eight consecutive tokens
// (rows 8*rgrp .. 8*rgrp+7) of eight consecutive channels: a wave's load touches four rows with 16 bytes per lane,
// and a channel's eight codes of those tokens are eight consecutive bytes of the transposed output, written to the
// LDS tile as one 8-byte word (16-byte chunks of a tile row are XOR-swizzled by the channel octet, so the sixteen
// threads of a row group do not meet in one bank).  The eight loads of a thread are issued together, past the
// segment's end too (a branch around each made them wait for one another: 16384 x 28672 bf16 309 -> 287 us, 16384 x
// 14336 codes 133 -> 100).  Channel maxima are reduced over the wave's four row groups with shuffles and over the four
// waves through LDS.  Global memory sees 16-byte lanes forming 128-byte rows (one channel x 128 tokens).
template <typename T>
__global__ void __launch_bounds__(256) quant_tgroup_kernel(const T* __restrict__ src,
                                                           const float* __restrict__ src_row_scale, int cols,
                                                           const int32_t* __restrict__ offsets,
                                                           const int32_t* __restrict__ pad_offsets, int E,
                                                           uint8_t* __restrict__ codes_t, long ldt,
                                                           uint8_t* __restrict__ e8m0, int slabs) {
  constexpr int CH = 128;                           // channels per block
  __shared__ float cmax[4][CH];
  __shared__ __attribute__((aligned(16))) uint8_t tile[CH][128 + 16];
  const int g = blockIdx.x / slabs;
  const int tok0 = g * 128;                         // padded token column of this group
  if (tok0 >= pad_offsets[E]) return;
  int lo = 0, hi = E;                               // expert whose padded range holds tok0
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pad_offsets[mid] <= tok0) lo = mid; else hi = mid;
  }
  const int e = lo;
  const int r0 = offsets[e] + (tok0 - pad_offsets[e]);      // first source row of the group
  const int r_end = offsets[e + 1];
  const int cq = threadIdx.x % 16, rgrp = threadIdx.x / 16;
  const int c0 = (blockIdx.x % slabs) * CH;
  // the thread's eight channels: one run, or for fp32 two of four, 64 apart, so that every load reads whole lines
  constexpr int V = sizeof(T) == 4 ? 4 : 8;
  auto chan = [&](int j) __attribute__((always_inline)) { return slab_col<V>(cq, j / V) + j % V; };
  // every load is issued before the first value is used; rows past the segment's end re-read its last row and count as 0
  constexpr int LB = 8 * (int)sizeof(T);            // bytes per row and thread
  const int last = cols - V;                        // cols is a multiple of 16: all V channels of a run or none
  unsigned raw[8][LB / 4];
  float rs[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = min(r0 + rgrp * 8 + i, r_end - 1);
    const T* p = src + (long)r * cols;
    if constexpr (LB == 8) {
      const u32x2 w = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p + min(c0 + cq * 8, last)));
      raw[i][0] = w[0]; raw[i][1] = w[1];
      rs[i] = src_row_scale[r];
    } else {
#pragma unroll
      for (int l = 0; l < LB / 16; ++l) {
        const u32x4 w = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p + min(c0 + slab_col<V>(cq, l), last)));
#pragma unroll
        for (int q = 0; q < 4; ++q) raw[i][4 * l + q] = w[q];
      }
    }
  }
  float v[8][8];
  float amax[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) amax[j] = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const bool in = r0 + rgrp * 8 + i < r_end;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float t;
      if constexpr (LB == 8) {
        // e4m3 codes with one scale per source row: the value is code * scale, rounded once to fp32
        const int w = (int)raw[i][j / 4];
        t = (j % 4 == 0 ? __builtin_amdgcn_cvt_f32_fp8(w, 0) : j % 4 == 1 ? __builtin_amdgcn_cvt_f32_fp8(w, 1)
             : j % 4 == 2 ? __builtin_amdgcn_cvt_f32_fp8(w, 2) : __builtin_amdgcn_cvt_f32_fp8(w, 3)) * rs[i];
      } else if constexpr (LB == 16) {
        t = __uint_as_float(j % 2 ? raw[i][j / 2] & 0xffff0000u : raw[i][j / 2] << 16);      // bf16 is the upper half of fp32
      } else {
        t = __uint_as_float(raw[i][j]);
      }
      v[i][j] = in ? t : 0.f;
      amax[j] = fmaxf(amax[j], fabsf(v[i][j]));
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    amax[j] = fmaxf(amax[j], __shfl_xor(amax[j], 16));
    amax[j] = fmaxf(amax[j], __shfl_xor(amax[j], 32));
  }
  if ((threadIdx.x & 63) < 16) {
#pragma unroll
    for (int j = 0; j < 8; ++j) cmax[threadIdx.x >> 6][chan(j)] = amax[j];
  }
  __syncthreads();
  float inv[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int ch = chan(j);
    const float m = fmaxf(fmaxf(cmax[0][ch], cmax[1][ch]), fmaxf(cmax[2][ch], cmax[3][ch]));
    int k = 0;
    if (m > 0.f) {
      const unsigned bits = __float_as_uint(m);
      k = (int)((bits >> 23) & 0xffu) - 127 - 8 + ((bits & 0x7fffffu) > 0x600000u ? 1 : 0);
      k = max(-126, min(127, k));
    }
    inv[j] = __uint_as_float((unsigned)(127 - k) << 23);          // 2^-k, exact
    if (rgrp == 0 && c0 + ch < cols) e8m0[(long)g * cols + c0 + ch] = (uint8_t)(k + 127);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    uint2 w;
    w.x = pack4_e4m3(v[0][j] * inv[j], v[1][j] * inv[j], v[2][j] * inv[j], v[3][j] * inv[j]);
    w.y = pack4_e4m3(v[4][j] * inv[j], v[5][j] * inv[j], v[6][j] * inv[j], v[7][j] * inv[j]);
    const int ch = chan(j), chunk = ((rgrp >> 1) ^ ((ch >> 3) & 7)) << 4;       // swizzled 16-byte chunk of the tile row
    *reinterpret_cast<uint2*>(&tile[ch][chunk + ((rgrp & 1) << 3)]) = w;
  }
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < 4; ++pass) {
    const int ch = pass * 32 + threadIdx.x / 8, seg = threadIdx.x % 8;
    if (c0 + ch < cols)
      *reinterpret_cast<uint4*>(codes_t + (long)(c0 + ch) * ldt + tok0 + seg * 16) =
          *reinterpret_cast<const uint4*>(&tile[ch][(seg ^ ((ch >> 3) & 7)) << 4]);
  }
}

// A thread makes 16 bytes of output at a time (8 bf16 or 4 fp32 of a row: a wave's store is one run of 1 KiB), U such pieces a
// block apart with all loads in flight together.  (Four codes per thread, an element-index division for each and scalar
// stores: 8192 x 4096 to bf16, from memory, 27.7 us with row scales, 28.5 with channel scales; now 20.2 and 24.1.)
enum ScaleRead { ROW_SCALE, GROUP_SCALES, GROUP_SCALES_VEC };     // VEC: the scales are 16-byte aligned
template <typename T, ScaleRead SR, int U>
__global__ void __launch_bounds__(256) dequant_kernel(const uint8_t* __restrict__ codes,
                                                      const float* __restrict__ scales, int rows, int cols,
                                                      T* __restrict__ dst) {
  constexpr int P = 16 / sizeof(T);
  const int per_row = cols / P;
  const long n = (long)rows * per_row;
  for (long base = blockIdx.x * (256L * U) + threadIdx.x; base < n; base += (long)gridDim.x * (256 * U)) {
    unsigned w[U][P / 4];
    float s[U][P];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long i = min(base + u * 256, n - 1);            // past the end: the last piece again, not stored
      const int r = n <= 0x7fffffffL ? (int)((unsigned)i / (unsigned)per_row) : (int)(i / per_row);
      const int c = (int)(i - (long)r * per_row) * P;
      const uint8_t* src = codes + (long)r * cols + c;
      if constexpr (P == 8) {
        const u32x2 t = *reinterpret_cast<const u32x2*>(src);
        w[u][0] = t[0]; w[u][1] = t[1];
      } else {
        w[u][0] = *reinterpret_cast<const unsigned*>(src);
      }
      const float* sp = SR == ROW_SCALE ? scales + r : scales + (long)(r / 128) * cols + c;
#pragma unroll
      for (int q = 0; q < P / 4; ++q) {
        float4 t;
        if constexpr (SR == GROUP_SCALES_VEC) t = *reinterpret_cast<const float4*>(sp + 4 * q);
        else if constexpr (SR == GROUP_SCALES) t = make_float4(sp[4 * q], sp[4 * q + 1], sp[4 * q + 2], sp[4 * q + 3]);
        else t = make_float4(sp[0], sp[0], sp[0], sp[0]);
        s[u][4 * q] = t.x; s[u][4 * q + 1] = t.y; s[u][4 * q + 2] = t.z; s[u][4 * q + 3] = t.w;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (base + u * 256 >= n) break;
      Vec16<T> o;
#pragma unroll
      for (int q = 0; q < P / 4; ++q) {
        o.v[4 * q + 0] = from_f32<T>(__builtin_amdgcn_cvt_f32_fp8((int)w[u][q], 0) * s[u][4 * q + 0]);
        o.v[4 * q + 1] = from_f32<T>(__builtin_amdgcn_cvt_f32_fp8((int)w[u][q], 1) * s[u][4 * q + 1]);
        o.v[4 * q + 2] = from_f32<T>(__builtin_amdgcn_cvt_f32_fp8((int)w[u][q], 2) * s[u][4 * q + 2]);
        o.v[4 * q + 3] = from_f32<T>(__builtin_amdgcn_cvt_f32_fp8((int)w[u][q], 3) * s[u][4 * q + 3]);
      }
      *reinterpret_cast<Vec16<T>*>(dst + (base + u * 256) * P) = o;
    }
  }
}

}  // namespace

int launch_quant_fp8(const void* src, moe_dtype src_dt, int rows, int cols, moe_qmode mode, uint8_t* codes,
                     float* scales, hipStream_t s) {
  if (rows == 0 || cols == 0) return MOE_OK;
  if (mode == MOE_Q_ROW) {
    const int grid = rows < 256 * 16 ? rows : 256 * 16;
    const int nvec = cols / (16 / (int)dtype_size(src_dt));
    const bool wide = nvec > 256 * 8;                    // more vectors than 256 threads can hold
    if (nvec <= 64 * 8) {
      constexpr int kMaxRows = 1 << 25;                  // per launch, which holds less than 2^32 threads
      for (long r0 = 0; r0 < rows; r0 += kMaxRows) {
        const int n = rows - r0 < kMaxRows ? (int)(rows - r0) : kMaxRows, waves = cdiv(n, 4);
        uint8_t* const c = codes + r0 * cols;
#define MOE_WAVE_ROWS(TT)                                                                                      \
  const TT* const p = (const TT*)src + r0 * cols;                                                              \
  if (nvec <= 64 * 2) quant_rows_wave_kernel<TT, 2><<<waves, 256, 0, s>>>(p, n, cols, c, scales + r0);         \
  else if (nvec <= 64 * 4) quant_rows_wave_kernel<TT, 4><<<waves, 256, 0, s>>>(p, n, cols, c, scales + r0);    \
  else quant_rows_wave_kernel<TT, 8><<<waves, 256, 0, s>>>(p, n, cols, c, scales + r0);
        if (src_dt == MOE_F32) { MOE_WAVE_ROWS(float) } else { MOE_WAVE_ROWS(bf16) }
#undef MOE_WAVE_ROWS
        MOE_LAUNCH_CHECK();
      }
    } else if (src_dt == MOE_F32) {
      if (wide) quant_rows_kernel<float, 1024><<<grid, 1024, 0, s>>>((const float*)src, rows, cols, codes, scales);
      else quant_rows_kernel<float, 256><<<grid, 256, 0, s>>>((const float*)src, rows, cols, codes, scales);
    } else {
      if (wide && nvec <= 256 * 16) quant_rows_kernel<bf16, 256, 16><<<rows < 256 * 64 ? rows : 256 * 64, 256, 0, s>>>((const bf16*)src, rows, cols, codes, scales);
      else if (wide) quant_rows_kernel<bf16, 1024><<<grid, 1024, 0, s>>>((const bf16*)src, rows, cols, codes, scales);
      else quant_rows_kernel<bf16, 256><<<grid, 256, 0, s>>>((const bf16*)src, rows, cols, codes, scales);
    }
  } else {
    // Narrow tensors take a narrower slab, of which more threads have columns (2^20 x 16 bf16: slabs of 32 / 64 / 128 columns
    // 22 / 23 / 32 us; x 64 columns and more the wide one: 8192 x 1040 15.4 / 9.3 / 7.9).  Streaming loads: for bf16 always (8192
    // x 4096 from memory 19.5 against 21.4, from the last-level cache 19.5 against 17.4; 8192 x 28672 109 against 130), for
    // fp32 only what that cache cannot hold (8192 x 4096 30 against 35 and 30 against 27; 8192 x 28672 210 against 225).
    const int cq = cols <= 32 ? 4 : cols <= 64 ? 8 : 16;
    const int slabs = cdiv(cols, cq * 8);
    const int grid = cdiv(rows, 128) * slabs;
#define MOE_COLGROUP(TT, CQ, NT) quant_colgroup_kernel<TT, CQ, NT><<<grid, 256, 0, s>>>((const TT*)src, rows, cols, codes, scales, slabs)
    if (src_dt == MOE_F32) {
      if (cq == 4) MOE_COLGROUP(float, 4, false);
      else if (cq == 8) MOE_COLGROUP(float, 8, false);
      else if ((long)rows * cols < (1L << 26)) MOE_COLGROUP(float, 16, false);
      else MOE_COLGROUP(float, 16, true);
    } else {
      if (cq == 4) MOE_COLGROUP(bf16, 4, true);
      else if (cq == 8) MOE_COLGROUP(bf16, 8, true);
      else MOE_COLGROUP(bf16, 16, true);
    }
#undef MOE_COLGROUP
  }
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

int launch_tgroup_offsets(const int32_t* offsets, int E, int32_t* pad_offsets, hipStream_t s) {
  tgroup_offsets_kernel<<<1, 64, 0, s>>>(offsets, E, pad_offsets);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

int launch_quant_tgroup(const void* src, const float* src_row_scale, moe_dtype src_dt, int rows, int cols, const int32_t* offsets,
                        const int32_t* pad_offsets, int E, uint8_t* codes_t, long ldt, uint8_t* e8m0, hipStream_t s) {
  if (cols == 0) return MOE_OK;
  const int slabs = cdiv(cols, 128);
  const int groups = cdiv(rows, 128) + E;              // upper bound on the padded group count
  const long grid = (long)groups * slabs;
  if (grid <= 0 || grid > 0x7fffffffL) return MOE_ERR_UNSUPPORTED;
  if (src_dt == MOE_F32)
    quant_tgroup_kernel<float><<<(int)grid, 256, 0, s>>>((const float*)src, nullptr, cols, offsets, pad_offsets, E, codes_t, ldt, e8m0, slabs);
  else if (src_dt == MOE_BF16)
    quant_tgroup_kernel<bf16><<<(int)grid, 256, 0, s>>>((const bf16*)src, nullptr, cols, offsets, pad_offsets, E, codes_t, ldt, e8m0, slabs);
  else
    quant_tgroup_kernel<uint8_t><<<(int)grid, 256, 0, s>>>((const uint8_t*)src, src_row_scale, cols, offsets, pad_offsets, E, codes_t, ldt, e8m0, slabs);
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

int launch_dequant_fp8(const uint8_t* codes, const float* scales, int rows, int cols, moe_qmode mode, void* dst,
                       moe_dtype dst_dt, hipStream_t s) {
  if (rows == 0 || cols == 0) return MOE_OK;
  const long pieces = (long)rows * (cols / (16 / (int)dtype_size(dst_dt)));
  // Few pieces: one per thread, so that they make enough waves (64 x 4096 2.5 -> 2.05 us).  With channel scales, four vectors of
  // them beside each piece, one piece per thread is the faster one up to larger sizes (bf16, from memory: 8192 x 4096 30.7 ->
  // 24.1, 8192 x 6000 44.5 -> 37.8, 2^20 x 256 147 -> 162; fp32 1000 x 8192 12.4 -> 11.5), but not on narrow rows (2^20 x 16 bf16
  // 8.8 -> 9.5, fp32 17.9 -> 20.0).
  const bool few = pieces <= (mode == MOE_Q_ROW || cols < 128 ? 1L << 18 : dst_dt == MOE_BF16 ? 1L << 23 : 1L << 21);
  long blocks = few ? (pieces + 255) / 256 : (pieces + 1023) / 1024;
  if (blocks > 256 * 64) blocks = 256 * 64;
#define MOE_DEQUANT(TT, SR)                                                                                          \
  if (few) dequant_kernel<TT, SR, 1><<<(int)blocks, 256, 0, s>>>(codes, scales, rows, cols, (TT*)dst);               \
  else dequant_kernel<TT, SR, 4><<<(int)blocks, 256, 0, s>>>(codes, scales, rows, cols, (TT*)dst)
#define MOE_DEQUANT_SR(TT)                                                \
  if (mode == MOE_Q_ROW) { MOE_DEQUANT(TT, ROW_SCALE); }                  \
  else if (aligned16(scales)) { MOE_DEQUANT(TT, GROUP_SCALES_VEC); }      \
  else { MOE_DEQUANT(TT, GROUP_SCALES); }
  if (dst_dt == MOE_F32) { MOE_DEQUANT_SR(float) } else { MOE_DEQUANT_SR(bf16) }
#undef MOE_DEQUANT_SR
#undef MOE_DEQUANT
  MOE_LAUNCH_CHECK();
  return MOE_OK;
}

}  // namespace moe
