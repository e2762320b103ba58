// Device helpers shared by the libjpi kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#include "jpi_internal.h"

namespace jpi {

// Launch with optional start/stop events tied to the dispatch itself.
#define JPI_LAUNCH(kern, grid, block, shm, strm, evs, eve, ...)                           \
  do {                                                                                    \
    if ((evs) || (eve))                                                                   \
      hipExtLaunchKernelGGL(kern, grid, block, shm, strm, evs, eve, 0, __VA_ARGS__);      \
    else                                                                                  \
      hipLaunchKernelGGL(kern, grid, block, shm, strm, __VA_ARGS__);                      \
  } while (0)

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <typename T>
struct Mfma;

template <>
struct Mfma<bf16> {
  static constexpr int KPL = 8;    // k values per lane per instruction
  static constexpr int KSUB = 32;  // k depth of one instruction
  typedef bf16x8 frag;
  static __device__ __forceinline__ frag load(const bf16* p) { return *reinterpret_cast<const bf16x8*>(p); }
  static __device__ __forceinline__ f32x4 run(frag a, frag b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

template <>
struct Mfma<float> {
  static constexpr int KPL = 1;
  static constexpr int KSUB = 4;
  typedef float frag;
  static __device__ __forceinline__ frag load(const float* p) { return *p; }
  static __device__ __forceinline__ f32x4 run(frag a, frag b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

template <typename T>
__device__ __forceinline__ T from_f32(float v) { return static_cast<T>(v); }

// Value of another lane of the same 16-lane row through a DPP operand
// modifier (one VALU move; no LDS crossbar round trip).
template <int CTRL>
__device__ __forceinline__ float dpp_row(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
constexpr int DPP_QUAD_XOR1 = 0xb1;   // quad_perm [1,0,3,2]
constexpr int DPP_QUAD_XOR2 = 0x4e;   // quad_perm [2,3,0,1]
constexpr int DPP_HALF_MIRROR = 0x141;  // lane i <-> 7 - i within each half-row
constexpr int DPP_MIRROR = 0x140;       // lane i <-> 15 - i within each row

// Sum over the 16 lanes that share lane / 16 (one row group of an MFMA tile).
// Every stage pairs lanes whose partial results are equal, so all 16 lanes
// end with the same bits.
__device__ __forceinline__ float group16_sum(float v) {
  v += dpp_row<DPP_QUAD_XOR1>(v);
  v += dpp_row<DPP_QUAD_XOR2>(v);
  v += dpp_row<DPP_HALF_MIRROR>(v);
  v += dpp_row<DPP_MIRROR>(v);
  return v;
}
__device__ __forceinline__ float group16_max(float v) {
  v = fmaxf(v, dpp_row<DPP_QUAD_XOR1>(v));
  v = fmaxf(v, dpp_row<DPP_QUAD_XOR2>(v));
  v = fmaxf(v, dpp_row<DPP_HALF_MIRROR>(v));
  v = fmaxf(v, dpp_row<DPP_MIRROR>(v));
  return v;
}

// Whole-wave sum, the same in every lane: row sums, then the four rows in order.
__device__ __forceinline__ float wave_sum(float v) {
  v = group16_sum(v);
  const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0));
  const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16));
  const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32));
  const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 48));
  return ((r0 + r1) + r2) + r3;
}

__device__ __forceinline__ float wave_max(float v) {
  v = group16_max(v);
  const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0));
  const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16));
  const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32));
  const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 48));
  return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}


// Block of 256 threads: fixed-order sum (wave sums, then the 4 wave totals in order).
__device__ __forceinline__ float block_sum_256(float v, float* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

// GELU, tanh form: 0.5 z (1 + tanh(u)), u = sqrt(2/pi) (z + 0.044715 z^3),
// evaluated through the identity 0.5 (1 + tanh u) = 1 / (1 + 2^(-2u log2 e)):
// one exp2 and one reciprocal instead of the library tanh (whose cost showed
// in every GeGLU epilogue); relative error about 2e-6, below the bf16 rounding
// of its uses.  Saturates correctly: the exponential overflows to inf (result
// -0) for large negative z and underflows to 0 (result z) for large positive z.
__device__ __forceinline__ float gelu_tanh(float z) {
  const float u2 = 2.f * 0.7978845608028654f * (z + 0.044715f * z * z * z);
  return z * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * u2));
}

// Rotation factors of an EPI_QKV result pair (row, col_lo), or (1, 0) where
// none applies (V columns, rows past M).  They do not depend on the product,
// so a kernel can load them before its K loop and pass them to the epilogue.
__device__ __forceinline__ float2 qkv_rope_factor(const EpiParams& ep, int M, int N, int row, int col_lo) {
  const int Dh = ep.head_dim, qcols = ep.n_heads * Dh;
  if (row >= M || col_lo >= N || col_lo >= qcols + Dh) return float2{1.f, 0.f};
  const int within = col_lo & (Dh - 1);  // Dh is a power of two
  const int d = (within >> 5) * 16 + (within & 15);
  return ep.rope[(size_t)row * (Dh >> 1) + d];  // row = b * H + i
}

// Rollouts and rows in them of a lane's four result rows row0 .. row0 + 3, taken once per row tile: with the
// divisions by the horizon and the head size taken per element, the epilogue cost more than the product
// (QKV at M = 3200, N = 2560, K = 1024: 31.3 us with it, 17 without; 25.4 as it is).
struct QkvRows {
  unsigned b[4], i[4];
};
__device__ __forceinline__ QkvRows qkv_rows(const EpiParams& ep, int row0) {
  QkvRows r;
  const unsigned H = ep.horizon;
  unsigned b = (unsigned)row0 / H, i = (unsigned)row0 - b * H;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    r.b[e] = b;
    r.i[e] = i++;
    if (i == H) i = 0, ++b;
  }
  return r;
}

// EPI_QKV epilogue of a result pair tile (columns col_lo and col_lo + 16 of rows row0 ..) with the rotation
// factors in hand.  A 16-column tile lies in one q head, in k or in v.  V is stored transposed: four
// consecutive tokens of a rollout leave as 8- or 4-byte stores where their place allows it.
__device__ __forceinline__ void epilogue_qkv_tile(const EpiParams& ep, const QkvRows& r, int M, int N, int row0, int col_lo,
                                                  f32x4 lo, f32x4 hi, const float2 (&cs)[4]) {
  if (col_lo >= N) return;
  const int Dh = ep.head_dim, half = Dh >> 1, H = ep.horizon;
  const int hn = __builtin_amdgcn_readfirstlane(col_lo >> (31 - __builtin_clz(Dh))), within = col_lo & (Dh - 1);
  if (hn <= ep.n_heads) {
    const int d = (within >> 5) * 16 + (within & 15);
    const bool is_k = hn == ep.n_heads;
    bf16* base = is_k ? reinterpret_cast<bf16*>(ep.ks) + d
                      : reinterpret_cast<bf16*>(ep.q) + (size_t)hn * (size_t)(H * Dh) + d;
    const size_t bs = is_k && ep.ks_bstride ? (size_t)ep.ks_bstride : (size_t)(is_k ? 1 : ep.n_heads) * (size_t)(H * Dh);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (row0 + e >= M) continue;
      bf16* p = base + r.b[e] * bs + r.i[e] * (size_t)Dh;
      p[0] = from_f32<bf16>(lo[e] * cs[e].x - hi[e] * cs[e].y);
      p[half] = from_f32<bf16>(lo[e] * cs[e].y + hi[e] * cs[e].x);
    }
    return;
  }
  typedef bf16 b4 __attribute__((ext_vector_type(4)));
  typedef bf16 b2 __attribute__((ext_vector_type(2)));
  const b4 x = b4{(bf16)lo[0], (bf16)lo[1], (bf16)lo[2], (bf16)lo[3]}, y = b4{(bf16)hi[0], (bf16)hi[1], (bf16)hi[2], (bf16)hi[3]};
  bf16* p = reinterpret_cast<bf16*>(ep.vst) + ((size_t)r.b[0] * Dh + within) * ep.vst_ld + r.i[0];
  bf16* q = p + (size_t)16 * ep.vst_ld;
  if (row0 + 3 < M && r.i[0] + 3 < (unsigned)H && ((r.i[0] | ep.vst_ld) & 1) == 0) {
    if (((r.i[0] | ep.vst_ld) & 3) == 0) {
      *reinterpret_cast<b4*>(p) = x;
      *reinterpret_cast<b4*>(q) = y;
    } else {
      *reinterpret_cast<b2*>(p) = b2{x[0], x[1]};
      *reinterpret_cast<b2*>(p + 2) = b2{x[2], x[3]};
      *reinterpret_cast<b2*>(q) = b2{y[0], y[1]};
      *reinterpret_cast<b2*>(q + 2) = b2{y[2], y[3]};
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (row0 + e >= M) continue;
    bf16* v = reinterpret_cast<bf16*>(ep.vst) + ((size_t)r.b[e] * Dh + within) * ep.vst_ld + r.i[e];
    v[0] = x[e];
    v[(size_t)16 * ep.vst_ld] = y[e];
  }
}

// s_waitcnt with vmcnt = N and the other counters not waited for
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// wait until at most `later` (<= L) stages of INS loads each are outstanding
template <int INS, int L>
__device__ __forceinline__ void wait_later(int later) {
  if constexpr (L == 0) {
    wait_vm<0>();
  } else {
    if (later >= L) wait_vm<L * INS>();
    else wait_later<INS, L - 1>(later);
  }
}

typedef __attribute__((address_space(3))) char dma_lds_t;
typedef __attribute__((address_space(3))) const bf16x8 dma_lds_frag;

// One 1 KB direct-to-LDS load: 16 bytes per lane from base + byte offset
// `off` (zero past `bytes`) into LDS at dst + 16 * lane.
__device__ __forceinline__ void dma_load_1k(const void* base, unsigned bytes, unsigned off, dma_lds_t* dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(
      __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000), dst, 16, off, 0, 0, 0);
}

}  // namespace jpi
