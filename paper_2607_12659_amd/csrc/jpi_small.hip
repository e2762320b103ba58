// Five-launch decoder layers for few activation rows (bf16): QKV, attention
// (jpi_flash.hip), O projection, gate/up, Down, with no row kernels between.
//
// With a few hundred rows every kernel of a layer is far shorter than the
// chip's rates would allow: a launch costs 1.55 us in a graph whatever it does
// and each dependent memory round trip about 1 us more.  So a layer should have
// few launches, and each of them one round trip:
//
// * The norm is folded into the products around it.  The kernel that updates
//   the residual stream (O, Down, the step's head) writes u = bf16(h (1 + scale))
//   with the next norm's scale and, per row and 16 columns, the sum of squares
//   of h; the product that follows multiplies u, scales its result row by
//   r = 1 / sqrt(mean h^2 + eps) and adds c[n] = sum_k shift[k] W[n][k], which
//   depends on the weights and the step only and comes from a table:
//   sum_k (r h_k (1 + scale_k) + shift_k) W[n][k] = r sum_k u_k W[n][k] + c[n].
//   What is rounded to bf16 is h (1 + scale), not the normalised value: where a
//   shift cancels a large activation the product's error is 2^-9 of the
//   activation (cancelled 4 / 16 times over: 2.7 / 6 times the error of the
//   eight-launch layers), where a shift dominates it is smaller than theirs.
// * O and Down are not split over workgroups: a workgroup computes a tile over
//   the whole contraction, so it can update the residual stream in its epilogue.
// * A workgroup's waves split the contraction; each wave issues every load of
//   its share at once and the partial tiles meet in LDS.  Both operands are
//   stored in fragment order (16 x 32 blocks, lane-linear KiB), so every load
//   instruction reads one contiguous KiB.  Row-major activations took up to
//   twice as long (rows 2 to 8 KiB apart meet in the same L2 channels): Down at
//   100 rows 5.9 -> 10.2 us.
#include <algorithm>

#include "jpi_device.h"
#include "jpi_internal.h"

namespace jpi {

namespace {

typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));

typedef unsigned int u32;
typedef u32 u32x2 __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

// 2 GiB from p on, for loads by byte offset that read nothing (and give 0) at offset 2^31
__device__ __forceinline__ rsrc_t whole(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, 0x7fffffff, 0x00020000);
}
__device__ __forceinline__ float loadf(rsrc_t r, u32 off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

// Sum over `TPR` (a power of two <= 64) consecutive lanes, fixed order.
template <int TPR>
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
  for (int o = TPR / 2; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// A wave's 16 x 16 result tile (lane: rows 4 (lane / 16) + i, column lane % 16) into a
// fragment-ordered matrix of `KSd` 32-column blocks per row group, column tile t: through
// 512 bytes of LDS, so that it leaves as 16-byte pieces that cover 512 contiguous bytes.
// LDS accesses of one wave are ordered.
__device__ __forceinline__ void store_frag_tile(bf16* dst, int rg, int KSd, int t, bf16* lds, const float (&v)[4]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < 4; ++i) lds[(4 * (lane >> 4) + i) * 16 + (lane & 15)] = from_f32<bf16>(v[i]);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (lane < 32) {
    const int p = lane >> 4, r = lane & 15;
    const bf16x8 x = *reinterpret_cast<const bf16x8*>(lds + r * 16 + p * 8);
    *reinterpret_cast<bf16x8*>(dst + (((size_t)rg * KSd + (t >> 1)) * 64 + (2 * (t & 1) + p) * 16 + r) * 8) = x;
  }
}

// The same for rows 4 q .. 4 q + 3 of a 16 x 16 result tile (lane: row 4 q + lane / 16, column lane % 16)
// through 128 bytes of LDS: two runs of 64 contiguous bytes.
__device__ __forceinline__ void store_frag_quad(bf16* dst, int rg, int KSd, int t, int q, bf16* lds, float v) {
  const int lane = threadIdx.x & 63;
  lds[lane] = from_f32<bf16>(v);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (lane < 8) {
    const int p = lane >> 2, r = lane & 3;
    const bf16x8 x = *reinterpret_cast<const bf16x8*>(lds + r * 16 + p * 8);
    *reinterpret_cast<bf16x8*>(dst + (((size_t)rg * KSd + (t >> 1)) * 64 + (2 * (t & 1) + p) * 16 + 4 * q + r) * 8) = x;
  }
}

// Have every field of the arguments in scalar registers from here on.
__device__ __forceinline__ void pin_args(const SmallGemm& g) {
  asm volatile("" :: "s"(g.A), "s"(g.W), "s"(g.M), "s"(g.N), "s"(g.KS));
  asm volatile("" :: "s"(g.ssq), "s"(g.n_ssq), "s"(g.inv_w), "s"(g.eps), "s"(g.c), "s"(g.seq));
  asm volatile("" :: "s"(g.h), "s"(g.h_in), "s"(g.h_ld), "s"(g.gate), "s"(g.scale));
  asm volatile("" :: "s"(g.ssq_out), "s"(g.u));
  asm volatile("" :: "s"(g.ep.q), "s"(g.ep.skvf));
  asm volatile("" :: "s"(g.ep.rope), "s"(g.ep.n_heads), "s"(g.ep.head_dim), "s"(g.ep.horizon), "s"(g.ep.rope_shared));
}

// Tile of 16 MT x 16 NT over the whole contraction; NWV waves each take K
// blocks of KW 32-deep steps in turn.  One memory round trip when
// K = 32 NWV KW.
template <int MT, int NT, int NWV, int KW, SmallEpi EPI, bool T0>
__global__ __launch_bounds__(64 * NWV) void k_small(SmallGemm g) {
  using MF = Mfma<bf16>;
  constexpr bool FOLD = EPI == SE_QKV || EPI == SE_GEGLU || EPI == SE_F32;
  constexpr int PN = FOLD ? 2 : 1;             // column tiles per epilogue unit (RoPE and gate/up pairs)
  constexpr int UNITS = MT * NT / PN;
  constexpr int WPU = NWV / UNITS >= 4 ? 4 : 1;  // waves that share a unit, one row quad each, or a wave per unit
  constexpr int QW = 4 / WPU;  // result rows per lane
  constexpr int TPR = 64 * NWV / (16 * MT) > 64 ? 64 : 64 * NWV / (16 * MT);  // threads per row: sums of squares
  constexpr int NCH = TPR >= 16 ? 1 : 16 / TPR;  // 4-float pieces of a row's sums of squares per thread (W <= 1024)
  static_assert(UNITS <= NWV && (!FOLD || (TPR & (TPR - 1)) == 0), "waves for every unit");
  static_assert(NT % PN == 0, "column pairs stay in one tile");
  __shared__ f32x4 red[NWV][MT * NT][64];
  __shared__ float rs[16 * MT];
  __shared__ __attribute__((aligned(16))) bf16 stage[NWV][WPU == 4 ? 64 : 256];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Everything the kernel reads from its arguments, in one go: read where they are used, they
  // cost several dependent trips to the argument block.
  const SmallGemm& h = g;
  pin_args(h);
  const int fr = lane & 15, M = h.M, KS = h.KS, RG = (M + 15) / 16;
  const int n0 = blockIdx.x * NT, m0 = blockIdx.y * MT;  // in 16-wide tiles

  const bf16 *ap[MT], *wp[NT];
#pragma unroll
  for (int m = 0; m < MT; ++m) ap[m] = h.A + ((size_t)min(m0 + m, RG - 1) * KS * 64 + lane) * 8;
#pragma unroll
  for (int n = 0; n < NT; ++n) wp[n] = h.W + ((size_t)(n0 + n) * KS * 64 + lane) * 8;
  MF::frag wf[KW][NT], af[KW][MT];
  auto load = [&](int kb) {
#pragma unroll
    for (int k = 0; k < KW; ++k)
#pragma unroll
      for (int n = 0; n < NT; ++n) wf[k][n] = MF::load(wp[n] + (size_t)(kb + k) * 512);
#pragma unroll
    for (int k = 0; k < KW; ++k)
#pragma unroll
      for (int m = 0; m < MT; ++m) af[k][m] = MF::load(ap[m] + (size_t)(kb + k) * 512);
  };
  constexpr u32 NONE = 0x80000000u;
  f32x4 sq[NCH];
  const int sr = tid / TPR, sc = tid % TPR;  // row and share of the sums of squares
  if constexpr (FOLD) {
    const rsrc_t rq = whole(h.ssq);
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      const int c4 = 4 * (sc + j * TPR), row = min((int)blockIdx.y * MT * 16 + sr, M - 1);
      sq[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                            rq, c4 < h.n_ssq ? (u32)(row * h.n_ssq + c4) * 4 : NONE, 0, 0));
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  load(wave * KW);
  __builtin_amdgcn_sched_barrier(0);  // every operand load goes out before anything waits

  // Then the epilogue's operands, which do not depend on the product.  Buffer loads whose offset
  // lies outside the range in waves without a unit (nothing is read): a branch around ordinary
  // loads made the compiler wait for them where it ends, before the products.
  const int uw = wave / WPU, q0 = wave % WPU;              // this wave's unit and row quad
  const int um = uw / (NT / PN), un = (uw % (NT / PN)) * PN;
  const int rl0 = um * 16 + (WPU == 4 ? 4 * q0 + (lane >> 4) : 4 * (lane >> 4));  // row j: rl0 + j
  const int row0 = m0 * 16 + rl0, col0 = (n0 + un) * 16 + fr;
  const bool unit = wave < UNITS * WPU && (m0 + um) < RG;
  float e0[QW], e1[QW], e2[QW];  // per result row: (c lo, c hi) or (h, gate, scale)
  u32x2 rope[EPI == SE_QKV ? QW : 1];
  u32 dst[EPI == SE_QKV ? QW : 1];  // element offset of the first of the pair
  u32 dst2 = 0;                     // from it to the second
  const u32 coff = unit ? (u32)col0 * 4 : NONE;
  if constexpr (FOLD) {
    const float c0 = loadf(whole(h.c), coff), c1 = loadf(whole(h.c + 16), coff);
#pragma unroll
    for (int j = 0; j < QW; ++j) {
      e0[j] = c0;
      e1[j] = c1;
    }
  } else if constexpr (EPI == SE_RESID) {
    const float gt = loadf(whole(h.gate), coff), sl = loadf(whole(h.scale), coff);
    const rsrc_t rh = whole(h.h_in);
#pragma unroll
    for (int j = 0; j < QW; ++j) {
      e0[j] = loadf(rh, unit ? (u32)(min(row0 + j, M - 1) * h.h_ld + col0) * 4 : NONE);
      e1[j] = gt;
      e2[j] = sl;
    }
  } else {
    const float c0 = loadf(whole(h.c), coff);
#pragma unroll
    for (int j = 0; j < QW; ++j) e0[j] = c0;
  }
  if constexpr (EPI == SE_QKV) {
    // q heads and k: RoPE pairs (d, d + Dh/2), d = 16 t + c of 32-column group t; v: stored transposed
    const int Dh = h.ep.head_dim, half = Dh >> 1, dsh = 31 - __builtin_clz(Dh), H = h.ep.horizon, nH = h.ep.n_heads;
    const int hn = col0 >> dsh, within = col0 & (Dh - 1), d = (within >> 5) * 16 + (within & 15);
    const bool is_v = hn > nH;
    const rsrc_t rr = whole(h.ep.rope);
    dst2 = is_v ? 512 : hn == nH ? half * 16 : half;  // in blocks: the next 16 dims, Dh / 2 dims on
    const int nbs = (H + 31) / 32;
#pragma unroll
    for (int j = 0; j < QW; ++j) {
      const int row = min(row0 + j, M - 1), b = row / H, q = row - b * H;
      rope[j] = __builtin_amdgcn_raw_buffer_load_b64(rr, unit && !is_v ? (u32)((h.ep.rope_shared ? q : row) * half + d) * 8 : NONE, 0, 0);
      const int kb = (b * nbs + (q >> 5)) * 64 * Dh;  // KvBlock; key q & 31 of it
      dst[j] = is_v       ? kb + 32 * Dh + ((within >> 4) * 64 + ((q & 31) >> 3) * 16 + (within & 15)) * 8 + (q & 7)
               : hn == nH ? kb + ((((q >> 2) & 1) * (Dh >> 5) + (d >> 5)) * 64 + ((d & 31) >> 3) * 16 + 4 * ((q & 31) >> 3) + (q & 3)) * 8 + (d & 7)
                          : ((b * nH + hn) * H + q) * Dh + d;
    }
  }
  if constexpr (T0) {  // committed rows at t = 0 take the t = 0 table row
#pragma unroll
    for (int j = 0; j < QW; ++j) {
      const int ia = (row0 + j) % h.seq - h.n_lead;
      const bool t0 = ia >= 0 && ia < h.n_t0;
      if constexpr (FOLD) {
        const float c0 = loadf(whole(h.c + h.c_t0), coff), c1 = loadf(whole(h.c + h.c_t0 + 16), coff);
        e0[j] = t0 ? c0 : e0[j];
        e1[j] = t0 ? c1 : e1[j];
      } else if constexpr (EPI == SE_RESID) {
        const float gt = loadf(whole(h.gate + h.t0_delta), coff), sl = loadf(whole(h.scale + h.t0_delta), coff);
        e1[j] = t0 ? gt : e1[j];
        e2[j] = t0 ? sl : e2[j];
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (FOLD) {
    f32x4 t = sq[0];
#pragma unroll
    for (int j = 1; j < NCH; ++j) t += sq[j];
    const float s = group_sum<TPR>((t[0] + t[1]) + (t[2] + t[3]));
    if (sc == 0 && sr < 16 * MT) rs[sr] = 1.0f / sqrtf(s * h.inv_w + h.eps);
  }

  f32x4 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kb = wave * KW;;) {
#pragma unroll
    for (int k = 0; k < KW; ++k)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[m][n] = MF::run(af[k][m], wf[k][n], acc[m][n]);
    kb += NWV * KW;
    if (kb >= KS) break;
    load(kb);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) red[wave][m * NT + n][lane] = acc[m][n];
  __syncthreads();
  if (!unit) return;
  // Sum of the waves' partial tiles, in wave order.  With a row quad q per wave a lane takes row 4 q + lane / 16:
  // the 256 bytes of lanes 16 q .. 16 q + 15 of each partial, one conflict-free read.
  float v[QW][PN];
  if constexpr (WPU == 4) {
    float pt[NWV][PN];
#pragma unroll
    for (int w = 0; w < NWV; ++w)
#pragma unroll
      for (int p = 0; p < PN; ++p)
        pt[w][p] = reinterpret_cast<const float*>(&red[w][um * NT + un + p][16 * q0 + fr])[lane >> 4];
    __builtin_amdgcn_sched_barrier(0);  // every LDS read in flight before the sums
#pragma unroll
    for (int p = 0; p < PN; ++p) {
      v[0][p] = pt[0][p];
#pragma unroll
      for (int w = 1; w < NWV; ++w) v[0][p] += pt[w][p];
    }
  } else {
    f32x4 pt[NWV][PN];
#pragma unroll
    for (int w = 0; w < NWV; ++w)
#pragma unroll
      for (int p = 0; p < PN; ++p) pt[w][p] = red[w][um * NT + un + p][lane];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < PN; ++p) {
      f32x4 t = pt[0][p];
#pragma unroll
      for (int w = 1; w < NWV; ++w) t += pt[w][p];
#pragma unroll
      for (int j = 0; j < QW; ++j) v[j][p] = t[j];
    }
  }
  float out[QW];  // what goes to the next product
#pragma unroll
  for (int j = 0; j < QW; ++j) {
    const int row = row0 + j;
    if constexpr (EPI == SE_QKV) {
      const int hn = col0 >> (31 - __builtin_clz(h.ep.head_dim));
      bf16* base = reinterpret_cast<bf16*>(hn < h.ep.n_heads ? h.ep.q : h.ep.skvf);
      const bool is_v = hn > h.ep.n_heads;
      if (row >= M) continue;
      const float r = rs[rl0 + j], lo = fmaf(r, v[j][0], e0[j]), hi = fmaf(r, v[j][PN - 1], e1[j]);
      const u32 rc = rope[j][0], rsn = rope[j][1];
      const float cx = is_v ? 1.f : __builtin_bit_cast(float, rc), cy = __builtin_bit_cast(float, rsn);  // v: (0, 0) read
      base[dst[j]] = from_f32<bf16>(lo * cx - hi * cy);
      base[dst[j] + dst2] = from_f32<bf16>(lo * cy + hi * cx);
    } else if constexpr (EPI == SE_F32) {
      if (row >= M) continue;
      const float r = rs[rl0 + j];
      h.h[(size_t)row * h.N + col0] = fmaf(r, v[j][0], e0[j]);
      h.h[(size_t)row * h.N + col0 + 16] = fmaf(r, v[j][PN - 1], e1[j]);
    } else if constexpr (EPI == SE_GEGLU) {
      const float r = rs[rl0 + j];
      out[j] = gelu_tanh(fmaf(r, v[j][0], e0[j])) * fmaf(r, v[j][PN - 1], e1[j]);
    } else if constexpr (EPI == SE_SWISH) {
      const float x = v[j][0] + e0[j];
      out[j] = x / (1.0f + expf(-x));
    } else {
      const float h2 = e0[j] + e1[j] * v[j][0];
      const float ss = group16_sum(h2 * h2);
      if (row < M) {
        h.h[(size_t)row * h.N + col0] = h2;
        if (fr == 0) h.ssq_out[(size_t)row * (h.N / 16) + n0 + un] = ss;
      }
      out[j] = h2 * (1.0f + e2[j]);
    }
  }
  if constexpr (EPI != SE_QKV && EPI != SE_F32) {
    if (EPI == SE_RESID && !h.u) return;
    const int KSd = h.N / (32 * PN), t = (n0 + un) / PN;
    if constexpr (WPU == 4) store_frag_quad(h.u, m0 + um, KSd, t, q0, stage[wave], out[0]);
    else store_frag_tile(h.u, m0 + um, KSd, t, stage[wave], out);
  }
}

// ---------------------------------------------------------------------------
// The folded products (QKV, gate/up) for more rows: a ring of direct-to-LDS
// stages over fragment-ordered operands, as k_gemm_dma.  Every load and every
// LDS read is one lane-linear KiB.  At 150 / 400 rows gate/up takes 9 / 12 us
// here and 12 / 21 us with a tile of k_small, whose waves read A once per 64
// columns.
// ---------------------------------------------------------------------------
template <int BM_, int BN_, int NW_, int NS_, int WGM_>
struct RingShape {
  static constexpr int BM = BM_, BN = BN_, NW = NW_, NS = NS_, BK = 64, KF = BK / 32, NT = 64 * NW;
  static constexpr int WGM = WGM_, WGN = NW / WGM, TM = BM / WGM / 16, TN = BN / WGN / 16;
  static constexpr int A_INS = BM / 16 * KF, W_INS = BN / 16 * KF, INS = (A_INS + W_INS) / NW;
  static constexpr int STAGE = (A_INS + W_INS) * 1024;  // bytes
  static_assert((A_INS + W_INS) % NW == 0 && TN % 2 == 0, "loads split evenly, column pairs in one wave");
};

template <typename S, SmallEpi EPI, bool T0>
__global__ __launch_bounds__(S::NT) void k_small_ring(SmallGemm g) {
  using MF = Mfma<bf16>;
  constexpr int TPR = S::NT / S::BM, NCH = 16 / TPR;  // threads per row, 4-float pieces each (W <= 1024)
  __shared__ __attribute__((aligned(1024))) char ring[S::NS * S::STAGE];
  const SmallGemm& h = g;
  pin_args(h);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / S::WGN, wn = wave % S::WGN, fr = lane & 15;
  const int m0 = blockIdx.y * S::BM, n0 = blockIdx.x * S::BN, M = h.M, N = h.N, KS = h.KS, nkt = KS / S::KF;
  // epilogue operands, requested before the ring's loads: sums of squares, c, rotation factors
  const int sr = tid / TPR, sc = tid % TPR;
  f32x4 sq[NCH];
  const rsrc_t rq = whole(h.ssq);
#pragma unroll
  for (int j = 0; j < NCH; ++j) {
    const int c4 = 4 * (sc + j * TPR), row = min(m0 + sr, M - 1);
    sq[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                          rq, c4 < h.n_ssq ? (u32)(row * h.n_ssq + c4) * 4 : 0x80000000u, 0, 0));
  }
  float cl[S::TN], ct[T0 ? S::TN : 1];
#pragma unroll
  for (int b = 0; b < S::TN; ++b) {
    const int col = min(n0 + (wn * S::TN + b) * 16 + fr, N - 1);
    cl[b] = h.c[col];
    if constexpr (T0) ct[b] = h.c[h.c_t0 + col];
  }
  u32x2 rope[EPI == SE_QKV ? S::TM : 1][EPI == SE_QKV ? S::TN / 2 : 1][4];
  const int Dh = h.ep.head_dim, half = Dh >> 1, dsh = EPI == SE_QKV ? 31 - __builtin_clz(Dh) : 0, nH = h.ep.n_heads;
  if constexpr (EPI == SE_QKV) {
    const rsrc_t rr = whole(h.ep.rope);
#pragma unroll
    for (int b = 0; b < S::TN; b += 2) {
      const int col = n0 + (wn * S::TN + b) * 16 + fr, hn = col >> dsh, within = col & (Dh - 1);
      const int d = (within >> 5) * 16 + (within & 15);
#pragma unroll
      for (int a = 0; a < S::TM; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = min(m0 + (wm * S::TM + a) * 16 + 4 * (lane >> 4) + i, M - 1);
          rope[a][b / 2][i] = __builtin_amdgcn_raw_buffer_load_b64(rr, hn <= nH ? (u32)((h.ep.rope_shared ? row % h.ep.horizon : row) * half + d) * 8 : 0x80000000u, 0, 0);
        }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  // slice kt into its stage: instruction j loads fragment j (A's row groups, then W's); groups past M or N read as zero
  const unsigned a_bytes = (unsigned)((M + 15) / 16) * KS * 1024u, w_bytes = (unsigned)(N / 16) * KS * 1024u;
  auto issue = [&](int kt) {
    dma_lds_t* st = (dma_lds_t*)ring + (kt % S::NS) * S::STAGE;
#pragma unroll
    for (int i = 0; i < S::INS; ++i) {
      const int j = wave + S::NW * i;
      if (j < S::A_INS) dma_load_1k(h.A, a_bytes, ((unsigned)(m0 / 16 + j / S::KF) * KS + kt * S::KF + j % S::KF) * 1024u + lane * 16u, st + j * 1024);
      else {
        const int jw = j - S::A_INS;
        dma_load_1k(h.W, w_bytes, ((unsigned)(n0 / 16 + jw / S::KF) * KS + kt * S::KF + jw % S::KF) * 1024u + lane * 16u, st + j * 1024);
      }
    }
  };
  f32x4 acc[S::TM][S::TN];
#pragma unroll
  for (int a = 0; a < S::TM; ++a)
#pragma unroll
    for (int b = 0; b < S::TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < S::NS - 1; ++s)
    if (s < nkt) issue(s);
  for (int kt = 0; kt < nkt; ++kt) {
    wait_later<S::INS, S::NS - 2>(min(S::NS - 2, nkt - 1 - kt));
    __builtin_amdgcn_s_barrier();  // every wave's part of slice kt; slice kt - 1 fully consumed
    if (kt + S::NS - 1 < nkt) issue(kt + S::NS - 1);
    const dma_lds_t* As = (const dma_lds_t*)ring + (kt % S::NS) * S::STAGE;
    const dma_lds_t* Ws = As + S::A_INS * 1024;
#pragma unroll
    for (int kk = 0; kk < S::KF; ++kk) {
      MF::frag af[S::TM], wf[S::TN];
#pragma unroll
      for (int a = 0; a < S::TM; ++a) af[a] = *(dma_lds_frag*)(As + (((wm * S::TM + a) * S::KF + kk) * 64 + lane) * 16);
#pragma unroll
      for (int b = 0; b < S::TN; ++b) wf[b] = *(dma_lds_frag*)(Ws + (((wn * S::TN + b) * S::KF + kk) * 64 + lane) * 16);
#pragma unroll
      for (int a = 0; a < S::TM; ++a)
#pragma unroll
        for (int b = 0; b < S::TN; ++b) acc[a][b] = MF::run(af[a], wf[b], acc[a][b]);
    }
  }
  __syncthreads();  // the ring is free: row factors and staging
  float* rs = reinterpret_cast<float*>(ring);
  bf16* stage = reinterpret_cast<bf16*>(ring + 4 * S::BM) + wave * 256;
  {
    f32x4 t = sq[0];
#pragma unroll
    for (int j = 1; j < NCH; ++j) t += sq[j];
    const float s = group_sum<TPR>((t[0] + t[1]) + (t[2] + t[3]));
    if (sc == 0) rs[sr] = 1.0f / sqrtf(s * h.inv_w + h.eps);
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < S::TM; ++a) {
    const int rl = (wm * S::TM + a) * 16 + 4 * (lane >> 4), row0 = m0 + rl;
    float r[4];
    bool t0[4];
    int rb[4], rq4[4];  // QKV: rollout and row in it
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      r[i] = rs[rl + i];
      t0[i] = false;
      if constexpr (T0) {
        const int ia = (row0 + i) % h.seq - h.n_lead;
        t0[i] = ia >= 0 && ia < h.n_t0;
      }
      if constexpr (EPI == SE_QKV) {
        rb[i] = (row0 + i) / h.ep.horizon;
        rq4[i] = (row0 + i) - rb[i] * h.ep.horizon;
      }
    }
#pragma unroll
    for (int b = 0; b < S::TN; b += 2) {
      const int ct0 = n0 / 16 + wn * S::TN + b, col = ct0 * 16 + fr;
      float z[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float lo = fmaf(r[i], acc[a][b][i], T0 && t0[i] ? ct[T0 ? b : 0] : cl[b]);
        const float hi = fmaf(r[i], acc[a][b + 1][i], T0 && t0[i] ? ct[T0 ? b + 1 : 0] : cl[b + 1]);
        if constexpr (EPI == SE_GEGLU) {
          z[i] = gelu_tanh(lo) * hi;
        } else {
          if (row0 + i >= M || col >= N) continue;
          const int hn = col >> dsh, within = col & (Dh - 1), d = (within >> 5) * 16 + (within & 15), q = rq4[i];
          const bool is_v = hn > nH;
          const u32 rc = rope[a][b / 2][i][0], rsn = rope[a][b / 2][i][1];
          const float cx = is_v ? 1.f : __builtin_bit_cast(float, rc), cy = __builtin_bit_cast(float, rsn);
          bf16* base = reinterpret_cast<bf16*>(hn < nH ? h.ep.q : h.ep.skvf);
          const int kb = (rb[i] * ((h.ep.horizon + 31) / 32) + (q >> 5)) * 64 * Dh;
          const int dst = is_v       ? kb + 32 * Dh + ((within >> 4) * 64 + ((q & 31) >> 3) * 16 + (within & 15)) * 8 + (q & 7)
                          : hn == nH ? kb + ((((q >> 2) & 1) * (Dh >> 5) + (d >> 5)) * 64 + ((d & 31) >> 3) * 16 + 4 * ((q & 31) >> 3) + (q & 3)) * 8 + (d & 7)
                                     : ((rb[i] * nH + hn) * h.ep.horizon + q) * Dh + d;
          base[dst] = from_f32<bf16>(lo * cx - hi * cy);
          base[dst + (is_v ? 512 : hn == nH ? half * 16 : half)] = from_f32<bf16>(lo * cy + hi * cx);
        }
      }
      if constexpr (EPI == SE_GEGLU)
        if (row0 - 4 * (lane >> 4) < M && col < N) store_frag_tile(h.u, (m0 + rl) / 16, N / 64, ct0 / 2, stage, z);
    }
  }
}

// One activation row (256 threads): the end of one Euler step and the start of
// the next, both local to the row.  Action rows: v = adaRMSNorm(h) W_out^T +
// b_out, x += dt v (do_out), then h = x W_in^T + b_in with the first norm's u and
// sums of squares (do_in).  Correction rows restart from their token.  Every
// operand that does not depend on the row's chain (W_out, W_in, biases) is
// requested before it starts.
__global__ __launch_bounds__(256) void k_small_head(SmallHead a) {
  __shared__ __attribute__((aligned(16))) float ys[1024];  // W <= 1024: four columns per thread
  __shared__ float xs[64], dots[64], red[4];
  const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int W = a.W, A = a.A, b = m / a.seq, i = m % a.seq - a.n_lead;  // i < 0: a correction row
  const int64_t t0 = i >= 0 && i < a.n_t0 ? 1 : 0;
  const size_t xrow = ((size_t)b * (a.seq - a.n_lead) + i) * A;
  if (i >= 0 && tid < A) xs[tid] = a.x[xrow + tid];
  // the first eight outputs' rows of W_out per wave (all of them at A = 32)
  constexpr int NO = 8;
  bf16x8 wo[NO][2];
  if (a.do_out && i >= 0) {
#pragma unroll
    for (int o = 0; o < NO; ++o)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        wo[o][j] = *reinterpret_cast<const bf16x8*>(a.w_out + (size_t)min(wave + 4 * o, A - 1) * W + min(8 * lane + 512 * j, W - 8));
  }
  const int k = 4 * tid;  // this thread's columns
  if (a.do_out && i >= 0) {
    f32x4 hv, sc, sh;
    float ss = 0.f;
    if (k < W) {
      hv = *reinterpret_cast<const f32x4*>(a.h + (size_t)m * W + k);
      sc = *reinterpret_cast<const f32x4*>(a.scale_f + t0 * a.t0_delta + k);
      sh = *reinterpret_cast<const f32x4*>(a.shift_f + t0 * a.t0_delta + k);
      ss = hv[0] * hv[0] + hv[1] * hv[1] + hv[2] * hv[2] + hv[3] * hv[3];
    }
    const float r = 1.0f / sqrtf(block_sum_256(ss, red) * a.inv_w + a.eps);
    if (k < W) *reinterpret_cast<f32x4*>(ys + k) = hv * r * (1.0f + sc) + sh;
    __syncthreads();
    // wave w: outputs w, w + 4, ..; lane: columns 8 lane + 512 j .. + 7
    auto dot = [&](const bf16x8 (&w)[2]) {
      float p = 0.f;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = 8 * lane + 512 * j;
        if (c >= W) continue;
        const f32x4 y0 = *reinterpret_cast<const f32x4*>(ys + c), y1 = *reinterpret_cast<const f32x4*>(ys + c + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p = fmaf(y0[e], (float)w[j][e], p);
          p = fmaf(y1[e], (float)w[j][4 + e], p);
        }
      }
      return wave_sum(p);
    };
#pragma unroll
    for (int o = 0; o < NO; ++o) {
      const float p = dot(wo[o]);
      if (lane == 0 && wave + 4 * o < A) dots[wave + 4 * o] = p;
    }
    for (int o = wave + 4 * NO; o < A; o += 4) {
      bf16x8 w[2];
#pragma unroll
      for (int j = 0; j < 2; ++j)
        w[j] = *reinterpret_cast<const bf16x8*>(a.w_out + (size_t)o * W + min(8 * lane + 512 * j, W - 8));
      const float p = dot(w);
      if (lane == 0) dots[o] = p;
    }
    __syncthreads();
    if (tid < A && i >= a.n_fixed) {
      const float x2 = xs[tid] + a.dt * (dots[tid] + a.b_out[tid]);
      xs[tid] = x2;
      a.x[xrow + tid] = x2;
    }
  }
  if (!a.do_in) return;
  __syncthreads();
  if (k < W) {
    f32x4 h;
    if (i < 0) {
      h = *reinterpret_cast<const f32x4*>(a.corr + ((size_t)b * a.n_lead + m % a.seq) * W + k);
    } else {
      h = f32x4{0.f, 0.f, 0.f, 0.f};
      if (A % 8 == 0) {
        for (int q = 0; q < A; q += 8) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bf16x8 w = *reinterpret_cast<const bf16x8*>(a.w_in + (size_t)(k + e) * A + q);
#pragma unroll
            for (int z = 0; z < 8; ++z) h[e] = fmaf(xs[q + z], (float)w[z], h[e]);
          }
        }
      } else {
        for (int q = 0; q < A; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) h[e] = fmaf(xs[q], (float)a.w_in[(size_t)(k + e) * A + q], h[e]);
      }
      h += *reinterpret_cast<const f32x4*>(a.b_in + k);
    }
    *reinterpret_cast<f32x4*>(a.h + (size_t)m * W + k) = h;
    const f32x4 u = h * (1.0f + *reinterpret_cast<const f32x4*>(a.scale + t0 * a.t0_delta_in + k));
    *reinterpret_cast<bf16x4*>(a.u + (((size_t)(m / 16) * (W / 32) + k / 32) * 64 + ((k % 32) / 8) * 16 + m % 16) * 8 + k % 8) =
        bf16x4{(bf16)u[0], (bf16)u[1], (bf16)u[2], (bf16)u[3]};
    // 16 columns: four lanes
    float ss = (h[0] * h[0] + h[1] * h[1]) + (h[2] * h[2] + h[3] * h[3]);
    ss += dpp_row<DPP_QUAD_XOR1>(ss);
    ss += dpp_row<DPP_QUAD_XOR2>(ss);
    if ((tid & 3) == 0) a.ssq[(size_t)m * (W / 16) + k / 16] = ss;
  }
}

// c[row][n] = sum_k shift[row][k] w[n][k] in fp64, layer blockIdx.y: a wave takes four columns n and
// six table rows at a time (one column per wave read the shifts from L2 four times as often: 0.8 -> 0.3 ms
// for the pi0.5 shape's 18 layers and 11 rows).
__global__ __launch_bounds__(256) void k_small_shift(const float* __restrict__ shift, int64_t shift_ld,
                                                     int64_t shift_lstride, const bf16* __restrict__ w,
                                                     int64_t w_lstride, float* __restrict__ out, int64_t out_ld,
                                                     int64_t out_lstride, int rows, int N, int K) {
  constexpr int C = 4, R = 6;
  const int lane = threadIdx.x & 63, n0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * C;
  if (n0 >= N) return;
  shift += blockIdx.y * shift_lstride;
  w += blockIdx.y * w_lstride;
  out += blockIdx.y * out_lstride;
  for (int r0 = 0; r0 < rows; r0 += R) {
    double acc[R][C];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < C; ++c) acc[r][c] = 0.0;
    for (int k = 8 * lane; k < K; k += 512) {
      bf16x8 wv[C];
#pragma unroll
      for (int c = 0; c < C; ++c) wv[c] = *reinterpret_cast<const bf16x8*>(w + (size_t)(n0 + c) * K + k);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float* s = shift + (size_t)min(r0 + r, rows - 1) * shift_ld + k;
        const f32x4 a = *reinterpret_cast<const f32x4*>(s), b = *reinterpret_cast<const f32x4*>(s + 4);
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[r][c] += (double)a[e] * (double)(float)wv[c][e] + (double)b[e] * (double)(float)wv[c][4 + e];
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const double t = wave_sum_d(acc[r][c]);
        if (lane == 0 && r0 + r < rows) out[(size_t)(r0 + r) * out_ld + n0 + c] = (float)t;
      }
  }
}

// u[m] = W_a x[m] + b_a (fragment-ordered), one workgroup per action row, 4 columns per thread
__global__ __launch_bounds__(256) void k_action_embed_frag(const float* __restrict__ x, const bf16* __restrict__ w,
                                                           const float* __restrict__ b, bf16* __restrict__ u, int W, int A) {
  __shared__ float xs[64];
  const int m = blockIdx.x;
  if (threadIdx.x < A) xs[threadIdx.x] = x[(size_t)m * A + threadIdx.x];
  __syncthreads();
  for (int k = 4 * threadIdx.x; k < W; k += 1024) {
    f32x4 h = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int q = 0; q < A; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = fmaf(xs[q], (float)w[(size_t)(k + e) * A + q], h[e]);
    h += *reinterpret_cast<const f32x4*>(b + k);
    *reinterpret_cast<bf16x4*>(u + (((size_t)(m / 16) * (W / 32) + k / 32) * 64 + ((k % 32) / 8) * 16 + m % 16) * 8 + k % 8) =
        bf16x4{(bf16)h[0], (bf16)h[1], (bf16)h[2], (bf16)h[3]};
  }
}

__global__ __launch_bounds__(256) void k_small_rows(const float* __restrict__ h, const float* __restrict__ scale,
                                                    bf16* __restrict__ u, float* __restrict__ ssq, int W) {
  const int m = blockIdx.x;
  for (int k = threadIdx.x; k < W; k += 256) {
    const float v = h[(size_t)m * W + k], s = group16_sum(v * v);
    u[(((size_t)(m / 16) * (W / 32) + k / 32) * 64 + ((k % 32) / 8) * 16 + m % 16) * 8 + k % 8] = from_f32<bf16>(v * (1.0f + scale[k]));
    if (k % 16 == 0) ssq[(size_t)m * (W / 16) + k / 16] = s;
  }
}

// h[b] = W_s state[b] + b_s in fp64, its u and sums of squares; one workgroup per 16 columns of a
// row, 16 threads per column
__global__ __launch_bounds__(256) void k_small_state(const float* __restrict__ state, const bf16* __restrict__ w,
                                                     const float* __restrict__ bias, int W, int D,
                                                     const float* __restrict__ scale, float* __restrict__ h,
                                                     bf16* __restrict__ u, float* __restrict__ ssq) {
  __shared__ float hv[16];
  const int b = blockIdx.y, k = blockIdx.x * 16 + threadIdx.x / 16, t = threadIdx.x % 16;
  double acc = 0.0;
  for (int d = t; d < D; d += 16) acc += (double)state[(size_t)b * D + d] * (double)(float)w[(size_t)k * D + d];
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (t == 0) {
    const float v = (float)(acc + (double)bias[k]);
    hv[threadIdx.x / 16] = v;
    h[(size_t)b * W + k] = v;
    u[(((size_t)(b / 16) * (W / 32) + k / 32) * 64 + ((k % 32) / 8) * 16 + b % 16) * 8 + k % 8] = from_f32<bf16>(v * (1.0f + scale[k]));
  }
  __syncthreads();
  if (threadIdx.x < 16) {
    const float v = hv[threadIdx.x], s = group16_sum(v * v);
    if (threadIdx.x == 0) ssq[(size_t)b * (W / 16) + blockIdx.x] = s;
  }
}

typedef RingShape<64, 64, 8, 4, 4> Ring64;    // 64 KB ring, two workgroups per unit; waves 4 x 2 of 16 x 32
typedef RingShape<128, 128, 8, 4, 2> Ring128;  // 128 KB ring; waves 2 x 4 of 64 x 32

template <typename S, SmallEpi EPI>
hipError_t launch_ring(const SmallGemm& g, hipStream_t s) {
  const dim3 grid((g.N + S::BN - 1) / S::BN, (g.M + S::BM - 1) / S::BM);
  if (g.n_t0 > 0) JPI_LAUNCH((k_small_ring<S, EPI, true>), grid, dim3(S::NT), 0, s, g.ev_start, g.ev_stop, g);
  else JPI_LAUNCH((k_small_ring<S, EPI, false>), grid, dim3(S::NT), 0, s, g.ev_start, g.ev_stop, g);
  return hipGetLastError();
}

template <int MT, int NT, int NWV, int KW, SmallEpi EPI>
hipError_t launch_t(const SmallGemm& g, hipStream_t s) {
  const dim3 grid(g.N / 16 / NT, ((g.M + 15) / 16 + MT - 1) / MT);
  if constexpr (EPI != SE_SWISH && EPI != SE_F32)
    if (g.n_t0 > 0) {
      JPI_LAUNCH((k_small<MT, NT, NWV, KW, EPI, true>), grid, dim3(64 * NWV), 0, s, g.ev_start, g.ev_stop, g);
      return hipGetLastError();
    }
  JPI_LAUNCH((k_small<MT, NT, NWV, KW, EPI, false>), grid, dim3(64 * NWV), 0, s, g.ev_start, g.ev_stop, g);
  return hipGetLastError();
}

}  // namespace

bool small_supported(jpi_dtype dt, int W, int nH, int Dh, int F) {
  // 8 waves x one 32-deep step divide every contraction, 16 pieces hold a row's sums of squares
  return dt == JPI_BF16 && W % 256 == 0 && F % 256 == 0 && (nH * Dh) % 256 == 0 && W <= 1024;
}

// Tiles, measured as graph chains on one MI355X (us at 50 / 100 / 150 / 200 / 400 rows):
//   QKV (N 2560, K 1024):  16x32 4.0 5.0 5.9 6.6 9.6   32x64 4.5 4.6 4.8 6.1 8.2
//   O (N 1024, K 2048):    16x16 3.5 4.4 5.4 6.4 9.5   32x16 4.2 4.2 5.1 5.4 8.7   64x32 6.4 6.3 6.2 6.3 6.5
//   Down (N 1024, K 4096): 16x16 5.0 6.8 9.0 11 18     32x16 6.0 5.9 8.8 9.0 16    64x16 8.6 8.1 8.0 8.1 16   64x32 9.8 9.5 9.4 9.5 10
//   gate/up (N 8192, K 1024): 64x32 6.8 10 13          64x64 8.2 8.1 12 12 22
// At these widths, on 256 units, the smallest tile that still gives at most about
// one and a half workgroups per unit wins; past that each workgroup's operands
// are read too often.  The rule below is that choice written as row-group
// thresholds: it looks at the rows (and at the contraction's length), not at N or
// the unit count, so narrower products (the correction module's N 1536, 1024 and
// 4096, experts below width 1024) take the tiles of the widths above unmeasured.
hipError_t launch_small(SmallEpi epi, const SmallGemm& g, hipStream_t s) {
  const int RG = (g.M + 15) / 16;
  const bool k32 = g.KS % 32 == 0;  // the wide variants take 32 steps a turn (64 or 128 below)
  if (g.M < 1 || g.KS % 8 != 0 || g.N % 64 != 0) return hipErrorInvalidValue;
  switch (epi) {
    case SE_QKV:
      if (!k32) return launch_t<2, 2, 8, 1, SE_QKV>(g, s);
      if (RG > 12) return launch_ring<Ring64, SE_QKV>(g, s);
      return RG <= 4 ? launch_t<1, 2, 8, 4, SE_QKV>(g, s) : launch_t<2, 4, 8, 4, SE_QKV>(g, s);
    case SE_GEGLU:
      if (!k32) {
        // narrow experts (W 256, 512, 768): small tiles up to about six workgroups per unit, past that the rings (us a layer,
        // small tiles / rings: W 512, F 2048 at 260 rows 30.6 / 32.0, F 4096 at 190 rows 38.5 / 37.0 and 510 rows 51.4 / 44.9,
        // F 8192 at 510 rows 71 / 60; W 256, F 1024 at 510 rows 26.4 / 27.5)
        if (RG <= 4 || (g.N / 32) * ((RG + 1) / 2) <= 1536) return launch_t<2, 2, 8, 1, SE_GEGLU>(g, s);
        return RG <= 16 || g.N < 8192 ? launch_ring<Ring64, SE_GEGLU>(g, s) : launch_ring<Ring128, SE_GEGLU>(g, s);
      }
      if (RG == 1) return launch_t<1, 2, 8, 4, SE_GEGLU>(g, s);
      if (RG <= 4) return launch_t<4, 2, 16, 2, SE_GEGLU>(g, s);
      return RG <= 16 ? launch_ring<Ring64, SE_GEGLU>(g, s) : launch_ring<Ring128, SE_GEGLU>(g, s);
    case SE_F32:
      if (!k32) return launch_t<2, 2, 8, 1, SE_F32>(g, s);
      return RG <= 4 ? launch_t<1, 2, 8, 4, SE_F32>(g, s) : launch_t<2, 4, 8, 4, SE_F32>(g, s);
    case SE_SWISH:
      if (!k32) return launch_t<2, 1, 8, 1, SE_SWISH>(g, s);
      return RG <= 4 ? launch_t<1, 1, 8, 4, SE_SWISH>(g, s) : launch_t<2, 1, 8, 4, SE_SWISH>(g, s);
    case SE_RESID:
      if (!k32) return launch_t<2, 1, 8, 1, SE_RESID>(g, s);
      if (RG <= 4) {
        if (g.KS % 128 == 0) return launch_t<1, 1, 16, 8, SE_RESID>(g, s);
        if (g.KS % 64 == 0) return launch_t<1, 1, 8, 8, SE_RESID>(g, s);
        return launch_t<1, 1, 8, 4, SE_RESID>(g, s);
      }
      if (g.KS % 64 == 0) {
        if (RG <= (g.KS >= 128 ? 8 : 16)) return launch_t<2, 1, 16, 4, SE_RESID>(g, s);
        if (RG <= 16) return launch_t<4, 1, 16, 4, SE_RESID>(g, s);
      }
      if (RG <= 16) return launch_t<2, 1, 8, 4, SE_RESID>(g, s);
      return launch_t<4, 2, 16, 2, SE_RESID>(g, s);
  }
  return hipErrorInvalidValue;
}

hipError_t enqueue_small_layer(const SmallLayer& y, hipStream_t s) {
  const int HD = y.nH * y.Dh;
  hipError_t e;
  SmallGemm base{};
  base.M = y.B * y.S;
  base.ssq = base.ssq_out = y.ssq;
  base.n_ssq = y.W / 16;
  base.inv_w = 1.0f / (float)y.W;
  base.eps = y.eps;
  base.c_t0 = y.c_t0;
  base.t0_delta = y.t0_delta;
  base.seq = y.S;
  base.n_lead = y.n_lead;
  base.n_t0 = y.n_t0;
  base.h = y.h;
  base.h_ld = y.W;
  auto timed = [&](SmallGemm& g, int kind) {
    g.ev_start = y.ev[kind][0];
    g.ev_stop = y.ev[kind][1];
  };
  SmallGemm g = base;
  if (!y.own_done) {
    g.A = y.u_in;
    g.W = y.w;
    g.N = HD + 2 * y.Dh;
    g.KS = y.W / 32;
    g.c = y.c_qkv;
    g.ep.q = y.q;
    g.ep.skvf = y.skvf;
    g.ep.rope = y.rope;
    g.ep.rope_shared = y.rope_shared;
    g.ep.n_heads = y.nH;
    g.ep.head_dim = y.Dh;
    g.ep.horizon = y.S;
    timed(g, JPI_KERNEL_QKV);
    if ((e = launch_small(SE_QKV, g, s)) != hipSuccess) return e;
  }
  AttnLaunch a{};
  a.q = y.q;
  a.skvf = y.skvf;
  a.kvf = y.kvf;
  a.kvf_bstride = y.kvf_bstride;
  a.prefix_len = y.plen;
  a.B = y.B;
  a.nH = y.nH;
  a.H = y.S;
  a.P = y.P;
  a.Dh = y.Dh;
  a.opart = y.opart;
  a.out = y.o;
  a.out_frag = 1;
  a.n_cu = y.n_cu;
  a.ev_start = y.ev[JPI_KERNEL_ATTENTION][0];
  a.ev_stop = y.ev[JPI_KERNEL_ATTENTION][1];
  if ((e = launch_flash_rows(a, flash_rows_splits(y.B, y.nH, y.S, y.P, y.Dh, y.n_cu), s)) != hipSuccess) return e;
  g = base;
  g.A = (const bf16*)y.o;
  g.W = y.w + y.off_o;
  g.N = y.W;
  g.KS = HD / 32;
  g.h_in = y.h_in;
  g.gate = y.gate_attn;
  g.scale = y.scale_mlp;
  g.u = y.u;
  timed(g, JPI_KERNEL_OPROJ);
  if ((e = launch_small(SE_RESID, g, s)) != hipSuccess) return e;
  g = base;
  g.A = y.u;
  g.W = y.w + y.off_gu;
  g.N = 2 * y.F;
  g.KS = y.W / 32;
  g.c = y.c_gu;
  g.u = (bf16*)y.z;
  timed(g, JPI_KERNEL_GATEUP);
  if ((e = launch_small(SE_GEGLU, g, s)) != hipSuccess) return e;
  g = base;
  g.A = (const bf16*)y.z;
  g.W = y.w + y.off_d;
  g.N = y.W;
  g.KS = y.F / 32;
  g.h_in = y.h;
  g.gate = y.gate_mlp;
  g.scale = y.scale_next;
  g.u = y.u_out ? y.u : nullptr;
  timed(g, JPI_KERNEL_DOWN);
  return launch_small(SE_RESID, g, s);
}

hipError_t launch_small_head(const SmallHead& a, hipStream_t s) {
  if (a.M < 1 || a.W > 1024 || a.W % 32 != 0 || a.A < 1 || a.A > 64 || a.seq <= a.n_lead) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_small_head, dim3(a.M), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_small_rows(const float* h, const float* scale, int M, int W, void* u, float* ssq, hipStream_t s) {
  if (M < 1 || W % 256 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_small_rows, dim3(M), dim3(256), 0, s, h, scale, (bf16*)u, ssq, W);
  return hipGetLastError();
}

hipError_t launch_action_embed_frag(const float* x, const void* w, const float* b, void* u, int M, int W, int A,
                                    hipStream_t s) {
  if (M < 1 || A > 64 || W % 32 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_action_embed_frag, dim3(M), dim3(256), 0, s, x, (const bf16*)w, b, (bf16*)u, W, A);
  return hipGetLastError();
}

hipError_t launch_small_state(const float* state, const void* w, const float* b, int B, int W, int state_dim,
                              const float* scale, float* h, void* u, float* ssq, hipStream_t s) {
  if (B < 1 || W % 32 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_small_state, dim3(W / 16, B), dim3(256), 0, s, state, (const bf16*)w, b, W, state_dim, scale, h,
                     (bf16*)u, ssq);
  return hipGetLastError();
}

hipError_t launch_small_shift(const float* shift, int64_t shift_ld, int64_t shift_lstride, const void* w,
                              int64_t w_lstride, float* out, int64_t out_ld, int64_t out_lstride, int layers, int rows,
                              int N, int K, hipStream_t s) {
  if (K % 8 != 0 || N % 4 != 0 || rows < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_small_shift, dim3((N + 15) / 16, layers), dim3(256), 0, s, shift, shift_ld, shift_lstride,
                     (const bf16*)w, w_lstride, out, out_ld, out_lstride, rows, N, K);
  return hipGetLastError();
}

}  // namespace jpi
