// Batched prefix + self attention (bf16) for the multi-kernel path.
//
// Queries come from the action tokens; keys and values are the prefix KV of
// the layer followed by the action tokens' own (Appendix, action expert).
// All query heads share the single KV head, so one rollout's nH x H query rows
// form one [nH*H][Dh] matrix (row r = head * H + i) against one key sequence.
// A workgroup (eight waves, two per SIMD) takes 128 of those rows, 16 per
// wave, and a range of 32-key blocks.  The blocks stream through a
// four-stage LDS ring by direct-to-LDS buffer loads, up to three blocks ahead
// of the one being multiplied, so the loads of later blocks overlap the
// products of this one.  A running (max, sum) per row gives the online
// softmax.
// With one key range the workgroup writes the normalised output; with several
// it writes a bf16 partial normalised by its own sum plus (max, sum), merged by k_flash_merge.
//
// Products use v_mfma_f32_16x16x32_bf16 with the operands swapped:
// S^T = K q^T puts one query row in each lane (lane % 16) and four keys of a
// 16-key tile in its four result elements; O^T = V^T P^T then takes P^T
// straight from those registers.  The K rows of the two 16-key tiles of a
// block are interleaved (tile jj, A row 4g + e <-> key 8g + 4jj + e) so that
// a lane's eight probabilities are eight consecutive keys, which makes each
// V^T operand one 16-byte piece of a V^T row.
//
// Key order: the action keys come first (blocks of 32, masked past H), then
// the prefix (masked past prefix_len[b]).  The softmax does not depend on the
// order.  Masked keys get probability 0 and their V entries are zeroed, so
// stale or non-finite memory in unused slots never reaches the output.
#include <algorithm>
#include <math.h>

#include "jpi_device.h"
#include "jpi_internal.h"

namespace jpi {

typedef unsigned int u32;
typedef u32 u32x4 __attribute__((ext_vector_type(4)));
typedef u32 u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));

template <int DH>
struct Flash {
  static constexpr int NW = 8;              // waves per workgroup (two per SIMD)
  static constexpr int RT = 1;              // 16-row query tiles per wave
  static constexpr int KB = 32;             // keys per block
  static constexpr int NS = 4;              // ring stages: three blocks in flight while one is multiplied
  static constexpr int QT = 16 * RT * NW;   // query rows per workgroup
  static constexpr int NST = DH / 32;       // k steps of S^T over the head dim
  static constexpr int NT = DH / 16;        // 16-wide output tiles over the head dim
  static constexpr int KFR = 2 * NST;       // 1 KB K fragments per block (two key tiles)
  static constexpr int VFR = NT;            // 1 KB V^T fragments per block
  static constexpr int LDW = (KFR + VFR) / NW;  // direct-to-LDS loads per wave per block
  static constexpr int STAGE = (KFR + VFR) * 1024;
  static_assert((KFR + VFR) % NW == 0 && LDW >= 1, "fragments split evenly over the waves");
  // fragment w + NW * u is a K fragment iff is_k(w, u); with KFR a multiple of
  // NW that depends on u alone, so every wave's load sequence is known when
  // compiling (which keeps the compiler's count of outstanding loads exact)
  static __device__ __forceinline__ bool is_k(int w, int u) {
    return KFR % NW == 0 ? u < KFR / NW : w + NW * u < KFR;
  }
  static_assert(2 * LDW < 64, "vmcnt range");
};

constexpr int FLASH_MAX_SPLITS = 16;
constexpr float FLASH_LIMIT = 64.f;  // log2 headroom of the probabilities over the row reference

// elements n_ok .. 7 of 8 packed bf16 set to zero (all of them when n_ok <= 0)
__device__ __forceinline__ u32x4 mask8(u32x4 v, int n_ok) {
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] &= (2 * q < n_ok ? 0x0000ffffu : 0u) | (2 * q + 1 < n_ok ? 0xffff0000u : 0u);
  return v;
}

// s_waitcnt: vmcnt = N, lgkmcnt = 0 when L, other counters not waited for
template <int N, bool L>
__device__ __forceinline__ void flash_wait() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | ((L ? 0 : 15) << 8));
}

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef __attribute__((address_space(3))) char lds_t;  // LDS byte pointer (direct-to-LDS loads)

// Buffer resource over [base, base + bytes): loads past the end return zero.
__device__ __forceinline__ rsrc_t rsrc(const void* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// Key sources of one rollout.  Action (suffix) keys: K rows [H][Dh], V^T
// rows [Dh][vst_ld].  Prefix keys: K rows [prefix_len][Dh], V^T rows
// [Dh][vpt_dstride].  The K ranges end at the last valid key, so rows past
// it read as zero.
struct FlashSrc {
  rsrc_t k_act, v_act, k_pre, v_pre;
  int nbs, H, pl;  // action blocks (they come first), action keys, prefix keys
  int last;        // last block of the sequence
  rsrc_t blk;      // prefix as KvBlocks (then k_pre and v_pre are not used)
};

// Direct-to-LDS loads of block jb into one ring stage.  Wave w loads
// fragments w, w + NW, ...: the first KFR are K fragments f = kt * NST + st
// (lane row 4g' + e of the A operand is key 8g' + 4kt + e, k values
// st * 32 + 8g .. + 8; g = lane / 16, g' and e from lane % 16), the next VFR
// are V^T fragments nt (dim nt * 16 + lane % 16, keys 8g .. + 8).  The
// per-lane part of each address (koff, vaoff, vpoff) is fixed for the
// launch; the per-fragment part and the block's first key are added to it,
// so that the whole offset is range-checked (an offset in the scalar
// operand is not part of the buffer's range check): K rows past the last
// valid key read as zero and nothing past the source is touched.  Returns
// the block's valid key count (>= 1).
template <int DH, bool BLK>
__device__ __forceinline__ int flash_issue(lds_t* stage, const FlashSrc& src, int jb, u32 koff, u32 vaoff, u32 vpoff,
                                           int vst_ld, int vpt_ld) {
  using FS = Flash<DH>;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool act = jb < src.nbs;
  const int key0 = (act ? jb : jb - src.nbs) * FS::KB;
  if (BLK && !act) {
    // a KvBlock is a stage's content in order: whole KiB per load, from where they lie.  A block past the
    // sequence is never multiplied; the last one (or block 0 of an empty prefix) is read in its place.
    const u32 at = (u32)max(min(jb, src.last) - src.nbs, 0) * FS::STAGE;
    const u32 lo = (threadIdx.x & 63) * 16;
#pragma unroll
    for (int u = 0; u < FS::LDW; ++u) {
      const int fi = w + FS::NW * u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(src.blk, stage + fi * 1024, 16, lo, at + fi * 1024, 0, 0);
    }
    const int n = src.pl - key0;
    return n < FS::KB ? n : FS::KB;
  }
  const rsrc_t rk = act ? src.k_act : src.k_pre;
  const rsrc_t rv = act ? src.v_act : src.v_pre;
  const u32 voff = act ? vaoff : vpoff;
  const int vld = act ? vst_ld : vpt_ld;
#pragma unroll
  for (int u = 0; u < FS::LDW; ++u) {
    const int fi = w + FS::NW * u;
    if (FS::is_k(w, u)) {
      const int kt = fi / FS::NST, st = fi - kt * FS::NST;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, stage + fi * 1024, 16,
                                               koff + (u32)(((key0 + 4 * kt) * DH + st * 32) * 2), 0, 0, 0);
    } else {
      const int nt = fi - FS::KFR;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, stage + fi * 1024, 16, voff + (u32)((nt * 16 * vld + key0) * 2),
                                               0, 0, 0);
    }
  }
  const int n = (act ? src.H : src.pl) - key0;
  return n < FS::KB ? n : FS::KB;
}

// After this thread's direct-to-LDS loads of a block have landed: zero the
// V^T entries of keys past the valid ones in the pieces it loaded (pieces
// past the end of a V^T row hold other data).  Only a block with fewer than
// KB valid keys has any.
template <int DH>
__device__ __forceinline__ void flash_fix(char* stage, int n_valid) {
  using FS = Flash<DH>;
  if (n_valid >= FS::KB) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int n_ok = n_valid - 8 * (lane >> 4);
  if (n_ok >= 8) return;
#pragma unroll
  for (int u = 0; u < FS::LDW; ++u) {
    const int fi = w + FS::NW * u;
    if (!FS::is_k(w, u)) {
      u32x4* p = reinterpret_cast<u32x4*>(stage + (fi * 64 + lane) * 16);
      *p = mask8(*p, n_ok);
    }
  }
}

// Maximum over the four lanes that hold one query row (lanes r, r + 16,
// r + 32, r + 48): two lane-swap instructions, no LDS round trip.  (The
// swapped pair is copied into scalars before the bit casts: a bit cast of an
// element of the returned vector reads element 0 for both.)
__device__ __forceinline__ float row4_max(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(u32, v), __builtin_bit_cast(u32, v), false, false);
  const u32 a0 = a[0], a1 = a[1];
  v = fmaxf(__builtin_bit_cast(float, a0), __builtin_bit_cast(float, a1));
  const auto b = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(u32, v), __builtin_bit_cast(u32, v), false, false);
  const u32 b0 = b[0], b1 = b[1];
  return fmaxf(__builtin_bit_cast(float, b0), __builtin_bit_cast(float, b1));
}

// One 32-key block for this wave's 16-row query tiles.
// Softmax in the log2 domain against a per-row reference m_ref: the maximum
// of the row's first block.  A later block whose maximum exceeds the
// reference by more than FLASH_LIMIT (probabilities up to 2^FLASH_LIMIT)
// moves the reference up to that maximum and rescales the row's running
// output and sum by 2^(old - new); otherwise the reference stays, so rows
// whose scores stay within that headroom are never rescaled.  The reference
// is the same in the four lanes of a row.  Keys n_valid .. 31 of the block
// are masked.
template <int DH>
__device__ __forceinline__ void flash_compute(const char* cur, int n_valid,
                                              const bf16x8 (&qf)[Flash<DH>::RT][Flash<DH>::NST],
                                              f32x4 (&o)[Flash<DH>::RT][Flash<DH>::NT], float (&m_ref)[Flash<DH>::RT],
                                              float (&l_run)[Flash<DH>::RT], float qscale) {
  using FS = Flash<DH>;
  using MF = Mfma<bf16>;
  constexpr int NST = FS::NST, NT = FS::NT, RT = FS::RT;
  const int lane = threadIdx.x & 63, g = lane >> 4;
  // S^T = K q^T: all K fragments of the block are read from LDS first, then multiplied
  MF::frag kf[NST][2];
#pragma unroll
  for (int st = 0; st < NST; ++st)
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) kf[st][kt] = *reinterpret_cast<const MF::frag*>(cur + ((kt * NST + st) * 64 + lane) * 16);
  f32x4 sc[RT][2];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) sc[rt][0] = sc[rt][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int st = 0; st < NST; ++st)
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) sc[rt][kt] = MF::run(kf[st][kt], qf[rt][st], sc[rt][kt]);
  // the V^T fragments are read while the softmax runs
  MF::frag vf[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) vf[nt] = *reinterpret_cast<const MF::frag*>(cur + ((FS::KFR + nt) * 64 + lane) * 16);
  __builtin_amdgcn_sched_group_barrier(0x100, 2 * NST, 0);
  __builtin_amdgcn_sched_group_barrier(0x008, 2 * NST * RT, 0);
  __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);

  if (n_valid < FS::KB) {
    asm volatile("" ::: "memory");  // a real branch: full blocks skip the masking
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[rt][kt][e] = 8 * g + 4 * kt + e < n_valid ? sc[rt][kt][e] : -INFINITY;
  }
  MF::frag pb[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float m = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int e = 0; e < 4; ++e) m = fmaxf(m, sc[rt][kt][e]);
    const float mx = row4_max(m) * qscale;  // finite: the block holds a valid key
    const bool over = mx > m_ref[rt] + FLASH_LIMIT;  // always on the row's first block (m_ref = -inf)
    if (__any(over)) {
      // 2^(-inf) = 0 on the first block, where the output and sum are still zero
      const float f = over ? __builtin_amdgcn_exp2f(m_ref[rt] - mx) : 1.f;
      l_run[rt] *= f;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) o[rt][nt] *= f;
      m_ref[rt] = over ? mx : m_ref[rt];
    }
    // P^T as the B operand: slot j of the lane's eight <-> key 8g + j.  The
    // row sum adds the same bf16-rounded probabilities that weight V, so a
    // row dominated by one key returns that key's value row exactly.
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bf16 lo = static_cast<bf16>(__builtin_amdgcn_exp2f(fmaf(sc[rt][0][e], qscale, -m_ref[rt])));
      const bf16 hi = static_cast<bf16>(__builtin_amdgcn_exp2f(fmaf(sc[rt][1][e], qscale, -m_ref[rt])));
      pb[rt][e] = lo;
      pb[rt][4 + e] = hi;
      sum += static_cast<float>(lo) + static_cast<float>(hi);
    }
    l_run[rt] += sum;
  }
  // O^T += V^T P^T
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) o[rt][nt] = MF::run(vf[nt], pb[rt], o[rt][nt]);
}

// Work items (rollout, 128-row query tile, key range) in that order, T of
// them; the grid is T rounded up to a multiple of 8 workgroups.  The hardware
// hands workgroup i to XCD i % 8, so item (i % 8) * (grid / 8) + i / 8 puts
// consecutive items, which share a rollout's keys and values, in one XCD's L2.
template <int DH, bool BLK>
__global__ __launch_bounds__(512) void k_flash(AttnLaunch a, int S, int nqt, int qrows, void* part, float2* ml) {
  using FS = Flash<DH>;
  using MF = Mfma<bf16>;
  constexpr int NST = FS::NST, NT = FS::NT, RT = FS::RT, NS = FS::NS, LDW = FS::LDW;
  // one LDS array: the compiler then does not make the ring's LDS reads wait
  // for every outstanding direct-to-LDS load
  __shared__ __attribute__((aligned(1024))) char lds[NS * FS::STAGE];
  static_assert(FS::NW * 64 == 512, "launch bounds");

  const int item = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
  if (item >= a.B * nqt * S) return;
  const int b = item / (nqt * S), split = item % S, qt = (item / S) % nqt;
  const int H = a.H, R = a.nH * H;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int g = lane >> 4, fr = lane & 15;
  const int pl = a.prefix_len[b];
  FlashSrc src;
  src.nbs = (H + FS::KB - 1) / FS::KB;
  src.H = H;
  src.pl = pl;
  const int nb = src.nbs + (pl + FS::KB - 1) / FS::KB;
  src.last = nb - 1;
  if constexpr (BLK)
    src.blk = rsrc(reinterpret_cast<const bf16*>(a.kvf) + (size_t)b * a.kvf_bstride, (int64_t)a.kvf_bstride * 2);
  const int jb0 = (int)((int64_t)split * nb / S), jb1 = (int)((int64_t)(split + 1) * nb / S);
  const int nblk = jb1 - jb0;
  // this wave's first query row; tile qt holds rows [qt * qrows, (qt + 1) * qrows)
  const int row0 = qt * qrows + w * 16 * RT;

  // each split writes its (max, sum) even when it has no keys
  if (nblk == 0) {
    if (S > 1) {
      for (int t = threadIdx.x; t < qrows; t += FS::NW * 64) {
        const int r = qt * qrows + t;
        if (r < R) ml[((size_t)split * a.B + b) * R + r] = float2{-INFINITY, 0.f};
      }
    }
    return;
  }

  src.k_act = rsrc(reinterpret_cast<const bf16*>(a.ks) + (size_t)b * (a.ks_bstride ? a.ks_bstride : (int64_t)H * DH),
                   (int64_t)H * DH * 2);
  src.v_act = rsrc(reinterpret_cast<const bf16*>(a.vst) + (size_t)b * DH * a.vst_ld, (int64_t)DH * a.vst_ld * 2);
  src.k_pre = rsrc(reinterpret_cast<const bf16*>(a.kp) + (size_t)b * a.kp_bstride, (int64_t)pl * DH * 2);
  src.v_pre = rsrc(reinterpret_cast<const bf16*>(a.vpt) + (size_t)b * a.vpt_bstride, (int64_t)DH * a.vpt_dstride * 2);
  const int vst_ld = (int)a.vst_ld, vpt_ld = (int)a.vpt_dstride;
  const u32 koff = (u32)(((8 * (fr >> 2) + (fr & 3)) * DH + 8 * g) * 2);
  const u32 vaoff = (u32)((fr * vst_ld + 8 * g) * 2), vpoff = (u32)((fr * vpt_ld + 8 * g) * 2);

  // query fragments (B operand of S^T): lane holds row fr of tile rt, dims st*32 + 8g .. + 8
  MF::frag qf[RT][NST];
  const bf16* qb = reinterpret_cast<const bf16*>(a.q) + (size_t)b * R * DH;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int r = row0 + 16 * rt + fr;
#pragma unroll
    for (int st = 0; st < NST; ++st) qf[rt][st] = r < R ? MF::load(qb + (size_t)r * DH + st * 32 + 8 * g) : MF::frag{};
  }
  const bool active = row0 < R && 16 * RT * w < qrows;  // wave has query rows of this tile (uniform per wave)

  lds_t* ring = (lds_t*)lds;
  // valid keys of the blocks in the ring, by stage.  The first NS - 1 blocks
  // are issued whatever the range's length (a block past the range reads
  // zeros or other keys into a stage that is never multiplied), so that the
  // count of loads issued after the query fragments is fixed: waiting until
  // at most that many are pending means the fragments have landed, without
  // draining the ring.
  int nval[NS];
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    nval[s] = flash_issue<DH, BLK>(ring + s * FS::STAGE, src, jb0 + s, koff, vaoff, vpoff, vst_ld, vpt_ld);
  flash_wait<(NS - 1) * LDW, false>();

  // log2-domain scores: s * log2(e) / sqrt(Dh)
  const float qscale = 1.4426950408889634f / sqrtf((float)DH);
  f32x4 o[RT][NT];
  float m_ref[RT], l_run[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    m_ref[rt] = -INFINITY;
    l_run[rt] = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) o[rt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  for (int j = 0; j < nblk; ++j) {
    const int slot = j % NS;
    int n_valid = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) n_valid = s == slot ? nval[s] : n_valid;
    // block j has landed once at most min(NS - 2, nblk - 1 - j) later blocks
    // of the range are pending (blocks issued past the range, when it is
    // shorter than NS - 1, only make this wait longer)
    const int later = nblk - 1 - j;
    if (later >= 2) flash_wait<2 * LDW, false>();
    else if (later == 1) flash_wait<LDW, false>();
    else flash_wait<0, false>();
    flash_fix<DH>(lds + slot * FS::STAGE, n_valid);
    // the V^T masks visible; every wave's part of block j landed; block j - 1
    // fully consumed, so its stage can take block j + NS - 1
    flash_wait<63, true>();
    __builtin_amdgcn_s_barrier();
    if (j + NS - 1 < nblk) {
      const int ns = (j + NS - 1) % NS;
      const int nv = flash_issue<DH, BLK>(ring + ns * FS::STAGE, src, jb0 + j + NS - 1, koff, vaoff, vpoff, vst_ld, vpt_ld);
#pragma unroll
      for (int s = 0; s < NS; ++s) nval[s] = s == ns ? nv : nval[s];
    }
    if (active) flash_compute<DH>(lds + slot * FS::STAGE, n_valid, qf, o, m_ref, l_run, qscale);
  }
  if (!active) return;

  // O^T: lane holds dims nt*16 + 4g .. + 4 of query row fr of each tile
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float l = l_run[rt];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    const int r = row0 + 16 * rt + fr;
    if (r >= R) continue;
    const float rl = 1.0f / l;
    if (S == 1) {
      const int hn = r / H, i = r - hn * H;
      const size_t base = ((size_t)b * H + i) * (size_t)a.nH * DH + (size_t)hn * DH + 4 * g;
      if (a.out_f32) {
        float* out = reinterpret_cast<float*>(a.out) + base;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) *reinterpret_cast<f32x4*>(out + nt * 16) = o[rt][nt] * rl;
      } else {
        bf16* out = reinterpret_cast<bf16*>(a.out) + base;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const f32x4 v = o[rt][nt] * rl;
          *reinterpret_cast<bf16x4*>(out + nt * 16) = bf16x4{static_cast<bf16>(v[0]), static_cast<bf16>(v[1]),
                                                             static_cast<bf16>(v[2]), static_cast<bf16>(v[3])};
        }
      }
    } else {
      const size_t rowi = ((size_t)split * a.B + b) * R + r;
      bf16* out = reinterpret_cast<bf16*>(part) + rowi * DH + 4 * g;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const f32x4 v = o[rt][nt] * rl;
        *reinterpret_cast<bf16x4*>(out + nt * 16) = bf16x4{static_cast<bf16>(v[0]), static_cast<bf16>(v[1]),
                                                           static_cast<bf16>(v[2]), static_cast<bf16>(v[3])};
      }
      if (g == 0) ml[rowi] = float2{m_ref[rt], m_ref[rt] == -INFINITY ? 0.f : l};
    }
  }
}

// address of columns col .. col + 3 (col a multiple of 4) of a row of the attention output
__device__ __forceinline__ size_t attn_out_at(const AttnLaunch& a, int DH, int m, int col) {
  const int C = a.nH * DH;
  if (!a.out_frag) return (size_t)m * C + col;
  return (((size_t)(m >> 4) * (C / 32) + (col >> 5)) * 64 + ((col & 31) >> 3) * 16 + (m & 15)) * 8 + (col & 7);
}

// out row (b, head, i) = sum_s 2^(m_s - m) l_s O_s / sum_s 2^(m_s - m) l_s, ranges in order; a
// range with m_s = -inf (no keys, or no weight: l_s = 0) is skipped unless l_s is NaN.  Dh / 4 threads per query row, 4 dims each.  S is
// known when compiling, so that the loads of a row's partials are one round trip
// (16 predicated ones took 7 us at three rollouts whatever S was).
template <int DH, int S, typename TO>
__global__ __launch_bounds__(256) void k_flash_merge(AttnLaunch a, const bf16* part, const float2* ml) {
  constexpr int TPR = DH / 4, RPB = 256 / TPR;
  const int R = a.nH * a.H;
  const int t = threadIdx.x, rr = blockIdx.x * RPB + t / TPR, q4 = t % TPR;
  if (rr >= a.B * R) return;
  const int b = rr / R, r = rr - b * R;
  const int hn = r / a.H, i = r - hn * a.H;
  float2 mv[S];
  u32x2 ov[S];
  float m = -INFINITY;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const size_t rowi = ((size_t)s * a.B + b) * R + r;
    mv[s] = ml[rowi];
    ov[s] = *reinterpret_cast<const u32x2*>(part + rowi * DH + 4 * q4);
  }
#pragma unroll
  for (int s = 0; s < S; ++s) m = fmaxf(m, mv[s].x);
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  float lsum = 0.f;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const bool some = mv[s].x != -INFINITY;
    const float wl = some ? __builtin_amdgcn_exp2f(mv[s].x - m) * mv[s].y : mv[s].y;
    const f32x4 v = f32x4{__builtin_bit_cast(float, ov[s][0] << 16), __builtin_bit_cast(float, ov[s][0] & 0xffff0000u),
                          __builtin_bit_cast(float, ov[s][1] << 16), __builtin_bit_cast(float, ov[s][1] & 0xffff0000u)};
    if (some) acc += wl * v;  // the partial of a range without keys is not written
    lsum += wl;
  }
  acc *= 1.0f / lsum;
  TO* out = reinterpret_cast<TO*>(a.out) + attn_out_at(a, DH, b * a.H + i, hn * DH + 4 * q4);
#pragma unroll
  for (int e = 0; e < 4; ++e) out[e] = from_f32<TO>(acc[e]);
}

template <int DH, typename TO>
static hipError_t launch_merge(const AttnLaunch& a, int S, const bf16* part, const float2* ml, hipStream_t s) {
  constexpr int RPB = 256 / (DH / 4);
  const size_t rows = (size_t)a.B * a.nH * a.H;
  const dim3 grid((unsigned)((rows + RPB - 1) / RPB));
#define MERGE(N) \
  case N: JPI_LAUNCH((k_flash_merge<DH, N, TO>), grid, dim3(256), 0, s, (hipEvent_t) nullptr, a.ev_stop, a, part, ml); break;
  switch (S) {
    MERGE(2) MERGE(3) MERGE(4) MERGE(5) MERGE(6) MERGE(7) MERGE(8) MERGE(9) MERGE(10) MERGE(11) MERGE(12) MERGE(13)
    MERGE(14) MERGE(15) MERGE(16)
    default: return hipErrorInvalidValue;
  }
#undef MERGE
  return hipGetLastError();
}

// Key ranges per (rollout, 128-row tile), one workgroup per compute unit at a time: the count that
// makes rounds x (fixed + blocks per range) least, where a workgroup's start, first load and stores take about
// as long as six 32-key blocks and several ranges cost a merge (three more).  A count just past a whole round was the
// costly case of "enough workgroups to cover the chip once": the 816-token prefill's 51 tiles at 6 ranges are 306
// workgroups in two rounds, at 5 ranges 255 in one.
struct Ranges {
  int S;      // key ranges
  long cost;  // the estimate of the launch that they make least
};
static Ranges flash_ranges(int B, int nH, int H, int P, int n_cu) {
  const int nqt = (nH * H + 127) / 128, nb = kv_blocks(H) + kv_blocks(P);
  Ranges best{1, -1};
  for (int s = 1; s <= FLASH_MAX_SPLITS && (s == 1 || s <= nb / 2); ++s) {
    const long rounds = ((long)B * nqt * s + n_cu - 1) / n_cu;
    const long cost = rounds * (6 + (nb + s - 1) / s) + (s > 1 ? 3 : 0);
    if (best.cost < 0 || cost < best.cost) best = Ranges{s, cost};
  }
  return best;
}
int flash_splits(int B, int nH, int H, int P, int n_cu) { return flash_ranges(B, nH, H, P, n_cu).S; }

template <int DH>
static hipError_t launch_flash_t(const AttnLaunch& a, int S, hipStream_t s) {
  // ceil(rows / 128) tiles per rollout, the rows spread evenly in whole 16-row wave tiles (400 rows: four
  // tiles of 112 instead of 128 + 128 + 128 + 16, so that the critical tiles keep seven waves busy)
  const int R = a.nH * a.H;
  const int nqt = (R + Flash<DH>::QT - 1) / Flash<DH>::QT;
  const int qrows = ((R + nqt - 1) / nqt + 15) / 16 * 16;
  const size_t rows = (size_t)a.B * a.nH * a.H;
  // partial outputs (bf16) then (max, sum) pairs, inside the opart scratch
  void* part = a.opart;
  float2* ml = reinterpret_cast<float2*>(reinterpret_cast<char*>(a.opart) + (size_t)S * rows * DH * 2);
  const int items = a.B * nqt * S;
  if (a.kvf && a.P > 0)
    JPI_LAUNCH((k_flash<DH, true>), dim3((items + 7) / 8 * 8), dim3(Flash<DH>::NW * 64), 0, s, a.ev_start,
               S == 1 ? a.ev_stop : (hipEvent_t) nullptr, a, S, nqt, qrows, part, ml);
  else
    JPI_LAUNCH((k_flash<DH, false>), dim3((items + 7) / 8 * 8), dim3(Flash<DH>::NW * 64), 0, s, a.ev_start,
               S == 1 ? a.ev_stop : (hipEvent_t) nullptr, a, S, nqt, qrows, part, ml);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || S == 1) return e;
  return a.out_f32 ? launch_merge<DH, float>(a, S, (const bf16*)part, ml, s) : launch_merge<DH, bf16>(a, S, (const bf16*)part, ml, s);
}

size_t flash_scratch_bytes(int B, int nH, int H, int Dh, int S) {
  return (size_t)S * B * nH * H * ((size_t)Dh * 2 + sizeof(float2));
}

hipError_t launch_flash(const AttnLaunch& a, int S, hipStream_t s) {
  if (S < 1 || S > FLASH_MAX_SPLITS || a.H < 1 || a.B < 1) return hipErrorInvalidValue;
  switch (a.Dh) {
    case 64: return launch_flash_t<64>(a, S, s);
    case 128: return launch_flash_t<128>(a, S, s);
    case 256: return launch_flash_t<256>(a, S, s);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Few query rows (the five-launch layers).  With one to eight rollouts the tiles of k_flash
// leave the chip idle or need many key ranges, and its ring pays a barrier and
// a memory round trip per 32-key block.  Here a workgroup takes 16 query rows and its
// four waves split the keys: a wave loads a whole 32-key block (K and V^T,
// 32 KiB at Dh 256) straight into registers, all at once, multiplies it, and takes the
// block 4 S further on; the waves' running outputs meet once in LDS.  No barrier
// inside the loop.  The keys come from their fragment-ordered blocks (KvBlock), so every
// load reads one contiguous KiB; gathered from the row-major K and V^T the same
// kernel ran at a third of that rate (batch 8: 29 us).  Every workgroup reads its range's keys
// from the XCD's L2, so this pays while B * (rows / 16) * keys stays small; from
// there k_flash, which shares each block between 112 rows, reads less.
// ---------------------------------------------------------------------------

constexpr int ROWS_NW = 4;  // waves of k_flash_rows

template <int DH>
__global__ __launch_bounds__(64 * ROWS_NW, 2) void k_flash_rows(AttnLaunch a, int S, int ntile, bf16* part, float2* ml) {
  using FS = Flash<DH>;
  using MF = Mfma<bf16>;
  constexpr int NST = FS::NST, NT = FS::NT, NW = ROWS_NW, KB = 32;
  __shared__ f32x4 red[NW][NT][64];
  __shared__ float2 mls[NW][16];
  // items (rollout, key range, tile), consecutive ones on one XCD: they share the range's keys
  const int item = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
  if (item >= a.B * ntile * S) return;
  const int b = item / (ntile * S), split = (item / ntile) % S, row0 = (item % ntile) * 16;
  const int H = a.H, R = a.nH * H;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, fr = lane & 15;
  const int nbs = (H + KB - 1) / KB;
  const bf16* act_base = reinterpret_cast<const bf16*>(a.skvf) + (size_t)b * nbs * KvBlock<DH>::ELEMS + lane * 8;
  const bf16* pre_base = reinterpret_cast<const bf16*>(a.kvf) + (size_t)b * a.kvf_bstride + lane * 8;
  MF::frag kf[2][NST];
  u32x4 vf[NT];
  // action blocks first, then the prefix
  auto block = [&](int jb) {
    return jb < nbs ? act_base + (size_t)jb * KvBlock<DH>::ELEMS : pre_base + (size_t)(jb - nbs) * KvBlock<DH>::ELEMS;
  };
  auto load_k = [&](const bf16* p) {
#pragma unroll
    for (int st = 0; st < NST; ++st)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) kf[kt][st] = MF::load(p + (kt * NST + st) * 512);
  };
  auto load_v = [&](const bf16* p) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) vf[nt] = *reinterpret_cast<const u32x4*>(p + (2 * NST + nt) * 512);
  };
  // the first block does not wait for prefix_len: any block below the bound P may be read (a rollout has
  // kv_blocks(P) of them, checked before the launch)
  const int jb0 = split * NW + w;
  MF::frag qf[NST];
  const bf16* qb = reinterpret_cast<const bf16*>(a.q) + ((size_t)b * R + min(row0 + fr, R - 1)) * DH + 8 * g;
#pragma unroll
  for (int st = 0; st < NST; ++st) qf[st] = MF::load(qb + st * 32);
  const bf16* p0 = block(min(jb0, nbs + (a.P + KB - 1) / KB - 1));
  load_k(p0);
  load_v(p0);
  __builtin_amdgcn_sched_barrier(0);
  const int pl = a.prefix_len ? a.prefix_len[b] : a.P;
  const int nb = nbs + (pl + KB - 1) / KB;
  const float qscale = 1.4426950408889634f / sqrtf((float)DH);
  f32x4 o[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) o[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_ref = -INFINITY, l = 0.f;

  for (int jb = jb0; jb < nb; jb += S * NW) {
    const bool act = jb < nbs;
    const int n_valid = min(act ? H - jb * KB : pl - (jb - nbs) * KB, KB);
    // the next block's K is requested as soon as this one's is multiplied, its V^T after P V: the
    // registers are free by then (the last turn reads its own block again)
    const bf16* next = block(jb + S * NW < nb ? jb + S * NW : jb);
    f32x4 sc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int st = 0; st < NST; ++st)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) sc[kt] = MF::run(kf[kt][st], qf[st], sc[kt]);
    __builtin_amdgcn_sched_barrier(0);
    load_k(next);
    __builtin_amdgcn_sched_barrier(0);
    if (n_valid < KB) {  // keys past the valid ones: score -inf, V zero (their memory may hold anything)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[kt][e] = 8 * g + 4 * kt + e < n_valid ? sc[kt][e] : -INFINITY;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) vf[nt] = mask8(vf[nt], n_valid - 8 * g);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int e = 0; e < 4; ++e) mx = fmaxf(mx, sc[kt][e]);
    mx = row4_max(mx) * qscale;  // -inf where every score is -inf or NaN (fmaxf drops a NaN)
    const bool over = mx > m_ref + FLASH_LIMIT;  // always on the first block with another score
    if (__any(over)) {
      const float f = over ? __builtin_amdgcn_exp2f(m_ref - mx) : 1.f;
      l *= f;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) o[nt] *= f;
      m_ref = over ? mx : m_ref;
    }
    MF::frag pb;
    float sum = 0.f;
    // a row without a reference yet: scores of -inf give 0 and NaN stays NaN, in the sum and in the output
    const float ref = m_ref == -INFINITY ? 0.f : m_ref;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bf16 lo = static_cast<bf16>(__builtin_amdgcn_exp2f(fmaf(sc[0][e], qscale, -ref)));
      const bf16 hi = static_cast<bf16>(__builtin_amdgcn_exp2f(fmaf(sc[1][e], qscale, -ref)));
      pb[e] = lo;
      pb[4 + e] = hi;
      sum += static_cast<float>(lo) + static_cast<float>(hi);
    }
    l += sum;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) o[nt] = MF::run(__builtin_bit_cast(MF::frag, vf[nt]), pb, o[nt]);
    __builtin_amdgcn_sched_barrier(0);
    load_v(next);
  }

  const int r = row0 + fr;
  if (split * NW >= nb) {  // a range without keys (S > 1), the same for every row: skipped by the merge
    if (w == 0 && g == 0 && r < R) ml[((size_t)split * a.B + b) * R + r] = float2{-INFINITY, 0.f};
    return;
  }
  // the waves' outputs against one reference per row: the largest.  Where there is none (every score of the
  // range -inf or NaN) the sum is 0 or NaN: with one range the quotient below is NaN, with several the merge decides.
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (g == 0) mls[w][fr] = float2{m_ref, l};
  __syncthreads();
  float m = -INFINITY, lsum = 0.f;
#pragma unroll
  for (int v = 0; v < NW; ++v) m = fmaxf(m, mls[v][fr].x);
#pragma unroll
  for (int v = 0; v < NW; ++v) {
    const float2 t = mls[v][fr];
    lsum += t.x == -INFINITY ? t.y : __builtin_amdgcn_exp2f(t.x - m) * t.y;
  }
  if (S > 1 && w == 0 && g == 0 && r < R) ml[((size_t)split * a.B + b) * R + r] = float2{m, lsum};
  const float f = (m_ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_ref - m)) / lsum;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) red[w][nt][lane] = o[nt] * f;
  __syncthreads();
  if (r >= R) return;
  const int hn = r / H, i = r - hn * H;
#pragma unroll
  for (int t = 0; t < (NT + NW - 1) / NW; ++t) {
    const int nt = w + NW * t;
    if (nt >= NT) break;
    f32x4 v = red[0][nt][lane];
#pragma unroll
    for (int u = 1; u < NW; ++u) v += red[u][nt][lane];
    if (S == 1 && a.out_f32) {
      *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + attn_out_at(a, DH, b * H + i, hn * DH + nt * 16 + 4 * g)) = v;
      continue;
    }
    const bf16x4_t p4 = bf16x4_t{static_cast<bf16>(v[0]), static_cast<bf16>(v[1]), static_cast<bf16>(v[2]), static_cast<bf16>(v[3])};
    bf16* dst = S == 1 ? reinterpret_cast<bf16*>(a.out) + attn_out_at(a, DH, b * H + i, hn * DH + nt * 16 + 4 * g)
                       : part + (((size_t)split * a.B + b) * R + r) * DH + nt * 16 + 4 * g;
    *reinterpret_cast<bf16x4_t*>(dst) = p4;
  }
}

// Key ranges per 16-row tile: the least estimated time (0.1 us; rounds of one workgroup per unit, each a start and the
// turns of its waves over 32-key blocks - a memory round trip and the block's bytes - and the merge with its launch).  A
// second workgroup on a unit costs almost a whole round, so ranges pay only while they fit one.  Measured with the merge
// (Dh 256, 8 heads of 50 rows, 816 tokens; 1, 2, 4, 8 ranges): one rollout 13.5, 12.3, 10.6, 10.2 us; two 13.2,
// 12.4, 10.7, 13.6; five 13.7, 13.6, 17.1; eight 13.4, 18.7.  With "enough for the chip" (three rollouts four
// ranges, eight two) batch 8 took 11.65 ms instead of 11.13 and batch 3 9.74 instead of 9.54.  Eight waves a
// workgroup and 32 rows a workgroup were slower throughout.
static Ranges rows_ranges(int B, int nH, int H, int P, int Dh, int n_cu) {
  const int ntile = (nH * H + 15) / 16, nb = kv_blocks(H) + kv_blocks(P);
  Ranges best{1, -1};
  for (int s = 1; s <= 8 && (s == 1 || 2 * s < nb); s *= 2) {
    const long rounds = ((long)B * ntile * s + n_cu - 1) / n_cu;
    const long cost = rounds * (52 + (6 + 6 * Dh / 256) * ((nb + ROWS_NW * s - 1) / (ROWS_NW * s))) + (s > 1 ? 35 : 0);
    if (best.cost < 0 || cost < best.cost) best = Ranges{s, cost};
  }
  return best;
}
int flash_rows_splits(int B, int nH, int H, int P, int Dh, int n_cu) { return rows_ranges(B, nH, H, P, Dh, n_cu).S; }

// Whether layers with this kernel are faster than the eight-launch layers with k_flash.  Every 16-row tile reads all
// of its rollout's keys (128 rows share them there), so many tiles over a long prefix are bound by those reads, about
// 16 TB/s from the L2s; k_flash's unit above is 0.3 + 0.9 Dh / 256 us, and the eight-launch layers cost about 18 us a
// layer more elsewhere.  Fitted to 240 shapes (Dh 64, 128, 256; 1 .. 50 rollouts, up to 500 rows; 256 .. 25600
// tokens), wrong by at most 6 %.  us a layer, these / those: Dh 256, 50 rows a rollout, 10 rollouts of 1600 tokens
// 70 / 87, of 4800 115 / 102, of 25600 357 / 217; 4 of 25600 198 / 120; 1 of 25600 61 / 106; Dh 128, 16 rows, 32 of
// 12800 152 / 103.
bool flash_rows_pays(int B, int nH, int H, int P, int Dh, int n_cu) {
  const double tiles = (double)B * ((nH * H + 15) / 16), nb = kv_blocks(H) + kv_blocks(P);
  const double reads = tiles * nb * kv_block_elems(Dh) * 2 / (16e6 * n_cu / 256);  // us
  const double rows = std::max(0.1 * (double)rows_ranges(B, nH, H, P, Dh, n_cu).cost, reads);
  return rows <= (0.3 + 0.9 * Dh / 256) * (double)flash_ranges(B, nH, H, P, n_cu).cost + 18.0;
}

template <int DH, typename TO>
static hipError_t launch_flash_rows_t(const AttnLaunch& a, int S, hipStream_t s) {
  const int ntile = (a.nH * a.H + 15) / 16, items = a.B * ntile * S;
  const size_t rows = (size_t)a.B * a.nH * a.H;
  bf16* part = reinterpret_cast<bf16*>(a.opart);
  float2* ml = reinterpret_cast<float2*>(part + (size_t)S * rows * DH);
  JPI_LAUNCH((k_flash_rows<DH>), dim3((items + 7) / 8 * 8), dim3(64 * ROWS_NW), 0, s, a.ev_start,
             S == 1 ? a.ev_stop : (hipEvent_t) nullptr, a, S, ntile, part, ml);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || S == 1) return e;
  return launch_merge<DH, TO>(a, S, part, ml, s);
}

hipError_t launch_flash_rows(const AttnLaunch& a, int S, hipStream_t s) {
  if ((S != 1 && S != 2 && S != 4 && S != 8) || a.H < 1 || a.B < 1) return hipErrorInvalidValue;
  if (a.P < 0 || (int64_t)(kv_blocks(a.P) * kv_block_elems(a.Dh)) > a.kvf_bstride) return hipErrorInvalidValue;
  switch (a.Dh) {
    case 64: return a.out_f32 ? launch_flash_rows_t<64, float>(a, S, s) : launch_flash_rows_t<64, bf16>(a, S, s);
    case 128: return a.out_f32 ? launch_flash_rows_t<128, float>(a, S, s) : launch_flash_rows_t<128, bf16>(a, S, s);
    case 256: return a.out_f32 ? launch_flash_rows_t<256, float>(a, S, s) : launch_flash_rows_t<256, bf16>(a, S, s);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Prefix hand-off: one workgroup per (32-key block, rollout, layer) reads the
// caller's K and V once and writes the resident K and V (unless they are the
// caller's), the transposed V and, for the bf16 kernels that take them, the
// fragment-ordered block.  One launch instead of two strided copies and a
// transpose per layer: batch 8, 816 tokens, 18 layers 316 us before.
// ---------------------------------------------------------------------------
template <typename T, int DH>
__global__ __launch_bounds__(256) void k_bind(BindLaunch a) {
  constexpr int VEC = 16 / sizeof(T), CPR = DH / VEC, LD = DH + (sizeof(T) == 2 ? 2 : 1);
  __shared__ T vt[32 * LD];
  const int key0 = blockIdx.x * 32, b = blockIdx.y, l = blockIdx.z, tid = threadIdx.x;
  const size_t src = ((size_t)l * a.B + b) * a.P, dst = ((size_t)l * a.Bmax + b) * a.Pmax;
  const bool in_place = a.in_place;
  // the caller's K and V may start at any element
  typedef u32x4 __attribute__((aligned(2))) piece;
  const T* k = reinterpret_cast<const T*>(a.k) + (in_place ? dst : src) * DH;
  const T* v = reinterpret_cast<const T*>(a.v) + (in_place ? dst : src) * DH;
  T* kp = reinterpret_cast<T*>(a.kp) + dst * DH;
  T* vp = reinterpret_cast<T*>(a.vp) + dst * DH;
  T* vpt = reinterpret_cast<T*>(a.vpt) + ((size_t)l * a.Bmax + b) * DH * a.Ppad;
  T* blk = a.kvf ? reinterpret_cast<T*>(a.kvf) + (((size_t)l * a.Bmax + b) * a.NBmax + blockIdx.x) * KvBlock<DH>::ELEMS : nullptr;
  const u32x4 zero = u32x4{0, 0, 0, 0};
#pragma unroll
  for (int e = tid; e < 32 * CPR; e += 256) {
    // fragment order: chunk c of key kk; lanes of a wave cover 16 keys x 4 chunks
    const int f = e / 64, ln = e % 64;
    const int kt = f / (CPR / 4), c = (f % (CPR / 4)) * 4 + (ln >> 4), row = ln & 15;
    const int kk = 8 * (row >> 2) + 4 * kt + (row & 3), key = key0 + kk;
    const bool ok = key < a.P;
    const u32x4 x = ok ? *reinterpret_cast<const piece*>(k + (size_t)key * DH + c * VEC) : zero;
    const u32x4 y = ok ? *reinterpret_cast<const piece*>(v + (size_t)key * DH + c * VEC) : zero;
    if (ok && !in_place) {
      *reinterpret_cast<u32x4*>(kp + (size_t)key * DH + c * VEC) = x;
      *reinterpret_cast<u32x4*>(vp + (size_t)key * DH + c * VEC) = y;
    }
    if constexpr (sizeof(T) == 2)
      if (blk) *reinterpret_cast<u32x4*>(blk + (size_t)e * 8) = x;  // e is the piece's place: (kt, k step, lane)
    T tmp[VEC];
    __builtin_memcpy(tmp, &y, 16);
#pragma unroll
    for (int i = 0; i < VEC; ++i) vt[kk * LD + c * VEC + i] = tmp[i];
  }
  __syncthreads();
  // V^T pieces of VEC keys: dim d, keys key0 + VEC q ..
  constexpr int Q = 32 / VEC;
#pragma unroll
  for (int e = tid; e < DH * Q; e += 256) {
    const int d = sizeof(T) == 2 ? (e >> 6) * 16 + (e & 15) : e / Q, q = sizeof(T) == 2 ? (e & 63) >> 4 : e % Q;
    T tmp[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) tmp[i] = vt[(VEC * q + i) * LD + d];
    u32x4 x;
    __builtin_memcpy(&x, tmp, 16);
    if (key0 + VEC * q < a.P) *reinterpret_cast<u32x4*>(vpt + (size_t)d * a.Ppad + key0 + VEC * q) = x;
    if constexpr (sizeof(T) == 2)
      if (blk) *reinterpret_cast<u32x4*>(blk + KvBlock<DH>::V + (size_t)e * 8) = x;
  }
}

// The fragment-ordered blocks from the resident K and V^T (after a producer that wrote those).
template <int DH>
__global__ __launch_bounds__(256) void k_kv_blocks(BindLaunch a) {
  const int key0 = blockIdx.x * 32, b = blockIdx.y, l = blockIdx.z;
  const size_t lb = (size_t)l * a.Bmax + b;
  const bf16* kp = reinterpret_cast<const bf16*>(a.kp) + lb * a.Pmax * DH;
  const bf16* vpt = reinterpret_cast<const bf16*>(a.vpt) + lb * DH * a.Ppad;
  bf16* blk = reinterpret_cast<bf16*>(a.kvf) + (lb * a.NBmax + blockIdx.x) * KvBlock<DH>::ELEMS;
  const u32x4 zero = u32x4{0, 0, 0, 0};
#pragma unroll
  for (int e = threadIdx.x; e < 32 * DH / 8; e += 256) {
    const int f = e / 64, ln = e % 64, kt = f / (DH / 32), c = (f % (DH / 32)) * 4 + (ln >> 4), row = ln & 15;
    const int key = key0 + 8 * (row >> 2) + 4 * kt + (row & 3), d = f * 16 + row, kv = key0 + 8 * (ln >> 4);
    *reinterpret_cast<u32x4*>(blk + (size_t)e * 8) = key < a.P ? *reinterpret_cast<const u32x4*>(kp + (size_t)key * DH + c * 8) : zero;
    *reinterpret_cast<u32x4*>(blk + KvBlock<DH>::V + (size_t)e * 8) =
        kv < a.P ? *reinterpret_cast<const u32x4*>(vpt + (size_t)d * a.Ppad + kv) : zero;
  }
}

size_t kv_block_elems(int Dh) { return (size_t)64 * Dh; }

hipError_t launch_bind(jpi_dtype dt, const BindLaunch& a, hipStream_t s) {
  if (a.P < 1 || a.B < 1 || a.L < 1) return hipSuccess;
  const dim3 grid((a.P + 31) / 32, a.B, a.L);
#define BIND_DH(DH)                                                                              \
  do {                                                                                           \
    if (dt == JPI_BF16) hipLaunchKernelGGL((k_bind<bf16, DH>), grid, dim3(256), 0, s, a);        \
    else hipLaunchKernelGGL((k_bind<float, DH>), grid, dim3(256), 0, s, a);                      \
  } while (0)
  switch (a.Dh) {
    case 64: BIND_DH(64); break;
    case 128: BIND_DH(128); break;
    case 256: BIND_DH(256); break;
    default: return hipErrorInvalidValue;
  }
#undef BIND_DH
  return hipGetLastError();
}

hipError_t launch_kv_blocks(const BindLaunch& a, hipStream_t s) {
  if (a.P < 1 || a.B < 1 || a.L < 1) return hipSuccess;
  const dim3 grid((a.P + 31) / 32, a.B, a.L);
  switch (a.Dh) {
    case 64: hipLaunchKernelGGL(k_kv_blocks<64>, grid, dim3(256), 0, s, a); break;
    case 128: hipLaunchKernelGGL(k_kv_blocks<128>, grid, dim3(256), 0, s, a); break;
    case 256: hipLaunchKernelGGL(k_kv_blocks<256>, grid, dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace jpi
