// Sizes that kernels rely on and that the host allocates by: plain C++, so
// that the arithmetic can be checked without a GPU (tests/test_bounds_cpu.py).
#ifndef JPI_BOUNDS_H_
#define JPI_BOUNDS_H_

#include <cstddef>

namespace jpi {

// KvBlocks (32 keys each) that hold `keys` keys.
inline int kv_blocks(int keys) { return (keys + 31) / 32; }

// Most keys a rollout's rows can find in its prefix slots: the bound prefix and,
// in the action-time variant, the state token in slot prefix_len.  That slot is
// below max_prefix for every binding that is accepted, so the bound is too:
// kernels may touch any block below kv_blocks(bound) before they know prefix_len.
inline int key_bound(int prefix, int max_prefix, bool state_slot) {
  return state_slot && prefix < max_prefix ? prefix + 1 : prefix;
}

// K slices of the correction module's product of the VLM tokens' keys and values
// (M tokens, N = 2 Dh columns; d_VLM is a multiple of 256, so four slices are
// whole 64-deep steps).  By its 64 x 64 tiles T: the slices fill the chip where
// T does not and cost their write and read where it does.  A refresh (us) with
// 1 / 2 / 4 slices on 256 units: 816 tokens (T = 52) 112 / 111 / 111, 4 x 816
// (204) 120 / 124 / 119, 4 x 1600 (400) 130 / 123 / 123, 8 x 1600 (800)
// 148 / 138 / 144, 16 x 1600 (1600) 159 / 163 / 206, 48 x 1600 323 / 347 / 407.
inline int xkv_slices(int M, int N, int n_cu) {
  const long tiles = (long)((M + 63) / 64) * ((N + 63) / 64);
  if (M <= 64 || tiles > 4l * n_cu) return 1;
  return tiles > n_cu ? 2 : 4;
}

// Floats that those slices take for any number of tokens up to Mmax: at most
// two slices of 4 n_cu tiles.
inline size_t xkv_slice_elems(size_t Mmax, int N, int n_cu) {
  const size_t all = 4 * Mmax * N, most = (size_t)2 * 4 * n_cu * 64 * 64;
  return all < most ? all : most;
}

// Columns of the buffer z for every row: the GeGLU output (F) and, in the
// action-time variant, the action-time MLP's swish output (W).
inline size_t z_columns(size_t W, size_t F, bool action_time) { return action_time && W > F ? W : F; }

}  // namespace jpi

#endif
