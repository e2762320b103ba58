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

// Columns of the buffer z for every row: the GeGLU output (F) and, in the
// action-time variant, the action-time MLP's swish output (W).
inline size_t z_columns(size_t W, size_t F, bool action_time) { return action_time && W > F ? W : F; }

}  // namespace jpi

#endif
