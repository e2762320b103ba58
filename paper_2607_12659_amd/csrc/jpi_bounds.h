// Sizes that kernels rely on and that the host allocates by: plain C++, so
// that the arithmetic can be checked without a GPU (tests/test_bounds_cpu.py).
#ifndef JPI_BOUNDS_H_
#define JPI_BOUNDS_H_

#include <cstddef>

namespace jpi {

// Columns of the buffer z for every row: the GeGLU output (F) and, in the
// action-time variant, the action-time MLP's swish output (W).
inline size_t z_columns(size_t W, size_t F, bool action_time) { return action_time && W > F ? W : F; }

}  // namespace jpi

#endif
