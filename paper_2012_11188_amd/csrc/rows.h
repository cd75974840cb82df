// Where the kernels' reads of a row go, also of a row that is shorter than its
// readers or empty. Graphs are not checked unless SCAN_VALIDATE asks for it, so
// a vertex without neighbours of its own may still be met as one; what comes
// out for such a graph is not defined, but every read stays inside its arrays.
// Plain functions, so that they can be checked without a GPU.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define SCAN_ROWS_FN __host__ __device__ __forceinline__
#else
#define SCAN_ROWS_FN static inline
#endif

namespace scan {

// First slot of a row that starts at `off`; an empty one (which may start
// where the slots end) stands at slot 0.
SCAN_ROWS_FN int64_t row_start(int64_t off, int32_t deg) { return deg > 0 ? off : 0; }

// Position p >= 0 of a row; past its end its last one (0 where it has none).
// (In this form one instruction, the middle of three, after the subtraction.)
SCAN_ROWS_FN int32_t row_position(int32_t p, int32_t deg) {
  const int32_t q = p < deg - 1 ? p : deg - 1;
  return q > 0 ? q : 0;
}

// The number of a vertex among the `used` ones with neighbours, from the count
// of those before it. One without (met as a neighbour all the same) may have
// them all before it; its number stays below `used` too, as the id windows and
// the bitmap reach no further.
SCAN_ROWS_FN int32_t used_number(int64_t before, int32_t used) {
  return (int32_t)(before < used ? before : used - 1);
}

}  // namespace scan
