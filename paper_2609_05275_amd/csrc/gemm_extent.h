// Extents of the buffer descriptors through which the 256-wide GEMM tiles read
// their operands, in bytes from a tile's first row (bf16 elements).  Plain C++,
// so that host code can check them.
#pragma once

#include <stdint.h>

namespace ld {

// k-contiguous operand X[r * ld + k], rows r0..R-1: whole rows (k past the end
// of the last one is cut off by the loads' own test).
constexpr int64_t kc_extent(int64_t R, int64_t r0, int64_t ld) { return (R - r0) * ld * 2; }

// mn-contiguous operand X[k * ld + r], K k rows of R elements each: up to the
// last row's last element.  A tile fetches 256 elements of every k row; with
// ld > R (a column slice of a wider matrix) those past R in the last row may lie
// outside the matrix the slice was taken from.  What is left from k row k0 on
// (none, or a negative number, from K on) is one subtraction of the offset the
// tile's base needs anyway: worked out from K - k0 at each load, it cost the
// backward GEMMs 6-8%.
constexpr int64_t mc_extent(int64_t K, int64_t R, int64_t ld) { return K > 0 ? ((K - 1) * ld + R) * 2 : 0; }
constexpr int64_t mc_offset(int64_t k0, int64_t ld) { return k0 * ld * 2; }

}  // namespace ld
