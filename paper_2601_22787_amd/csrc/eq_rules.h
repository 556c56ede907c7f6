// Host rules that choose how a call is launched.  No device code, so that
// they can be checked without a GPU.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace eq_detail {

// Version 1, rows that are not whole steps: whether the GEMV decodes and
// multiplies in one kernel, or decodes to codes first and multiplies those, a
// block per row.  In the fused kernel every row that ends inside a chunk costs
// its wavefront some 0.1 to 0.5 us of its chain (more with more batch rows).
// That is hidden where compute units have several chunks each (fewer are
// enough for long rows, whose separate product has more to read) and small
// where a chunk holds few rows.  Both ways timed at 5340 points (65 to 11000
// columns, chunks of 1024 to 65536, 64 to 256 lanes, 4 to 16384 chunks, batch 1
// to 8): the rule's choice takes 1.01 times the faster one's time on average,
// 1.43 at worst (always the fused kernel: 1.17 at batch 1 to 1.60 at batch 8,
// 16 at worst; never: 1.61 to 1.29, 13 at worst).
inline bool ragged_fused(uint32_t n_chunks, uint32_t cols, uint32_t chunk_syms, uint32_t B,
                         uint32_t cus) {
  const double t = B == 1 ? 1.0 : B == 2 ? 1.25 : B <= 4 ? 2.0 : 3.0;
  return n_chunks * (1.0 + double(B) * cols / 8192.0) >= t * cus ||
         cols >= (B == 1 ? 0.25 : 0.4) * chunk_syms;
}

}  // namespace eq_detail
