// Detection epilogue of the matrix-core kernels: the offers of one lane's
// four consecutive outputs, out of line.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "ols_variants.hpp"

namespace fdas {

// The offers of a lane's four consecutive outputs, the first of them kept
// output `o` of the block's segment (plane column r0 + o, powers v), out of
// line: the wave calls it together, and only when one of its lanes has a power
// at or above the threshold, so the registers the offers need are not held
// across a template loop (the caller's live registers are saved around the
// call, on that rare path).
typedef float cand_f4 __attribute__((ext_vector_type(4)));
static __device__ __attribute__((noinline)) void offer4(CandOut cd, CandLds *lds, cand_f4 v, int o,
                                                        int nkeep, int64_t r0, int row) {
  const float p[4] = {v[0], v[1], v[2], v[3]};
  cand_offer(cd, lds, row, p, [&](int i) { return o + i; }, nkeep, 0, r0);
}

}  // namespace fdas
