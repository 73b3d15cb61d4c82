// Device front end (frontend.hip): series -> normalised spectrum.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "fft_batch.hpp"
#include "fft_radix.hpp"

namespace fdas {

// How an M-point transform is split: one transform of length N1 (N2 == 1),
// or the four-step N1 x N2 with both lengths compiled.
struct FrontendGeom {
  int64_t M;
  int N1, N2;
  const FftVariant *f1;  // the one transform when N2 == 1
  const c32 *tw1, *tw2;  // twiddle tables of lengths N1 and N2: W_N1^j, or with
                         // N2 > 1 the stage tables of both
};

size_t frontend_sel_bytes();
// The twiddles of the n-point transforms of an M-point one in the order their
// stages read them: for each stage, factor k of suffix mi at (k - 1) S + mi, so
// that consecutive threads read consecutive entries. (Picked out of W_n^j one
// load of a wave touches up to 60 lines.) At most n factors; those of short
// series come with their rounding errors, two entries each.
constexpr int kStageTableEntries = 2;
hipError_t launch_stage_table(c32 *out, int n, int64_t M, hipStream_t s);
hipError_t launch_frontend(const FrontendGeom &g, const float *series, c32 *spectrum, c32 *work,
                           float *pw, void *sel, float *stats, hipStream_t s);

}  // namespace fdas
