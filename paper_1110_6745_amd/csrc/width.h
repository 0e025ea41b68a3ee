// Internal declarations of the width pass (not part of the C ABI).
#pragma once

#include "okpz_internal.h"

namespace okpz {

// Width, through `rows` scratch (width_scratch_words(Ly) int64): out[0..3] = {S1' lo, S1' hi,
// S2' lo, S2' hi} (128-bit two's complement halves of the sums relative to H0),
// out[4] = *h0, and with t >= 0 out[-1] = t.  out may be host memory that the
// device can write.
hipError_t launch_width(const LatticeView &v, int64_t *rows, const int64_t *h0, int64_t *out, int64_t t,
                        hipStream_t st);

size_t width_scratch_words(int64_t Ly);

}  // namespace okpz
