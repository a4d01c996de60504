// Pivot rule of the binary searches (Section IV, Algorithm 1), shared by
// the device kernels and the host code that builds the LDS tile.  Plain
// C++ so that a CPU test can check it at the largest text length.
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#define SAMATCH_HD __host__ __device__
#else
#define SAMATCH_HD
#endif

namespace samatch {

// Row halfway through the open range (L, R), -1 <= L < R <= 2^31 - 1.  The
// paper's (L + R) / 2 overflows 32 bits near n = 2^31, and so does R - L
// in signed arithmetic (L = -1, R = 2^31 - 1); the difference is taken in
// unsigned arithmetic, where it always fits, and half of it keeps L + d
// within [L, R].
SAMATCH_HD inline int midpoint(int L, int R) {
    return L + (int)(((uint32_t)R - (uint32_t)L) >> 1);
}

// Row that lane `lane` (0..63) of a wave looks at in the rows [lo, hi), which
// the wave narrows down together, lo < hi <= 2^31 - 1: every row when there
// are at most 64 (a result of hi or more: none for this lane), else the
// (lane + 1)-th of 64 evenly spaced ones.  Rows and their sums are
// unsigned: lo + lane passes 2^31 near the end of the longest texts.
SAMATCH_HD inline uint32_t wave_probe_row(uint32_t lo, uint32_t hi, int lane) {
    const uint32_t rows = hi - lo;
    if (rows <= 64) return lo + (uint32_t)lane;
    const uint32_t share = 0xFFFFFFFFu / 65u * (uint32_t)(lane + 1);  // of the rows, times 2^32
    return lo + (uint32_t)(((uint64_t)rows * share) >> 32);
}

}  // namespace samatch
