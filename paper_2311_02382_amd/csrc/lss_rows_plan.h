// Which launches LayerNorm's backward takes, from sizes alone.  Plain C++ without a HIP header, so that a host program can go over the choice
// (tests/host/rows_plan_check.cpp).
#pragma once
#include <stdint.h>

namespace lss {

// Whether one launch makes dx, dgamma and dbeta (layernorm_bwd_short_kernel): the second of two waits for the first, 4 us whatever its size, but a
// column workgroup of the one launch walks all rows, whose bytes come from the last-level cache where they have just been written.
// 4700 launches between one that makes dy and one that reads dx, the whole sequence, one launch less two: up to 1024 columns -1.9 us up to 128 rows,
// -1.4 at 350, -0.8 at 540, -0.2 to -0.5 at 700, +0.1 at 800, +0.3 to +1.3 at 1024; wider rows, which the two launches take 1 us longer for, -1.7 to
// -1.0 up to a million elements.
inline bool layernorm_bwd_short(int64_t rows, int E) { return E <= 2048 && rows * E <= 1024 * 1024 && rows <= (E <= 1024 ? 720 : 1024); }

} // namespace lss
