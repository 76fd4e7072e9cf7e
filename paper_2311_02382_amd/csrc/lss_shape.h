// One segment's problem, as host code and kernels see it.  Plain C++ without a HIP header, so that a host program can go over
// the rules that choose launches by it.
#pragma once
#include <stdint.h>

namespace lss {

// Eq. 2 of Section 3 for one segment (device pointers are passed beside it)
struct SegShape {
    int64_t s0;      // global index of the segment's first query row
    int l_s, l_x;    // query rows of the segment, key/value rows of the sequence
    int B, H, d;
    int causal;
    int skip_tail;   // causal backward: leave key tiles that no query of the segment sees unwritten (not zero-filled)
};

} // namespace lss
