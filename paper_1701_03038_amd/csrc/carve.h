// Byte offsets of a workgroup's arrays in its state memory (LDS or a slot of
// global memory), for the kernels that lay them out and the host code that
// sizes them.  Plain constexpr functions: 64-bit arrays start at multiples of
// 8, which 64-bit LDS accesses are compiled for.
#pragma once

#include <cstddef>
#include <cstdint>

namespace wfst {

// forward_sweep: two vectors of Q + 1 floats, the step's segment values and
// chunk values (FP64), and the segments' keys.
struct LseCarve {
    size_t vval, part, vkey, end;
};
constexpr LseCarve lse_carve(int64_t Q, int64_t max_segs, int64_t max_slots)
{
    const size_t segs = (size_t)(max_segs > 1 ? max_segs : 1), slots = (size_t)(max_slots > 1 ? max_slots : 1);
    const size_t vval = 2 * (size_t)(Q + 1) * 4;  // a multiple of 8
    const size_t part = vval + segs * 8, vkey = part + slots * 8;
    return LseCarve{vval, part, vkey, vkey + segs * 4};
}

// rest_backward: the same, then the chunks' sums (part holds their maxima) and
// three sets of Q + 1 state marks.
struct RestCarve {
    LseCarve lse;
    size_t part_s, marks, end;
};
constexpr RestCarve rest_carve(int64_t Q, int64_t max_segs, int64_t max_slots)
{
    const LseCarve l = lse_carve(Q, max_segs, max_slots);
    const size_t slots = (size_t)(max_slots > 1 ? max_slots : 1), marks = l.end + slots * 4;
    return RestCarve{l, l.end, marks, marks + 3 * (size_t)(Q + 1)};
}

}  // namespace wfst
