// Whole-number helpers of the refinement that need no device: constexpr, so
// that kernels call them as they are and the host can check them with a
// sanitizer.
#pragma once

#include <cstdint>

namespace polymh {

// A vertex as a whole number that falls along an edge that points down, or is
// horizontal and points right: the edges whose tie-break threshold
// (p_edge_threshold) is negative.  Any x and y.
constexpr int64_t down_right_key(int32_t x, int32_t y)
{
    return (int64_t)(((uint64_t)(uint32_t)y << 32) | (0x7fffffffu - (uint32_t)x));
}

// Edge pairs of two rings of any size.
constexpr int64_t edge_pairs(int32_t n, int32_t m) { return (int64_t)n * m; }

}  // namespace polymh
