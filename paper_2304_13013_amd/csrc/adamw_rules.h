// Size rules of the StableAdamW step: host arithmetic alone (no HIP in this file), so that they can be compiled and checked
// without a GPU.
#pragma once
#include <stdint.h>

namespace sb {

constexpr int kAdamwThreads = 256;
constexpr int kAdamwElementsPerBlock = kAdamwThreads * 4 * 4;  // four quads per lane before the grid stride matters
constexpr int kAdamwPartials = 2048;  // upper bound on the workgroups, and partial sums, of one tensor

// Workgroups of a tensor, in a step of its own and in a batched one.
inline int adamw_blocks(int64_t count) {
    const int64_t blocks = (count + kAdamwElementsPerBlock - 1) / kAdamwElementsPerBlock;
    return blocks < 1 ? 1 : blocks > kAdamwPartials ? kAdamwPartials : (int)blocks;
}

// Both passes are bound by memory.  While all of a step's arrays fit the 256 MiB last-level cache together, plain
// accesses in one direction serve the second pass (and the next step) from it.  Above that (STREAM) the second pass walks
// the workgroups backwards, so that it starts at the moments the first pass wrote last, and what only one pass touches
// (gradient, parameters) is accessed non-temporally, so that it does not push the moments out.  A transformer block's ten
// tensors, both passes, bf16 / binary32 gradients: width 2048 (0.7 / 0.8 GB) 338 / 356 us plain, 286 / 298 us streaming;
// width 1280 (275 / 315 MB) 107.7 / 112.6 and 104.8 / 110.7; width 768 (99 / 113 MB) 42.4 / 44.9 and 45.6 / 48.4.
// (Four quads per lane in flight at once, loads ahead of the partial sums: 6 % slower at width 1280, the same at 768.)
inline bool adamw_streams(int64_t elements, bool grad_bf16) {
    return elements * (12 + (grad_bf16 ? 2 : 4)) > (int64_t)256 << 20;
}

// The element counts of a batched step live in device memory.  Its host knows the tensors and their workgroups, which
// bound the sum from below: all workgroups of a tensor but its last are full.  Only that bound decides, so that a step
// that fits the cache never streams (5000 tensors of 256 elements, 20 MB, taken for 5000 whole workgroups: 21.7 / 26.4 us).
// A tensor of more than kAdamwPartials workgroups' elements (8.4 million) counts as that many: a batched step of a few
// such tensors may stay below the line although its arrays exceed the cache, and then runs as if they did not.
inline int64_t adamw_elements_at_least(int64_t total_blocks, int64_t n) {
    return (total_blocks - n) * kAdamwElementsPerBlock + n;
}

}  // namespace sb
