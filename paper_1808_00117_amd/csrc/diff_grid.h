// Grid of the diff kernel.  Host code without HIP, so that it can be checked on
// any machine.
#pragma once
#include <stdint.h>

namespace crum {

// Largest value of CRUM_PARAM_DIFF_BLOCKS, and its default: a wave for every unit
// up to 16 GiB of 4 KiB units, 64 GiB of 16 KiB ones.
constexpr uint32_t kDiffBlocksMax = 1u << 20;

// A launch holds fewer than 2^32 work-items along a dimension: with 256 a
// workgroup, at most this many.  The waves stride, so a smaller grid does the
// same work.
constexpr uint64_t kGridMax = (1ull << 24) - 1;

// Workgroups of four waves for `units` diff units, `group` consecutive ones a wave,
// in a grid of at most `blocks`.
inline uint32_t diff_grid(uint64_t units, uint32_t group, uint32_t blocks)
{
    const uint64_t waves = units / group + (units % group != 0);
    const uint64_t need = waves / 4 + (waves % 4 != 0);
    const uint64_t most = blocks < kGridMax ? blocks : kGridMax;
    return (uint32_t)(need < most ? need : most);
}

}  // namespace crum
