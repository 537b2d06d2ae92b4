// rk_device.h -- device helpers shared by the fill kernels.
#pragma once

#include "rk_internal.h"

namespace rk {

// ---------------------------------------------------------------------------------------
// Workgroups of a launch go to the 8 XCDs round-robin (id g to XCD g mod 8), and each XCD
// has its own L2.  Tiles are laid out as column chunks x n_idx tiles per chunk, and XCD x
// (g mod 8) takes the chunks x, x + 8, x + 16, ..., each with its n_idx tiles in order.
// Every XCD then keeps whole column chunks (tiles that share operand rows share its L2, at
// about the same time) and gets chunks from the whole budget range, so work that shrinks
// with the budget column (tiles past the store-everything budget) stays even over the
// XCDs.  Launches hold 8 ceil(n_chunks / 8) n_idx workgroups; *chunk >= n_chunks marks a
// spare one.  Correctness does not depend on the dispatch order.
// ---------------------------------------------------------------------------------------
__device__ inline void chunk_tile(uint32_t g, uint32_t n_idx, int32_t *chunk, int32_t *idx)
{
    const uint32_t j = g / 8;
    // scalars: the division is expanded with vector instructions, and without the hint
    // every address derived from the tile would be computed (and loaded) per lane
    *chunk = __builtin_amdgcn_readfirstlane((int32_t)(g % 8 + 8 * (j / n_idx)));
    *idx = __builtin_amdgcn_readfirstlane((int32_t)(j % n_idx));
}
static inline uint32_t chunk_grid(int32_t n_chunks, int32_t n_idx)
{
    return (uint32_t)(8 * ((n_chunks + 7) / 8) * n_idx);
}

// load at a byte offset from a wave-uniform base (one scalar base + one 32-bit lane offset)
__device__ inline int32_t ldb(const int32_t *base, uint32_t byte_off)
{
    return *(const int32_t *)((const char *)base + byte_off);
}

}  // namespace rk
