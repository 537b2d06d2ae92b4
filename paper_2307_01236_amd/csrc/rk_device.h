// rk_device.h -- device helpers shared by the fill kernels.
#pragma once

#include <type_traits>

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

// Maximum of a 32-bit value over the 64 lanes of a wavefront (all lanes active): DPP
// exchanges inside each row of 16 lanes, then the four row maxima read as scalars.
__device__ inline uint32_t wave_max_u32(uint32_t v)
{
    v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, false));   // quad_perm 1,0,3,2
    v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, false));   // quad_perm 2,3,0,1
    v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x124, 0xf, 0xf, false));  // row_ror 4
    v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, false));  // row_ror 8
    const uint32_t r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
    const uint32_t r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
    return max(max(r0, r1), max(r2, r3));
}

// Calls f(integral_constant<int, U>) for U = B .. E-1 in order: a loop unrolled by
// construction, whose index is a compile-time constant in the body.
template <int B, int E, typename F>
__device__ inline void static_for(F &&f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// load at a byte offset from a wave-uniform base (one scalar base + one 32-bit lane offset)
__device__ inline int32_t ldb(const int32_t *base, uint32_t byte_off)
{
    return *(const int32_t *)((const char *)base + byte_off);
}

// A store marked nontemporal: its line is the first the caches let go.  The finalize writes
// several rows per cell that only later launches read, most of them on other XCDs; with
// these stores so marked the fill measured 0.13 ms faster (0.33 ms with the saving sweep),
// the products and mids included, which keep more of their operands in L2.
__device__ inline void st_nt(int32_t v, int32_t *p) { __builtin_nontemporal_store(v, p); }

}  // namespace rk
