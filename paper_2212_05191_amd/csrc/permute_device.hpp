// Row moves shared by the permutation and routing kernels: a row is d * elem bytes, moved as 16-byte pieces by LPR
// consecutive lanes, so that every access of those lanes is one contiguous run.
#pragma once

#include "smile_internal.hpp"

namespace smile {

namespace {

constexpr int kPieces = 4;   // loads in flight per lane

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

// Copy (or gate-scale) one row of ppr pieces, up to kPieces loads in flight per lane.  F maps a loaded piece to the stored one.
template <int LPR, typename F>
__device__ __forceinline__ void move_row(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, int ppr, int sub, F f)
{
    for (int c0 = sub; c0 < ppr; c0 += LPR * kPieces) {
        u32x4 v[kPieces];
#pragma unroll
        for (int i = 0; i < kPieces; ++i)
            if (c0 + i * LPR < ppr) v[i] = src[c0 + i * LPR];
#pragma unroll
        for (int i = 0; i < kPieces; ++i)
            if (c0 + i * LPR < ppr) dst[c0 + i * LPR] = f(v[i]);
    }
}

// zero one row by `lanes` lanes
__device__ __forceinline__ void zero_row(u32x4 *row, int ppr, int sub, int lanes)
{
    for (int c = sub; c < ppr; c += lanes) row[c] = u32x4{0u, 0u, 0u, 0u};
}

// lanes per row: the largest power of two <= min(ppr, 32), at least 8
inline int lanes_per_row(int ppr)
{
    int l = 8;
    while (l * 2 <= ppr && l < 32) l *= 2;
    return l;
}

}  // namespace

}  // namespace smile
