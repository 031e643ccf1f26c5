// Router logits on the matrix cores: operand types shared by the stand-alone gate kernel and the kernel that routes in the same
// launch, and the latter's product: one unit of four waves multiplies RT x 16 token rows by CT x 16 router columns, the waves taking the
// contraction in turns (wave w: chunks w, w + 4, ...).  Operands go straight from global memory into the MFMA layout: a
// lane reads 32 contiguous bytes of its row, four lanes a full 128-byte line.  A chunk is 64 elements of a 16-bit type
// (two v_mfma_f32_16x16x32) or 32 floats (eight v_mfma_f32_16x16x4_f32).  The four partial sums are added in wave order by
// whoever holds them, so every kernel gives the same bits for a token.
#pragma once

#include "smile_internal.hpp"

namespace smile {

namespace {

constexpr int kGateWaves = 4;   // waves of a unit: K-split factor

// DT: SMILE_DTYPE_*
template <int DT>
struct GateType;

template <typename E>
struct GateHalf {
    typedef E elem;
    typedef typename Half<E>::vec8 vec;
    static constexpr int kChunk = 64;
    __device__ static __forceinline__ mfma_f32x4 mfma(vec a, vec b, mfma_f32x4 c) { return Half<E>::mfma_16x16x32(a, b, c); }
};
template <>
struct GateType<SMILE_DTYPE_BF16> : GateHalf<__bf16> {};
template <>
struct GateType<SMILE_DTYPE_F16> : GateHalf<_Float16> {};
template <>
struct GateType<SMILE_DTYPE_F32> {
    typedef float elem;
    typedef mfma_f32x4 vec;
    static constexpr int kChunk = 32;
    __device__ static __forceinline__ mfma_f32x4 mfma(vec a, vec b, mfma_f32x4 c)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], c, 0, 0, 0);
        return c;
    }
};

// acc[rt][ct]: this wave's part of rows row0 + 16 rt .. + 15 (clamped to T) and router columns col0 + 16 ct .. + 15
// (inter, then intra; zero beyond n + m).  U: chunks in flight.  Element i of lane (kg = lane / 16, r = lane % 16) is row 4 kg + i, column r.
template <int DT, int CT, int RT, int U>
__device__ __forceinline__ void gate_partial(const void *x_, const void *w_inter_, const void *w_intra_, int row0, int T, int d,
                                             int n, int m, int col0, int wave, mfma_f32x4 (&acc)[RT][CT])
{
    typedef typename GateType<DT>::elem E;
    typedef typename GateType<DT>::vec vec;
    constexpr int kChunk = GateType<DT>::kChunk, kLane = kChunk / 4, kVec = kChunk / 8;   // elements per lane, per 16 bytes
    const E *x = static_cast<const E *>(x_), *w_inter = static_cast<const E *>(w_inter_), *w_intra = static_cast<const E *>(w_intra_);
    const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
    // rows of x as 32-bit offsets from the unit's first row, which is uniform (route_plan: 16 RT d <= 2^32)
    unsigned xoff[RT];
    const E *wrow[CT];
    x += (size_t)row0 * d;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) xoff[rt] = (unsigned)min(rt * 16 + r, T - 1 - row0) * d + kg * kLane;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const int c = col0 + ct * 16 + r;
        wrow[ct] = c < n ? w_inter + (size_t)c * d : (c < n + m ? w_intra + (size_t)(c - n) * d : nullptr);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt][ct] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int chunks = (d + kChunk - 1) / kChunk;
    for (int c0 = wave; c0 < chunks; c0 += kGateWaves * U) {
        // the operands of U chunks are requested before the first is used
        vec a[U][2][RT], b[U][2][CT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // the contraction index may be visited in any order as long as both operands agree: lane group kg takes
            // kLane consecutive elements, half of them for each of the two steps
            const int c = c0 + u * kGateWaves, k = c * kChunk + kg * kLane;
            // 16-bit rows are whole chunks; a float row may end inside one (d is a multiple of 8)
            const bool in = c < chunks && (DT != SMILE_DTYPE_F32 || k < d);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    a[u][h][rt] = vec{};
                    if (in) a[u][h][rt] = *reinterpret_cast<const vec *>(x + xoff[rt] + (c * kChunk + h * kVec));
                }
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    b[u][h][ct] = vec{};
                    if (in && wrow[ct]) b[u][h][ct] = *reinterpret_cast<const vec *>(wrow[ct] + k + h * kVec);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c0 + u * kGateWaves >= chunks) break;   // uniform
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int h = 0; h < 2; ++h) acc[rt][ct] = GateType<DT>::mfma(a[u][h][rt], b[u][h][ct], acc[rt][ct]);
        }
    }
}

}  // namespace

}  // namespace smile
