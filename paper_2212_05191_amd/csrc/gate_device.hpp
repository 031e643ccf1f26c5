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

// Columns that gate_wide takes in its one pass, and the LDS it needs (two stages of one chunk of the weights).
typedef uint32_t gate_piece __attribute__((ext_vector_type(4)));   // 16 bytes
constexpr int kWideTiles = 9, kWideCols = 16 * kWideTiles, kWideLds = 2 * kWideCols * 128;

// The same product for 64 rows and up to kWideCols columns of a 16-bit type, by a workgroup of four waves, wave w for
// rows row0 + 16 w .. + 15: every wave walks all chunks, with one set of accumulators for each wave that would have had the chunk above,
// and adds the four in wave order, so the bits are the same.  What bounds wide routers is not the read of x but the latency of the
// operands: with the contraction split over the waves, 64 rows x 80 columns leave registers for one chunk in flight, 129 columns
// take a second pass over x, and every wave fetches its own weights in pieces of 16 bytes.  Here x is read once, two chunks ahead, straight to
// registers; the weights, loaded two chunks ahead too, pass through `stage`, which the four waves share, at one barrier a chunk.  The
// 144 accumulators and the loads in flight fill 246 registers; two workgroups share a CU.
// 32768 x 768 with 129 columns, 16-bit: 60 -> 32 us with the routing decision (50 MB of x: 1.6 TB/s), whole pass of 128 experts 470 -> 444.
// out[ct]: the logits of columns 16 ct + lane % 16, rows 4 (lane / 16) + i of the wave's.
template <int DT>
__device__ __forceinline__ void gate_wide(const void *x_, const void *w_inter_, const void *w_intra_, int row0, int T, int d, int n, int m,
                                          gate_piece *stage, mfma_f32x4 (&out)[kWideTiles])
{
    typedef typename GateType<DT>::elem E;
    typedef typename GateType<DT>::vec vec;
    constexpr int PIECES = kWideCols * 8, NW = (PIECES + 255) / 256;   // 16-byte pieces of a chunk; loads per thread
    static_assert(sizeof(E) == 2 && PIECES % 64 == 0, "whole waves load the weights");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, kg = lane >> 4, cols = n + m;
    const int chunks = d / 64;   // d is a multiple of 64 for the 16-bit types
    const E *xrow = static_cast<const E *>(x_) + (size_t)min(row0 + wave * 16 + r, T - 1) * d + kg * 16;
    const E *wsrc[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int q = tid + 256 * i, c = min(q >> 3, cols - 1);   // columns beyond the last repeat it; nobody reads their logits
        wsrc[i] = (c < n ? static_cast<const E *>(w_inter_) + (size_t)c * d : static_cast<const E *>(w_intra_) + (size_t)(c - n) * d) + (q & 7) * 8;
    }
    mfma_f32x4 acc[kGateWaves][kWideTiles];
#pragma unroll
    for (int p = 0; p < kGateWaves; ++p)
#pragma unroll
        for (int ct = 0; ct < kWideTiles; ++ct) acc[p][ct] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
    gate_piece w[2][NW];
    vec a[2][2];
    // unconditional (the last chunk again beyond the end), so that the compiler can count the loads in flight
    auto load = [&](int c_, gate_piece (&wc)[NW], vec (&ac)[2]) {
        const int c = min(c_, chunks - 1);
#pragma unroll
        for (int h = 0; h < 2; ++h) ac[h] = *reinterpret_cast<const vec *>(xrow + c * 64 + h * 8);
#pragma unroll
        for (int i = 0; i < NW; ++i) wc[i] = *reinterpret_cast<const gate_piece *>(wsrc[i] + c * 64);
    };
    load(0, w[0], a[0]);
    load(1, w[1], a[1]);
    for (int c0 = 0; c0 < chunks; c0 += kGateWaves) {
#pragma unroll
        for (int p = 0; p < kGateWaves; ++p) {
            const int c = c0 + p;
            if (c >= chunks) break;   // uniform
            gate_piece *at = stage + (p & 1) * PIECES;
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const int q = tid + 256 * i, row = q >> 3;
                if (256 * (i + 1) <= PIECES || q < PIECES) at[row * 8 + ((q & 7) ^ ((row >> 1) & 7))] = w[p & 1][i];
            }
            const vec ac[2] = {a[p & 1][0], a[p & 1][1]};
            load(c + 2, w[p & 1], a[p & 1]);
            // one barrier a chunk: a wave that passes it has read the other stage, which is written next, to the end
            __syncthreads();
#pragma unroll
            for (int ct = 0; ct < kWideTiles; ++ct)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int row = ct * 16 + r;
                    const vec b = __builtin_bit_cast(vec, at[row * 8 + ((kg * 2 + h) ^ ((row >> 1) & 7))]);
                    acc[p][ct] = GateType<DT>::mfma(ac[h], b, acc[p][ct]);
                }
        }
    }
#pragma unroll
    for (int ct = 0; ct < kWideTiles; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i) out[ct][i] = acc[0][ct][i] + acc[1][ct][i] + acc[2][ct][i] + acc[3][ct][i];
}

}  // namespace

}  // namespace smile
