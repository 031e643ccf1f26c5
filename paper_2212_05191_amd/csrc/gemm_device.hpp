// Device-side pieces shared by the grouped expert GEMM kernels (HIP, gfx950): vector types, the activation
// functions of the epilogues and their derivatives, the kernel argument block, direct-to-LDS load helpers, the transposing LDS read and
// the LDS bank swizzle.
#pragma once

#include "smile_internal.hpp"

namespace smile {

// Arguments of the 16-bit grouped GEMM kernels (one block for every variant).
struct GemmArgs {
    const void *x;          // [N][C][K]; with x_rows: the token matrix [T][K]
    const void *w;          // [N][Nout][K]
    const void *bias;       // [N][Nout] or null
    void *y;                // [N][C][Nout], or null when only the scattered output is wanted
    const int32_t *kept;    // [N]
    int C, Nout, K;
    int row_tiles, col_tiles, tiles;   // tiles = N*row_tiles*col_tiles
    // Permutation fused into the GEMM (both optional, [N][C] token index of each buffer row):
    const int32_t *x_rows;  // gather: input row r of expert e is x[x_rows[e*C + r]]  (dispatch fused in)
    const int32_t *y_rows;  // scatter: output row also goes to y_tok[y_rows[e*C + r]] * gate  (combine fused in)
    void *y_tok;            // [T][Nout]
    const float *gate;      // [T]
    void *y2 = nullptr;     // [N][C][Nout]: the same product without the activation (DUAL kernels only)
    int N = 0;                   // experts (PERSIST kernels walk the live row tiles of all of them)
    bool backwards = false;      // ring kernels: walk the tiles from the last expert to the first
    int tokens = 0;              // T: rows of the gathered matrix, and what the experts' rows add up to at most (0: full buffers)
};

namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;

constexpr int kXcds = 8;

// ACT: 0 none, 1 ReLU, 2 GELU (erff; fp32 path), 3 GELU (rational erfc; 16-bit path)
template <int ACT>
__device__ __forceinline__ float activate(float v)
{
    if constexpr (ACT == 1) return v > 0.f ? v : 0.f;
    else if constexpr (ACT == 2) return 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
    else if constexpr (ACT == 3) {
        // GELU(v) = v * Phi(v) = max(v,0) - |v| * erfc(|v|/sqrt2)/2, with erfc from the rational
        // approximation 7.1.26 of Abramowitz & Stegun (|error| < 1.5e-7, far below bf16 resolution):
        // erfc(z) = (a1 t + ... + a5 t^5) exp(-z^2), t = 1/(1 + p z).  ~15 VALU ops, no branches.  The exponential is a factor, so
        // the tail keeps its relative accuracy as far as bf16 has values: 0.5 % at v = -6.5, 2 % at -10, 4 % at -13.  2^P(|v|) with one
        // polynomial P of degree 8 is one transcendental less (128 experts x 256 rows, 768 -> 3072: 492.7 -> 487.2 us a pass, the
        // base layer 122.6 -> 122.5), but is off by 10 % at -8 and by 90 % at -10.
        // A product that overflowed to infinity counts as the largest finite value, which rounds to infinity in 16 bits (infinity
        // times the tail's 0 would be NaN).  Medians instead of fmaxf and fminf, which the compiler gives a second instruction each
        // to quieten a signalling NaN: the clamp costs nothing over the plain form.
        const float av = fabsf(v);
        const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, av, 1.0f));
        float poly = fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
        poly = fmaf(poly, t, 0.5f * 1.421413741f);
        poly = fmaf(poly, t, 0.5f * -0.284496736f);
        poly = fmaf(poly, t, 0.5f * 0.254829592f);
        const float ex = __builtin_amdgcn_exp2f(v * v * (-0.5f * 1.4426950408889634f));
        float most;   // in a scalar register: the compiler would keep it in a vector register, of which the ring kernels have none to spare
        asm("s_mov_b32 %0, 0x7f7fffff" : "=s"(most));
        return __builtin_amdgcn_fmed3f(v, 0.f, most) - __builtin_amdgcn_fmed3f(av, 0.f, most) * (poly * t * ex);
    } else return v;
}

// ------------------------------------------------------------------------------------ bf16 / fp16: MFMA

// One 16-byte piece (8 elements) times a gate: fp32 product, rounded to the storage type (nearest even) --
// the same arithmetic as the stand-alone combine kernel.
template <typename E>
__device__ __forceinline__ u32x4 scale_x8(u32x4 v, float g)
{
    u32x4 r;
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = Half<E>::pack(Half<E>::lo(v[k]) * g, Half<E>::hi(v[k]) * g);
    return r;
}

#define SMILE_GPTR(p) ((const __attribute__((address_space(1))) void *)(p))
#define SMILE_LPTR(p) ((__attribute__((address_space(3))) void *)(p))

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);   // expcnt, lgkmcnt: no wait
}

// d/dv GELU(v) = Phi(v) + v phi(v) (POST 2), or the step function (POST 1); Phi from the rational erfc approximation 7.1.26 of
// Abramowitz & Stegun (|error| < 1.5e-7), phi sharing its exponential
template <int POST>
__device__ __forceinline__ float activate_grad(float v)
{
    if constexpr (POST == 1) return v > 0.f ? 1.f : 0.f;
    else {
        const float av = fabsf(v);
        const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, av, 1.0f));
        float poly = fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
        poly = fmaf(poly, t, 0.5f * 1.421413741f);
        poly = fmaf(poly, t, 0.5f * -0.284496736f);
        poly = fmaf(poly, t, 0.5f * 0.254829592f);
        const float ex = __builtin_amdgcn_exp2f(v * v * (-0.5f * 1.4426950408889634f));
        const float q = poly * t * ex;   // 1 - Phi(|v|)
        return fmaf(v * 0.3989422804014327f, ex, v >= 0.f ? 1.0f - q : q);
    }
}

typedef __attribute__((address_space(3))) char lds_char;

// The two transposing reads of one fragment, HALF bytes apart.  Unless the compiler knows that they do not touch what the
// global -> LDS loads in flight write, it waits for all of those before each read, which undoes the ring: restrict pointers for the
// stage read and the stage filled tell it.  Measured at 48 experts x 512 rows, 1600 x 6400, bf16, on the two-stage kernel:
// dxe 376 -> 261 us, dpre 303 -> 250, dW2 235 -> 227, dW1 254 -> 247.
template <int HALF, typename V>
__device__ __forceinline__ void read_transposed(V &f, const lds_char *at)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    struct { s16x4 lo, hi; } t;
    t.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)at);
    t.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(at + HALF));
    f = __builtin_bit_cast(V, t);
}

// source of k-rows beyond a ragged contraction length
__device__ __attribute__((aligned(16))) const uint32_t kZeroPiece[4] = {0u, 0u, 0u, 0u};

// Swizzle term of a row of 64 k (128 bytes): consecutive rows must land on different banks.
__device__ __forceinline__ int swz(int row)
{
    return (row >> 1) & 7;
}

}  // namespace

}  // namespace smile
