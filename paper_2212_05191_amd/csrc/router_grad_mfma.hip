// The two skinny products of the backward pass that involve the router weights, on the matrix cores (bf16 storage):
//
//   dx[t,:]   = dxe[row(t),:] + dlp[t,:] . W_p + dlq[t,:] . W_q           (chain rule through Eq. 1 of both levels)
//   dW_p[i,:] = sum_t dlp[t,i] x[t,:],   dW_q[j,:] = sum_t dlq[t,j] x[t,:]
//
// The logit gradients are fp32 and have to stay fp32-accurate, the weights and tokens are bf16.  An fp32 value is
// the exact sum of three bf16 values (8 + 8 + 8 mantissa bits: hi = bf16(v), mid = bf16(v - hi), lo = bf16(v - hi -
// mid)) and a bf16 x bf16 product is exact in the fp32 accumulator of v_mfma_f32_32x32x16_bf16, so three MFMAs per
// 16 logit columns give the fp32 product, at 1/20 of the vector-ALU time of the FMA formulation (which has to
// widen every bf16 weight for every token).
//
// MFMA operand layout used below (same as the expert GEMMs): for D = A . B, lane l supplies 8 consecutive k of
// row (l & 31) of A and of column (l & 31) of B, k-group l >> 5; accumulator element v of lane l is row
// 8*(v/4) + 4*(l>>5) + v%4, column l & 31 of D.
#include "smile_internal.hpp"

namespace smile {

namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef Half<__bf16>::vec8 bf16x8;

constexpr int kThreads = 256;

// v = hi + mid + lo exactly (up to 2^-24 relative), each representable in bf16
__device__ __forceinline__ void split3(float v, __bf16 &hi, __bf16 &mid, __bf16 &lo)
{
    hi = (__bf16)v;
    const float r1 = v - (float)hi;
    mid = (__bf16)r1;
    lo = (__bf16)(r1 - (float)mid);
}

// ------------------------------------------------------------------------------------ dx

// columns of d per workgroup: 256, or 128 when the transposed weights of 256 would leave room for one workgroup per CU
constexpr int dx_cols(int kc) { return kc <= 6 ? 256 : 128; }
constexpr int kDxTokens = 128;   // tokens per workgroup: 32 per wave
constexpr int kDxMaxChunks = 10; // 16-wide chunks of logit columns (inter, then intra) kept in registers

// Row i of an MFMA A tile holds weight column perm(i) of the 32-column tile, so that a lane's 16 accumulator
// elements are 16 CONSECUTIVE columns (16 * (lane >> 5) + v) of its token: two 16-byte pieces per tile.
__device__ __forceinline__ int perm_col(int i) { return 16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3); }

// Workgroup = 128 tokens x 256 (or 128) columns.  The weight rows of the column range are transposed into LDS once
// (wt[column][logit column], bf16); each wave splits the logit gradients of its 32 tokens into bf16 planes once
// (registers) and then walks the column range 64 columns at a time: 2*KC*3 MFMAs, add the expert-buffer row, round,
// store; rows are read and written whole (128 bytes of a row per 8 lanes), through a per-wave LDS tile.
struct DxArgs {
    const __bf16 *dxe;
    const int32_t *group_idx, *local_idx, *slot;
    const float *dlp, *dlq;
    const __bf16 *w_inter, *w_intra;
    __bf16 *dx;
    int T, d, n, m, C, kp;   // kp: 16-wide chunks of inter columns
};
template <int KC>
struct DxLds {
    static constexpr int kStride = KC * 16 + 8;   // row stride of the weights in elements (+8: bank spread, keeps 16-byte alignment)
    typedef __bf16 Weights[dx_cols(KC) * kStride] __attribute__((aligned(16)));
    typedef u32x4 Rows[kThreads / 64][32 * 9];     // per wave: 32 rows x 8 pieces (+1: bank spread)
};

template <int KC>
__device__ __forceinline__ void dispatch_backward_block(const DxArgs &args, typename DxLds<KC>::Weights &wt, typename DxLds<KC>::Rows &io, int token_block,
                                                        int col_block)
{
    constexpr int kDxCols = dx_cols(KC), RS = DxLds<KC>::kStride;
    const __bf16 *__restrict__ dxe = args.dxe, *__restrict__ w_inter = args.w_inter, *__restrict__ w_intra = args.w_intra;
    const int32_t *__restrict__ group_idx = args.group_idx, *__restrict__ local_idx = args.local_idx, *__restrict__ slot = args.slot;
    const float *__restrict__ dlp = args.dlp, *__restrict__ dlq = args.dlq;
    __bf16 *__restrict__ dx = args.dx;
    const int T = args.T, d = args.d, n = args.n, m = args.m, C = args.C, kp = args.kp;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c_base = col_block * kDxCols;

    // ---- weights of this column range, transposed: piece = 8 columns of one weight row
    for (int p = tid; p < KC * 16 * (kDxCols / 8); p += kThreads) {
        const int r = p / (kDxCols / 8), c8 = (p - r * (kDxCols / 8)) * 8;
        const int ri = r < kp * 16 ? r : r - kp * 16;                    // row inside its router
        const bool inter = r < kp * 16;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (c_base + c8 < d && ri < (inter ? n : m))
            v = *reinterpret_cast<const u32x4 *>((inter ? w_inter : w_intra) + (size_t)ri * d + c_base + c8);
        const __bf16 *e = reinterpret_cast<const __bf16 *>(&v);
#pragma unroll
        for (int j = 0; j < 8; ++j) wt[(c8 + j) * RS + r] = e[j];
    }

    // ---- logit gradients of this wave's tokens as bf16 planes: lane = (token lane & 31, k-group lane >> 5)
    const int t = token_block * kDxTokens + wave * 32 + (lane & 31), g = lane >> 5;
    const bool t_ok = t < T;
    bf16x8 plane[KC][3];
#pragma unroll
    for (int ch = 0; ch < KC; ++ch) {
        const bool inter = ch < kp;
        const int r0 = (inter ? ch : ch - kp) * 16 + 8 * g, cnt = inter ? n : m;
        const float *dl = inter ? dlp + (size_t)t * n : dlq + (size_t)t * m;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float v = (t_ok && r0 + j < cnt) ? dl[r0 + j] : 0.f;
            __bf16 hi, mid, lo;
            split3(v, hi, mid, lo);
            plane[ch][0][j] = hi, plane[ch][1][j] = mid, plane[ch][2][j] = lo;
        }
    }
    const int sl = t_ok ? slot[t] : -1;
    const __bf16 *src = sl >= 0 ? dxe + ((size_t)(group_idx[t] * m + local_idx[t]) * C + sl) * d : nullptr;

    // ---- memory side: 64 columns (128 bytes of a row) at a time, whole rows per instruction.  Lane = (row lane / 8 +
    // 8 it, 16-byte piece lane % 8) for it = 0..3; the rows' source pointers live in the lanes that own the tokens
    // and are fetched from there once.  The tile goes through a per-wave LDS buffer to the lanes that hold the
    // matching accumulators (token lane & 31, columns 32 u + 16 g + 8 h of the 64: piece 4 u + 2 g + h) and back.
    const int mrow = lane >> 3, mpiece = lane & 7;
    const __bf16 *msrc[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const unsigned long long p = reinterpret_cast<unsigned long long>(src);
        const unsigned lo = __shfl((unsigned)p, mrow + 8 * it, 64), hi = __shfl((unsigned)(p >> 32), mrow + 8 * it, 64);
        msrc[it] = reinterpret_cast<const __bf16 *>(((unsigned long long)hi << 32) | lo);
    }
    const int t_wave = token_block * kDxTokens + wave * 32;   // first token of the wave
    u32x4 *tile = io[wave];
    __syncthreads();

    const int arow = perm_col(lane & 31);
    u32x4 in[4];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            in[it] = u32x4{0u, 0u, 0u, 0u};
            if (msrc[it]) in[it] = *reinterpret_cast<const u32x4 *>(msrc[it] + c0 + mpiece * 8);
        }
    };
    if (c_base < d) fetch(c_base);
#pragma unroll 1
    for (int cs = 0; cs < kDxCols / 64; ++cs) {
        const int c0 = c_base + cs * 64;
        if (c0 >= d) break;   // uniform (d is a multiple of 64)
#pragma unroll
        for (int it = 0; it < 4; ++it) tile[(mrow + 8 * it) * 9 + mpiece] = in[it];
        if (c0 + 64 < d && cs + 1 < kDxCols / 64) fetch(c0 + 64);   // in flight during the MFMAs
        f32x16 acc[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[u][v] = 0.f;
#pragma unroll
            for (int ch = 0; ch < KC; ++ch) {
                const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&wt[(cs * 64 + u * 32 + arow) * RS + ch * 16 + 8 * g]);
#pragma unroll
                for (int p = 0; p < 3; ++p) acc[u] = Half<__bf16>::mfma_32x32x16(a, plane[ch][p], acc[u]);
            }
        }
        // lane holds columns c0 + 32 u + 16 g + 0..15 of token (lane & 31): add the expert-buffer row, round once
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x4 *cell = &tile[(lane & 31) * 9 + 4 * u + 2 * g + h];
                const u32x4 v = *cell;
                u32x4 o;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    o[k] = Half<__bf16>::pack(Half<__bf16>::lo(v[k]) + acc[u][8 * h + 2 * k],
                                              Half<__bf16>::hi(v[k]) + acc[u][8 * h + 2 * k + 1]);
                *cell = o;
            }
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int row = mrow + 8 * it;
            const u32x4 o = tile[row * 9 + mpiece];
            if (t_wave + row < T) *reinterpret_cast<u32x4 *>(dx + (size_t)(t_wave + row) * d + c0 + mpiece * 8) = o;
        }
    }
}

// ------------------------------------------------------------------------------------ dW_p, dW_q

constexpr int kGwCb = 256;         // columns of x per workgroup
constexpr int kGwMaxRowTiles = 5;  // 32-wide tiles of logit columns (inter and intra concatenated)
typedef short s16x4 __attribute__((ext_vector_type(4)));

// partial[b][r][c] = sum over the tokens of block b of dl[t][r] * x[t][c], r over the n + m logit columns (dlp first,
// then dlq).  D = A . B with A = x^T (row = column c of x, k = token) and B = the bf16 planes of dl (column = logit
// column r, k = token).  Both are stored token-major, i.e. with k as the slow index:
//   * the x tile (64 tokens x 256 columns) is written to LDS as it is in memory and its fragments are fetched with
//     the transposing LDS read (ds_read_b64_tr_b16: within 16 lanes, lane 4a+b receives element b of the 8-byte
//     rows addressed by lanes a, a+4, a+8, a+12; so lane i addresses token i/4 and the 4-column block i%4 and ends
//     up with 4 consecutive tokens of its own column).  A token row's 16-byte pieces are rotated by 4*(token&3)
//     positions so that the 8 token rows a wave touches per read spread over all banks;
//   * the planes are written transposed, pl[plane][r][token], by the threads that split the values.
// The next tile's global loads are in flight while the current one is multiplied.  Tokens are summed in a fixed
// order and the blocks are added by the reduce kernel in index order: deterministic.
struct GwArgs {
    const __bf16 *x;
    const float *dlp, *dlq;
    float *partial;
    int T, d, n, m, tokens_per_block;
};
template <int RT>
struct GwLds {
    static constexpr int kStride = 64 + 8;   // row stride of a plane in elements (+8: bank spread, keeps 16-byte alignment)
    typedef u32x4 Tokens[64 * kGwCb / 8];
    typedef __bf16 Planes[3][RT * 32][kStride] __attribute__((aligned(16)));
};

template <int RT>
__device__ __forceinline__ void gate_weights_block(const GwArgs &args, typename GwLds<RT>::Tokens &xs, typename GwLds<RT>::Planes &pl, int token_block,
                                                   int col_block)
{
    constexpr int PPK = kGwCb / 8;   // 16-byte pieces per token row of the tile
    constexpr int PS = GwLds<RT>::kStride;
    constexpr int XP = 64 * PPK / kThreads;   // x pieces per thread
    constexpr int DLV = (64 * RT * 32 + kThreads - 1) / kThreads;   // dl values per thread (upper bound)
    const __bf16 *__restrict__ x = args.x;
    const float *__restrict__ dlp = args.dlp, *__restrict__ dlq = args.dlq;
    const int T = args.T, d = args.d, n = args.n, m = args.m;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c_base = col_block * kGwCb, R = n + m;
    const int t_begin = token_block * args.tokens_per_block, t_end = min(T, t_begin + args.tokens_per_block);

    // rows of the planes beyond the n + m logit columns stay zero
    for (int i = tid; i < 3 * RT * 32 * PS / 8; i += kThreads) reinterpret_cast<u32x4 *>(&pl[0][0][0])[i] = u32x4{0u, 0u, 0u, 0u};

    f32x16 acc[2][RT];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[u][rt][v] = 0.f;

    // fragment addressing of the x tile: lane = 16 tg + 4 tj + ta addresses token 8 (tg / 2) + tj (+4: second read,
    // +16 per k-step) and the 4 columns 16 (tg % 2) + 4 ta of its 32-column tile
    const int tg = lane >> 4, tj = (lane >> 2) & 3, ta = lane & 3;
    const int tk0 = 8 * (tg >> 1) + tj;
    int xoff[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int col = (wave * 2 + u) * 32 + 16 * (tg & 1) + 4 * ta;
        xoff[u] = (tk0 * PPK + ((col >> 3) + 4 * tj) % PPK) * 16 + (col & 4) * 2;
    }

    u32x4 xr[XP];
    float dv[DLV];
    // (index arithmetic is redone from an opaque copy of the thread id wherever it is needed, so that the compiler
    // does not keep two dozen precomputed addresses in registers across the token loop)
    auto opaque_tid = [&]() {
        int v = tid;
        asm volatile("" : "+v"(v));
        return v;
    };
    auto prefetch = [&](int t0) {
        const int tid = opaque_tid();
#pragma unroll
        for (int q = 0; q < XP; ++q) {
            const int id = tid + q * kThreads, k = id / PPK, p = id - k * PPK;
            xr[q] = u32x4{0u, 0u, 0u, 0u};
            if (t0 + k < t_end && c_base + p * 8 < d)
                xr[q] = *reinterpret_cast<const u32x4 *>(x + (size_t)(t0 + k) * d + c_base + p * 8);
        }
#pragma unroll
        for (int q = 0; q < DLV; ++q) {
            const int id = tid + q * kThreads, k = id / R, r = id - k * R;
            dv[q] = 0.f;
            if (k < 64 && t0 + k < t_end) dv[q] = r < n ? dlp[(size_t)(t0 + k) * n + r] : dlq[(size_t)(t0 + k) * m + r - n];
        }
    };
    prefetch(t_begin);
    for (int t0 = t_begin; t0 < t_end; t0 += 64) {
        __syncthreads();   // the previous tile has been read by every wave (first pass: the zero fill is complete)
        const int tid = opaque_tid();
#pragma unroll
        for (int q = 0; q < XP; ++q) {
            const int id = tid + q * kThreads, k = id / PPK, p = id - k * PPK;
            xs[k * PPK + (p + 4 * (k & 3)) % PPK] = xr[q];
        }
#pragma unroll
        for (int q = 0; q < DLV; ++q) {
            const int id = tid + q * kThreads, k = id / R, r = id - k * R;
            if (k < 64) {
                __bf16 hi, mid, lo;
                split3(dv[q], hi, mid, lo);
                pl[0][r][k] = hi, pl[1][r][k] = mid, pl[2][r][k] = lo;
            }
        }
        __syncthreads();
        if (t0 + 64 < t_end) prefetch(t0 + 64);
        const char *xb = reinterpret_cast<const char *>(xs);
#pragma unroll 1
        for (int kk = 0; kk < 4; ++kk) {
            bf16x8 a[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const char *p = xb + xoff[u] + kk * 16 * PPK * 16;
                struct { s16x4 lo, hi; } t;
                t.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
                t.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p + 4 * PPK * 16));
                a[u] = __builtin_bit_cast(bf16x8, t);
            }
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    const bf16x8 b = *reinterpret_cast<const bf16x8 *>(&pl[p][rt * 32 + (lane & 31)][16 * kk + 8 * (lane >> 5)]);
#pragma unroll
                    for (int u = 0; u < 2; ++u) acc[u][rt] = Half<__bf16>::mfma_32x32x16(a[u], b, acc[u][rt]);
                }
        }
    }

    // accumulator element v of a lane: logit column rt*32 + (lane & 31), x column 8*(v/4) + 4*(lane>>5) + v%4
    float *out = args.partial + (size_t)token_block * R * d;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int r = rt * 32 + (lane & 31);
        if (r >= R) continue;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c = c_base + (wave * 2 + u) * 32 + 8 * q + 4 * (lane >> 5);
                if (c < d)
                    *reinterpret_cast<f32x4 *>(out + (size_t)r * d + c) =
                        f32x4{acc[u][rt][4 * q], acc[u][rt][4 * q + 1], acc[u][rt][4 * q + 2], acc[u][rt][4 * q + 3]};
            }
    }
}

// Both products of a backward pass in one launch: they do not depend on each other, and neither fills the chip with latency to spare (few
// workgroups, or rows that wait for memory).  The first dx.blocks workgroups take dx, the others the router weights.
struct RouterGradArgs {
    DxArgs dx;
    GwArgs gw;
    int dx_blocks, dx_col_blocks, gw_col_blocks;   // workgroups of the dx part, column blocks of the two parts
};

// KC, RT 0: without that part, its LDS and its registers.  What one part alone needs are arrays of their own, which the compiler can tell
// apart; the parts that share a launch share their LDS.  dx on its own has its column blocks in blockIdx.y.
template <int KC, int RT>
__global__ __launch_bounds__(kThreads) void router_grad_mfma_kernel(RouterGradArgs a)
{
    const int b = blockIdx.x;
    if constexpr (RT == 0) {
        __shared__ typename DxLds<KC>::Weights wt;
        __shared__ typename DxLds<KC>::Rows io;
        dispatch_backward_block<KC>(a.dx, wt, io, b, blockIdx.y);
    } else if constexpr (KC == 0) {
        __shared__ typename GwLds<RT>::Tokens xs;
        __shared__ typename GwLds<RT>::Planes pl;
        gate_weights_block<RT>(a.gw, xs, pl, b / a.gw_col_blocks, b % a.gw_col_blocks);
    } else {
        union Lds {
            __device__ Lds() {}
            struct {
                typename DxLds<KC>::Weights wt;
                typename DxLds<KC>::Rows io;
            } dx;
            struct {
                typename GwLds<RT>::Tokens xs;
                typename GwLds<RT>::Planes pl;
            } gw;
        };
        __shared__ Lds lds;
        if (b < a.dx_blocks) dispatch_backward_block<KC>(a.dx, lds.dx.wt, lds.dx.io, b / a.dx_col_blocks, b % a.dx_col_blocks);
        else gate_weights_block<RT>(a.gw, lds.gw.xs, lds.gw.pl, (b - a.dx_blocks) / a.gw_col_blocks, (b - a.dx_blocks) % a.gw_col_blocks);
    }
}
}  // namespace

bool dispatch_backward_mfma_applies(const smile_layer_desc &d)
{
    const int kc = (d.n_groups + 15) / 16 + (d.m_local + 15) / 16;
    return d.dtype == SMILE_DTYPE_BF16 && kc <= kDxMaxChunks && d.d_model % 8 == 0;
}

bool gate_weights_mfma_applies(const smile_layer_desc &d)
{
    return d.dtype == SMILE_DTYPE_BF16 && (d.n_groups + d.m_local + 31) / 32 <= kGwMaxRowTiles && d.d_model % 8 == 0;
}

// Tokens per partial-sum block: a multiple of `granule` (the block size the workspace was laid out for, so that
// fewer, larger blocks always fit), grown until the grid is down to about four workgroups per CU.
int gate_weights_mfma_block_tokens(const smile_layer_desc &d, int granule)
{
    const long long col_blocks = (d.d_model + kGwCb - 1) / kGwCb;
    int k = 1;
    while (k < 8 && ((long long)d.T / (granule * 2 * k)) * col_blocks >= 1024) k *= 2;
    return granule * k;
}

hipError_t launch_router_grad_mfma(const LayerDesc &d, const RouterGradIo &io, bool with_dx, bool with_gw, float *partial, int blocks,
                                   int tokens_per_block, hipStream_t s)
{
    const int kp = (d.n_groups + 15) / 16, kc = kp + (d.m_local + 15) / 16, rt = (d.n_groups + d.m_local + 31) / 32;
    // One launch for both where the two parts need about the same LDS (39 and 46 KB with two chunks of logit columns), or where there are
    // few workgroups of dx.  us, dx and router weights apart -> in one launch: 8192 x 768, 2 + 8 columns 12.1 + 9.0 -> 13.9; 8192 x 1600
    // 19.2 + 11.6 -> 24.3; 32768 x 768, 16 + 8 28.8 + 20.3 -> 44.3; but 65536 x 1024, 32 + 8 (47 and 60 KB, 2048 workgroups) 77.3 + 61.4 -> 146.3.
    // Two chunks gain at every size, less as both parts fill the chip (a whole backward pass of narrow experts, apart -> in one launch: 8192 x 768 73.0 ->
    // 65.8; 65536 x 1024, 16 + 16, 2048 workgroups of dx 393.6 -> 391.0; 65536 x 1600, 16 + 16, 3584 592.1 -> 585.4; 131072 x 1024, 2 + 8, 4096 714.9 -> 711.7).
    const long long dx_groups = (long long)((d.T + kDxTokens - 1) / kDxTokens) * ((d.d_model + dx_cols(kc) - 1) / dx_cols(kc));
    if (with_dx && with_gw && (kc > 3 || (kc == 3 && dx_groups > 2 * (d.tune.cus > 0 ? d.tune.cus : 256)))) {
        const hipError_t err = launch_router_grad_mfma(d, io, true, false, nullptr, 0, 0, s);
        return err == hipSuccess ? launch_router_grad_mfma(d, io, false, true, partial, blocks, tokens_per_block, s) : err;
    }
    RouterGradArgs a{};
    a.dx = {static_cast<const __bf16 *>(io.dxe), io.group_idx, io.local_idx, io.slot, io.dlp, io.dlq, static_cast<const __bf16 *>(io.w_inter),
            static_cast<const __bf16 *>(io.w_intra), static_cast<__bf16 *>(io.dx), d.T, d.d_model, d.n_groups, d.m_local, d.capacity, kp};
    a.gw = {static_cast<const __bf16 *>(io.x), io.dlp, io.dlq, partial, d.T, d.d_model, d.n_groups, d.m_local, tokens_per_block};
    a.dx_col_blocks = (d.d_model + dx_cols(kc) - 1) / dx_cols(kc), a.gw_col_blocks = (d.d_model + kGwCb - 1) / kGwCb;
    const int dx_token_blocks = (d.T + kDxTokens - 1) / kDxTokens;
    a.dx_blocks = with_dx ? dx_token_blocks * a.dx_col_blocks : 0;
    const dim3 block(kThreads), grid = with_gw ? dim3(a.dx_blocks + blocks * a.gw_col_blocks) : dim3(dx_token_blocks, a.dx_col_blocks);
#define SMILE_CASE(K, R) SMILE_LAUNCH((router_grad_mfma_kernel<K, R>), grid, block, 0, s, a); break;
    if (with_dx && with_gw) {
        switch (kc * 4 + rt) {
        case 2 * 4 + 1: SMILE_CASE(2, 1)
        case 3 * 4 + 1: SMILE_CASE(3, 1)
        case 3 * 4 + 2: SMILE_CASE(3, 2)
        default: return hipErrorInvalidValue;
        }
    } else if (with_dx) {
        switch (kc) {
        case 2: SMILE_CASE(2, 0)
        case 3: SMILE_CASE(3, 0)
        case 4: SMILE_CASE(4, 0)
        case 5: SMILE_CASE(5, 0)
        case 6: SMILE_CASE(6, 0)
        case 7: SMILE_CASE(7, 0)
        case 8: SMILE_CASE(8, 0)
        case 9: SMILE_CASE(9, 0)
        case 10: SMILE_CASE(10, 0)
        default: return hipErrorInvalidValue;
        }
    } else {
        switch (rt) {
        case 1: SMILE_CASE(0, 1)
        case 2: SMILE_CASE(0, 2)
        case 3: SMILE_CASE(0, 3)
        case 4: SMILE_CASE(0, 4)
        case 5: SMILE_CASE(0, 5)
        default: return hipErrorInvalidValue;
        }
    }
#undef SMILE_CASE
    return hipGetLastError();
}

}  // namespace smile
