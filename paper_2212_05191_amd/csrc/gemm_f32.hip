// Grouped fp32 GEMM of the expert FFN on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 products and
// sums, 256 flop per clock and CU, twice what FMA instructions give), for the forward products and, with
// the contraction index as the slow index of one or both operands, for the four gradient products:
//
//   y[e][i][j] = sum_k X(i,k) W(j,k),  X(i,k) = x[e][i][k] or x[e][k][i] (XT),  W(j,k) = w[e][j][k] or w[e][k][j] (WT)
//
// with the row gather, bias, activation, second output, activation-gradient factor and gate-weighted scatter of the
// 16-bit kernels in the epilogue.
//
// Bound: fp32 layers are small (the weights of a group fit L2 many times over), so what counts is how many workgroups
// there are and how long one takes.  Hence small tiles, chosen by the launcher so that the chip has about two
// workgroups per CU, and four waves per workgroup that share one tile: 2 x 2 over a 64 x 64 or 64 x 128 tile, or, when
// there are few tiles, split along k (each wave takes a part of every slab, the parts are added through LDS in a
// fixed order), which shortens the serial chain of a tile by the same factor.
//
// K slabs of 32 go global -> LDS directly (16 bytes per lane) into a ring of three buffers.  A normal operand lands as
// [row][32 k] with its eight 16-byte pieces XOR-swizzled by row as in the 16-bit kernels, a transposed one as it lies
// in memory, [32 k][columns].  One MFMA takes two k: lane half h supplies the k of its half.  A normal operand is read
// 16 bytes at a time: the halves take neighbouring pieces, and element i of the two pieces is one MFMA, so that MFMA
// contracts k = 8 p + 4 h + i.  A transposed operand is read one float per lane at the same k.
// k beyond the end of the contraction (K % 32, or an expert's row count) is loaded from a zero block.
//
// Measured, 8 experts of about 256 rows of 256 x 1024 (forward and backward products in order): 22, 22, 23, 16, 22, 16 us
// (49-67 TFLOP/s); the FMA kernel of 64 x 64 tiles this replaces took 32, 74, 34, 28, 65, 28 us and six transposed copies
// of 4-5 us in the backward pass.  Forced tiles on the same products: 64 x 64 17-29 us, 32 x 64 17-27, 32 x 32 19-26,
// 64 x 128 17-45; the rule in launch_shape picks the best of them for every product.
#include "gemm_device.hpp"

namespace smile {

namespace {

struct F32Args {
    const float *x, *w, *bias;
    float *y, *y2;
    const float *aux;
    const int32_t *rows_valid, *k_valid, *x_rows, *y_rows;
    float *y_tok;
    const float *gate;
    int Mrows, Nout, K, ldx, ldw;
    long long sx, sw, sy;
    int act, post;
    int row_tiles, col_tiles, tiles;
};

// act'(p) and act(f) with the exact erf form (1 ReLU, 2 GELU)
__device__ __forceinline__ float f32_act(int act, float f)
{
    if (act == 1) return activate<1>(f);
    return act == 2 ? activate<2>(f) : f;
}
__device__ __forceinline__ float f32_act_grad(int post, float p)
{
    if (post == 1) return p > 0.f ? 1.f : 0.f;
    return 0.5f * (1.0f + erff(p * 0.70710678118654752f)) + p * 0.3989422804014327f * expf(-0.5f * p * p);
}

// Source address of linear 16-byte piece q of an operand tile of EXT rows / columns starting at tile0.  k0: first k of
// the piece inside the slab (the piece holds k0 .. k0+3 of one row, or columns of the single row k0).
template <int EXT, bool T>
__device__ __forceinline__ const float *f32_source(const float *base, int q, int tile0, int ext_valid, int ld, int &k0)
{
    if constexpr (!T) {
        const int row = q >> 3, piece = (q & 7) ^ ((row >> 1) & 7);
        k0 = piece * 4;
        return base + (size_t)min(tile0 + row, ext_valid - 1) * ld + piece * 4;
    } else {
        constexpr int PPK = EXT / 4;
        const int k = q / PPK, piece = q - k * PPK;
        k0 = k;
        return base + (size_t)k * ld + min(tile0 + piece * 4, ext_valid - 4);
    }
}

// BM x BN tile; 4 waves = WGM x WGN x WGK, a wave owns a (BM / WGM) x (BN / WGN) part of the tile and every WGK-th
// pair of pieces of a slab.
template <int BM, int BN, int WGM, int WGN, int WGK, bool XT, bool WT>
__global__ __launch_bounds__(256) void grouped_gemm_f32_kernel(F32Args a)
{
    static_assert(WGM * WGN * WGK == 4, "four waves");
    constexpr int BK = 32, STAGES = 3;
    constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 32, TN = WN / 32;
    constexpr int XI = BM / 8, WI = BN / 8, GPW = (XI + WI) / 4;   // load instructions per slab: x tile, w tile, per wave
    constexpr int STAGE = (BM + BN) * 8;                            // 16-byte pieces
    static_assert((XI + WI) % 4 == 0 && XI % 4 == 0, "load instructions must divide over the waves");
    static_assert((WGK - 1) * BM * BN / 4 <= STAGES * STAGE, "partial tiles must fit in the slab ring");
    __shared__ u32x4 lds[STAGES * STAGE];

    // ---- which tile: ids are remapped so that each XCD gets a contiguous range (shared operands meet in one L2)
    const int per_xcd = (a.tiles + kXcds - 1) / kXcds;
    const int lid = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if (lid >= a.tiles) return;
    const int per_group = a.row_tiles * a.col_tiles;
    const int e = lid / per_group, rem = lid - e * per_group;
    const int ct = rem / a.row_tiles, rt = rem - ct * a.row_tiles;
    const int rows = a.rows_valid ? min(a.rows_valid[e], a.Mrows) : a.Mrows;
    if (rt * BM >= rows) return;
    const int kv = a.k_valid ? min(a.k_valid[e], a.K) : a.K;
    const int slabs = (kv + BK - 1) / BK;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WGK, wm = (wave / WGK) % WGM, wn = wave / WGK / WGM;

    // ---- loads
    const float *X = a.x + (a.x_rows ? 0 : (size_t)e * a.sx), *W = a.w + (size_t)e * a.sw;
    const float *zero = reinterpret_cast<const float *>(kZeroPiece);
    const float *src[GPW];
    int k0[GPW];
    const size_t adv_x = XT ? (size_t)BK * a.ldx : BK, adv_w = WT ? (size_t)BK * a.ldw : BK;
#pragma unroll
    for (int i = 0; i < GPW; ++i) {
        const int inst = wave + i * 4;
        if (i < XI / 4) {
            const int q = inst * 64 + lane;
            if (!XT && a.x_rows) {   // gathered rows of the token matrix
                const int row = q >> 3, piece = (q & 7) ^ ((row >> 1) & 7);
                k0[i] = piece * 4;
                src[i] = X + (size_t)a.x_rows[(size_t)e * a.Mrows + min(rt * BM + row, rows - 1)] * a.ldx + piece * 4;
            } else {
                // a transposed x holds the output rows along its fast index: all Mrows columns exist in memory
                src[i] = f32_source<BM, XT>(X, q, rt * BM, XT ? a.Mrows : rows, a.ldx, k0[i]);
            }
        } else {
            src[i] = f32_source<BN, WT>(W, (inst - XI) * 64 + lane, ct * BN, a.Nout, a.ldw, k0[i]);
        }
    }
    auto issue = [&](int slab, int stage) {
#pragma unroll
        for (int i = 0; i < GPW; ++i) {
            const float *p = src[i] + (size_t)slab * (i < XI / 4 ? adv_x : adv_w);
            if (slab * BK + k0[i] >= kv) p = zero;
            __builtin_amdgcn_global_load_lds(SMILE_GPTR(p), SMILE_LPTR(&lds[stage * STAGE + (wave + i * 4) * 64]), 16, 0, 0);
        }
    };
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
        if (s < slabs) issue(s, s);

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const int frow = lane & 31, h = lane >> 5, fsw = (frow >> 1) & 7;
    int stage = 0;
    for (int s = 0; s < slabs; ++s) {
        if (s + 1 < slabs) wait_vmcnt<GPW>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();   // slab s is there for every wave, and nobody reads the buffer refilled next
        if (s + STAGES - 1 < slabs) issue(s + STAGES - 1, stage == 0 ? STAGES - 1 : stage - 1);
        const u32x4 *xb = lds + stage * STAGE, *wb = xb + BM * 8;
        // element i of lane half h: k = 8 p + 4 h + i of row / column tile0 + frow
        auto fetch = [&](const u32x4 *t, auto transposed, int ext, int tile0, int p) {
            f32x4 f;
            if constexpr (decltype(transposed)::value) {
                const float *q = reinterpret_cast<const float *>(t) + (8 * p + 4 * h) * ext + tile0 + frow;
#pragma unroll
                for (int i = 0; i < 4; ++i) f[i] = q[i * ext];
            } else {
                f = __builtin_bit_cast(f32x4, t[(tile0 + frow) * 8 + ((2 * p + h) ^ fsw)]);
            }
            return f;
        };
#pragma unroll
        for (int pp = 0; pp < 4 / WGK; ++pp) {
            const int p = pp * WGK + wk;
            f32x4 xf[TM], wf[TN];
#pragma unroll
            for (int j = 0; j < TM; ++j) xf[j] = fetch(xb, std::integral_constant<bool, XT>{}, BM, wm * WM + j * 32, p);
#pragma unroll
            for (int i = 0; i < TN; ++i) wf[i] = fetch(wb, std::integral_constant<bool, WT>{}, BN, wn * WN + i * 32, p);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int j = 0; j < TM; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[i][q], xf[j][q], acc[i][j], 0, 0, 0);
        }
        stage = stage + 1 == STAGES ? 0 : stage + 1;
    }

    // ---- waves that split k: the parts are added in wave order by the wave with wk == 0
    if constexpr (WGK > 1) {
        __syncthreads();
        f32x4 *red = reinterpret_cast<f32x4 *>(lds);
        constexpr int PART = TN * TM * 4 * 64;   // one wave's accumulators, in 16-byte units
        const int pair = wn * WGM + wm;
        if (wk > 0) {
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        red[(pair * (WGK - 1) + wk - 1) * PART + ((i * TM + j) * 4 + q) * 64 + lane] =
                            f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int o = 0; o < WGK - 1; ++o)
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 v = red[(pair * (WGK - 1) + o) * PART + ((i * TM + j) * 4 + q) * 64 + lane];
#pragma unroll
                        for (int k = 0; k < 4; ++k) acc[i][j][4 * q + k] += v[k];
                    }
    }

    // ---- epilogue: accumulator element v of a lane is (column 8*(v/4) + 4*h + v%4, row lane % 32) of its 32 x 32 tile
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int row = rt * BM + wm * WM + j * 32 + frow;
        if (row >= rows) continue;
        const int tok = a.y_rows ? a.y_rows[(size_t)e * a.Mrows + row] : 0;
        const float g = a.y_rows ? a.gate[tok] : 0.f;
        const size_t at = (size_t)e * a.sy + (size_t)row * a.Nout;
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = ct * BN + wn * WN + i * 32 + 8 * q + 4 * h;
                if (col >= a.Nout) continue;   // Nout is a multiple of 8: whole groups of four
                f32x4 f = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                if (a.bias) f += *reinterpret_cast<const f32x4 *>(a.bias + (size_t)e * a.Nout + col);
                if (a.y2) *reinterpret_cast<f32x4 *>(a.y2 + at + col) = f;
                if (a.post) {
                    const f32x4 p = *reinterpret_cast<const f32x4 *>(a.aux + at + col);
#pragma unroll
                    for (int k = 0; k < 4; ++k) f[k] *= f32_act_grad(a.post, p[k]);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) f[k] = f32_act(a.act, f[k]);
                if (a.y) *reinterpret_cast<f32x4 *>(a.y + at + col) = f;
                if (a.y_rows) *reinterpret_cast<f32x4 *>(a.y_tok + (size_t)tok * a.Nout + col) = f * g;
            }
    }
}

template <int BM, int BN, int WGM, int WGN, int WGK, bool XT, bool WT>
hipError_t launch_tile(F32Args a, int N, hipStream_t s)
{
    a.row_tiles = (a.Mrows + BM - 1) / BM;
    a.col_tiles = (a.Nout + BN - 1) / BN;
    a.tiles = N * a.row_tiles * a.col_tiles;
    SMILE_LAUNCH((grouped_gemm_f32_kernel<BM, BN, WGM, WGN, WGK, XT, WT>), dim3((a.tiles + kXcds - 1) / kXcds * kXcds), dim3(256),
                 0, s, a);
    return hipGetLastError();
}

template <bool XT, bool WT>
hipError_t launch_shape(const F32Args &a, int N, const Tuning &tune, hipStream_t s)
{
    // the largest tile that still gives about two workgroups per CU: tiles are counted over the whole buffers (the host does not
    // know how many rows are live), which is right within the capacity factor
    auto tiles = [&](int bm, int bn) { return (long long)N * ((a.Mrows + bm - 1) / bm) * ((a.Nout + bn - 1) / bn); };
    const long long want = 2LL * (tune.cus > 0 ? tune.cus : 256);
    if (tiles(64, 128) >= 2 * want) return launch_tile<64, 128, 2, 2, 1, XT, WT>(a, N, s);
    if (tiles(64, 64) >= want) return launch_tile<64, 64, 2, 2, 1, XT, WT>(a, N, s);
    if (tiles(32, 64) >= want) return launch_tile<32, 64, 1, 2, 2, XT, WT>(a, N, s);
    return launch_tile<32, 32, 1, 1, 4, XT, WT>(a, N, s);
}

}  // namespace

hipError_t launch_grouped_gemm_f32(const F32Gemm &g, hipStream_t s)
{
    if (g.K < 1 || g.Mrows < 1 || g.Nout % 8 || g.ldx % 4 || g.ldw % 4) return hipErrorInvalidValue;
    if (g.x_transposed && (!g.w_transposed || g.Mrows % 4)) return hipErrorInvalidValue;   // not needed by any caller
    if (!(g.x_transposed && g.w_transposed) && g.K % 4) return hipErrorInvalidValue;       // pieces of a normal operand
    F32Args a{};
    a.x = static_cast<const float *>(g.x), a.w = static_cast<const float *>(g.w), a.bias = static_cast<const float *>(g.bias);
    a.y = static_cast<float *>(g.y), a.y2 = static_cast<float *>(g.y2), a.aux = static_cast<const float *>(g.aux);
    a.rows_valid = g.rows_valid, a.k_valid = g.k_valid, a.x_rows = g.x_rows, a.y_rows = g.y_rows;
    a.y_tok = static_cast<float *>(g.y_tok), a.gate = g.gate;
    a.Mrows = g.Mrows, a.Nout = g.Nout, a.K = g.K, a.ldx = g.ldx, a.ldw = g.ldw;
    a.sx = g.sx, a.sw = g.sw, a.sy = g.sy, a.act = g.act, a.post = g.post;
    if (g.x_transposed) return launch_shape<true, true>(a, g.N, g.tune, s);
    if (g.w_transposed) return launch_shape<false, true>(a, g.N, g.tune, s);
    return launch_shape<false, false>(a, g.N, g.tune, s);
}

}  // namespace smile
