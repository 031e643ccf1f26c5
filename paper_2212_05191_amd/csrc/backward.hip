// Backward pass of the layer: the chain rule on Eq. 3 and Eq. 4 with the discrete routing decisions and
// the fractions f of Eq. 4 held constant (as for the Switch loss of Section 2), in the reverse order of
// the forward steps:
//
//   combine_backward       dye[row(t)] = gate_t * dy[t],  dgate[t] = <dy[t], ye[row(t)]>     (HBM streaming)
//   route_backward         softmax Jacobians of the two routers: dgate and the Eq. 4 terms -> dlogits (in the chained pass in
//                          the same launch as combine_backward)
//   expert_ffn_backward    (pre, h) = xe . W1^T   unless saved by the forward pass (one launch of the forward kernel)
//                          dpre = (dye . W2) * act'(pre),  dxe = dpre . W1,
//                          dW2 = dye^T . h,  dW1 = dpre^T . xe   (contraction over the expert's rows)
//                          four launches of the MFMA kernels that read operands whose contraction index is
//                          the slow one, nothing transposed in memory
//   dispatch_backward      dx[t] = dxe[row(t)] + dlp[t,:] . W_p + dlq[t,:] . W_q
//   gate_weights_backward  dW_p = dlp^T . x, dW_q = dlq^T . x: per-block partial sums, then a fixed-order
//                          reduction over the blocks (bit-reproducible, no atomics); the partial sums in the same launch as
//                          dispatch_backward where both are small
#include <type_traits>


#include "smile_internal.hpp"

namespace smile {

namespace {

constexpr int kThreads = 256;
constexpr int kMaxGridX = 1 << 20;   // workgroups in x where a grid is dealt out over x and y

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

// A 16-byte piece as 4 (fp32) or 8 (16-bit types) floats and back.  DT: SMILE_DTYPE_*.
template <int DT>
struct Piece {
    static constexpr int kElems = DT == SMILE_DTYPE_F32 ? 4 : 8;
    using H = Half<std::conditional_t<DT == SMILE_DTYPE_F16, _Float16, __bf16>>;
    __device__ static __forceinline__ void unpack(u32x4 v, float (&f)[kElems])
    {
        if constexpr (DT != SMILE_DTYPE_F32) {
#pragma unroll
            for (int k = 0; k < 4; ++k) { f[2 * k] = H::lo(v[k]); f[2 * k + 1] = H::hi(v[k]); }
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = __uint_as_float(v[k]);
        }
    }
    __device__ static __forceinline__ u32x4 pack(const float (&f)[kElems])
    {
        u32x4 r;
        if constexpr (DT != SMILE_DTYPE_F32) {
#pragma unroll
            for (int k = 0; k < 4; ++k) r[k] = H::pack(f[2 * k], f[2 * k + 1]);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) r[k] = __float_as_uint(f[k]);
        }
        return r;
    }
};

// ------------------------------------------------------------------------------------ combine and route backward

__device__ __forceinline__ float exp_neg(float v) { return __builtin_amdgcn_exp2f(v * 1.4426950408889634f); }

// Sum over the LPR lanes of a token, in a fixed order; every lane gets it.
template <int LPR>
__device__ __forceinline__ float token_sum(float v)
{
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

struct RouteBackwardArgs {
    const float *logits_inter, *logits_intra, *bias_inter, *bias_intra;
    const int32_t *group_idx, *local_idx, *group_count, *local_count;
    int T, n, m;
    float coef_inter, coef_intra;
    float *dlp, *dlq;
};

// One softmax row backwards by the LPR lanes of a token, columns sub, sub + LPR, ...: with z = sum exp(a - a_top) (so the top
// probability is 1 / z) and u_k = coef * count_k + [k == top] * extra,  dl_k = p_k * (u_k - sum_i u_i p_i).
// Rows of up to HELD * LPR columns stay in registers; wider ones are read again by each of the three passes.
// VIRTUAL: the bits of VIRTUAL * LPR lanes, or of any more that have no columns (their zeros change nothing), for rows of at most HELD * LPR columns:
// column k of a lane's own belongs to virtual lane k % VIRTUAL, whose terms are added in a chain, and the virtual lanes are added in the order
// of token_sum.
template <int LPR, int HELD = 2, int VIRTUAL = 1>
struct SoftmaxRow {
    static_assert(VIRTUAL == 1 || VIRTUAL == 2 || VIRTUAL == 4, "see sum()");
    const float *row, *bias;
    int len, top, sub;
    float held[HELD], mx, inv_z;
    __device__ __forceinline__ float at(int i) const { return bias ? __fadd_rn(row[i], bias[i]) : row[i]; }
    template <typename F>
    __device__ __forceinline__ void each(F f) const
    {
        if (VIRTUAL > 1 || len <= HELD * LPR) {
#pragma unroll
            for (int k = 0; k < HELD; ++k)
                if (sub + k * LPR < len) f(sub + k * LPR, held[k], k);
        } else {
            for (int i = sub; i < len; i += LPR) f(i, at(i), 0);
        }
    }
    // add(i, a, s) = s and column i's term
    template <typename F>
    __device__ __forceinline__ float sum(F add) const
    {
        float s[VIRTUAL] = {};
        each([&](int i, float a, int k) { s[k % VIRTUAL] = add(i, a, s[k % VIRTUAL]); });
        if constexpr (VIRTUAL == 4) s[0] += s[2], s[1] += s[3];
        if constexpr (VIRTUAL >= 2) s[0] += s[1];
        return token_sum<LPR>(s[0]);
    }
    // reads the row; 1 / z is the top probability
    __device__ __forceinline__ SoftmaxRow(const float *row_, const float *bias_, int len_, int top_, int sub_)
        : row(row_), bias(bias_), len(len_), top(top_), sub(sub_)
    {
#pragma unroll
        for (int k = 0; k < HELD; ++k) held[k] = sub + k * LPR < len ? at(sub + k * LPR) : 0.f;
        mx = at(top);
    }
    __device__ __forceinline__ void normalise()
    {
        inv_z = 1.0f / sum([&](int, float a, float s) { return s + exp_neg(a - mx); });
    }
    __device__ __forceinline__ void backward(float coef, const int32_t *__restrict__ count, float extra, float *__restrict__ out) const
    {
        auto u = [&](int i) { return coef * (float)count[i] + (i == top ? extra : 0.f); };
        const float dot = sum([&](int i, float a, float s) { return fmaf(u(i), exp_neg(a - mx) * inv_z, s); });
        each([&](int i, float a, int) { out[i] = exp_neg(a - mx) * inv_z * (u(i) - dot); });
    }
};

template <typename Row>
__device__ __forceinline__ void route_backward_token(Row &p, Row &q, const RouteBackwardArgs &a, int t, float dg)
{
    p.normalise();
    q.normalise();
    p.backward(a.coef_inter, a.group_count, dg * q.inv_z, a.dlp + (size_t)t * a.n);
    q.backward(a.coef_intra, a.local_count, dg * p.inv_z, a.dlq + (size_t)t * a.m);
}

// LPR consecutive lanes own one token row (as in the forward dispatch / combine kernels).  ROUTE: they go on with the token's two softmax
// rows, whose logits were requested in front of the rows of dy and ye.  Bound: the rows (3 K d elements); the softmax part on its own is a
// launch of small loads.  Against two launches, the second with a thread for each token (us): 8192 x 768 with 2 + 8 columns 9.1 + 7.4 -> 10.9,
// 32768 x 768 with 1 + 128 28.1 + 39.4 -> 42.2, 65536 x 1024 with 32 + 8 24.0 + 31.4 -> 42.7, fp32 2048 x 256 with 2 + 4 4.3 + 5.6 -> 5.3.
template <int DT, int LPR, bool ROUTE>
__global__ __launch_bounds__(kThreads) void combine_backward_kernel(
    const u32x4 *__restrict__ dy, const u32x4 *__restrict__ ye, const int32_t *__restrict__ slot, const float *__restrict__ gate,
    u32x4 *__restrict__ dye, float *__restrict__ dgate, int ppr, int C, RouteBackwardArgs a)
{
    constexpr int E = Piece<DT>::kElems;
    const int t = blockIdx.x * (kThreads / LPR) + threadIdx.x / LPR, sub = threadIdx.x % LPR;
    // every lane of a row group takes the same branch, and a group never straddles a wave
    if (t >= a.T) return;
    const int sl = slot[t], g = a.group_idx[t], l = a.local_idx[t];
    auto rows = [&]() {
        if (sl < 0) return 0.f;
        const float gt = gate[t];
        const size_t row = (size_t)(g * a.m + l) * C + sl;
        const u32x4 *src = dy + (size_t)t * ppr, *act = ye + row * ppr;
        u32x4 *dst = dye + row * ppr;
        float dot = 0.f;
        for (int c = sub; c < ppr; c += LPR) {
            float x[E], y[E], o[E];
            Piece<DT>::unpack(src[c], x);
            Piece<DT>::unpack(act[c], y);
#pragma unroll
            for (int k = 0; k < E; ++k) {
                dot = fmaf(x[k], y[k], dot);
                o[k] = x[k] * gt;
            }
            dst[c] = Piece<DT>::pack(o);
        }
        return token_sum<LPR>(dot);
    };
    if constexpr (ROUTE) {
        SoftmaxRow<LPR> p(a.logits_inter + (size_t)t * a.n, a.bias_inter, a.n, g, sub);
        SoftmaxRow<LPR> q(a.logits_intra + (size_t)t * a.m, a.bias_intra ? a.bias_intra + (size_t)g * a.m : nullptr, a.m, l, sub);
        const float dg = rows();
        if (sub == 0) dgate[t] = dg;
        route_backward_token(p, q, a, t, dg);
    } else {
        const float dg = rows();
        if (sub == 0) dgate[t] = dg;
    }
}

// The softmax part on its own, with the bits of the kernel above (launch_route_backward: by how many lanes).  The token blocks are dealt out over
// blockIdx.x and y: a launch has fewer than 2^32 threads in x.
template <int LPR, int VIRTUAL>
__global__ __launch_bounds__(kThreads) void route_backward_kernel(const float *__restrict__ dgate, RouteBackwardArgs a)
{
    const long long token = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * (kThreads / LPR) + threadIdx.x / LPR;
    if (token >= a.T) return;
    const int t = (int)token, sub = threadIdx.x % LPR;
    const int g = a.group_idx[t], l = a.local_idx[t];
    typedef SoftmaxRow<LPR, 4, VIRTUAL> Row;
    Row p(a.logits_inter + (size_t)t * a.n, a.bias_inter, a.n, g, sub);
    Row q(a.logits_intra + (size_t)t * a.m, a.bias_intra ? a.bias_intra + (size_t)g * a.m : nullptr, a.m, l, sub);
    route_backward_token(p, q, a, t, dgate[t]);
}

// ------------------------------------------------------------------------------------ dispatch backward

// dx[t] = dxe[row(t)] (kept tokens) + sum_i dlp[t,i] W_p[i] + sum_j dlq[t,j] W_q[j], one rounding.
struct DispatchBackwardArgs {
    const u32x4 *dxe;
    const int32_t *group_idx, *local_idx, *slot;
    const float *dlp, *dlq;
    const u32x4 *w_inter, *w_intra;
    u32x4 *dx;
    int T, ppr, n, m, C;
};
template <int DT, int LPR>
__device__ __forceinline__ void dispatch_backward_block(const DispatchBackwardArgs &a, int block)
{
    constexpr int E = Piece<DT>::kElems;
    const u32x4 *__restrict__ dxe = a.dxe, *__restrict__ w_inter = a.w_inter, *__restrict__ w_intra = a.w_intra;
    const int32_t *__restrict__ group_idx = a.group_idx, *__restrict__ local_idx = a.local_idx, *__restrict__ slot = a.slot;
    const float *__restrict__ dlp = a.dlp, *__restrict__ dlq = a.dlq;
    u32x4 *__restrict__ dx = a.dx;
    const int T = a.T, ppr = a.ppr, n = a.n, m = a.m, C = a.C;
    const int t = block * (kThreads / LPR) + threadIdx.x / LPR, sub = threadIdx.x % LPR;
    if (t >= T) return;
    const int sl = slot[t];
    const u32x4 *src = sl >= 0 ? dxe + ((size_t)(group_idx[t] * m + local_idx[t]) * C + sl) * ppr : nullptr;
    const float *lp = dlp + (size_t)t * n, *lq = dlq + (size_t)t * m;
    for (int c = sub; c < ppr; c += LPR) {
        float acc[E], w[E];
        if (src) Piece<DT>::unpack(src[c], acc);
        else {
#pragma unroll
            for (int k = 0; k < E; ++k) acc[k] = 0.f;
        }
        // acc += sum_i dl[i] * rows[i][c], eight rows at a time with all their loads issued first
        auto add_rows = [&](const u32x4 *__restrict__ rows, const float *__restrict__ dl, int count) {
            for (int i0 = 0; i0 < count; i0 += 8) {
                u32x4 wp[8];
                float g[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int i = min(i0 + q, count - 1);
                    wp[q] = rows[(size_t)i * ppr + c];
                    g[q] = dl[i];
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    if (i0 + q < count) {
                        Piece<DT>::unpack(wp[q], w);
#pragma unroll
                        for (int k = 0; k < E; ++k) acc[k] = fmaf(g[q], w[k], acc[k]);
                    }
                }
            }
        };
        add_rows(w_inter, lp, n);
        add_rows(w_intra, lq, m);
        dx[(size_t)t * ppr + c] = Piece<DT>::pack(acc);
    }
}

// ------------------------------------------------------------------------------------ router weights backward

constexpr int kGwTokens = 128;   // tokens per workgroup
constexpr int kGwCols = 64;      // columns of x per workgroup
constexpr int kGwChunk = 16;     // logit columns per pass over the token tile

// partial[b][i][k] = sum over the block's tokens of dl[t][i] * x[t][k], i over the n + m logit columns
// (dlp first, then dlq).  The x tile (fp32) and a chunk of 16 logit-gradient columns sit in LDS; lane =
// column of x, wave w owns logit columns 4w .. 4w+3 of the chunk, so its four dl values of a token come
// from one broadcast LDS read.  Tokens are summed serially: a fixed order.
struct GateWeightsArgs {
    const void *x;
    const float *dlp, *dlq;
    float *partial;
    int T, d, n, m;
};
template <int DT>
__device__ __forceinline__ void gate_weights_block(const GateWeightsArgs &a, int b, int col_block)
{
    __shared__ float xs[kGwTokens][kGwCols + 1];
    __shared__ __attribute__((aligned(16))) float dls[kGwTokens][kGwChunk];
    const void *__restrict__ x = a.x;
    const float *__restrict__ dlp = a.dlp, *__restrict__ dlq = a.dlq;
    float *__restrict__ partial = a.partial;
    const int T = a.T, d = a.d, n = a.n, m = a.m, k0 = col_block * kGwCols;
    const int t0 = b * kGwTokens;
    const int cnt = min(kGwTokens, T - t0);
    {
        // x tile: 16-byte pieces, all of a thread's loads issued before the first LDS write (d % 8 == 0)
        constexpr int E = Piece<DT>::kElems, PPT = kGwCols / E, PER = kGwTokens * PPT / kThreads;
        u32x4 v[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int id = threadIdx.x + q * kThreads, tt = id / PPT, k = (id - tt * PPT) * E;
            v[q] = u32x4{0u, 0u, 0u, 0u};
            if (tt < cnt && k0 + k < d)
                v[q] = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(x) +
                                                        ((size_t)(t0 + tt) * d + k0 + k) * (16 / E));
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int id = threadIdx.x + q * kThreads, tt = id / PPT, k = (id - tt * PPT) * E;
            float f[E];
            Piece<DT>::unpack(v[q], f);
#pragma unroll
            for (int j = 0; j < E; ++j) xs[tt][k + j] = f[j];
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int cols = n + m;
    for (int c0 = 0; c0 < cols; c0 += kGwChunk) {
        __syncthreads();   // x tile ready / previous chunk consumed
        for (int id = threadIdx.x; id < kGwTokens * kGwChunk; id += kThreads) {
            const int tt = id / kGwChunk, i = c0 + (id - tt * kGwChunk);
            float v = 0.f;
            if (tt < cnt && i < cols)
                v = i < n ? dlp[(size_t)(t0 + tt) * n + i] : dlq[(size_t)(t0 + tt) * m + (i - n)];
            dls[tt][id - tt * kGwChunk] = v;
        }
        __syncthreads();
        float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll 8
        for (int tt = 0; tt < cnt; ++tt) {
            const float xv = xs[tt][lane];
            const float4 g = *reinterpret_cast<const float4 *>(&dls[tt][4 * wave]);
            s0 = fmaf(g.x, xv, s0);
            s1 = fmaf(g.y, xv, s1);
            s2 = fmaf(g.z, xv, s2);
            s3 = fmaf(g.w, xv, s3);
        }
        if (k0 + lane < d) {
            const float sv[4] = {s0, s1, s2, s3};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = c0 + 4 * wave + j;
                if (i < cols) partial[((size_t)b * cols + i) * d + k0 + lane] = sv[j];
            }
        }
    }
}

// dx by the first dx_blocks workgroups, the partial sums of the router weights by the others (DX, GW: with that part)
template <int DT, int LPR, bool DX, bool GW>
__global__ __launch_bounds__(kThreads) void router_grad_kernel(DispatchBackwardArgs dx, GateWeightsArgs gw, int dx_blocks, int gw_col_blocks)
{
    const int b = blockIdx.x;
    if constexpr (DX) {
        if (!GW || b < dx_blocks) return dispatch_backward_block<DT, LPR>(dx, b);
    }
    if constexpr (!DX) gate_weights_block<DT>(gw, b, blockIdx.y);
    else if constexpr (GW) gate_weights_block<DT>(gw, (b - dx_blocks) / gw_col_blocks, (b - dx_blocks) % gw_col_blocks);
}

// dw[i][k] = sum_b partial[b][i][k]: PARTS runs of the blocks side by side, each in index order, then the runs in order.  A thread that adds all
// blocks itself waits for memory once per eight of them; with less than a workgroup per CU nothing hides that, so eight threads share an
// element there, from 48 blocks on (us: 512 blocks of 16 x 64 22.7 -> 5.3, 256 of 24 x 768 12.5 -> 4.8, 128 of 40 x 1024 6.9 -> 4.9, 64 of 10 x 64 and of
// 10 x 768 3.8 -> 2.4 and 3.9; but 32 of them 2.5 and 3.0, 8 of 10 x 64 1.5 and 2.3; 256 of 129 x 768, 387 workgroups, 15.3 and 16.6).
template <int PARTS>
__global__ __launch_bounds__(kThreads) void gate_weights_reduce_kernel(
    const float *__restrict__ partial, float *__restrict__ dw_inter, float *__restrict__ dw_intra, int B, int d, int n,
    int m)
{
    constexpr int ELEMS = kThreads / PARTS;
    const int part = PARTS > 1 ? threadIdx.x / ELEMS : 0, elem = threadIdx.x % ELEMS;
    const long long id = (long long)blockIdx.x * ELEMS + elem;
    const long long total = (long long)(n + m) * d;
    const int per = (B + PARTS - 1) / PARTS, b1 = PARTS > 1 ? min(B, (part + 1) * per) : B;
    float s = 0.f;
    if (id < total) {
#pragma unroll 8
        for (int b = part * per; b < b1; ++b) s += partial[(size_t)b * total + id];
    }
    if constexpr (PARTS > 1) {
        __shared__ float sums[PARTS][ELEMS];
        sums[part][elem] = s;
        __syncthreads();
        if (part != 0) return;
#pragma unroll
        for (int p = 1; p < PARTS; ++p) s += sums[p][elem];
    }
    if (id >= total) return;
    if (id < (long long)n * d) dw_inter[id] = s;
    else dw_intra[id - (long long)n * d] = s;
}

int lanes_per_row(int ppr)
{
    int l = 8;
    while (l * 2 <= ppr && l < 32) l *= 2;
    return l;
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace

#define SMILE_BWD_LPR_SWITCH(lpr, CALL)             \
    switch (lpr) {                                  \
    case 8: { constexpr int L = 8; CALL; } break;   \
    case 16: { constexpr int L = 16; CALL; } break; \
    default: { constexpr int L = 32; CALL; } break; \
    }

// CALL with the compile-time constant DT set to the runtime storage type
#define SMILE_DTYPE_SWITCH(dtype, CALL)                                             \
    switch (dtype) {                                                                \
    case SMILE_DTYPE_BF16: { constexpr int DT = SMILE_DTYPE_BF16; CALL; } break;    \
    case SMILE_DTYPE_F16: { constexpr int DT = SMILE_DTYPE_F16; CALL; } break;      \
    default: { constexpr int DT = SMILE_DTYPE_F32; CALL; } break;                   \
    }

BackwardLayout backward_workspace_layout(const smile_layer_desc &d)
{
    BackwardLayout L{};
    const size_t esz = elem_size(d.dtype);
    const size_t N = (size_t)d.n_groups * d.m_local, C = (size_t)d.capacity;
    const size_t dm = (size_t)d.d_model, F = (size_t)d.d_ff;
    L.gw_blocks = (d.T + kGwTokens - 1) / kGwTokens;
    size_t off = 0;
    L.off_pre = off;     off = align_up(off + N * C * F * esz, 256);
    L.off_h = off;       off = align_up(off + N * C * F * esz, 256);
    L.off_dpre = off;    off = align_up(off + N * C * F * esz, 256);
    L.off_gw_partial = off;
    off = align_up(off + (size_t)L.gw_blocks * (size_t)(d.n_groups + d.m_local) * dm * sizeof(float), 256);
    L.total = off;
    return L;
}

static RouteBackwardArgs route_backward_args(const smile_layer_desc &d, const RouteBackwardIo &io, float dloss)
{
    // d(alpha * n * sum_i f_i P_i) / dp[t,i] = alpha * n * (count_i / T) / T
    const float inv_t2 = 1.0f / ((float)d.T * (float)d.T);
    return {io.logits_inter, io.logits_intra, io.bias_inter, io.bias_intra, io.group_idx, io.local_idx, io.group_count, io.local_count,
            d.T, d.n_groups, d.m_local, dloss * d.alpha * (float)d.n_groups * inv_t2, dloss * d.beta * (float)d.m_local * inv_t2, io.dlp, io.dlq};
}

hipError_t launch_combine_backward(const smile_layer_desc &d, const void *dy, const void *ye, const int32_t *slot, const float *gate, void *dye,
                                   float *dgate, const RouteBackwardIo &io, bool route, float dloss, hipStream_t s)
{
    const int ppr = d.d_model * elem_size(d.dtype) / 16;
    const int lpr = lanes_per_row(ppr);
    const RouteBackwardArgs a = route_backward_args(d, io, dloss);
    const dim3 grid((d.T + kThreads / lpr - 1) / (kThreads / lpr)), block(kThreads);
    auto launch = [&](auto with) {
        constexpr bool ROUTE = decltype(with)::value;
        SMILE_DTYPE_SWITCH(d.dtype, SMILE_BWD_LPR_SWITCH(
            lpr, SMILE_LAUNCH((combine_backward_kernel<DT, L, ROUTE>), grid, block, 0, s, static_cast<const u32x4 *>(dy),
                              static_cast<const u32x4 *>(ye), slot, gate, static_cast<u32x4 *>(dye), dgate, ppr, d.capacity, a)));
    };
    if (route) launch(std::true_type{});
    else launch(std::false_type{});
    return hipGetLastError();
}

hipError_t launch_route_backward(const smile_layer_desc &d, const float *dgate, const RouteBackwardIo &io, float dloss, hipStream_t s)
{
    // As few lanes a token as hold the wider row, two columns each up to 16 and four beyond, up to those that the chained pass gives it: that pass
    // has them for the rows of dy, here the ones without a column would be most of the launch.  us, 524288 tokens, rows of 1536 bytes, 32 lanes -> here (a
    // kernel of one thread a token, or through LDS from 32 columns on): 1 + 1 columns 92 -> 4.4 (4.3), 2 + 8 93 -> 16.5 (33), 16 + 16 96 -> 35 (44),
    // 32 + 8 95 -> 40 (69); 65536 tokens: 2 + 8 11.4 -> 4.2 (6.7), 1 + 64 15.3 -> 11.1 (21.9).  Two columns and four: 8 + 8 19.7 and 23.8, 16 + 16 35.0 and 35.4 (at
    // 8192 tokens 3.6 and 4.4), 24 + 8 57.3 and 34.7, 32 + 32 82 and 69.
    const int most = lanes_per_row(d.d_model * elem_size(d.dtype) / 16), width = d.n_groups > d.m_local ? d.n_groups : d.m_local;
    const int columns = width <= 16 ? 2 : 4;
    int lanes = 1;
    while (lanes < most && columns * lanes < width) lanes *= 2;
    const RouteBackwardArgs a = route_backward_args(d, io, dloss);
    const long long blocks = ((long long)d.T * lanes + kThreads - 1) / kThreads;
    const dim3 grid((unsigned)(blocks < kMaxGridX ? blocks : kMaxGridX), (unsigned)((blocks + kMaxGridX - 1) / kMaxGridX));
#define SMILE_CASE(L, V) case L * 8 + V: SMILE_LAUNCH((route_backward_kernel<L, V>), grid, dim3(kThreads), 0, s, dgate, a); break;
    switch (lanes * 8 + (most / lanes < 4 ? most / lanes : 4)) {
        SMILE_CASE(1, 4) SMILE_CASE(2, 4) SMILE_CASE(4, 4) SMILE_CASE(8, 4)
        SMILE_CASE(4, 2) SMILE_CASE(8, 2) SMILE_CASE(16, 2)
        SMILE_CASE(8, 1) SMILE_CASE(16, 1) SMILE_CASE(32, 1)
    }
#undef SMILE_CASE
    return hipGetLastError();
}

hipError_t launch_expert_ffn_backward(const LayerDesc &d, void *workspace, const void *xe,
                                      const int32_t *kept_count, const void *w1, const void *w2, const void *dye,
                                      const void *h_saved, const void *pre_saved, void *dxe, void *dw1, void *dw2,
                                      hipStream_t s)
{
    const BackwardLayout L = backward_workspace_layout(d);
    char *b = static_cast<char *>(workspace);
    void *dpre = b + L.off_dpre;
    const int N = d.n_groups * d.m_local, C = d.capacity, dm = d.d_model, F = d.d_ff;
    const int act = d.act == SMILE_ACT_RELU ? 1 : 2;
    hipError_t err;
#define SMILE_TRY(call) do { err = (call); if (err != hipSuccess) return err; } while (0)

    // hidden activation and its pre-activation: saved by the forward pass, or recomputed here
    const void *h = h_saved, *pre = pre_saved;
    if (!h) {
        void *h_ws = b + L.off_h, *pre_ws = b + L.off_pre;
        SMILE_TRY(launch_grouped_gemm_nt(d.dtype, GroupedGemm{xe, w1, h_ws, pre_ws, kept_count, N, C, F, dm, act, nullptr, nullptr, d.tune, d.T}, s));
        h = h_ws;
        pre = pre_ws;
    }
    // kernels that read operands with the contraction index as the slow index: no transposed copies
    const long long cd = (long long)C * dm, cf = (long long)C * F, df = (long long)dm * F;
    auto product = [&](const void *x, const void *w, void *y, const void *aux, const int32_t *rows, const int32_t *k, int M,
                       int Nout, int K, int ldx, int ldw, long long sx, long long sw, long long sy, bool xt, int post) {
        if (is_half(d.dtype))
            return launch_grouped_gemm_t(d.dtype, TransposedGemm{x, w, y, aux, rows, k, N, M, Nout, K, ldx, ldw, sx, sw, sy, xt, true,
                                                                 post, d.tune, d.T}, s);
        F32Gemm g{};
        g.x = x, g.w = w, g.y = y, g.aux = aux, g.rows_valid = rows, g.k_valid = k;
        g.N = N, g.Mrows = M, g.Nout = Nout, g.K = K, g.ldx = ldx, g.ldw = ldw, g.sx = sx, g.sw = sw, g.sy = sy;
        g.x_transposed = xt, g.w_transposed = true, g.post = post, g.tune = d.tune;
        return launch_grouped_gemm_f32(g, s);
    };
    // dpre[r,f] = (sum_c dye[r,c] W2[c,f]) * act'(pre[r,f])
    SMILE_TRY(product(dye, w2, dpre, pre, kept_count, nullptr, C, F, dm, dm, F, cd, df, cf, false, act));
    // dW2[c,f] = sum_r dye[r,c] h[r,f]
    SMILE_TRY(product(dye, h, dw2, nullptr, nullptr, kept_count, dm, F, C, dm, F, cd, cf, df, true, 0));
    // dxe[r,k] = sum_f dpre[r,f] W1[f,k]
    SMILE_TRY(product(dpre, w1, dxe, nullptr, kept_count, nullptr, C, dm, F, F, dm, cf, df, cd, false, 0));
    // dW1[f,k] = sum_r dpre[r,f] xe[r,k]
    SMILE_TRY(product(dpre, xe, dw1, nullptr, nullptr, kept_count, F, dm, C, F, dm, cf, cd, df, true, 0));
#undef SMILE_TRY
    return hipSuccess;
}

// The vector-ALU kernels (fp32, fp16, wide routers)
static hipError_t launch_router_grad_valu(const LayerDesc &d, const RouterGradIo &io, bool with_dx, bool with_gw, float *partial, int blocks, hipStream_t s)
{
    const int ppr = d.d_model * elem_size(d.dtype) / 16, lpr = lanes_per_row(ppr), per_block = kThreads / lpr;
    const int dx_blocks = with_dx ? (d.T + per_block - 1) / per_block : 0, col_blocks = (d.d_model + kGwCols - 1) / kGwCols;
    // In one launch while a CU has at most two workgroups of dx (us: fp32 2048 x 256, 256 of them, 4.7 + 9.6 -> 7.5): beyond, the registers and
    // the LDS of the other part keep theirs from sharing a CU (fp16 8192 x 768, 1024 of them, 13.3 + 12.1 -> 28.3).
    if (with_dx && with_gw && dx_blocks > 2 * (d.tune.cus > 0 ? d.tune.cus : 256)) {
        const hipError_t err = launch_router_grad_valu(d, io, true, false, nullptr, 0, s);
        return err == hipSuccess ? launch_router_grad_valu(d, io, false, true, partial, blocks, s) : err;
    }
    const DispatchBackwardArgs dx{static_cast<const u32x4 *>(io.dxe), io.group_idx, io.local_idx, io.slot, io.dlp, io.dlq,
                                  static_cast<const u32x4 *>(io.w_inter), static_cast<const u32x4 *>(io.w_intra), static_cast<u32x4 *>(io.dx),
                                  d.T, ppr, d.n_groups, d.m_local, d.capacity};
    const GateWeightsArgs gw{io.x, io.dlp, io.dlq, partial, d.T, d.d_model, d.n_groups, d.m_local};
    const dim3 block(kThreads), grid = with_dx ? dim3(dx_blocks + (with_gw ? blocks * col_blocks : 0)) : dim3(blocks, col_blocks);
    auto launch = [&](auto dx_tag, auto gw_tag) {
        constexpr bool DX = decltype(dx_tag)::value, GW = decltype(gw_tag)::value;
        SMILE_DTYPE_SWITCH(d.dtype, SMILE_BWD_LPR_SWITCH(
            DX ? lpr : 8, SMILE_LAUNCH((router_grad_kernel<DT, (DX ? L : 8), DX, GW>), grid, block, 0, s, dx, gw, dx_blocks, col_blocks)));
    };
    if (with_dx && with_gw) launch(std::true_type{}, std::true_type{});
    else if (with_dx) launch(std::true_type{}, std::false_type{});
    else launch(std::false_type{}, std::true_type{});
    return hipGetLastError();
}

hipError_t launch_router_gradients(const LayerDesc &d, void *workspace, const RouterGradIo &io, bool with_dx, bool with_gw, hipStream_t s)
{
    // Tuning::router_grad_mfma = 0 keeps the vector-ALU kernels (tuning / comparison runs)
    const bool mfma = d.tune.router_grad_mfma != 0, dx_mfma = mfma && dispatch_backward_mfma_applies(d), gw_mfma = mfma && gate_weights_mfma_applies(d);
    const BackwardLayout L = backward_workspace_layout(d);
    float *partial = with_gw ? reinterpret_cast<float *>(static_cast<char *>(workspace) + L.off_gw_partial) : nullptr;
    int blocks = L.gw_blocks, tokens = kGwTokens;
    if (gw_mfma) {
        tokens = gate_weights_mfma_block_tokens(d, kGwTokens);
        blocks = (d.T + tokens - 1) / tokens;   // <= L.gw_blocks: the partial sums fit the same scratch area
    }
    hipError_t err = hipSuccess;
    if (with_dx && with_gw && dx_mfma == gw_mfma) {
        err = dx_mfma ? launch_router_grad_mfma(d, io, true, true, partial, blocks, tokens, s)
                      : launch_router_grad_valu(d, io, true, true, partial, blocks, s);
    } else {
        if (with_dx) err = dx_mfma ? launch_router_grad_mfma(d, io, true, false, nullptr, 0, 0, s) : launch_router_grad_valu(d, io, true, false, nullptr, 0, s);
        if (with_gw && err == hipSuccess)
            err = gw_mfma ? launch_router_grad_mfma(d, io, false, true, partial, blocks, tokens, s)
                          : launch_router_grad_valu(d, io, false, true, partial, blocks, s);
    }
    if (!with_gw || err != hipSuccess) return err;
    const long long total = (long long)(d.n_groups + d.m_local) * d.d_model;
    const long long groups = (total + kThreads - 1) / kThreads;   // workgroups of a thread an element
    if (blocks >= 48 && groups < (d.tune.cus > 0 ? d.tune.cus : 256))
        SMILE_LAUNCH(gate_weights_reduce_kernel<8>, dim3((unsigned)((total + kThreads / 8 - 1) / (kThreads / 8))), dim3(kThreads), 0, s, partial,
                     io.dw_inter, io.dw_intra, blocks, d.d_model, d.n_groups, d.m_local);
    else
        SMILE_LAUNCH(gate_weights_reduce_kernel<1>, dim3((unsigned)groups), dim3(kThreads), 0, s, partial, io.dw_inter, io.dw_intra, blocks,
                     d.d_model, d.n_groups, d.m_local);
    return hipGetLastError();
}

}  // namespace smile
