// Dispatch and combine: the token <-> expert-buffer row permutation (Section 3.2.1; on one GPU the
// paper's inter- and intra-node hops are composed into a single row move) and the gate-weighted
// return (Eq. 3).  Both are pure HBM streaming: a row is d*elem bytes (1.5-2 KiB for the bf16
// configurations), moved as 16-byte pieces; 8-32 consecutive lanes own a row, so every access is a
// run of full cache lines, the routing indices are read once per row, and up to kPieces loads are
// in flight per lane.
#include "permute_device.hpp"

namespace smile {

namespace {

constexpr int kThreads = 256;

// Row mapping shared by the kernels below: LPR consecutive lanes own one token row and walk its ppr
// 16-byte pieces LPR at a time (so every access of those lanes is one contiguous run), kThreads / LPR
// rows per workgroup.  The routing indices are read once per row, not once per piece.
template <int LPR>
struct RowLanes {
    static constexpr int kRowsPerBlock = kThreads / LPR;
    int t, sub;
    __device__ __forceinline__ RowLanes() : t(blockIdx.x * kRowsPerBlock + threadIdx.x / LPR), sub(threadIdx.x % LPR) {}
};

// xe[(g*m+l)*C + slot] <- x[t] for kept tokens.  ppr = 16-byte pieces per row.
template <int LPR>
__global__ __launch_bounds__(kThreads) void dispatch_kernel(
    const u32x4 *__restrict__ x, const int32_t *__restrict__ group_idx, const int32_t *__restrict__ local_idx,
    const int32_t *__restrict__ slot, u32x4 *__restrict__ xe, int T, int ppr, int m, int C)
{
    const RowLanes<LPR> rl;
    if (rl.t >= T) return;
    const int sl = slot[rl.t];
    if (sl < 0) return;
    const size_t row = (size_t)(group_idx[rl.t] * m + local_idx[rl.t]) * C + sl;
    move_row<LPR>(x + (size_t)rl.t * ppr, xe + row * ppr, ppr, rl.sub, [](u32x4 v) { return v; });
}

// First hop alone: xg[g*rows + pos_in_group] <- x[t] while the group's buffer has a row for it.
template <int LPR>
__global__ __launch_bounds__(kThreads) void dispatch_hop1_kernel(
    const u32x4 *__restrict__ x, const int32_t *__restrict__ group_idx, const int32_t *__restrict__ pos_in_group,
    u32x4 *__restrict__ xg, int T, int ppr, int rows)
{
    const RowLanes<LPR> rl;
    if (rl.t >= T) return;
    const int pos = pos_in_group[rl.t];
    if (pos < 0 || pos >= rows) return;
    const size_t row = (size_t)group_idx[rl.t] * rows + pos;
    move_row<LPR>(x + (size_t)rl.t * ppr, xg + row * ppr, ppr, rl.sub, [](u32x4 v) { return v; });
}

// Second hop alone: xe[(g*m+l)*C + slot] <- xg[g*rows + pos_in_group] for kept tokens.
template <int LPR>
__global__ __launch_bounds__(kThreads) void dispatch_hop2_kernel(
    const u32x4 *__restrict__ xg, const int32_t *__restrict__ group_idx, const int32_t *__restrict__ local_idx,
    const int32_t *__restrict__ pos_in_group, const int32_t *__restrict__ slot, u32x4 *__restrict__ xe,
    int T, int ppr, int m, int C, int rows)
{
    const RowLanes<LPR> rl;
    if (rl.t >= T) return;
    const int sl = slot[rl.t], pos = pos_in_group[rl.t];
    if (sl < 0 || sl >= C || pos < 0 || pos >= rows) return;
    const int g = group_idx[rl.t];
    const size_t src = (size_t)g * rows + pos, dst = (size_t)(g * m + local_idx[rl.t]) * C + sl;
    move_row<LPR>(xg + src * ppr, xe + dst * ppr, ppr, rl.sub, [](u32x4 v) { return v; });
}

// Dispatch fused with the last routing step of a chained forward pass with many routing blocks (scanned histograms): every
// thread derives the token's final slot from the workspace (block offset of its expert + rank inside the block,
// dropped at or beyond C); the thread moving piece 0 of a token also writes slot / pos_in_group and
// the slot -> token map; the output rows of dropped tokens are zeroed here (the down-projection
// returns the gate-weighted rows of the kept ones, so no combine kernel follows).
template <int LPR>
__global__ __launch_bounds__(kThreads) void dispatch_finalize_kernel(RouteIo io, Workspace ws, RouteTail tail, int T, int RB, int Bp, int ppr,
                                                                     int n, int m, int C, float alpha, float beta)
{
    // Eq. 4 from the (complete) routing statistics, by the first wave of the last workgroup
    if (tail.loss3 && blockIdx.x == gridDim.x - 1 && threadIdx.x < 64)
        aux_loss_wave(io.group_count, io.local_count, io.p_sum, io.q_sum, T, n, m, alpha, beta, tail.loss3);
    const RowLanes<LPR> rl;
    if (rl.t >= T) return;
    const int t = rl.t, b = t / RB;
    const int g = io.group_idx[t], e = g * m + io.local_idx[t];
    const int rank = ws.block_expert_hist[(size_t)e * Bp + b] + ws.rank_in_block[t];
    const int sl = rank < C ? rank : -1;
    if (rl.sub == 0) {
        io.slot[t] = sl;
        io.pos_in_group[t] = ws.block_group_hist[(size_t)g * Bp + b] + ws.pos_in_block[t];
        if (sl >= 0) tail.slot_token[(size_t)e * C + sl] = t;   // for the down-projection's gate-weighted return
    }
    if (sl < 0) {   // a dropped token's output row is zero (Eq. 3 gives it no expert output)
        zero_row(static_cast<u32x4 *>(tail.y) + (size_t)t * ppr, ppr, rl.sub, LPR);
        return;
    }
    move_row<LPR>(static_cast<const u32x4 *>(tail.x) + (size_t)t * ppr, static_cast<u32x4 *>(tail.xe) + ((size_t)e * C + sl) * ppr, ppr, rl.sub,
                  [](u32x4 v) { return v; });
}

// DT: storage type of the piece (SMILE_DTYPE_*)
template <int DT>
__device__ __forceinline__ u32x4 scale_piece(u32x4 v, float gt)
{
    u32x4 r;
    if constexpr (DT == SMILE_DTYPE_BF16) {
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = Half<__bf16>::pack(Half<__bf16>::lo(v[k]) * gt, Half<__bf16>::hi(v[k]) * gt);
    } else if constexpr (DT == SMILE_DTYPE_F16) {
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = Half<_Float16>::pack(Half<_Float16>::lo(v[k]) * gt, Half<_Float16>::hi(v[k]) * gt);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = __float_as_uint(__uint_as_float(v[k]) * gt);
    }
    return r;
}

// y[t] <- gate[t] * ye[(g*m+l)*C + slot] for kept tokens, 0 for dropped ones.
template <int DT, int LPR>
__global__ __launch_bounds__(kThreads) void combine_kernel(
    const u32x4 *__restrict__ ye, const int32_t *__restrict__ group_idx, const int32_t *__restrict__ local_idx,
    const int32_t *__restrict__ slot, const float *__restrict__ gate, u32x4 *__restrict__ y,
    int T, int ppr, int m, int C)
{
    const RowLanes<LPR> rl;
    if (rl.t >= T) return;
    const int sl = slot[rl.t];
    u32x4 *dst = y + (size_t)rl.t * ppr;
    if (sl < 0) {
        zero_row(dst, ppr, rl.sub, LPR);
        return;
    }
    const float gt = gate[rl.t];
    const size_t row = (size_t)(group_idx[rl.t] * m + local_idx[rl.t]) * C + sl;
    move_row<LPR>(ye + row * ppr, dst, ppr, rl.sub, [gt](u32x4 v) { return scale_piece<DT>(v, gt); });
}

}  // namespace

#define SMILE_LPR_SWITCH(lpr, CALL)          \
    switch (lpr) {                           \
    case 8: { constexpr int L = 8; CALL; } break;   \
    case 16: { constexpr int L = 16; CALL; } break; \
    default: { constexpr int L = 32; CALL; } break; \
    }

hipError_t launch_dispatch(const smile_layer_desc &d, const void *x, const int32_t *group_idx,
                           const int32_t *local_idx, const int32_t *slot, void *xe, hipStream_t s)
{
    const int ppr = d.d_model * elem_size(d.dtype) / 16;
    const int lpr = lanes_per_row(ppr);
    const dim3 grid((d.T + kThreads / lpr - 1) / (kThreads / lpr)), block(kThreads);
    SMILE_LPR_SWITCH(lpr, SMILE_LAUNCH(dispatch_kernel<L>, grid, block, 0, s, static_cast<const u32x4 *>(x),
                                             group_idx, local_idx, slot, static_cast<u32x4 *>(xe), d.T, ppr, d.m_local,
                                             d.capacity));
    return hipGetLastError();
}

hipError_t launch_dispatch_hop1(const smile_layer_desc &d, const void *x, const int32_t *group_idx,
                                const int32_t *pos_in_group, int group_rows, void *xg, hipStream_t s)
{
    const int ppr = d.d_model * elem_size(d.dtype) / 16;
    const int lpr = lanes_per_row(ppr);
    const dim3 grid((d.T + kThreads / lpr - 1) / (kThreads / lpr)), block(kThreads);
    SMILE_LPR_SWITCH(lpr, SMILE_LAUNCH(dispatch_hop1_kernel<L>, grid, block, 0, s, static_cast<const u32x4 *>(x),
                                             group_idx, pos_in_group, static_cast<u32x4 *>(xg), d.T, ppr, group_rows));
    return hipGetLastError();
}

hipError_t launch_dispatch_hop2(const smile_layer_desc &d, const void *xg, const int32_t *group_idx,
                                const int32_t *local_idx, const int32_t *pos_in_group, const int32_t *slot,
                                int group_rows, void *xe, hipStream_t s)
{
    const int ppr = d.d_model * elem_size(d.dtype) / 16;
    const int lpr = lanes_per_row(ppr);
    const dim3 grid((d.T + kThreads / lpr - 1) / (kThreads / lpr)), block(kThreads);
    SMILE_LPR_SWITCH(lpr, SMILE_LAUNCH(dispatch_hop2_kernel<L>, grid, block, 0, s,
                                             static_cast<const u32x4 *>(xg), group_idx, local_idx, pos_in_group, slot,
                                             static_cast<u32x4 *>(xe), d.T, ppr, d.m_local, d.capacity, group_rows));
    return hipGetLastError();
}

hipError_t launch_dispatch_finalize(const smile_layer_desc &d, const Workspace &ws, const RoutePlan &p, const RouteIo &io,
                                    const RouteTail &tail, hipStream_t s)
{
    const int ppr = d.d_model * elem_size(d.dtype) / 16;
    const int lpr = lanes_per_row(ppr);
    const dim3 grid((d.T + kThreads / lpr - 1) / (kThreads / lpr)), block(kThreads);
    SMILE_LPR_SWITCH(lpr, SMILE_LAUNCH(dispatch_finalize_kernel<L>, grid, block, 0, s, io, ws, tail, d.T, p.rb, p.stride, ppr, d.n_groups,
                                       d.m_local, d.capacity, d.alpha, d.beta));
    return hipGetLastError();
}

hipError_t launch_combine(const smile_layer_desc &d, const void *ye, const int32_t *group_idx,
                          const int32_t *local_idx, const int32_t *slot, const float *gate, void *y, hipStream_t s)
{
    const int ppr = d.d_model * elem_size(d.dtype) / 16;
    const int lpr = lanes_per_row(ppr);
    const dim3 grid((d.T + kThreads / lpr - 1) / (kThreads / lpr)), block(kThreads);
#define SMILE_COMBINE(DT)                                                                                          \
    SMILE_LPR_SWITCH(lpr, SMILE_LAUNCH((combine_kernel<DT, L>), grid, block, 0, s,                             \
                                             static_cast<const u32x4 *>(ye), group_idx, local_idx, slot, gate,       \
                                             static_cast<u32x4 *>(y), d.T, ppr, d.m_local, d.capacity))
    if (d.dtype == SMILE_DTYPE_BF16) { SMILE_COMBINE(SMILE_DTYPE_BF16); }
    else if (d.dtype == SMILE_DTYPE_F16) { SMILE_COMBINE(SMILE_DTYPE_F16); }
    else { SMILE_COMBINE(SMILE_DTYPE_F32); }
#undef SMILE_COMBINE
    return hipGetLastError();
}

}  // namespace smile
