// Bi-level top-1 routing with per-expert capacity (Section 3.2.1, Section 3.2.2 statistics,
// Section 4.2 capacity).  Tokens are cut into routing blocks; a workgroup decides one block, and the blocks are put in
// order afterwards:
//
//   gate_logits_route  one workgroup per block of 16, 32, 64 or 256 tokens: (chained forward pass, up to 64 tokens) the router
//                      logits of the block on the matrix cores, then from an LDS tile of the logits: top-1 group and local expert, the
//                      two softmax probabilities (Eq. 1 read as a softmax), the gate p*q (Eq. 3), column sums of p and
//                      q, the token's rank among EARLIER tokens of the block with the same group / the same expert
//                      (wave64 ballots + per-wave LDS counters combined after one barrier), block histograms.
//   route_finish       one workgroup per block: the offsets of the block (sum of the histograms of the blocks before
//                      it, one 16-byte load per lane and column), final slots with the capacity cut, and, as the caller
//                      needs, the slot -> token map, zero output rows of dropped tokens, the row move into the expert
//                      buffers; the first and last workgroup write the totals, the sums and the loss.
//
// Two launches; a batch small enough for a single workgroup (route_plan) needs only the first one.  More
// than 256 blocks, or histograms too large for every workgroup to read, take the column scan (route_scan) as a
// launch of its own, and routers too wide for an LDS tile the kernel that re-reads its rows (route_decide).
//
// With a group capacity (a first-hop buffer of Cg rows per group, Section 3.2.3) route_first_hop
// recomputes the in-block expert ranks over the tokens whose stage-1 position is below Cg only (the others get a rank
// no capacity admits) between the two.
//
// Histograms and partial sums are stored per column, [column][block], so that one load of a wave covers 64-256 blocks.
//
// Everything that decides an integer is integer arithmetic or an fp32 compare of the logits,
// so the result depends only on the logits and the token order, never on the launch geometry.  No
// atomics order, no inter-workgroup waiting, no memory that must be cleared beforehand.
#include <algorithm>

#include "gate_device.hpp"
#include "permute_device.hpp"

namespace smile {

namespace {

typedef mfma_f32x4 f32x4;

__device__ __forceinline__ unsigned long long lanemask_lt()
{
    const unsigned lane = __lane_id();
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Lanes of this wave (among `valid` ones) holding the same key; key < 2^bits.
__device__ __forceinline__ unsigned long long match_any(int key, int bits, bool valid)
{
    unsigned long long mask = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
        const bool set = (key >> b) & 1;
        const unsigned long long bal = __ballot(valid && set);
        mask &= set ? bal : ~bal;
    }
    return mask;
}

// exp(v) for v <= 0 by the hardware exp2 (v_exp_f32 is accurate to about 1 ulp; the scaling by
// log2(e) adds a relative error of about |v| * 6e-8, far inside the 1e-5 tolerance of the gates).
// The kernel is instruction-bound (one wave per SIMD at T = 65536), which is why this matters.
__device__ __forceinline__ float exp_neg(float v)
{
    return __builtin_amdgcn_exp2f(v * 1.4426950408889634f);
}

constexpr int kLoadChunk = 8;   // logits fetched per lane before any of them is used (loads in flight)

// kLoadChunk biased logits starting at column i0 (one fp32 add each; columns >= len give `fill`).
// All loads are issued before the first use, so a lane waits for memory once per chunk, not per logit.
__device__ __forceinline__ void load_biased(const float *__restrict__ row, const float *__restrict__ bias, int i0,
                                            int len, float fill, float (&a)[kLoadChunk])
{
    float v[kLoadChunk], bv[kLoadChunk];
#pragma unroll
    for (int k = 0; k < kLoadChunk; ++k) {
        const int i = min(i0 + k, len - 1);
        v[k] = row[i];
        bv[k] = bias ? bias[i] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < kLoadChunk; ++k) a[k] = i0 + k < len ? (bias ? __fadd_rn(v[k], bv[k]) : v[k]) : fill;
}

// Top-1 over `len` biased logits: lowest index of the maximum, and 1/sum(exp(a - max)) which is
// the softmax probability of that maximum.  `row` and `bias` (may be null) are read twice.
__device__ __forceinline__ void top1_softmax(const float *__restrict__ row, const float *__restrict__ bias,
                                             int len, int &arg, float &mx, float &inv_z)
{
    arg = 0;
    mx = -INFINITY;
    float a[kLoadChunk];
    for (int i0 = 0; i0 < len; i0 += kLoadChunk) {
        load_biased(row, bias, i0, len, -INFINITY, a);
#pragma unroll
        for (int k = 0; k < kLoadChunk; ++k)
            if (a[k] > mx) { mx = a[k]; arg = i0 + k; }   // strict: the lowest index of the maximum wins
    }
    float z = 0.f;
    for (int i0 = 0; i0 < len; i0 += kLoadChunk) {
        load_biased(row, bias, i0, len, -INFINITY, a);
#pragma unroll
        for (int k = 0; k < kLoadChunk; ++k) z += exp_neg(a[k] - mx);   // exp2(-inf) = 0 for the padding
    }
    inv_z = 1.0f / z;
}

constexpr int kColChunk = 32;   // probability columns summed per LDS pass

// Column sums over the block's tokens of prob[t, c] = exp(a[t,c] - mx_t) * inv_z_t, written to out[c * out_stride]:
// the probabilities go through an LDS tile, 32 columns at a time, and are summed
// in a fixed order (8 segments of 32 tokens serially, then the 8 partials serially).  GET(c) yields the biased
// logit of column c.
template <typename Get>
__device__ __forceinline__ void block_column_sums_tile(Get get, int len, float mx, float inv_z, bool valid,
                                                       float (*tile)[kColChunk + 1], float (*part)[kColChunk],
                                                       float *__restrict__ out, int out_stride)
{
    const int tid = threadIdx.x;
    for (int c0 = 0; c0 < len; c0 += kColChunk) {
        const int w = min(kColChunk, len - c0);
        get(c0, w, tile[tid]);   // tile[tid][k] = biased logit of column c0 + k for k < w (valid threads only)
        if (valid) {
            for (int k = 0; k < w; ++k) tile[tid][k] = exp_neg(tile[tid][k] - mx) * inv_z;
        } else {
            for (int k = 0; k < w; ++k) tile[tid][k] = 0.f;
        }
        __syncthreads();
        const int col = tid & (kColChunk - 1), seg = tid / kColChunk;   // 8 segments of 32 tokens
        if (col < w) {
            float s = 0.f;
            for (int j = 0; j < kRouteBlock / 8; ++j) s += tile[seg * (kRouteBlock / 8) + j][col];
            part[seg][col] = s;
        }
        __syncthreads();
        if (tid < w) {
            float s = 0.f;
            for (int sg = 0; sg < 8; ++sg) s += part[sg][tid];
            out[(size_t)(c0 + tid) * out_stride] = s;
        }
        __syncthreads();
    }
}

// Zero the output rows of the block's dropped tokens (to[tk] < 0; Eq. 3 gives them no expert output): a wave looks at 64 tokens
// at a time and takes every waves-th of the dropped ones.
__device__ __forceinline__ void zero_dropped_rows(const int32_t *to, int live, int t0, u32x4 *y, int ppr, int wave, int waves)
{
    const int lane = __lane_id();
    int k = 0;
    for (int tk0 = 0; tk0 < live; tk0 += 64) {
        unsigned long long mask = __ballot(tk0 + lane < live && to[min(tk0 + lane, live - 1)] < 0);
        for (; mask; mask &= mask - 1, k = k + 1 == waves ? 0 : k + 1)
            if (k == wave) zero_row(y + (size_t)(t0 + tk0 + __ffsll((long long)mask) - 1) * ppr, ppr, lane, 64);
    }
}

// ------------------------------------------------------------------------------------ decision from an LDS tile

struct RouteArgs {
    const void *x, *w_inter, *w_intra;   // GATE kernels: the logits are computed here
    int d;
    RouteIo io;
    int T, n, m, bits_n, bits_N, Bp;     // Bp: blocks per column of the histograms
    Workspace ws;
    // a batch of one block is finished here
    bool one;
    int C, Cg, ppr;
    RouteTail tail;
    float alpha, beta;
};

template <int CTRL>
__device__ __forceinline__ int dpp(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true); }
template <int CTRL>
__device__ __forceinline__ float dpp(float v) { return __int_as_float(dpp<CTRL>(__float_as_int(v))); }

// F combines the lane's value with those of the other lanes of its aligned group of P (4, 8 or 16), one step per factor of two:
// quad permutations, then mirrored halves (every lane of a finished half holds the same value).
template <int P, typename F>
__device__ __forceinline__ void group_reduce(F step)
{
    step(std::integral_constant<int, 0xB1>{});                       // lane ^ 1
    step(std::integral_constant<int, 0x4E>{});                       // lane ^ 2
    if constexpr (P >= 8) step(std::integral_constant<int, 0x141>{});    // mirror of 8
    if constexpr (P >= 16) step(std::integral_constant<int, 0x140>{});   // mirror of 16
}

// LDS written before by lanes of this wave may be read after by others of it (a wave's LDS operations complete in order, so
// this only holds the compiler back).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Softmax and top-1 of one logit row in LDS by the P neighbouring lanes that own the token (columns part, part + P, ...):
// lowest index of the maximum of row + bias, its probability, and the row overwritten with all probabilities (zeros
// for a token that does not exist).  K > 0: at most K P columns, held in registers between the passes.
// Every lane adds the whole denominator up in column order, from the exponentials in LDS: p_top, and with it the gate,
// then has the same bits for every block size and in the kernel for very wide routers.
template <int P, int K>
__device__ __forceinline__ void softmax_top1(float *row, const float *__restrict__ bias, int len, int part, bool valid, int &arg,
                                             float &p_top)
{
    float mx = -INFINITY, z = 0.f, v[K > 0 ? K : 1];
    arg = len;
    auto look = [&](int c, float a) {
        if (a > mx) { mx = a; arg = c; }   // strict: the lowest index of the maximum wins
    };
    if constexpr (K > 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int c = part + k * P;
            v[k] = c < len ? row[c] : -INFINITY;
            if (bias && c < len) v[k] = __fadd_rn(v[k], bias[c]);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) look(part + k * P, v[k]);
    } else {
        for (int c = part; c < len; c += P) {
            float a = row[c];
            if (bias) { a = __fadd_rn(a, bias[c]); row[c] = a; }
            look(c, a);
        }
    }
    group_reduce<P>([&](auto ctrl) {
        const float ov = dpp<decltype(ctrl)::value>(mx);
        const int oa = dpp<decltype(ctrl)::value>(arg);
        if (ov > mx || (ov == mx && oa < arg)) { mx = ov; arg = oa; }
    });
    if (arg == len) arg = 0;   // nothing above -inf: a row of -inf or NaN
    if constexpr (K > 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            v[k] = exp_neg(v[k] - mx);
            if (part + k * P < len) row[part + k * P] = v[k];
        }
    } else {
        for (int c = part; c < len; c += P) row[c] = exp_neg(row[c] - mx);
    }
    wave_lds_fence();
#pragma unroll 8
    for (int c = 0; c < len; ++c) z += row[c];
    wave_lds_fence();
    p_top = 1.0f / z;
    if constexpr (K > 0) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (part + k * P < len) row[part + k * P] = valid ? v[k] * p_top : 0.f;
    } else {
        for (int c = part; c < len; c += P) row[c] = valid ? row[c] * p_top : 0.f;
    }
}

// Waves per SIMD the registers must leave room for: four 4-wave blocks per CU hide each other's reads of x; with five column tiles a
// chunk's operands and accumulators alone are more than 128 registers, and one column tile spends its registers on chunks in flight instead
// (170 with three chunks over 64 tokens: two blocks per CU).
constexpr int gate_waves_per_simd(int NT, int CT) { return NT == 1024 || (CT > 1 && CT <= 3) ? 4 : 2; }

// Chunks in flight of the logits (gate_partial's U): as many, up to three, as fit the registers without spilling -- 8 (RT + CT) of
// operands a chunk, 4 RT CT of accumulators, the addresses and about 24 others, in the 128 of four waves per SIMD, else in about 170.
// One chunk more spilled 44-96 bytes per lane: with 40 columns 8192 x 768 took 17.2 us instead of 13.9, 4096 x 768 14.8 instead of 12.7.
constexpr int gate_chunks_in_flight(int CT, int RT, int waves)
{
    for (int u = 3; u > 1; --u)
        if (8 * u * (RT + CT) + 4 * RT * CT + RT + 2 * CT + 24 <= (waves == 4 ? 128 : 168)) return u;
    return 1;
}

// NT threads, P per token: blocks of NT / P tokens.  GATE: logits from x and the router weights (16 * CT columns per pass
// over the block's rows, which come from L2 after the first), else from memory.
// Dynamic LDS (route_lds_bytes): logit / probability tile, 8 segment sums per column, packed decisions, per-wave counters,
// counts and sums for the loss.
// Bound: the read of x (GATE), else latency.  One CU draws about 28 GB/s from HBM however much it requests, so the blocks
// are as small as leaves 256 of them; several threads per token because a token's serial loops over its columns are what
// a wave spends its time on.  Measured against a gate kernel and a decision kernel with one thread per token (us, routing
// and block order included): 512 tokens fp32 13 -> 10, 128 tokens of 768 17 -> 11, 8192 of 768 20 -> 16, 16384 of
// 1024 22 -> 22, 32768 of 768 with 16 + 8 columns 36 -> 33 and with 129 columns 117 -> 70; whole layers of 64-wide experts gain
// the launch too (16384 of 1024: 64 -> 50, 65536 of 1024: 170 -> 141).
template <int DT, int CT, int NT, int P, bool GATE>
__global__ __launch_bounds__(NT, gate_waves_per_simd(NT, CT)) void gate_logits_route_kernel(RouteArgs a)
{
    constexpr int RB = NT / P, kRankWaves = (RB + 63) / 64, kWaves = NT / 64;
    extern __shared__ float lds_f[];
    const int n = a.n, m = a.m, N = n * m, cols = n + m, stride = cols | 1, NC = N + n;
    float *tile = lds_f;                                                    // [RB][stride]
    float *seg_sum = tile + RB * stride;                                    // [8][cols]
    int32_t *decision = reinterpret_cast<int32_t *>(seg_sum + 8 * cols);    // [RB] e | g << 12, -1 beyond T
    int32_t *hist = decision + RB;                                          // [kRankWaves][N experts, then n groups]
    int32_t *cnt = hist + kRankWaves * NC;                                  // [cols]  (one block only)
    float *sum = reinterpret_cast<float *>(cnt + cols);                     // [cols]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.x, t0 = b * RB, live = min(RB, a.T - t0);

    constexpr bool WIDE = GATE && CT == kWideTiles;
    if (!WIDE)
        for (int i = tid; i < kRankWaves * NC; i += NT) hist[i] = 0;

    // logit rows between memory and the tile: a power-of-two number of neighbouring threads per row (no divisions)
    auto copy_rows = [&](auto to_lds, float *at, const float *src, float *dst, int len) {
        const int sh = min(32 - __clz(max(len, 2) - 1), 6), rows = NT >> sh;
        for (int r = tid >> sh; r < live; r += rows)
            for (int c = tid & ((1 << sh) - 1); c < len; c += 1 << sh) {
                if constexpr (decltype(to_lds)::value) at[r * stride + c] = src[(size_t)r * len + c];
                else dst[(size_t)r * len + c] = at[r * stride + c];
            }
    };
    if constexpr (WIDE) {
        f32x4 logits[CT];
        gate_wide<DT>(a.x, a.w_inter, a.w_intra, t0, a.T, a.d, n, m, reinterpret_cast<gate_piece *>(lds_f), logits);
        __syncthreads();   // the stages lie where the tile and the counters come
        for (int i = tid; i < kRankWaves * NC; i += NT) hist[i] = 0;
        float *at = tile + (wave * 16 + (lane >> 4) * 4) * stride + (lane & 15);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
            if (ct * 16 + (lane & 15) < cols)
#pragma unroll
                for (int i = 0; i < 4; ++i) at[i * stride + ct * 16] = logits[ct][i];
        __syncthreads();
    } else if constexpr (GATE) {
        constexpr int RT = RB < 64 ? RB / 16 : 4;               // row tiles per unit of four waves: at most 64 tokens
        constexpr int kAhead = gate_chunks_in_flight(CT, RT, gate_waves_per_simd(NT, CT));
        const int unit = wave / kGateWaves, uw = wave % kGateWaves, r16 = lane & 15, kg = lane >> 4;
        const bool any = unit * 64 < live;
#pragma unroll 1
        for (int col0 = 0; col0 < cols; col0 += 16 * CT) {
            f32x4 acc[RT][CT];
            if (any) gate_partial<DT, CT, RT, kAhead>(a.x, a.w_inter, a.w_intra, t0 + unit * 64, a.T, a.d, n, m, col0, uw, acc);
            // the four partial sums are added in wave order (all reads of a turn before its writes)
            float *at = tile + (unit * 64 + kg * 4) * stride + col0 + r16;
#pragma unroll 1
            for (int w = 0; w < kGateWaves; ++w) {
                if (any && uw == w) {
                    if (w > 0) {
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                            for (int ct = 0; ct < CT; ++ct)
                                if (col0 + ct * 16 + r16 < cols)
#pragma unroll
                                    for (int i = 0; i < 4; ++i) acc[rt][ct][i] = at[(rt * 16 + i) * stride + ct * 16] + acc[rt][ct][i];
                    }
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                        for (int ct = 0; ct < CT; ++ct)
                            if (col0 + ct * 16 + r16 < cols)
#pragma unroll
                                for (int i = 0; i < 4; ++i) at[(rt * 16 + i) * stride + ct * 16] = acc[rt][ct][i];
                }
                __syncthreads();
            }
        }
    }
    if constexpr (GATE) {
        copy_rows(std::false_type{}, tile, nullptr, a.io.logits_inter + (size_t)t0 * n, n);
        copy_rows(std::false_type{}, tile + n, nullptr, a.io.logits_intra + (size_t)t0 * m, m);
    } else {
        copy_rows(std::true_type{}, tile, a.io.logits_inter + (size_t)t0 * n, nullptr, n);
        copy_rows(std::true_type{}, tile + n, a.io.logits_intra + (size_t)t0 * m, nullptr, m);
    }
    __syncthreads();

    {   // ---- top-1 at both levels
        const int tk = tid / P, part = tid % P, t = t0 + tk;
        const bool valid = tk < live;
        int g, l;
        float p_top, q_top;
        float *row = tile + tk * stride;
        auto level = [&](float *r, const float *bias, int len, int &arg, float &top) {
            if (len <= 2 * P) softmax_top1<P, 2>(r, bias, len, part, valid, arg, top);
            else if (len <= 8 * P) softmax_top1<P, 8>(r, bias, len, part, valid, arg, top);
            else softmax_top1<P, 0>(r, bias, len, part, valid, arg, top);
        };
        level(row, a.io.bias_inter, n, g, p_top);
        level(row + n, a.io.bias_intra && valid ? a.io.bias_intra + (size_t)g * m : nullptr, m, l, q_top);
        if (part == 0) decision[tk] = valid ? (g * m + l) | (g << 12) : -1;
        if (valid && part == 0) {
            a.io.group_idx[t] = g;
            a.io.local_idx[t] = l;
            a.io.p_top[t] = p_top;
            a.io.q_top[t] = q_top;
            a.io.gate[t] = p_top * q_top;
        }
    }
    __syncthreads();

    // ---- rank among earlier tokens of this block with the same expert / the same group: one thread per token
    const bool ranks = tid < RB;
    const int dec = ranks ? decision[tid] : -1, e = dec & 4095, g = dec >> 12;
    const bool ok = dec >= 0;
    int rank = 0, pos = 0;
    // counts the tokens of `in` by expert (and group) into the per-wave counters
    auto count = [&](bool in, unsigned long long &me, unsigned long long *mg) {
        me = match_any(e, a.bits_N, in);
        if (mg) *mg = match_any(g, a.bits_n, in);
        if (in) {   // the last lane of each matching set publishes the wave's count
            if (63 - __clzll(me) == lane) hist[wave * NC + e] = __popcll(me);
            if (mg && 63 - __clzll(*mg) == lane) hist[wave * NC + N + g] = __popcll(*mg);
        }
    };
    auto total = [&](int i) {
        int c = 0;
#pragma unroll
        for (int w = 0; w < kRankWaves; ++w) c += hist[w * NC + i];
        return c;
    };
    unsigned long long me = 0, mg = 0;
    if (ranks) count(ok, me, &mg);
    // column sums of p and q in a fixed order: eight segments of the block, then the eight
    for (int seg = kWaves - 1 - wave; seg < 8; seg += kWaves)   // the waves without a rank start first
        for (int c = lane; c < cols; c += 64) {
            float s = 0.f;
#pragma unroll 8
            for (int j = 0; j < RB / 8; ++j) s += tile[(seg * (RB / 8) + j) * stride + c];
            seg_sum[seg * cols + c] = s;
        }
    __syncthreads();
    if (ok) {
        for (int w = 0; w < wave; ++w) {
            rank += hist[w * NC + e];
            pos += hist[w * NC + N + g];
        }
        rank += __popcll(me & lanemask_lt());
        pos += __popcll(mg & lanemask_lt());
    }
    for (int c = tid; c < cols; c += NT) {
        float s = seg_sum[c];
#pragma unroll
        for (int seg = 1; seg < 8; ++seg) s += seg_sum[seg * cols + c];
        if (a.one) {
            sum[c] = s;
            (c < n ? a.io.p_sum : a.io.q_sum - n)[c] = s;
        } else if (c < n) {
            a.ws.block_p_sum[(size_t)c * a.Bp + b] = s;
        } else {
            a.ws.block_q_sum[(size_t)(c - n) * a.Bp + b] = s;
        }
    }
    for (int j = tid; j < cols; j += NT) {   // counts by group and, summed over the groups, by local index
        int c = 0;
        if (j < n) c = total(N + j);
        else for (int i = 0; i < n; ++i) c += total(i * m + j - n);
        if (a.one) {
            cnt[j] = c;
            (j < n ? a.io.group_count : a.io.local_count - n)[j] = c;
        } else {
            a.ws.block_group_hist[(size_t)j * a.Bp + b] = c;
        }
    }
    if (!a.one) {
        for (int i = tid; i < N; i += NT) a.ws.block_expert_hist[(size_t)i * a.Bp + b] = total(i);
        if (ok) {
            a.ws.rank_in_block[t0 + tid] = rank;
            a.ws.pos_in_block[t0 + tid] = pos;
        }
        return;
    }

    // ---- the only block: ranks and counts are final
    for (int i = tid; i < N; i += NT) {
        const int c = total(i);
        a.io.expert_count[i] = c;
        if (a.Cg == 0) a.io.kept_count[i] = min(c, a.C);
    }
    if (a.Cg > 0) {   // ranks again over the tokens that pass the first hop
        const bool through = ok && pos < a.Cg;
        __syncthreads();
        for (int i = tid; i < kRankWaves * NC; i += NT) hist[i] = 0;
        __syncthreads();
        if (ranks) count(through, me, nullptr);
        __syncthreads();
        rank = kHop1Dropped;
        if (through) {
            rank = __popcll(me & lanemask_lt());
            for (int w = 0; w < wave; ++w) rank += hist[w * NC + e];
        }
        for (int i = tid; i < N; i += NT) a.io.kept_count[i] = min(total(i), a.C);
    }
    if (ok) {
        const int sl = rank < a.C ? rank : -1;
        a.io.slot[t0 + tid] = sl;
        a.io.pos_in_group[t0 + tid] = pos;
        if (sl >= 0 && a.tail.slot_token) a.tail.slot_token[(size_t)e * a.C + sl] = t0 + tid;
        decision[tid] = sl;
    }
    __syncthreads();
    if (a.tail.loss3 && wave == 0) aux_loss_wave(cnt, cnt + n, sum, sum + n, a.T, n, m, a.alpha, a.beta, a.tail.loss3);
    if (a.tail.y) zero_dropped_rows(decision, live, t0, static_cast<u32x4 *>(a.tail.y), a.ppr, wave, kWaves);
}

// ------------------------------------------------------------------------------------ decision, very wide routers

// One thread per token, rows re-read from memory by every pass, probabilities through a 32-column LDS tile.
// PERWAVE: every wave counts into its own copy of the LDS histograms and the copies are combined after one
// barrier (needs 4 x (N + n) counters); otherwise the four waves take turns on one copy.
template <bool PERWAVE>
__global__ __launch_bounds__(kRouteBlock) void route_decide_kernel(RouteArgs a)
{
    // [N] expert counters then [n] group counters (PERWAVE: one such set per wave)
    extern __shared__ int32_t hist[];
    __shared__ float tile[kRouteBlock][kColChunk + 1];
    __shared__ float part8[8][kColChunk];
    constexpr int kWaves = kRouteBlock / 64;

    const int T = a.T, n = a.n, m = a.m, N = n * m, NC = N + n;
    const int tid = threadIdx.x;
    const int b = blockIdx.x;
    const int t = b * kRouteBlock + tid;
    const bool valid = t < T;

    for (int i = tid; i < (PERWAVE ? kWaves : 1) * NC; i += kRouteBlock) hist[i] = 0;

    int g = 0, l = 0;
    float mx_p = 0.f, iz_p = 0.f, mx_q = 0.f, iz_q = 0.f;
    const float *rp = a.io.logits_inter + (size_t)(valid ? t : 0) * n;
    const float *rq = a.io.logits_intra + (size_t)(valid ? t : 0) * m;
    const float *bq = nullptr;
    if (valid) {
        top1_softmax(rp, a.io.bias_inter, n, g, mx_p, iz_p);
        bq = a.io.bias_intra ? a.io.bias_intra + (size_t)g * m : nullptr;
        top1_softmax(rq, bq, m, l, mx_q, iz_q);
        a.io.group_idx[t] = g;
        a.io.local_idx[t] = l;
        a.io.p_top[t] = iz_p;
        a.io.q_top[t] = iz_q;
        a.io.gate[t] = iz_p * iz_q;
    }
    __syncthreads();   // counters are zero

    // rank among earlier tokens of this block with the same expert / the same group
    const int e = g * m + l;
    const unsigned long long me = match_any(e, a.bits_N, valid);
    const unsigned long long mg = match_any(g, a.bits_n, valid);
    const unsigned long long lt = lanemask_lt();
    const int lane = __lane_id();
    const int wave = tid >> 6;
    if constexpr (PERWAVE) {
        int32_t *mine = hist + wave * NC;
        if (valid) {   // the last lane of each matching set publishes the wave's count
            if (63 - __clzll(me) == lane) mine[e] = __popcll(me);
            if (63 - __clzll(mg) == lane) mine[N + g] = __popcll(mg);
        }
        __syncthreads();
        if (valid) {
            int base_e = 0, base_g = 0;
            for (int w = 0; w < wave; ++w) {
                base_e += hist[w * NC + e];
                base_g += hist[w * NC + N + g];
            }
            a.ws.rank_in_block[t] = base_e + __popcll(me & lt);
            a.ws.pos_in_block[t] = base_g + __popcll(mg & lt);
        }
    } else {
        int32_t *ghist = hist + N;
        for (int w = 0; w < kWaves; ++w) {   // the waves take turns in token order
            if (wave == w && valid) {
                const int base_e = hist[e];
                const int base_g = ghist[g];
                a.ws.rank_in_block[t] = base_e + __popcll(me & lt);
                a.ws.pos_in_block[t] = base_g + __popcll(mg & lt);
                if (63 - __clzll(me) == lane) hist[e] = base_e + __popcll(me);
                if (63 - __clzll(mg) == lane) ghist[g] = base_g + __popcll(mg);
            }
            __syncthreads();
        }
    }
    auto total = [&](int i) {
        int c = 0;
#pragma unroll
        for (int w = 0; w < (PERWAVE ? kWaves : 1); ++w) c += hist[w * NC + i];
        return c;
    };
    for (int i = tid; i < N; i += kRouteBlock) a.ws.block_expert_hist[(size_t)i * a.Bp + b] = total(i);
    // counts by group, then by local index (summed over groups)
    for (int j = tid; j < n + m; j += kRouteBlock) {
        int c = 0;
        if (j < n) c = total(N + j);
        else for (int i = 0; i < n; ++i) c += total(i * m + j - n);
        a.ws.block_group_hist[(size_t)j * a.Bp + b] = c;
    }
    __syncthreads();

    auto from = [&](const float *row, const float *bias, int len) {
        return [=](int c0, int w, float *dst) {
            if (!valid) return;
            for (int i0 = 0; i0 < w; i0 += kLoadChunk) {
                float v[kLoadChunk];
                load_biased(row, bias, c0 + i0, len, -INFINITY, v);
#pragma unroll
                for (int k = 0; k < kLoadChunk; ++k)
                    if (i0 + k < w) dst[i0 + k] = v[k];
            }
        };
    };
    block_column_sums_tile(from(rp, a.io.bias_inter, n), n, mx_p, iz_p, valid, tile, part8, a.ws.block_p_sum + b, a.Bp);
    block_column_sums_tile(from(rq, bq, m), m, mx_q, iz_q, valid, tile, part8, a.ws.block_q_sum + b, a.Bp);
}

// ------------------------------------------------------------------------------------ order of the blocks

__device__ __forceinline__ int wave_sum(int v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sums over the blocks before block b (b <= 256) of `count` histogram columns ([column][Bp], Bp a multiple of 4): out(c, sum) is
// called by one lane per column.  A column of Bp counts is Bp / 4 16-byte loads, so 2^sh >= Bp / 4 lanes take a column, a wave 64 >> sh
// of them at once, eight such groups in flight.
template <typename Out>
__device__ __forceinline__ void column_prefixes(const int32_t *__restrict__ hist, int Bp, int count, int b, int wave, int waves, Out out)
{
    const int lane = __lane_id();
    const int sh = 32 - __clz(max((Bp >> 2) - 1, 0)), per = 64 >> sh;   // Bp <= 256: sh <= 6
    const int k = 4 * (lane & ((1 << sh) - 1)), sub = lane >> sh;
    constexpr int kFlight = 8;
    for (int c0 = wave * per; c0 < count; c0 += waves * per * kFlight) {
        int4 v[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int c = c0 + u * waves * per + sub;
            v[u] = int4{0, 0, 0, 0};
            if (c < count && k < b) v[u] = *reinterpret_cast<const int4 *>(hist + (size_t)c * Bp + k);   // k + 3 < Bp
        }
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            if (c0 + u * waves * per >= count) break;   // uniform
            int s = v[u].x + (k + 1 < b ? v[u].y : 0) + (k + 2 < b ? v[u].z : 0) + (k + 3 < b ? v[u].w : 0);
            // window sums over 2^sh lanes ending at each lane; the last lane of a column has its total
            if (sh > 0) s += dpp<0x111>(s);   // row_shr 1, 2, 4, 8: rows of 16 lanes
            if (sh > 1) s += dpp<0x112>(s);
            if (sh > 2) s += dpp<0x114>(s);
            if (sh > 3) s += dpp<0x118>(s);
            if (sh > 4) s += dpp<0x142>(s);   // row_bcast 15, 31: the last lane of the row(s) before
            if (sh > 5) s += dpp<0x143>(s);
            const int c = c0 + u * waves * per + sub;
            if (k == 4 * ((1 << sh) - 1) && c < count) out(c, s);
        }
    }
}

struct FinishArgs {
    RouteIo io;
    Workspace ws;
    const int32_t *expert_off_hist;   // histograms the slots follow: block_expert_hist, or those of the first hop
    int T, RB, B, Bp, n, m, C, ppr;
    RouteTail tail;
    float alpha, beta;
};

// Two workgroups for the totals (dispatched first, they take longest): workgroup 0 writes the counts by
// group and local index, the probability sums and the loss, workgroup 1 the expert counts.  Then one per routing block, tokens of a
// block <= its threads.  LPR > 0: the rows of the block's tokens are
// moved to the expert buffers by LPR lanes each.  Dynamic LDS: [N + n] offsets, [RB] destinations, or [n + m] counts, [n + m] sums.
// Latency-bound except for the row moves: one round of loads for the offsets, one for the tokens, the stores.
template <int LPR>
__global__ __launch_bounds__(1024) void route_finish_kernel(FinishArgs a)
{
    extern __shared__ int32_t lds_i[];
    const int n = a.n, m = a.m, N = n * m, cols = n + m, b = (int)blockIdx.x - 2, Bp = a.Bp;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
    if (b == -2) {
        int32_t *cnt = lds_i;
        float *sum = reinterpret_cast<float *>(cnt + cols);
        column_prefixes(a.ws.block_group_hist, Bp, cols, a.B, wave, waves, [&](int c, int s) {
            cnt[c] = s;
            (c < n ? a.io.group_count : a.io.local_count - n)[c] = s;
        });
        for (int c0 = wave; c0 < cols; c0 += waves * 4) {   // four columns in flight
            float s[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * waves;
                s[u] = 0.f;
                if (c < cols)
                    for (int k = lane; k < a.B; k += 64) s[u] += c < n ? a.ws.block_p_sum[(size_t)c * Bp + k] : a.ws.block_q_sum[(size_t)(c - n) * Bp + k];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * waves;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) s[u] += __shfl_xor(s[u], off, 64);
                if (lane == 0 && c < cols) {
                    sum[c] = s[u];
                    (c < n ? a.io.p_sum : a.io.q_sum - n)[c] = s[u];
                }
            }
        }
        __syncthreads();
        if (a.tail.loss3 && wave == 0) aux_loss_wave(cnt, cnt + n, sum, sum + n, a.T, n, m, a.alpha, a.beta, a.tail.loss3);
        return;
    }
    if (b == -1) {
        const int32_t *own = a.ws.block_expert_hist;
        const bool hop = a.expert_off_hist != own;   // with a first-hop limit the counts before drops come from other histograms
        column_prefixes(a.expert_off_hist, Bp, N, a.B, wave, waves, [&](int e, int s) {
            a.io.kept_count[e] = min(s, a.C);
            if (!hop) a.io.expert_count[e] = s;
        });
        if (hop) column_prefixes(own, Bp, N, a.B, wave, waves, [&](int e, int s) { a.io.expert_count[e] = s; });
        return;
    }

    int32_t *dest = lds_i + N + n;
    const int t0 = b * a.RB, live = min(a.RB, a.T - t0);
    int g = 0, e = 0, rank = 0, pos = 0;
    if (tid < live) {   // requested before the offsets
        const int t = t0 + tid;
        g = a.io.group_idx[t], e = g * m + a.io.local_idx[t];
        rank = a.ws.rank_in_block[t], pos = a.ws.pos_in_block[t];
    }
    column_prefixes(a.expert_off_hist, Bp, N, b, wave, waves, [&](int c, int s) { lds_i[c] = s; });
    column_prefixes(a.ws.block_group_hist, Bp, n, b, wave, waves, [&](int c, int s) { lds_i[N + c] = s; });
    __syncthreads();
    if (tid < live) {
        const int t = t0 + tid;
        rank += lds_i[e];
        const int sl = rank < a.C ? rank : -1;
        a.io.slot[t] = sl;
        a.io.pos_in_group[t] = lds_i[N + g] + pos;
        if (sl >= 0 && a.tail.slot_token) a.tail.slot_token[(size_t)e * a.C + sl] = t;
        dest[tid] = sl < 0 ? -1 : e * a.C + sl;   // N*C < 2^31
    }
    __syncthreads();
    if constexpr (LPR > 0) {
        const int rows = blockDim.x / LPR, sub = tid % LPR;
        for (int tk = tid / LPR; tk < live; tk += rows) {
            const int to = dest[tk];
            const size_t t = t0 + tk;
            if (to < 0) zero_row(static_cast<u32x4 *>(a.tail.y) + t * a.ppr, a.ppr, sub, LPR);
            else
                move_row<LPR>(static_cast<const u32x4 *>(a.tail.x) + t * a.ppr, static_cast<u32x4 *>(a.tail.xe) + (size_t)to * a.ppr, a.ppr, sub,
                              [](u32x4 v) { return v; });
        }
    } else if (a.tail.y) {
        zero_dropped_rows(dest, live, t0, static_cast<u32x4 *>(a.tail.y), a.ppr, wave, waves);
    }
}

// Exclusive scan along the block axis of one histogram column by one wave, 1024 blocks per step with all their loads in
// flight; returns the column total.  hist[col*Bp + b] is rewritten in place.
__device__ __forceinline__ int wave_scan_column(int32_t *__restrict__ hist, int B, int Bp, int col)
{
    constexpr int kFlight = 16;
    const int lane = __lane_id();
    int32_t *h = hist + (size_t)col * Bp;
    int carry = 0;
    for (int b0 = 0; b0 < B; b0 += 64 * kFlight) {
        int v[kFlight];
#pragma unroll
        for (int k = 0; k < kFlight; ++k) v[k] = b0 + k * 64 + lane < B ? h[b0 + k * 64 + lane] : 0;
#pragma unroll
        for (int k = 0; k < kFlight; ++k) {
            if (b0 + k * 64 >= B) break;   // uniform
            int incl = v[k];               // inclusive prefix over the wave: rows of 16 lanes, then across rows
            incl += dpp<0x111>(incl);
            incl += dpp<0x112>(incl);
            incl += dpp<0x114>(incl);
            incl += dpp<0x118>(incl);
            incl += __builtin_amdgcn_update_dpp(0, incl, 0x142, 0xA, 0xF, false);   // lane 15 of rows 0, 2 to rows 1, 3
            incl += __builtin_amdgcn_update_dpp(0, incl, 0x143, 0xC, 0xF, false);   // lane 31 to rows 2, 3
            if (b0 + k * 64 + lane < B) h[b0 + k * 64 + lane] = carry + incl - v[k];
            carry += __builtin_amdgcn_readlane(incl, 63);
        }
    }
    return carry;
}

// One wave per column of the work list
//   [N expert columns | n group columns | n p-sum columns | m q-sum columns | m local-count columns],
// 4 waves per workgroup; the columns are independent, so the grid spreads them over the chip.
constexpr int kScanWaves = 4;

__global__ __launch_bounds__(64 * kScanWaves) void route_scan_kernel(RouteIo io, Workspace ws, int B, int Bp, int n, int m, int C)
{
    const int N = n * m;
    const int lane = threadIdx.x & 63;
    const int w = blockIdx.x * kScanWaves + (threadIdx.x >> 6);
    if (w < N) {
        const int total = wave_scan_column(ws.block_expert_hist, B, Bp, w);
        if (lane == 0) {
            io.expert_count[w] = total;
            io.kept_count[w] = min(total, C);
        }
    } else if (w < N + n) {
        const int total = wave_scan_column(ws.block_group_hist, B, Bp, w - N);
        if (lane == 0) io.group_count[w - N] = total;
    } else if (w < N + 2 * n) {
        const float s = wave_sum_column(ws.block_p_sum, B, Bp, w - N - n);
        if (lane == 0) io.p_sum[w - N - n] = s;
    } else if (w < N + 2 * n + m) {
        const float s = wave_sum_column(ws.block_q_sum, B, Bp, w - N - 2 * n);
        if (lane == 0) io.q_sum[w - N - 2 * n] = s;
    } else if (w < N + 2 * n + 2 * m) {
        const int j = w - N - 2 * n - m;   // local_count[j] = tokens whose local index is j, over all groups
        int s = 0;
        for (int b = lane; b < B; b += 64) s += ws.block_group_hist[(size_t)(n + j) * Bp + b];
        s = wave_sum(s);
        if (lane == 0) io.local_count[j] = s;
    }
}

// Group capacity: tokens whose stage-1 position (block offset of the group + in-block
// position) reaches Cg are dropped at the first hop.  The in-block expert ranks are rebuilt over the remaining tokens,
// overwriting those of the decision, and so are the block histograms of the experts (into hist_out).
// SCANNED: the group histograms hold block offsets already; otherwise they are summed here (at most 256 blocks).
template <bool SCANNED>
__global__ __launch_bounds__(kRouteBlock) void route_first_hop_kernel(RouteIo io, Workspace ws, int T, int RB, int Bp, int n, int m, int Cg,
                                                                      int bits_N, int32_t *__restrict__ hist_out)
{
    extern __shared__ int32_t hist[];   // [N], then [n] group offsets
    const int N = n * m;
    const int tid = threadIdx.x;
    const int b = blockIdx.x;
    const int t = b * RB + tid;
    const bool valid = tid < RB && t < T;
    const int lane = __lane_id();
    const int wave = tid >> 6;
    for (int i = tid; i < N; i += kRouteBlock) hist[i] = 0;
    if constexpr (SCANNED) {
        for (int i = tid; i < n; i += kRouteBlock) hist[N + i] = ws.block_group_hist[(size_t)i * Bp + b];
    } else {
        column_prefixes(ws.block_group_hist, Bp, n, b, wave, kRouteBlock / 64, [&](int c, int s) { hist[N + c] = s; });
    }
    __syncthreads();
    int e = 0;
    bool through = false;
    if (valid) {
        const int g = io.group_idx[t];
        e = g * m + io.local_idx[t];
        through = hist[N + g] + ws.pos_in_block[t] < Cg;
    }
    const unsigned long long me = match_any(e, bits_N, through);
    const unsigned long long lt = lanemask_lt();
    for (int w = 0; w < kRouteBlock / 64; ++w) {
        if (wave == w && through) {
            const int base = hist[e];
            ws.rank_in_block[t] = base + __popcll(me & lt);
            if (63 - __clzll(me) == lane) hist[e] = base + __popcll(me);
        }
        __syncthreads();
    }
    if (valid && !through) ws.rank_in_block[t] = kHop1Dropped;
    for (int i = tid; i < N; i += kRouteBlock) hist_out[(size_t)i * Bp + b] = hist[i];
}

// Group capacity, many blocks: block offsets of the rebuilt expert histograms; kept_count = tokens that
// reached the expert, cut at C.
__global__ __launch_bounds__(64 * kScanWaves) void route_scan_experts_kernel(
    int B, int Bp, int N, int C, int32_t *__restrict__ block_expert_hist, int32_t *__restrict__ kept_count)
{
    const int w = blockIdx.x * kScanWaves + (threadIdx.x >> 6);
    if (w >= N) return;
    const int total = wave_scan_column(block_expert_hist, B, Bp, w);
    if ((threadIdx.x & 63) == 0) kept_count[w] = min(total, C);
}

// Final slots from scanned histograms (many blocks), one thread per token; see RouteTail for what else is written.
// (The row move of the chained forward pass is a kernel of its own: dispatch_finalize.)
__global__ __launch_bounds__(256) void route_slots_kernel(FinishArgs a)
{
    const int n = a.n, m = a.m;
    if (a.tail.loss3 && blockIdx.x == gridDim.x - 1 && threadIdx.x < 64)
        aux_loss_wave(a.io.group_count, a.io.local_count, a.io.p_sum, a.io.q_sum, a.T, n, m, a.alpha, a.beta, a.tail.loss3);
    const int t = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63, t0 = t - lane;
    bool dropped = false;
    if (t < a.T) {
        const int b = t / a.RB, g = a.io.group_idx[t], e = g * m + a.io.local_idx[t];
        const int rank = a.ws.block_expert_hist[(size_t)e * a.Bp + b] + a.ws.rank_in_block[t];
        const int sl = rank < a.C ? rank : -1;
        a.io.slot[t] = sl;
        a.io.pos_in_group[t] = a.ws.block_group_hist[(size_t)g * a.Bp + b] + a.ws.pos_in_block[t];
        if (sl >= 0 && a.tail.slot_token) a.tail.slot_token[(size_t)e * a.C + sl] = t;
        dropped = sl < 0;
    }
    if (!a.tail.y) return;
    unsigned long long mask = __ballot(dropped);
    while (mask) {   // output rows of dropped tokens, a wave at a time (Eq. 3 gives them no expert output)
        const int src = __ffsll((long long)mask) - 1;
        zero_row(static_cast<u32x4 *>(a.tail.y) + (size_t)(t0 + src) * a.ppr, a.ppr, lane, 64);
        mask &= mask - 1;
    }
}

int ceil_log2(int v)
{
    int b = 0;
    while ((1 << b) < v) ++b;
    return b;
}

size_t route_lds_bytes(int rb, int n, int m)
{
    const size_t cols = n + m, NC = (size_t)n * m + n;
    return 4 * (rb * (cols | 1) + 8 * cols + rb + (rb + 63) / 64 * NC + 2 * cols);
}

template <int NT, int P, bool GATE, int DT, int CT>
hipError_t launch_block(const RouteArgs &a, int blocks, size_t lds, hipStream_t s)
{
    SMILE_LAUNCH((gate_logits_route_kernel<DT, CT, NT, P, GATE>), dim3(blocks), dim3(NT), lds, s, a);
    return hipGetLastError();
}

// Column tiles per pass: all of them while the accumulators (RT x CT tiles of 4 registers) fit beside the operands.  Three over the
// four row tiles of 64 tokens do not (24 bytes spilled); route_plan leaves those logits to the gate kernel.
template <int NT, int P, int DT>
hipError_t launch_gate_ct(const RouteArgs &a, int blocks, size_t lds, hipStream_t s)
{
    const int ct = (a.n + a.m + 15) / 16;
    if (ct <= 1) return launch_block<NT, P, true, DT, 1>(a, blocks, lds, s);
    if (ct <= 2) return launch_block<NT, P, true, DT, 2>(a, blocks, lds, s);
    if constexpr (NT / P < 64)
        if (ct <= 3) return launch_block<NT, P, true, DT, 3>(a, blocks, lds, s);
    // Blocks of 64 tokens and 49 to 144 columns of a 16-bit type (gate_wide), against the contraction split over the waves with five column tiles
    // a pass (this kernel, us): 8300 x 768 with 49 / 80 / 129 columns 24.5 / 29.8 / 46.2 -> 17.6 / 20.7 / 23.3, 12288 x 1024 with 49 / 144
    // 27.3 / 55.9 -> 19.8 / 30.9, 32768 x 768 with 65 / 129 37.0 / 60.2 -> 24.7 / 31.9, 65536 x 1024 with 129 121.5 -> 72.4.  A batch of one
    // block keeps the split, which has more of its only block's loads in flight.
    if constexpr (NT == 256 && NT / P == 64 && DT != SMILE_DTYPE_F32)
        if (ct > 3 && ct <= kWideTiles && !a.one) return launch_block<NT, P, true, DT, kWideTiles>(a, blocks, std::max(lds, (size_t)kWideLds), s);
    return launch_block<NT, P, true, DT, 5>(a, blocks, lds, s);
}

template <int NT, int P>
hipError_t launch_decide(int dtype, bool gate, const RouteArgs &a, int blocks, size_t lds, hipStream_t s)
{
    if (!gate) return launch_block<NT, P, false, SMILE_DTYPE_F32, 1>(a, blocks, lds, s);
    if constexpr (NT / P > 64) return hipErrorInvalidValue;   // route_plan: larger blocks read logits
    else if (dtype == SMILE_DTYPE_BF16) return launch_gate_ct<NT, P, SMILE_DTYPE_BF16>(a, blocks, lds, s);
    else if (dtype == SMILE_DTYPE_F16) return launch_gate_ct<NT, P, SMILE_DTYPE_F16>(a, blocks, lds, s);
    else return launch_gate_ct<NT, P, SMILE_DTYPE_F32>(a, blocks, lds, s);
}

}  // namespace

// How a layer's tokens are routed; a function of the layer description only, so that every entry point sums
// in the same order.
RoutePlan route_plan(const smile_layer_desc &d)
{
    const int n = d.n_groups, m = d.m_local, N = n * m;
    constexpr size_t kLdsMost = 64 * 1024;
    RoutePlan p{};
    // One workgroup does it all while reading the batch through one CU (28 GB/s) is faster than a second launch (4 us)
    if (d.T <= 64 && (size_t)d.T * d.d_model * elem_size(d.dtype) <= 64 * 1024) {
        const int rb = d.T <= 16 ? 16 : d.T <= 32 ? 32 : 64;
        if (route_lds_bytes(rb, n, m) <= kLdsMost) {
            p.rb = rb, p.tile = p.one = p.gate = true;
            p.blocks = p.stride = 1;
            return p;
        }
    }
    // Blocks as small as leaves at most 256 of them (more CUs read x, and 256 blocks are one load in route_finish), from 64
    // tokens on as many blocks as there are: several share a CU then, and one block's latency hides under another's reads.
    // 256 tokens where the histograms would grow past 2 MB otherwise.
    auto blocks_of = [&](int tokens) { return ((size_t)d.T + tokens - 1) / tokens; };   // T may be 2^31 - 1
    int rb = d.T <= 16 * 256 ? 16 : d.T <= 32 * 256 ? 32 : 64;
    if (d.T > 65536 || blocks_of(rb) * (N + 2 * n + 2 * m) > 512 * 1024) rb = 256;
    // The 1024 threads of a 256-token block are alone on their CU anyway and may have nearly all of its LDS: routers of about 60 to 140
    // columns (bf16, 131072 x 768, decision of 64 / 68 / 129 columns 32 / 33 / 66 us; the kernel that re-reads its rows 62 / 71 / 117).
    p.tile = route_lds_bytes(rb, n, m) <= (rb == kRouteBlock ? 152 * 1024 : kLdsMost);
    if (!p.tile) rb = kRouteBlock;
    p.rb = rb;
    p.blocks = (int)blocks_of(rb);
    // every workgroup of route_finish reads the histograms of the blocks before it: worth a launch up to 128 KB
    const int padded = (p.blocks + 3) / 4 * 4;
    // Logits in the routing launch: with blocks of up to 64 tokens.  256 tokens are one workgroup per CU, whose waves all wait for the same
    // barriers (bf16, routing us, in one launch against two: 70000 x 768 with 10 / 24 / 40 columns 63 / 78 / 95 against 46 / 56 / 67, 131072 x 768
    // 84 / 95 / 107 against 77 / 87 / 92).  33 to 48 columns over 64 tokens spill (launch_gate_ct): 40 columns, 65536 x 1024 67 against 64,
    // 12000 x 768 31.4 against 30.1.  The kernel's row offsets inside a block are 32-bit.
    const int cols = n + m;
    p.gate = p.tile && rb <= 64 && (rb < 64 || cols <= 32 || cols > 48) && (int64_t)rb * d.d_model <= (int64_t)1 << 32;
    p.scan_inline = p.blocks <= 256 && (size_t)(N + n) * padded * 4 <= 128 * 1024;
    p.stride = p.scan_inline ? padded : p.blocks;
    return p;
}

hipError_t launch_routing(const smile_layer_desc &d, const Workspace &ws, const GateInputs *gate, const RouteIo &io, const RouteTail &tail,
                          hipStream_t s)
{
    const int n = d.n_groups, m = d.m_local, N = n * m;
    const RoutePlan p = route_plan(d);
    const int ppr = d.d_model * elem_size(d.dtype) / 16;
    hipError_t err;
    RouteArgs a{};
    if (gate) a.x = gate->x, a.w_inter = gate->w_inter, a.w_intra = gate->w_intra;
    a.d = d.d_model, a.io = io, a.T = d.T, a.n = n, a.m = m, a.bits_n = ceil_log2(n), a.bits_N = ceil_log2(N), a.Bp = p.stride, a.ws = ws;
    a.one = p.one, a.C = d.capacity, a.Cg = d.group_capacity, a.ppr = ppr, a.tail = tail, a.alpha = d.alpha, a.beta = d.beta;
    if (gate && !p.gate) {
        err = launch_gate_logits(d, gate->x, gate->w_inter, gate->w_intra, io.logits_inter, io.logits_intra, s);
        if (err != hipSuccess) return err;
        gate = nullptr;
    }
    if (p.tile) {
        const size_t lds = route_lds_bytes(p.rb, n, m);
        if (p.rb == 16) err = launch_decide<256, 16>(d.dtype, gate != nullptr, a, p.blocks, lds, s);
        else if (p.rb == 32) err = launch_decide<256, 8>(d.dtype, gate != nullptr, a, p.blocks, lds, s);
        else if (p.rb == 64) err = launch_decide<256, 4>(d.dtype, gate != nullptr, a, p.blocks, lds, s);
        else err = launch_decide<1024, 4>(d.dtype, gate != nullptr, a, p.blocks, lds, s);
    } else {
        // one histogram copy per wave while four of them fit beside the kernel's static LDS in 64 KB: N + n <= 1920
        constexpr size_t kStaticLds = sizeof(float) * (kRouteBlock * (kColChunk + 1) + 8 * kColChunk);
        const bool per_wave = (size_t)(N + n) * (kRouteBlock / 64) * sizeof(int32_t) + kStaticLds <= 64 * 1024;
        const size_t lds = sizeof(int32_t) * (size_t)(N + n) * (per_wave ? kRouteBlock / 64 : 1);
        if (per_wave) SMILE_LAUNCH(route_decide_kernel<true>, dim3(p.blocks), dim3(kRouteBlock), lds, s, a);
        else SMILE_LAUNCH(route_decide_kernel<false>, dim3(p.blocks), dim3(kRouteBlock), lds, s, a);
        err = hipGetLastError();
    }
    if (err != hipSuccess) return err;
    if (p.one) {   // everything but the row move is done
        if (tail.xe) err = launch_dispatch(d, tail.x, io.group_idx, io.local_idx, io.slot, tail.xe, s);
        return err;
    }
    FinishArgs f{io, ws, ws.block_expert_hist, d.T, p.rb, p.blocks, p.stride, n, m, d.capacity, ppr, tail, d.alpha, d.beta};
    const size_t hop_lds = sizeof(int32_t) * (size_t)(N + n);
    if (p.scan_inline) {
        if (d.group_capacity > 0) {
            SMILE_LAUNCH(route_first_hop_kernel<false>, dim3(p.blocks), dim3(kRouteBlock), hop_lds, s, io, ws, d.T, p.rb, p.stride, n, m,
                         d.group_capacity, a.bits_N, ws.block_expert_hist2);
            err = hipGetLastError();
            if (err != hipSuccess) return err;
            f.expert_off_hist = ws.block_expert_hist2;
        }
        const size_t lds = sizeof(int32_t) * (size_t)std::max(N + n + p.rb, 2 * (n + m));
        const dim3 grid(p.blocks + 2);
        if (tail.xe) {
            const int lpr = lanes_per_row(ppr), threads = std::min(std::max(p.rb * 16, 256), 1024);   // half the block's rows at once
            if (lpr == 8) SMILE_LAUNCH(route_finish_kernel<8>, grid, dim3(threads), lds, s, f);
            else if (lpr == 16) SMILE_LAUNCH(route_finish_kernel<16>, grid, dim3(threads), lds, s, f);
            else SMILE_LAUNCH(route_finish_kernel<32>, grid, dim3(threads), lds, s, f);
        } else {
            // enough waves to have the loads of all columns in flight at once
            SMILE_LAUNCH(route_finish_kernel<0>, grid, dim3(N > 32 || p.rb > 64 ? 1024 : 256), lds, s, f);
        }
        return hipGetLastError();
    }
    const int columns = N + 2 * n + 2 * m;
    SMILE_LAUNCH(route_scan_kernel, dim3((columns + kScanWaves - 1) / kScanWaves), dim3(64 * kScanWaves), 0, s, io, ws, p.blocks, p.stride, n,
                 m, d.capacity);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    if (d.group_capacity > 0) {
        SMILE_LAUNCH(route_first_hop_kernel<true>, dim3(p.blocks), dim3(kRouteBlock), hop_lds, s, io, ws, d.T, p.rb, p.stride, n, m,
                     d.group_capacity, a.bits_N, ws.block_expert_hist);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
        SMILE_LAUNCH(route_scan_experts_kernel, dim3((N + kScanWaves - 1) / kScanWaves), dim3(64 * kScanWaves), 0, s, p.blocks, p.stride, N,
                     d.capacity, ws.block_expert_hist, io.kept_count);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    if (tail.xe) return launch_dispatch_finalize(d, ws, p, io, tail, s);
    SMILE_LAUNCH(route_slots_kernel, dim3(((size_t)d.T + 255) / 256), dim3(256), 0, s, f);
    return hipGetLastError();
}

}  // namespace smile
