// Router logits r(x) = W_r x (Section 2, text before Eq. 1) for the inter router W_p[n,d] and the
// intra router W_q[m,d] (Section 3.2.1: two tied routers reading the same token), computed as one
// skinny product [T,d] x [d,n+m].  n+m is 10-40 in the paper-shaped workloads (up to 257 for the flat
// one-level router the paper compares against), so the kernel is
// bound by the single read of x from HBM; the weights (<= 80 KB) stay in L2.
//
// One workgroup of 4 waves owns RT x 16 token rows and takes the contraction in turns; the 4 partial accumulators are summed
// through LDS in a fixed order.  Every workgroup re-reads the router weights from L2, so RT grows with T (weight
// traffic / RT) while keeping >= 512 workgroups: RT = 1 for the smallest paper-shaped batch (T = 8192), 4 from
// T = 32768.
//
// One chunk and one column tile's weights at a time: what keeps HBM busy here is the number of waves, so registers count.
// Against the loop of the routing kernel (gate_device.hpp: two chunks in flight, all weights of a chunk requested at once), bf16, us:
// 131072 x 768, 10 / 24 / 40 / 72 columns: 41 / 47 / 51 / 83 against 48 / 53 / 59 / 96; 65536 x 1024: 23 / 26 / 32 / 55
// against 24 / 30 / 36 / 61; 32768 x 768: 10.5 / 13.0 / 15.4 / 23.4 against 12.2 / 14.0 / 16.7 / 24.0; equal below 16384 rows.  Only with eight
// column tiles over several row tiles (16-bit) are the weights of a chunk worth requesting at once: 65536 x 1024 with 129 columns 107
// against 119.  Products and order are the same in both: the same bits.
#include <algorithm>

#include "gate_device.hpp"

namespace smile {

namespace {

typedef mfma_f32x4 f32x4;

// CT = number of 16-column tiles covering the logit columns of this pass; RT = 16-row tiles per workgroup.
template <int DT, int CT, int RT>
__global__ __launch_bounds__(64 * kGateWaves) void gate_logits_kernel(
    const void *__restrict__ x, const void *__restrict__ w_inter, const void *__restrict__ w_intra,
    float *__restrict__ logits_inter, float *__restrict__ logits_intra, int T, int d, int n, int m, int col0)
{
    __shared__ f32x4 red[kGateWaves - 1][RT][CT][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, kg = lane >> 4;
    const int row0 = blockIdx.x * 16 * RT;

    typedef typename GateType<DT>::elem E;
    typedef typename GateType<DT>::vec vec;
    constexpr int kChunk = GateType<DT>::kChunk, kLane = kChunk / 4, kVec = kChunk / 8;   // elements per lane, per 16 bytes
    constexpr bool kAtOnce = CT == 8 && RT > 1 && DT != SMILE_DTYPE_F32;
    const E *xrow[RT], *wrow[CT];   // wrow: the weight row of this lane in column tile ct, null beyond n + m
    f32x4 acc[RT][CT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) xrow[rt] = static_cast<const E *>(x) + (size_t)min(row0 + rt * 16 + r, T - 1) * d;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const int c = col0 + ct * 16 + r;
        wrow[ct] = c < n ? static_cast<const E *>(w_inter) + (size_t)c * d
                         : (c < n + m ? static_cast<const E *>(w_intra) + (size_t)(c - n) * d : nullptr);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int chunks = (d + kChunk - 1) / kChunk;
    for (int chunk = wave; chunk < chunks; chunk += kGateWaves) {
        const int k = chunk * kChunk + kg * kLane;
        const bool in = DT != SMILE_DTYPE_F32 || k < d;   // 16-bit rows are whole chunks; a float row may end inside one
        vec a[RT][2];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int h = 0; h < 2; ++h) a[rt][h] = in ? *reinterpret_cast<const vec *>(xrow[rt] + k + h * kVec) : vec{};
        vec b[kAtOnce ? CT : 1][2];
        auto weights = [&](int ct) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                b[kAtOnce ? ct : 0][h] = in && wrow[ct] ? *reinterpret_cast<const vec *>(wrow[ct] + k + h * kVec) : vec{};
        };
        if constexpr (kAtOnce) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) weights(ct);
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            if constexpr (!kAtOnce) weights(ct);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int h = 0; h < 2; ++h) acc[rt][ct] = GateType<DT>::mfma(a[rt][h], b[kAtOnce ? ct : 0][h], acc[rt][ct]);
        }
    }
    if (wave > 0) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) red[wave - 1][rt][ct][lane] = acc[rt][ct];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                f32x4 s = acc[rt][ct];
#pragma unroll
                for (int w = 0; w < kGateWaves - 1; ++w) s += red[w][rt][ct][lane];
                const int c = col0 + ct * 16 + r;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = row0 + rt * 16 + kg * 4 + i;
                    if (row < T) {
                        if (c < n) logits_inter[(size_t)row * n + c] = s[i];
                        else if (c < n + m) logits_intra[(size_t)row * m + (c - n)] = s[i];
                    }
                }
            }
    }
}

template <int CT, int RT>
void launch_rt(const smile_layer_desc &d, const void *x, const void *w_inter, const void *w_intra, float *logits_inter,
               float *logits_intra, int col0, hipStream_t s)
{
    const dim3 grid((d.T + 16 * RT - 1) / (16 * RT)), block(64 * kGateWaves);
#define SMILE_GATE(DT) \
    SMILE_LAUNCH((gate_logits_kernel<DT, CT, RT>), grid, block, 0, s, x, w_inter, w_intra, logits_inter, logits_intra, d.T, \
                 d.d_model, d.n_groups, d.m_local, col0)
    if (d.dtype == SMILE_DTYPE_BF16) SMILE_GATE(SMILE_DTYPE_BF16);
    else if (d.dtype == SMILE_DTYPE_F16) SMILE_GATE(SMILE_DTYPE_F16);
    else SMILE_GATE(SMILE_DTYPE_F32);
#undef SMILE_GATE
}

// columns [col0, col0 + 16*CT)
template <int CT>
void launch_ct(const smile_layer_desc &d, const void *x, const void *w_inter, const void *w_intra,
               float *logits_inter, float *logits_intra, int col0, hipStream_t s)
{
    // the accumulators of RT x CT tiles must stay in registers: RT * CT <= 16
    if (d.T >= 32768 && CT <= 4) launch_rt<CT, 4>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s);
    else if (d.T >= 16384) launch_rt<CT, 2>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s);
    else launch_rt<CT, 1>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s);
}

}  // namespace

hipError_t launch_gate_logits(const smile_layer_desc &d, const void *x, const void *w_inter, const void *w_intra,
                              float *logits_inter, float *logits_intra, hipStream_t s)
{
    // up to 128 columns per pass over x (8 accumulator tiles); wider routers (a flat one-level
    // router over all N experts) take several passes
    const int cols = d.n_groups + d.m_local;
    for (int col0 = 0; col0 < cols; col0 += 128) {
        switch ((std::min(cols - col0, 128) + 15) / 16) {
        case 1: launch_ct<1>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s); break;
        case 2: launch_ct<2>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s); break;
        case 3: launch_ct<3>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s); break;
        case 4: launch_ct<4>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s); break;
        case 5: launch_ct<5>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s); break;
        case 6: launch_ct<6>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s); break;
        case 7: launch_ct<7>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s); break;
        default: launch_ct<8>(d, x, w_inter, w_intra, logits_inter, logits_intra, col0, s); break;
        }
    }
    return hipGetLastError();
}

}  // namespace smile
