// Expert FFN E_e of Eq. 3 (Section 4.1: hidden -> intermediate -> hidden with GELU) for all N
// experts at once, as two grouped "NT" GEMMs with device-resident, ragged row counts:
//
//   h [e] = act(xe[e] . w1[e]^T + b1[e])      rows r < kept[e],  xe[e]: [C,d],  w1[e]: [F,d]
//   ye[e] =      h[e] . w2[e]^T + b2[e]                          h[e]:  [C,F],  w2[e]: [d,F]
//
// Both operands of either product are K-contiguous, which is exactly the MFMA register layout
// (8 consecutive k per lane), so tiles go global -> LDS -> registers as 16-byte pieces with no
// transposition anywhere.
//
// Large buffers of the 16-bit types run on the ring kernels (gemm_ring.hpp), which keep more loads in flight.  The two-stage
// kernel below takes small buffers and narrow layers (64-row tiles, pick_tile) and what a ring does not take: contractions of fewer
// than three slabs and operands whose offsets need more than 32 bits.
//
// Two-stage kernel (bf16 or fp16 storage).  One workgroup computes a BM x BN tile
// of one expert with v_mfma_f32_32x32x16_bf16 / _f16 and fp32 accumulators.
//   * K is cut into slabs of BK = 64 elements.  A slab travels global -> LDS directly
//     (global_load_lds_dwordx4: no staging registers, no ds_write) into a ring of STAGES buffers
//     with STAGES-1 slabs in flight.  Per slab: wait until this wave's part has landed (s_waitcnt
//     vmcnt), one s_barrier (every wave's part landed, and every wave is done reading the buffer
//     about to be refilled), issue the loads of the slab STAGES-1 ahead beside the MFMAs.  The wait for the next slab comes
//     before the LAST k-step of a slab, so that no LDS read at a slab's start is waited for with the matrix cores idle.
//   * A direct load writes 64 lanes x 16 bytes to consecutive LDS addresses, i.e. whole rows of a
//     slab.  The bank swizzle is therefore applied on the global side: the lane that fills position
//     p of a row fetches piece p ^ f(row), so piece c of a row sits at position c ^ f(row) and the
//     32 rows a wave reads for one MFMA operand fall on distinct banks.
//   * The weight tile is the MFMA "A" operand and the token tile the "B" operand, so a lane ends up
//     with 4 consecutive output columns of one token row.  The epilogue (activation, round
//     to the storage type) writes them to LDS and the workgroup then stores whole rows, 16 bytes per lane, so
//     every global store instruction covers full cache lines.
//   * Traffic L2 -> LDS per flop falls as 1/BM + 1/BN; that path (about 64 B/clk per CU at best)
//     and not HBM is what bounds small tiles, so tiles are as large as the workload can still
//     spread over 256 CUs.
//
// Plain grid (at most a few tiles per workgroup slot of the chip): it covers every (expert, column tile,
// row tile); tiles whose first row is >= kept[e] exit at once, so no host synchronisation on the routing
// result is needed.  Workgroup ids are dealt round-robin to the 8 XCDs by the hardware; the id is remapped
// so that each XCD (own L2) works on a contiguous range of tiles: the row tiles sharing a weight tile and
// the column tiles sharing a token tile then meet in the same L2.
// Persistent grid (many tiles per slot): one workgroup per slot walks the live tiles only, in the same
// order (LiveTileWalk), again without any host knowledge of the row counts.  When experts are far below
// capacity this is up to 25 % faster: a workgroup of an empty tile still has to wait for a free slot (its
// LDS) before it can exit, in turn with the live ones.
//
// fp32 storage: gemm_f32.hip.
#include <algorithm>
#include <type_traits>

#include <hip/hip_ext.h>

#include "gemm_device.hpp"

namespace smile {

namespace {

// OCC: waves per SIMD the register allocation must leave room for (workgroups per CU when the
// workgroup has 4 waves).
// DUAL: the epilogue runs twice, storing act(product) to y and the bare product to y2 (the hidden
// activation and its pre-activation from one GEMM, for the backward pass).
// E: the 16-bit storage type (__bf16 or _Float16).
template <typename E, int BM, int BN, int WGM, int WGN, int STAGES, int OCC, int ACT, bool DUAL = false, bool PERSIST = false>
__global__ __launch_bounds__(WGM *WGN * 64, OCC) void grouped_gemm_nt_kernel(GemmArgs a)
{
    typedef typename Half<E>::vec8 bf16x8;                                  // one MFMA operand: 8 elements
    typedef __attribute__((__vector_size__(4 * sizeof(E)))) E bf16x4;       // 4 rounded outputs
    constexpr int NW = WGM * WGN, NT = NW * 64;
    constexpr int WM = BM / WGM, WN = BN / WGN;   // wave tile
    constexpr int TM = WM / 32, TN = WN / 32;     // MFMA tiles per wave
    constexpr int BK = 64;                        // slab depth
    constexpr int PPR = BK / 8;                   // 16-byte pieces per LDS row
    constexpr int RPI = 64 / PPR;                 // rows filled by one direct-load instruction
    constexpr int ROWS = BM + BN;                 // LDS rows per stage: token tile, then weight tile
    constexpr int GPW = ROWS / RPI / NW;          // load instructions per wave per slab
    constexpr int STAGE = ROWS * PPR;             // 16-byte units per stage
    constexpr int OROWS = WGM * 32;               // output rows staged per epilogue pass
    constexpr int OSTRIDE = BN / 8 + 1;           // staged row length in 16-byte units (+1: bank spread)
    static_assert(BM % (WGM * 32) == 0 && BN % (WGN * 32) == 0, "wave tile must be a multiple of 32");
    static_assert(ROWS % (RPI * NW) == 0 && BM % RPI == 0, "slab must divide into load instructions over the waves");
    static_assert(STAGES >= 2 && STAGES <= 4 && (STAGES - 2) * GPW < 64, "pipeline depth");
    static_assert(OROWS * OSTRIDE <= STAGES * STAGE, "epilogue staging must fit in the pipeline buffers");

    __shared__ u32x4 lds[STAGES * STAGE];

    const int K = a.K, Nout = a.Nout;
    const int slabs = K / BK;

    // ---- which tile(s).
    // Plain kernels: one tile per workgroup; the id is remapped so that each XCD gets a contiguous range
    // (the hardware deals workgroup ids round-robin to the 8 XCDs).
    // PERSIST kernels: one workgroup per slot of the chip walks the live tiles (LiveTileWalk).  The first
    // slabs of the next tile are requested before the epilogue of the current one (PREFETCH), which then
    // stages its output in the one pipeline buffer those loads do not touch.
    constexpr bool PREFETCH = PERSIST && OROWS * OSTRIDE <= STAGE;
    constexpr int STG = PREFETCH ? (STAGES - 1) * STAGE : 0;   // staging area, in 16-byte units
    LiveTileWalk<BM> walk;
    if constexpr (PERSIST) walk.init(a.kept, a.N, a.C, a.col_tiles, false);
    struct Tile {
        int e, rt, ct, rows;
    };
    // the tile of the current ticket (PERSIST) / of this workgroup (plain); false when there is none
    auto select = [&](Tile &t) {
        if constexpr (PERSIST) {
            return walk.tile(t.e, t.rt, t.ct, t.rows);
        } else {
            const int per_xcd = (a.tiles + kXcds - 1) / kXcds;
            const int lid = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
            if (lid >= a.tiles) return false;
            const int per_expert = a.row_tiles * a.col_tiles;
            t.e = lid / per_expert;
            const int rem = lid - t.e * per_expert;
            t.ct = rem / a.row_tiles, t.rt = rem - t.ct * a.row_tiles;
        }
        t.rows = a.kept ? min(a.kept[t.e], a.C) : a.C;   // never trust a count beyond the buffer
        return t.rt * BM < t.rows;
    };

    // ---- loads.  src: this lane's source address in each of the wave's load instructions of a slab.
    const E *src[GPW];
    auto issue = [&](int wave, int slab, int stage) {
#pragma unroll
        for (int i = 0; i < GPW; ++i)
            __builtin_amdgcn_global_load_lds(SMILE_GPTR(src[i] + slab * BK),
                                             SMILE_LPTR(&lds[stage * STAGE + (wave + i * NW) * 64]), 16, 0, 0);
    };
    // Per-lane indices are derived afresh wherever they are needed (PERSIST: through an opaque copy of the
    // thread id), so that nothing computed from them stays in registers from one tile to the next.
    auto thread_id = [&]() {
        int tid = threadIdx.x;
        if constexpr (PERSIST) asm volatile("" : "+v"(tid));
        return tid;
    };
    // source addresses of a tile and the requests for its first STAGES-1 slabs
    auto start_tile = [&](const Tile &t) {
        const int tid = thread_id(), lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int lr = lane / PPR, lp = lane % PPR;
        const E *X = static_cast<const E *>(a.x) + (a.x_rows ? (size_t)0 : (size_t)t.e * a.C * K);
        const E *W = static_cast<const E *>(a.w) + (size_t)t.e * Nout * K;
        const int32_t *x_rows = a.x_rows ? a.x_rows + (size_t)t.e * a.C : nullptr;
#pragma unroll
        for (int i = 0; i < GPW; ++i) {
            const int row = (wave + i * NW) * RPI + lr;            // row of the stage
            const int piece = lp ^ swz(row);
            // rows past the end of the expert's tokens / of the weight matrix re-read the last valid one
            if (row < BM) {
                const int xr = min(t.rt * BM + row, t.rows - 1);
                src[i] = X + (size_t)(x_rows ? x_rows[xr] : xr) * K + piece * 8;
            } else {
                src[i] = W + (size_t)min(t.ct * BN + row - BM, Nout - 1) * K + piece * 8;
            }
        }
#pragma unroll
        for (int s = 0; s < STAGES - 1; ++s)
            if (s < slabs) issue(wave, s, s);
    };

    Tile cur;
    if (!select(cur)) return;
    start_tile(cur);
    for (;;) {
    const int e = cur.e, rt = cur.rt, ct = cur.ct, rows = cur.rows;
    const int tid = thread_id(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WGM, wn = wave / WGM;
    // LDS -> MFMA operands: lane reads row (lane & 31), pieces 2*kk + (lane >> 5)
    const int frow = lane & 31, fhi = lane >> 5, fsw = swz(lane);   // tile bases are multiples of 32
    const int xbase = (wm * WM + frow) * PPR, wbase = (BM + wn * WN + frow) * PPR;

    // The accumulators start at the bias: element v of a lane is column 8*(v/4) + 4*(lane/32) + v%4 of its 32x32 tile, four
    // columns to an 8-byte load (Nout % 8 == 0, so a block of four is inside the row or outside as a whole).  Added in the
    // epilogue element by element it was 96 waits in a row (15 experts x 334 rows, 960 x 3840, f16 with biases: 186 -> 159 us).
    f32x16 acc[TN][TM];
    if (a.bias) {
        const E *bias = static_cast<const E *>(a.bias) + (size_t)e * Nout;
        bf16x4 b[TN][4];
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                b[i][q] = *reinterpret_cast<const bf16x4 *>(bias + min(ct * BN + wn * WN + i * 32 + 8 * q + 4 * fhi, Nout - 4));
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = (float)b[i][v / 4][v % 4];
    } else {
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    }

    const bool wave_live = rt * BM + wm * WM < rows;   // wave-uniform
    constexpr int KS = BK / 16, NM = TM * TN, NF = TM + TN;
    bf16x8 xf[2][TM], wf[2][TN];   // fragments of the k-step being multiplied and of the next one
    auto fetch_one = [&](auto slot, auto kstep, const u32x4 *from) {   // fragment `slot` (token tiles first) of k-step `kstep`
        constexpr int F = decltype(slot)::value, KK = decltype(kstep)::value;
        const int p = (2 * KK + fhi) ^ fsw;
        if constexpr (F < TM) xf[KK & 1][F] = __builtin_bit_cast(bf16x8, from[xbase + F * 32 * PPR + p]);
        else wf[KK & 1][F - TM] = __builtin_bit_cast(bf16x8, from[wbase + (F - TM) * 32 * PPR + p]);
    };
    auto issue_one = [&](int i, int slab, int to) {
        __builtin_amdgcn_global_load_lds(SMILE_GPTR(src[i] + slab * BK), SMILE_LPTR(&lds[to * STAGE + (wave + i * NW) * 64]), 16, 0, 0);
    };
    // Waits for slab `s` (this wave's part landed, then everybody's).  Every wave is then also done reading slab s-1, so
    // slab s-1+STAGES may overwrite it.  `issued_after`: slabs requested after s by now.
    auto enter_slab = [&](int issued_after, bool first) {
        // a prefetched tile's first slabs were requested before the previous tile's stores: wait for all
        if (PREFETCH && first) wait_vmcnt<0>();
        else if (STAGES >= 4 && issued_after == 2) wait_vmcnt<2 * GPW>();
        else if (STAGES >= 3 && issued_after == 1) wait_vmcnt<GPW>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
    };
    // One K slab, its first fragments already in registers.  MORE: slabs kt+1 .. kt+STAGES-1 exist (steady state).  The wait
    // and the barrier for slab kt+1 stand in front of this slab's LAST k-step, whose MFMAs cover the LDS reads of the next
    // slab's first fragments; the load instructions of slab kt+STAGES-1 are spread over the other k-steps.  Inside a k-step
    // the reads come right behind the first MFMAs, so that the last MFMAs cover their latency (the order is pinned).
    auto slab_step = [&](auto more_tag, int kt, int stage) {
        constexpr bool MORE = decltype(more_tag)::value;
        const int nstage = stage == 0 ? STAGES - 1 : stage - 1, next = stage + 1 == STAGES ? 0 : stage + 1;
        for_constants<KS>([&](auto kstep) {
            constexpr int KK = decltype(kstep)::value;
            constexpr bool LAST = KK + 1 == KS;
            constexpr int L0 = LAST ? 0 : GPW * KK / (KS - 1), L1 = LAST ? 0 : GPW * (KK + 1) / (KS - 1);
            __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this k-step's fragments
            if (LAST && (MORE || kt + 1 < slabs)) enter_slab(MORE ? STAGES - 2 : min(STAGES - 2, slabs - 2 - kt), false);
            __builtin_amdgcn_sched_barrier(0);
            const u32x4 *from = lds + (LAST ? next : stage) * STAGE;   // after the last slab: stale, and never multiplied
            for_constants<NM>([&](auto m) {
                constexpr int R = decltype(m)::value;
                acc[R / TM][R % TM] = Half<E>::mfma_32x32x16(wf[KK & 1][R / TM], xf[KK & 1][R % TM], acc[R / TM][R % TM]);
                constexpr int F0 = min_int(NF, 2 * R), F1 = min_int(NF, 2 * R + 2);
                for_constants<F1 - F0>([&](auto f) {
                    fetch_one(std::integral_constant<int, F0 + decltype(f)::value>{}, std::integral_constant<int, (KK + 1) % KS>{}, from);
                });
                constexpr int G0 = L0 + (L1 - L0) * R / NM, G1 = L0 + (L1 - L0) * (R + 1) / NM;
                if constexpr (MORE)
                    for_constants<G1 - G0>([&](auto g) { issue_one(G0 + decltype(g)::value, kt + STAGES - 1, nstage); });
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    // the next tile is chosen before the main loop, so that the loads of its row counts are long back when
    // the epilogue needs them (after it where registers are short: DUAL)
    Tile nxt_tile;
    bool more = false;
    if constexpr (PERSIST && !DUAL) {
        walk.advance();
        more = select(nxt_tile);
    }
    enter_slab(min(STAGES - 2, slabs - 1), true);
    if (wave_live) {
        for_constants<NF>([&](auto f) { fetch_one(f, std::integral_constant<int, 0>{}, lds); });
        int kt = 0, stage = 0;
        for (; kt + STAGES - 1 < slabs; ++kt) {
            slab_step(std::true_type{}, kt, stage);
            stage = stage + 1 == STAGES ? 0 : stage + 1;
        }
        for (; kt < slabs; ++kt) {
            slab_step(std::false_type{}, kt, stage);
            stage = stage + 1 == STAGES ? 0 : stage + 1;
        }
    } else {
        // none of this wave's token rows exists (ragged tile): it only helps loading
        int stage = 0;
        for (int kt = 0; kt < slabs; ++kt) {
            if (kt > 0) enter_slab(min(STAGES - 2, slabs - 1 - kt), false);
            if (kt + STAGES - 1 < slabs) issue(wave, kt + STAGES - 1, stage == 0 ? STAGES - 1 : stage - 1);
            stage = stage + 1 == STAGES ? 0 : stage + 1;
        }
    }
    if constexpr (PERSIST && DUAL) {
        walk.advance();
        more = select(nxt_tile);
    }

    // ---- epilogue.  Accumulator element v of a lane is (column 8*(v/4) + 4*(lane/32) + v%4,
    // row lane%32) of its 32x32 tile.  One pass per 32-row slice of the wave tiles:
    // activation + rounding, 8-byte writes into a [OROWS][BN] staging tile, then row-contiguous
    // 16-byte global stores by the whole workgroup.
    const int32_t *y_rows = a.y_rows ? a.y_rows + (size_t)e * a.C : nullptr;
    u32x2 *stg = reinterpret_cast<u32x2 *>(lds + STG);
    constexpr int OPR = BN / 8;   // 16-byte pieces per output row
#pragma unroll
    for (int pass = 0; pass < (DUAL ? 2 : 1); ++pass) {
        void *dst = pass == 0 ? a.y : a.y2;
        E *Y = dst ? static_cast<E *>(dst) + (size_t)e * a.C * Nout : nullptr;
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave's LDS reads are done
            __builtin_amdgcn_s_barrier();          // main-loop reads / the previous pass's stores are finished
            if (PREFETCH && pass == 0 && j == 0 && more) start_tile(nxt_tile);
#pragma unroll
            for (int i = 0; i < TN; ++i) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int lcol = wn * WN + i * 32 + 8 * q + 4 * fhi;      // column inside the tile
                    bf16x4 out;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float f = acc[i][j][4 * q + v];
                        out[v] = (E)(pass == 0 ? activate<ACT>(f) : f);
                    }
                    stg[((wm * 32 + frow) * OSTRIDE) * 2 + (lcol >> 2)] = __builtin_bit_cast(u32x2, out);
                }
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);
            __builtin_amdgcn_s_barrier();
            // staged piece `id` (already read into v) -> global memory
            auto store_piece = [&](int id, u32x4 v) {
                const int orow = id / OPR, piece = id - orow * OPR;
                const int row = rt * BM + (orow >> 5) * WM + j * 32 + (orow & 31);
                const int col = ct * BN + piece * 8;
                if (id < OROWS * OPR && row < rows && col < Nout) {
                    if (Y) *reinterpret_cast<u32x4 *>(Y + (size_t)row * Nout + col) = v;
                    if (pass == 0 && y_rows) {   // gate-weighted return to token order (Eq. 3), fused
                        const int tok = y_rows[row];
                        *reinterpret_cast<u32x4 *>(static_cast<E *>(a.y_tok) + (size_t)tok * Nout + col) =
                            scale_x8<E>(v, a.gate[tok]);
                    }
                }
            };
            if constexpr (DUAL) {
                // the accumulators are needed again: registers are short, one piece at a time
                for (int id = tid; id < OROWS * OPR; id += NT) {
                    const int orow = id / OPR;
                    store_piece(id, lds[STG + orow * OSTRIDE + id - orow * OPR]);
                }
            } else {
                // all of the thread's staged pieces are read before the first store, so that the LDS latencies overlap
                constexpr int NIT = (OROWS * OPR + NT - 1) / NT;
                u32x4 outv[NIT];
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    const int id = min(tid + it * NT, OROWS * OPR - 1);
                    const int orow = id / OPR;
                    outv[it] = lds[STG + orow * OSTRIDE + id - orow * OPR];
                }
#pragma unroll
                for (int it = 0; it < NIT; ++it) store_piece(tid + it * NT, outv[it]);
            }
        }
    }
    if (!more) return;
    if constexpr (!PREFETCH) {
        // the next tile's first loads overwrite the staging area: every wave must be done reading it
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        start_tile(nxt_tile);
    }
    cur = nxt_tile;
    }   // tile loop
}

// t0/t1 (both or neither): events that receive the begin / end timestamps of the kernel itself.
template <typename Kernel>
void launch_timed(Kernel k, dim3 grid, dim3 block, hipStream_t s, hipEvent_t t0, hipEvent_t t1, const GemmArgs &a)
{
    if (t0 && t1) hipExtLaunchKernelGGL(k, grid, block, 0, s, t0, t1, 0, a);
    else launch_kernel("grouped_gemm_nt_kernel", k, grid, block, 0, s, a);
}

template <typename E, int BM, int BN, int WGM, int WGN, int STAGES, int OCC>
hipError_t launch_half_tile(GemmArgs a, int N, int act, const Tuning &tune, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    a.row_tiles = (a.C + BM - 1) / BM;
    a.col_tiles = (a.Nout + BN - 1) / BN;
    a.tiles = N * a.row_tiles * a.col_tiles;
    a.N = N;
    const int slots = workgroup_slots(tune, workgroups_per_cu(WGM * WGN, OCC, STAGES * (BM + BN) * 64 * 2));
    const dim3 block(WGM * WGN * 64);
    if (use_persistent_grid(tune, N, a.tiles, slots)) {
        const dim3 grid(slots);
        if (act == 0) launch_timed(grouped_gemm_nt_kernel<E, BM, BN, WGM, WGN, STAGES, OCC, 0, false, true>, grid, block, s, t0, t1, a);
        else if (act == 1) launch_timed(grouped_gemm_nt_kernel<E, BM, BN, WGM, WGN, STAGES, OCC, 1, false, true>, grid, block, s, t0, t1, a);
        else launch_timed(grouped_gemm_nt_kernel<E, BM, BN, WGM, WGN, STAGES, OCC, 3, false, true>, grid, block, s, t0, t1, a);
        return hipGetLastError();
    }
    const dim3 grid((a.tiles + kXcds - 1) / kXcds * kXcds);
    if (act == 0) launch_timed(grouped_gemm_nt_kernel<E, BM, BN, WGM, WGN, STAGES, OCC, 0>, grid, block, s, t0, t1, a);
    else if (act == 1) launch_timed(grouped_gemm_nt_kernel<E, BM, BN, WGM, WGN, STAGES, OCC, 1>, grid, block, s, t0, t1, a);
    else launch_timed(grouped_gemm_nt_kernel<E, BM, BN, WGM, WGN, STAGES, OCC, 3>, grid, block, s, t0, t1, a);
    return hipGetLastError();
}

// The dual-output launch (a.y2 given: act(product) and the bare product) of one tile shape, four waves.
template <typename E, int BM, int BN, int STAGES, int OCC>
hipError_t launch_half_dual(GemmArgs a, int N, int act, const Tuning &tune, hipStream_t s)
{
    a.row_tiles = (a.C + BM - 1) / BM;
    a.col_tiles = (a.Nout + BN - 1) / BN;
    a.tiles = N * a.row_tiles * a.col_tiles;
    a.N = N;
    const int slots = workgroup_slots(tune, workgroups_per_cu(4, OCC, STAGES * (BM + BN) * 64 * 2));
    const bool persist = use_persistent_grid(tune, N, a.tiles, slots);
    const dim3 grid(persist ? slots : (a.tiles + kXcds - 1) / kXcds * kXcds), block(256);
    if (act == 1 && persist) SMILE_LAUNCH((grouped_gemm_nt_kernel<E, BM, BN, 2, 2, STAGES, OCC, 1, true, true>), grid, block, 0, s, a);
    else if (act == 1) SMILE_LAUNCH((grouped_gemm_nt_kernel<E, BM, BN, 2, 2, STAGES, OCC, 1, true>), grid, block, 0, s, a);
    else if (persist) SMILE_LAUNCH((grouped_gemm_nt_kernel<E, BM, BN, 2, 2, STAGES, OCC, 3, true, true>), grid, block, 0, s, a);
    else SMILE_LAUNCH((grouped_gemm_nt_kernel<E, BM, BN, 2, 2, STAGES, OCC, 3, true>), grid, block, 0, s, a);
    return hipGetLastError();
}

// `tile` as pick_tile says, with the shapes that exist for two outputs
template <typename E>
hipError_t launch_half_dual_typed(const GemmArgs &a, int N, int act, int tile, const Tuning &tune, hipStream_t s)
{
    if (tile == 9 || tile == 7) return launch_half_dual<E, 64, 64, 3, 3>(a, N, act, tune, s);
    if (tile == 8 || tile == 5) return launch_half_dual<E, 64, 128, 3, 2>(a, N, act, tune, s);
    return launch_half_dual<E, 128, 192, 2, 2>(a, N, act, tune, s);
}

// Tile shapes of grouped_gemm_nt_kernel: id -> (BM, BN, waves along M, waves along N, stages, waves/SIMD budget).  0 is the
// shape for contractions of one or two slabs, which the ring kernels do not take; the 64-row tiles are for few or small buffers: see
// pick_tile.
template <typename E>
hipError_t launch_half_typed(const GemmArgs &a, int N, int act, int tile, const Tuning &tune, hipStream_t s,
                             hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr)
{
    switch (tile) {
    case 0: return launch_half_tile<E, 128, 192, 2, 2, 2, 2>(a, N, act, tune, s, t0, t1);
    case 5: return launch_half_tile<E, 64, 256, 1, 4, 2, 2>(a, N, act, tune, s, t0, t1);
    case 7: return launch_half_tile<E, 64, 64, 2, 2, 4, 2>(a, N, act, tune, s, t0, t1);
    case 8: return launch_half_tile<E, 64, 128, 2, 2, 3, 2>(a, N, act, tune, s, t0, t1);
    case 9: return launch_half_tile<E, 64, 64, 2, 2, 3, 3>(a, N, act, tune, s, t0, t1);
    default: return hipErrorInvalidValue;
    }
}
constexpr int kRingTile0 = 1;   // ids 1 .. 4: the shapes of the ring kernels (RingTile)
constexpr bool is_ring_tile(int tile) { return tile >= kRingTile0 && tile < kRingTile0 + kRingTiles; }

RingArgs ring_args(const GemmArgs &g, int N)
{
    RingArgs a{};
    a.x = g.x, a.w = g.w, a.y = g.y, a.y2 = g.y2, a.bias = g.bias, a.rows_valid = g.kept, a.x_rows = g.x_rows, a.y_rows = g.y_rows;
    a.y_tok = g.y_tok, a.gate = g.gate, a.N = N, a.Mrows = g.C, a.Nout = g.Nout, a.K = g.K, a.ldx = g.K, a.ldw = g.K;
    a.sx = (long long)g.C * g.K, a.sw = (long long)g.Nout * g.K, a.sy = (long long)g.C * g.Nout, a.backwards = g.backwards;
    return a;
}

}  // namespace

// Tile choice; Tuning::ffn_tile (0..9 without 6) overrides it for tuning runs.  Large buffers take the ring kernels
// (pick_ring_tile).  Small buffers and narrow layers leave most of the chip
// without a 128-row tile (16 experts x 768 columns: 64 tiles of 192 columns on 256 CUs, each a serial chain of K / 64 slabs),
// so they take 64-row tiles as long as those are few; the counts are those of 64 x 64 tiles over the whole buffers, and in one rule of the
// down-projection (`live`) over the rows that an expert expects (tiles of empty rows exit at once).  bf16, us:
//   * up, one round of three workgroups per CU (<= 768): 64 x 64, three stages.  16 experts x 16 rows, 768 -> 3072: 22.3 -> 15.9;
//     32 x 188 rows, 256 -> 512: 10.8 -> 6.6; 4 x 100 rows, 960 -> 3840: 19.9 -> 9.1.  Beyond the line, 16 x 80 rows (1536 tiles): 24.4 -> 28.2.  At
//     most one a CU and from eleven slabs on, a fourth stage: 5 x 28 rows, 704 -> 2816 (220) 6.9 -> 5.9, 4 x 35, 960 -> 2880 (180) 7.9 -> 6.9; of shorter
//     ones the fill is longer than the sum (16 x 15, 256 -> 1024 4.3 -> 5.0, 6 x 248, 128 -> 384 4.5 -> 5.2), and where a CU has two they share it (4 x
//     13, 1472 -> 4416 (276) 11.6 -> 12.7).
//   * up, one round of two per CU of 64 x 128 (<= 512 of them): 16 experts x 203 rows, 256 -> 1024: 9.5 -> 8.1; 21 x 173, 320 -> 960 11.8 -> 9.0; 4 x
//     107, 1152 -> 3456 15.4 -> 13.8; at 528 16 x 185, 448 -> 1344 13.0 -> 14.0.  Contractions of one slab, and of two up to 4096 tiles, which
//     have nothing to pipeline: 64 x 551, 128 -> 256 21.1 -> 14.9, 128 x 591, 64 -> 256 29.2 -> 22.8, 16 x 4063, 64 -> 256 22.4 -> 18.6; two slabs, 16 x 4063,
//     128 -> 512 (8192) 33.6 -> 37.2.  Not where 128-wide tiles pad what 192-wide ones do not: 10 x 6493, 64 -> 192 13.8, 64 x 128 19.0; 30 x 2122 13.7 and
//     18.0.  (191 such products: 0.78 of the time in 128 x 192 tiles on the average; where those fit one round of two per CU a few are slower, by up to an
//     eighth: 31 x 990 in half-full buffers, 128 -> 384 14.9 -> 16.7, but 42 x 594, 128 -> 512 17.8 -> 16.1.)
//   * up, buffers of at most 64 rows: 64 x 128 up to 8192 (64 x 6 rows, 1024 -> 4096: 107.6 -> 93.1; 128 x 16, 768 -> 3072: 123.8 -> 114.8),
//     beyond that the chip is full anyway and 64 x 256 reads the token rows least often (256 x 63 rows, 1024 -> 4096: 444.6 -> 404.4; 64 x 128: 415.1).
//   * down, one round of two per CU (<= 512): 64 x 64 with four stages, K is long.  16 x 16 rows, 3072 -> 768: 31.0 -> 17.2;
//     8 x 469 rows, 1024 -> 256: 17.2 -> 7.2; 64 x 6, 4096 -> 1024: 123.1 -> 97.0; 5 x 488 rows, 3072 -> 768 (480 of 600 expected) 22.1, ring 26.8.
//   * down, a second round of those (to 1024) is where the ring's 128-row tiles are faster: 16 x 209 rows, 3840 -> 960 (960) 64.4 -> 39.2; 32 x 79,
//     3584 -> 896 (896) 62.8 -> 50.5; 5 x 395, 2816 -> 1408 (770) 35.1 -> 26.4; 16 x 256, 3072 -> 768 (768) 35.4 -> 31.0.  Of more than 64 experts a skewed
//     router leaves most without a row, and the few live tiles of 128 rows leave CUs idle: 90 x 82, 1280 -> 320, 21 experts live, 9.2, ring 16.8; 144 x 143, 256 ->
//     128, 9 live, 4.8 and 7.0 (evenly spread, N > 64: 0.85 to 0.93).  What narrow layers have to 768 fits one round of three per CU with three stages:
//     21 x 644, 576 -> 192 (693) 11.4 -> 8.8, ring 9.4; 88 x 107, 1024 -> 256 (704) 0.90 of four stages; beyond, half-empty buffers of many experts
//     still do by the rows expected: 160 x 177, 512 -> 128 (960, 640 live) 0.83.
//   * down, buffers of at most 64 rows, which would leave half of a 128-row tile empty: three stages and three per CU to 768 where the sum is short and
//     experts expect three rows or more, so that nearly all are live: 128 x 26, 1536 -> 384 34.8 -> 31.0; 189 x 6, 768 -> 256 0.92; but 112 x 2, 1280 -> 320 11.2 and
//     13.2, 32 x 57, 5120 -> 1280 91.0 and 93.4, 80 x 24, 1792 -> 448 skewed 12.0 and 13.8.  From there to 1024 64 x 128 where it pads nothing and as many as 64 experts
//     are live: 54 x 56, 4096 -> 1024 0.92, 50 x 8, 2304 -> 1152 0.90; but 74 x 1, 2816 -> 704 22.0 and 31.6, 60 x 4, 4096 -> 1024 1.06, 200 x 49, 1280 -> 320 39.2 and 48.2, 140
//     x 32, 1152 -> 384 skewed 9.2 and 11.2.  Then 64 x 128 up to 2048 (128 x 16 rows, 3072 -> 768: 117.0 -> 104.9), then 64 x 256 (256 x 63 rows, 4096 -> 1024:
//     374.9 -> 369.2; 64 x 128: 379.8).
// Every tile adds a row's products in the same order: the results are the same bits.
int pick_forward_tile(const Tuning &tune, int N, int C, int Nout, int K, int tokens, bool gathered)
{
    RingArgs ring{};
    ring.N = N, ring.Mrows = C, ring.Nout = Nout, ring.K = ring.ldx = ring.ldw = K;
    const bool ring_ok = ring_applies(ring, gathered ? tokens : C, false, false);
    if (tune.ffn_tile >= 0 && tune.ffn_tile != 6) return is_ring_tile(tune.ffn_tile) && !ring_ok ? 0 : tune.ffn_tile;
    const long long cols = (Nout + 63) / 64, small = N * ((C + 63ll) / 64) * cols;   // 64 x 64 tiles
    const int rows = tokens > 0 ? std::min(C, (tokens - 1) / N + 1) : C;              // that an expert expects
    if (Nout >= K) {
        if (small <= 256 && K >= 704) return 7;
        if (small <= 768) return 9;
        if (C <= 64) return small <= 8192 ? 8 : 5;
        const long long wide = (Nout + 127) / 128;
        if ((K <= 64 || (K < 192 && small <= 4096)) && wide * 128 * 10 <= Nout * 11ll) return 8;
        if (N * ((C + 63ll) / 64) * wide <= 512) return 8;
    } else if (small <= 1024) {
        const long long live = rows > 64 ? N * ((rows + 63ll) / 64) * cols : small;
        if (live <= 512 || !ring_ok) return 7;
        if (C <= 64 && small <= 768) return rows >= 3 && K <= 1536 ? 9 : 7;
        if (C <= 64) return rows >= 5 && N <= 64 && Nout % 128 == 0 ? 8 : 7;
        if (Nout <= 320 && (small <= 768 || (N > 64 && live <= 768))) return 9;
        if (N > 64) return 7;
    } else if (C <= 64) {
        return small <= 2048 ? 8 : 5;
    }
    if (!ring_ok) return 0;
    return kRingTile0 + pick_ring_tile(tune, ring, rows, false);
}

namespace {

int pick_tile(const Tuning &tune, const GemmArgs &g, int N)
{
    return pick_forward_tile(tune, N, g.C, g.Nout, g.K, g.tokens, g.x_rows != nullptr);
}

// dtype dispatch of the two MFMA launchers
hipError_t launch_half(int dtype, const GemmArgs &a, int N, int act, int tile, const Tuning &tune, hipStream_t s,
                       hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr)
{
    if (is_ring_tile(tile)) return launch_ring_forward(dtype, ring_args(a, N), act, RingTile(tile - kRingTile0), tune, s, t0, t1);
    if (dtype == SMILE_DTYPE_BF16) return launch_half_typed<__bf16>(a, N, act, tile, tune, s, t0, t1);
    return launch_half_typed<_Float16>(a, N, act, tile, tune, s, t0, t1);
}

hipError_t launch_half_dual(int dtype, const GemmArgs &a, int N, int act, const Tuning &tune, hipStream_t s)
{
    const int tile = pick_tile(tune, a, N);
    if (is_ring_tile(tile)) return launch_ring_forward(dtype, ring_args(a, N), act, RingTile(tile - kRingTile0), tune, s);
    if (dtype == SMILE_DTYPE_BF16) return launch_half_dual_typed<__bf16>(a, N, act, tile, tune, s);
    return launch_half_dual_typed<_Float16>(a, N, act, tile, tune, s);
}

}  // namespace

bool use_persistent_grid(const Tuning &tune, int N, long long tiles, int slots)
{
    if (N > 4096) return false;   // the tile walk keeps one lane per 64 groups
    if (tune.persist >= 0) return tune.persist != 0;
    return tiles >= 4LL * slots;
}

// the fp32 product of the same description (gemm_f32.hip)
static F32Gemm f32_gemm(const GroupedGemm &g)
{
    F32Gemm f{};
    f.x = g.x, f.w = g.w, f.y = g.y, f.y2 = g.y2, f.bias = g.bias, f.x_rows = g.x_rows;
    f.rows_valid = g.kept, f.N = g.N, f.Mrows = g.C, f.Nout = g.Nout, f.K = g.K, f.ldx = g.K, f.ldw = g.K;
    f.sx = (long long)g.C * g.K, f.sw = (long long)g.Nout * g.K, f.sy = (long long)g.C * g.Nout;
    f.act = g.act, f.tune = g.tune;
    return f;
}

hipError_t launch_grouped_gemm_nt(int dtype, const GroupedGemm &g, hipStream_t s)
{
    const int act = g.act == 0 ? 0 : (g.act == 1 ? 1 : 2);
    if (g.y2 && act == 0) return hipErrorInvalidValue;
    if (!is_half(dtype)) return launch_grouped_gemm_f32(f32_gemm(g), s);
    if (g.K % 64 || g.Nout % 8) return hipErrorInvalidValue;
    GemmArgs a{g.x, g.w, g.bias, g.y, g.kept, g.C, g.Nout, g.K, 0, 0, 0, g.x_rows, nullptr, nullptr, nullptr, g.y2};
    a.tokens = g.tokens;
    if (g.y2) return launch_half_dual(dtype, a, g.N, act, g.tune, s);
    return launch_half(dtype, a, g.N, act, pick_tile(g.tune, a, g.N), g.tune, s);
}

hipError_t launch_expert_ffn_up(const LayerDesc &d, const Workspace &ws, const void *xe,
                                const int32_t *kept_count, const void *w1, const void *b1, hipStream_t s,
                                hipEvent_t t0, hipEvent_t t1, const void *x_tokens, void *h_save, void *pre_save)
{
    const int N = d.n_groups * d.m_local;
    const int act = d.act == SMILE_ACT_RELU ? 1 : 2;
    // x_tokens: read the rows straight from the token matrix through the slot -> token map
    const int32_t *x_rows = x_tokens ? ws.slot_token : nullptr;
    const void *src = x_tokens ? x_tokens : xe;
    if (h_save) {   // training: the hidden activation and its pre-activation go to the caller's buffers
        if (t0 && t1) (void)hipEventRecord(t0, s);
        const hipError_t err = launch_grouped_gemm_nt(
            d.dtype, GroupedGemm{src, w1, h_save, pre_save, kept_count, N, d.capacity, d.d_ff, d.d_model, act, b1, x_rows,
                                 d.tune, d.T}, s);
        if (t0 && t1) (void)hipEventRecord(t1, s);
        return err;
    }
    if (is_half(d.dtype)) {
        GemmArgs g{src, w1, b1, ws.hidden, kept_count, d.capacity, d.d_ff, d.d_model, 0, 0, 0, x_rows, nullptr, nullptr, nullptr};
        g.tokens = d.T;
        return launch_half(d.dtype, g, N, act, pick_tile(d.tune, g, N), d.tune, s, t0, t1);
    }
    if (t0 && t1) (void)hipEventRecord(t0, s);
    const hipError_t err = launch_grouped_gemm_f32(
        f32_gemm(GroupedGemm{src, w1, ws.hidden, nullptr, kept_count, N, d.capacity, d.d_ff, d.d_model, act, b1, x_rows, d.tune}), s);
    if (t0 && t1) (void)hipEventRecord(t1, s);
    return err;
}

hipError_t launch_expert_ffn_down(const LayerDesc &d, const Workspace &ws, const int32_t *kept_count,
                                  const void *w2, const void *b2, void *ye, hipStream_t s, void *y_tokens,
                                  const float *gate, const void *h_saved)
{
    const int N = d.n_groups * d.m_local;
    const void *hidden = h_saved ? h_saved : ws.hidden;
    // y_tokens: also (or, with ye == null, only) return the rows to token order, times the gate
    const int32_t *y_rows = y_tokens ? ws.slot_token : nullptr;
    if (is_half(d.dtype)) {
        GemmArgs g{hidden, w2, b2, ye, kept_count, d.capacity, d.d_model, d.d_ff, 0, 0, 0, nullptr, y_rows, y_tokens, gate};
        // From the last expert to the first: what the up-projection wrote last is still in the 256 MB memory-side cache (128 experts x 256
        // rows, 768 x 3072, 188 MB of h: 447.0 -> 441.9 us a pass; behind the flat router 479.6 -> 474.9; others within 0.3 %)
        g.backwards = true;
        g.tokens = d.T;
        return launch_half(d.dtype, g, N, 0, pick_tile(d.tune, g, N), d.tune, s);
    }
    F32Gemm f = f32_gemm(GroupedGemm{hidden, w2, ye, nullptr, kept_count, N, d.capacity, d.d_model, d.d_ff, 0, b2, nullptr, d.tune});
    f.y_rows = y_rows, f.y_tok = y_tokens, f.gate = gate;
    return launch_grouped_gemm_f32(f, s);
}

}  // namespace smile
