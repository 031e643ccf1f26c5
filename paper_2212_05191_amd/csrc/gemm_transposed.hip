// Grouped 16-bit (bf16 / fp16) MFMA GEMM whose operands may be stored with the contraction index as the SLOW index
// ("transposed"): the four gradient GEMMs of the expert FFN backward pass,
//
//     dpre[r,f] = sum_c dye[r,c] W2[c,f]      x normal,      w transposed      (K = d)
//     dxe [r,k] = sum_f dpre[r,f] W1[f,k]     x normal,      w transposed      (K = F)
//     dW2 [c,f] = sum_r dye[r,c] h[r,f]       x transposed,  w transposed      (K = rows of the expert)
//     dW1 [f,k] = sum_r dpre[r,f] xe[r,k]     x transposed,  w transposed      (K = rows of the expert)
//
// without materialising any transposed copy.  y[e][i][j] = sum_k X(i,k) W(j,k) per group e, where a
// normal operand is stored [i][k] (k contiguous) and a transposed one [k][i] (i contiguous).
//
// Most of these products run on the ring kernels (gemm_ring.hpp).  The two-stage kernel below takes weight gradients of few rows and
// other small products (launch_grouped_gemm_t), normal operands of fewer than three slabs and operands whose offsets need more than 32 bits.
// weight_gradient_kernel takes the weight gradients of short sums where there are many tiles.
//
// Design (gfx950):
//   * global -> LDS with the direct 16-byte loads of the forward kernel, two stages of K slabs
//     (BK = 64).  A normal operand lands as [row][64 k] (8 pieces per row, XOR-swizzled); a transposed
//     one lands as it is in memory, [k][BM or BN columns] (16 or 32 pieces per row).
//   * MFMA 32x32x16 bf16 wants, per lane, 8 consecutive k of one row/column.  From a normal tile that
//     is one 16-byte LDS read.  From a transposed tile it is two transposing LDS reads
//     (ds_read_b64_tr_b16): within each group of 16 lanes, lane 4a+b receives element b of the four
//     8-byte rows addressed by lanes a, a+4, a+8, a+12.  Lane i of a group therefore addresses
//     k-row (i / 4) [+4 for the second read] and the 4-column block (i % 4) of its 16-column span,
//     and every lane ends up with k, k+1, k+2, k+3 of its own column -- the same k order as a
//     normal operand, so the two kinds mix in one MFMA.
//   * transposed tiles are swizzled by k: a row's pieces are rotated by 4 * (k & 3) positions.  The 8
//     k-rows a wave touches in one read then cover all 64 banks twice, the minimum for 512 bytes
//     (rows of 16, 24 or 32 pieces alike; with 24 the last group of four pieces wraps onto a used bank).
//   * the contraction length of the weight-gradient GEMMs is the expert's row count: slabs beyond it
//     are skipped, and k-rows beyond it inside the last slab are loaded from a zero block instead
//     (no zero-padded copies, no work on empty buffer rows).
//   * epilogue as in the forward kernel: fp32 -> bf16, staged through LDS, row-contiguous 16-byte
//     stores; POST multiplies by act'(aux) there (the gradient at the pre-activation).
#include <algorithm>
#include <climits>
#include <type_traits>

#include "gemm_device.hpp"

namespace smile {

namespace {

constexpr int BK = 64, STAGES = 2, kWorkgroupsPerCu = 2;   // one workgroup's loads and epilogue hide behind the other's MFMAs

// E: the 16-bit storage type (__bf16 or _Float16)
template <typename E>
struct TGemmArgs {
    const E *x, *w;
    E *y;
    const E *aux;             // POST: [N][rows][Nout] like y
    const int32_t *rows_valid;   // [N] valid output rows per group, or null: Mrows for all
    const int32_t *k_valid;      // [N] valid contraction length per group, or null: K for all
    int Mrows, Nout, K;          // output extents per group and the full contraction length
    int ldx, ldw;                // leading dimensions (elements) of x and w
    long long sx, sw, sy;        // per-group strides (elements) of x, w and y / aux
    int row_tiles, col_tiles, tiles;
    int N;                       // groups
};

// One operand tile of a stage, as seen by the loader and by the MFMA fragment reader.
//   T == false: [EXT rows][8 pieces], piece ^= (row >> 1) & 7
//   T == true : [64 k][EXT / 8 pieces], position = (piece + 4 * (k & 3)) mod (EXT / 8)
template <typename E, int EXT, bool T>
struct OperandTile {
    static constexpr int kPieces = EXT * BK / 8;
    static constexpr int kPiecesPerK = EXT / 8;

    // global source of linear LDS piece q (slab 0) and whether / how it depends on k
    __device__ static __forceinline__ const E *source(const E *base, int q, int tile0, int ext_valid, int ld,
                                                      int &k_row)
    {
        if constexpr (!T) {
            const int row = q >> 3, piece = (q & 7) ^ ((row >> 1) & 7);
            k_row = -1;   // all k of this piece are inside the slab; no k bound needed (K % 64 == 0)
            return base + (size_t)min(tile0 + row, ext_valid - 1) * ld + piece * 8;
        } else {
            const int k = q / kPiecesPerK, pos = q - k * kPiecesPerK;
            const int piece = pos - 4 * (k & 3) + (pos < 4 * (k & 3) ? kPiecesPerK : 0);   // the piece rotated to pos
            k_row = k;
            return base + (size_t)k * ld + min(tile0 + piece * 8, ext_valid - 8);
        }
    }
};

template <typename E, int BM, int BN, bool XT, bool WT, int POST, bool PERSIST = false>
__global__ __launch_bounds__(256, kWorkgroupsPerCu) void grouped_gemm_t_kernel(TGemmArgs<E> a)
{
    typedef typename Half<E>::vec8 bf16x8;                              // one MFMA operand: 8 elements
    typedef __attribute__((__vector_size__(4 * sizeof(E)))) E bf16x4;   // 4 rounded outputs
    constexpr int WGM = 2, WGN = 2, NW = WGM * WGN, NT = NW * 64;   // waves along rows and columns
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int TM = WM / 32, TN = WN / 32;
    using XTile = OperandTile<E, BM, XT>;
    using WTile = OperandTile<E, BN, WT>;
    constexpr int XI = XTile::kPieces / 64, WI = WTile::kPieces / 64;   // load instructions per slab
    constexpr int GPW = (XI + WI) / NW;
    constexpr int STAGE = XTile::kPieces + WTile::kPieces;
    constexpr int OROWS = WGM * 32, OSTRIDE = BN / 8 + 1, OPR = BN / 8;
    static_assert((XI + WI) % NW == 0, "load instructions must divide over the waves");
    static_assert(BM % 32 == 0 && BN % 32 == 0 && BM >= 128 && BN >= 128, "rotation swizzle: rows of at least 16 pieces");
    static_assert(OROWS * OSTRIDE <= STAGES * STAGE, "epilogue staging must fit in the pipeline buffers");

    __shared__ u32x4 lds[STAGES * STAGE];

    // ---- which tile(s): one per workgroup (plain grid, ids remapped so that each XCD gets a contiguous range) or
    // PERSIST: one workgroup per slot of the chip walks the live tiles (LiveTileWalk) and requests the first
    // slabs of its next tile before the epilogue of the current one (PREFETCH), which then stages its output in
    // the one pipeline buffer those loads do not touch.
    constexpr bool PREFETCH = PERSIST && OROWS * OSTRIDE <= STAGE;
    constexpr int STG = PREFETCH ? (STAGES - 1) * STAGE : 0;   // staging area, in 16-byte units
    LiveTileWalk<BM> walk;
    if constexpr (PERSIST) walk.init(a.rows_valid, a.N, a.Mrows, a.col_tiles, XT && WT);
    struct Tile {
        int e, rt, ct, rows, kv;
    };
    auto select = [&](Tile &t) {
        if constexpr (PERSIST) {
            if (!walk.tile(t.e, t.rt, t.ct, t.rows)) return false;
        } else {
            const int per_xcd = (a.tiles + kXcds - 1) / kXcds;
            const int lid = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
            if (lid >= a.tiles) return false;
            const int per_group = a.row_tiles * a.col_tiles;
            t.e = lid / per_group;
            const int rem = lid - t.e * per_group;
            t.ct = rem / a.row_tiles, t.rt = rem - t.ct * a.row_tiles;
        }
        if constexpr (!PERSIST) t.rows = a.rows_valid ? min(a.rows_valid[t.e], a.Mrows) : a.Mrows;
        t.kv = a.k_valid ? min(a.k_valid[t.e], a.K) : a.K;
        return t.rt * BM < t.rows;
    };

    // ---- loader: this lane's source of each of the wave's load instructions (slab 0), the k-row it
    // holds (transposed operands; -1 otherwise) and its advance per slab
    // Instruction wave + i*NW of a slab: the first XI / NW values of i fill the x tile for every wave, the
    // rest the w tile (both counts are multiples of NW), so the kind of each load is known at compile time.
    static_assert(XI % NW == 0, "x tile instructions must divide over the waves");
    constexpr int XG = XI / NW;
    // The contraction length is ragged only in the weight-gradient GEMMs (both operands transposed).
    constexpr bool KRAGGED = XT && WT;
    const E *src[GPW];
    int krow[GPW];
    int kv = 0;   // contraction length of the tile whose loads are being issued
    const size_t adv_x = XT ? (size_t)BK * a.ldx : (size_t)BK, adv_w = WT ? (size_t)BK * a.ldw : (size_t)BK;
    const E *zero = reinterpret_cast<const E *>(kZeroPiece);
    // load instruction i of slab `slab` into `stage`
    auto load_one = [&](int wave, int i, int slab, lds_char *to) {
        const E *p = src[i] + (size_t)slab * (i < XG ? adv_x : adv_w);
        if (KRAGGED && slab * BK + krow[i] >= kv) p = zero;   // beyond the contraction length
        __builtin_amdgcn_global_load_lds(SMILE_GPTR(p), SMILE_LPTR(to + (wave + i * NW) * 1024), 16, 0, 0);
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
        const E *X = a.x + (size_t)t.e * a.sx;
        const E *W = a.w + (size_t)t.e * a.sw;
        kv = t.kv;
        const int slabs = (t.kv + BK - 1) / BK;
#pragma unroll
        for (int i = 0; i < GPW; ++i) {
            const int inst = wave + i * NW;
            if (i < XG) {
                // a transposed x holds the output rows along its fast index: all Mrows columns exist in memory
                src[i] = XTile::source(X, inst * 64 + lane, t.rt * BM, XT ? a.Mrows : t.rows, a.ldx, krow[i]);
            } else {
                src[i] = WTile::source(W, (inst - XI) * 64 + lane, t.ct * BN, a.Nout, a.ldw, krow[i]);
            }
        }
#pragma unroll
        for (int s = 0; s < STAGES - 1; ++s)
            if (s < slabs) {
#pragma unroll
                for (int i = 0; i < GPW; ++i) load_one(wave, i, s, (lds_char *)(lds + s * STAGE));
            }
    };

    Tile cur;
    if (!select(cur)) return;
    start_tile(cur);
    for (;;) {
    const int e = cur.e, rt = cur.rt, ct = cur.ct, rows = cur.rows;
    const int slabs = (cur.kv + BK - 1) / BK;
    const int tid = thread_id(), lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WGM, wn = wave / WGM;

    // ---- fragment addressing
    // normal: lane reads row (lane & 31), pieces 2*kk + (lane >> 5)
    const int frow = lane & 31, fhi = lane >> 5, fsw = (frow >> 1) & 7;
    // transposed: lane = 16 g + 4 j + a addresses k-row 8 (g / 2) + j (+4: second read, +16 kk) and the
    // 4 columns 16 (g % 2) + 4 a of the 32-column tile
    const int tg = lane >> 4, tj = (lane >> 2) & 3, ta = lane & 3;
    const int tk0 = 8 * (tg >> 1) + tj;
    const int tcol = 16 * (tg & 1) + 4 * ta;   // column inside the 32-column tile
    int xoff[TM], woff[TN];                    // byte offsets inside the stage for kk = 0, first read
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        if constexpr (XT) {
            const int col = wm * WM + j * 32 + tcol;
            xoff[j] = (tk0 * XTile::kPiecesPerK + ((col >> 3) + 4 * tj) % XTile::kPiecesPerK) * 16 + (col & 4) * 2;
        } else {
            xoff[j] = ((wm * WM + j * 32 + frow) * 8) * 16;
        }
    }
#pragma unroll
    for (int i = 0; i < TN; ++i) {
        if constexpr (WT) {
            const int col = wn * WN + i * 32 + tcol;
            woff[i] = (XTile::kPieces + tk0 * WTile::kPiecesPerK + ((col >> 3) + 4 * tj) % WTile::kPiecesPerK) * 16 +
                      (col & 4) * 2;
        } else {
            woff[i] = ((XTile::kPieces + (wn * WN + i * 32 + frow) * 8)) * 16;
        }
    }

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    const bool wave_live = rt * BM + wm * WM < rows;   // wave-uniform
    constexpr int KS = BK / 16, NM = TM * TN, NF = TM + TN;
    bf16x8 xf[2][TM], wf[2][TN];   // fragments of the k-step being multiplied and of the next one
    auto fetch_one = [&](auto slot, auto kstep, const lds_char *from) {   // fragment `slot` (x tiles first) of k-step `kstep`
        constexpr int F = decltype(slot)::value, KK = decltype(kstep)::value;
        if constexpr (F < TM) {
            if constexpr (XT) read_transposed<4 * XTile::kPiecesPerK * 16>(xf[KK & 1][F], from + xoff[F] + KK * 16 * XTile::kPiecesPerK * 16);
            else xf[KK & 1][F] = *(const __attribute__((address_space(3))) bf16x8 *)(from + xoff[F] + (((2 * KK + fhi) ^ fsw) * 16));
        } else {
            constexpr int I = F - TM;
            if constexpr (WT) read_transposed<4 * WTile::kPiecesPerK * 16>(wf[KK & 1][I], from + woff[I] + KK * 16 * WTile::kPiecesPerK * 16);
            else wf[KK & 1][I] = *(const __attribute__((address_space(3))) bf16x8 *)(from + woff[I] + (((2 * KK + fhi) ^ fsw) * 16));
        }
    };
    // Waits for the slab requested last (this wave's part landed, then everybody's); every wave is then also done reading the slab
    // before it, whose buffer may be filled again.
    auto enter_slab = [&]() {
        wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
    };
    // The MFMAs of k-step KK, and behind the first of them the reads of the k-step after it, so that the last ones cover
    // the reads' latency; load instructions L0 .. L1-1 of slab `slab` are spread over all (the order is pinned).
    auto multiply = [&](auto kstep, auto l0, auto l1, const lds_char *from, int slab, lds_char *fill) {
        constexpr int KK = decltype(kstep)::value, L0 = decltype(l0)::value, L1 = decltype(l1)::value;
        __builtin_amdgcn_sched_barrier(0);
        for_constants<NM>([&](auto m) {
            constexpr int R = decltype(m)::value;
            acc[R / TM][R % TM] = Half<E>::mfma_32x32x16(wf[KK & 1][R / TM], xf[KK & 1][R % TM], acc[R / TM][R % TM]);
            constexpr int F0 = min_int(NF, 2 * R), F1 = min_int(NF, 2 * R + 2);
            for_constants<F1 - F0>([&](auto f) {
                fetch_one(std::integral_constant<int, F0 + decltype(f)::value>{}, std::integral_constant<int, (KK + 1) % KS>{}, from);
            });
            constexpr int G0 = L0 + (L1 - L0) * R / NM, G1 = L0 + (L1 - L0) * (R + 1) / NM;
            for_constants<G1 - G0>([&](auto g) { load_one(wave, G0 + decltype(g)::value, slab, fill); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // All k-steps of a slab but the last, its first fragments already in registers, reading `from`.  MORE: with the load
    // instructions of slab `slab`, into `fill`, the other stage.
    auto front_steps = [&](auto more_tag, int slab, const lds_char *__restrict from, lds_char *__restrict fill) {
        constexpr int G = decltype(more_tag)::value ? GPW : 0;
        for_constants<KS - 1>([&](auto kstep) {
            constexpr int KK = decltype(kstep)::value;
            __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this k-step's fragments
            multiply(kstep, std::integral_constant<int, G * KK / (KS - 1)>{}, std::integral_constant<int, G * (KK + 1) / (KS - 1)>{}, from, slab, fill);
        });
    };
    // One K slab.  MORE: slabs kt+1 .. kt+STAGES-1 exist (steady state).  The wait and the barrier for slab kt+1 stand in front
    // of this slab's LAST k-step, whose MFMAs cover the LDS reads of the next slab's first fragments, as in the forward kernel (a training
    // step of 256 skewed experts, whose contractions are a slab or two long, neither gains nor loses: 3569 -> 3584 us).
    auto slab_step = [&](auto more_tag, int kt, int stage) {
        constexpr bool MORE = decltype(more_tag)::value;
        const int fill = stage == 0 ? STAGES - 1 : stage - 1, next = stage + 1 == STAGES ? 0 : stage + 1;
        front_steps(more_tag, kt + STAGES - 1, (const lds_char *)(lds + stage * STAGE), (lds_char *)(lds + fill * STAGE));
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the last k-step's fragments, this wave's last reads of the slab
        if (MORE || kt + 1 < slabs) enter_slab();
        // after the last slab: stale fragments, never multiplied
        multiply(std::integral_constant<int, KS - 1>{}, std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{},
                 (const lds_char *)(lds + next * STAGE), 0, nullptr);
    };
    // the next tile is chosen before the main loop, so that the loads of its row counts are long back when
    // the epilogue needs them
    Tile nxt_tile;
    bool more = false;
    if constexpr (PERSIST) {
        walk.advance();
        more = select(nxt_tile);
    }
    if (slabs > 0) enter_slab();
    int kt = 0, stage = 0;
    if (wave_live) {
        if (slabs > 0) for_constants<NF>([&](auto f) { fetch_one(f, std::integral_constant<int, 0>{}, (const lds_char *)lds); });
        for (; kt + STAGES - 1 < slabs; ++kt) {
            slab_step(std::true_type{}, kt, stage);
            stage = stage + 1 == STAGES ? 0 : stage + 1;
        }
        for (; kt < slabs; ++kt) {
            slab_step(std::false_type{}, kt, stage);
            stage = stage + 1 == STAGES ? 0 : stage + 1;
        }
    } else {
        // none of this wave's rows exists: it only helps loading
        for (; kt < slabs; ++kt) {
            if (kt > 0) enter_slab();
            if (kt + STAGES - 1 < slabs) {
                lds_char *fill = (lds_char *)(lds + (stage == 0 ? STAGES - 1 : stage - 1) * STAGE);
#pragma unroll
                for (int i = 0; i < GPW; ++i) load_one(wave, i, kt + STAGES - 1, fill);
            }
            stage = stage + 1 == STAGES ? 0 : stage + 1;
        }
    }

    // ---- epilogue.  Accumulator element v of a lane is (column 8*(v/4) + 4*(lane/32) + v%4, row lane%32)
    // of its 32x32 tile: rounded to bf16, staged as a [OROWS][BN] tile, stored row-contiguously.
    E *Y = a.y + (size_t)e * a.sy;
    u32x2 *stg = reinterpret_cast<u32x2 *>(lds + STG);
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave's LDS reads are done
        __builtin_amdgcn_s_barrier();
        if (PREFETCH && j == 0 && more) start_tile(nxt_tile);
#pragma unroll
        for (int i = 0; i < TN; ++i) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int lcol = wn * WN + i * 32 + 8 * q + 4 * fhi;
                bf16x4 out;
#pragma unroll
                for (int v = 0; v < 4; ++v) out[v] = (E)acc[i][j][4 * q + v];
                stg[((wm * 32 + frow) * OSTRIDE) * 2 + (lcol >> 2)] = __builtin_bit_cast(u32x2, out);
            }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        // all of the thread's staged pieces are read before the first store, so that the LDS latencies overlap
        constexpr int NIT = (OROWS * OPR + NT - 1) / NT;
        u32x4 outv[NIT];
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int id = min(tid + it * NT, OROWS * OPR - 1);
            const int orow = id / OPR, piece = id - orow * OPR;
            outv[it] = lds[STG + orow * OSTRIDE + piece];
        }
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int id = tid + it * NT;
            const int orow = id / OPR, piece = id - orow * OPR;
            const int row = rt * BM + (orow >> 5) * WM + j * 32 + (orow & 31);
            const int col = ct * BN + piece * 8;
            if (id < OROWS * OPR && row < rows && col < a.Nout) {
                u32x4 v = outv[it];
                if constexpr (POST != 0) {
                    const u32x4 p = *reinterpret_cast<const u32x4 *>(a.aux + (size_t)e * a.sy + (size_t)row * a.Nout + col);
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        v[k] = Half<E>::pack(Half<E>::lo(v[k]) * activate_grad<POST>(Half<E>::lo(p[k])),
                                             Half<E>::hi(v[k]) * activate_grad<POST>(Half<E>::hi(p[k])));
                }
                u32x4 *dst = reinterpret_cast<u32x4 *>(Y + (size_t)row * a.Nout + col);
                // weight gradients are not read again soon: keep them out of the way of the operands in L2
                if constexpr (KRAGGED) __builtin_nontemporal_store(v, dst);
                else *dst = v;
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

// Weight gradients whose contraction is short: y[e][i][j] = sum over the group's rows of X(i,k) W(j,k), both operands transposed, 128 x 128
// outputs for a workgroup of four waves.  A tile is a slab or a few of them and then its stores, a serial chain (load, wait, multiply, stage,
// store) whose latencies no prefetch inside one workgroup covers, so here many workgroups share a CU instead of pipelining one: a
// single slab buffer (32 KB, which the epilogue stages in) and 128 registers leave room for four, on a plain grid that the hardware
// deals out.  256 skewed experts (55 rows on average) of 1024 x 4096, 2.15 GB of gradients, us: ring 650, two-stage 649, here 571; with nothing to
// contract, stores alone, 364 (5.9 TB/s); without the stores 281: a quarter of the time is neither, mostly loads that wait behind stores.
// Three or five workgroups on a CU instead of four: 571, 585; cached stores 606 and the next kernel 11 % slower.
// Stores are whole lines (rows of 64 columns, 128 bytes): tiles written in runs of 64 bytes reach 3.9 TB/s, of 128 bytes 5.9.
// The XCDs take chunks of tiles in turn, as the weight gradients of the ring kernels do (LiveTileWalk).
template <typename E>
__global__ __launch_bounds__(256, 4) void weight_gradient_kernel(TGemmArgs<E> a)
{
    typedef typename Half<E>::vec8 vec8;
    typedef __attribute__((__vector_size__(4 * sizeof(E)))) E vec4;
    constexpr int BM = 128, BN = 128, NW = 4, OPERAND = BK * 256;   // bytes of an operand's slab: [64 k][16 pieces], rotated by 4 * (k & 3)
    __shared__ __attribute__((aligned(16))) char slab_lds[2 * OPERAND];
    lds_char *const lds = (lds_char *)slab_lds;

    const int chunks = max(1, (a.tiles + 1023) / 1024), chunk = (a.tiles + 8 * chunks - 1) / (8 * chunks);
    const int local = blockIdx.x / kXcds, ticket = ((local / chunk) * kXcds + blockIdx.x % kXcds) * chunk + local % chunk;
    if (ticket >= a.tiles) return;
    const int per_group = a.row_tiles * a.col_tiles;
    // neighbours go along the longer side, so that they share the operand tile of the shorter one
    const int e = ticket / per_group, rem = ticket - e * per_group, fast = a.row_tiles > a.col_tiles ? a.row_tiles : a.col_tiles;
    const int slow_tile = rem / fast, fast_tile = rem - slow_tile * fast;
    const int rt = a.row_tiles > a.col_tiles ? fast_tile : slow_tile, ct = a.row_tiles > a.col_tiles ? slow_tile : fast_tile;
    const int kv = a.k_valid ? min(a.k_valid[e], a.K) : a.K, slabs = (kv + BK - 1) / BK;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wn = wave >> 1;
    // loads: instruction wave + 4 i of an operand is its k-rows 4 (wave + 4 i) .. + 3
    const int krow = lane >> 4, piece = ((lane & 15) - 4 * (krow & 3)) & 15;
    const E *const x = a.x + (size_t)e * a.sx + min(rt * BM + piece * 8, a.Mrows - 8);
    const E *const w = a.w + (size_t)e * a.sw + min(ct * BN + piece * 8, a.Nout - 8);
    const E *const zero = reinterpret_cast<const E *>(kZeroPiece);

    f32x16 acc[2][2];   // [columns][rows] of the wave's 64 x 64
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // fragments: lane = 16 g + 4 j + b addresses k-row 8 (g / 2) + j and the 4 columns 16 (g % 2) + 4 b of its 32 (see the header)
    const int tj = (lane >> 2) & 3, tk0 = 8 * (lane >> 5) + tj, tcol = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    int xoff[2], woff[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int xc = wm * 64 + b * 32 + tcol, wc = wn * 64 + b * 32 + tcol;
        xoff[b] = tk0 * 256 + (((xc >> 3) + 4 * tj) & 15) * 16 + (xc & 4) * 2;
        woff[b] = OPERAND + tk0 * 256 + (((wc >> 3) + 4 * tj) & 15) * 16 + (wc & 4) * 2;
    }
    for (int s = 0; s < slabs; ++s) {
        if (s > 0) __syncthreads();   // every wave is done with the slab before
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int inst = wave + i * NW, k = s * BK + inst * 4 + krow;
            __builtin_amdgcn_global_load_lds(SMILE_GPTR(k < kv ? x + (size_t)k * a.ldx : zero), SMILE_LPTR(lds + inst * 1024), 16, 0, 0);
            __builtin_amdgcn_global_load_lds(SMILE_GPTR(k < kv ? w + (size_t)k * a.ldw : zero), SMILE_LPTR(lds + OPERAND + inst * 1024), 16, 0, 0);
        }
        wait_vmcnt<0>();
        __syncthreads();
        for_constants<BK / 16>([&](auto kk) {
            constexpr int AT = decltype(kk)::value * 16 * 256;
            vec8 xf[2], wf[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                read_transposed<4 * 256>(xf[b], lds + xoff[b] + AT);
                read_transposed<4 * 256>(wf[b], lds + woff[b] + AT);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = Half<E>::mfma_32x32x16(wf[i], xf[j], acc[i][j]);
        });
    }

    // ---- epilogue: a block of 32 rows x 64 columns of each wave at a time through the wave's own 4 KB (piece c of a row at c ^ ((row >> 1) & 7))
    if (slabs > 0) __syncthreads();
    E *const y = a.y + (size_t)e * a.sy;
    lds_char *const stg = lds + wave * 4096;
    const int col = ct * BN + wn * 64 + (lane & 7) * 8;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row0 = rt * BM + wm * 64 + j * 32;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                vec4 out;
#pragma unroll
                for (int v = 0; v < 4; ++v) out[v] = (E)acc[i][j][4 * q + v];
                const int r = lane & 31;
                *(__attribute__((address_space(3))) vec4 *)(stg + r * 128 + (((i * 4 + q) ^ ((r >> 1) & 7)) * 16) + (lane >> 5) * 8) = out;
            }
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int r = it * 8 + (lane >> 3);
            const u32x4 v = *(const __attribute__((address_space(3))) u32x4 *)(stg + r * 128 + (((lane & 7) ^ ((r >> 1) & 7)) * 16));
            // weight gradients are not read again soon: keep them out of the way of the operands in L2
            if (row0 + r < a.Mrows && col < a.Nout) __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(y + (size_t)(row0 + r) * a.Nout + col));
        }
    }
}

template <typename E>
hipError_t launch_weight_gradient(TGemmArgs<E> a, int N, hipStream_t s)
{
    a.row_tiles = (a.Mrows + 127) / 128, a.col_tiles = (a.Nout + 127) / 128, a.tiles = N * a.row_tiles * a.col_tiles, a.N = N;
    const int chunks = std::max(1, (a.tiles + 1023) / 1024), chunk = (a.tiles + 8 * chunks - 1) / (8 * chunks);
    SMILE_LAUNCH(weight_gradient_kernel<E>, dim3(8 * chunks * chunk), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <typename E, int BM, int BN, bool XT, bool WT, int POST>
hipError_t launch_tile(TGemmArgs<E> a, int N, const Tuning &tune, hipStream_t s)
{
    a.row_tiles = (a.Mrows + BM - 1) / BM;
    a.col_tiles = (a.Nout + BN - 1) / BN;
    a.tiles = N * a.row_tiles * a.col_tiles;
    a.N = N;
    const int slots = workgroup_slots(tune, kWorkgroupsPerCu);
    if (use_persistent_grid(tune, N, a.tiles, slots)) {
        SMILE_LAUNCH((grouped_gemm_t_kernel<E, BM, BN, XT, WT, POST, true>), dim3(slots), dim3(256),
                           0, s, a);
    } else {
        const int per_xcd = (a.tiles + kXcds - 1) / kXcds;
        SMILE_LAUNCH((grouped_gemm_t_kernel<E, BM, BN, XT, WT, POST>), dim3(per_xcd * kXcds),
                           dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

// wide: 192 columns a tile; short_sums: weight_gradient_kernel (weight gradients only)
template <typename E>
hipError_t launch_typed(const TransposedGemm &g, bool wide, bool short_sums, hipStream_t s)
{
    TGemmArgs<E> a{static_cast<const E *>(g.x), static_cast<const E *>(g.w), static_cast<E *>(g.y),
                   static_cast<const E *>(g.aux), g.rows_valid, g.k_valid, g.Mrows, g.Nout, g.K, g.ldx, g.ldw,
                   g.sx, g.sw, g.sy, 0, 0, 0, g.N};
    if (g.x_transposed) {
        if (short_sums) return launch_weight_gradient<E>(a, g.N, s);
        if (wide) return launch_tile<E, 128, 192, true, true, 0>(a, g.N, g.tune, s);
        return launch_tile<E, 128, 128, true, true, 0>(a, g.N, g.tune, s);
    }
    if (g.post == 1) return launch_tile<E, 128, 128, false, true, 1>(a, g.N, g.tune, s);
    if (g.post == 2) return launch_tile<E, 128, 128, false, true, 2>(a, g.N, g.tune, s);
    return launch_tile<E, 128, 128, false, true, 0>(a, g.N, g.tune, s);
}

}  // namespace

hipError_t launch_grouped_gemm_t(int dtype, const TransposedGemm &g, hipStream_t s)
{
    if (!is_half(dtype)) return hipErrorInvalidValue;
    if (g.K < 1 || g.Mrows < 1 || g.Nout % 64 || g.ldx % 8 || g.ldw % 8) return hipErrorInvalidValue;
    if (!g.x_transposed && g.K % BK) return hipErrorInvalidValue;   // a normal operand is read in whole 64-k slabs
    if (!g.w_transposed) return hipErrorInvalidValue;               // not needed by any caller
    if (g.x_transposed && (g.Mrows % 8 || g.post)) return hipErrorInvalidValue;
    RingArgs a{};
    a.x = g.x, a.w = g.w, a.y = g.y, a.aux = g.aux, a.rows_valid = g.rows_valid, a.k_valid = g.k_valid, a.N = g.N, a.Mrows = g.Mrows;
    a.Nout = g.Nout, a.K = g.K, a.ldx = g.ldx, a.ldw = g.ldw, a.sx = g.sx, a.sw = g.sw, a.sy = g.sy;
    const int expected = g.tokens > 0 ? (g.tokens + g.N - 1) / g.N : INT_MAX;   // rows per group if the tokens spread evenly
    const RingTile tile = g.tune.tgemm_tile > 0 ? RingTile(g.tune.tgemm_tile - 1)
                                                : pick_ring_tile(g.tune, a, std::min(g.rows_valid ? expected : INT_MAX, g.Mrows), true);
    const bool wide = g.x_transposed && tile == kRing128x192x2;
    // The two-stage kernel keeps what is over before a ring pays.
    //   * Weight gradients of few rows and few tiles, by the rows a group is expected to contract and not by its buffer: they are bound by their
    //     stores, which leave here in whole rows of a tile and from the ring in runs of 64 and 128 bytes.  Up to 320 rows where the
    //     tiles are 128 wide, 192 where they are 192 wide.  us, both kernels in the width they take, dW2: 96 experts x 80 rows in
    //     buffers of 80, 1024 x 4096 283, ring 313; 64 x 96 in 144, 768 x 3072 114 and 133; 48 x 96 in 144, 1600 x 6400 340 and 381;
    //     64 x 176, 768 x 3072 142 and 140; 64 x 208, 1024 x 4096 274 and 269; 64 x 300 309 and 294; 128 wide: 64 x 180,
    //     256 x 1024 14.2 and 15.0; 21 x 240, 192 x 576 7.4 and 8.5; 64 x 800, 256 x 1024 47 and 46.
    //   * Other products with rows for half a tile, less than eight slabs and at most two tiles per CU, or four slabs and at most one
    //     tile per CU, where the plain grid needs no walk (us: 111 experts x 4 rows, 128 x 384: dxe 6.2, ring 6.5; 43 x 10, 192 x 768:
    //     dpre 6.6 and 7.3; but 27 x 11, 128 x 512: dxe, eight slabs, 7.6 and 7.1; 7 x 600, 320 x 1280: dpre 16.3 and 12.1).
    const long long tiles = (long long)g.N * ((g.Mrows + 127) / 128) * ((g.Nout + 127) / 128);   // of 128 x 128
    // With more than four tiles per CU, weight gradients of at most 256 expected rows take weight_gradient_kernel, which hides a tile's chain behind the
    // other workgroups of its CU.  us, dW2 / dW1, the better one of the ring and the two-stage kernel first: 16 experts x 125 rows, 768 x 3072
    // 22.4 / 22.4 -> 20.7 / 21.3; x 188 26.5 / 26.6 -> 25.4 / 25.4; x 256 32.7 / 34.1 -> 32.8 / 31.1; x 288 (not taken) 36.0 / 33.9 -> 34.9 / 35.7; x 375 (not
    // taken) 43.4 / 42.4 -> 45.3 / 47.4; 64 experts x 140 rows 117 / 116 -> 108 / 108; x 256, 1024 x 4096 264 / 274 -> 252 / 246; 48 x 188, 1600 x 6400
    // 383 / 383 -> 362 / 368; 256 skewed experts, 1024 x 4096 650 / 662 -> 571 / 570; 128 x 234, 256 x 768 26.4 / 26.4 -> 27.8 / 24.9.  With fewer tiles nothing
    // hides the chain: 32 x 200, 256 x 1024 (512 tiles) 8.0 / 7.9 -> 8.7 / 8.5; 21 x 238, 192 x 576 6.0 / 6.1 -> 6.5 / 6.5.
    const bool short_sums = g.x_transposed && g.tune.tgemm_tile < 0 && tiles > 4LL * (g.tune.cus > 0 ? g.tune.cus : 256) &&
                            std::min(g.k_valid ? expected : INT_MAX, g.K) <= 256;
    const bool small = g.x_transposed ? short_sums || std::min(g.k_valid ? expected : INT_MAX, g.K) <= (wide ? 192 : 320)
                                      : (g.Mrows <= 64 && g.K < 512 && tiles <= 2 * g.tune.cus) || (g.K <= 256 && tiles <= g.tune.cus);
    if ((g.tune.tgemm_tile > 0 || (g.tune.tgemm_tile < 0 && !small)) && ring_applies(a, g.Mrows, g.x_transposed, true))
        return launch_ring_gradient(dtype, a, g.x_transposed, g.post, tile, g.tune, s);
    if (dtype == SMILE_DTYPE_BF16) return launch_typed<__bf16>(g, wide, short_sums, s);
    return launch_typed<_Float16>(g, wide, short_sums, s);
}

}  // namespace smile
