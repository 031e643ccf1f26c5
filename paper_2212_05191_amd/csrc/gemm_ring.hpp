// Grouped 16-bit (bf16 / fp16) MFMA GEMM with a ring of operand units: y[e][i][j] = sum_k X(i,k) W(j,k) per group e, where either
// operand may be stored with the contraction index as its slow index ("transposed").  A workgroup of four waves computes
// 64*(QA0+QA1) x 64*(QB0+QB1) outputs at a time and walks the live tiles of the launch (LiveTileWalk); OCC of them share a CU.
//
// What bounds it and why this form.  The two-stage kernels (grouped_gemm_nt_kernel, grouped_gemm_t_kernel) request a K slab during the
// slab in front of it, so that less than one slab is in flight, while a weight line takes about 2 us from HBM under load.  Here:
//   * a slab (64 k) is four units: the rows of X that belong to the first and second half of every wave's blocks (A0, A1)
//     and the same of W (B0, B1).  A wave reads a whole unit into registers one phase before it multiplies with it, which frees the unit's
//     LDS slot one phase later.  The four products of a slab are its phases, in the order A0 B0, A0 B1, A1 B1, A1 B0, which leaves the
//     registers of A0 and of A1 free exactly when their next unit is due; B0 has a second set.  Slots are refilled in the
//     order of reading, two slabs ahead, so that 6 to 7 of the 8 slots are in flight at any time, at one barrier a phase;
//   * the stream of units runs on into the next tile, whose first seven units (four where the epilogue stages in the last
//     stage of the ring) are requested before this tile's epilogue;
//   * block q of a wave is at row q*64 + wm*32 of a unit, so that a tile whose rows end in A0 multiplies nothing with A1;
//   * the epilogue is private to a wave: 32 x 32 or 32 x 64 outputs pass through its own piece of LDS and leave as runs of 64 or 128 bytes.
// With 128 x 192 tiles, two on a CU, L2 -> LDS traffic reaches 18 TB/s during the contractions, its limit with 8 waves on a CU (18.7
// measured), and the set-up, GELU and stores of one tile hide behind the other's contraction; 128 x 256 and 256 x 192 alone on a CU move 10 and
// 30 % less, which wins where contractions are long (pick_ring_tile).  Every tile adds a row's products in the order of k: same bits.
// Measured against the two-stage kernels, whole passes, both sides in turn on one card, us: 64 experts 1024 x 4096 forward
// 467 -> 440, 128 experts 768 x 3072 487 -> 444, 15 experts x 334 rows 960 x 3840 fp16 159 -> 132, 16 experts 768 x 3072 training
// 423 -> 389, 1600 x 6400 training 1747 -> 1441.
//
// Operand tiles in LDS.  Normal: [row][64 k], piece c (16 bytes) of a row at c ^ ((row >> 1) & 7), MFMA fragments by one
// 16-byte read.  Transposed: as in memory, [64 k][columns], fragments by two transposing reads (ds_read_b64_tr_b16, see
// gemm_transposed.hip); the pieces of k-row k are rotated so that four successive k-rows fall on distinct banks: by 4 * (k & 3) in rows
// of 16 pieces (256 bytes), by 4 * ((k >> 1) & 1) in rows of 8.
//
// What the compiler's own waits undo: it cannot count loads across the loop over slabs, so a value loaded before the loop and used after it
// costs a wait for all loads, i.e. the whole ring.  Row indices, tokens and gates are requested early enough to have arrived (tokens and the
// next tile's row indices at the start of a tile, gates in the phase D = -7), but the forward kernels, which may gather or scatter, do wait
// for all that is in flight at D = -7, where the next tile's addresses are taken, and in front of the epilogue; the gradient kernels of
// a normal x do not.  128 x 192 tiles fill the 256 registers of two workgroups on a CU and spill: forward 2 (4 with GELU), weight gradients 10 (in the
// code for one and two slabs, too); what is reloaded at the start of a tile, of the walk, waits for its first units and the stores of the
// tile before.  The other shapes spill no vector register.  Contractions of one or two slabs, whose waits would cover nothing, have code of
// their own.
#pragma once

#include <type_traits>

#include "gemm_device.hpp"

namespace smile {

namespace {

// QA0, QA1 / QB0, QB1: 32-wide blocks per wave in the units A0, A1 / B0, B1.  XT, WT: operand stored transposed.
// ACT: activation of the epilogue; DUAL: the product without it to y2 as well; POST: times act'(aux).
template <typename E, int QA0, int QA1, int QB0, int QB1, int OCC, bool XT, bool WT, int ACT, bool DUAL, int POST>
__global__ __launch_bounds__(256, OCC) void grouped_gemm_ring_kernel(RingArgs a)
{
    typedef typename Half<E>::vec8 vec8;                               // one MFMA operand: 8 elements
    typedef __attribute__((__vector_size__(4 * sizeof(E)))) E vec4;    // 4 rounded outputs
    constexpr int NW = 4, BM = 64 * (QA0 + QA1), BN = 64 * (QB0 + QB1), TM = QA0 + QA1, TN = QB0 + QB1;
    enum { A0, B0, B1, A1 };
    constexpr int kExt[4] = {64 * QA0, 64 * QB0, 64 * QB1, 64 * QA1};   // rows (columns) of a unit
    constexpr int kOff[4] = {0, kExt[0] * 128, (kExt[0] + kExt[1]) * 128, (kExt[0] + kExt[1] + kExt[2]) * 128};
    constexpr int kCnt[8] = {2 * QA0, 2 * QB0, 2 * QB1, 2 * QA1, 2 * QA0, 2 * QB0, 2 * QB1, 2 * QA1};   // load instructions per wave
    constexpr int kFirst[4] = {0, kCnt[0], kCnt[0] + kCnt[1], kCnt[0] + kCnt[1] + kCnt[2]};
    constexpr int kFrags[4] = {4 * QA0, 4 * QB0, 4 * QB1, 4 * QA1};     // fragments per wave
    constexpr int GPW = 2 * (TM + TN), STAGE = (BM + BN) * 128;
    constexpr bool KRAGGED = XT && WT;   // the contraction length is the group's row count
    constexpr int SROW = (QB0 > QB1 ? QB0 : QB1) * 64 + 16;  // bytes of a staged row
    static_assert(QA0 <= 2 && QA1 <= 2 && QB0 <= 2 && QA0 >= 1 && QA1 >= 1 && QB1 >= 1, "units of 64 or 128 rows");

    constexpr bool SHARED = 2 * STAGE + NW * 32 * SROW + BM * 8 > kLdsPerCu / OCC;   // the epilogue stages in the tile's last stage
    __shared__ __attribute__((aligned(16))) char ring_lds[2 * STAGE + (SHARED ? 0 : NW * 32 * SROW + BM * 8)];
    lds_char *const lds = (lds_char *)ring_lds;

    LiveTileWalk<BM> walk;
    walk.init(a.rows_valid, a.N, a.Mrows, a.col_tiles, KRAGGED, a.backwards);
    struct Tile {
        int e, rt, ct, rows, kv;
    };
    auto select = [&](Tile &t) {
        if (!walk.tile(t.e, t.rt, t.ct, t.rows)) return false;
        t.kv = KRAGGED && a.k_valid ? min(a.k_valid[t.e], a.K) : a.K;
        return true;
    };
    // Per-lane indices are derived afresh wherever they are needed, from an opaque copy of the thread id, so that nothing
    // computed from them stays in registers from one part of a tile to the next.
    auto thread_id = [&]() {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    };
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave & 1, wn = wave >> 1;

    // ---- loader.  off: this lane's byte offset from the tile's operand (xb / wb, slab 0) in each load instruction of a slab
    uint32_t off[GPW];
    const char *xb = nullptr, *wb = nullptr;
    int kv = 0;   // contraction length of the tile whose units are being requested
    const size_t adv_x = 2 * (XT ? (size_t)64 * a.ldx : 64), adv_w = 2 * (WT ? (size_t)64 * a.ldw : 64);
    // (row or k-row, piece) that a lane fetches in instruction `inst` of a unit of EXT rows / columns
    auto place = [&](auto ext, auto transposed, int lane, int inst, int &r, int &piece) __attribute__((always_inline)) {
        constexpr int EXT = decltype(ext)::value;
        if constexpr (!decltype(transposed)::value) {
            r = inst * 8 + (lane >> 3);
            piece = (lane & 7) ^ ((r >> 1) & 7);
        } else {
            constexpr int P = EXT / 8;
            const int q = inst * 64 + lane;
            r = q / P;
            const int rot = P == 16 ? 4 * (r & 3) : 4 * ((r >> 1) & 1);
            piece = (q - r * P - rot) & (P - 1);
        }
    };
    // gathered operand: this lane's entries of x_rows for the tile to come, in the order of the load instructions of A0, A1
    int gathered[2 * TM];
    auto fetch_rows = [&](const Tile &t) __attribute__((always_inline)) {
        if constexpr (!XT && !WT) {
            if (a.x_rows) {
                const int32_t *x_rows = a.x_rows + (size_t)t.e * a.Mrows;
                const int lane = thread_id() & 63;
#pragma unroll
                for (int i = 0; i < 2 * TM; ++i) {
                    const int r = (i < kCnt[A0] ? (wave + i * NW) * 8 : kExt[A0] + (wave + (i - kCnt[A0]) * NW) * 8) + (lane >> 3);
                    gathered[i] = x_rows[min(t.rt * BM + r, t.rows - 1)];
                }
            }
        }
    };
    auto set_sources = [&](const Tile &t) __attribute__((always_inline)) {
        kv = t.kv;
        const bool gather = !XT && !WT && a.x_rows;
        xb = static_cast<const char *>(a.x) + (gather ? (size_t)0 : (size_t)t.e * a.sx * 2);
        wb = static_cast<const char *>(a.w) + (size_t)t.e * a.sw * 2;
        const int lane = thread_id() & 63;
        for_constants<4>([&](auto type) {
            constexpr int T = decltype(type)::value;
            constexpr bool IS_X = T == A0 || T == A1, TR = IS_X ? XT : WT;
            const int first = IS_X ? t.rt * BM + (T == A1 ? kExt[A0] : 0) : t.ct * BN + (T == B1 ? kExt[B0] : 0);
            const uint32_t ld = IS_X ? a.ldx : a.ldw;
#pragma unroll
            for (int i = 0; i < kCnt[T]; ++i) {
                int r, piece;
                place(std::integral_constant<int, kExt[T]>{}, std::integral_constant<bool, TR>{}, lane, wave + i * NW, r, piece);
                if constexpr (TR) {
                    const int ext = IS_X ? a.Mrows : a.Nout;   // columns beyond the matrix re-read its last ones
                    off[kFirst[T] + i] = 2 * ((uint32_t)r * ld + min(first + piece * 8, ext - 8));
                } else {
                    const int ext = IS_X ? t.rows : a.Nout;    // rows beyond the last valid one re-read it
                    int row = min(first + r, ext - 1);
                    if constexpr (IS_X && !WT) {
                        if (gather) row = gathered[(T == A1 ? kCnt[A0] : 0) + i];
                    }
                    off[kFirst[T] + i] = 2 * ((uint32_t)row * ld + piece * 8);
                }
            }
        });
    };
    // load instruction i of unit `type` of slab `slab`, into the stage `stage` bytes into LDS.  LAST: it may be the last slab.
    auto load_one = [&](auto type, auto last, int i, int slab, int stage) __attribute__((always_inline)) {
        constexpr int T = decltype(type)::value;
        constexpr bool IS_X = T == A0 || T == A1;
        const char *base = (IS_X ? xb : wb) + (size_t)slab * (IS_X ? adv_x : adv_w);
        uint32_t o = off[kFirst[T] + i];
        asm volatile("" : "+v"(o));   // scalar base + 32-bit offset, not a 64-bit sum kept per lane
        const auto to = SMILE_LPTR(lds + stage + kOff[T] + (wave + i * NW) * 1024);
        if constexpr (KRAGGED && decltype(last)::value) {   // k-rows beyond the contraction length are zero
            constexpr int P = kExt[T] / 8;
            const char *p = slab * 64 + (wave + i * NW) * (64 / P) + (int)(thread_id() & 63) / P < kv ? base + o : reinterpret_cast<const char *>(kZeroPiece);
            __builtin_amdgcn_global_load_lds(SMILE_GPTR(p), to, 16, 0, 0);
            return;
        }
        __builtin_amdgcn_global_load_lds(SMILE_GPTR(base + o), to, 16, 0, 0);
    };
    auto load_unit = [&](auto type, int slab, int stage) __attribute__((always_inline)) {
        for_constants<kCnt[decltype(type)::value]>([&](auto i) { load_one(type, std::true_type{}, decltype(i)::value, slab, stage); });
    };
    // units FROM .. TO - 1 of a tile whose first slab lies in `stage`, as far as it has them
    auto load_first = [&](auto from, auto to, int units, int stage) __attribute__((always_inline)) {
        for_constants<7>([&](auto v) {
            constexpr int V = decltype(v)::value;
            if (V >= decltype(from)::value && V < decltype(to)::value && V < units) load_unit(std::integral_constant<int, V & 3>{}, V / 4, V < 4 ? stage : STAGE - stage);
        });
    };
    auto load_bias = [&](const Tile &t, vec4 (&b)[TN][4]) {
        const E *bias = static_cast<const E *>(a.bias) + (size_t)t.e * a.Nout;
        const int fhi = (thread_id() >> 5) & 1;
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = t.ct * BN + (i < QB0 ? wn * QB0 * 32 + i * 32 : kExt[B0] + wn * QB1 * 32 + (i - QB0) * 32) + 8 * q + 4 * fhi;
                b[i][q] = *reinterpret_cast<const vec4 *>(bias + min(col, a.Nout - 4));
            }
    };

    Tile cur;
    if (!select(cur)) return;
    fetch_rows(cur);
    set_sources(cur);
    int stage0 = 0;   // where the tile's slab 0 lies in LDS (0 or STAGE)
    load_first(std::integral_constant<int, 0>{}, std::integral_constant<int, 7>{}, 4 * ((cur.kv + 63) / 64), stage0);
    vec4 bias_regs[TN][4];
    if (a.bias) load_bias(cur, bias_regs);

    for (;;) {
    const int S = (cur.kv + 63) / 64;
    walk.advance();
    Tile nxt;
    const bool more = select(nxt);
    const int next_units = more ? 4 * ((nxt.kv + 63) / 64) : 0;
    const bool full = next_units >= 7 && S >= 3;   // the next tile's first seven units follow this tile's without a gap
    if (more) fetch_rows(nxt);
    const bool scatter = !XT && !WT && a.y_rows;
    const bool upper = cur.rows - cur.rt * BM > kExt[A0];   // rows in A1
    int token = 0;     // of row tid of the tile, and its gate (scatter)
    float gate = 0.f;
    if constexpr (!XT && !WT) {
        if (scatter) token = a.y_rows[(size_t)cur.e * a.Mrows + min(cur.rt * BM + thread_id() % BM, cur.rows - 1)];
    }

    // ---- fragment addressing: byte offsets of this lane in stage 0
    const int tid = thread_id(), lane = tid & 63, frow = lane & 31, fhi = lane >> 5;
    const int tj = (lane >> 2) & 3, tk0 = 8 * fhi + tj;             // transposed: k-row and column of the first read
    const int tcol = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    // normal: block q of A at row q*64 + wm*32, of B at wn*QB*32 + q*32; fragment kk at piece (2 kk + fhi) ^ swizzle
    int noff[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) noff[kk] = frow * 128 + (((2 * kk + fhi) ^ ((frow >> 1) & 7)) * 16);
    vec8 fa0[QA0][4], fa1[QA1][4], fb0[QB0][4], fb1[QB1][4], fb0n[QB0][4];   // fb0n: B0 of the next slab
    auto read_one = [&](auto type, auto index, const lds_char *stage) __attribute__((always_inline)) {   // fragment `index` = kk * Q + q
        constexpr int T = decltype(type)::value, Q = T == A0 ? QA0 : T == A1 ? QA1 : T == B0 ? QB0 : QB1;
        constexpr bool IS_X = T == A0 || T == A1, TR = IS_X ? XT : WT;
        constexpr int KK = decltype(index)::value / Q, q = decltype(index)::value % Q;
        const int first = IS_X ? wm * 32 + q * 64 : wn * Q * 32 + q * 32;
        vec8 v;
        if constexpr (!TR) {
            v = *(const __attribute__((address_space(3))) vec8 *)(stage + kOff[T] + first * 128 + noff[KK]);
        } else {
            constexpr int P = kExt[T] / 8, PITCH = P * 16;
            const int col = first + tcol;
            const int rot = P == 16 ? 4 * tj : 4 * ((tj >> 1) & 1);   // k-rows tk0 + 4 n: the same k & 3
            const lds_char *at = stage + kOff[T] + tk0 * PITCH + (((col >> 3) + rot) & (P - 1)) * 16 + (col & 4) * 2;
            read_transposed<4 * PITCH>(v, at + KK * 16 * PITCH);
        }
        if constexpr (T == A0) fa0[q][KK] = v;
        else if constexpr (T == A1) fa1[q][KK] = v;
        else if constexpr (T == B0) fb0n[q][KK] = v;
        else fb1[q][KK] = v;
    };

    f32x16 acc[TN][TM];
    if (a.bias) {
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = (float)bias_regs[i][v / 4][v % 4];
    } else {
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    }

    // Phase f: waits for unit f (every wave is then also done reading unit f - 1, whose slot is free), reads it, requests the
    // unit seven places on and multiplies fragments JA, JB (0 / 1; -1: none).  Unit f is of type f mod 4; D = f - U (U units in the
    // tile), or -32 in the steady state.  Behind unit f six units have been requested when it is waited for: of this tile, then of
    // the next one (unit v in phase U - 7 + v) if `full`.  from, to: stages of unit f and of unit f + 7; slab7: its slab.
    constexpr auto behind = [](int type, int n) {   // load instructions of the n units after one of type `type`
        int c = 0;
        for (int i = 1; i <= n; ++i) c += kCnt[(type + i) & 3];
        return c;
    };
    constexpr int AHEAD = SHARED ? 4 : 7;   // units of the next tile requested before the epilogue
    auto phase = [&](auto ja, auto jb, auto type, auto d, auto follow, int from, int slab7, int to) __attribute__((always_inline)) {
        constexpr int JA = decltype(ja)::value, JB = decltype(jb)::value, RT = decltype(type)::value, D = decltype(d)::value;
        constexpr int LT = (RT + 3) & 3;
        // in the steady state unit f + 7 is of slab s + 2 of S >= s + 4, or A0 of slab s + 3 (three slabs: B0 of the last)
        const std::integral_constant<bool, D != -32 || LT == A0 || JA == -1> last{};
        const bool next_follows = decltype(follow)::value && full;
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave's reads of unit f - 1
        if constexpr (D <= -7) wait_vmcnt<behind(RT, 6)>();
        else if constexpr (D < 0) {
            if (next_follows) wait_vmcnt<behind(RT, -1 - D) + behind(3, min_int(D + 7, AHEAD))>();
            else wait_vmcnt<behind(RT, -1 - D)>();
        }
        if constexpr (D < 1) __builtin_amdgcn_s_barrier();
        if constexpr (D >= -7 && D < AHEAD - 7) {
            if constexpr (D == -7 && !XT && !WT) {
                if (scatter) gate = a.gate[token];
            }
            if (next_follows) {
                if constexpr (D == -7) set_sources(nxt);
                load_unit(std::integral_constant<int, LT>{}, (D + 7) / 4, to);
            }
        }
        constexpr int QA = JA < 0 ? 0 : JA == 0 ? QA0 : QA1, QB = JB < 0 ? 0 : JB == 0 ? QB0 : QB1;
        constexpr int NM = QA * QB * 4, NR = D >= 0 ? 0 : kFrags[RT], NL = D < -7 ? kCnt[LT] : 0;
        // the stage read and the stage filled do not overlap (see gemm_transposed.hip on restrict)
        auto body = [&](auto with, const lds_char *__restrict stage) __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NM == 0 || !decltype(with)::value) {
                for_constants<NL>([&](auto l) { load_one(std::integral_constant<int, LT>{}, last, decltype(l)::value, slab7, to); });
                for_constants<NR>([&](auto r) { read_one(std::integral_constant<int, RT>{}, r, stage); });
            } else {
                // reads in the first half of the MFMAs, so that the others cover their latency; loads spread over all (pinned order)
                constexpr int RPM = NM ? (2 * NR + NM - 1) / NM : 0;
                for_constants<NM>([&](auto m) {
                    constexpr int M = decltype(m)::value, KK = M / (QA * QB), q = M % (QA * QB), i = q / QA, j = q % QA;
                    constexpr int ai = (JB == 0 ? 0 : QB0) + i, aj = (JA == 0 ? 0 : QA0) + j;
                    vec8 wv, xv;
                    if constexpr (JB == 0) wv = fb0[i][KK];
                    else wv = fb1[i][KK];
                    if constexpr (JA == 0) xv = fa0[j][KK];
                    else xv = fa1[j][KK];
                    acc[ai][aj] = Half<E>::mfma_32x32x16(wv, xv, acc[ai][aj]);
                    constexpr int R0 = min_int(NR, RPM * M), R1 = min_int(NR, RPM * (M + 1));
                    for_constants<R1 - R0>([&](auto r) { read_one(std::integral_constant<int, RT>{}, std::integral_constant<int, R0 + decltype(r)::value>{}, stage); });
                    constexpr int L0 = NL * M / NM, L1 = NL * (M + 1) / NM;
                    for_constants<L1 - L0>([&](auto l) { load_one(std::integral_constant<int, LT>{}, last, L0 + decltype(l)::value, slab7, to); });
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
        };
        if constexpr (JA == 1 && !KRAGGED) {   // nothing to multiply where the tile's rows all lie in A0
            if (upper) body(std::true_type{}, lds + from);
            else body(std::false_type{}, lds + from);
        } else {
            body(std::true_type{}, lds + from);
        }
    };
    auto take_b0 = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < QB0; ++q)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) fb0[q][kk] = fb0n[q][kk];
    };
#define SMILE_IC(v) std::integral_constant<int, (v)>{}
    // The four phases 4 s + 2 .. 4 s + 5 of slab s, which lies in `stage`; D of the first of them, or -32.  Units f + 7 of the first
    // three are of slab s + 2 (same stage), of the last of slab s + 3.
    auto slab = [&](auto d, auto follow, int s, int stage) __attribute__((always_inline)) {
        constexpr int D = decltype(d)::value, N1 = D == -32 ? 0 : 1;
        phase(SMILE_IC(0), SMILE_IC(0), SMILE_IC(B1), SMILE_IC(D), follow, stage, s + 2, stage);
        phase(SMILE_IC(0), SMILE_IC(1), SMILE_IC(A1), SMILE_IC(D + N1), follow, stage, s + 2, stage);
        phase(SMILE_IC(1), SMILE_IC(1), SMILE_IC(A0), SMILE_IC(D + 2 * N1), follow, STAGE - stage, s + 2, stage);
        phase(SMILE_IC(1), SMILE_IC(0), SMILE_IC(B0), SMILE_IC(D + 3 * N1), follow, STAGE - stage, s + 3, STAGE - stage);
        take_b0();
    };
    const std::integral_constant<int, -1> none{};
    if (!KRAGGED || S >= 3) {   // (whole contraction lengths: three slabs or more, by the rule of the dispatch)
        const std::true_type follow{};
        phase(none, none, SMILE_IC(A0), SMILE_IC(-32), follow, stage0, 1, STAGE - stage0);
        phase(none, none, SMILE_IC(B0), SMILE_IC(-32), follow, stage0, 2, stage0);
        take_b0();
        int s = 0, stage = stage0;
        for (; s + 3 < S; ++s, stage = STAGE - stage) slab(SMILE_IC(-32), follow, s, stage);
        slab(SMILE_IC(-10), follow, s, stage);
        slab(SMILE_IC(-6), follow, s + 1, STAGE - stage);
        slab(SMILE_IC(-2), follow, s + 2, stage);
        stage0 = STAGE - stage;   // the next tile's slabs follow
    } else if (S > 0) {
        // one or two slabs: nothing of the next tile is requested in between, and what the wait counts of longer tiles rest
        // on does not pass through here
        const std::false_type follow{};
        if (S == 2) {
            phase(none, none, SMILE_IC(A0), SMILE_IC(-8), follow, stage0, 1, STAGE - stage0);
            phase(none, none, SMILE_IC(B0), SMILE_IC(-7), follow, stage0, 0, stage0);
            take_b0();
            slab(SMILE_IC(-6), follow, 0, stage0);
            slab(SMILE_IC(-2), follow, 1, STAGE - stage0);
        } else {
            phase(none, none, SMILE_IC(A0), SMILE_IC(-4), follow, stage0, 0, 0);
            phase(none, none, SMILE_IC(B0), SMILE_IC(-3), follow, stage0, 0, 0);
            take_b0();
            slab(SMILE_IC(-2), follow, 0, stage0);
            stage0 = STAGE - stage0;
        }
    }
#undef SMILE_IC
    if (more) {
        if (!full) {   // its first units all at once; their slots were last read two phases and a barrier ago
            set_sources(nxt);
            load_first(std::integral_constant<int, 0>{}, std::integral_constant<int, AHEAD>{}, next_units, stage0);
        }
        if (a.bias) load_bias(nxt, bias_regs);
    }

    // ---- epilogue.  Accumulator element v of a lane is (column 8*(v/4) + 4*(lane/32) + v%4, row lane%32) of its 32 x 32
    // block: rounded, staged as [32 rows][QB * 32 columns], stored row-contiguously.
    const int e = cur.e, rows = cur.rows, Nout = a.Nout;
    const int otid = thread_id(), olane = otid & 63;
    lds_char *const staging = lds + (SHARED ? STAGE - stage0 : 2 * STAGE);
    lds_char *const stg = staging + wave * 32 * SROW;
    lds_char *const meta = staging + NW * 32 * SROW;   // [BM] token, [BM] gate of the tile's rows (scatter)
    E *Y = a.y ? static_cast<E *>(a.y) + (size_t)e * a.sy : nullptr;
    if (scatter) {
        if (otid < BM) {
            *(__attribute__((address_space(3))) int *)(meta + otid * 4) = token;
            *(__attribute__((address_space(3))) float *)(meta + BM * 4 + otid * 4) = gate;
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
    }
    for_constants<TM>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        const int row0 = (j < QA0 ? j * 64 : kExt[A0] + (j - QA0) * 64) + wm * 32;   // inside the tile
        if (cur.rt * BM + row0 >= rows) return;
        // The second factor of the row block is requested before anything of it is staged: one wait in place of two (dpre, us: 128 experts 768 x 3072
        // 266 -> 260, 1600 x 6400 224 -> 220, 16 experts 768 x 3072 63.3 -> 61.9; for the whole tile at once it spills).  Pieces of part 0, then of 1.
        u32x4 aux[POST != 0 ? 2 * TN : 1];
        if constexpr (POST != 0) {
            for_constants<2>([&](auto part) {
                constexpr int H = decltype(part)::value, P = (H == 0 ? QB0 : QB1) * 4;
                const int col0 = cur.ct * BN + (H == 0 ? wn * QB0 * 32 : kExt[B0] + wn * QB1 * 32);
#pragma unroll
                for (int it = 0; it < P / 2; ++it) {
                    const int id = it * 64 + olane, lrow = id / P, row = cur.rt * BM + row0 + lrow, col = col0 + (id - lrow * P) * 8;
                    aux[(H == 0 ? 0 : 2 * QB0) + it] = *reinterpret_cast<const u32x4 *>(
                        static_cast<const E *>(a.aux) + (size_t)e * a.sy + (size_t)min(row, rows - 1) * Nout + min(col, Nout - 8));
                }
            });
        }
        for_constants<2>([&](auto part) {
            constexpr int H = decltype(part)::value, QB = H == 0 ? QB0 : QB1, P = QB * 4, NIT = 32 * P / 64;
            const int col0 = cur.ct * BN + (H == 0 ? wn * QB0 * 32 : kExt[B0] + wn * QB1 * 32);
            if (col0 >= Nout) return;
            auto at = [&](int it, int &row, int &col, int &lrow) {   // piece it * 64 + olane of the staged block
                const int id = it * 64 + olane;
                lrow = id / P;
                row = cur.rt * BM + row0 + lrow, col = col0 + (id - lrow * P) * 8;
            };
#pragma unroll
            for (int pass = 0; pass < (DUAL ? 2 : 1); ++pass) {
#pragma unroll
                for (int i = 0; i < QB; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        vec4 out;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const float val = acc[(H == 0 ? 0 : QB0) + i][j][4 * q + v];
                            out[v] = (E)(pass == 0 ? activate<ACT>(val) : val);
                        }
                        *(__attribute__((address_space(3))) vec4 *)(stg + (olane & 31) * SROW + (i * 32 + 8 * q + 4 * (olane >> 5)) * 2) = out;
                    }
                u32x4 staged[NIT];
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    const int id = it * 64 + olane, lrow = id / P;
                    staged[it] = *(const __attribute__((address_space(3))) u32x4 *)(stg + lrow * SROW + (id - lrow * P) * 16);
                }
                E *dst = DUAL && pass == 1 ? static_cast<E *>(a.y2) + (size_t)e * a.sy : Y;
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
                    int row, col, lrow;
                    at(it, row, col, lrow);
                    if (row < rows && col < Nout) {
                        u32x4 v = staged[it];
                        if constexpr (POST != 0) {
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                v[k] = Half<E>::pack(Half<E>::lo(v[k]) * activate_grad<POST>(Half<E>::lo(aux[(H == 0 ? 0 : 2 * QB0) + it][k])),
                                                     Half<E>::hi(v[k]) * activate_grad<POST>(Half<E>::hi(aux[(H == 0 ? 0 : 2 * QB0) + it][k])));
                        }
                        if (dst) {
                            u32x4 *to = reinterpret_cast<u32x4 *>(dst + (size_t)row * Nout + col);
                            // weight gradients are not read again soon: keep them out of the way of the operands in L2
                            if constexpr (KRAGGED) __builtin_nontemporal_store(v, to);
                            else *to = v;
                        }
                        if (pass == 0 && scatter) {   // gate-weighted return to token order (Eq. 3)
                            const int tok = *(const __attribute__((address_space(3))) int *)(meta + (row0 + lrow) * 4);
                            const float g = *(const __attribute__((address_space(3))) float *)(meta + BM * 4 + (row0 + lrow) * 4);
                            // No kernel of the pass reads y again, so its rows pass the L2 by and leave it to w2 and h (128
                            // experts of 768 -> 3072, 32768 tokens: 437 -> 431 us a pass; 16 experts, 8192: 114.6 -> 113.8;
                            // the same at 64 experts of 1024 -> 4096, 429 us).  With a reader right behind (y + x): 465.3 -> 460.8,
                            // 117.1 -> 116.7, 459.2 -> 458.4; 2048 and 4096 tokens the same.
                            __builtin_nontemporal_store(scale_x8<E>(v, g), reinterpret_cast<u32x4 *>(static_cast<E *>(a.y_tok) + (size_t)tok * Nout + col));
                        }
                    }
                }
            }
        });
    });
    if (!more) return;
    if constexpr (SHARED) {   // every wave is done with the staging area
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        load_first(std::integral_constant<int, AHEAD>{}, std::integral_constant<int, 7>{}, next_units, stage0);
    }
    cur = nxt;
    }   // tile loop
}

template <typename E, int QA0, int QA1, int QB0, int QB1, int OCC, bool XT, bool WT, int ACT, bool DUAL, int POST>
hipError_t launch_ring_kernel(RingArgs a, const Tuning &tune, hipStream_t s, hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr)
{
    constexpr int BM = 64 * (QA0 + QA1), BN = 64 * (QB0 + QB1);
    a.col_tiles = (a.Nout + BN - 1) / BN;
    const long long tiles = (long long)a.N * ((a.Mrows + BM - 1) / BM) * a.col_tiles;
    const int slots = workgroup_slots(tune, OCC);
    const int grid = tiles < slots ? (int)((tiles + 7) / 8 * 8) : slots;
    const auto kernel = grouped_gemm_ring_kernel<E, QA0, QA1, QB0, QB1, OCC, XT, WT, ACT, DUAL, POST>;
    if (t0 && t1) hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, s, t0, t1, 0, a);
    else launch_kernel("grouped_gemm_ring_kernel", kernel, dim3(grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace

}  // namespace smile
