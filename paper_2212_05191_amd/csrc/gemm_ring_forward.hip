// Forward expert GEMMs on the ring kernel (gemm_ring.hpp): both operands K-contiguous.
#include "gemm_ring.hpp"

#include <algorithm>
#include <cmath>

namespace smile {

namespace {

template <typename E, int QA0, int QA1, int QB0, int QB1, int OCC>
hipError_t launch_shape(const RingArgs &a, int act, const Tuning &tune, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    if (a.y2) {
        if (act == 1) return launch_ring_kernel<E, QA0, QA1, QB0, QB1, OCC, false, false, 1, true, 0>(a, tune, s, t0, t1);
        return launch_ring_kernel<E, QA0, QA1, QB0, QB1, OCC, false, false, 3, true, 0>(a, tune, s, t0, t1);
    }
    if (act == 0) return launch_ring_kernel<E, QA0, QA1, QB0, QB1, OCC, false, false, 0, false, 0>(a, tune, s, t0, t1);
    if (act == 1) return launch_ring_kernel<E, QA0, QA1, QB0, QB1, OCC, false, false, 1, false, 0>(a, tune, s, t0, t1);
    return launch_ring_kernel<E, QA0, QA1, QB0, QB1, OCC, false, false, 3, false, 0>(a, tune, s, t0, t1);
}

template <typename E>
hipError_t launch_typed(const RingArgs &a, int act, RingTile tile, const Tuning &tune, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    switch (tile) {
    case kRing128x192x2: return launch_shape<E, 1, 1, 1, 2, 2>(a, act, tune, s, t0, t1);
    case kRing128x256: return launch_shape<E, 1, 1, 2, 2, 1>(a, act, tune, s, t0, t1);
    case kRing256x192: return launch_shape<E, 2, 2, 1, 2, 1>(a, act, tune, s, t0, t1);
    case kRing128x128x2: return launch_shape<E, 1, 1, 1, 1, 2>(a, act, tune, s, t0, t1);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool ring_applies(const RingArgs &a, long long x_rows, bool x_transposed, bool w_transposed)
{
    const long long limit = 1ll << 31;   // elements of two bytes
    const long long x = x_transposed ? 64ll * a.ldx + a.Mrows : x_rows * a.ldx;
    const long long w = w_transposed ? 64ll * a.ldw + a.Nout : (long long)a.Nout * a.ldw;
    return (x_transposed || a.K >= 192) && x < limit && w < limit;
}

// Tile shapes.  With tiles for many rounds of the chip, measured on the forward passes and training steps of the bf16 workloads (us per pass,
// the other GEMMs unchanged):
//   * short contractions (Nout >= K: up-projection, dpre) and the weight gradients: 128 x 192, two on a CU, so that one tile's epilogue
//     overlaps the other's contraction (up, 64 experts 1024 -> 4096: 443; 128 x 256 alone on a CU 457, 256 x 192 506; dW of
//     1600 x 6400: 1611 against 1666 and 1643).  Outputs that 192-wide tiles would pad by more than a quarter over 128-wide ones (up to
//     128, 193 .. 256 columns, ...): 128 x 128;
//   * long contractions where 192-wide tiles pad by more than a tenth (1024 columns): 128 x 128 forward (64 experts x 256 rows,
//     4096 -> 1024: 437; 128 x 256 443, 128 x 192 449), 128 x 256 for dxe, whose transposed operand makes narrow tiles dearer
//     (256 skewed experts: 3514 against 3531), unless that pads by more than a fifth;
//   * else 256 x 192 where buffers are expected to be full, so that one tile takes all rows of an expert and its weights cross L2 once
//     (128 experts x 256 rows, 3072 -> 768: 441; 128 x 256 451, 128 x 192 455), and 128 x 256 where their fill varies and a second
//     row tile would be nearly empty (16 experts x 512 rows in buffers of 1024, 6400 -> 1600: dxe 1486; 128 x 192 1507, 256 x 192 1511).
// Up to three rounds the last one decides: another shape is taken where this one needs 15 % longer by the estimate rounds x time of a
// round, whose weights are what a CU multiplies in a round.  Measured on 800 products of 4 to 256 experts, 8 to 2700 rows, 128 x 512 to
// 1600 x 6400 (us per kernel): down, 16 experts x 144 rows, 6400 -> 1600: 224 tiles of 128 x 256 117, 288 of 128 x 192 154; 21 x 144: 360
// of 128 x 192 in one round 166, 281 of 128 x 256 in two 214; dxe, 64 x 240, 1280 -> 320: 384 of 128 x 128 25, 256 of 128 x 256, which pad by a
// third, 44; dpre, 16 x 128, 1024 -> 4096: one round of 512 of 128 x 128 37, 352 of 128 x 192 46; up, 64 x 96, 256 -> 1024: 16.4 and 19.7.
// `rows`: tokens per group if they spread evenly.
namespace {

struct RingShape {
    int rows, cols, per_cu;   // tile, workgroups on a CU
    double weight;            // time of a round
};
constexpr RingShape kShapes[kRingTiles] = {{128, 192, 2, 1.5}, {128, 256, 1, 1.0}, {256, 192, 1, 1.25}, {128, 128, 2, 1.0}};

// Row tiles of a group on the average of a random assignment of `rows` tokens to each: one, and one more for every boundary between tiles,
// weighted with the chance (normal with the variance `rows`) that the group's count passes it
double expected_row_tiles(const RingArgs &a, int rows, int tile_rows)
{
    if (rows >= a.Mrows) return (double)(((long long)a.Mrows + tile_rows - 1) / tile_rows);
    const double sd = std::sqrt((double)rows);
    const long long sure = std::max(0ll, (long long)std::floor((rows - 4.0 * sd) / tile_rows));   // boundaries that every group passes
    double n = 1.0 + sure;
    for (long long edge = (sure + 1) * tile_rows; edge < a.Mrows && edge < rows + 4.0 * sd; edge += tile_rows)
        n += 0.5 * std::erfc((edge - rows) / (sd * std::sqrt(2.0)));
    return n;
}

double rounds(const Tuning &tune, const RingArgs &a, int rows, RingTile tile)
{
    const RingShape &s = kShapes[tile];
    return a.N * expected_row_tiles(a, rows, s.rows) * ((a.Nout + s.cols - 1) / s.cols) / ((double)tune.cus * s.per_cu);
}

double estimated_time(const Tuning &tune, const RingArgs &a, int rows, RingTile tile)
{
    const int per_cu = kShapes[tile].per_cu;
    double n = rounds(tune, a, rows, tile);
    if (n > (per_cu == 2 ? 2.0 : 3.0)) {
        n += 0.25;   // by now workgroups are out of step and share the last round
    } else if (per_cu == 2) {
        const double tiles_of_cu = std::ceil(2.0 * n), pairs = std::floor(tiles_of_cu / 2.0);
        n = tiles_of_cu > 2.0 * pairs ? pairs + 0.55 : pairs;   // a workgroup alone on its CU takes little more than half of two
    } else {
        n = std::ceil(n);
    }
    return kShapes[tile].weight * n;
}

}  // namespace

RingTile pick_ring_tile(const Tuning &tune, const RingArgs &a, int rows, bool gradient)
{
    auto padded = [&](int width) { return ((long long)a.Nout + width - 1) / width * width; };
    const bool is_short = a.Nout >= a.K || a.k_valid;
    RingTile best;
    if (is_short) best = padded(192) * 4 > padded(128) * 5 ? kRing128x128x2 : kRing128x192x2;
    else if (padded(192) * 10 > padded(128) * 11)
        best = gradient && padded(256) * 10 <= padded(128) * 12 ? kRing128x256 : kRing128x128x2;
    else best = rows >= a.Mrows && a.Mrows > 128 ? kRing256x192 : kRing128x256;
    if (rounds(tune, a, rows, best) > 3.0) {
        // Where a second 256-row tile is filled to a third at most, three row tiles of 128 x 256 pad less, if three of them side by side cover the
        // columns of four of 256 x 192 (us: down, 128 experts x 300 rows, 3072 -> 768 271 -> 264, x 320 291 -> 263; 1536 columns: 128 x 300 572 -> 460, 80 x
        // 288 660 -> 573; dxe, 128 x 320, 768 columns 283 -> 244; skewed counts: 128 x 288, 768 columns 190 -> 178, 192 x 320 207 -> 220).  Fewer than 32
        // rows more than a tile cost little, and from 350 on three tiles cost what two do: 128 x 384, 768 columns, 264 and 281, skewed 128 x 368 156 and 171.
        // Other widths gain or lose by how their tiles fall: 960 columns 0.79 to 1.03, 576 1.08 to 1.22.
        const bool third = best == kRing256x192 && a.Mrows >= 288 && a.Mrows <= 336 && (a.Nout + 255) / 256 * 4 <= (a.Nout + 191) / 192 * 3;
        return third ? kRing128x256 : best;
    }
    double time = estimated_time(tune, a, rows, best) / 1.15;
    for (const RingTile t : {kRing128x128x2, kRing128x192x2, kRing128x256}) {
        if (is_short && t == kRing128x256) continue;
        const double other = estimated_time(tune, a, rows, t);
        if (other < time) time = other, best = t;
    }
    return best;
}

hipError_t launch_ring_forward(int dtype, const RingArgs &a, int act, RingTile tile, const Tuning &tune, hipStream_t s, hipEvent_t t0,
                               hipEvent_t t1)
{
    if (dtype == SMILE_DTYPE_BF16) return launch_typed<__bf16>(a, act, tile, tune, s, t0, t1);
    return launch_typed<_Float16>(a, act, tile, tune, s, t0, t1);
}

}  // namespace smile
