// Forward expert GEMMs on the ring kernel (gemm_ring.hpp): both operands K-contiguous.
#include "gemm_ring.hpp"

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

// Tile shapes, measured on the forward passes and training steps of the bf16 workloads (us per pass, the other GEMMs unchanged) and on
// small training steps (us per kernel):
//   * short contractions (Nout >= K: up-projection, dpre) and the weight gradients: 128 x 192, two on a CU, so that one tile's epilogue
//     overlaps the other's contraction (up, 64 experts 1024 -> 4096: 443; 128 x 256 alone on a CU 457, 256 x 192 506; dW of
//     1600 x 6400: 1611 against 1666 and 1643).  Outputs that 192-wide tiles would pad by more than a quarter over 128-wide ones (up to
//     128, 193 .. 256 columns, ...): 128 x 128.  So too where that leaves the chip few enough tiles: weight gradients with one per CU at
//     most (7 experts x 600 rows, 320 x 1280: 10.6 against 12.3; 11 x 251, 576 x 1728, three per CU: 12.0 against 10.4), others
//     with at most two, if 128 x 192 are at most one per CU and rows fill more than half of them (dpre of the two: 12.1 against 15.8, 14.4
//     against 17.8; 8 x 36 rows, 1152 x 4608: 21.2 against 18.5).
//   * long contractions, at most one 128 x 128 tile per CU: that (dxe of the three: 13.7 against 17.1 in 128 x 192, 17.2 against
//     20.9, 34.8 against 39.5); at most one 128 x 192: that (down, 16 experts x 512 rows, 3072 -> 768: 101; 128 x 256 102, 256 x 192 113; dxe
//     397, 128 x 128 409; down, 15 experts x 334 rows, 3840 -> 960: 125 against 134 and 134).
//   * else, where 192-wide tiles pad by more than a tenth (1024 columns): 128 x 128 forward (64 experts x 256 rows, 4096 -> 1024: 437; 128 x 256
//     443, 128 x 192 449), 128 x 256 for dxe, whose transposed operand makes narrow tiles dearer (256 skewed experts: 3514 against 3531).
//   * else 256 x 192 where buffers are expected to be full, so that one tile takes all rows of an expert and its weights cross L2 once
//     (128 experts x 256 rows, 3072 -> 768: 441; 128 x 256 451, 128 x 192 455), and 128 x 256 where their fill varies and a second
//     row tile would be nearly empty (16 experts x 512 rows in buffers of 1024, 6400 -> 1600: dxe 1486; 128 x 192 1507, 256 x 192 1511).
// `rows`: tokens per group if they spread evenly; with room in the buffers half a tile more is counted.
RingTile pick_ring_tile(const Tuning &tune, const RingArgs &a, int rows, bool gradient)
{
    auto padded = [&](int width) { return (a.Nout + width - 1) / width * width; };
    const double row_tiles = rows >= a.Mrows ? (a.Mrows + 127) / 128 : rows / 128.0 + 0.5;
    const double tiles128 = a.N * row_tiles * (padded(128) / 128), tiles192 = a.N * row_tiles * (padded(192) / 192);
    if (a.Nout >= a.K || a.k_valid) {
        const bool few = a.k_valid ? tiles128 <= tune.cus : tiles192 <= tune.cus && tiles128 <= 2 * tune.cus && a.Mrows > 64;
        return few || padded(192) * 4 > padded(128) * 5 ? kRing128x128x2 : kRing128x192x2;
    }
    if (tiles128 <= tune.cus) return kRing128x128x2;
    if (tiles192 <= tune.cus) return kRing128x192x2;
    if (padded(192) * 10 > padded(128) * 11) return gradient ? kRing128x256 : kRing128x128x2;
    return rows >= a.Mrows && a.Mrows > 128 ? kRing256x192 : kRing128x256;
}

hipError_t launch_ring_forward(int dtype, const RingArgs &a, int act, RingTile tile, const Tuning &tune, hipStream_t s, hipEvent_t t0,
                               hipEvent_t t1)
{
    if (dtype == SMILE_DTYPE_BF16) return launch_typed<__bf16>(a, act, tile, tune, s, t0, t1);
    return launch_typed<_Float16>(a, act, tile, tune, s, t0, t1);
}

}  // namespace smile
