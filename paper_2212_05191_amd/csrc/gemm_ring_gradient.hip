// Gradient expert GEMMs on the ring kernel (gemm_ring.hpp): w, and for the weight gradients x too, transposed.
#include "gemm_ring.hpp"

namespace smile {

namespace {

template <typename E, int QA0, int QA1, int QB0, int QB1, int OCC>
hipError_t launch_shape(const RingArgs &a, bool x_transposed, int post, const Tuning &tune, hipStream_t s)
{
    if constexpr (OCC == 2) {   // weight gradients: contractions of a few slabs, never one workgroup on a CU
        if (x_transposed) return launch_ring_kernel<E, QA0, QA1, QB0, QB1, OCC, true, true, 0, false, 0>(a, tune, s);
    }
    if (post == 1) return launch_ring_kernel<E, QA0, QA1, QB0, QB1, OCC, false, true, 0, false, 1>(a, tune, s);
    if (post == 2) return launch_ring_kernel<E, QA0, QA1, QB0, QB1, OCC, false, true, 0, false, 2>(a, tune, s);
    return launch_ring_kernel<E, QA0, QA1, QB0, QB1, OCC, false, true, 0, false, 0>(a, tune, s);
}

template <typename E>
hipError_t launch_typed(const RingArgs &a, bool x_transposed, int post, RingTile tile, const Tuning &tune, hipStream_t s)
{
    if (x_transposed && tile != kRing128x128x2) tile = kRing128x192x2;
    switch (tile) {
    case kRing128x192x2: return launch_shape<E, 1, 1, 1, 2, 2>(a, x_transposed, post, tune, s);
    case kRing128x256: return launch_shape<E, 1, 1, 2, 2, 1>(a, x_transposed, post, tune, s);
    case kRing256x192: return launch_shape<E, 2, 2, 1, 2, 1>(a, x_transposed, post, tune, s);
    case kRing128x128x2: return launch_shape<E, 1, 1, 1, 1, 2>(a, x_transposed, post, tune, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_ring_gradient(int dtype, const RingArgs &a, bool x_transposed, int post, RingTile tile, const Tuning &tune, hipStream_t s)
{
    if (dtype == SMILE_DTYPE_BF16) return launch_typed<__bf16>(a, x_transposed, post, tile, tune, s);
    return launch_typed<_Float16>(a, x_transposed, post, tile, tune, s);
}

}  // namespace smile
