// Batched persistent kernels, float32 storage.
#include "batch_kernels.hpp"

namespace fmm {

template <class TS, class TD, int L, bool ROWS> static BatchKernelFn pick(int rw, int cw)
{
    constexpr int VW = 16 / (int)sizeof(TS);
    constexpr int W = 64 / L;
    if (!rw && !cw) return batch_kernel<TS, TD, L, VW, 1, 1, ROWS>;
    if (!rw && cw) return batch_kernel<TS, TD, L, VW, 1, W, ROWS>;
    if (rw && !cw) return batch_kernel<TS, TD, L, VW, W, 1, ROWS>;
    return batch_kernel<TS, TD, L, VW, W, W, ROWS>;
}

template <class TS, class TD, int L, bool ROWS> static BatchQueueKernelFn pick_queue(int rw, int cw)
{
    constexpr int VW = 16 / (int)sizeof(TS);
    constexpr int W = 64 / L;
    if (!rw && !cw) return batch_queue_kernel<TS, TD, L, VW, 1, 1, ROWS>;
    if (!rw && cw) return batch_queue_kernel<TS, TD, L, VW, 1, W, ROWS>;
    if (rw && !cw) return batch_queue_kernel<TS, TD, L, VW, W, 1, ROWS>;
    return batch_queue_kernel<TS, TD, L, VW, W, W, ROWS>;
}

template <> BatchKernelFn batch_kernel_for<float, float>(int L, int rw, int cw, bool rows)
{
    switch (L) {
    case 4: return rows ? pick<float, float, 4, true>(rw, cw) : pick<float, float, 4, false>(rw, cw);
    case 8: return rows ? pick<float, float, 8, true>(rw, cw) : pick<float, float, 8, false>(rw, cw);
    case 16: return rows ? pick<float, float, 16, true>(rw, cw) : pick<float, float, 16, false>(rw, cw);
    case 32: return rows ? pick<float, float, 32, true>(rw, cw) : pick<float, float, 32, false>(rw, cw);
    case 64: return rows ? pick<float, float, 64, true>(rw, cw) : pick<float, float, 64, false>(rw, cw);
    default: return nullptr;
    }
}

template <> BatchQueueKernelFn batch_queue_kernel_for<float, float>(int L, int rw, int cw, bool rows)
{
    switch (L) {
    case 4: return rows ? pick_queue<float, float, 4, true>(rw, cw) : pick_queue<float, float, 4, false>(rw, cw);
    case 8: return rows ? pick_queue<float, float, 8, true>(rw, cw) : pick_queue<float, float, 8, false>(rw, cw);
    case 16: return rows ? pick_queue<float, float, 16, true>(rw, cw) : pick_queue<float, float, 16, false>(rw, cw);
    case 32: return rows ? pick_queue<float, float, 32, true>(rw, cw) : pick_queue<float, float, 32, false>(rw, cw);
    case 64: return rows ? pick_queue<float, float, 64, true>(rw, cw) : pick_queue<float, float, 64, false>(rw, cw);
    default: return nullptr;
    }
}

}  // namespace fmm
