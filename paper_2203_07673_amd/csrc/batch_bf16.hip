// Batched persistent kernels, bfloat16 storage (float32 accumulation and outputs), with a
// float32 or a bfloat16 upstream gradient.
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

template <> BatchKernelFn batch_kernel_for<bf16_t, float>(int L, int rw, int cw, bool rows)
{
    switch (L) {
    case 4: return rows ? pick<bf16_t, float, 4, true>(rw, cw) : pick<bf16_t, float, 4, false>(rw, cw);
    case 8: return rows ? pick<bf16_t, float, 8, true>(rw, cw) : pick<bf16_t, float, 8, false>(rw, cw);
    case 16: return rows ? pick<bf16_t, float, 16, true>(rw, cw) : pick<bf16_t, float, 16, false>(rw, cw);
    case 32: return rows ? pick<bf16_t, float, 32, true>(rw, cw) : pick<bf16_t, float, 32, false>(rw, cw);
    case 64: return rows ? pick<bf16_t, float, 64, true>(rw, cw) : pick<bf16_t, float, 64, false>(rw, cw);
    default: return nullptr;
    }
}

template <> BatchKernelFn batch_kernel_for<bf16_t, bf16_t>(int L, int rw, int cw, bool rows)
{
    switch (L) {
    case 4: return rows ? pick<bf16_t, bf16_t, 4, true>(rw, cw) : pick<bf16_t, bf16_t, 4, false>(rw, cw);
    case 8: return rows ? pick<bf16_t, bf16_t, 8, true>(rw, cw) : pick<bf16_t, bf16_t, 8, false>(rw, cw);
    case 16: return rows ? pick<bf16_t, bf16_t, 16, true>(rw, cw) : pick<bf16_t, bf16_t, 16, false>(rw, cw);
    case 32: return rows ? pick<bf16_t, bf16_t, 32, true>(rw, cw) : pick<bf16_t, bf16_t, 32, false>(rw, cw);
    case 64: return rows ? pick<bf16_t, bf16_t, 64, true>(rw, cw) : pick<bf16_t, bf16_t, 64, false>(rw, cw);
    default: return nullptr;
    }
}

template <> BatchQueueKernelFn batch_queue_kernel_for<bf16_t, float>(int L, int rw, int cw, bool rows)
{
    switch (L) {
    case 4: return rows ? pick_queue<bf16_t, float, 4, true>(rw, cw) : pick_queue<bf16_t, float, 4, false>(rw, cw);
    case 8: return rows ? pick_queue<bf16_t, float, 8, true>(rw, cw) : pick_queue<bf16_t, float, 8, false>(rw, cw);
    case 16: return rows ? pick_queue<bf16_t, float, 16, true>(rw, cw) : pick_queue<bf16_t, float, 16, false>(rw, cw);
    case 32: return rows ? pick_queue<bf16_t, float, 32, true>(rw, cw) : pick_queue<bf16_t, float, 32, false>(rw, cw);
    case 64: return rows ? pick_queue<bf16_t, float, 64, true>(rw, cw) : pick_queue<bf16_t, float, 64, false>(rw, cw);
    default: return nullptr;
    }
}

template <> BatchQueueKernelFn batch_queue_kernel_for<bf16_t, bf16_t>(int L, int rw, int cw, bool rows)
{
    switch (L) {
    case 4: return rows ? pick_queue<bf16_t, bf16_t, 4, true>(rw, cw) : pick_queue<bf16_t, bf16_t, 4, false>(rw, cw);
    case 8: return rows ? pick_queue<bf16_t, bf16_t, 8, true>(rw, cw) : pick_queue<bf16_t, bf16_t, 8, false>(rw, cw);
    case 16: return rows ? pick_queue<bf16_t, bf16_t, 16, true>(rw, cw) : pick_queue<bf16_t, bf16_t, 16, false>(rw, cw);
    case 32: return rows ? pick_queue<bf16_t, bf16_t, 32, true>(rw, cw) : pick_queue<bf16_t, bf16_t, 32, false>(rw, cw);
    case 64: return rows ? pick_queue<bf16_t, bf16_t, 64, true>(rw, cw) : pick_queue<bf16_t, bf16_t, 64, false>(rw, cw);
    default: return nullptr;
    }
}

}  // namespace fmm
