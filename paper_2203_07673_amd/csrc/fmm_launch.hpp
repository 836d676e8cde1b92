// Launcher for the line kernels: picks the compiled (L, NV, VW, U) variant for r,
// sizes the grid (chunk blocks first, then line blocks) and runs the merge of split
// lines.  Included only by the per-dtype instantiation units.
#pragma once

#include "fmm_internal.hpp"
#include "fmm_merge.hpp"

namespace fmm {

template <int OP> constexpr bool two_row() { return OP == OP_SPMM2 || OP == OP_FUSED2; }

// Entries loaded ahead per group: enough gathers in flight without spilling.  A lane
// holds U * NV vectors of 16 bytes per gathered matrix.
// Batch depth of class CLS (1 deep, 2 medium, 3 shallow): entries per batch for the
// one-row passes, half that for the two-row passes, divided by the vectors per lane.
template <int OP, int NV, int CLS> constexpr int unroll_for() {
    constexpr bool two = two_row<OP>();
    constexpr int one = CLS == 1 ? 8 : CLS == 2 ? 4 : 2;
    constexpr int u = (two ? one / 2 : one) / NV;
    return u < 1 ? 1 : u;
}

// Whether the chunks of split lines take a wave each (line_wave_kernel): where a group is less
// than a wave, for float32 sums (the gradient-check path keeps the one kernel), from 2^14
// chunks.  With fewer, chunks by groups are all resident at once and the extra waves only
// hold back the line blocks.  A training step on R-MAT, float32 at r = 64 unless named, a
// group / a wave per chunk in us: 3500 chunks 146 / 154, 6500 138 / 154 and (64 per row) 113 /
// 121, 7900 144 / 139, 10800 210 / 197, 11600 244 / 247, 16000 (r = 16) 201 / 212, 19800 414 /
// 394 and (bfloat16) 317 / 305, 24300 (r = 32) 186 / 181, 29500 311 / 302, 129000 (r = 32, 64
// per row) 825 / 745.
//
// A one-row pass by narrow groups needs chunks of full length besides: the groups of a wave
// load 64 / L batches of U entries at once, more than a short chunk holds.  2^17 lines of 150,
// chunks of 128 and 22, forward, group / wave: bfloat16 r = 16 257 / 333, r = 32 295 / 333, r = 64
// (with float32 dC) 379 / 423, r = 128 695 / 678, float32 r = 8 254 / 279; lines of 250, chunks of
// 128 and 122: bfloat16 r = 16 495 / 379, float32 r = 8 496 / 365.  Two-row passes gain either
// way (bfloat16 r = 16, 150: 615 / 560).
constexpr int32_t kWaveChunks = 1 << 14;
template <class Acc, int L> constexpr bool has_wave_kernel() { return L < 64 && sizeof(Acc) == 4; }
template <int OP, int L, int U> bool chunks_by_waves(const LineArgs &a)
{
    if (a.n_chunks < kWaveChunks) return false;
    if (two_row<OP>() || 64 / L * U <= 32) return true;
    return (double)a.nnz >= 0.75 * a.long_len * a.n_chunks;  // the entries bound the chunks' mean length
}

// Whether gather hints are followed: where a wave holds a row.  R-MAT scale 22, 16 per row,
// float32, in us without / with hints for 32 MB of rows: r = 256 (64 lanes) 9217 / 8973 forward,
// 17817 / 17574 column pass; scale 20, r = 512 4468 / 4265 and 9255 / 8919.  With fewer lanes a
// row the branch costs more than the kept rows give, in every pass: r = 128 5036 / 5144 and 9132 /
// 9183, r = 64 3066 / 3282 and 5315 / 5714, bfloat16 r = 256 5918 / 5980 and 13883 / 14083.
constexpr bool has_hints(int lanes) { return lanes == 64; }

template <int OP, class TH, class TG1, class TG2, class Acc, int L, int NV, int VW, int U, bool WAVE = false, bool HINT = false>
hipError_t launch_one(const LineArgs &a, hipStream_t stream)
{
    constexpr int GPB = kBlock / L;
    constexpr int CPB = WAVE ? kBlock / 64 : GPB;  // chunks per block
    const int64_t nb_chunk = a.n_chunks > 0 ? ((int64_t)a.n_chunks + CPB - 1) / CPB : 0;
    const int64_t nb_line = ((int64_t)a.nlines + GPB - 1) / GPB;
    const int64_t nb = nb_chunk + nb_line;
    if (nb == 0) return hipSuccess;
    if (nb > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    if constexpr (WAVE)
        hipLaunchKernelGGL((line_wave_kernel<OP, TH, TG1, TG2, Acc, L, NV, VW, U>), dim3((unsigned)nb), dim3(kBlock), 0,
                           stream, a, (int32_t)nb_chunk);
    else
        hipLaunchKernelGGL((line_kernel<OP, TH, TG1, TG2, Acc, L, NV, VW, U, HINT>), dim3((unsigned)nb), dim3(kBlock), 0,
                           stream, a, (int32_t)nb_chunk);
    return hipGetLastError();
}

template <int OP, class TH, class TG1, class TG2, class Acc, int L, int NV, int VW, int U>
hipError_t launch_kind(const LineArgs &a, hipStream_t stream)
{
    if constexpr (has_wave_kernel<Acc, L>() && !(VW == 1 && L == 32))  // small patterns, where groups are faster
        if (chunks_by_waves<OP, L, U>(a)) return launch_one<OP, TH, TG1, TG2, Acc, L, NV, VW, U, true>(a, stream);
    if constexpr (has_hints(L))
        if (a.hot) return launch_one<OP, TH, TG1, TG2, Acc, L, NV, VW, U, false, true>(a, stream);
    return launch_one<OP, TH, TG1, TG2, Acc, L, NV, VW, U>(a, stream);
}

#define FMM_SHAPE_CASE(Lv, NVv)                                                                  \
    if (shape.L == Lv && shape.NV == NVv) {                                                      \
        if (a.uclass == 1) return launch_kind<OP, TH, TG1, TG2, Acc, Lv, NVv, VW, unroll_for<OP, NVv, 1>()>(a, stream); \
        if (a.uclass == 2) return launch_kind<OP, TH, TG1, TG2, Acc, Lv, NVv, VW, unroll_for<OP, NVv, 2>()>(a, stream); \
        return launch_kind<OP, TH, TG1, TG2, Acc, Lv, NVv, VW, unroll_for<OP, NVv, 3>()>(a, stream);                    \
    }

template <int OP, class TH, class TG1, class TG2, class Acc, int VW>
hipError_t launch_shape(const LineArgs &a, Shape shape, hipStream_t stream)
{
    FMM_SHAPE_CASE(1, 1)
    FMM_SHAPE_CASE(2, 1)
    FMM_SHAPE_CASE(4, 1)
    FMM_SHAPE_CASE(8, 1)
    FMM_SHAPE_CASE(16, 1)
    // one element per lane: up to 16 of them, in float32 up to 64 (line_vectors)
    if constexpr (VW > 1 || sizeof(Acc) == 4) {
        FMM_SHAPE_CASE(32, 1)
        FMM_SHAPE_CASE(64, 1)
    }
    if constexpr (VW > 1) {
        FMM_SHAPE_CASE(16, 2)
        FMM_SHAPE_CASE(32, 2)
        FMM_SHAPE_CASE(64, 2)
        FMM_SHAPE_CASE(64, 4)
    }
    return hipErrorInvalidValue;
}
#undef FMM_SHAPE_CASE

// Smallest element size among the operands decides the vector width (16-byte loads).
template <class TH, class TG1, class TG2> constexpr int vector_width() {
    constexpr int a = (int)sizeof(TH), b = (int)sizeof(TG1), c = (int)sizeof(TG2);
    constexpr int mn = a < b ? (a < c ? a : c) : (b < c ? b : c);
    return 16 / mn;
}

template <int OP, class TH, class TG1, class TG2, class Acc>
hipError_t launch_lines(const LineArgs &a, int32_t n_splits, const int32_t *splits, Shape hint,
                        hipStream_t stream)
{
    constexpr int VWV = vector_width<TH, TG1, TG2>();
    constexpr bool has_bf16 = sizeof(TH) == 2 || sizeof(TG1) == 2 || sizeof(TG2) == 2;
    const int rows = two_row<OP>() ? 2 : OP == OP_FUSED1 || (OP == OP_SPMM1 && a.wperm) ? 1 : 0;
    const auto [vw, shape] = line_shape(a, rows, VWV, hint);
    if (!shape_supported(shape, a.r, vw)) return hipErrorInvalidValue;
    hipError_t e;
    if (vw > 1) {
        e = launch_shape<OP, TH, TG1, TG2, Acc, VWV>(a, shape, stream);
    } else {
        if constexpr (has_bf16) {
            return hipErrorInvalidValue;  // bfloat16 rows are whole vectors (r a multiple of 8)
        } else {
            e = launch_shape<OP, TH, TG1, TG2, Acc, 1>(a, shape, stream);
        }
    }
    if (e != hipSuccess) return e;
    if (OP != OP_SDDMM && n_splits > 0 && a.out != nullptr) {
        const Acc *partial = static_cast<const Acc *>(a.partial);
        if constexpr (has_bf16) {
            if (a.out16)
                return launch_merge<Acc>(splits, n_splits, a.n_chunks, a.r, partial,
                                         MergeBf16{static_cast<bf16_t *>(a.out), a.r}, stream);
        }
        e = launch_merge<Acc>(splits, n_splits, a.n_chunks, a.r, partial,
                              MergePlain<Acc>{static_cast<Acc *>(a.out), a.beta, a.r}, stream);
    }
    return e;
}

#define FMM_INSTANTIATE(OP, TH, TG1, TG2, Acc)                                                   \
    template hipError_t launch_lines<OP, TH, TG1, TG2, Acc>(const LineArgs &, int32_t, const int32_t *, \
                                                            Shape, hipStream_t);

}  // namespace fmm
