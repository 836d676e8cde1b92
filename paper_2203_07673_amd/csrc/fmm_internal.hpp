// Host-side declarations shared by the C-ABI layer and the kernel translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fmm.h"
#include "fmm_lines.hpp"

namespace fmm {

// Storage-driven vector width: elements per 16-byte load of A/B (F32: 4, BF16: 8, F64: 2).
enum Path { PATH_F32 = 0, PATH_BF16 = 1, PATH_F64 = 2 };

// Lane-group shapes the line kernels are built for (L lanes per line, NV vectors per lane).
struct Shape {
    int L, NV;
};

// Rows in 16-byte vectors of vw elements, or one element per lane.  A row whose length is no
// multiple of the vector ends in one that overlaps the one before (RowVec).  That can pay above
// 16 elements (64 bytes).  Below, element by element keeps more lanes on a line, which read its
// indices together: 2^17 x 2^17 R-MAT, 16 per row, r = 9, forward and column pass 42 and 64 us
// by elements against 50 and 71 in vectors.
inline bool vector_rows(int r, int vw) { return r % vw == 0 || r * (16 / vw) > 64; }

// What a line pass takes of the two, by the rows it gathers per entry: 2 (OP_FUSED2, OP_SPMM2),
// 1 (OP_FUSED1, and OP_SPMM1 with weights read through a permutation) or 0 (the others, always
// in vectors).  Vectors that start at any element take more cache accesses for a row than
// dwords do; they win where the row leaves many of the 32 or 64 lanes of the other form idle,
// where lines are short (more of them share a wave), and where the gathered rows mostly hit L2,
// as on power-law patterns (which have split lines).  float32, elements / vectors in us:
//   fused forward  uniform, 300k, 30 per row: r = 21 237 / 246, 27 273 / 284, 33 376 / 301;
//                  2^17, 16 per row: r = 21 (11 MB) 59 / 53, 27 (14 MB) 62 / 66; 2^18, 8 per
//                  row: r = 27 81 / 71; R-MAT 2^19, 16 per row: r = 25 235 / 184
//   weights by permutation  uniform, 300k, 30 per row: r = 17 368 / 386, 27 420 / 448, 33 468 /
//                  464; 2^17, 16 per row: r = 17 (9 MB) 81 / 86; with weights in order, 300k:
//                  r = 17 253 / 221, 27 280 / 283, 33 424 / 302
//   two rows       uniform, 300k, 30 per row: r = 17 433 / 475, 27 545 / 599, 38 641 / 671, 61
//                  894 / 929, 75 1018 / 1039; 60k, 30 per row: r = 21 (10 MB) 74 / 78, 38 (18 MB)
//                  125 / 115; 2^17, 16 per row: r = 38 (40 MB) 158 / 150, 61 (64 MB) 205 / 212;
//                  2^18, 8 per row: r = 46 190 / 184; 2^20, 16 per row: r = 50 (420 MB) 1514 /
//                  1489; R-MAT 2^17, 16 per row: r = 17 80 / 73, 46 165 / 107
//   no rule needed  dS with its gradient, 300k: r = 17 398 / 250, 31 410 / 326; SDDMM 268 / 240
//                  and 313 / 320
// Wider rows of a two-row pass lie within 2% either way.  float64 stays in vectors.
//
// Small patterns with split lines go by elements up to 64 of them: there the longest chains
// decide, and a chunk goes faster with 32 or 64 lanes than with the 8 or 16 of the vectors, while
// the chip has waves to spare.  The line lies at entries times lanes.  R-MAT, 2^13 lines, 8 per
// row: r = 54 one row 20 / 24, two rows 30 / 38, r = 17 19 / 23 and 27 / 36; one row at 2^24: 2^15
// lines, 8 per row, r = 54 28 / 32, 2^16, r = 23 28 / 34; at 2^25: 2^16, 8 per row, r = 54 41 / 36,
// 2^17, r = 23 39 / 39; two rows at 2^25: 53 / 57 and 50 / 61 (weights by permutation 42 / 45 and
// 43 / 51), at 2^26 98 / 73 and (2^17, 16 per row, r = 17) 79 / 73.
inline bool line_vectors(const LineArgs &a, int rows, int vw)
{
    const int r = a.r;
    if (r % vw == 0 || vw != 4 || r <= 16) return vector_rows(r, vw);
    if (a.n_chunks > 0 && r <= 64)
        return (double)a.nnz * (r > 32 ? 64 : 32) > (rows == 2 || a.wperm ? 1 << 25 : 1 << 24);
    if (rows == 0 || a.n_chunks > 0 || r > 32 * rows) return true;
    const double mb = 1e-6 * rows * 4 * r * a.nminor;  // of gathered matrices
    const bool short_lines = (double)a.nnz < 12.0 * a.nlines;
    if (rows == 1) return short_lines || mb <= (a.wperm ? 8 : 12);
    return r <= 32 ? mb <= 8 : short_lines || mb <= 48 || mb > 400;
}

// Chosen by the launcher from r (and the vector width vw) unless a valid hint is given.
// A shape is supported when it is one of the compiled ones and L * NV vectors of vw
// elements cover r.
Shape default_shape(int r, int vw);
bool shape_supported(Shape s, int r, int vw);

// The form of a pass: elements per vector and lane-group shape.  A shape given by hint that
// covers r in vectors is taken as it is.
struct LineShape {
    int vw;
    Shape shape;
};
inline LineShape line_shape(const LineArgs &a, int rows, int vw, Shape hint)
{
    if (vector_rows(a.r, vw)) {
        if (shape_supported(hint, a.r, vw)) return {vw, hint};
        if (line_vectors(a, rows, vw)) return {vw, default_shape(a.r, vw)};
    }
    return {1, default_shape(a.r, 1)};
}

// Tuning knobs (process-wide; set through fmm_set_tuning for experiments and the autotuner).
struct Tuning {
    int lanes;  // 0 = automatic
    int nv;     // 0 = automatic
};
Tuning &tuning();

// Record the hipError_t that fmm_last_hip_error() reports for this thread.
void set_last_hip_error(int32_t e);

// One launch of a line kernel (plus the merge of split lines for the accumulating ops).
// Instantiated in lines_<dtype>.hip for the type combinations the C ABI uses.
template <int OP, class TH, class TG1, class TG2, class Acc>
hipError_t launch_lines(const LineArgs &a, int32_t n_splits, const int32_t *splits, Shape hint,
                        hipStream_t stream);

// The argument checks of the batched CG on its pattern, gathered rows and split workspace (api.hip).
fmm_status gram_check(const fmm_sparse *S, const void *F, int32_t r, int32_t dtype, void *ws, size_t ws_bytes);

// Pattern preparation kernels (pattern.hip).
size_t transpose_workspace_bytes(int64_t m, int64_t n, int64_t nnz);
hipError_t csr_to_csc(int32_t m, int32_t n, int32_t nnz, const int32_t *rowptr, const int32_t *colidx,
                      const void *val, int val_bytes, int32_t *colptr, int32_t *rowidx, void *valT,
                      int32_t *perm, void *ws, hipStream_t s);
hipError_t validate(int32_t nmajor, int32_t nminor, int32_t nnz, const int32_t *ptr, const int32_t *idx,
                    int32_t *flag_dev, hipStream_t s);
hipError_t gather_values(const int32_t *perm, const void *src, void *dst, int32_t nnz, int val_bytes, hipStream_t s);
hipError_t gather_hints(const int32_t *idx, const int32_t *minor_ptr, int32_t nnz, int32_t min_len, uint8_t *hot,
                        hipStream_t s);
size_t line_order_workspace_bytes(int64_t nlines);
hipError_t line_order(const int32_t *ptr, int32_t nlines, int32_t long_len, int32_t *order, void *ws, hipStream_t s);
size_t schedule_workspace_bytes(int64_t nmajor);
hipError_t schedule_count(const int32_t *ptr, int32_t nmajor, int32_t long_len, int32_t chunk, int32_t *totals_host,
                          void *ws, hipStream_t s);
hipError_t schedule_fill(const int32_t *ptr, int32_t nmajor, int32_t long_len, int32_t chunk, int32_t *chunks,
                         int32_t *splits, void *ws, hipStream_t s);
hipError_t f32_to_bf16(const float *x, uint16_t *y, int64_t n, hipStream_t s);

}  // namespace fmm
