// Alternating least squares support (Section VI-E of the paper): batched conjugate
// gradients whose query vectors M p for every line come from one pass over the sparse
// pattern (the batching of Zhao and Canny the paper adopts), and the Frobenius residual
// ||C~ - SDDMM(A, B, S)|| over the stored entries.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "fmm.h"
#include "fmm_internal.hpp"

namespace fmm {
namespace {

fmm_status hipfail(hipError_t e)
{
    set_last_hip_error((int32_t)e);
    return FMM_ERR_HIP;
}

// Vectors of an r-row, at four-byte alignment: rows of any r start anywhere.  The
// instruction is the same 16-byte load or store.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
template <class T, int VW> struct Row;
template <> struct Row<float, 1> {
    float x;
    __device__ __forceinline__ void load(const float *p) { x = p[0]; }
    __device__ __forceinline__ void zero() { x = 0.f; }
    __device__ __forceinline__ void pin() {}
    __device__ __forceinline__ float get(int) const { return x; }
};
template <> struct Row<float, 4> {
    f32x4_t x;
    __device__ __forceinline__ void load(const float *p) { x = *reinterpret_cast<const f32x4_u *>(p); }
    __device__ __forceinline__ void zero() { x = f32x4_t{0.f, 0.f, 0.f, 0.f}; }
    __device__ __forceinline__ void pin() {}
    __device__ __forceinline__ float get(int e) const { return x[e]; }
};
template <> struct Row<bf16_t, 8> : Raw<bf16_t, 8> {};

template <int VW> __device__ __forceinline__ void ld_row(const float *p, float *o)
{
    if constexpr (VW == 1) {
        o[0] = p[0];
    } else {
#pragma unroll
        for (int q = 0; q < VW / 4; ++q) {
            const f32x4_u v = *reinterpret_cast<const f32x4_u *>(p + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) o[4 * q + e] = v[e];
        }
    }
}
template <int VW> __device__ __forceinline__ void st_row(float *p, const float *o)
{
    if constexpr (VW == 1) {
        p[0] = o[0];
    } else {
#pragma unroll
        for (int q = 0; q < VW / 4; ++q)
            *reinterpret_cast<f32x4_u *>(p + 4 * q) = f32x4_u{o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]};
    }
}

struct CgArgs {
    int32_t nlines, r, iters;
    const int32_t *ptr, *idx, *order;
    int32_t long_len, n_chunks;  // lines the split schedule takes are left out
    const void *F;
    const float *rhs;            // lines x r, or NULL: rhs_line = sum_p val_p F_j
    const float *val;            // S's values for rhs == NULL (NULL = 1)
    float lambda;
    float *X;
};

// The vectors of an r-row that a lane of a group of L owns, and the sums of products over them.
//
// A row whose length is no multiple of the vector: the last vector ends at element r - 1
// and repeats elements of the one before it (rep of them; RAG).  Repeated elements follow the
// same arithmetic, so both lanes hold and store the same bits; dot products leave them out.
// Idle vectors hold zeros, in held and in gathered rows.
//
// A solve goes on after short lines have converged, where alpha and beta are quotients of
// rounding errors, so another order of summation shows in the result (R-MAT, 16 per row, r =
// 64, 10 iterations: 3e-2 of B).  All sums keep one order for every kernel here: dot products
// an FMA chain over a lane's elements and a tree over the lanes of the power of two of vectors
// in a row, or for r of up to 64 that is no multiple of four a tree over elements; sums of
// rows a chain in entry order, chunk by chunk for split lines.  In float32 that is the order
// of a pass of the line kernels per iteration.  Rows of over 64 elements in no whole vectors
// have lanes of elements 64 apart for it, which costs (2^15 lines of 20, r = 99, 10 iterations:
// 914 us, 471 in overlapping vectors; 1433 with a pass per iteration).  Chains of bfloat16 rows
// are eight elements long.
template <class TF, int L, int NV, int VW, bool RAG> struct LaneRow {
    static_assert(!RAG || L <= 16, "r of up to 64");
    bool act[NV], full;
    int off[NV], rep[NV];
    __device__ __forceinline__ LaneRow(int lane, int r) {
        const int C = (r + VW - 1) / VW;
        full = C == L * NV;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int c = v * L + lane;
            act[v] = c < C;
            off[v] = act[v] ? (RAG ? min(c * VW, r - VW) : c * VW) : 0;
            rep[v] = RAG && act[v] ? c * VW - off[v] : 0;
        }
    }
    // what a dot product takes of a vector: repeated elements as 0
    __device__ __forceinline__ void once(const float *y, float *o) const {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int e = 0; e < VW; ++e) o[v * VW + e] = RAG && e < rep[v] ? 0.f : y[v * VW + e];
    }
    __device__ __forceinline__ void load(const float *row, float *y) const {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            ld_row<VW>(row + off[v], y + v * VW);
#pragma unroll
            for (int e = 0; e < VW; ++e) y[v * VW + e] = act[v] ? y[v * VW + e] : 0.f;
        }
    }
    // after the loads of N gathered rows
    template <int N> __device__ __forceinline__ void idle(Row<TF, VW> (*row)[NV]) const {
        if (full) return;
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
            for (int v = 0; v < NV; ++v)
                if (!act[v]) row[u][v].zero();
    }
    // this lane's part of <y, z>, for a y that went through once()
    template <class Get> __device__ __forceinline__ float part(const float *y, Get z) const {
        if constexpr (RAG) {
            float m[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) m[e] = fmadd(y[e], z(0, e), 0.f);
            const float lo = rep[0] == 1 ? m[1] + m[2] : m[0] + m[1];  // one repeated: pairs begin at 1
            return lo + (rep[0] == 1 ? m[3] : m[2] + m[3]);
        }
        float s = 0.f;
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int e = 0; e < VW; ++e) s = fmadd(y[v * VW + e], z(v, e), s);
        return s;
    }
    __device__ __forceinline__ float dot(const float *y, const float *z) const {
        float ym[NV * VW];
        once(y, ym);
        return group_sum<L>(part(ym, [&](int v, int e) { return z[v * VW + e]; }));
    }
    // <y, y>, where the chain begins at the second element
    __device__ __forceinline__ float square(const float *y) const {
        float ym[NV * VW];
        once(y, ym);
        if constexpr (VW == 1 || RAG) return group_sum<L>(part(ym, [&](int v, int e) { return ym[v * VW + e]; }));
        float s = fmadd(ym[0], ym[0], ym[1 % (NV * VW)] * ym[1 % (NV * VW)]);
#pragma unroll
        for (int e = 2; e < NV * VW; ++e) s = fmadd(ym[e], ym[e], s);
        return group_sum<L>(s);
    }
    __device__ __forceinline__ void store(float *row, const float *y) const {
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (act[v]) st_row<VW>(row + off[v], y + v * VW);
    }
};

// One CG step on a line's iterate x, residual res and direction p, with q = (sum_j F_j F_j^T) p and
// rr = <res, res>; returns the new rr.
template <class TF, int L, int NV, int VW, bool RAG>
__device__ __forceinline__ float cg_step(const LaneRow<TF, L, NV, VW, RAG> &at, float lam, float rr, float *p, float *q,
                                         float *x, float *res)
{
    constexpr int E = NV * VW;
#pragma unroll
    for (int e = 0; e < E; ++e) q[e] = fmadd(lam, p[e], q[e]);
    const float pq = at.dot(p, q);
    const float alpha = (rr > 0.f && pq > 0.f) ? rr / pq : 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        x[e] = fmadd(alpha, p[e], x[e]);
        res[e] = fmadd(-alpha, q[e], res[e]);
    }
    const float rrn = at.square(res);
    const float beta = rr > 0.f ? rrn / rr : 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) p[e] = fmadd(beta, p[e], res[e]);
    return rrn;
}

// out += sum of c_u F_u over N rows, in order: c_u = <y, F_u> (DOT; y went through once()) or
// w_u.  Entries from n on are left out.
template <bool DOT, int N, int L, int NV, int VW, bool RAG, class TF>
__device__ __forceinline__ void add_rows(const LaneRow<TF, L, NV, VW, RAG> &at, Row<TF, VW> (*row)[NV], int32_t n,
                                         const float *y, const float *w, float *out)
{
    float d[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        if constexpr (DOT) {
#pragma unroll
            for (int v = 0; v < NV; ++v) row[u][v].pin();
            d[u] = at.part(y, [&](int v, int e) { return row[u][v].get(e); });
        } else {
            d[u] = w[u];
        }
    }
    if constexpr (DOT) {
#pragma unroll
        for (int u = 0; u < N; ++u) d[u] = group_sum<L>(d[u]);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const float c = u < n ? d[u] : 0.f;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            row[u][v].pin();
#pragma unroll
            for (int e = 0; e < VW; ++e) out[v * VW + e] = fmadd(c, row[u][v].get(e), out[v * VW + e]);
        }
    }
}

// The split lines' solve: iterate, residual and direction of every line, <residual, residual>, and
// the chunks' partials.
struct SplitCg {
    const int32_t *splits;
    int32_t n_splits, r;
    float lambda;
    const float *rhs;
    float *X, *R, *P, *rr;
    const float *partial;
};

// The whole CG solve of a line by a group of L lanes that holds an r-row, with the gathered
// rows F_j in registers for every iteration.  A line's iterations depend on no other line, so
// each row comes from memory once where a pass per iteration gathers it iters + 1 times (and
// once more for the right-hand side).
//
// A lane holds S rows (NV vectors each: about 160 registers, which leaves two waves per SIMD);
// entries past S are gathered again in every iteration, OV at a time with the indices of the
// next read ahead.  With lines of 32 and r = 128 that is none in the rows and one column in
// fourteen.  Slots go in blocks of SB that a line without entries there skips; inside a block
// entries past the end repeat the line's last row and weigh 0.  One group sums a line's rows,
// since the order of that sum is fixed; several groups a line took 3.95 ms for the sweep below,
// in another order.
//
// Bound by vector issue: about 16 instructions per entry and iteration for two lines of a
// wave.  A sweep over 2^18 x 2^18, 32 per row, r = 128, 10 iterations a side, with the loss,
// where a pass per iteration took 16.7 ms: 4.2 ms.  Slots, block and rows past them of other
// splits: 48, 8, 4 4.3 ms; 40, 4, 8 4.3; 36, 6, 12 4.9 (spills); at three waves per SIMD 32, 4, 2
// 4.1 and 30, 3, 2 4.5, but with lines of 40, r = 128 3.4 ms at 32 slots and 2.7 at 40, with
// lines of 38, r = 32 0.97 and 0.72.
template <class TF, int L, int NV, int VW, bool RAG, int S, int SB>
__global__ __launch_bounds__(kBlock, 2) void cg_resident_kernel(CgArgs a)
{
    constexpr int E = NV * VW;
    constexpr int OV = VW == 1 ? 8 : NV > 1 ? 2 : VW == 8 ? 4 : 8;  // rows in flight past the slots
    static_assert(S % SB == 0, "whole blocks of slots");
    const int lane = threadIdx.x % L;
    const int64_t k = (int64_t)blockIdx.x * (kBlock / L) + threadIdx.x / L;
    if (k >= a.nlines) return;
    const int32_t line = a.order ? a.order[k] : (int32_t)k;
    const int32_t begin = a.ptr[line], len = a.ptr[line + 1] - begin;
    if (a.n_chunks > 0 && len > a.long_len) return;
    const int r = a.r;
    const LaneRow<TF, L, NV, VW, RAG> at(lane, r);
    const TF *F = static_cast<const TF *>(a.F);
    const int32_t *idx = a.idx + begin;

    Row<TF, VW> f[S][NV];
#pragma unroll
    for (int b = 0; b < S; b += SB) {
        if (b < len) {
            int32_t j[SB];
#pragma unroll
            for (int u = 0; u < SB; ++u) j[u] = idx[min(b + u, len - 1)];
#pragma unroll
            for (int u = 0; u < SB; ++u)
#pragma unroll
                for (int v = 0; v < NV; ++v) f[b + u][v].load(F + (size_t)j[u] * r + at.off[v]);
        }
    }
    at.template idle<S>(f);
    float *Xrow = a.X + (size_t)line * r;
    float x[E], res[E], p[E], q[E];
    at.load(Xrow, x);

    // out = sum over the line of c_t F_j, with c_t = <y, F_j> or val_t
    auto gather = [&](auto dot_tag, const float *y, const float *val, float *out) {
        constexpr bool DOT = decltype(dot_tag)::value;
        float ym[E];
        if constexpr (DOT) at.once(y, ym);
#pragma unroll
        for (int e = 0; e < E; ++e) out[e] = 0.f;
        auto weights = [&](int32_t t, float *w, int n) {
            if constexpr (!DOT) {
#pragma unroll
                for (int u = 0; u < n; ++u) w[u] = 1.f;
                if (val)
#pragma unroll
                    for (int u = 0; u < n; ++u) w[u] = val[min(t + u, len - 1)];
            }
        };
#pragma unroll
        for (int b = 0; b < S; b += SB)
            if (b < len) {
                float w[SB];
                weights(b, w, SB);
                add_rows<DOT, SB>(at, f + b, len - b, ym, w, out);
            }
        int32_t j[OV];  // of the next rows, which arrive while these are summed
        auto indices = [&](int32_t t) {
#pragma unroll
            for (int u = 0; u < OV; ++u) j[u] = idx[min(t + u, len - 1)];
        };
        if (S < len) indices(S);
        for (int32_t t = S; t < len; t += OV) {
            Row<TF, VW> o[OV][NV];
            float w[OV];
            weights(t, w, OV);
#pragma unroll
            for (int u = 0; u < OV; ++u)
#pragma unroll
                for (int v = 0; v < NV; ++v) o[u][v].load(F + (size_t)j[u] * r + at.off[v]);
            indices(t + OV);
            at.template idle<OV>(o);
            add_rows<DOT, OV>(at, o, len - t, ym, w, out);
        }
    };
    const float lam = a.lambda;
    if (a.rhs) {
        at.load(a.rhs + (size_t)line * r, res);
    } else {
        gather(std::false_type{}, x, a.val ? a.val + begin : nullptr, res);
    }
    gather(std::true_type{}, x, nullptr, q);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        res[e] -= fmadd(lam, x[e], q[e]);
        p[e] = res[e];
    }
    float rr = at.square(res);
    for (int it = 0; it < a.iters; ++it) {
        gather(std::true_type{}, p, nullptr, q);
        rr = cg_step(at, lam, rr, p, q, x, res);
    }
    at.store(Xrow, x);
}

// Split lines keep a pass per iteration, which spreads a long line over the chip: a group
// per chunk, and a group per line for the step, which adds the chunks' sums in chunk order.
// R-MAT of 16 per row at 2^17, r = 64, the sweep with the whole lines above: 2.07 ms with all
// lines in passes, 1.09 now; at 2^13, r = 50 0.69 and 0.67.  16 rows in flight in a chunk: 8 and
// 32 take 1.14.
// partial_c = sum over chunk c of <H_line, F_j> F_j (DOT) or of val_p F_j
template <class TF, int L, int NV, int VW, bool RAG, bool DOT>
__global__ __launch_bounds__(kBlock) void cg_chunk_kernel(int32_t n_chunks, int32_t r, const int32_t *__restrict__ chunks,
                                                          const int32_t *__restrict__ idx,
                                                          const float *__restrict__ val, const float *__restrict__ H,
                                                          const TF *__restrict__ F, float *__restrict__ partial)
{
    constexpr int E = NV * VW;
    constexpr int U = (VW == 8 ? 8 : 16) / NV;
    const int lane = threadIdx.x % L;
    const int64_t c = (int64_t)blockIdx.x * (kBlock / L) + threadIdx.x / L;
    if (c >= n_chunks) return;
    const int32_t line = chunks[3 * c], begin = chunks[3 * c + 1], end = chunks[3 * c + 2];
    const LaneRow<TF, L, NV, VW, RAG> at(lane, r);
    float h[E], hm[E], acc[E];
    if constexpr (DOT) {
        at.load(H + (size_t)line * r, h);
        at.once(h, hm);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
    int32_t j[U];  // of the next rows, which arrive while these are summed
    auto indices = [&](int32_t t) {
#pragma unroll
        for (int u = 0; u < U; ++u) j[u] = idx[min(t + u, end - 1)];
    };
    if (begin < end) indices(begin);
    for (int32_t t = begin; t < end; t += U) {
        Row<TF, VW> f[U][NV];
        float w[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < NV; ++v) f[u][v].load(F + (size_t)j[u] * r + at.off[v]);
        if constexpr (!DOT) {
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = 1.f;
            if (val) {
#pragma unroll
                for (int u = 0; u < U; ++u) w[u] = val[min(t + u, end - 1)];
            }
        }
        indices(t + U);
        at.template idle<U>(f);
        add_rows<DOT, U>(at, f, end - t, hm, w, acc);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v)
        if (at.act[v]) st_row<VW>(partial + (size_t)c * r + at.off[v], acc + v * VW);
}

// The sum of a line's chunks in chunk order, for VW elements from `off` of split line s.
template <int VW>
__device__ __forceinline__ void chunk_sum(const int32_t *__restrict__ split, int32_t r, int32_t off,
                                          const float *__restrict__ partial, float *out)
{
    const float *p = partial + (size_t)split[1] * r + off;
    const int32_t cnt = split[2];
#pragma unroll
    for (int e = 0; e < VW; ++e) out[e] = 0.f;
    for (int32_t c = 0; c < cnt; c += 8) {
        float v[8][VW];
#pragma unroll
        for (int u = 0; u < 8; ++u) ld_row<VW>(p + (size_t)min(c + u, cnt - 1) * r, v[u]);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int e = 0; e < VW; ++e) out[e] = c + u < cnt ? out[e] + v[u][e] : out[e];
    }
}

// out_line = the sum of the line's chunks
__global__ __launch_bounds__(kBlock) void cg_chunk_sum_kernel(const int32_t *__restrict__ splits, int32_t n_splits,
                                                              int32_t r, const float *__restrict__ partial,
                                                              float *__restrict__ out)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= (int64_t)n_splits * r) return;
    const int32_t s = (int32_t)(t / r), k = (int32_t)(t % r);
    chunk_sum<1>(splits + 3 * s, r, k, partial, out + (size_t)splits[3 * s] * r + k);
}

// Q = (sum_j F_j F_j^T) y for the line of split s, from its chunks' partials.
template <class TF, int L, int NV, int VW, bool RAG>
__device__ __forceinline__ void chunk_sums(const LaneRow<TF, L, NV, VW, RAG> &at, const int32_t *__restrict__ split,
                                           int32_t r, const float *__restrict__ partial, float *q)
{
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        chunk_sum<VW>(split, r, at.off[v], partial, q + v * VW);
#pragma unroll
        for (int e = 0; e < VW; ++e) q[v * VW + e] = at.act[v] ? q[v * VW + e] : 0.f;
    }
}

// Start of CG: R = rhs - (Q + lambda X), P = R, rr = <R, R>.  rhs may be R itself.
template <class TF, int L, int NV, int VW, bool RAG>
__global__ __launch_bounds__(kBlock) void cg_start_kernel(SplitCg a)
{
    constexpr int E = NV * VW;
    const int64_t k = (int64_t)blockIdx.x * (kBlock / L) + threadIdx.x / L;
    if (k >= a.n_splits) return;
    const LaneRow<TF, L, NV, VW, RAG> at(threadIdx.x % L, a.r);
    const int32_t line = a.splits[3 * k];
    const size_t row = (size_t)line * a.r;
    float x[E], q[E], res[E];
    at.load(a.rhs + row, res);
    at.load(a.X + row, x);
    chunk_sums(at, a.splits + 3 * k, a.r, a.partial, q);
#pragma unroll
    for (int e = 0; e < E; ++e) res[e] -= fmadd(a.lambda, x[e], q[e]);
    const float rr = at.square(res);
    at.store(a.R + row, res);
    at.store(a.P + row, res);
    if (threadIdx.x % L == 0) a.rr[line] = rr;
}

// One CG step, with Q = (sum_j F_j F_j^T) P:
//   alpha = rr / <P, Q + lambda P>;  X += alpha P;  R -= alpha (Q + lambda P);
//   beta = <R, R>_new / rr;  P = R + beta P;  rr = <R, R>_new.
// A line whose residual or curvature is zero keeps its iterate (alpha = beta = 0).
template <class TF, int L, int NV, int VW, bool RAG>
__global__ __launch_bounds__(kBlock) void cg_step_kernel(SplitCg a)
{
    constexpr int E = NV * VW;
    const int64_t k = (int64_t)blockIdx.x * (kBlock / L) + threadIdx.x / L;
    if (k >= a.n_splits) return;
    const LaneRow<TF, L, NV, VW, RAG> at(threadIdx.x % L, a.r);
    const int32_t line = a.splits[3 * k];
    const size_t row = (size_t)line * a.r;
    float p[E], q[E], x[E], res[E];
    at.load(a.P + row, p);
    at.load(a.X + row, x);
    at.load(a.R + row, res);
    chunk_sums(at, a.splits + 3 * k, a.r, a.partial, q);
    const float rr = cg_step(at, a.lambda, a.rr[line], p, q, x, res);
    at.store(a.X + row, x);
    at.store(a.R + row, res);
    at.store(a.P + row, p);
    if (threadIdx.x % L == 0) a.rr[line] = rr;
}

// Per-block partial sums of (val[p] - R[p])^2 in float64, then one block adds the
// partials in block order: a fixed summation order, so the result is reproducible.
__global__ __launch_bounds__(256) void residual_partial_kernel(int64_t nnz, const float *__restrict__ val,
                                                               const float *__restrict__ R, double *__restrict__ part)
{
    __shared__ double sh[256];
    double acc = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < nnz; p += (int64_t)gridDim.x * 256) {
        const double d = (double)(val ? val[p] : 1.f) - (double)R[p];
        acc += d * d;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(256) void residual_final_kernel(int32_t nparts, const double *__restrict__ part,
                                                             double *__restrict__ out)
{
    __shared__ double sh[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 256) acc += part[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0];
}

constexpr int kResidualBlocks = 1024;

template <class TF, int L, int NV, int VW, bool RAG, int S, int SB>
hipError_t launch_resident(const CgArgs &a, hipStream_t st)
{
    constexpr int LPB = kBlock / L;
    const unsigned nb = (unsigned)(((int64_t)a.nlines + LPB - 1) / LPB);
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL((cg_resident_kernel<TF, L, NV, VW, RAG, S, SB>), dim3(nb), dim3(kBlock), 0, st, a);
    return hipGetLastError();
}

// Partials of the chunks, to ws: of <H_line, F_j> F_j, or of val_p F_j for H NULL.
template <class TF, int L, int NV, int VW, bool RAG>
hipError_t launch_chunks(const fmm_sparse *S, const void *F, int32_t r, const float *H, void *ws, hipStream_t st)
{
    constexpr int GPB = kBlock / L;
    const int64_t nb = ((int64_t)S->n_chunks + GPB - 1) / GPB;
    if (nb > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const float *val = H ? nullptr : static_cast<const float *>(S->val);
    float *partial = static_cast<float *>(ws);
    if (H)
        hipLaunchKernelGGL((cg_chunk_kernel<TF, L, NV, VW, RAG, true>), dim3((unsigned)nb), dim3(kBlock), 0, st, S->n_chunks,
                           r, S->chunks, S->idx, val, H, static_cast<const TF *>(F), partial);
    else
        hipLaunchKernelGGL((cg_chunk_kernel<TF, L, NV, VW, RAG, false>), dim3((unsigned)nb), dim3(kBlock), 0, st,
                           S->n_chunks, r, S->chunks, S->idx, val, H, static_cast<const TF *>(F), partial);
    return hipGetLastError();
}

// Lanes per row by the number of vectors in a row.
template <class TF, int VW, bool RAG, class Fn> hipError_t by_width(int r, Fn fn)
{
    const int C = (r + VW - 1) / VW;
#define CG_WIDTH(Lv, NVv) fn(std::integral_constant<int, Lv>{}, std::integral_constant<int, NVv>{})
    if (C <= 4) return CG_WIDTH(4, 1);
    if constexpr (VW == 1) {  // r < 4 or over 64
        if (C <= 128) return CG_WIDTH(64, 2);
        return CG_WIDTH(64, 4);
    } else {
        if (C <= 8) return CG_WIDTH(8, 1);
        if (C <= 16) return CG_WIDTH(16, 1);
        if constexpr (!RAG) {  // r of up to 64
            if (C <= 32) return CG_WIDTH(32, 1);
            if (C <= 64) return CG_WIDTH(64, 1);
            if (C <= 128) return CG_WIDTH(64, 2);
            if constexpr (VW == 4) return CG_WIDTH(64, 4);
        }
    }
#undef CG_WIDTH
    return hipErrorInvalidValue;
}

// The form of a row for every kernel here: fn with its type, vector and overlap, then its lanes.
// Above 64 elements a row of no whole vectors goes by elements, 64 apart in a lane.
template <class Fn> hipError_t by_row(int32_t dtype, int r, Fn fn)
{
    auto with = [&](auto tf, auto vw, auto rag) {
        return by_width<decltype(tf), decltype(vw)::value, decltype(rag)::value>(r, [&](auto L, auto NV) { return fn(tf, L, NV, vw, rag); });
    };
    typedef std::integral_constant<int, 1> V1;
    typedef std::integral_constant<int, 4> V4;
    if (dtype == FMM_BF16) return with(bf16_t(), std::integral_constant<int, 8>{}, std::false_type{});
    if (r % 4 == 0) return with(float(), V4{}, std::false_type{});
    if (r < 4 || r > 64) return with(float(), V1{}, std::false_type{});
    return with(float(), V4{}, std::true_type{});
}

// Slots that fill the registers of two waves per SIMD beside the line's four or five vectors.
hipError_t resident_lines(int32_t dtype, const CgArgs &a, hipStream_t st)
{
    return by_row(dtype, a.r, [&](auto tf, auto L, auto NV, auto VW, auto RAG) {
        typedef decltype(tf) TF;
        constexpr int l = L.value, nv = NV.value, vw = VW.value;
        constexpr bool rag = RAG.value;
        if constexpr (nv == 1) return launch_resident<TF, l, nv, vw, rag, 40, vw == 8 ? 4 : 8>(a, st);
        else if constexpr (vw == 1) return launch_resident<TF, l, nv, vw, rag, nv == 2 ? 72 : 36, nv == 2 ? 8 : 4>(a, st);
        else if constexpr (nv == 2) return launch_resident<TF, l, nv, vw, rag, vw == 8 ? 12 : 18, 2>(a, st);
        else return launch_resident<TF, l, nv, vw, rag, 4, 2>(a, st);
    });
}

// begin: the start of the iteration; else one step.
template <class TF, int L, int NV, int VW, bool RAG>
hipError_t launch_split_cg(const SplitCg &c, bool begin, hipStream_t st)
{
    const unsigned nb = (unsigned)(((int64_t)c.n_splits + kBlock / L - 1) / (kBlock / L));
    if (nb == 0) return hipSuccess;
    if (begin) hipLaunchKernelGGL((cg_start_kernel<TF, L, NV, VW, RAG>), dim3(nb), dim3(kBlock), 0, st, c);
    else hipLaunchKernelGGL((cg_step_kernel<TF, L, NV, VW, RAG>), dim3(nb), dim3(kBlock), 0, st, c);
    return hipGetLastError();
}

// CG for every line of S: those of up to long_len entries in one kernel, the split ones by
// a pass per iteration.  rhs NULL: the right-hand side is sum_p val_p F_j.
fmm_status solve_lines(const fmm_sparse *S, const void *F, int32_t r, int32_t dtype, const float *rhs, float lambda,
                       int32_t iters, float *X, float *work, size_t work_bytes, void *ws, size_t ws_bytes,
                       hipStream_t stream)
{
    if (!S) return FMM_ERR_NULL;
    if (S->orient != FMM_CSR && S->orient != FMM_CSC) return FMM_ERR_ORIENT;
    const int32_t n = S->orient == FMM_CSR ? S->rows : S->cols;
    const int32_t minor = S->orient == FMM_CSR ? S->cols : S->rows;
    if (n < 0 || minor < 0 || r < 1 || iters < 0 || !(lambda >= 0.f)) return FMM_ERR_DIM;
    if (dtype != FMM_F32 && dtype != FMM_BF16) return FMM_ERR_DTYPE;
    if (n > 0 && (!X || !work)) return FMM_ERR_NULL;
    if (minor > 0 && !F) return FMM_ERR_NULL;
    size_t need = 0;
    fmm_cg_work_size(n, r, &need);
    if (work_bytes < need) return FMM_ERR_WORKSPACE;
    const int vw = r % 4 == 0 ? 4 : 1;
    if (r > 64 * 4 * vw) return FMM_ERR_DTYPE;
    if (vw == 4 && ((uintptr_t)rhs % 16 || (uintptr_t)X % 16 || (uintptr_t)work % 16)) return FMM_ERR_UNSUPPORTED;
    fmm_status s = gram_check(S, F, r, dtype, ws, ws_bytes);
    if (s != FMM_OK) return s;
    CgArgs a;
    memset(&a, 0, sizeof(a));
    a.nlines = n;
    a.r = r;
    a.iters = iters;
    a.ptr = S->ptr;
    a.idx = S->idx;
    a.order = S->order;
    a.long_len = S->long_len;
    a.n_chunks = S->n_chunks;
    a.F = F;
    a.rhs = rhs;
    a.val = static_cast<const float *>(S->val);
    a.lambda = lambda;
    a.X = X;
    hipError_t e;
    if (S->n_chunks > 0) {
        SplitCg c;
        c.splits = S->splits;
        c.n_splits = S->n_splits;
        c.r = r;
        c.lambda = lambda;
        c.X = X;
        c.R = work;
        c.P = work + (size_t)n * r;
        c.partial = static_cast<const float *>(ws);
        c.rr = work + 2 * (size_t)n * r;
        c.rhs = rhs ? rhs : c.R;
        auto partials = [&](const float *H) {  // of <H_line, F_j> F_j, or for NULL of val_p F_j
            return by_row(dtype, r, [&](auto tf, auto L, auto NV, auto VW, auto RAG) {
                return launch_chunks<decltype(tf), L.value, NV.value, VW.value, RAG.value>(S, F, r, H, ws, stream);
            });
        };
        if (!rhs) {
            e = partials(nullptr);
            if (e != hipSuccess) return hipfail(e);
            const int64_t nb = ((int64_t)S->n_splits * r + kBlock - 1) / kBlock;
            if (nb > 0x7fffffffLL) return hipfail(hipErrorInvalidConfiguration);
            if (nb > 0) {
                hipLaunchKernelGGL(cg_chunk_sum_kernel, dim3((unsigned)nb), dim3(kBlock), 0, stream, S->splits,
                                   S->n_splits, r, c.partial, c.R);
                e = hipGetLastError();
                if (e != hipSuccess) return hipfail(e);
            }
        }
        for (int32_t it = -1; it < iters; ++it) {
            e = partials(it < 0 ? X : c.P);
            if (e != hipSuccess) return hipfail(e);
            e = by_row(dtype, r, [&](auto tf, auto L, auto NV, auto VW, auto RAG) {
                return launch_split_cg<decltype(tf), L.value, NV.value, VW.value, RAG.value>(c, it < 0, stream);
            });
            if (e != hipSuccess) return hipfail(e);
        }
    }
    e = resident_lines(dtype, a, stream);
    return e == hipSuccess ? FMM_OK : hipfail(e);
}

}  // namespace
}  // namespace fmm

using namespace fmm;

extern "C" {

fmm_status fmm_cg_work_size(int32_t nmajor, int32_t r, size_t *bytes)
{
    if (!bytes) return FMM_ERR_NULL;
    if (nmajor < 0 || r < 1) return FMM_ERR_DIM;
    *bytes = (2 * (size_t)nmajor * r + (size_t)nmajor) * sizeof(float);  // residual and direction of split lines, <R, R>
    return FMM_OK;
}

fmm_status fmm_cg_lines(const fmm_sparse *S, const void *F, int32_t r, int32_t dtype, const float *rhs, float lambda,
                        int32_t iters, float *X, float *work, size_t work_bytes, void *ws, size_t ws_bytes,
                        hipStream_t stream)
{
    if (S && (S->orient == FMM_CSR ? S->rows : S->cols) > 0 && !rhs) return FMM_ERR_NULL;
    return solve_lines(S, F, r, dtype, rhs, lambda, iters, X, work, work_bytes, ws, ws_bytes, stream);
}

fmm_status fmm_als_lines(const fmm_sparse *S, const void *F, int32_t r, int32_t dtype, float lambda, int32_t iters,
                         float *X, float *work, size_t work_bytes, void *ws, size_t ws_bytes, hipStream_t stream)
{
    return solve_lines(S, F, r, dtype, nullptr, lambda, iters, X, work, work_bytes, ws, ws_bytes, stream);
}

fmm_status fmm_residual_workspace(const fmm_sparse *S, size_t *bytes)
{
    if (!S || !bytes) return FMM_ERR_NULL;
    if (S->nnz < 0) return FMM_ERR_DIM;
    *bytes = ((size_t)S->nnz * sizeof(float) + 255) / 256 * 256 + kResidualBlocks * sizeof(double);
    return FMM_OK;
}

fmm_status fmm_sddmm_residual(const fmm_sparse *S_csr, const void *A, const void *B, int32_t r, int32_t dtype,
                              double *out, void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (!S_csr || !out) return FMM_ERR_NULL;
    if (S_csr->orient != FMM_CSR) return FMM_ERR_ORIENT;
    if (dtype != FMM_F32 && dtype != FMM_BF16) return FMM_ERR_DTYPE;
    size_t need = 0;
    fmm_residual_workspace(S_csr, &need);
    if (!ws || ws_bytes < need || (uintptr_t)ws % 16) return FMM_ERR_WORKSPACE;
    float *R = static_cast<float *>(ws);
    double *part = reinterpret_cast<double *>(static_cast<char *>(ws) + ((size_t)S_csr->nnz * sizeof(float) + 255) /
                                                                             256 * 256);
    fmm_sparse pat = *S_csr;  // the model's prediction uses the pattern alone
    pat.val = nullptr;
    fmm_status s = fmm_sddmm(&pat, A, B, r, dtype, R, 0.0, nullptr, 0, stream);
    if (s != FMM_OK) return s;
    hipLaunchKernelGGL(residual_partial_kernel, dim3(kResidualBlocks), dim3(256), 0, stream, (int64_t)S_csr->nnz,
                       static_cast<const float *>(S_csr->val), (const float *)R, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hipfail(e);
    hipLaunchKernelGGL(residual_final_kernel, dim3(1), dim3(256), 0, stream, kResidualBlocks, (const double *)part,
                       out);
    e = hipGetLastError();
    return e == hipSuccess ? FMM_OK : hipfail(e);
}

}  // extern "C"
