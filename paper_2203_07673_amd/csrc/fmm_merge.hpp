// Merges of split lines: the r-vectors that a line's chunks left in `partial` (chunk order)
// are added up, one wave for a line of up to kMergeAlone chunks and a block for a longer
// one.  Lanes hold a 16-byte vector of the row each, and lane groups that a short row leaves
// over take every NG-th chunk; the groups' sums, then the waves', are added in a fixed tree.
// Where split lines are many (PACK), each lane group takes a line of its own if it has at most
// kMergeFew chunks, in chunk order, and the wave or the block the others as before.
//
// One thread per element walking all chunks made the longest line's chunks one chain: on R-MAT
// scale 22, r = 256 (250 MB of partials, 760 chunks in the longest line) a merge takes 118 us,
// 180 that way; the softmax merge on scale 20, r = 128 takes 27 us, 200 that way (every thread
// walked the chunks' maxima as well).
#pragma once

#include "fmm_lines.hpp"

namespace fmm {

// Packed: enough lines to leave 4096 waves of them (four per SIMD), or a quarter of that where
// lines have few chunks.  2^17 lines of two chunks, the forward without / with: r = 8 279 / 239 us,
// r = 16 276 / 238, r = 64 667 / 640; attention step on 2^16 of them, r = 8 444 / 365.  R-MAT of 64
// per row at 2^17 (9400 lines of 4.8 chunks, r = 64, 2350 waves) 153 / 157; 2^20, 16 per row
// (21700 lines of 4.1, 5400 waves) 517 / 516.  Two groups a wave gain nothing: layered calls on
// 2^17, r = 100 (3200 lines of 3.3, 1600 waves) 667 / 673.
inline bool pack_merges(int32_t n_splits, int32_t n_chunks, int groups)
{
    const int64_t waves = n_splits / groups;
    return groups > 2 && (waves >= 4096 || (waves >= 1024 && n_chunks < 4 * (int64_t)n_splits));
}

constexpr int32_t kMergeAlone = 32;
constexpr int32_t kMergeFew = 8;
constexpr int kMergeWaves = kBlock / 64;

// What a merge does besides adding: begin (per line, by a whole wave: state for the weights) or
// begin_few (by a lane group, chunk after chunk), weight of a chunk, and the store of elements
// k .. k + VW - 1 of the line.
template <class Acc> struct MergePlain {
    Acc *out;
    double beta;
    int32_t r;
    struct State {};
    __device__ __forceinline__ State begin(int32_t, int32_t, int32_t, bool) const { return {}; }
    __device__ __forceinline__ State begin_few(int32_t, int32_t, int32_t, bool) const { return {}; }
    __device__ __forceinline__ Acc weigh(const State &, int32_t, Acc x) const { return x; }
    template <int VW> __device__ __forceinline__ void store(const State &, int32_t line, int k, Acc *v) const {
        Acc *o = out + (size_t)line * r + k;
        if (beta != 0.0) {
            Acc old[VW];
            Ld<Acc, VW, Acc>::run(o, old);
#pragma unroll
            for (int e = 0; e < VW; ++e) v[e] = Acc(beta) * old[e] + v[e];
        }
        St<Acc, VW>::run(o, v);
    }
};

// The sum as bfloat16 (rows of a multiple of 8 elements).
struct MergeBf16 {
    bf16_t *out;
    int32_t r;
    struct State {};
    __device__ __forceinline__ State begin(int32_t, int32_t, int32_t, bool) const { return {}; }
    __device__ __forceinline__ State begin_few(int32_t, int32_t, int32_t, bool) const { return {}; }
    __device__ __forceinline__ float weigh(const State &, int32_t, float x) const { return x; }
    template <int VW> __device__ __forceinline__ void store(const State &, int32_t line, int k, float *v) const {
        if constexpr (VW == 4) st_bf16<VW>(out + (size_t)line * r + k, v);
    }
};

template <class Acc> __device__ __forceinline__ Acc wave_sum(Acc x)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) x += __shfl_xor(x, d, 64);
    return x;
}
template <class Acc> __device__ __forceinline__ Acc wave_max(Acc x)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const Acc y = __shfl_xor(x, d, 64);
        x = y > x ? y : x;
    }
    return x;
}

// lpr: lanes per row (a power of two up to 64); rows of more than 64 vectors go in tiles.
// PACK: lpr < 64, so a row is one tile; a wave has the lines of its lane groups.
template <class Acc, int VW, class Op, bool PACK>
__global__ __launch_bounds__(kBlock) void merge_kernel(const int32_t *__restrict__ splits, int32_t n_splits, int32_t r,
                                                       int lpr, const Acc *__restrict__ partial, Op op)
{
    __shared__ Acc red[kMergeWaves][64 * VW];
    __shared__ uint64_t whole[kMergeWaves];
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int cv = lane % lpr, g = lane / lpr, ng = 64 / lpr;
    const int C = (r + VW - 1) / VW;

    // chunks c0, c0 + step, ... of a line, for vector v of the row
    auto chain = [&](const typename Op::State &st, int32_t first, int32_t cnt, int v, int32_t c0, int32_t step, Acc *acc) {
#pragma unroll
        for (int e = 0; e < VW; ++e) acc[e] = Acc(0);
        if (v < C) {
            const Acc *p = partial + (size_t)first * r + v * VW;
            int32_t c = c0;
            for (; c + 3 * step < cnt; c += 4 * step) {  // four vectors in flight
                Acc x[4][VW];
#pragma unroll
                for (int u = 0; u < 4; ++u) Ld<Acc, VW, Acc>::run(p + (size_t)(c + u * step) * r, x[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int e = 0; e < VW; ++e) acc[e] += op.weigh(st, first + c + u * step, x[u][e]);
            }
            for (; c < cnt; c += step) {
                Acc x[VW];
                Ld<Acc, VW, Acc>::run(p + (size_t)c * r, x);
#pragma unroll
                for (int e = 0; e < VW; ++e) acc[e] += op.weigh(st, first + c, x[e]);
            }
        }
    };
    // this lane group's chain, and the sum over the wave's groups
    auto part = [&](const typename Op::State &st, int32_t first, int32_t cnt, int v, int32_t c0, int32_t step, Acc *acc) {
        chain(st, first, cnt, v, c0, step, acc);
        for (int d = lpr; d < 64; d <<= 1)
#pragma unroll
            for (int e = 0; e < VW; ++e) acc[e] += __shfl_xor(acc[e], d, 64);
    };

    const int per_wave = PACK ? ng : 1;
    const int32_t s0 = (int32_t)blockIdx.x * (kMergeWaves * per_wave);
    const int32_t own = s0 + w * per_wave + (PACK ? g : 0);
    const int32_t own_cnt = own < n_splits ? splits[3 * own + 2] : 0;
    const bool speaks = lane == (PACK ? g * lpr : 0);  // one lane per line
    if (PACK && own_cnt > 0 && own_cnt <= kMergeFew) {
        const int32_t line = splits[3 * own], first = splits[3 * own + 1];
        const typename Op::State st = op.begin_few(line, first, own_cnt, cv == 0);
        Acc acc[VW];
        chain(st, first, own_cnt, cv, 0, 1, acc);
        if (cv < C) op.template store<VW>(st, line, cv * VW, acc);
    }
    // lines for the wave
    for (uint64_t m = __ballot(speaks && own_cnt > (PACK ? kMergeFew : 0) && own_cnt <= kMergeAlone); m; m &= m - 1) {
        const int32_t s = s0 + w * per_wave + (PACK ? (__ffsll((unsigned long long)m) - 1) / lpr : 0);
        const int32_t line = splits[3 * s], first = splits[3 * s + 1], cnt = splits[3 * s + 2];
        const typename Op::State st = op.begin(line, first, cnt, true);
        for (int t = 0; t < C; t += lpr) {
            Acc acc[VW];
            part(st, first, cnt, t + cv, g, ng, acc);
            if (g == 0 && t + cv < C) op.template store<VW>(st, line, (t + cv) * VW, acc);
        }
    }
    // lines for the block, which all its waves go through together
    const uint64_t mine = __ballot(speaks && own_cnt > kMergeAlone);
    if (lane == 0) whole[w] = mine;
    __syncthreads();
    for (int q = 0; q < kMergeWaves; ++q) {
        for (uint64_t m = whole[q]; m; m &= m - 1) {
            const int32_t s = s0 + q * per_wave + (PACK ? (__ffsll((unsigned long long)m) - 1) / lpr : 0);
            const int32_t line = splits[3 * s], first = splits[3 * s + 1], cnt = splits[3 * s + 2];
            const typename Op::State st = op.begin(line, first, cnt, w == 0);
            for (int t = 0; t < C; t += lpr) {
                Acc acc[VW];
                part(st, first, cnt, t + cv, w * ng + g, kMergeWaves * ng, acc);
                if (g == 0) {
#pragma unroll
                    for (int e = 0; e < VW; ++e) red[w][cv * VW + e] = acc[e];
                }
                __syncthreads();
                if (w == 0 && g == 0 && t + cv < C) {
#pragma unroll
                    for (int e = 0; e < VW; ++e)
                        acc[e] = (red[0][cv * VW + e] + red[1][cv * VW + e]) + (red[2][cv * VW + e] + red[3][cv * VW + e]);
                    op.template store<VW>(st, line, (t + cv) * VW, acc);
                }
                __syncthreads();
            }
        }
    }
}

template <class Acc, int VW, class Op>
hipError_t launch_merge_rows(const int32_t *splits, int32_t n_splits, int32_t n_chunks, int32_t r, const Acc *partial,
                             const Op &op, hipStream_t st)
{
    static_assert(kMergeWaves == 4, "the block's waves are added as two pairs");
    int lpr = 1;
    while (lpr < 64 && lpr * VW < r) lpr <<= 1;
    const int ng = 64 / lpr;
    const bool pack = pack_merges(n_splits, n_chunks, ng);
    const int64_t lines = (int64_t)kMergeWaves * (pack ? ng : 1);  // of a block
    const dim3 grid((unsigned)((n_splits + lines - 1) / lines));
    if (pack)
        hipLaunchKernelGGL((merge_kernel<Acc, VW, Op, true>), grid, dim3(kBlock), 0, st, splits, n_splits, r, lpr, partial, op);
    else
        hipLaunchKernelGGL((merge_kernel<Acc, VW, Op, false>), grid, dim3(kBlock), 0, st, splits, n_splits, r, lpr, partial, op);
    return hipGetLastError();
}

template <class Acc, class Op>
hipError_t launch_merge(const int32_t *splits, int32_t n_splits, int32_t n_chunks, int32_t r, const Acc *partial,
                        const Op &op, hipStream_t st)
{
    constexpr int VWV = 16 / (int)sizeof(Acc);
    return r % VWV == 0 ? launch_merge_rows<Acc, VWV>(splits, n_splits, n_chunks, r, partial, op, st)
                        : launch_merge_rows<Acc, 1>(splits, n_splits, n_chunks, r, partial, op, st);
}

}  // namespace fmm
