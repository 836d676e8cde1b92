// Graph attention on the FusedMM access pattern (Section VI-E of the paper): the
// sampled product is replaced by the attention score a^T (H_i || H_j) = s_i + t_j,
// passed through LeakyReLU, optionally normalised by a softmax over each row's stored
// entries, and the result weights an SpMM with H:
//
//   out_i = sum_j w_ij H_j,   e_ij = LeakyReLU(S_ij (s_i + t_j)),
//   w_ij = e_ij, or w_ij = exp(e_ij - max_k e_ik) / sum_k exp(e_ik - max_k e_ik).
//
// The fused kernel keeps the softmax state of a row (running maximum m, normaliser l
// and the weighted sum) in registers and rescales it when the maximum grows, so a row
// is read once and no edge value is written to memory.  Long rows are split into
// chunks whose (sum, m, l) triples are combined afterwards in a fixed order.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

#include "fmm.h"
#include "fmm_internal.hpp"
#include "fmm_merge.hpp"

namespace fmm {
namespace {

template <class Acc> __device__ __forceinline__ Acc exp_acc(Acc x);
template <> __device__ __forceinline__ float exp_acc<float>(float x) { return expf(x); }
template <> __device__ __forceinline__ double exp_acc<double>(double x) { return exp(x); }
template <class Acc> __device__ __forceinline__ Acc log_acc(Acc x);
template <> __device__ __forceinline__ float log_acc<float>(float x) { return logf(x); }
template <> __device__ __forceinline__ double log_acc<double>(double x) { return log(x); }
template <class Acc> __device__ __forceinline__ Acc neg_inf();
template <> __device__ __forceinline__ float neg_inf<float>() { return -__builtin_huge_valf(); }
template <> __device__ __forceinline__ double neg_inf<double>() { return -__builtin_huge_val(); }

// s_i = a1 . H_i and t_i = a2 . H_i for every row: one lane group per row, kScoreRows rows in
// flight per group.  H is gathered from next; where it is larger than the 256 MB behind the
// L2s can hold it is streamed (kStreamBytes), which leaves those caches to the gathers' rows:
// an attention step with two heads on R-MAT scale 20, r = 128 (H of 512 MB), 7.45 -> 7.35 ms.
constexpr size_t kStreamBytes = (size_t)256 << 20;
constexpr int kScoreRows = 4;
template <class TH, class Acc, int L, int NV, int VW, bool RAG>
__global__ __launch_bounds__(kBlock) void gat_scores_kernel(const TH *__restrict__ H, int32_t n, int32_t r,
                                                            const Acc *__restrict__ a1, const Acc *__restrict__ a2,
                                                            Acc *__restrict__ s, Acc *__restrict__ t, bool stream)
{
    constexpr int GPB = kBlock / L;
    const int lane = threadIdx.x % L;
    const int64_t row0 = (int64_t)blockIdx.x * (GPB * kScoreRows) + threadIdx.x / L;
    RowVec<VW, RAG> rv[NV];
    Raw<TH, VW> h[kScoreRows][NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) rv[v] = RowVec<VW, RAG>(v * L + lane, r);
#pragma unroll
    for (int u = 0; u < kScoreRows; ++u) {
        const int64_t row = min(row0 + u * GPB, (int64_t)n - 1);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (stream) h[u][v].load_nt(H + row * r + rv[v].off);
            else h[u][v].load(H + row * r + rv[v].off);
        }
    }
    Acc x[kScoreRows], y[kScoreRows];
#pragma unroll
    for (int u = 0; u < kScoreRows; ++u) x[u] = y[u] = Acc(0);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if (!rv[v].act) continue;
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            if (RAG && e < rv[v].rep) continue;
            const Acc b1 = a1[rv[v].off + e], b2 = a2[rv[v].off + e];
#pragma unroll
            for (int u = 0; u < kScoreRows; ++u) {
                x[u] += b1 * Acc(h[u][v].get(e));
                y[u] += b2 * Acc(h[u][v].get(e));
            }
        }
    }
#pragma unroll
    for (int u = 0; u < kScoreRows; ++u) {
        const Acc xs = group_sum<L>(x[u]), ys = group_sum<L>(y[u]);
        const int64_t row = row0 + u * GPB;
        if (lane == 0 && row < n) {
            s[row] = xs;
            t[row] = ys;
        }
    }
}

// Edge values of every stored entry, in CSR order (the unfused form: written to memory
// for a separate SpMM).  A group of L lanes owns a row; lanes take the row's entries in
// turn.  Softmax: the row maximum and the sum of exponentials are reduced over the group
// (a fixed tree), then every value is rescaled.
template <class Acc, int L>
__global__ __launch_bounds__(kBlock) void gat_edges_kernel(int32_t n, const int32_t *__restrict__ ptr,
                                                           const int32_t *__restrict__ idx, const Acc *__restrict__ val,
                                                           const Acc *__restrict__ s, const Acc *__restrict__ t,
                                                           Acc slope, bool softmax, Acc *__restrict__ w)
{
    const int lane = threadIdx.x % L;
    const int64_t row = (int64_t)blockIdx.x * (kBlock / L) + threadIdx.x / L;
    if (row >= n) return;
    const int32_t b = ptr[row], e = ptr[row + 1];
    const Acc si = s[row];
    Acc mx = neg_inf<Acc>();
    for (int32_t p = b + lane; p < e; p += L) {
        const Acc x = (val ? val[p] : Acc(1)) * (si + t[idx[p]]);
        const Acc v = x >= Acc(0) ? x : slope * x;
        w[p] = v;
        mx = v > mx ? v : mx;
    }
    if (!softmax) return;
    // group maximum: max is exact, so any reduction order gives the same bits
#pragma unroll
    for (int o = 1; o < L; o <<= 1) {
        const Acc y = __shfl_xor(mx, o, L);
        mx = y > mx ? y : mx;
    }
    Acc sum = Acc(0);
    for (int32_t p = b + lane; p < e; p += L) {
        const Acc v = exp_acc<Acc>(w[p] - mx);
        w[p] = v;
        sum += v;
    }
    sum = group_sum<L>(sum);
    const Acc inv = sum > Acc(0) ? Acc(1) / sum : Acc(0);
    for (int32_t p = b + lane; p < e; p += L) w[p] *= inv;
}

struct GatArgs {
    int32_t nlines, r;
    const int32_t *ptr, *idx;
    const void *val;  // S values (Acc) or NULL for a 0/1 adjacency
    const void *s, *t;
    const void *H;
    void *out;
    double slope;
    int32_t long_len, n_chunks;
    const int32_t *chunks;
    void *partial;  // n_chunks x r sums, then n_chunks x 2 (m, l)
    const int32_t *order;  // row processing order, NULL = index order
    void *lse;             // softmax: per-row log-sum-exp of the edge values (Acc), or NULL
};

template <class TH, class Acc, int L, int NV, int VW, int U, bool SOFTMAX, bool RAG>
__global__ __launch_bounds__(kBlock) void gat_kernel(GatArgs a, int32_t nb_chunk_blocks)
{
    constexpr int GPB = kBlock / L;
    constexpr int E = NV * VW;
    const int lane = threadIdx.x % L;
    const int gib = threadIdx.x / L;
    const int r = a.r;
    int32_t line, begin, end, chunk = -1;
    if ((int32_t)blockIdx.x < nb_chunk_blocks) {
        chunk = blockIdx.x * GPB + gib;
        if (chunk >= a.n_chunks) return;
        line = a.chunks[3 * chunk];
        begin = a.chunks[3 * chunk + 1];
        end = a.chunks[3 * chunk + 2];
    } else {
        const int32_t k = (blockIdx.x - nb_chunk_blocks) * GPB + gib;
        if (k >= a.nlines) return;
        line = a.order ? a.order[k] : k;
        begin = a.ptr[line];
        end = a.ptr[line + 1];
        if (a.n_chunks > 0 && end - begin > a.long_len) return;
    }
    RowVec<VW, RAG> rv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) rv[v] = RowVec<VW, RAG>(v * L + lane, r);
    const int32_t *__restrict__ idx = a.idx;
    const Acc *__restrict__ val = static_cast<const Acc *>(a.val);
    const Acc *__restrict__ tv = static_cast<const Acc *>(a.t);
    const TH *__restrict__ H = static_cast<const TH *>(a.H);
    const Acc si = static_cast<const Acc *>(a.s)[line];
    const Acc slope = Acc(a.slope);

    Acc acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = Acc(0);
    Acc m = neg_inf<Acc>(), l = Acc(0);

    // Column indices and edge values of the batch at p0; entries past `end` reread the
    // last entry, so every load is in bounds.
    auto load_meta = [&](int32_t p0, int32_t *j, Acc *sc) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t p = p0 + u;
            const int32_t pc = p < end ? p : end - 1;
            j[u] = idx[pc];
            sc[u] = val ? val[pc] : Acc(1);
        }
    };
    int32_t j[U], jn[U];
    Acc sc[U], scn[U];
    if (begin < end) load_meta(begin, j, sc);
    for (int32_t p0 = begin; p0 < end; p0 += U) {
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) ok[u] = p0 + u < end;
        Raw<TH, VW> g[U][NV];
        Acc tj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            tj[u] = tv[j[u]];
            if (ok[u]) {
#pragma unroll
                for (int v = 0; v < NV; ++v) g[u][v].load(H + (size_t)j[u] * r + rv[v].off);
            }
        }
        // the next batch's operands arrive while this batch waits for its rows
        if (p0 + U < end) load_meta(p0 + U, jn, scn);
        // LeakyReLU of the sampled score; entries past the end get weight 0 (softmax: -inf)
        Acc ev[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const Acc x = sc[u] * (si + tj[u]);
            ev[u] = x >= Acc(0) ? x : slope * x;
        }
        Acc w[U];
        if constexpr (SOFTMAX) {
            Acc mb = m;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (ok[u]) mb = ev[u] > mb ? ev[u] : mb;
            const Acc scale = exp_acc<Acc>(m - mb);  // m == -inf on the first batch: 0
            l *= scale;
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] *= scale;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                w[u] = ok[u] ? exp_acc<Acc>(ev[u] - mb) : Acc(0);
                l += w[u];
            }
            m = mb;
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = ok[u] ? ev[u] : Acc(0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!ok[u]) continue;
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int e = 0; e < VW; ++e) acc[v * VW + e] += w[u] * Acc(g[u][v].get(e));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            j[u] = jn[u];
            sc[u] = scn[u];
        }
    }

    Acc *dst;
    Acc inv = Acc(1);
    if (chunk >= 0) {
        dst = static_cast<Acc *>(a.partial) + (size_t)chunk * r;
        if (lane == 0) {
            Acc *ml = static_cast<Acc *>(a.partial) + (size_t)a.n_chunks * r + 2 * (size_t)chunk;
            ml[0] = m;
            ml[1] = l;
        }
    } else {
        dst = static_cast<Acc *>(a.out) + (size_t)line * r;
        if (SOFTMAX) inv = l > Acc(0) ? Acc(1) / l : Acc(0);
        if (SOFTMAX && a.lse && lane == 0)
            static_cast<Acc *>(a.lse)[line] = l > Acc(0) ? m + log_acc<Acc>(l) : Acc(0);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if (!rv[v].act) continue;
        Acc o[VW];
#pragma unroll
        for (int e = 0; e < VW; ++e) o[e] = acc[v * VW + e] * inv;
        rv[v].template store<kNtStore>(dst, o);
    }
}

// Combine the chunks of each split row: with M the largest chunk maximum and L = sum_c l_c
// exp(m_c - M), out = sum_c acc_c exp(m_c - M) / L and lse = M + log L.
template <class Acc> struct MergeSoftmax {
    Acc *out, *lse;
    const Acc *ml;  // (m, l) of every chunk
    int32_t r;
    struct State {
        Acc M, inv;
    };
    __device__ __forceinline__ State begin(int32_t line, int32_t first, int32_t cnt, bool writes) const {
        const int lane = threadIdx.x % 64;
        Acc M = neg_inf<Acc>(), L = Acc(0);
        for (int32_t c = lane; c < cnt; c += 64) {
            const Acc m = ml[2 * (size_t)(first + c)];
            M = m > M ? m : M;
        }
        M = wave_max(M);
        for (int32_t c = lane; c < cnt; c += 64)
            L += ml[2 * (size_t)(first + c) + 1] * exp_acc<Acc>(ml[2 * (size_t)(first + c)] - M);
        L = wave_sum(L);
        if (writes && lse && lane == 0) lse[line] = L > Acc(0) ? M + log_acc<Acc>(L) : Acc(0);
        return State{M, L > Acc(0) ? Acc(1) / L : Acc(0)};
    }
    __device__ __forceinline__ State begin_few(int32_t line, int32_t first, int32_t cnt, bool writes) const {
        Acc M = neg_inf<Acc>(), L = Acc(0);
        for (int32_t c = first; c < first + cnt; ++c) {
            const Acc m = ml[2 * (size_t)c];
            M = m > M ? m : M;
        }
        for (int32_t c = first; c < first + cnt; ++c) L += ml[2 * (size_t)c + 1] * exp_acc<Acc>(ml[2 * (size_t)c] - M);
        if (writes && lse) lse[line] = L > Acc(0) ? M + log_acc<Acc>(L) : Acc(0);
        return State{M, L > Acc(0) ? Acc(1) / L : Acc(0)};
    }
    __device__ __forceinline__ Acc weigh(const State &st, int32_t chunk, Acc x) const {
        return x * exp_acc<Acc>(ml[2 * (size_t)chunk] - st.M);
    }
    template <int VW> __device__ __forceinline__ void store(const State &st, int32_t line, int k, Acc *v) const {
#pragma unroll
        for (int e = 0; e < VW; ++e) v[e] *= st.inv;
        St<Acc, VW>::run(out + (size_t)line * r + k, v);
    }
};

template <class Acc>
hipError_t merge_rows(const fmm_sparse *S, int32_t r, bool softmax, const void *ws, void *out, void *lse, hipStream_t st)
{
    const Acc *partial = static_cast<const Acc *>(ws);
    if (softmax)
        return launch_merge<Acc>(S->splits, S->n_splits, S->n_chunks, r, partial,
                                 MergeSoftmax<Acc>{static_cast<Acc *>(out), static_cast<Acc *>(lse),
                                                   partial + (size_t)S->n_chunks * r, r}, st);
    return launch_merge<Acc>(S->splits, S->n_splits, S->n_chunks, r, partial,
                             MergePlain<Acc>{static_cast<Acc *>(out), 0.0, r}, st);
}

template <class TH, class Acc, int L, int NV, int VW, int U, bool RAG>
hipError_t launch_gat_shape(const GatArgs &a, bool softmax, hipStream_t st)
{
    constexpr int GPB = kBlock / L;
    const int64_t nbc = a.n_chunks > 0 ? ((int64_t)a.n_chunks + GPB - 1) / GPB : 0;
    const int64_t nbl = ((int64_t)a.nlines + GPB - 1) / GPB;
    if (nbc + nbl == 0) return hipSuccess;
    if (softmax)
        hipLaunchKernelGGL((gat_kernel<TH, Acc, L, NV, VW, U, true, RAG>), dim3((unsigned)(nbc + nbl)), dim3(kBlock), 0,
                           st, a, (int32_t)nbc);
    else
        hipLaunchKernelGGL((gat_kernel<TH, Acc, L, NV, VW, U, false, RAG>), dim3((unsigned)(nbc + nbl)), dim3(kBlock), 0,
                           st, a, (int32_t)nbc);
    return hipGetLastError();
}

template <class TH, class Acc, int L, int NV, int VW, bool RAG>
hipError_t launch_scores_shape(const TH *H, int32_t n, int32_t r, const Acc *a1, const Acc *a2, Acc *s, Acc *t,
                               hipStream_t st)
{
    constexpr int RPB = kBlock / L * kScoreRows;
    const int64_t nb = ((int64_t)n + RPB - 1) / RPB;
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL((gat_scores_kernel<TH, Acc, L, NV, VW, RAG>), dim3((unsigned)nb), dim3(kBlock), 0, st, H, n, r, a1,
                       a2, s, t, (size_t)n * r * sizeof(TH) > kStreamBytes);
    return hipGetLastError();
}

// With one element per lane (see vector_rows) the first five cover every r.
#define GAT_SHAPES(X)                                                                            \
    X(1, 1) X(2, 1) X(4, 1) X(8, 1) X(16, 1)                                                     \
    if constexpr (VW > 1) { X(32, 1) X(64, 1) X(64, 2) X(64, 4) }

template <class TH, class Acc, int VW, bool RAG = false>
hipError_t dispatch_gat(const GatArgs &a, Shape sh, bool softmax, int uclass, hipStream_t st)
{
#define GAT_CASE(Lv, NVv)                                                                        \
    if (sh.L == Lv && sh.NV == NVv) {                                                            \
        if (uclass == 1) return launch_gat_shape<TH, Acc, Lv, NVv, VW, (8 / NVv > 0 ? 8 / NVv : 1), RAG>(a, softmax, st); \
        return launch_gat_shape<TH, Acc, Lv, NVv, VW, (4 / NVv > 0 ? 4 / NVv : 1), RAG>(a, softmax, st);                   \
    }
    GAT_SHAPES(GAT_CASE)
#undef GAT_CASE
    return hipErrorInvalidValue;
}

template <class TH, class Acc, int VW, bool RAG = false>
hipError_t dispatch_scores(const TH *H, int32_t n, int32_t r, const Acc *a1, const Acc *a2, Acc *s, Acc *t, Shape sh,
                           hipStream_t st)
{
#define SC_CASE(Lv, NVv)                                                                         \
    if (sh.L == Lv && sh.NV == NVv) return launch_scores_shape<TH, Acc, Lv, NVv, VW, RAG>(H, n, r, a1, a2, s, t, st);
    GAT_SHAPES(SC_CASE)
#undef SC_CASE
    return hipErrorInvalidValue;
}

// Shapes for the attention kernels: the default line shape, with NV = 2 rounded up to 4
// only where L = 64 (the compiled set above).
// Rows of whole 16-byte vectors, rows that end in an overlapping one, or element by element
// (vector_rows; for a training step on 2^17 x 2^17 R-MAT the line lies where it does for the
// line kernels: r = 13, 266 us in vectors and 244 by elements; r = 25, 275 and 350).  Up to 256
// lanes' worth of vectors, or 256 elements where r is no multiple of the vector.
enum RowForm { ROW_WHOLE, ROW_RAGGED, ROW_SHORT };
inline RowForm row_form(int r, int full)
{
    return r % full == 0 ? ROW_WHOLE : vector_rows(r, full) ? ROW_RAGGED : ROW_SHORT;
}
inline bool row_ok(int r, int full) { return r <= (r % full == 0 ? 256 * full : 256); }

Shape gat_shape(int r, int vw)
{
    Shape s = default_shape(r, vw);
    if (s.NV == 2 && s.L != 64) s = Shape{64, 1};
    return s;
}

template <class T, int VW>
hipError_t scores_rows(RowForm form, const void *H, int32_t n, int32_t r, const void *a1, const void *a2, void *s, void *t,
                       hipStream_t st)
{
    const T *h = (const T *)H, *x = (const T *)a1, *y = (const T *)a2;
    if (form == ROW_WHOLE) return dispatch_scores<T, T, VW>(h, n, r, x, y, (T *)s, (T *)t, gat_shape(r, VW), st);
    if (form == ROW_RAGGED) return dispatch_scores<T, T, VW, true>(h, n, r, x, y, (T *)s, (T *)t, gat_shape(r, VW), st);
    return dispatch_scores<T, T, 1>(h, n, r, x, y, (T *)s, (T *)t, gat_shape(r, 1), st);
}

template <class T, int VW> hipError_t gat_rows(RowForm form, const GatArgs &a, bool softmax, int uc, hipStream_t st)
{
    if (form == ROW_WHOLE) return dispatch_gat<T, T, VW>(a, gat_shape(a.r, VW), softmax, uc, st);
    if (form == ROW_RAGGED) return dispatch_gat<T, T, VW, true>(a, gat_shape(a.r, VW), softmax, uc, st);
    return dispatch_gat<T, T, 1>(a, gat_shape(a.r, 1), softmax, uc, st);
}

fmm_status hipfail(hipError_t e)
{
    set_last_hip_error((int32_t)e);
    return FMM_ERR_HIP;
}

int gat_uclass(const fmm_sparse *S)
{
    if (S->variant == FMM_VARIANT_DEEP) return 1;
    if (S->variant >= FMM_VARIANT_MEDIUM) return 2;
    const double mean = S->rows > 0 ? (double)S->nnz / S->rows : 0.0;
    return mean >= 24.0 ? 1 : 2;
}

}  // namespace
}  // namespace fmm

using namespace fmm;

extern "C" {

fmm_status fmm_gat_scores(const void *H, int32_t n, int32_t r, int32_t dtype, const void *a1, const void *a2, void *s,
                          void *t, hipStream_t stream)
{
    if (n < 0 || r < 1) return FMM_ERR_DIM;
    if (n > 0 && (!H || !s || !t)) return FMM_ERR_NULL;
    if (!a1 || !a2) return FMM_ERR_NULL;
    hipError_t e;
    if (dtype == FMM_F32) {
        const RowForm form = row_form(r, 4);
        if (!row_ok(r, 4)) return FMM_ERR_DTYPE;
        if (form == ROW_WHOLE && (uintptr_t)H % 16) return FMM_ERR_UNSUPPORTED;
        e = scores_rows<float, 4>(form, H, n, r, a1, a2, s, t, stream);
    } else if (dtype == FMM_BF16) {
        if (r % 8 != 0 || r > 1024) return FMM_ERR_DTYPE;
        if ((uintptr_t)H % 16) return FMM_ERR_UNSUPPORTED;
        e = dispatch_scores<bf16_t, float, 8>((const bf16_t *)H, n, r, (const float *)a1, (const float *)a2,
                                              (float *)s, (float *)t, gat_shape(r, 8), stream);
    } else if (dtype == FMM_F64) {
        const RowForm form = row_form(r, 2);
        if (!row_ok(r, 2)) return FMM_ERR_DTYPE;
        if (form == ROW_WHOLE && (uintptr_t)H % 16) return FMM_ERR_UNSUPPORTED;
        e = scores_rows<double, 2>(form, H, n, r, a1, a2, s, t, stream);
    } else {
        return FMM_ERR_DTYPE;
    }
    return e == hipSuccess ? FMM_OK : hipfail(e);
}

fmm_status fmm_gat_forward(const fmm_sparse *S, const void *s, const void *t, const void *H, int32_t r, int32_t dtype,
                           double negative_slope, int32_t flags, void *out, void *lse, void *ws, size_t ws_bytes,
                           hipStream_t stream)
{
    if (!S) return FMM_ERR_NULL;
    if (S->orient != FMM_CSR) return FMM_ERR_ORIENT;
    if (S->rows < 0 || S->rows != S->cols || S->nnz < 0 || r < 1) return FMM_ERR_DIM;
    if (!S->ptr || (S->nnz > 0 && !S->idx)) return FMM_ERR_NULL;
    if (S->rows > 0 && (!s || !t || !H || !out)) return FMM_ERR_NULL;
    if (flags & ~FMM_GAT_SOFTMAX) return FMM_ERR_DIM;
    if (S->n_chunks < 0 || S->n_splits < 0) return FMM_ERR_DIM;
    if (S->n_chunks > 0 && (!S->chunks || !S->splits || S->long_len < 1)) return FMM_ERR_NULL;
    const size_t ob = dtype == FMM_F64 ? 8 : 4;
    const size_t need = S->n_chunks > 0 ? (size_t)S->n_chunks * ((size_t)r + 2) * ob : 0;
    if (need && (!ws || ws_bytes < need || (uintptr_t)ws % 16)) return FMM_ERR_WORKSPACE;
    GatArgs a;
    memset(&a, 0, sizeof(a));
    a.nlines = S->rows;
    a.r = r;
    a.ptr = S->ptr;
    a.idx = S->idx;
    a.val = S->val;
    a.s = s;
    a.t = t;
    a.H = H;
    a.out = out;
    a.slope = negative_slope;
    a.long_len = S->long_len;
    a.n_chunks = S->n_chunks;
    a.chunks = S->chunks;
    a.order = S->order;
    a.partial = ws;
    a.lse = lse;
    const bool softmax = (flags & FMM_GAT_SOFTMAX) != 0;
    const int uc = gat_uclass(S);
    hipError_t e;
    if (dtype == FMM_F32) {
        const RowForm form = row_form(r, 4);
        if (!row_ok(r, 4)) return FMM_ERR_DTYPE;
        if (form == ROW_WHOLE && ((uintptr_t)H % 16 || (uintptr_t)out % 16)) return FMM_ERR_UNSUPPORTED;
        e = gat_rows<float, 4>(form, a, softmax, uc, stream);
    } else if (dtype == FMM_BF16) {
        if (r % 8 != 0 || r > 1024) return FMM_ERR_DTYPE;
        if ((uintptr_t)H % 16 || (uintptr_t)out % 16) return FMM_ERR_UNSUPPORTED;
        e = dispatch_gat<bf16_t, float, 8>(a, gat_shape(r, 8), softmax, uc, stream);
    } else if (dtype == FMM_F64) {
        const RowForm form = row_form(r, 2);
        if (!row_ok(r, 2)) return FMM_ERR_DTYPE;
        if (form == ROW_WHOLE && ((uintptr_t)H % 16 || (uintptr_t)out % 16)) return FMM_ERR_UNSUPPORTED;
        e = gat_rows<double, 2>(form, a, softmax, uc, stream);
    } else {
        return FMM_ERR_DTYPE;
    }
    if (e != hipSuccess) return hipfail(e);
    if (S->n_chunks > 0 && S->n_splits > 0) {
        e = dtype == FMM_F64 ? merge_rows<double>(S, r, softmax, ws, out, lse, stream)
                             : merge_rows<float>(S, r, softmax, ws, out, lse, stream);
        if (e != hipSuccess) return hipfail(e);
    }
    return FMM_OK;
}

fmm_status fmm_gat_workspace(const fmm_sparse *S, int32_t r, int32_t dtype, size_t *bytes)
{
    if (!S || !bytes) return FMM_ERR_NULL;
    if (r < 1) return FMM_ERR_DIM;
    if (dtype != FMM_F32 && dtype != FMM_BF16 && dtype != FMM_F64) return FMM_ERR_DTYPE;
    const size_t ob = dtype == FMM_F64 ? 8 : 4;
    *bytes = S->n_chunks > 0 ? (size_t)S->n_chunks * ((size_t)r + 2) * ob : 0;
    return FMM_OK;
}

fmm_status fmm_gat_edge_values(const fmm_sparse *S, const void *s, const void *t, int32_t dtype, double negative_slope,
                               int32_t flags, void *w, hipStream_t stream)
{
    if (!S) return FMM_ERR_NULL;
    if (S->orient != FMM_CSR) return FMM_ERR_ORIENT;
    if (S->rows < 0 || S->rows != S->cols || S->nnz < 0) return FMM_ERR_DIM;
    if (!S->ptr || (S->nnz > 0 && (!S->idx || !w))) return FMM_ERR_NULL;
    if (S->rows > 0 && (!s || !t)) return FMM_ERR_NULL;
    if (flags & ~FMM_GAT_SOFTMAX) return FMM_ERR_DIM;
    const bool softmax = (flags & FMM_GAT_SOFTMAX) != 0;
    constexpr int L = 16;
    const unsigned nb = (unsigned)(((int64_t)S->rows + kBlock / L - 1) / (kBlock / L));
    if (nb == 0) return FMM_OK;
    if (dtype == FMM_F64)
        hipLaunchKernelGGL((gat_edges_kernel<double, L>), dim3(nb), dim3(kBlock), 0, stream, S->rows, S->ptr, S->idx,
                           (const double *)S->val, (const double *)s, (const double *)t, negative_slope, softmax,
                           (double *)w);
    else if (dtype == FMM_F32 || dtype == FMM_BF16)
        hipLaunchKernelGGL((gat_edges_kernel<float, L>), dim3(nb), dim3(kBlock), 0, stream, S->rows, S->ptr, S->idx,
                           (const float *)S->val, (const float *)s, (const float *)t, (float)negative_slope, softmax,
                           (float *)w);
    else
        return FMM_ERR_DTYPE;
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FMM_OK : hipfail(e);
}

}  // extern "C"
