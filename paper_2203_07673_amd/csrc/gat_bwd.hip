// Adjoint of the graph-attention head (the forward is Section VI-E; its gradient follows
// from the definition by the chain rule).  With upstream gradient dO and the forward's
// scores s, t and output out:
//
//   x_ij = S_ij (s_i + t_j),  e = LeakyReLU(x),  w = e or exp(e_ij - lse_i) (row softmax)
//   dw_ij = <dO_i, H_j>
//   de_ij = dw_ij, or w_ij (dw_ij - D_i) with D_i = sum_j w_ij dw_ij = <dO_i, out_i>
//   dx_ij = de_ij (1 if x_ij > 0 else slope)
//   dS_ij = dx_ij (s_i + t_j),  ds_i = sum_j dx_ij S_ij,  dt_j = sum_i dx_ij S_ij
//   dH_j  = sum_i w_ij dO_i + ds_j a1 + dt_j a2,  da1 = H^T ds,  da2 = H^T dt
//
// dt and the sum over w dO need a column pass on the stored transpose that gathers dO_i and
// per-row scalars (held H_j); it recomputes the edge weight (from the forward's per-row
// log-sum-exp) and dw in registers like the fused adjoints.  ds sums the same dx over rows:
//
//   one gather  (1) D_i and the packed row scalars, (2) the column pass, which leaves every
//               entry's dx_ij S_ij at its CSR place (through perm), (3) the merge of split
//               columns, (4) per row ds_i from its entries, dH_i += ds_i a1 + dt_i a2, and the
//               blocks' sums of da1, da2, (5) their sum.
//   two gathers (1) a row pass that gathers H_j and recomputes dw for D_i, ds and dS, (2) the
//               column pass, which adds ds_j a1 + dt_j a2 as it stores dH_j, (3) merges, (4)
//               the blocks' sums of da1, da2, (5) their sum.
//
// No atomics anywhere.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <initializer_list>
#include <type_traits>

#include "fmm.h"
#include "fmm_internal.hpp"
#include "fmm_merge.hpp"

namespace fmm {
namespace {

template <class Acc> __device__ __forceinline__ Acc bexp(Acc x);
template <> __device__ __forceinline__ float bexp<float>(float x) { return expf(x); }
template <> __device__ __forceinline__ double bexp<double>(double x) { return exp(x); }

constexpr int kFinishBlocks = 2048;  // most blocks of the pass that sums da1 and da2

// The three per-row scalars the column pass gathers for every entry, packed so that one
// 16-byte (float) or 32-byte (double) load fetches them: s_i, lse_i, D_i.
template <class Acc> struct RowScalars;
template <> struct RowScalars<float> {
    float4 v;
    __device__ __forceinline__ void load(const void *base, int32_t i) { v = static_cast<const float4 *>(base)[i]; }
    static __device__ __forceinline__ void store(void *base, int32_t i, float s, float l, float d) {
        static_cast<float4 *>(base)[i] = make_float4(s, l, d, 0.f);
    }
    __device__ __forceinline__ float s() const { return v.x; }
    __device__ __forceinline__ float lse() const { return v.y; }
    __device__ __forceinline__ float D() const { return v.z; }
};
template <> struct RowScalars<double> {
    double2 a, b;
    __device__ __forceinline__ void load(const void *base, int32_t i) {
        a = static_cast<const double2 *>(base)[2 * i];
        b = static_cast<const double2 *>(base)[2 * i + 1];
    }
    static __device__ __forceinline__ void store(void *base, int32_t i, double s, double l, double d) {
        static_cast<double2 *>(base)[2 * i] = make_double2(s, l);
        static_cast<double2 *>(base)[2 * i + 1] = make_double2(d, 0.0);
    }
    __device__ __forceinline__ double s() const { return a.x; }
    __device__ __forceinline__ double lse() const { return a.y; }
    __device__ __forceinline__ double D() const { return b.x; }
};

struct GatBwdArgs {
    int32_t nlines, r;
    const int32_t *ptr, *idx;
    const void *val;          // S's values in this orientation (Acc), NULL = 1
    const void *s, *t;        // scores (Acc, per node)
    const void *lse;          // per row log-sum-exp from the forward (softmax; Acc)
    void *rs;                 // packed per-row (s_i, lse_i, D_i): written by the row pass, gathered by the column pass
    const void *out;          // forward output (row pass)
    const void *a1, *a2;      // attention vectors (column pass)
    const void *ds;           // ds from the row pass (column pass)
    const void *held;         // held matrix: dO (row pass, Acc) or H (column pass, TH)
    const void *gath;         // gathered matrix: H (row pass, TH) or dO (column pass, Acc)
    double slope;
    int32_t softmax;
    int32_t long_len, n_chunks;
    const int32_t *chunks;
    const int32_t *order;
    void *out_vec;            // column pass: sum_i w_ij dO_i per column (Acc, lines x r)
    int32_t out16;            // two gathers: out_vec is bfloat16
    void *out_sc;             // per-line scalar: ds (row pass) or dt (column pass)
    void *part_vec, *part_sc; // chunk partials
    void *dS;                 // dL/dS in CSR order (Acc), or NULL
    const int32_t *perm;      // column pass, one gather: CSR place of each entry
    void *dxs;                // and dx_ij S_ij of every entry, in CSR order
};

// Line (or chunk) of this lane group, as in the forward kernels.  Returns false when the
// group has no work.
__device__ __forceinline__ bool pick_line(const GatBwdArgs &a, int32_t nb_chunk_blocks, int gpb, int gib,
                                          int32_t &line, int32_t &begin, int32_t &end, int32_t &chunk)
{
    chunk = -1;
    if ((int32_t)blockIdx.x < nb_chunk_blocks) {
        chunk = blockIdx.x * gpb + gib;
        if (chunk >= a.n_chunks) return false;
        line = a.chunks[3 * chunk];
        begin = a.chunks[3 * chunk + 1];
        end = a.chunks[3 * chunk + 2];
        return true;
    }
    const int32_t k = (blockIdx.x - nb_chunk_blocks) * gpb + gib;
    if (k >= a.nlines) return false;
    line = a.order ? a.order[k] : k;
    begin = a.ptr[line];
    end = a.ptr[line + 1];
    return !(a.n_chunks > 0 && end - begin > a.long_len);
}

// Indices and stored values of the batch at p0 (entries past `end` reread the last one).
template <class Acc, int U>
__device__ __forceinline__ void load_entries(const int32_t *__restrict__ idx, const Acc *__restrict__ val, int32_t p0,
                                             int32_t end, int32_t *j, Acc *v)
{
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int32_t pc = p0 + u < end ? p0 + u : end - 1;
        j[u] = idx[pc];
        v[u] = val ? val[pc] : Acc(1);
    }
}

// Per-entry backward scalars from the recomputed forward values.
template <class Acc>
__device__ __forceinline__ void entry_grad(Acc v, Acc score, Acc lse_i, Acc D_i, Acc dw, Acc slope, bool softmax,
                                           Acc &w, Acc &dx)
{
    const Acc x = v * score;
    const Acc e = x >= Acc(0) ? x : slope * x;
    w = softmax ? bexp<Acc>(e - lse_i) : e;
    const Acc de = softmax ? w * (dw - D_i) : dw;
    dx = de * (x > Acc(0) ? Acc(1) : slope);
}

// (1) of the one-gather form: D_i = <dO_i, out_i> (= sum_j w_ij dw_ij) and the packed scalars
// of every row.  A lane group takes kDotRows rows, whose loads are in flight together: 2^20 rows
// of r = 128 in 170 us, 6.3 TB/s.
constexpr int kDotRows = 4;
template <class TO, class Acc, int L, int NV, int VW, bool RAG>
__global__ __launch_bounds__(kBlock) void gat_bwd_dots_kernel(int32_t n, int32_t r, const TO *__restrict__ dO,
                                                              const Acc *__restrict__ out, const Acc *__restrict__ s,
                                                              const Acc *__restrict__ lse, bool softmax,
                                                              void *__restrict__ rs)
{
    constexpr int GPB = kBlock / L;
    const int lane = threadIdx.x % L;
    const int64_t row0 = (int64_t)blockIdx.x * (GPB * kDotRows) + threadIdx.x / L;
    if (!softmax) {  // D is not used
        if (lane == 0)
            for (int u = 0; u < kDotRows; ++u)
                if (row0 + u * GPB < n) RowScalars<Acc>::store(rs, (int32_t)(row0 + u * GPB), s[row0 + u * GPB], Acc(0), Acc(0));
        return;
    }
    RowVec<VW, RAG> rv[NV];
    Raw<TO, VW> x[kDotRows][NV];
    Acc y[kDotRows][NV * VW];
#pragma unroll
    for (int v = 0; v < NV; ++v) rv[v] = RowVec<VW, RAG>(v * L + lane, r);
#pragma unroll
    for (int u = 0; u < kDotRows; ++u) {
        const int64_t row = min(row0 + u * GPB, (int64_t)n - 1);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            x[u][v].load(dO + row * r + rv[v].off);
            Ld<Acc, VW, Acc>::template run<true>(out + row * r + rv[v].off, y[u] + v * VW);
        }
    }
#pragma unroll
    for (int u = 0; u < kDotRows; ++u) {
        Acc d = Acc(0);
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int e = 0; e < VW; ++e)
                if (rv[v].act && (!RAG || e >= rv[v].rep)) d += Acc(x[u][v].get(e)) * y[u][v * VW + e];
        d = group_sum<L>(d);
        const int64_t row = row0 + u * GPB;
        if (lane == 0 && row < n) RowScalars<Acc>::store(rs, (int32_t)row, s[row], lse[row], d);
    }
}

// (1) of the two-gather form, on S_csr: held dO_i (stored as TO), gathered H_j.  D_i, ds_i =
// sum_j dx_ij S_ij and dS_ij.
template <class TH, class TO, class Acc, int L, int NV, int VW, int U, bool RAG>
__global__ __launch_bounds__(kBlock) void gat_bwd_rows_kernel(GatBwdArgs a, int32_t nb_chunk_blocks)
{
    constexpr int GPB = kBlock / L;
    constexpr int E = NV * VW;
    const int lane = threadIdx.x % L;
    int32_t line, begin, end, chunk;
    if (!pick_line(a, nb_chunk_blocks, GPB, threadIdx.x / L, line, begin, end, chunk)) return;
    const int r = a.r;
    const TO *dO = static_cast<const TO *>(a.held);
    const TH *H = static_cast<const TH *>(a.gath);
    const Acc *val = static_cast<const Acc *>(a.val);
    const Acc *t = static_cast<const Acc *>(a.t);
    const Acc *out = static_cast<const Acc *>(a.out);
    const Acc si = static_cast<const Acc *>(a.s)[line];
    const bool softmax = a.softmax != 0;
    const Acc lse_i = softmax ? static_cast<const Acc *>(a.lse)[line] : Acc(0);
    const Acc slope = Acc(a.slope);
    Acc *dS = static_cast<Acc *>(a.dS);
    RowVec<VW, RAG> rv[NV];
    Acc hd[E];
    Acc dd = Acc(0);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        rv[v] = RowVec<VW, RAG>(v * L + lane, r);
        Raw<TO, VW> x;
        Raw<Acc, VW> y;
        if (rv[v].act) {
            x.load(dO + (size_t)line * r + rv[v].off);
            y.load(out + (size_t)line * r + rv[v].off);
            if constexpr (RAG) {
                x.drop(rv[v].rep);
                y.drop(rv[v].rep);
            }
        } else {
            x.zero();
            y.zero();
        }
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            hd[v * VW + e] = Acc(x.get(e));
            dd += Acc(x.get(e)) * Acc(y.get(e));
        }
    }
    // D_i = <dO_i, out_i> (= sum_j w_ij dw_ij); every chunk of a split row writes the same bits
    const Acc D_i = group_sum<L>(dd);
    if (lane == 0) RowScalars<Acc>::store(a.rs, line, si, lse_i, D_i);
    Acc dsum = Acc(0);
    // indices and values of the next batch are loaded while this batch's rows arrive
    int32_t j[U], jn[U];
    Acc v[U], vn[U];
    if (begin < end) load_entries<Acc, U>(a.idx, val, begin, end, j, v);
    for (int32_t p0 = begin; p0 < end; p0 += U) {
        bool ok[U];
        Acc tj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) ok[u] = p0 + u < end;
        Raw<TH, VW> g[U][NV];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            tj[u] = t[j[u]];
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                if (ok[u] && rv[q].act) g[u][q].load(H + (size_t)j[u] * r + rv[q].off);
                else g[u][q].zero();
            }
        }
        if (p0 + U < end) load_entries<Acc, U>(a.idx, val, p0 + U, end, jn, vn);
        if constexpr (RAG) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < NV; ++q) g[u][q].drop(rv[q].rep);
        }
        Acc dw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            Acc x = Acc(0);
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int e = 0; e < VW; ++e) x += hd[q * VW + e] * Acc(g[u][q].get(e));
            dw[u] = group_sum<L>(x);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!ok[u]) continue;
            const Acc score = si + tj[u];
            Acc w, dx;
            entry_grad<Acc>(v[u], score, lse_i, D_i, dw[u], slope, softmax, w, dx);
            dsum += dx * v[u];
            if (dS && lane == (u % L)) dS[p0 + u] = dx * score;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            j[u] = jn[u];
            v[u] = vn[u];
        }
    }
    if (lane == 0) {
        if (chunk >= 0) static_cast<Acc *>(a.part_sc)[chunk] = dsum;
        else static_cast<Acc *>(a.out_sc)[line] = dsum;
    }
}

// (2) Column pass on the stored transpose: held H_j, gathered dO_i (stored as TO) and the row
// scalars.  dt_j = sum_i dx_ij S_ij and sum_i w_ij dO_i.  SCATTER (one gather): dx_ij S_ij, and
// dS_ij where asked for, go to the entry's CSR place; lane u of the group writes entry u of a
// batch, whose place it loads with the batch's rows.
template <class TH, class TO, class Acc, int L, int NV, int VW, int U, bool RAG, bool SCATTER>
__global__ __launch_bounds__(kBlock) void gat_bwd_cols_kernel(GatBwdArgs a, int32_t nb_chunk_blocks)
{
    constexpr int GPB = kBlock / L;
    constexpr int E = NV * VW;
    constexpr bool kBf16 = std::is_same<TH, bf16_t>::value;
    const int lane = threadIdx.x % L;
    int32_t line, begin, end, chunk;
    if (!pick_line(a, nb_chunk_blocks, GPB, threadIdx.x / L, line, begin, end, chunk)) return;
    const int r = a.r;
    const TH *H = static_cast<const TH *>(a.held);
    const TO *dO = static_cast<const TO *>(a.gath);
    const Acc *val = static_cast<const Acc *>(a.val);
    const Acc tj = static_cast<const Acc *>(a.t)[line];
    const Acc slope = Acc(a.slope);
    const bool softmax = a.softmax != 0;
    RowVec<VW, RAG> rv[NV];
    Acc hh[E], acc[E];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        rv[v] = RowVec<VW, RAG>(v * L + lane, r);
        Raw<TH, VW> x;
        if (rv[v].act) {
            x.load(H + (size_t)line * r + rv[v].off);
            if constexpr (RAG) x.drop(rv[v].rep);
        } else {
            x.zero();
        }
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            hh[v * VW + e] = Acc(x.get(e));
            acc[v * VW + e] = Acc(0);
        }
    }
    Acc dtsum = Acc(0);
    constexpr int PU = (U + L - 1) / L;  // entries of a batch that a lane writes
    int32_t i[U], in_[U];
    Acc v[U], vn[U];
    if (begin < end) load_entries<Acc, U>(a.idx, val, begin, end, i, v);
    for (int32_t p0 = begin; p0 < end; p0 += U) {
        bool ok[U];
        RowScalars<Acc> rsc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) ok[u] = p0 + u < end;
        Raw<TO, VW> g[U][NV];
        int32_t place[PU];
        if constexpr (SCATTER) {
#pragma unroll
            for (int k = 0; k < PU; ++k) {
                const int32_t p = p0 + k * L + lane;
                place[k] = k * L + lane < U && p < end ? a.perm[p] : -1;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            rsc[u].load(a.rs, i[u]);
#pragma unroll
            for (int q = 0; q < NV; ++q) {
                if (ok[u] && rv[q].act) g[u][q].load(dO + (size_t)i[u] * r + rv[q].off);
                else g[u][q].zero();
            }
        }
        if (p0 + U < end) load_entries<Acc, U>(a.idx, val, p0 + U, end, in_, vn);
        if constexpr (RAG) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < NV; ++q) g[u][q].drop(rv[q].rep);
        }
        Acc dw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            Acc x = Acc(0);
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int e = 0; e < VW; ++e) x += hh[q * VW + e] * Acc(g[u][q].get(e));
            dw[u] = group_sum<L>(x);
        }
        Acc dxs[PU], ds_e[PU];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!ok[u]) continue;
            Acc w, dx;
            entry_grad<Acc>(v[u], rsc[u].s() + tj, rsc[u].lse(), rsc[u].D(), dw[u], slope, softmax, w, dx);
            const Acc x = dx * v[u];
            dtsum += x;
            if constexpr (SCATTER) {
                dxs[u / L] = u % L == 0 || lane == u % L ? x : dxs[u / L];
                ds_e[u / L] = u % L == 0 || lane == u % L ? dx * (rsc[u].s() + tj) : ds_e[u / L];
            }
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
                for (int e = 0; e < VW; ++e) acc[q * VW + e] += w * Acc(g[u][q].get(e));
        }
        if constexpr (SCATTER) {
#pragma unroll
            for (int k = 0; k < PU; ++k) {
                if (place[k] < 0) continue;
                static_cast<Acc *>(a.dxs)[place[k]] = dxs[k];
                if (a.dS) static_cast<Acc *>(a.dS)[place[k]] = ds_e[k];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            i[u] = in_[u];
            v[u] = vn[u];
        }
    }
    Acc *dst;
    if (chunk >= 0) {
        dst = static_cast<Acc *>(a.part_vec) + (size_t)chunk * r;
    } else if constexpr (SCATTER) {
        dst = static_cast<Acc *>(a.out_vec) + (size_t)line * r;
    } else {  // a whole column: add the rank-one terms ds_j a1 + dt_j a2 here
        dst = static_cast<Acc *>(a.out_vec) + (size_t)line * r;
        const Acc dsj = static_cast<const Acc *>(a.ds)[line];
        const Acc *a1 = static_cast<const Acc *>(a.a1);
        const Acc *a2 = static_cast<const Acc *>(a.a2);
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (rv[v].act)
#pragma unroll
                for (int e = 0; e < VW; ++e)
                    acc[v * VW + e] += dsj * a1[rv[v].off + e] + dtsum * a2[rv[v].off + e];
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if (!rv[v].act) continue;
        if constexpr (kBf16 && !SCATTER) {
            if (a.out16 && chunk < 0) {
                st_bf16<VW>(static_cast<bf16_t *>(a.out_vec) + (size_t)line * r + rv[v].off, acc + v * VW);
                continue;
            }
        }
        rv[v].template store<kNtStore>(dst, acc + v * VW);
    }
    if (lane == 0) {
        if (chunk >= 0) static_cast<Acc *>(a.part_sc)[chunk] = dtsum;
        else static_cast<Acc *>(a.out_sc)[line] = dtsum;
    }
}

// (3) Merge of the split columns: dt_j and sum_i w_ij dO_i, plus the rank-one terms where ds is
// known (two gathers).
template <class Acc> struct MergeColumns {
    Acc *dH, *dt;
    const Acc *part_sc;              // dt of every chunk
    const Acc *ds, *a1, *a2;         // ds NULL: no rank-one terms yet
    int32_t r;
    bool out16;                      // dH is bfloat16 (r a multiple of 8)
    struct State {
        Acc ds, dt;
    };
    __device__ __forceinline__ State begin(int32_t line, int32_t first, int32_t cnt, bool writes) const {
        const int lane = threadIdx.x % 64;
        Acc x = Acc(0);
        for (int32_t c = lane; c < cnt; c += 64) x += part_sc[first + c];
        x = wave_sum(x);
        if (writes && lane == 0) dt[line] = x;
        return State{ds ? ds[line] : Acc(0), x};
    }
    __device__ __forceinline__ State begin_few(int32_t line, int32_t first, int32_t cnt, bool writes) const {
        Acc x = Acc(0);
        for (int32_t c = first; c < first + cnt; ++c) x += part_sc[c];
        if (writes) dt[line] = x;
        return State{ds ? ds[line] : Acc(0), x};
    }
    __device__ __forceinline__ Acc weigh(const State &, int32_t, Acc x) const { return x; }
    template <int VW> __device__ __forceinline__ void store(const State &st, int32_t line, int k, Acc *v) const {
        if (ds) {
#pragma unroll
            for (int e = 0; e < VW; ++e) v[e] += st.ds * a1[k + e] + st.dt * a2[k + e];
        }
        if constexpr (VW == 4) {
            if (out16) {
                st_bf16<VW>(reinterpret_cast<bf16_t *>(dH) + (size_t)line * r + k, v);
                return;
            }
        }
        St<Acc, VW>::run(dH + (size_t)line * r + k, v);
    }
};

// (4) of the one-gather form, split rows: ds_i from the row's entries, a wave for a row of up to
// kLongRow of them and the block for a longer one.
constexpr int32_t kLongRow = 2048;
template <class Acc>
__global__ __launch_bounds__(kBlock) void gat_bwd_long_rows_kernel(const int32_t *__restrict__ splits, int32_t n_splits,
                                                                   const int32_t *__restrict__ ptr,
                                                                   const Acc *__restrict__ dxs, Acc *__restrict__ ds)
{
    constexpr int W = kBlock / 64;
    static_assert(W == 4, "the waves are added as two pairs");
    __shared__ Acc red[W];
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    auto sum = [&](int32_t b, int32_t e, int32_t t, int32_t step) {
        Acc x = Acc(0);
        int32_t p = b + t;
        for (; p + 3 * step < e; p += 4 * step) {
            Acc y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) y[u] = dxs[p + u * step];
#pragma unroll
            for (int u = 0; u < 4; ++u) x += y[u];
        }
        for (; p < e; p += step) x += dxs[p];
        return wave_sum(x);
    };
    const int32_t s0 = (int32_t)blockIdx.x * W;
    if (s0 + w < n_splits) {
        const int32_t line = splits[3 * (s0 + w)];
        const int32_t b = ptr[line], e = ptr[line + 1];
        if (e - b <= kLongRow) {
            const Acc x = sum(b, e, lane, 64);
            if (lane == 0) ds[line] = x;
        }
    }
    for (int i = 0; i < W && s0 + i < n_splits; ++i) {  // the same for the whole block
        const int32_t line = splits[3 * (s0 + i)];
        const int32_t b = ptr[line], e = ptr[line + 1];
        if (e - b <= kLongRow) continue;
        const Acc x = sum(b, e, threadIdx.x, kBlock);
        if (lane == 0) red[w] = x;
        __syncthreads();
        if (threadIdx.x == 0) ds[line] = (red[0] + red[1]) + (red[2] + red[3]);
        __syncthreads();
    }
}

struct GatFinishArgs {
    int32_t n, r, rows_per_block;
    const int32_t *ptr;       // S_csr's, and its long_len where it has a split schedule
    int32_t long_len;
    const void *dxs;          // one gather: dx_ij S_ij in CSR order
    const void *ds, *dt;      // ds of the split rows (one gather) or of every row
    const void *H, *a1, *a2;
    const void *dHp;          // one gather: sum_i w_ij dO_i (Acc), may be dH
    void *dH, *part;
    int32_t out16;            // dH is bfloat16
};

// (4) The blocks' sums of ds_j H_j and dt_j H_j.  UPDATE (one gather): ds_j is summed here from
// the row's entries, and dH_j += ds_j a1 + dt_j a2.  A lane group takes every GPB-th row of
// the block's range; the groups' sums are added in a fixed tree.  Bound by memory: 2^20 rows
// of r = 128 move 1.6 GB in 362 us (0.5 GB without UPDATE).  For da1 and da2 alone a block
// took 512 rows, one thread a column: six blocks for 3000 rows, 20 us; 4 us now.
template <class TH, class Acc, int L, int NV, int VW, bool RAG, bool UPDATE>
__global__ __launch_bounds__(kBlock) void gat_bwd_finish_kernel(GatFinishArgs a)
{
    constexpr int GPB = kBlock / L, E = NV * VW, W = kBlock / 64;
    __shared__ Acc red[W][2][L * E];
    const int lane = threadIdx.x % L;
    const int r = a.r;
    const TH *H = static_cast<const TH *>(a.H);
    const Acc *dxs = static_cast<const Acc *>(a.dxs), *ds = static_cast<const Acc *>(a.ds);
    const Acc *dt = static_cast<const Acc *>(a.dt);
    const Acc *dHp = static_cast<const Acc *>(a.dHp);
    constexpr bool kBf16 = std::is_same<TH, bf16_t>::value;
    RowVec<VW, RAG> rv[NV];
    Acc a1[UPDATE ? E : 1], a2[UPDATE ? E : 1];
    Acc p1[E], p2[E];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        rv[v] = RowVec<VW, RAG>(v * L + lane, r);
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            if constexpr (UPDATE) {
                a1[v * VW + e] = static_cast<const Acc *>(a.a1)[rv[v].off + e];
                a2[v * VW + e] = static_cast<const Acc *>(a.a2)[rv[v].off + e];
            }
            p1[v * VW + e] = p2[v * VW + e] = Acc(0);
        }
    }
    const int64_t r1 = min((int64_t)a.n, (int64_t)(blockIdx.x + 1) * a.rows_per_block);
    int64_t j = (int64_t)blockIdx.x * a.rows_per_block + threadIdx.x / L;
    int32_t b = 0, e = 0;
    if (UPDATE && j < r1) {
        b = a.ptr[j];
        e = a.ptr[j + 1];
    }
    for (; j < r1; j += GPB) {
        Raw<TH, VW> h[NV];
        Acc out[NV][VW];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            h[v].load(H + j * r + rv[v].off);
            if constexpr (UPDATE) Ld<Acc, VW, Acc>::run(dHp + j * r + rv[v].off, out[v]);
        }
        const Acc dtj = dt[j];
        Acc dsj;
        if constexpr (UPDATE) {
            const int32_t p0 = b, p1e = e;
            if (j + GPB < r1) {  // the next row's entries
                b = a.ptr[j + GPB];
                e = a.ptr[j + GPB + 1];
            }
            if (p1e - p0 > a.long_len) {
                dsj = ds[j];
            } else {
                Acc x = Acc(0);
                for (int32_t p = p0 + lane; p < p1e; p += L) x += dxs[p];
                dsj = group_sum<L>(x);
            }
        } else {
            dsj = ds[j];
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
#pragma unroll
            for (int q = 0; q < VW; ++q) {
                const Acc x = Acc(h[v].get(q));
                p1[v * VW + q] += dsj * x;
                p2[v * VW + q] += dtj * x;
                if constexpr (UPDATE) out[v][q] += dsj * a1[v * VW + q] + dtj * a2[v * VW + q];
            }
            if constexpr (UPDATE) {
                if (!rv[v].act) continue;
                if constexpr (kBf16) {
                    if (a.out16) {
                        st_bf16<VW>(static_cast<bf16_t *>(a.dH) + j * r + rv[v].off, out[v]);
                        continue;
                    }
                }
                rv[v].template store<true>(static_cast<Acc *>(a.dH) + j * r, out[v]);
            }
        }
    }
    // groups of a wave, then waves
#pragma unroll
    for (int k = 0; k < E; ++k) {
        for (int d = L; d < 64; d <<= 1) {
            p1[k] += __shfl_xor(p1[k], d, 64);
            p2[k] += __shfl_xor(p2[k], d, 64);
        }
    }
    const int w = threadIdx.x / 64;
    if (threadIdx.x % 64 < L) {
#pragma unroll
        for (int k = 0; k < E; ++k) {
            red[w][0][k * L + lane] = p1[k];
            red[w][1][k * L + lane] = p2[k];
        }
    }
    __syncthreads();
    if (threadIdx.x >= 2 * L) return;
    const int which = threadIdx.x / L;
    Acc *part = static_cast<Acc *>(a.part) + (size_t)blockIdx.x * 2 * r + which * r;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        if (!rv[v].act) continue;
#pragma unroll
        for (int q = 0; q < VW; ++q) {
            const int k = (v * VW + q) * L + lane;
            if (!RAG || q >= rv[v].rep)
                part[rv[v].off + q] = (red[0][which][k] + red[1][which][k]) + (red[2][which][k] + red[3][which][k]);
        }
    }
}

// (5) da1 = sum_b part[b][0:r], da2 = sum_b part[b][r:2r]: 32 columns a block, every 32nd
// partial in one thread, their sums in order.
template <class Acc>
__global__ __launch_bounds__(1024) void gat_bwd_reduce_kernel(int32_t nb, int32_t r, const Acc *__restrict__ part,
                                                              Acc *__restrict__ da1, Acc *__restrict__ da2)
{
    __shared__ Acc red[32][33];
    const int c = threadIdx.x % 32, g = threadIdx.x / 32;
    const int k = blockIdx.x * 32 + c;
    Acc sum = Acc(0);
    if (k < 2 * r) {
        int32_t b = g;
        for (; b + 96 < nb; b += 128) {
            Acc x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = part[(size_t)(b + 32 * u) * 2 * r + k];
#pragma unroll
            for (int u = 0; u < 4; ++u) sum += x[u];
        }
        for (; b < nb; b += 32) sum += part[(size_t)b * 2 * r + k];
    }
    red[g][c] = sum;
    __syncthreads();
    if (g != 0 || k >= 2 * r) return;
    sum = Acc(0);
    for (int q = 0; q < 32; ++q) sum += red[q][c];
    if (k < r) da1[k] = sum;
    else da2[k - r] = sum;
}

inline size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

struct BwdLayout {
    size_t rs, ds, dt, dxs, dh, psc_r, pvec_c, psc_c, pblk, total;
};

// Whether the backward gathers once: it needs the entries' CSR places, and has to save more
// than it costs.  It saves the gather of a row of H per entry (r elements of hb bytes).  It
// costs a scattered store per entry, about 192 bytes' worth of that gather, and reading and
// writing dH once more.  A training step on R-MAT scale 20, 16 per row, one head, once / twice:
// float32 r = 32 1535 / 1382 us, r = 64 2237 / 2331, r = 128 3900 / 4650; bfloat16 r = 64 2034 /
// 1814, r = 128 3284 / 3248.
bool one_gather(const fmm_sparse *S_csc, int32_t r, size_t hb, size_t ob)
{
    if (S_csc->perm == nullptr) return false;
    return ((double)r * hb - 192.0) * S_csc->nnz > 2.0 * ob * r * S_csc->rows;
}

BwdLayout bwd_layout(const fmm_sparse *S_csr, const fmm_sparse *S_csc, int32_t r, size_t hb, size_t ob)
{
    const int64_t n = S_csr->rows;
    const int64_t ncr = S_csr->n_chunks > 0 ? S_csr->n_chunks : 0;
    const int64_t ncc = S_csc->n_chunks > 0 ? S_csc->n_chunks : 0;
    const bool once = one_gather(S_csc, r, hb, ob);
    BwdLayout l;
    size_t o = 0;
    l.rs = o; o += al256((size_t)n * 4 * ob);
    l.ds = o; o += al256((size_t)n * ob);
    l.dt = o; o += al256((size_t)n * ob);
    l.dxs = o; o += once ? al256((size_t)S_csr->nnz * ob) : 0;
    l.dh = o; o += once && hb < ob ? al256((size_t)n * r * ob) : 0;  // dH before it is rounded to bfloat16
    l.psc_r = o; o += once ? 0 : al256((size_t)ncr * ob);
    l.pvec_c = o; o += al256((size_t)ncc * r * ob);
    l.psc_c = o; o += al256((size_t)ncc * ob);
    l.pblk = o; o += al256((size_t)(n < kFinishBlocks ? n : kFinishBlocks) * 2 * r * ob);
    l.total = o + 256;
    return l;
}

Shape bwd_shape(int r, int vw)
{
    Shape s = default_shape(r, vw);
    if (s.NV == 2 && s.L != 64) s = Shape{64, 1};
    return s;
}

template <class TH, class TO, class Acc, int L, int NV, int VW, bool RAG>
hipError_t run_bwd_shape(const fmm_sparse *S_csr, const fmm_sparse *S_csc, const TH *H, const Acc *a1, const Acc *a2,
                         const Acc *s, const Acc *t, const Acc *out, const Acc *lse, const TO *dO, int32_t r,
                         Acc slope, bool softmax, void *dH, bool out16, Acc *da1, Acc *da2, Acc *dS, char *ws, hipStream_t st)
{
    constexpr int GPB = kBlock / L;
    constexpr int UR = NV == 1 ? 8 : 4;  // batch depth of the row pass
    constexpr int UC = NV == 1 ? 4 : 2;  // and of the column pass (more live registers per entry)
    const int32_t n = S_csr->rows;
    const BwdLayout lay = bwd_layout(S_csr, S_csc, r, sizeof(TH), sizeof(Acc));
    void *rsb = ws + lay.rs;
    Acc *ds = reinterpret_cast<Acc *>(ws + lay.ds);
    Acc *dt = reinterpret_cast<Acc *>(ws + lay.dt);
    hipError_t e;
    const dim3 reduce_grid((unsigned)((2 * r + 31) / 32));
    if (n == 0) {  // da1 = da2 = 0
        hipLaunchKernelGGL((gat_bwd_reduce_kernel<Acc>), reduce_grid, dim3(1024), 0, st, 0, r, (const Acc *)nullptr, da1,
                           da2);
        return hipGetLastError();
    }
    const unsigned nb_rows = (unsigned)(((int64_t)n + GPB - 1) / GPB);
    const bool once = one_gather(S_csc, r, sizeof(TH), sizeof(Acc));
    const bool split_rows = S_csr->n_chunks > 0 && S_csr->n_splits > 0;

    GatBwdArgs a;
    memset(&a, 0, sizeof(a));
    a.r = r;
    a.s = s;
    a.t = t;
    a.lse = lse;
    a.rs = rsb;
    a.slope = (double)slope;
    a.softmax = softmax ? 1 : 0;
    a.nlines = n;
    a.dS = dS;
    int64_t nbc = 0;
    if (once) {
        hipLaunchKernelGGL((gat_bwd_dots_kernel<TO, Acc, L, NV, VW, RAG>), dim3((nb_rows + kDotRows - 1) / kDotRows),
                           dim3(kBlock), 0, st, n, r, dO, out, s, lse, softmax, rsb);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else {
        a.ptr = S_csr->ptr;
        a.idx = S_csr->idx;
        a.val = S_csr->val;
        a.held = dO;
        a.gath = H;
        a.out = out;
        a.long_len = S_csr->long_len;
        a.n_chunks = S_csr->n_chunks;
        a.chunks = S_csr->chunks;
        a.order = S_csr->order;
        a.out_sc = ds;
        a.part_sc = ws + lay.psc_r;
        nbc = a.n_chunks > 0 ? ((int64_t)a.n_chunks + GPB - 1) / GPB : 0;
        hipLaunchKernelGGL((gat_bwd_rows_kernel<TH, TO, Acc, L, NV, VW, UR, RAG>), dim3((unsigned)(nbc + nb_rows)),
                           dim3(kBlock), 0, st, a, (int32_t)nbc);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (split_rows) {
            e = launch_merge<Acc>(S_csr->splits, S_csr->n_splits, S_csr->n_chunks, 1, static_cast<const Acc *>(a.part_sc),
                                  MergePlain<Acc>{ds, 0.0, 1}, st);
            if (e != hipSuccess) return e;
        }
        a.dS = nullptr;
    }
    // the column pass
    a.ptr = S_csc->ptr;
    a.idx = S_csc->idx;
    a.val = S_csc->val;
    a.held = H;
    a.gath = dO;
    a.out = nullptr;
    a.a1 = a1;
    a.a2 = a2;
    a.ds = ds;
    a.long_len = S_csc->long_len;
    a.n_chunks = S_csc->n_chunks;
    a.chunks = S_csc->chunks;
    a.order = S_csc->order;
    void *sums = once && out16 ? static_cast<void *>(ws + lay.dh) : dH;  // where the column pass and its merge write
    a.out_vec = sums;
    a.out16 = out16 ? 1 : 0;
    a.out_sc = dt;
    a.part_vec = ws + lay.pvec_c;
    a.part_sc = ws + lay.psc_c;
    a.perm = S_csc->perm;
    a.dxs = ws + lay.dxs;
    nbc = a.n_chunks > 0 ? ((int64_t)a.n_chunks + GPB - 1) / GPB : 0;
    const dim3 col_grid((unsigned)(nbc + nb_rows));
    if (once)
        hipLaunchKernelGGL((gat_bwd_cols_kernel<TH, TO, Acc, L, NV, VW, UC, RAG, true>), col_grid, dim3(kBlock), 0, st, a,
                           (int32_t)nbc);
    else
        hipLaunchKernelGGL((gat_bwd_cols_kernel<TH, TO, Acc, L, NV, VW, UC, RAG, false>), col_grid, dim3(kBlock), 0, st, a,
                           (int32_t)nbc);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (S_csc->n_chunks > 0 && S_csc->n_splits > 0) {
        e = launch_merge<Acc>(S_csc->splits, S_csc->n_splits, S_csc->n_chunks, r, static_cast<const Acc *>(a.part_vec),
                              MergeColumns<Acc>{static_cast<Acc *>(sums), dt, static_cast<const Acc *>(a.part_sc),
                                                once ? nullptr : ds, a1, a2, r, out16 && !once},
                              st);
        if (e != hipSuccess) return e;
    }
    if (once && split_rows) {
        hipLaunchKernelGGL((gat_bwd_long_rows_kernel<Acc>), dim3((unsigned)(S_csr->n_splits + 3) / 4), dim3(kBlock),
                           0, st, S_csr->splits, S_csr->n_splits, S_csr->ptr, static_cast<const Acc *>(a.dxs), ds);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // ds, the rest of dH, da1 = H^T ds, da2 = H^T dt: whole rounds of the lane groups, at most
    // kFinishBlocks blocks
    GatFinishArgs f;
    f.n = n;
    f.r = r;
    f.rows_per_block = (int32_t)(((int64_t)n + (int64_t)kFinishBlocks * GPB - 1) / ((int64_t)kFinishBlocks * GPB)) * GPB;
    f.ptr = S_csr->ptr;
    f.long_len = split_rows ? S_csr->long_len : INT32_MAX;
    f.dxs = a.dxs;
    f.ds = ds;
    f.dt = dt;
    f.H = H;
    f.a1 = a1;
    f.a2 = a2;
    f.dHp = sums;
    f.dH = dH;
    f.out16 = out16 ? 1 : 0;
    f.part = ws + lay.pblk;
    const int32_t nbf = (int32_t)(((int64_t)n + f.rows_per_block - 1) / f.rows_per_block);
    if (once)
        hipLaunchKernelGGL((gat_bwd_finish_kernel<TH, Acc, L, NV, VW, RAG, true>), dim3((unsigned)nbf), dim3(kBlock), 0, st,
                           f);
    else
        hipLaunchKernelGGL((gat_bwd_finish_kernel<TH, Acc, L, NV, VW, RAG, false>), dim3((unsigned)nbf), dim3(kBlock), 0, st,
                           f);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((gat_bwd_reduce_kernel<Acc>), reduce_grid, dim3(1024), 0, st, nbf, r,
                       static_cast<const Acc *>(f.part), da1, da2);
    return hipGetLastError();
}

// With one element per lane (see vector_rows) the first five cover every r.
#define BWD_SHAPES(X)                                                                            \
    X(1, 1) X(2, 1) X(4, 1) X(8, 1) X(16, 1)                                                     \
    if constexpr (VW > 1) { X(32, 1) X(64, 1) X(64, 2) X(64, 4) }

template <class TH, class TO, class Acc, int VW, bool RAG = false>
hipError_t dispatch_bwd(Shape sh, const fmm_sparse *S_csr, const fmm_sparse *S_csc, const void *H, const void *a1,
                        const void *a2, const void *s, const void *t, const void *out, const void *lse,
                        const void *dO, int32_t r,
                        double slope, bool softmax, void *dH, bool out16, void *da1, void *da2, void *dS, void *ws,
                        hipStream_t st)
{
#define BWD_CASE(Lv, NVv)                                                                        \
    if (sh.L == Lv && sh.NV == NVv)                                                              \
        return run_bwd_shape<TH, TO, Acc, Lv, NVv, VW, RAG>(                                        \
            S_csr, S_csc, (const TH *)H, (const Acc *)a1, (const Acc *)a2, (const Acc *)s, (const Acc *)t, \
            (const Acc *)out, (const Acc *)lse, (const TO *)dO, r, (Acc)slope, softmax, dH, out16, (Acc *)da1, (Acc *)da2, \
            (Acc *)dS, (char *)ws, st);
    BWD_SHAPES(BWD_CASE)
#undef BWD_CASE
    return hipErrorInvalidValue;
}

}  // namespace
}  // namespace fmm

using namespace fmm;

extern "C" {

fmm_status fmm_gat_backward_workspace(const fmm_sparse *S_csr, const fmm_sparse *S_csc, int32_t r, int32_t dtype,
                                      size_t *bytes)
{
    if (!bytes || !S_csr || !S_csc) return FMM_ERR_NULL;
    if (r < 1 || S_csr->rows < 0) return FMM_ERR_DIM;
    if (dtype != FMM_F32 && dtype != FMM_BF16 && dtype != FMM_F64) return FMM_ERR_DTYPE;
    *bytes = bwd_layout(S_csr, S_csc, r, dtype == FMM_F64 ? 8 : dtype == FMM_BF16 ? 2 : 4, dtype == FMM_F64 ? 8 : 4).total;
    return FMM_OK;
}

fmm_status fmm_gat_backward(const fmm_sparse *S_csr, const fmm_sparse *S_csc, const void *H, const void *a1,
                            const void *a2, const void *s, const void *t, const void *out, const void *lse,
                            const void *dO, int32_t r,
                            int32_t dtype, double negative_slope, int32_t flags, void *dH, void *da1, void *da2,
                            void *dS, void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (!S_csr || !S_csc) return FMM_ERR_NULL;
    if (S_csr->orient != FMM_CSR || S_csc->orient != FMM_CSC) return FMM_ERR_ORIENT;
    const int32_t n = S_csr->rows;
    if (n < 0 || S_csr->cols != n || S_csc->rows != n || S_csc->cols != n || S_csr->nnz != S_csc->nnz ||
        S_csr->nnz < 0 || r < 1)
        return FMM_ERR_DIM;
    if (flags & ~(FMM_GAT_SOFTMAX | FMM_DC_BF16 | FMM_GRAD_BF16)) return FMM_ERR_DIM;
    const bool do16 = (flags & FMM_DC_BF16) != 0;  // dO stored as bfloat16 (bfloat16 H only)
    const bool grad16 = (flags & FMM_GRAD_BF16) != 0;  // and dH
    if ((do16 || grad16) && dtype != FMM_BF16) return FMM_ERR_UNSUPPORTED;
    if (!S_csr->ptr || !S_csc->ptr || (S_csr->nnz > 0 && (!S_csr->idx || !S_csc->idx))) return FMM_ERR_NULL;
    if (!a1 || !a2 || !da1 || !da2) return FMM_ERR_NULL;
    if (n > 0 && (!H || !s || !t || !out || !dO || !dH)) return FMM_ERR_NULL;
    if (n > 0 && (flags & FMM_GAT_SOFTMAX) && !lse) return FMM_ERR_NULL;
    for (const fmm_sparse *S : {S_csr, S_csc}) {
        if (S->n_chunks < 0 || S->n_splits < 0) return FMM_ERR_DIM;
        if (S->n_chunks > 0 && (!S->chunks || !S->splits || S->long_len < 1)) return FMM_ERR_NULL;
    }
    const size_t ob = dtype == FMM_F64 ? 8 : 4, hb = dtype == FMM_BF16 ? 2 : ob;
    if (!ws || ws_bytes < bwd_layout(S_csr, S_csc, r, hb, ob).total || (uintptr_t)ws % 256 != 0)
        return FMM_ERR_WORKSPACE;
    const bool softmax = (flags & FMM_GAT_SOFTMAX) != 0;
    auto misaligned = [](const void *p) { return ((uintptr_t)p % 16) != 0; };
    hipError_t e;
    if (dtype == FMM_F32) {
        if (r > (r % 4 == 0 ? 1024 : 256)) return FMM_ERR_DTYPE;
        if (r % 4 == 0 && (misaligned(H) || misaligned(out) || misaligned(dO) || misaligned(dH)))
            return FMM_ERR_UNSUPPORTED;
        if (r % 4 == 0)
            e = dispatch_bwd<float, float, float, 4>(bwd_shape(r, 4), S_csr, S_csc, H, a1, a2, s, t, out, lse, dO, r,
                                                      negative_slope, softmax, dH, grad16, da1, da2, dS, ws, stream);
        else if (vector_rows(r, 4))  // rows end in an overlapping vector
            e = dispatch_bwd<float, float, float, 4, true>(bwd_shape(r, 4), S_csr, S_csc, H, a1, a2, s, t, out, lse, dO,
                                                            r, negative_slope, softmax, dH, grad16, da1, da2, dS, ws, stream);
        else
            e = dispatch_bwd<float, float, float, 1>(bwd_shape(r, 1), S_csr, S_csc, H, a1, a2, s, t, out, lse, dO, r,
                                                  negative_slope, softmax, dH, grad16, da1, da2, dS, ws, stream);
    } else if (dtype == FMM_BF16) {
        if (r % 8 != 0 || r > 1024) return FMM_ERR_DTYPE;
        if (misaligned(H) || misaligned(out) || misaligned(dO) || misaligned(dH)) return FMM_ERR_UNSUPPORTED;
        e = do16 ? dispatch_bwd<bf16_t, bf16_t, float, 8>(bwd_shape(r, 8), S_csr, S_csc, H, a1, a2, s, t, out, lse,
                                                          dO, r, negative_slope, softmax, dH, grad16, da1, da2, dS, ws, stream)
                 : dispatch_bwd<bf16_t, float, float, 8>(bwd_shape(r, 8), S_csr, S_csc, H, a1, a2, s, t, out, lse,
                                                         dO, r, negative_slope, softmax, dH, grad16, da1, da2, dS, ws, stream);
    } else if (dtype == FMM_F64) {
        if (r > (r % 2 == 0 ? 512 : 256)) return FMM_ERR_DTYPE;
        if (r % 2 == 0 && (misaligned(H) || misaligned(out) || misaligned(dO) || misaligned(dH)))
            return FMM_ERR_UNSUPPORTED;
        if (r % 2 == 0)
            e = dispatch_bwd<double, double, double, 2>(bwd_shape(r, 2), S_csr, S_csc, H, a1, a2, s, t, out, lse, dO, r,
                                                      negative_slope, softmax, dH, grad16, da1, da2, dS, ws, stream);
        else if (vector_rows(r, 2))  // rows end in an overlapping vector
            e = dispatch_bwd<double, double, double, 2, true>(bwd_shape(r, 2), S_csr, S_csc, H, a1, a2, s, t, out, lse, dO,
                                                            r, negative_slope, softmax, dH, grad16, da1, da2, dS, ws, stream);
        else
            e = dispatch_bwd<double, double, double, 1>(bwd_shape(r, 1), S_csr, S_csc, H, a1, a2, s, t, out, lse, dO, r,
                                                  negative_slope, softmax, dH, grad16, da1, da2, dS, ws, stream);
    } else {
        return FMM_ERR_DTYPE;
    }
    if (e != hipSuccess) {
        set_last_hip_error((int32_t)e);
        return FMM_ERR_HIP;
    }
    return FMM_OK;
}

}  // extern "C"
