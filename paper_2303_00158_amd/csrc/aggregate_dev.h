// Device side of the neighbour aggregation over a sampled block, forward (pull over the block
// CSR) and backward (pull over its transpose, no atomics): the mean and GCN
// sums, and GraphSAGE's max aggregator with its argmax table.
//
// Work split: one wavefront per output row (the forward sums: up to two).  A
// row of f elements is cut into C = ceil(f / 4) chunks of 4; when C <= 32 the
// wavefront is divided into S = 64 / C slots that walk different edges of the
// row at once (f = 100: two slots of 25 lanes), and the slot partial sums are
// folded with lane shuffles at the end.  The backward walks a source's edges
// in sequence, several sources per wavefront for narrow rows.  Sums are fp32.
#pragma once

#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "internal.h"

namespace gnn {
namespace agg {

template <class T> struct Tag {
    using type = T;
};

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// Elements e0 .. e0+3 of a row starting at row_off (zero past f).  Loads are
// issued unconditionally from in-bounds addresses and masked afterwards.
template <bool VEC, class T>
__device__ __forceinline__ float4 load_chunk(const T *p, int64_t row_off, int64_t e0, int64_t f) {
    if constexpr (VEC) return load4(p, row_off + e0);
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool ok = e0 + q < f;
        const float x = Elem<T>::load(p, row_off + (ok ? e0 + q : f - 1));
        v[q] = ok ? x : 0.f;
    }
    return make_float4(v[0], v[1], v[2], v[3]);
}

template <bool VEC, class T>
__device__ __forceinline__ void store_chunk(T *p, int64_t row_off, int64_t e0, int64_t f, float4 v) {
    if constexpr (VEC) {
        store4(p, row_off + e0, v);
        return;
    }
    const float a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (e0 + q < f) Elem<T>::store(p, row_off + e0 + q, a[q]);
}

__device__ __forceinline__ void fma4(float4 &acc, float w, const float4 &v) {
    acc.x = fmaf(w, v.x, acc.x);
    acc.y = fmaf(w, v.y, acc.y);
    acc.z = fmaf(w, v.z, acc.z);
    acc.w = fmaf(w, v.w, acc.w);
}

__device__ __forceinline__ float4 shfl4(const float4 &v, int src) {
    return make_float4(__shfl(v.x, src, 64), __shfl(v.y, src, 64), __shfl(v.z, src, 64), __shfl(v.w, src, 64));
}

__device__ __forceinline__ float4 round_bf16(float4 v) {
    return make_float4(bf16_to_f32(f32_to_bf16(v.x)), bf16_to_f32(f32_to_bf16(v.y)), bf16_to_f32(f32_to_bf16(v.z)),
                       bf16_to_f32(f32_to_bf16(v.w)));
}
// ---------------------------------------------------------------------------
// forward
//
// A row is summed by S slots: within a window of 64 edges slot s takes edges s,
// s + S, ... one after another, and the slots are added in order at the end.
// S = 64 / ceil(f / 4) (1 when a row has more than 32 chunks of 4) fixes the
// order of the sums for every kernel that has to reproduce it. A lane holds E
// consecutive elements of its slot's sum, so a row takes S CL lanes, CL =
// ceil(f / E), and a wavefront R = 64 / (S CL) rows.
//
// The kernel is bound by the misses in flight, so what counts is that its
// whole grid is resident (at most 64 registers: FwdJob) and that a wavefront
// covers many edges at once.  bf16 rows use E = 8: one 16-byte
// load (4-byte aligned; the last lane's is moved back to end with the row)
// instead of two, two rows per wavefront for f = 100, and every lane loads the
// column indices of its own slot's edges instead of taking them from other
// lanes. 1.19M edges of 32,768 targets, f = 100: 74 us with 4 elements per
// lane, shuffled indices and 6 wavefronts per SIMD, now 50 us.
// ---------------------------------------------------------------------------

// E consecutive elements as loaded (add() adds w times their values).
template <class T, int E, bool VEC, bool ROUND> struct RowElems {
    float4 v;  // E = 4
    __device__ __forceinline__ void load(const T *p, int64_t row_off, int64_t e0, int64_t f) {
        v = load_chunk<VEC>(p, row_off, e0, f);
    }
    __device__ __forceinline__ void add(float (&acc)[4], float w) const {
        const float4 x = ROUND ? round_bf16(v) : v;
        acc[0] = fmaf(w, x.x, acc[0]);
        acc[1] = fmaf(w, x.y, acc[1]);
        acc[2] = fmaf(w, x.z, acc[2]);
        acc[3] = fmaf(w, x.w, acc[3]);
    }
};
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
template <bool VEC, bool ROUND> struct RowElems<uint16_t, 8, VEC, ROUND> {
    u32x4_a4 v;
    __device__ __forceinline__ void load(const uint16_t *p, int64_t row_off, int64_t e0, int64_t) {
        v = *reinterpret_cast<const u32x4_a4 *>(p + row_off + e0);
    }
    __device__ __forceinline__ void add(float (&acc)[8], float w) const {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[2 * i] = fmaf(w, __uint_as_float(v[i] << 16), acc[2 * i]);
            acc[2 * i + 1] = fmaf(w, __uint_as_float(v[i] & 0xffff0000u), acc[2 * i + 1]);
        }
    }
};
template <int E, bool VEC, class T>
__device__ __forceinline__ void store_elems(T *p, int64_t row_off, int64_t e0, int64_t f, const float (&a)[E]) {
    if constexpr (E == 4) {
        store_chunk<VEC>(p, row_off, e0, f, make_float4(a[0], a[1], a[2], a[3]));
    } else if constexpr (sizeof(T) == 2) {
        u32x4_a4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o[i] = static_cast<uint32_t>(f32_to_bf16(a[2 * i])) | (static_cast<uint32_t>(f32_to_bf16(a[2 * i + 1])) << 16);
        *reinterpret_cast<u32x4_a4 *>(p + row_off + e0) = o;
    } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4_a4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = __float_as_uint(a[4 * h + i]);
            *reinterpret_cast<u32x4_a4 *>(p + row_off + e0 + 4 * h) = o;
        }
    }
}

// A lane's place in its wavefront's rows.
struct RowLanes {
    int r, slot, chunk;
    bool active;
    __device__ __forceinline__ RowLanes(int CL, int S, int R) {
        const int lane = threadIdx.x & 63, per_row = S * CL;
        if (per_row > 64) {  // one row, a chunk group at a time
            r = slot = 0;
            chunk = lane;
            active = true;
            return;
        }
        r = lane / per_row;
        slot = lane % per_row / CL;
        chunk = lane % CL;  // (CL divides per_row)
        active = r < R;
    }
};

// Where a row's edges lie and whose rows they read: a block's own columns and
// its source rows ...
template <class TIn> struct BlockEdges {
    using T = TIn;
    static constexpr bool kRound = false;
    const int32_t *col;
    const float *norm;
    const TIn *x;
    int64_t stride;
    __device__ __forceinline__ int32_t at(int64_t, int64_t beg, int32_t p) const { return col[beg + p]; }
};
// ... or an fp32 feature table in device memory (the feature loading fused
// into the input layer's aggregation): row i's p-th sampled neighbour is the
// global vertex gids[i k + p] (the sampler's staging of the block, in the
// block's column order), whose table row is rounded to bf16 element by element,
// exactly as the gather would have stored it in X'. Same slots and order of
// summation as over X', so the result is bitwise the same. norm holds the
// graph's normalisers by global id (src_norm of the block holds the same
// values).
struct TableEdges {
    using T = float;
    static constexpr bool kRound = true;
    const int64_t *gids;
    int64_t k;
    const float *norm;
    const float *x;
    int64_t stride;
    __device__ __forceinline__ int32_t at(int64_t row, int64_t, int32_t p) const {
        return static_cast<int32_t>(gids[row * k + p]);  // (graphs of up to 2^31 - 1 vertices)
    }
};

// Rows row0 .. row0 + R - 1 of one wavefront. The GCN self term is row i of
// x_self.
template <int KIND, int E, bool VEC, class Edges, class TSelf, class TOut>
__device__ __forceinline__ void agg_fwd_rows(const Edges &edges, const int64_t *__restrict__ rowptr,
                                             const float *__restrict__ src_norm, const TSelf *__restrict__ x_self,
                                             int64_t n, int64_t f, int CL, int S, const RowLanes &L,
                                             TOut *__restrict__ out, int64_t row0) {
    using T = typename Edges::T;
    const int lane = threadIdx.x & 63;
    const bool live = L.active && row0 + L.r < n;
    const int64_t row = live ? row0 + L.r : row0;
    const int64_t beg = rowptr[row];
    const int32_t deg = static_cast<int32_t>(rowptr[row + 1] - beg), mine = live ? deg : 0;
    const float wi = (KIND == GNN_AGG_GCN_SYM) ? src_norm[row] : 1.f;
    for (int chunk = L.chunk; chunk < CL; chunk += 64) {
        const int64_t e0 = E == 8 ? min(static_cast<int64_t>(chunk) * 8, f - 8) : static_cast<int64_t>(chunk) * E;
        RowElems<TSelf, E, VEC, false> self;
        if (KIND == GNN_AGG_GCN_SYM) self.load(x_self, row * f, e0, f);  // issued before the neighbours
        float acc[E];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = 0.f;
        for (int32_t wb = 0; wb < mine; wb += 64) {
            const int wn = min(64, mine - wb);
            if constexpr (Edges::kRound) {
                for (int t = L.slot; t < wn; t += 4 * S) {
                    int32_t j[4];
                    float w[4];
                    RowElems<T, E, VEC, true> v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (t + q * S < wn) j[q] = edges.at(row, beg, wb + t + q * S);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (t + q * S < wn) {
                            w[q] = (KIND == GNN_AGG_GCN_SYM) ? wi * edges.norm[j[q]] : 1.f;
                            v[q].load(edges.x, static_cast<int64_t>(j[q]) * edges.stride, e0, f);
                        }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (t + q * S < wn) v[q].add(acc, w[q]);
                }
            } else {
                // Four edges that are all there (ALL) need no guard around each
                // load; the guards cost a small call more than its loads
                // (1,024 targets, f = 256, GCN: 8.1 us, now 6.2). The table's
                // launch above lost by it (23 us to 28 beside the sort of a
                // three-layer step).
                auto four = [&](int t, auto all) {
                    constexpr bool ALL = decltype(all)::value;
                    int32_t j[4];
                    float w[4];
                    RowElems<T, E, VEC, false> v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (ALL || t + q * S < wn) j[q] = edges.at(row, beg, wb + t + q * S);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (ALL || t + q * S < wn) {
                            w[q] = (KIND == GNN_AGG_GCN_SYM) ? wi * edges.norm[j[q]] : 1.f;
                            v[q].load(edges.x, static_cast<int64_t>(j[q]) * edges.stride, e0, f);
                        }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (ALL || t + q * S < wn) v[q].add(acc, w[q]);
                };
                int t = L.slot;
                for (; t + 3 * S < wn; t += 4 * S) four(t, std::true_type{});
                if (t < wn) four(t, std::false_type{});
            }
        }
        // fold the slots into slot 0
        for (int s2 = 1; s2 < S; ++s2) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const float o = __shfl(acc[e], lane + s2 * CL, 64);
                if (L.slot == 0) acc[e] += o;
            }
        }
        if (L.slot != 0 || !live) continue;
        if (KIND == GNN_AGG_SAGE_MEAN) {
            if (deg > 0) {
                const float d = static_cast<float>(deg);
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] /= d;
            }
        } else {
            self.add(acc, wi * wi);
        }
        store_elems<E, VEC>(out, row * f, e0, f, acc);
    }
}

// ---------------------------------------------------------------------------
// backward: d_src[j] = self(j) + sum_{i in csc(j)} w_ij d_a[i, nbr part]
//
// Rows of more than 128 elements take a wavefront each, which adds the source's
// edges one after another, four loads in flight; narrower ones share a
// wavefront (walk_narrow). Most sources have one or two edges: the kernel is a
// chain of three dependent loads per row (column pointer, rows, their
// gradients), so what counts is that many rows are in flight and that the grid
// is resident (54 and 62 registers for wide rows; narrow ones 71 to 91, so 5 to
// 7 wavefronts per SIMD: at 64 they spill and took up to twice the time).
// 8,192 targets, f = 256: 41 us, now 31, the maximum's 83 us, now 44.
// Gradients above 32 MiB used to bypass the caches in calls of their own,
// which made the call 1 to 3 us shorter and its reader 3 to 7 us longer (the
// backward and the update below it: 68.4 us, without 66.0; the maximum's 80.5
// and 76.8).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void add4(float4 &acc, const float4 &a, const float4 &b) {
    acc.x += a.x + b.x;
    acc.y += a.y + b.y;
    acc.z += a.z + b.z;
    acc.w += a.w + b.w;
}
// acc, a column's sum over its edges, becomes its gradient: the self term
// (weight ws) where j is a destination, and the ReLU mask.
template <bool VEC>
__device__ __forceinline__ void finish_grad(float4 acc, float ws, const float4 &self, const float4 &hb, int64_t n_dst,
                                            bool mask, int64_t f, uint32_t e0, float *__restrict__ d_src, int64_t j) {
    if (j < n_dst) fma4(acc, ws, self);
    if (mask) {
        if (!(hb.x > 0.f)) acc.x = 0.f;
        if (!(hb.y > 0.f)) acc.y = 0.f;
        if (!(hb.z > 0.f)) acc.z = 0.f;
        if (!(hb.w > 0.f)) acc.w = 0.f;
    }
    store_chunk<VEC>(d_src, j * f, e0, f, acc);
}
// What finish_grad takes of column j itself (ka: d_a's row length).
struct OwnTerms {
    float4 self, hb;
};
template <class THB, bool VEC>
__device__ __forceinline__ OwnTerms own_terms(int64_t n_dst, const float *__restrict__ d_a, int64_t ka,
                                              const THB *__restrict__ h_below, int64_t f, uint32_t e0, int64_t j) {
    OwnTerms o;
    if (j < n_dst) o.self = load_chunk<VEC>(d_a + j * ka, 0, e0, f);
    if (h_below) o.hb = load_chunk<VEC>(h_below + j * f, 0, e0, f);
    return o;
}
// The weight of row i's edge in the column of a source with normaliser wj.
template <int KIND>
__device__ __forceinline__ float edge_weight(const int64_t *__restrict__ rowptr, const float *__restrict__ src_norm,
                                             int32_t i, float wj) {
    if constexpr (KIND == GNN_AGG_GCN_SYM) return src_norm[i] * wj;
    return 1.f / static_cast<float>(static_cast<int32_t>(rowptr[i + 1]) - static_cast<int32_t>(rowptr[i]));
}
// Column j of a wavefront, its edges beg .. beg + len - 1, for rows of more
// than 32 lanes: the lanes load the indices and weights of 32 edges at a time
// (with a load per edge and lane the backward of 1,024 targets, f = 256, took 8.5
// us, now 7.0).
template <int KIND, class THB, bool VEC>
__device__ __forceinline__ void agg_bwd_row(int64_t n_dst, const int64_t *__restrict__ rowptr,
                                             const int32_t *__restrict__ cscrow, const float *__restrict__ src_norm,
                                             const float *__restrict__ d_a, int64_t f, int C, const RowLanes &L,
                                             const THB *__restrict__ h_below, float *__restrict__ d_src, int64_t j,
                                             int64_t beg, int32_t len) {
    const int64_t ka = (KIND == GNN_AGG_SAGE_MEAN) ? 2 * f : f;
    const int64_t nbr_off = (KIND == GNN_AGG_SAGE_MEAN) ? f : 0;
    const float wj = (KIND == GNN_AGG_GCN_SYM) ? src_norm[j] : 1.f;
    const bool mask = h_below != nullptr;
    const float ws = (KIND == GNN_AGG_GCN_SYM) ? wj * wj : 1.f;
    const int lane = threadIdx.x & 63;
    // (every lane that entered stays in the loop: its edges are read by the others)
    for (int c0 = 0; c0 < C; c0 += 64) {
        const bool active = c0 + L.chunk < C;
        const uint32_t e0 = active ? static_cast<uint32_t>(c0 + L.chunk) * 4 : 0;
        float4 self, hb;
        if (j < n_dst) self = load_chunk<VEC>(d_a + j * ka, 0, e0, f);
        if (mask) hb = load_chunk<VEC>(h_below + j * f, 0, e0, f);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int32_t wb = 0; wb < len; wb += 32) {  // (a row has more than 32 lanes)
            const int32_t wn = min(32, len - wb);
            const int32_t my_idx = lane < wn ? cscrow[beg + wb + lane] : 0;
            float4 v[4];
            auto load = [&](int32_t t) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (t + q < wn) {
                        const int64_t i = __builtin_amdgcn_readlane(my_idx, t + q);
                        v[q] = load_chunk<VEC>(d_a + (i * ka + nbr_off), 0, e0, f);
                    }
            };
            load(0);
            // (the weights behind the first rows: they wait for loads of their own)
            const float my_w = lane < wn ? edge_weight<KIND>(rowptr, src_norm, my_idx, wj) : 0.f;
            for (int32_t t = 0; t < wn; t += 4) {
                if (t > 0) load(t);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (t + q < wn)
                        fma4(acc, __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_w), t + q)), v[q]);
            }
        }
        if (active) finish_grad<VEC>(acc, ws, self, hb, n_dst, mask, f, e0, d_src, j);
    }
}

// This lane's part of a narrow column's sum: edges t0, t0 + step, ... of the
// column's len at cscrow, four at a time in two pairs (one running sum over
// all of them was further from the 64-bit result: 1.8e-8 against 1.6e-8 at 246
// targets, f = 128).
template <int KIND, bool VEC>
__device__ __forceinline__ float4 agg_bwd_part(const int64_t *__restrict__ rowptr, const int32_t *__restrict__ cscrow,
                                               const float *__restrict__ src_norm, const float *__restrict__ d_a,
                                               int64_t f, uint32_t e0, float wj, uint32_t len, uint32_t t0,
                                               uint32_t step) {
    const int64_t ka = (KIND == GNN_AGG_SAGE_MEAN) ? 2 * f : f;
    const int64_t nbr_off = (KIND == GNN_AGG_SAGE_MEAN) ? f : 0;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    auto four = [&](uint32_t t, auto all) {
        constexpr bool ALL = decltype(all)::value;
        int32_t i[4];
        float w[4];
        float4 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (ALL || t + q * step < len) i[q] = cscrow[t + q * step];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (ALL || t + q * step < len) {
                v[q] = load_chunk<VEC>(d_a + (static_cast<int64_t>(i[q]) * ka + nbr_off), 0, e0, f);
                w[q] = edge_weight<KIND>(rowptr, src_norm, i[q], wj);
            }
        float4 pair[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (ALL || t + q * step < len) fma4(pair[q / 2], w[q], v[q]);
        add4(acc, pair[0], pair[1]);
    };
    uint32_t t = t0;
    for (; t + 3 * step < len; t += 4 * step) four(t, std::true_type{});
    if (t < len) four(t, std::false_type{});
    return acc;
}

// The transpose's long columns (the graph's hubs): a wavefront that walks one
// alone, four edges in flight, is still at it when the rest of the grid has
// finished. Such columns are put aside (LongColumns) and summed by the
// whole workgroup afterwards, a thread per element and kLongAhead edges in
// flight, the edges in the same sequence, so the sums are the same bit for bit.
// At 8,192 targets (fanout 25, f = 256; the longest column has about 180
// of the 59k edges) the mean's backward took 36 us without, 32 with it, the
// maximum's 79 and 43. Columns of up to 32 or 64 edges left with their wavefront
// are no faster at 1,024 targets and 3 us slower at 8,192.
constexpr int kLong = 16;       // longest column of one wavefront
constexpr int kShare = 8;       // narrow rows: longest column of a row's own lanes
constexpr int kLongAhead = 16;
struct LongColumns {
    static constexpr int kCap = 16;  // per wavefront; columns past it stay with their wavefront
    int n[kWaves];
    int32_t j[kWaves][kCap];
    // A wavefront's n-th column; false where there is no room.
    __device__ __forceinline__ bool add(int &n, int64_t c) {
        if (n == kCap) return false;
        j[threadIdx.x >> 6][n++] = static_cast<int32_t>(c);  // (every lane writes the same)
        return true;
    }
    // fn(column) in all threads, for the columns of all wavefronts (n: this one's).
    template <class F> __device__ __forceinline__ void walk(int own, F &&fn) {
        n[threadIdx.x >> 6] = own;
        __syncthreads();
        for (int w = 0; w < kWaves; ++w)
            for (int i = 0; i < n[w]; ++i) fn(static_cast<int64_t>(j[w][i]));
    }
};
// One column per wavefront (rows of more than 128 elements): row(j, beg, len)
// in the lanes that the row takes, and long_row(j, beg, end) in all threads of
// the workgroup for those put aside.
template <class Row, class LongRow>
__device__ __forceinline__ void walk_columns(const gnn_block &b, int64_t blk, int64_t nblk, const RowLanes &L,
                                             Row &&row, LongRow &&long_row) {
    __shared__ LongColumns aside;
    const int64_t n_src = b.counts[1];
    int put = 0;
    for (int64_t j0 = blk * kWaves + (threadIdx.x >> 6); j0 < n_src; j0 += nblk * kWaves) {
        const int64_t j = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(j0));  // (local ids are 32-bit)
        const int64_t beg = b.cscptr[j], end = b.cscptr[j + 1];
        const int32_t len = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(end - beg));
        if (len > kLong && aside.add(put, j)) continue;
        if (L.active) row(j, beg, len);
    }
    aside.walk(put, [&](int64_t j) { long_row(j, b.cscptr[j], b.cscptr[j + 1]); });
}

// Rows of up to 128 elements: C = ceil(f / 4) <= 32 lanes each, S = 64 / C of them
// in a wavefront. Columns of up to kShare edges share a wavefront, as many as
// leave every wavefront of the grid one (at most S). A longer one is summed by a
// whole wavefront, S edges at a time (slots), and one of more than kLong S edges by the workgroup,
// 4 S at a time. part(e0, j, beg, len, t0, step) is a lane's part of a sum,
// edges t0, t0 + step, ...; the slots are added as a tree, the wavefronts of a
// workgroup in order. All of it depends on the column's length alone (a column
// for which the list has no room is summed in the same parts by one
// wavefront), so results are the same on every run.
// A block of 18,497 sources and 213k edges, the longest column 3,928: 12 us at f =
// 4, 20 at 16, 55 at 64, 104 at 128 (252, 186, 194 and 216 when a workgroup
// walked long columns one after another with a thread per element, most of
// them idle; its one running sum was up to 2.8 times further from the 64-bit
// sum of 4,000 edges). kShare: 4 is 10 to 25% slower at 32,768 targets (f up to
// 16), 16 20% slower at 1,024.
template <class Part, class Own, class Finish>
__device__ __forceinline__ void walk_narrow(const gnn_block &b, int64_t blk, int64_t nblk, int C, int S, Part &&part,
                                            Own &&own, Finish &&finish) {
    __shared__ LongColumns aside;
    __shared__ float4 sums[kWaves][32];
    const int64_t n_src = b.counts[1];
    const int64_t waves = nblk * kWaves;
    // (three quarters of the grid's wavefronts: what the registers leave resident)
    const uint32_t spread = static_cast<uint32_t>(waves * 3 / 4);
    const int R = n_src <= spread ? 1
                                  : static_cast<int>(min(static_cast<uint32_t>(S),
                                                         (static_cast<uint32_t>(n_src) + spread - 1) / spread));
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int slot = lane / C, chunk = lane - slot * C;
    const uint32_t e0 = static_cast<uint32_t>(chunk) * 4;
    // slots 1 .. S - 1 are added to slot 0
    auto fold = [&](float4 &acc) {
        for (int half = 32; half > 0; half >>= 1) {
            if (half >= S) continue;
            const float4 o = shfl4(acc, lane + half * C);
            if (slot < half && slot + half < S) acc = make_float4(acc.x + o.x, acc.y + o.y, acc.z + o.z, acc.w + o.w);
        }
    };
    int put = 0;
    for (int64_t j0 = (blk * kWaves + wave) * R; j0 < n_src; j0 += waves * R) {
        uint64_t longs;  // the first lanes of the longer columns
        {
            const bool live = slot < R && j0 + slot < n_src;
            const int64_t j = live ? j0 + slot : j0, beg = b.cscptr[j];
            const int32_t len = static_cast<int32_t>(b.cscptr[j + 1] - beg);
            longs = __ballot(live && len > kShare && chunk == 0);
            if (live && len <= kShare) {
                const OwnTerms o = own(e0, j);
                finish(e0, j, part(e0, j, beg, len, 0, 1), o);
            }
        }
        while (longs) {
            const int64_t j = j0 + __builtin_ctzll(longs) / C, beg = b.cscptr[j];
            const int32_t len = static_cast<int32_t>(b.cscptr[j + 1] - beg);
            longs &= longs - 1;
            const int shares = len > kLong * S ? kWaves : 1;
            if (shares > 1 && aside.add(put, j)) continue;
            const OwnTerms o = own(e0, j);
            float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
            for (int w = 0; w < shares; ++w) {
                float4 acc = part(e0, j, beg, len, slot < S ? w * S + slot : len, shares * S);
                fold(acc);
                sum = make_float4(sum.x + acc.x, sum.y + acc.y, sum.z + acc.z, sum.w + acc.w);
            }
            if (slot == 0) finish(e0, j, sum, o);
        }
    }
    aside.walk(put, [&](int64_t j) {
        const int64_t beg = b.cscptr[j];
        const int32_t len = static_cast<int32_t>(b.cscptr[j + 1] - beg);
        const OwnTerms o = own(e0, j);
        float4 acc = part(e0, j, beg, len, slot < S ? wave * S + slot : len, kWaves * S);
        fold(acc);
        if (slot == 0) sums[wave][lane] = acc;
        __syncthreads();
        if (wave == 0 && slot == 0) {
            float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int w = 0; w < kWaves; ++w) {
                const float4 x = sums[w][lane];
                sum = make_float4(sum.x + x.x, sum.y + x.y, sum.z + x.z, sum.w + x.w);
            }
            finish(e0, j, sum, o);
        }
        __syncthreads();  // the sums are free for the next column
    });
}

template <int KIND, class THB>
__device__ __forceinline__ void agg_bwd_long(int64_t n_dst, const int64_t *__restrict__ rowptr,
                                             const int32_t *__restrict__ cscrow, const float *__restrict__ src_norm,
                                             const float *__restrict__ d_a, int64_t f, const THB *__restrict__ h_below,
                                             float *__restrict__ d_src, int64_t j, int64_t beg, int64_t end) {
    const int lane = threadIdx.x & 63;
    const int64_t ka = (KIND == GNN_AGG_SAGE_MEAN) ? 2 * f : f;
    const int64_t nbr_off = (KIND == GNN_AGG_SAGE_MEAN) ? f : 0;
    const float wj = (KIND == GNN_AGG_GCN_SYM) ? src_norm[j] : 1.f;
    // a wavefront past the row has nothing to add (e0 is uniform in it)
    for (uint32_t e0 = threadIdx.x - lane; e0 < f; e0 += kThreads) {
        const uint32_t e = min(e0 + lane, static_cast<uint32_t>(f) - 1);
        const float self = (d_a + (j < n_dst ? j : 0) * ka)[e];
        const float hb = h_below ? Elem<THB>::load(h_below + j * f, e) : 1.f;
        float acc = 0.f;
        for (int64_t wb = beg; wb < end; wb += 64) {
            const int wn = static_cast<int>(min<int64_t>(64, end - wb));
            int32_t my_idx = 0;
            float my_w = 0.f;
            if (lane < wn) {
                my_idx = cscrow[wb + lane];
                my_w = edge_weight<KIND>(rowptr, src_norm, my_idx, wj);
            }
            for (int tb = 0; tb < wn; tb += kLongAhead) {
                float v[kLongAhead], w[kLongAhead];
#pragma unroll
                for (int u = 0; u < kLongAhead; ++u) {  // (lanes past the window hold row 0 with weight 0)
                    const int64_t i = __builtin_amdgcn_readlane(my_idx, tb + u);
                    w[u] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_w), tb + u));
                    v[u] = (d_a + i * ka + nbr_off)[e];
                }
#pragma unroll
                for (int u = 0; u < kLongAhead; ++u) v[u] = tb + u < wn ? v[u] : 0.f;
#pragma unroll
                for (int u = 0; u < kLongAhead; ++u) acc = fmaf(w[u], v[u], acc);
            }
        }
        if (j < n_dst) acc = fmaf((KIND == GNN_AGG_GCN_SYM) ? wj * wj : 1.f, self, acc);
        if (!(hb > 0.f)) acc = 0.f;
        if (e0 + lane < f) (d_src + j * f)[e] = acc;
    }
}

// One row per wavefront, the grid's wavefronts striding over the rows (a
// grid of at most kMaxBlocks workgroups: capacity-sized grids would mostly
// hold workgroups that read the row count only to exit).
constexpr int64_t kMaxBlocks = 2048;

template <int KIND, bool VEC>
struct FwdTableJob {
    gnn_block b;
    TableEdges edges;
    const uint16_t *x_self;
    int64_t f;
    int C, S;
    uint16_t *out;
    __device__ void run(int64_t blk, int64_t nblk) const {
        const int64_t n = b.counts[0];
        const RowLanes L(C, S, 1);
        for (int64_t row = blk * kWaves + (threadIdx.x >> 6); row < n; row += nblk * kWaves)
            agg_fwd_rows<KIND, 4, VEC>(edges, b.rowptr, b.src_norm, x_self, n, f, C, S, L, out, row);
    }
};

template <int KIND, class TIn, class TOut, int E, bool VEC>
struct FwdJob {
    gnn_block b;
    const TIn *h;
    int64_t f;
    int CL, S, R;
    TOut *out;
    // the grid's 8 workgroups per CU run at once (with more registers a
    // quarter of them would run alone afterwards)
    static constexpr int kWavesPerSimd = E == 8 || VEC ? 8 : 1;
    __device__ void run(int64_t blk, int64_t nblk) const {
        const int64_t n = b.counts[0];
        const RowLanes L(CL, S, R);
        const BlockEdges<TIn> edges{b.col, b.src_norm, h, f};
        for (int64_t row = (blk * kWaves + (threadIdx.x >> 6)) * R; row < n; row += nblk * kWaves * R)
            agg_fwd_rows<KIND, E, VEC>(edges, b.rowptr, b.src_norm, h, n, f, CL, S, L, out, row);
    }
};

template <int KIND, class THB, bool VEC, bool UNI>
struct BwdJob {
    gnn_block b;
    const float *d_a;
    int64_t f;
    int C, R;
    const THB *h_below;
    float *d_src;
    static constexpr int kWavesPerSimd = VEC && UNI ? 8 : 1;
    __device__ void run(int64_t blk, int64_t nblk) const {
        const int64_t n_dst = b.counts[0];
        if constexpr (UNI) {
            const RowLanes L(C, 1, 1);
            walk_columns(
                b, blk, nblk, L,
                [&](int64_t j, int64_t beg, int32_t len) {
                    agg_bwd_row<KIND, THB, VEC>(n_dst, b.rowptr, b.cscrow, b.src_norm, d_a, f, C, L, h_below, d_src, j,
                                                beg, len);
                },
                [&](int64_t j, int64_t beg, int64_t end) {
                    agg_bwd_long<KIND, THB>(n_dst, b.rowptr, b.cscrow, b.src_norm, d_a, f, h_below, d_src, j, beg, end);
                });
        } else {
            auto norm = [&](int64_t j) { return (KIND == GNN_AGG_GCN_SYM) ? b.src_norm[j] : 1.f; };
            walk_narrow(
                b, blk, nblk, C, R,
                [&](uint32_t e0, int64_t j, int64_t beg, int32_t len, int32_t t0, int32_t step) {
                    return agg_bwd_part<KIND, VEC>(b.rowptr, b.cscrow + beg, b.src_norm, d_a, f, e0, norm(j), len, t0,
                                                   step);
                },
                [&](uint32_t e0, int64_t j) {
                    return own_terms<THB, VEC>(n_dst, d_a, (KIND == GNN_AGG_SAGE_MEAN) ? 2 * f : f, h_below, f, e0, j);
                },
                [&](uint32_t e0, int64_t j, const float4 &sum, const OwnTerms &o) {
                    const float wj = norm(j);
                    finish_grad<VEC>(sum, (KIND == GNN_AGG_GCN_SYM) ? wj * wj : 1.f, o.self, o.hb, n_dst,
                                         h_below != nullptr, f, e0, d_src, j);
                });
        }
    }
};

// ---------------------------------------------------------------------------
// GraphSAGE's max aggregator, forward: out[i, c] = the maximum of h[u, c] over
// row i's edges, with argmax[i, c] the local source of the edge that holds it.
// Sequential rule: the row's first edge holds the running maximum and a later
// edge replaces it only when strictly greater (a tie, and a duplicate edge,
// go to the earliest edge).  The slots walk interleaved edges of the row,
// each applying the rule to its own edges with the row's first edge taken
// unconditionally (it belongs to slot 0); the fold keeps the greater value
// and, on equal values, the earlier edge.  That reproduces the sequential
// rule, NaN included: a NaN is only ever taken as the row's first edge, and
// then nothing replaces it.  A row without edges gives 0 and argmax -1.
// ---------------------------------------------------------------------------
struct MaxChunk {
    float v[4];
    int32_t pos[4];  // edge position in the row; INT32_MAX for none
    int32_t src[4];  // local source id; -1 for none
};

__device__ __forceinline__ void max_take(MaxChunk &m, int q, float v, int32_t pos, int32_t src) {
    m.v[q] = v;
    m.pos[q] = pos;
    m.src[q] = src;
}

template <bool VEC>
__device__ __forceinline__ void store_arg4(int32_t *p, int64_t row_off, int64_t e0, int64_t f, const int32_t *a) {
    if constexpr (VEC) {
        *reinterpret_cast<int4 *>(p + row_off + e0) = make_int4(a[0], a[1], a[2], a[3]);
        return;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (e0 + q < f) p[row_off + e0 + q] = a[q];
}

// argmax[row_off + e0 .. + 3], with `none` past f
template <bool VEC>
__device__ __forceinline__ int4 load_arg4(const int32_t *p, int64_t row_off, int64_t e0, int64_t f, int32_t none) {
    if constexpr (VEC) return *reinterpret_cast<const int4 *>(p + row_off + e0);
    int32_t a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bool ok = e0 + q < f;
        const int32_t x = p[row_off + (ok ? e0 + q : f - 1)];
        a[q] = ok ? x : none;
    }
    return make_int4(a[0], a[1], a[2], a[3]);
}

template <class TIn, class TOut, bool VEC>
__device__ __forceinline__ void agg_fwd_row_max(const int64_t *__restrict__ rowptr, const int32_t *__restrict__ col,
                                                const TIn *__restrict__ h, int64_t f, int C, int S,
                                                TOut *__restrict__ out, int32_t *__restrict__ argmax, int64_t row) {
    const int lane = threadIdx.x & 63;
    const int64_t beg = rowptr[row], end = rowptr[row + 1];
    const int groups = (C + 63) / 64;
    const int slot = (S > 1) ? lane / C : 0;
    for (int g = 0; g < groups; ++g) {
        const int chunk = (S > 1) ? lane % C : g * 64 + lane;
        const bool active = (S > 1) ? (slot < S) : (chunk < C);
        const int64_t e0 = active ? static_cast<int64_t>(chunk) * 4 : 0;
        MaxChunk m;
#pragma unroll
        for (int q = 0; q < 4; ++q) max_take(m, q, -INFINITY, INT32_MAX, -1);
        for (int64_t wb = beg; wb < end; wb += 64) {
            const int wn = static_cast<int>(min<int64_t>(64, end - wb));
            const int32_t base = static_cast<int32_t>(wb - beg);
            const int32_t my_idx = (lane < wn) ? col[wb + lane] : 0;
            for (int tb = 0; tb < wn; tb += 4 * S) {
                int32_t j[4];
                bool ok[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int t = tb + u * S + slot;
                    ok[u] = active && (t < wn);
                    j[u] = __shfl(my_idx, t & 63, 64);
                }
                float4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = load_chunk<VEC>(h, static_cast<int64_t>(j[u]) * f, e0, f);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (!ok[u]) continue;
                    const int32_t pos = base + tb + u * S + slot;
                    const float x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (pos == 0 || x[q] > m.v[q]) max_take(m, q, x[q], pos, j[u]);
                }
            }
        }
        // fold the slots into slot 0 in slot order
        for (int s2 = 1; s2 < S; ++s2) {
            const int src_lane = lane + s2 * C;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float ov = __shfl(m.v[q], src_lane, 64);
                const int32_t op = __shfl(m.pos[q], src_lane, 64);
                const int32_t os = __shfl(m.src[q], src_lane, 64);
                if (slot == 0 && (ov > m.v[q] || (ov == m.v[q] && op < m.pos[q]))) max_take(m, q, ov, op, os);
            }
        }
        if (slot != 0 || !active) continue;
        float r[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) r[q] = (m.src[q] < 0) ? 0.f : m.v[q];
        store_chunk<VEC>(out, row * f, e0, f, make_float4(r[0], r[1], r[2], r[3]));
        if (argmax) store_arg4<VEC>(argmax, row * f, e0, f, m.src);
    }
}

// Backward of the max aggregator for source j, pulled over the block's
// transpose: d_src[j, c] = [j < n_dst] d_a[j, c] + the sum of d_a[i, f + c]
// over the distinct rows i that sampled j with argmax[i, c] = j, then the
// ReLU mask.  A row that sampled j several times sits in consecutive entries
// of j's column (the columns are in ascending row order), and only the
// first of them counts: the maximum passes its gradient once.  The
// neighbour rows of d_a are read only for elements that j won.
template <class THB, bool VEC>
__device__ __forceinline__ void agg_bwd_row_max(int64_t n_dst, const int32_t *__restrict__ cscrow,
                                                const int32_t *__restrict__ argmax, const float *__restrict__ d_a,
                                                int64_t f, int C, const RowLanes &L,
                                                const THB *__restrict__ h_below, float *__restrict__ d_src, int64_t j,
                                                int64_t beg, int32_t len) {
    const int64_t ka = 2 * f;
    const int32_t jj = static_cast<int32_t>(j);
    const bool mask = h_below != nullptr;
    for (int chunk = L.chunk; chunk < C; chunk += 64) {
        const uint32_t e0 = static_cast<uint32_t>(chunk) * 4;
        float4 self, hb;
        if (j < n_dst) self = load_chunk<VEC>(d_a + j * ka, 0, e0, f);
        if (mask) hb = load_chunk<VEC>(h_below + j * f, 0, e0, f);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        int32_t before = -1;  // the last entry's row
        for (int32_t t = 0; t < len; t += 4) {
            int32_t i[4];
            int4 a[4];
            float4 v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (t + q < len) i[q] = cscrow[beg + t + q];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (t + q < len) {
                    i[q] = __builtin_amdgcn_readfirstlane(i[q]);
                    a[q] = load_arg4<VEC>(argmax + static_cast<int64_t>(i[q]) * f, 0, e0, f, -1);
                }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (t + q >= len) continue;
                const bool first = i[q] != before;
                before = i[q];
                a[q].x = first && a[q].x == jj;
                a[q].y = first && a[q].y == jj;
                a[q].z = first && a[q].z == jj;
                a[q].w = first && a[q].w == jj;
                if (a[q].x | a[q].y | a[q].z | a[q].w)
                    v[q] = load_chunk<VEC>(d_a + (static_cast<int64_t>(i[q]) * ka + f), 0, e0, f);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (t + q >= len || !(a[q].x | a[q].y | a[q].z | a[q].w)) continue;
                acc.x += a[q].x ? v[q].x : 0.f;
                acc.y += a[q].y ? v[q].y : 0.f;
                acc.z += a[q].z ? v[q].z : 0.f;
                acc.w += a[q].w ? v[q].w : 0.f;
            }
        }
        finish_grad<VEC>(acc, 1.f, self, hb, n_dst, mask, f, e0, d_src, j);
    }
}

// agg_bwd_part for the maximum.
template <bool VEC>
__device__ __forceinline__ float4 agg_bwd_part_max(const int32_t *__restrict__ cscrow,
                                                   const int32_t *__restrict__ argmax, const float *__restrict__ d_a,
                                                   int64_t f, uint32_t e0, int32_t j, uint32_t len, uint32_t t0,
                                                   uint32_t step) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (uint32_t t = t0; t < len; t += 4 * step) {
        int32_t i[4];
        int4 a[4];
        float4 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t u = t + q * step;
            i[q] = -1;
            if (u >= len) continue;
            i[q] = cscrow[u];
            if (u > 0 && cscrow[u - 1] == i[q]) i[q] = -1;  // a row's second and later entries
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (i[q] >= 0) a[q] = load_arg4<VEC>(argmax + static_cast<int64_t>(i[q]) * f, 0, e0, f, -1);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (i[q] >= 0 && (a[q].x == j || a[q].y == j || a[q].z == j || a[q].w == j))
                v[q] = load_chunk<VEC>(d_a + (static_cast<int64_t>(i[q]) * 2 * f + f), 0, e0, f);
        float4 pair[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (i[q] < 0) continue;
            pair[q / 2].x += a[q].x == j ? v[q].x : 0.f;
            pair[q / 2].y += a[q].y == j ? v[q].y : 0.f;
            pair[q / 2].z += a[q].z == j ? v[q].z : 0.f;
            pair[q / 2].w += a[q].w == j ? v[q].w : 0.f;
        }
        add4(acc, pair[0], pair[1]);
    }
    return acc;
}

// A long column of the maximum's backward, by the whole workgroup
// (agg_bwd_long's split and order).
template <class THB>
__device__ __forceinline__ void agg_bwd_long_max(int64_t n_dst, const int32_t *__restrict__ cscrow,
                                                 const int32_t *__restrict__ argmax, const float *__restrict__ d_a,
                                                 int64_t f, const THB *__restrict__ h_below,
                                                 float *__restrict__ d_src, int64_t j, int64_t beg, int64_t end) {
    const int lane = threadIdx.x & 63;
    const int64_t ka = 2 * f;
    const int32_t jj = static_cast<int32_t>(j);
    for (uint32_t e0 = threadIdx.x - lane; e0 < f; e0 += kThreads) {
        const uint32_t e = min(e0 + lane, static_cast<uint32_t>(f) - 1);
        const float self = (d_a + (j < n_dst ? j : 0) * ka)[e];
        const float hb = h_below ? Elem<THB>::load(h_below + j * f, e) : 1.f;
        float acc = 0.f;
        for (int64_t wb = beg; wb < end; wb += 64) {
            const int wn = static_cast<int>(min<int64_t>(64, end - wb));
            // a row's second and later entries count as no row (-1)
            int32_t my_idx = -1;
            if (lane < wn) {
                my_idx = cscrow[wb + lane];
                if (wb + lane > beg && cscrow[wb + lane - 1] == my_idx) my_idx = -1;
            }
            for (int tb = 0; tb < wn; tb += kLongAhead) {
                int32_t a[kLongAhead];
                float v[kLongAhead];
#pragma unroll
                for (int u = 0; u < kLongAhead; ++u) {
                    const int64_t i = __builtin_amdgcn_readlane(my_idx, tb + u);
                    a[u] = (argmax + (i < 0 ? 0 : i) * f)[e];
                }
#pragma unroll
                for (int u = 0; u < kLongAhead; ++u) {
                    const int64_t i = __builtin_amdgcn_readlane(my_idx, tb + u);
                    v[u] = 0.f;
                    if (i >= 0 && a[u] == jj) v[u] = (d_a + i * ka + f)[e];
                }
#pragma unroll
                for (int u = 0; u < kLongAhead; ++u) acc += v[u];
            }
        }
        if (j < n_dst) acc += self;
        if (!(hb > 0.f)) acc = 0.f;
        if (e0 + lane < f) (d_src + j * f)[e] = acc;
    }
}

template <class TIn, class TOut, bool VEC>
struct FwdMaxJob {
    gnn_block b;
    const TIn *h;
    int64_t f;
    int C, S;
    TOut *out;
    int32_t *argmax;
    __device__ void run(int64_t blk, int64_t nblk) const {
        const int64_t n = b.counts[0];
        for (int64_t row = blk * kWaves + (threadIdx.x >> 6); row < n; row += nblk * kWaves)
            agg_fwd_row_max<TIn, TOut, VEC>(b.rowptr, b.col, h, f, C, S, out, argmax, row);
    }
};

template <class THB, bool VEC, bool UNI>
struct BwdMaxJob {
    gnn_block b;
    const int32_t *argmax;
    const float *d_a;
    int64_t f;
    int C, R;
    const THB *h_below;
    float *d_src;
    static constexpr int kWavesPerSimd = VEC && UNI ? 8 : 1;
    __device__ void run(int64_t blk, int64_t nblk) const {
        const int64_t n_dst = b.counts[0];
        if constexpr (UNI) {
            const RowLanes L(C, 1, 1);
            walk_columns(
                b, blk, nblk, L,
                [&](int64_t j, int64_t beg, int32_t len) {
                    agg_bwd_row_max<THB, VEC>(n_dst, b.cscrow, argmax, d_a, f, C, L, h_below, d_src, j, beg, len);
                },
                [&](int64_t j, int64_t beg, int64_t end) {
                    agg_bwd_long_max<THB>(n_dst, b.cscrow, argmax, d_a, f, h_below, d_src, j, beg, end);
                });
        } else {
            walk_narrow(
                b, blk, nblk, C, R,
                [&](uint32_t e0, int64_t j, int64_t beg, int32_t len, int32_t t0, int32_t step) {
                    return agg_bwd_part_max<VEC>(b.cscrow + beg, argmax, d_a, f, e0, static_cast<int32_t>(j), len, t0,
                                                 step);
                },
                [&](uint32_t e0, int64_t j) { return own_terms<THB, VEC>(n_dst, d_a, 2 * f, h_below, f, e0, j); },
                [&](uint32_t e0, int64_t j, const float4 &sum, const OwnTerms &o) {
                    finish_grad<VEC>(sum, 1.f, o.self, o.hb, n_dst, h_below != nullptr, f, e0, d_src, j);
                });
        }
    }
};

inline void split_row(int64_t f, int *C, int *S) {
    const int64_t c = ceil_div(f, 4);
    *C = static_cast<int>(c);
    *S = (c <= 32) ? static_cast<int>(64 / c) : 1;
}

// Rows per wavefront when each takes ceil(f / 4) lanes.
inline int rows_per_wave(int64_t f) { return static_cast<int>(std::max<int64_t>(1, 64 / ceil_div(f, 4))); }

inline unsigned row_grid(int64_t rows) {
    return static_cast<unsigned>(std::min<int64_t>(ceil_div(rows > 0 ? rows : 1, kWaves), kMaxBlocks));
}

// f(job) with the table-reading forward job (fp32 table -> bf16 output).
template <class F>
void with_fwd_table_job(const gnn_block *b, int kind, const int64_t *gids, int32_t k, const float *gcn_norm,
                        const float *table, int64_t row_stride, const uint16_t *x_self, int64_t f, uint16_t *out,
                        F &&fn) {
    int C, S;
    split_row(f, &C, &S);
    const bool vec = (f % 4 == 0) && (row_stride % 4 == 0) && aligned(table, 16) && aligned(x_self, 8) &&
                     aligned(out, 8);
    auto go = [&](auto kind_tag) {
        constexpr int KIND = decltype(kind_tag)::value;
        const TableEdges edges{gids, k, gcn_norm, table, row_stride};
        if (vec) fn(FwdTableJob<KIND, true>{*b, edges, x_self, f, C, S, out});
        else fn(FwdTableJob<KIND, false>{*b, edges, x_self, f, C, S, out});
    };
    if (kind == GNN_AGG_SAGE_MEAN) go(std::integral_constant<int, GNN_AGG_SAGE_MEAN>{});
    else go(std::integral_constant<int, GNN_AGG_GCN_SYM>{});
}

// f(job) with the forward job for (kind, hdt -> odt); false if unsupported.
template <class F>
bool with_fwd_job(const gnn_block *b, int kind, const void *h, int hdt, int64_t f, void *out, int odt, F &&fn) {
    int C, S;
    split_row(f, &C, &S);
    const bool vec = (f % 4 == 0) && aligned(h, 4 * dtype_size(hdt)) && aligned(out, 4 * dtype_size(odt));
    auto by_kind = [&](auto kind_tag, auto ti_tag, auto to_tag) {
        constexpr int KIND = decltype(kind_tag)::value;
        using TI = typename decltype(ti_tag)::type;
        using TO = typename decltype(to_tag)::type;
        const TI *hp = static_cast<const TI *>(h);
        TO *op = static_cast<TO *>(out);
        if constexpr (sizeof(TI) == 2) {
            // eight elements per lane: even rows of at least eight, dword aligned
            if (f % 2 == 0 && f >= 8 && aligned(h, 4) && aligned(out, 4)) {
                const int CL = static_cast<int>(ceil_div(f, 8)), R = std::max(1, 64 / (S * CL));
                return fn(FwdJob<KIND, TI, TO, 8, false>{*b, hp, f, CL, S, R, op});
            }
        }
        if (vec) fn(FwdJob<KIND, TI, TO, 4, true>{*b, hp, f, C, S, 1, op});
        else fn(FwdJob<KIND, TI, TO, 4, false>{*b, hp, f, C, S, 1, op});
    };
    auto by_types = [&](auto kind_tag) {
        if (hdt == GNN_F32 && odt == GNN_F32) by_kind(kind_tag, Tag<float>{}, Tag<float>{});
        else if (hdt == GNN_F32 && odt == GNN_BF16) by_kind(kind_tag, Tag<float>{}, Tag<uint16_t>{});
        else if (hdt == GNN_BF16 && odt == GNN_F32) by_kind(kind_tag, Tag<uint16_t>{}, Tag<float>{});
        else by_kind(kind_tag, Tag<uint16_t>{}, Tag<uint16_t>{});
    };
    if (!((hdt == GNN_F32 || hdt == GNN_BF16) && (odt == GNN_F32 || odt == GNN_BF16))) return false;
    if (kind == GNN_AGG_SAGE_MEAN) by_types(std::integral_constant<int, GNN_AGG_SAGE_MEAN>{});
    else by_types(std::integral_constant<int, GNN_AGG_GCN_SYM>{});
    return true;
}

// f(job) with the backward job.
template <class F>
void with_bwd_job(const gnn_block *b, int kind, const float *d_a, int64_t f, const void *h_below, int hbdt,
                  float *d_src, F &&fn) {
    const int C = static_cast<int>(ceil_div(f, 4)), R = rows_per_wave(f);
    const bool vec = (f % 4 == 0) && aligned(d_a, 16) && aligned(d_src, 16) &&
                     (!h_below || aligned(h_below, 4 * dtype_size(hbdt)));
    auto by_type = [&](auto kind_tag, auto hb_tag) {
        constexpr int KIND = decltype(kind_tag)::value;
        using THB = typename decltype(hb_tag)::type;
        const THB *hb = static_cast<const THB *>(h_below);
        auto by_rows = [&](auto vec_tag) {
            constexpr bool V = decltype(vec_tag)::value;
            if (R == 1) fn(BwdJob<KIND, THB, V, true>{*b, d_a, f, C, R, hb, d_src});
            else fn(BwdJob<KIND, THB, V, false>{*b, d_a, f, C, R, hb, d_src});
        };
        if (vec) by_rows(std::true_type{});
        else by_rows(std::false_type{});
    };
    auto by_kind = [&](auto kind_tag) {
        if (!h_below || hbdt == GNN_F32) by_type(kind_tag, Tag<float>{});
        else by_type(kind_tag, Tag<uint16_t>{});
    };
    if (kind == GNN_AGG_SAGE_MEAN) by_kind(std::integral_constant<int, GNN_AGG_SAGE_MEAN>{});
    else by_kind(std::integral_constant<int, GNN_AGG_GCN_SYM>{});
}

// f(job) with the max aggregator's forward job (argmax may be null: the
// table is not kept); false if the dtypes are unsupported.
template <class F>
bool with_fwd_max_job(const gnn_block *b, const void *h, int hdt, int64_t f, void *out, int odt, int32_t *argmax,
                      F &&fn) {
    int C, S;
    split_row(f, &C, &S);
    const bool vec = (f % 4 == 0) && aligned(h, 4 * dtype_size(hdt)) && aligned(out, 4 * dtype_size(odt)) &&
                     aligned(argmax, 16);
    auto go = [&](auto ti_tag, auto to_tag) {
        using TI = typename decltype(ti_tag)::type;
        using TO = typename decltype(to_tag)::type;
        const TI *hp = static_cast<const TI *>(h);
        TO *op = static_cast<TO *>(out);
        if (vec) fn(FwdMaxJob<TI, TO, true>{*b, hp, f, C, S, op, argmax});
        else fn(FwdMaxJob<TI, TO, false>{*b, hp, f, C, S, op, argmax});
    };
    if (!((hdt == GNN_F32 || hdt == GNN_BF16) && (odt == GNN_F32 || odt == GNN_BF16))) return false;
    if (hdt == GNN_F32 && odt == GNN_F32) go(Tag<float>{}, Tag<float>{});
    else if (hdt == GNN_F32 && odt == GNN_BF16) go(Tag<float>{}, Tag<uint16_t>{});
    else if (hdt == GNN_BF16 && odt == GNN_F32) go(Tag<uint16_t>{}, Tag<float>{});
    else go(Tag<uint16_t>{}, Tag<uint16_t>{});
    return true;
}

// f(job) with the forward job of any aggregation kind; the max aggregator
// writes its argmax table to argmax (may be null).
template <class F>
bool with_fwd_kind_job(const gnn_block *b, int kind, const void *h, int hdt, int64_t f, void *out, int odt,
                       int32_t *argmax, F &&fn) {
    if (kind == GNN_AGG_SAGE_MAX) return with_fwd_max_job(b, h, hdt, f, out, odt, argmax, fn);
    return with_fwd_job(b, kind, h, hdt, f, out, odt, fn);
}

template <class F>
void with_bwd_max_job(const gnn_block *b, const int32_t *argmax, const float *d_a, int64_t f, const void *h_below,
                      int hbdt, float *d_src, F &&fn) {
    const int C = static_cast<int>(ceil_div(f, 4)), R = rows_per_wave(f);
    const bool vec = (f % 4 == 0) && aligned(d_a, 16) && aligned(d_src, 16) && aligned(argmax, 16) &&
                     (!h_below || aligned(h_below, 4 * dtype_size(hbdt)));
    auto go = [&](auto hb_tag) {
        using THB = typename decltype(hb_tag)::type;
        const THB *hb = static_cast<const THB *>(h_below);
        auto by_rows = [&](auto vec_tag) {
            constexpr bool V = decltype(vec_tag)::value;
            if (R == 1) fn(BwdMaxJob<THB, V, true>{*b, argmax, d_a, f, C, R, hb, d_src});
            else fn(BwdMaxJob<THB, V, false>{*b, argmax, d_a, f, C, R, hb, d_src});
        };
        if (vec) by_rows(std::true_type{});
        else by_rows(std::false_type{});
    };
    if (!h_below || hbdt == GNN_F32) go(Tag<float>{});
    else go(Tag<uint16_t>{});
}

}  // namespace agg
}  // namespace gnn
