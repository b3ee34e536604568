// Transpose of a sampled block (its CSC: for every local source, the rows
// that sampled it, in ascending row order), the structure the aggregation
// backward reads so that it gathers instead of scattering.
//
// Four phases, each a job (see jobs.h) that a step can run alongside other
// work, so the transpose costs no launch of its own:
//   count  per-column edge counts (atomic increments; done by the relabel of
//          the hop, which produces the edges' columns, into counters that
//          the hop's prepare cleared), each edge keeping its number in its
//          column (the order inside a column is arbitrary here)
//   scan   column pointers: exclusive scan of the counts, single pass with
//          ticket-ordered look-back
//   place  every edge to its slot of its column
//   sort   every column in ascending row order, which makes the result
//          unique: columns of up to kShort entries by one lane with a
//          sorting network, longer ones by a wavefront, the longest by the
//          workgroup
// Every index a phase derives
// from device data is range-checked; a violation flags samp::kErrRange in
// counts[3] and skips the access.
#pragma once

#include <type_traits>

#include "internal.h"
#include "sampler_dev.h"

namespace gnn {
namespace csc {

constexpr int kThreads = 256;
constexpr int kPer = 8;                          // columns per thread in the scan
constexpr int64_t kScanTile = kThreads * kPer;   // columns per scan workgroup
constexpr int kShort = 16;                       // longest column sorted by one lane

struct Args {
    int64_t *counts;         // block counts: n_dst, n_src, nnz, error flag
    const int32_t *bcol;     // [nnz] column (local source) of each edge
    int32_t *erow;           // [cap_nnz] row of each edge; scratch of the sort
    int32_t *eslot;          // [cap_nnz] number of each edge in its column
    int64_t cap_src, cap_nnz;
    int32_t *cnt;            // [cap_src] per-column counters
    uint64_t *status;        // [nb_scan] look-back words
    int *ticket;
    int64_t nb_scan;
    int64_t *cscptr;         // [cap_src + 1]
    int32_t *cscrow;         // [cap_nnz]
    int64_t cap_dst;         // most rows of the block
};

struct ScanJob {
    Args a;
    __device__ void run(int64_t blk, int64_t) const {
        const int64_t n_src = min(a.counts[1], a.cap_src);
        // workgroups that the capacity-sized grid has too many leave without
        // a ticket (tickets are atomics on one address, 11.5 ns apart)
        if (blk * kScanTile > n_src) return;
        const int64_t t = samp::take_ticket(a.ticket);
        const int64_t j0 = t * kScanTile;
        const int64_t jt = j0 + static_cast<int64_t>(threadIdx.x) * kPer;
        int32_t c[kPer];
        int64_t sum = 0;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int64_t j = jt + q;
            c[q] = j < n_src ? a.cnt[j] : 0;
            sum += c[q];
        }
        int64_t total;
        const int64_t excl = samp::block_excl_scan(sum, &total);
        __shared__ int64_t base;
        if (threadIdx.x < 64) {
            const int64_t b = samp::look_back(a.status, t, total, &a.counts[3]);
            if (threadIdx.x == 0) base = b;
        }
        __syncthreads();
        int64_t run = base + excl;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int64_t j = jt + q;
            if (j <= n_src) a.cscptr[j] = run;
            run += c[q];
        }
    }
};

struct PlaceJob {
    Args a;
    __device__ void run(int64_t blk, int64_t nblk) const {
        const int64_t nnz = min(a.counts[2], a.cap_nnz);
        const int64_t n_src = min(a.counts[1], a.cap_src);
        for (int64_t e = blk * kThreads + threadIdx.x; e < nnz; e += nblk * kThreads) {
            const int32_t c = a.bcol[e];
            if (c < 0 || c >= n_src) {
                samp::flag_error(&a.counts[3], samp::kErrRange);
                continue;
            }
            const int64_t beg = a.cscptr[c], p = beg + a.eslot[e];
            if (beg < 0 || p < beg || p >= nnz || p >= a.cscptr[c + 1]) {
                samp::flag_error(&a.counts[3], samp::kErrRange);
                continue;
            }
            a.cscrow[p] = a.erow[e];
        }
    }
};

__device__ __forceinline__ void cswap(int32_t &x, int32_t &y) {
    const int32_t lo = min(x, y), hi = max(x, y);
    x = lo;
    y = hi;
}

// One lane: sort seg[0, len) for len <= kShort (bitonic network on
// registers, padded with INT32_MAX).
__device__ __forceinline__ void sort_short(int32_t *seg, int64_t len) {
    int32_t v[kShort];
#pragma unroll
    for (int i = 0; i < kShort; ++i) v[i] = i < len ? seg[i] : INT32_MAX;
#pragma unroll
    for (int k = 2; k <= kShort; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
            for (int i = 0; i < kShort; ++i) {
                const int l = i ^ j;
                if (l > i) {
                    if ((i & k) == 0)
                        cswap(v[i], v[l]);
                    else
                        cswap(v[l], v[i]);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kShort; ++i)
        if (i < len) seg[i] = v[i];
}

// Orders one wavefront's LDS (and its own global) accesses before and after
// the call; the lanes of a wavefront run together, so no workgroup barrier.
__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// One wavefront: sort seg[0, len) for kShort < len <= 64, one entry per lane
// (v: the entry of this lane).  A lane's place is the number of smaller
// entries, equal ones in lane order; len uniform steps of a readlane, a
// compare and an add, with no exchange between lanes to wait for.
__device__ __forceinline__ void sort_wave(int32_t *seg, int32_t v, int len) {
    const int lane = threadIdx.x & 63;
    int rank = 0;
    for (int s = 0; s < len; ++s) {
        const int32_t o = __builtin_amdgcn_readlane(v, s);
        rank += (s < lane ? o <= v : o < v) ? 1 : 0;
    }
    if (lane < len) seg[rank] = v;
}

// Exclusive scan of v over T = 64 (a wavefront) or kThreads threads.
template <int T> __device__ __forceinline__ int excl_scan(int v) {
    if constexpr (T == 64) {
        const int lane = threadIdx.x & 63;
        int inc = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        return inc - v;
    } else {
        int64_t total;
        return static_cast<int>(samp::block_excl_scan(v, &total));
    }
}

// T threads: sort seg[0, n), n <= half, through 2 * half LDS words.  Rows are
// dealt to `half` buckets of equal row ranges; an entry's place is its
// bucket's start plus the smaller entries of its bucket (equal ones in slot
// order).  A hub's rows are spread over the block, so a bucket holds an
// entry or two; a column whose rows crowd into one range costs up to n steps
// per entry and stays correct.
// P: most entries and buckets per thread (n and half at most P T).
template <int T, int P, class Sync>
__device__ __forceinline__ void sort_buckets(uint32_t *words, int half, int32_t *seg, int n, int n_dst, int t,
                                             int64_t *err, Sync &&sync) {
    uint32_t *start = words;
    int32_t *key = reinterpret_cast<int32_t *>(words + half);
    const bool direct = n_dst <= half;  // a bucket per row
    const uint32_t scale =
        direct ? 0u : static_cast<uint32_t>((static_cast<uint64_t>(half) << 32) / static_cast<uint32_t>(n_dst));
    for (int i = t; i < half; i += T) start[i] = 0u;
    int32_t v[P];
    uint32_t b[P], at[P];
#pragma unroll
    for (int e = 0; e < P; ++e) v[e] = t + e * T < n ? seg[t + e * T] : 0;
    sync();
#pragma unroll
    for (int e = 0; e < P; ++e) {
        if (t + e * T >= n) continue;
        const bool ok = v[e] >= 0 && v[e] < n_dst;
        if (!ok) samp::flag_error(err, samp::kErrRange);
        b[e] = !ok ? 0u : direct ? static_cast<uint32_t>(v[e]) : __umulhi(static_cast<uint32_t>(v[e]), scale);
        at[e] = atomicAdd(&start[b[e]], 1u);
    }
    sync();
    // counts -> starts; thread t owns buckets [per t, per (t + 1))
    const int per = half / T;
    uint32_t c[P];
    int sum = 0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        c[q] = q < per ? start[t * per + q] : 0u;
        sum += static_cast<int>(c[q]);
    }
    uint32_t run = static_cast<uint32_t>(excl_scan<T>(sum));
#pragma unroll
    for (int q = 0; q < P; ++q) {
        if (q < per) start[t * per + q] = run;
        run += c[q];
    }
    sync();
#pragma unroll
    for (int e = 0; e < P; ++e)
        if (t + e * T < n) key[start[b[e]] + at[e]] = v[e];
    sync();
#pragma unroll
    for (int e = 0; e < P; ++e) {
        if (t + e * T >= n) continue;
        const uint32_t lo = start[b[e]], hi = b[e] + 1 < static_cast<uint32_t>(half) ? start[b[e] + 1] : n;
        const uint32_t own = lo + at[e];
        uint32_t place = lo;
        for (uint32_t q = lo; q < hi; ++q) place += (key[q] < v[e] || (key[q] == v[e] && q < own)) ? 1u : 0u;
        seg[place] = v[e];
    }
    sync();  // the next segment goes to the same words
}

// A workgroup: the rows of column segment out[0, len) in ascending order by
// counting, 2 * words rows at a time, into 16-bit LDS counters (two per
// word).  The counters are all zero before and after.  Thread t owns `per`
// consecutive words' worth of rows; its word q is at q * kThreads + t, so that
// the walk over the counters is free of bank conflicts.  src is where the
// unsorted rows are read (out itself when one window covers all rows, else a
// copy).
__device__ __forceinline__ void sort_counting(uint32_t *lds, int words, const int32_t *src, int32_t *out, int len,
                                              int n_dst, int64_t *err) {
    const int t = threadIdx.x, per = words / kThreads, window = 2 * words;
    int pos = 0;
    for (int w0 = 0; w0 < n_dst; w0 += window) {
        for (int i = t; i < len; i += kThreads) {
            const int r = src[i];
            if (r < 0 || r >= n_dst) {
                samp::flag_error(err, samp::kErrRange);
                continue;
            }
            const int o = r - w0, w = o >> 1;
            if (o >= 0 && o < window) atomicAdd(&lds[(w % per) * kThreads + w / per], 1u << (16 * (o & 1)));
        }
        __syncthreads();
        int mine = 0;
        for (int q = 0; q < per; ++q) {
            const uint32_t c = lds[q * kThreads + t];
            mine += static_cast<int>((c & 0xffffu) + (c >> 16));
        }
        int64_t total;
        int at = pos + static_cast<int>(samp::block_excl_scan(mine, &total));
        for (int q = 0; mine > 0 && q < per; ++q) {
            const uint32_t c = lds[q * kThreads + t];
            const int r = w0 + 2 * (t * per + q);
            for (uint32_t n = c & 0xffffu; n > 0; --n, ++at)
                if (at < len) out[at] = r;
            for (uint32_t n = c >> 16; n > 0; --n, ++at)
                if (at < len) out[at] = r + 1;
            lds[q * kThreads + t] = 0u;
        }
        pos += static_cast<int>(total);
        __syncthreads();
        if (w0 > n_dst - window) break;  // (w0 + window may not fit an int)
    }
}

// The sort phase.  A workgroup takes 256 columns at a time: a thread sorts
// its column in registers when it is short; longer ones go to two lists, one
// walked by the wavefronts (a column per wavefront) and one by the whole
// workgroup.  It is bound by latency (each list entry is a chain of one load,
// a few LDS passes and one store), so what counts is that few columns follow
// one another in one wavefront and that none walks all rows alone.
// Long columns come from the graph's hubs: a wavefront that counted the rows
// of every column above 16 entries by itself, 1,024 rows per pass, took 223 us
// for the second block of 1,024 targets (7.6k rows, 69k edges, fanouts 25 and
// 10) and 5.5 ms for that of 16,384 targets (83k rows, 719k edges); this form
// takes 10 and 26 us.
//
// P sets the LDS words (512 P) and the entries a thread holds.  2 when the
// block's rows fit one counting window of those words (2,048 rows), 4 up to 16
// windows (65,536 rows), else 8: a larger area keeps the number of windows down
// for hubs of large blocks, but its registers cost occupancy in the launches
// that the sort rides in (at P = 8 99 VGPRs instead of 71 beside layer 1's
// aggregation: a pipelined step of 1,024 targets lost 2.5%, a three-layer step
// takes 277 us with P = 8 for its 16,384-row block and 272 with 4).
template <int P> struct SortJob {
    Args a;
    __device__ void run(int64_t blk, int64_t nblk) const {
        constexpr int words = 512 * P, wave_words = words / (kThreads / 64);
        __shared__ __attribute__((aligned(16))) uint32_t sort_lds[words];
        // wavefront columns from the front, workgroup columns from the back
        __shared__ uint2 list[kThreads];  // segment (from the first column's), length
        __shared__ int wave_n, group_n;
        const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
        const int n_dst = static_cast<int>(min(a.counts[0], a.cap_dst));  // (local ids are 32-bit)
        const int64_t n_src = min(a.counts[1], a.cap_src);
        const int64_t nnz = min(a.counts[2], a.cap_nnz);
        // every thread of the workgroup runs the same rounds
        for (int64_t c0 = blk * kThreads; c0 < n_src; c0 += nblk * kThreads) {
            if (t == 0) wave_n = group_n = 0;
            __syncthreads();
            const int64_t c = c0 + t;
            const int64_t base = a.cscptr[c0];
            int64_t p0 = 0, len = 0;
            if (c < n_src) {
                p0 = a.cscptr[c];
                const int64_t p1 = a.cscptr[c + 1];
                if (base < 0 || p0 < base || p1 < p0 || p1 > nnz || p0 - base > UINT32_MAX || p1 - p0 > INT32_MAX)
                    samp::flag_error(&a.counts[3], samp::kErrRange);
                else
                    len = p1 - p0;
            }
            if (len > kShort) {
                const bool by_wave = len <= wave_words / 2;
                const int at = by_wave ? atomicAdd(&wave_n, 1) : kThreads - 1 - atomicAdd(&group_n, 1);
                list[at] = make_uint2(static_cast<uint32_t>(p0 - base), static_cast<uint32_t>(len));
            } else if (len >= 2) {
                sort_short(a.cscrow + p0, len);
            }
            __syncthreads();
            const int nw = wave_n, ng = group_n;
            for (int i = wave; i < nw; i += kThreads / 64) {
                int32_t *seg = a.cscrow + base + list[i].x;
                const int n = __builtin_amdgcn_readfirstlane(static_cast<int>(list[i].y));
                if (n <= 64)
                    sort_wave(seg, lane < n ? seg[lane] : 0, n);
                else
                    sort_buckets<64, P>(sort_lds + wave * wave_words, wave_words / 2, seg, n, n_dst, lane, &a.counts[3],
                                     [] { wave_sync_lds(); });
            }
            __syncthreads();  // the LDS words change hands
            bool zeroed = false;
            for (int i = 0; i < ng; ++i) {
                const uint2 item = list[kThreads - 1 - i];
                int32_t *out = a.cscrow + base + item.x;
                const int n = static_cast<int>(item.y);
                if constexpr (P > 2) {  // (at P = 2 one window holds all rows)
                    if (n_dst > 2 * words && n <= words / 2) {
                        sort_buckets<kThreads, P>(sort_lds, words / 2, out, n, n_dst, t, &a.counts[3],
                                                  [] { __syncthreads(); });
                        zeroed = false;
                        continue;
                    }
                }
                if (!zeroed)
                    for (int o = t; o < words; o += kThreads) sort_lds[o] = 0u;
                zeroed = true;
                const int32_t *src = out;
                if (n_dst > 2 * words) {
                    // several windows read the rows again: keep a copy in the
                    // edge-row scratch (free once the edges are placed)
                    int32_t *copy = a.erow + base + item.x;
                    for (int e = t; e < n; e += kThreads) copy[e] = out[e];
                    src = copy;
                }
                __syncthreads();
                sort_counting(sort_lds, words, src, out, n, n_dst, &a.counts[3]);
            }
            __syncthreads();  // the lists are free for the next round
        }
    }
};
// f(tag) with the P (an integral constant) of a block of cap_dst rows.
template <class F> void with_sort_size(int64_t cap_dst, F &&f) {
    if (cap_dst <= 2048) f(std::integral_constant<int, 2>{});
    else if (cap_dst <= 65536) f(std::integral_constant<int, 4>{});
    else f(std::integral_constant<int, 8>{});
}

struct Grids {
    unsigned scan, place, sort;
};

}  // namespace csc

// Host side (sampler.hip).  The transpose scratch of one block: the row of
// every edge, the per-column counters and the scan's look-back state.
size_t block_csc_ws_bytes(int64_t cap_src, int64_t cap_nnz);
// Arguments of the block's transpose in scratch sized for (ws_src, ws_nnz);
// the capacities used are the smaller of the block's and the scratch's.
csc::Args csc_args(const gnn_block *out, void *csc_ws, int64_t ws_src, int64_t ws_nnz);
csc::Grids csc_grids(const csc::Args &a);
// The scan, place and sort phases as three launches (after the relabel that
// counted).
gnn_status launch_block_csc(const csc::Args &a, hipStream_t s);

}  // namespace gnn
