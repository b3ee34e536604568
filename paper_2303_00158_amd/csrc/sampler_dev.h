// Device side of the sampler (see sampler.hip): the hop's argument block and
// the bodies of its kernels, each taking its logical workgroup index and
// count so that a launch can run it alongside other work.
#pragma once

#include "internal.h"

namespace gnn {
namespace csc {
struct Args;
}
namespace samp {

constexpr int kThreads = 256;
// Marks of the sampled vertices and of the destinations, a map each: a byte per
// vertex where a hop may mark an eighth of the graph or more, else a bit.
// Bytes are set with plain stores, bits with device-wide atomics (720k marks
// on the 2.4M-vertex graph: 7 us as bytes, 30-38 us as bits), but the emit phase
// reads eight times less of the bits: with bytes the blocks of 1,024 targets
// (77k marks) took 10.8 us to emit instead of 8.8.  The maps have room for bytes
// up to kByteMarks vertices and are all zero between hops, so hops of either
// kind share them.
constexpr int64_t kByteMarks = 64 << 20;
__host__ __device__ inline bool byte_marks(int64_t graph_n, int64_t cap_nnz) {
    return graph_n <= kByteMarks && cap_nnz >= graph_n / 8;
}
// marks per thread in the emit phase, in words of 32 vertices
constexpr int kBitWords = 8, kByteWords = 1;
constexpr uint64_t kFlagAgg = 1ull << 62, kFlagPrefix = 2ull << 62, kValueMask = (1ull << 62) - 1;
constexpr uint32_t kSpinLimit = 1u << 22;

__host__ __device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t load_status(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_status(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Logical workgroup index: the order in which workgroups started.
__device__ __forceinline__ int64_t take_ticket(int *ticket) {
    __shared__ int64_t t;
    if (threadIdx.x == 0) t = atomicAdd(ticket, 1);
    __syncthreads();
    return t;
}

__device__ __forceinline__ int64_t wave_sum64(int64_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Device error flags of a block (its counts[3]; gnn.h names them): set
// with an atomic OR, so that concurrent checks keep every flag.
constexpr int64_t kErrWait = 1;   // a bounded wait for an earlier workgroup gave up
constexpr int64_t kErrRange = 2;  // an index derived from device data was out of range
__device__ __forceinline__ void flag_error(int64_t *err, int64_t flag) {
    atomicOr(reinterpret_cast<unsigned long long *>(err), static_cast<unsigned long long>(flag));
}

// Called by all 64 lanes of one wavefront: publish this workgroup's
// aggregate, add up the aggregates / prefixes of earlier tickets 64 at a
// time (lane j reads ticket blk-1-j-64w), publish the inclusive prefix, and
// return the exclusive prefix.  Waits for an earlier ticket give up after
// spin_limit polls and flag kErrWait.  `silent` (normally -1) names a ticket
// that publishes nothing: a host-driven test of that path.
__device__ inline int64_t look_back(uint64_t *status, int64_t blk, int64_t agg, int64_t *err,
                                    uint32_t spin_limit = kSpinLimit, int64_t silent = -1) {
    const int lane = threadIdx.x & 63;
    const bool publish = blk != silent;
    if (blk == 0) {
        if (lane == 0 && publish) store_status(&status[0], kFlagPrefix | static_cast<uint64_t>(agg));
        return 0;
    }
    if (lane == 0 && publish) store_status(&status[blk], kFlagAgg | static_cast<uint64_t>(agg));
    int64_t excl = 0;
    int64_t hi = blk - 1;
    uint32_t spins = 0;
    while (true) {
        const int64_t p = hi - lane;
        // tickets before 0 read as a zero prefix, which ends every walk
        const uint64_t s = p >= 0 ? load_status(&status[p]) : kFlagPrefix;
        const uint64_t flag = s & ~kValueMask;
        const uint64_t pre = __ballot(flag == kFlagPrefix);
        const int first = pre ? static_cast<int>(__builtin_ctzll(pre)) : 63;
        const uint64_t need = (first == 63) ? ~0ull : ((1ull << (first + 1)) - 1);
        if (__ballot(flag == 0) & need) {
            if (++spins > spin_limit) {
                if (lane == 0) flag_error(err, kErrWait);  // an earlier workgroup never published
                break;
            }
            continue;
        }
        excl += wave_sum64(lane <= first ? static_cast<int64_t>(s & kValueMask) : 0);
        if (pre) break;
        hi -= 64;
    }
    if (lane == 0 && publish) store_status(&status[blk], kFlagPrefix | static_cast<uint64_t>(excl + agg));
    return excl;
}

__device__ __forceinline__ int64_t block_excl_scan(int64_t v, int64_t *total) {
    __shared__ int64_t sh[kThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) sh[wave] = inc;
    __syncthreads();
    int64_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) {
        if (w < wave) base += sh[w];
        tot += sh[w];
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

struct HopArgs {
    const int64_t *rowptr, *col;  // graph
    const float *gcn_norm;        // per vertex, or null
    const int64_t *dst;
    const int64_t *n_dst_dev;
    int64_t cap_dst;
    int32_t k;
    uint64_t key;                 // mix(mix(mix(seed) ^ step) ^ hop)
    // block
    int64_t *counts, *src_ids, *brow;
    int32_t *bcol;
    float *src_norm;
    // workspace
    int32_t *map;
    uint32_t *bits, *dbits;  // marks
    bool bytes;              // ... a byte each, else a bit
    int64_t graph_n;
    int64_t *gpad;      // [cap_dst][k] sampled global ids
    int32_t *cnt;       // [cap_dst] sample counts
    int32_t *erow;      // [cap_nnz] row of each edge (for the transpose) or null
    int32_t *eslot;     // [cap_nnz] the edge's number in its column, with erow
    uint64_t *status;   // [nb_rows + nb_bits] look-back words
    int *ticket;        // two: the row scan's and, 64 ints on, the sources'
    int64_t nb_rows, nb_bits;
    // count phase of the transpose (when erow is set): per-column counters
    // and the transpose scan's look-back state, reset by the prepare
    int32_t *csc_cnt;
    int64_t csc_cap_src;
    uint64_t *csc_status;
    int *csc_ticket;
    int64_t csc_nb;
    // the row scan's bounded wait (kSpinLimit polls) and its silent ticket
    // (-1: none), changed only by the host's error-path test hook
    uint32_t spin_limit;
    int64_t silent_row_tile;
};

constexpr int kTicketStride = 64;  // ints between the emit phase's two tickets

__device__ __forceinline__ void set_mark(uint32_t *marks, bool bytes, int64_t v) {
    if (bytes)
        reinterpret_cast<uint8_t *>(marks)[v] = 1;
    else
        atomicOr(&marks[v >> 5], 1u << (v & 31));
}

// 1. prepare: reset of the later phases' state, shared by the grid.
__device__ __forceinline__ int64_t hop_prepare_reset(const HopArgs &a, int64_t gtid, int64_t gsize) {
    const int64_t n_dst = a.n_dst_dev ? min(*a.n_dst_dev, a.cap_dst) : a.cap_dst;
    // the look-back state of the emit kernel and, for a block with a
    // transpose, its column counters and scan state
    for (int64_t i = gtid; i < a.nb_rows + a.nb_bits; i += gsize) a.status[i] = 0;
    if (a.erow) {
        for (int64_t i = gtid; i < a.csc_cap_src; i += gsize) a.csc_cnt[i] = 0;
        for (int64_t i = gtid; i < a.csc_nb; i += gsize) a.csc_status[i] = 0;
        if (gtid == 0) *a.csc_ticket = 0;
    }
    if (gtid == 0) {
        a.ticket[0] = 0;
        a.ticket[kTicketStride] = 0;
        a.counts[0] = n_dst;
        a.counts[3] = 0;
    }
    return n_dst;
}

// What a destination row records of itself (one thread per row).
__device__ __forceinline__ void hop_prepare_dst(const HopArgs &a, int64_t row, int64_t v, int64_t d) {
    a.map[v] = static_cast<int32_t>(row);
    a.src_ids[row] = v;
    if (a.src_norm) a.src_norm[row] = a.gcn_norm[v];
    a.cnt[row] = static_cast<int32_t>(d < a.k ? d : a.k);
    set_mark(a.dbits, a.bytes, v);
}

// Fanouts of up to G = 16 or 32: G lanes per destination row, draw t of the row
// in lane t of its group.  The kernel is bound by latency (destination id, row
// pointer, neighbour id: three dependent loads per row), so 64 / G rows per
// wavefront shorten the chain of rows that a wavefront walks: 83k rows with
// fanout 10 took 52 us with a wavefront per row, now 29 us.
//
// Floyd's algorithm without its draw-by-draw chain: draw t takes x_t unless
// that is among the values taken by draws s < t, and else j_t = d - k + t.  A
// value equal to x_t is there exactly when some x_s = x_t (draw s took it, or
// found it taken), or when draw s = x_t - (d - k) < t took its j_s, which only
// a draw that had to give way did.  The first test needs no order; the second
// refers to an earlier draw's outcome, so it is repeated until it settles (a
// chain of draws that gave way, nearly always none).
template <int G>
__device__ __forceinline__ void hop_prepare_group(const HopArgs &a, int64_t blk, int64_t nblk) {
    const int64_t gtid = blk * kThreads + threadIdx.x, gsize = nblk * kThreads;
    const int64_t n_dst = hop_prepare_reset(a, gtid, gsize);
    const int lane = threadIdx.x & 63, g = lane & (G - 1), first = lane - g;
    const int32_t k = a.k;
    // every lane of a wavefront runs the same rounds (row0 is the wavefront's)
    for (int64_t row0 = gtid / 64 * (64 / G); row0 < n_dst; row0 += gsize / G) {
        const int64_t row = row0 + lane / G;
        const bool live = row < n_dst;
        const int64_t v = a.dst[live ? row : row0];
        const int64_t beg = a.rowptr[v];
        const int64_t d = a.rowptr[v + 1] - beg;
        if (live && g == 0) hop_prepare_dst(a, row, v, d);
        // lanes past the row's draws take part in the exchanges only
        const bool draws = live && d > k && g < k;
        const uint64_t pk = mix64(a.key ^ static_cast<uint64_t>(v));
        const uint32_t low = static_cast<uint32_t>(d - k);  // (degrees are below 2^32)
        const uint64_t j = static_cast<uint64_t>(d - k + g);
        const uint32_t x = static_cast<uint32_t>(((mix64(pk ^ static_cast<uint64_t>(g)) >> 32) * (j + 1)) >> 32);
        bool taken = false;
#pragma unroll 8
        for (int s = 0; s < k; ++s) {
            const uint32_t xs = __shfl(x, first + s, 64);
            taken |= s < g && xs == x;
        }
        taken &= draws;
        const uint32_t ref = x - low;  // the draw whose j equals x, if x >= low
        const bool refers = draws && x >= low && ref < static_cast<uint32_t>(g);
        while (true) {
            const uint64_t m = __ballot(taken);
            const bool now = taken || (refers && ((m >> (first + (refers ? ref : 0u))) & 1ull));
            if (__ballot(now != taken) == 0) break;
            taken = now;
        }
        const uint32_t val = taken ? static_cast<uint32_t>(j) : x;
        // rank of each drawn position among all k (they are distinct)
        int rank = 0;
#pragma unroll 8
        for (int s = 0; s < k; ++s) rank += __shfl(val, first + s, 64) < val ? 1 : 0;
        const bool whole = live && d <= k && g < d;  // a row kept whole
        if (draws || whole) {
            const int64_t u = a.col[beg + (whole ? static_cast<uint32_t>(g) : val)];
            a.gpad[row * k + (whole ? g : rank)] = u;
            set_mark(a.bits, a.bytes, u);
        }
    }
}

// Larger fanouts: one wavefront per destination row.  R drawn positions per
// lane (slot s lives in lane s % 64, register s / 64).
template <int R>
__device__ __forceinline__ void hop_prepare_wave(const HopArgs &a, int64_t blk, int64_t nblk) {
    const int64_t gtid = blk * kThreads + threadIdx.x;
    const int64_t gsize = nblk * kThreads;
    const int64_t n_dst = hop_prepare_reset(a, gtid, gsize);
    const int lane = threadIdx.x & 63;
    // one destination row per wavefront, the grid's wavefronts striding
    // over the rows (the row is uniform per wavefront)
    for (int64_t row = gtid >> 6; row < n_dst; row += gsize >> 6) {
        const int64_t v = a.dst[row];
        const int64_t beg = a.rowptr[v];
        const int64_t d = a.rowptr[v + 1] - beg;
        const int32_t k = a.k;
        int64_t *out = a.gpad + row * k;
        if (lane == 0) hop_prepare_dst(a, row, v, d);
        if (d <= k) {
            for (int64_t p = lane; p < d; p += 64) {
                const int64_t u = a.col[beg + p];
                out[p] = u;
                set_mark(a.bits, a.bytes, u);
            }
            continue;
        }
        uint32_t slot[R];
#pragma unroll
        for (int r = 0; r < R; ++r) slot[r] = 0xffffffffu;
        const uint64_t pk = mix64(a.key ^ static_cast<uint64_t>(v));
        // The draws' candidates x_t = floor(u_t (j_t + 1)) do not depend on
        // one another: lane t computes draw t's hash (register t / 64), and
        // only the membership test below runs draw by draw.
        uint32_t cand[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t t = r * 64 + lane;
            const uint64_t j = static_cast<uint64_t>(d - k + t);
            const uint64_t key = mix64(pk ^ static_cast<uint64_t>(t));
            cand[r] = static_cast<uint32_t>(((key >> 32) * (j + 1)) >> 32);
        }
        for (int32_t t = 0; t < k; ++t) {
            const uint64_t j = static_cast<uint64_t>(d - k + t);
            uint32_t cr = 0;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (r == (t >> 6)) cr = cand[r];
            const uint32_t x = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(cr), t & 63));
            bool mine = false;
#pragma unroll
            for (int r = 0; r < R; ++r) mine |= (r * 64 + lane < t) && (slot[r] == x);
            const bool found = __ballot(mine) != 0ull;
            const uint32_t val = found ? static_cast<uint32_t>(j) : x;
            if (lane == (t & 63)) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (r == (t >> 6)) slot[r] = val;
            }
        }
        // rank of each drawn position among all k (they are distinct)
        int rank[R];
#pragma unroll
        for (int r = 0; r < R; ++r) rank[r] = 0;
        for (int32_t s = 0; s < k; ++s) {
            uint32_t mine = 0;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (r == (s >> 6)) mine = slot[r];
            const uint32_t other = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mine), s & 63));
#pragma unroll
            for (int r = 0; r < R; ++r) rank[r] += (other < slot[r]) ? 1 : 0;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r * 64 + lane < k) {
                const int64_t u = a.col[beg + slot[r]];
                out[rank[r]] = u;
                set_mark(a.bits, a.bytes, u);
            }
        }
    }
}

// The row tiles of the emit phase that hold rows (at least one).
__device__ __forceinline__ int64_t row_tiles(int64_t n_dst) { return n_dst > 0 ? ceil_div(n_dst, kThreads) : 1; }

// 2a. row pointer of the block: scan of the sample counts (logical block
// `blk` owns rows [256 blk, 256 blk + 256)).
__device__ __forceinline__ void emit_rows(const HopArgs &a, int64_t blk, int64_t n_dst) {
    const int64_t i = blk * kThreads + threadIdx.x;
    const int64_t c = (i < n_dst) ? a.cnt[i] : 0;
    int64_t total;
    const int64_t excl_in_block = block_excl_scan(c, &total);
    __shared__ int64_t base;
    if (threadIdx.x < 64) {
        const int64_t b = look_back(a.status, blk, total, &a.counts[3], a.spin_limit, a.silent_row_tile);
        if (threadIdx.x == 0) base = b;
    }
    __syncthreads();
    if (i < n_dst) a.brow[i + 1] = base + excl_in_block + c;
    if (blk == 0 && threadIdx.x == 0) a.brow[0] = 0;
    if (blk == row_tiles(n_dst) - 1 && threadIdx.x == 0) a.counts[2] = base + total;
}

// Bit i of the result: byte i of the 32 bytes at p is set (they hold 0 or 1).
__device__ __forceinline__ uint32_t marks_of_bytes(const uint4 &lo, const uint4 &hi) {
    const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    uint32_t m = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const uint32_t x = w[q];
        m |= ((x & 1u) | ((x >> 7) & 2u) | ((x >> 14) & 4u) | ((x >> 21) & 8u)) << (4 * q);
    }
    return m;
}
__device__ __forceinline__ bool any_mark(const uint4 &v) { return (v.x | v.y | v.z | v.w) != 0u; }

// 2b. new sources in ascending vertex order (logical block `blk` owns
// 32 W kThreads vertices, a thread 32 W of them; the maps are padded to whole
// words of 32 vertices); the marks are cleared.  A thread writes its new
// sources one after another, so many threads with few vertices each are what
// keeps this short where a block marks much of the graph: 256 vertices per
// thread (38 workgroups) took 68 us for the 180k new sources of 16,384
// targets, 32 take 17 us.
template <bool BYTES, int W>
__device__ __forceinline__ void emit_sources(const HopArgs &a, int64_t blk, int64_t n_dst) {
    const int64_t words = ceil_div(a.graph_n, 32);
    const int64_t w0 = (blk * kThreads + threadIdx.x) * W;
    uint32_t sw[W], dw[W];
    if constexpr (BYTES) {
        static_assert(W == 1, "a thread reads the bytes of one word");
        const int64_t w = w0 < words ? w0 : 0;
        uint4 *sp = reinterpret_cast<uint4 *>(a.bits) + 2 * w, *dp = reinterpret_cast<uint4 *>(a.dbits) + 2 * w;
        const uint4 s0 = sp[0], s1 = sp[1], d0 = dp[0], d1 = dp[1];
        sw[0] = marks_of_bytes(s0, s1);
        dw[0] = marks_of_bytes(d0, d1);
        if (w0 < words) {
            const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
            if (any_mark(s0)) sp[0] = zero;
            if (any_mark(s1)) sp[1] = zero;
            if (any_mark(d0)) dp[0] = zero;
            if (any_mark(d1)) dp[1] = zero;
        }
    } else {
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int64_t w = (w0 + q < words) ? w0 + q : 0;
            sw[q] = a.bits[w];
            dw[q] = a.dbits[w];
        }
    }
    int64_t c = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        if (w0 + q >= words) sw[q] = dw[q] = 0u;
        c += __popc(sw[q] & ~dw[q]);
    }
    int64_t total;
    const int64_t excl_in_block = block_excl_scan(c, &total);
    __shared__ int64_t base;
    if (threadIdx.x < 64) {
        const int64_t b = look_back(a.status + a.nb_rows, blk, total, &a.counts[3]);
        if (threadIdx.x == 0) base = b;
    }
    __syncthreads();
    int64_t r = n_dst + base + excl_in_block;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        uint32_t m = sw[q] & ~dw[q];
        const int64_t wbase = (w0 + q) * 32;
        while (m) {
            const int b = __builtin_ctz(m);
            m &= m - 1;
            const int64_t u = wbase + b;
            a.src_ids[r] = u;
            a.map[u] = static_cast<int32_t>(r);
            if (a.src_norm) a.src_norm[r] = a.gcn_norm[u];
            ++r;
        }
        if constexpr (!BYTES) {
            if (sw[q]) a.bits[w0 + q] = 0u;
            if (dw[q]) a.dbits[w0 + q] = 0u;
        }
    }
    if (blk == a.nb_bits - 1 && threadIdx.x == 0) a.counts[1] = n_dst + base + total;
}

// 2. one launch, two roles: as many workgroups as there are tiles with rows
// scan the rows, the next nb_bits emit the new sources, the rest of the
// capacity-sized grid has nothing to do and leaves without a ticket (tickets
// are atomics on one address, 11.5 ns apart: the 1,700 of a 425,984-row
// capacity took 20 us).  The role is uniform per workgroup.
__device__ __forceinline__ void hop_emit_body(const HopArgs &a, int64_t blk) {
    const int64_t n_dst = a.counts[0];
    const int64_t rows = row_tiles(n_dst);
    if (blk < rows) {
        emit_rows(a, take_ticket(a.ticket), n_dst);
    } else if (blk < rows + a.nb_bits) {
        const int64_t t = take_ticket(a.ticket + kTicketStride);
        if (a.bytes)
            emit_sources<true, kByteWords>(a, t, n_dst);
        else
            emit_sources<false, kBitWords>(a, t, n_dst);
    }
}

// 3. local source index of every sampled edge.
// With the transpose requested, also the row of every edge and the count
// phase of the transpose: the per-column counts, and the edge's number in its
// column (in the order of the atomics), with which the place phase finds the
// edge's slot without atomics of its own (42 us of them for 719k edges).
template <class Int>
__device__ __forceinline__ void relabel_rows(const HopArgs &a, int64_t gtid, int64_t gsize, int64_t total) {
    for (int64_t q = gtid; q < total; q += gsize) {
        const Int i = static_cast<Int>(q) / static_cast<Int>(a.k);
        const int32_t t = static_cast<int32_t>(static_cast<Int>(q) - i * static_cast<Int>(a.k));
        if (t >= a.cnt[i]) continue;
        const int64_t e = a.brow[i] + t;
        const int32_t c = a.map[a.gpad[q]];
        a.bcol[e] = c;
        if (a.erow) {
            a.erow[e] = static_cast<int32_t>(i);
            if (c >= 0 && c < a.csc_cap_src)
                a.eslot[e] = atomicAdd(&a.csc_cnt[c], 1);
            else
                flag_error(&a.counts[3], kErrRange);
        }
    }
}
__device__ __forceinline__ void hop_relabel_body(const HopArgs &a, int64_t blk, int64_t nblk) {
    const int64_t total = a.counts[0] * a.k;
    const int64_t gtid = blk * kThreads + threadIdx.x, gsize = nblk * kThreads;
    // (a 64-bit division costs about as much as the rest of an edge's work)
    if (total <= UINT32_MAX)
        relabel_rows<uint32_t>(a, gtid, gsize, total);
    else
        relabel_rows<int64_t>(a, gtid, gsize, total);
}

// Jobs (see jobs.h) of the prepare and relabel steps.
// PrepareJob<-G>: G lanes per row; PrepareJob<R>: a wavefront per row.
template <int R> struct PrepareJob {
    HopArgs a;
    __device__ void run(int64_t blk, int64_t nblk) const {
        if constexpr (R < 0)
            hop_prepare_group<-R>(a, blk, nblk);
        else
            hop_prepare_wave<R>(a, blk, nblk);
    }
};
struct RelabelJob {
    HopArgs a;
    __device__ void run(int64_t blk, int64_t nblk) const { hop_relabel_body(a, blk, nblk); }
};
// (The logical index picks the role; within it workgroups order themselves by
// ticket.)
struct EmitJob {
    HopArgs a;
    __device__ void run(int64_t blk, int64_t) const { hop_emit_body(a, blk); }
};

// Launch parameters of one hop.
struct HopPlan {
    HopArgs a;
    unsigned prep_grid, emit_grid, relabel_grid;
    int r;  // PrepareJob's variant: -16, -32 (lanes per row), 1, 2, 4, 8, 16 (draws per lane)
};

// Calls f(job) with the prepare job of the plan's fanout class.
template <class F> void with_prepare_job(const HopPlan &p, F &&f) {
    switch (p.r) {
        case -16: f(PrepareJob<-16>{p.a}); break;
        case -32: f(PrepareJob<-32>{p.a}); break;
        case 1: f(PrepareJob<1>{p.a}); break;
        case 2: f(PrepareJob<2>{p.a}); break;
        case 4: f(PrepareJob<4>{p.a}); break;
        case 8: f(PrepareJob<8>{p.a}); break;
        default: f(PrepareJob<16>{p.a}); break;
    }
}

}  // namespace samp

// Host side (sampler.hip).  A hop uses the shared part of a sampler
// workspace (vertex map and marks, sampler_shared_bytes) and a per-hop
// scratch (sampler_hop_bytes); hops whose steps overlap need distinct
// scratch.
size_t sampler_shared_bytes(int64_t graph_n);
size_t sampler_hop_bytes(int64_t graph_n, int64_t cap_dst, int32_t fanout);
// csc: the transpose's arguments when the hop's block gets one (the relabel
// then runs its count phase), else null.
samp::HopPlan plan_hop(const gnn_graph *g, const float *gcn_norm, const int64_t *dst_ids, const int64_t *n_dst_dev,
                       int32_t fanout, uint64_t seed, uint64_t step, int32_t hop, const gnn_block *out, void *shared,
                       void *scratch, const csc::Args *csc);
gnn_status launch_hop_prepare(const samp::HopPlan &p, hipStream_t s);
gnn_status launch_hop_emit(const samp::HopPlan &p, hipStream_t s);
}  // namespace gnn
