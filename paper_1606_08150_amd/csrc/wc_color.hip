// Graph coloring with workload consolidation (the GC benchmark of Sec. V, an
// irregular loop like Fig. 1(b)).
//
// Jones-Plassmann coloring of a symmetric graph: a vertex takes color r in the
// round after its last outranking neighbour was colored (r - 1), color 0 if no
// neighbour outranks it (larger priority, ties to the larger id).  This is the
// round-by-round definition (every uncolored vertex that outranks all of its
// uncolored neighbours takes the round's color) computed data-driven: wait[v]
// counts the outranking neighbours still uncolored; a vertex colored in round
// r loops over its neighbours and releases the ones it outranks, and a vertex
// whose count reaches zero joins the queue of round r + 1 with color r + 1.
// Every edge is visited once by the count pass and once by a release, instead
// of once per round.
//
// A queued vertex's release loop is the nested work; one with more than
// `threshold` neighbours is consolidated per mode:
//   wave  - the wave's ballot mask is the buffer; the wave walks each buffered
//           vertex's neighbours 64 x kUnroll at a time (no barrier).
//   block - thread-ordered LDS buffer; after the barrier the block walks the
//           concatenated neighbour ranges.
//   In both, a buffered vertex with more than one chunk (64 * items_per_lane)
//   of neighbours is handed on as chunks to a global buffer that a grid-wide
//   drain walks right after the parent, one wave per chunk (the KC_X rule of
//   Sec. IV.E: a warp's or block's child gets many blocks), in the count pass
//   and in every round.
//   grid  - global buffer of (vertex, neighbour range) chunks drained by a
//           moldable grid after the kernel boundary, one wave per chunk.  The
//           thread that readies a vertex buffers its range right away, so the
//           drain of round r is also the parent of round r + 1: one kernel
//           per round, and for consecutive small rounds one workgroup in one
//           kernel (color_narrow).
//   flat  - every vertex walks all of its neighbours itself.
// Outside grid mode `threshold` applies in the count pass and the rounds
// alike; in grid mode it applies to the count pass, and every readied
// vertex's range is buffered.
#include <algorithm>
#include <climits>
#include <cstring>
#include <type_traits>

#include "wc_block.h"
#include "wc_device.h"
#include "wc_internal.h"
#include "wc_stats.h"

namespace wc {
namespace {

constexpr int kPad = 32;        // ring entries on separate 128-byte lines
constexpr int kUnroll = 4;      // neighbours in flight per lane
constexpr int kNoRelease = INT_MIN;  // rcol flag: nothing to release along this edge

struct ColorArgs {
    const int *row_ptr;
    const int *col;
    const uint32_t *prio;
    int *color;       // -1 while uncolored
    int *wait;        // outranking neighbours not yet colored
    int *rcol;        // col with bit 31 set where the row's vertex does not outrank the neighbour
    int *queue0;      // vertices colored in even rounds
    int *queue1;      // ... in odd rounds
    int *qtail;       // ring of 3 (stride kPad): size of the queue of round r
    int *chunk_tail;  // ring of 3 (stride kPad)
    int4 *chunks;     // (v, begin, end, count pass: prio[v]); grid: the chunks of even rounds
    int4 *chunks1;    // grid: the chunks of odd rounds
    long long chunk_cap;
    int *colored;     // grid: vertices colored so far
    int *state;       // grid with narrow rounds: see color_narrow
    int n;
    int threshold;
    int chunk;
    unsigned long long *host_ring;
    DevStats *stats;
    int want_stats;
};

__device__ __forceinline__ bool above(uint32_t pu, int u, uint32_t pv, int v)
{
    return pu > pv || (pu == pv && u > v);
}

// Where readied vertices go: the next round's vertex queue, or (grid mode)
// the next round's chunk buffer, with the queue taking vertices whose chunks
// do not fit (buffer full).
struct Next {
    int *queue;
    int *queue_tail;
    int4 *chunks;
    int *chunk_tail;
};

// Readied vertex w (priority pw) takes color_next and is queued.  Every active
// lane of the wave calls this together.
template <bool CHUNKED>
__device__ __forceinline__ void push_ready(const ColorArgs &a, bool ready, int w, int color_next, const Next &nx,
                                           int &readied)
{
    if (ready) {
        a.color[w] = color_next;
        ++readied;
    }
    if constexpr (!CHUNKED) {
        const int s = wave_reserve(ready, nx.queue_tail);
        if (ready) nx.queue[s] = w;
    } else {
        int beg = 0, end = 0;
        if (ready) {
            beg = a.row_ptr[w];
            end = a.row_ptr[w + 1];
        }
        const int nch = (end - beg + a.chunk - 1) / a.chunk;
        const bool one = ready && nch == 1;
        const int s = wave_reserve(one, nx.chunk_tail);
        bool defer = false;
        if (one) {
            if (s < a.chunk_cap) nx.chunks[s] = make_int4(w, beg, end, 0);
            else defer = true;
        } else if (ready && nch > 1) {
            const long long base = atomic_add_dev(nx.chunk_tail, nch);
            if (base + nch <= a.chunk_cap) {
                for (int c = 0; c < nch; ++c) {
                    const int cb = beg + c * a.chunk;
                    nx.chunks[base + c] = make_int4(w, cb, min(end, cb + a.chunk), 0);
                }
            } else {
                // reserved slots below the capacity get empty ranges (the drain
                // reads no stale chunk there)
                for (long long c = base; c < base + nch && c < a.chunk_cap; ++c) nx.chunks[c] = make_int4(w, 0, 0, 0);
                defer = true;
            }
        }
        if (defer) {
            // buffer full: the next round walks w with one lane (fallback)
            a.stats->overflowed = 1;
            nx.queue[atomic_add_dev(nx.queue_tail, 1)] = w;
        }
    }
}

// Wave and block modes: the lanes with nch > 0 hand their vertex's range on
// as chunks (v, begin, end, tag) of the global buffer, one reservation per
// wave on `tail`; the wave writes each vertex's chunks together.  Returns
// false on a lane whose chunks do not all fit (buffer full): its reserved
// entries are marked empty and the lane walks the range itself (fallback).
// Every lane of the wave calls this.
__device__ __forceinline__ bool spill_chunks(const ColorArgs &a, int *tail, int v, int beg, int end, int nch, int tag)
{
    const int slot = wave_reserve_n(nch, tail);
    const bool fits = nch > 0 && (long long)slot + nch <= a.chunk_cap;
    uint64_t m = __ballot(fits);
    while (m) {
        const int b = __builtin_ctzll(m);
        m &= m - 1;
        const int s0 = readlane(slot, b), n0 = readlane(nch, b), rb = readlane(beg, b), re = readlane(end, b);
        const int rv = readlane(v, b), rt = readlane(tag, b);
        for (int c = lane_id(); c < n0; c += kWave) {
            const int cb = rb + c * a.chunk;
            a.chunks[s0 + c] = make_int4(rv, cb, min(re, cb + a.chunk), rt);
        }
    }
    if (nch > 0 && !fits) {
        for (long long c = slot; c < (long long)slot + nch && c < a.chunk_cap; ++c) a.chunks[c] = make_int4(v, 0, 0, 0);
        a.stats->overflowed = 1;
    }
    return nch == 0 || fits;
}

// A vertex colored in round r releases the neighbours e = first + k * stride
// < end of its row that it outranks (the count pass flagged the others in
// rcol); a neighbour whose count reaches zero is readied with color r + 1.
// Every active lane of the wave calls this together (the appends are
// wave-aggregated); first, stride and end may differ per lane.  Returns the
// number of releases.
template <bool CHUNKED>
__device__ __forceinline__ int release_range(const ColorArgs &a, int first, int stride, int end, int color_next,
                                             const Next &nx, int &readied)
{
    int rel = 0;
    for (int e0 = first; e0 < end; e0 += kUnroll * stride) {
        int w[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            const int e = e0 + k * stride;
            w[k] = e < end ? a.rcol[e] : kNoRelease;
        }
        int old[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            old[k] = w[k] >= 0 ? atomic_add_dev(&a.wait[w[k]], -1) : 0;
            rel += w[k] >= 0 ? 1 : 0;
        }
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) push_ready<CHUNKED>(a, old[k] == 1, w[k], color_next, nx, readied);
    }
    return rel;
}

// The consolidated child of a block (G = BLOCK) over its buffer of nb
// vertices: vertex i releases along rcol[beg_i, beg_i + deg_i),
// pre_i being the exclusive prefix of the degrees (total in all).  The group
// walks the concatenated ranges, G * kUnroll edges per step, thread t taking
// flattened edges t, t + G, ...; a cursor that only moves forward finds each
// edge's vertex.  Returns the number of releases.
template <int G>
__device__ __forceinline__ int release_items(const ColorArgs &a, const int *ibeg, const int *ipre, int nb, int total,
                                             int t, int color_next, const Next &nx, int &readied)
{
    int rel = 0, it = 0;
    for (int j0 = t; j0 < total; j0 += G * kUnroll) {
        int w[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            const int j = j0 + k * G;
            w[k] = kNoRelease;
            if (j < total) {
                while (it + 1 < nb && ipre[it + 1] <= j) ++it;
                w[k] = a.rcol[ibeg[it] + (j - ipre[it])];
            }
        }
        int old[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            old[k] = w[k] >= 0 ? atomic_add_dev(&a.wait[w[k]], -1) : 0;
            rel += w[k] >= 0 ? 1 : 0;
        }
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) push_ready<false>(a, old[k] == 1, w[k], color_next, nx, readied);
    }
    return rel;
}

template <int BLOCK>
struct ColorLds {
    int beg[BLOCK];
    int pre[BLOCK + 1];
    int scan_tmp[2 * (BLOCK / kWave)];
    int base;
};

// Round r outside grid mode: thread i takes the i-th vertex of the round's
// queue (colored r).
template <int MODE, int BLOCK>
__global__ __launch_bounds__(BLOCK) void color_round(ColorArgs a, int r)
{
    __shared__ ColorLds<BLOCK> sb;
    const int size = a.qtail[(r % 3) * kPad];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.qtail[((r + 2) % 3) * kPad] = 0;
        a.chunk_tail[((r + 2) % 3) * kPad] = 0;
        publish_host(a.host_ring, r % kHostRing, a.stats, size);
    }
    if (size == 0) return;
    const int *q = (r & 1) ? a.queue1 : a.queue0;
    const Next nx{(r & 1) ? a.queue0 : a.queue1, &a.qtail[((r + 1) % 3) * kPad], nullptr, nullptr};
    const int lane = lane_id();
    int readied = 0;
    StatAcc acc;
    for (int base = blockIdx.x * BLOCK; base < size; base += gridDim.x * BLOCK) {
        const int i = base + threadIdx.x;
        const bool member = i < size;
        int beg = 0, end = 0;
        if (member) {
            const int v = q[i];
            beg = a.row_ptr[v];
            end = a.row_ptr[v + 1];
        }
        const int deg = end - beg;
        const bool heavy = MODE != WC_FLAT && deg > a.threshold;
        if (a.want_stats) {
            acc.edges += deg;
            acc.buffered += heavy ? deg : 0;
            acc.items += heavy ? 1 : 0;
            if (MODE == WC_WAVE && __ballot(heavy) && lane == 0) acc.dispatches += 1;
        }
        // buffered vertices with more than one chunk go to the round's drain
        bool spill = heavy && deg > a.chunk, inline_walk = member && !heavy;
        if (__ballot(spill)) {
            const int v = spill ? q[i] : 0;
            if (!spill_chunks(a, &a.chunk_tail[(r % 3) * kPad], v, beg, end, spill ? (deg + a.chunk - 1) / a.chunk : 0,
                              0))
                inline_walk = true;
        }
        const bool mine = heavy && !spill;
        if (inline_walk) acc.updates += release_range<false>(a, beg, 1, end, r + 1, nx, readied);
        if constexpr (MODE == WC_WAVE) {
            // the ballot mask is the wave's buffer; the wave walks each buffered
            // vertex's range 64 x kUnroll neighbours at a time (walking the
            // concatenated ranges measured 12% slower here)
            uint64_t mask = __ballot(mine);
            while (mask) {
                const int b = __builtin_ctzll(mask);
                mask &= mask - 1;
                acc.updates_buffered +=
                    release_range<false>(a, readlane(beg, b) + lane, kWave, readlane(end, b), r + 1, nx, readied);
            }
        } else if constexpr (MODE == WC_BLOCK) {
            int k, off, nb, total;
            block_scan2<BLOCK>(mine ? 1 : 0, mine ? deg : 0, sb.scan_tmp, k, off, nb, total);
            if (mine) {
                sb.beg[k] = beg;
                sb.pre[k] = off;
            }
            if (a.want_stats && __syncthreads_or(heavy ? 1 : 0) && threadIdx.x == 0) acc.dispatches += 1;
            if (threadIdx.x == 0) sb.pre[nb] = total;
            __syncthreads();
            acc.updates_buffered += release_items<BLOCK>(a, sb.beg, sb.pre, nb, total, threadIdx.x, r + 1, nx, readied);
            __syncthreads();  // the LDS buffer is reused by the next window
        }
    }
    if (a.want_stats) stat_flush(a.stats, acc);
}

// Wave and block modes: the chunks that round r's parent handed on, one wave
// per chunk, right after the parent; readied vertices join round r + 1's queue.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void color_round_drain(ColorArgs a, int r)
{
    const int tail = a.chunk_tail[(r % 3) * kPad];
    const int total = (long long)tail < a.chunk_cap ? tail : (int)a.chunk_cap;
    if (total == 0) return;
    const Next nx{(r & 1) ? a.queue0 : a.queue1, &a.qtail[((r + 1) % 3) * kPad], nullptr, nullptr};
    const int gw = (blockIdx.x * BLOCK + threadIdx.x) / kWave;
    const int nw = gridDim.x * (BLOCK / kWave);
    int readied = 0;
    StatAcc acc;
    for (int c = gw; c < total; c += nw) {
        const int4 d = a.chunks[c];
        const int beg = __builtin_amdgcn_readfirstlane(d.y), end = __builtin_amdgcn_readfirstlane(d.z);
        acc.updates_buffered += release_range<false>(a, beg + lane_id(), kWave, end, r + 1, nx, readied);
    }
    if (a.want_stats) stat_flush(a.stats, acc);
}

// Where color_narrow left off (ColorArgs::state).
enum { kRound = 0, kWide = 1, kDone = 2, kStateInts = 3 };

// Round r in grid mode: one wave per buffered chunk (a readied vertex's
// neighbour range, buffered while round r - 1 ran), then one lane per vertex
// the buffer could not take.  Vertices readied here buffer their ranges for
// round r + 1.  Publishes whether it had work.  PHASED (in turn with color_narrow):
// r < 0 is the round that color_narrow found too large for itself, if it did, and
// host-ring entry `slot`, unless that is negative, gets the number of chunks.
template <int BLOCK, bool PHASED>
__global__ __launch_bounds__(BLOCK) void color_round_grid(ColorArgs a, int r, int slot)
{
    if (PHASED && r < 0) {
        if (!a.state[kWide]) return;
        r = a.state[kRound];
    }
    const int nchunks = a.chunk_tail[(r % 3) * kPad];
    const int ndefer = a.qtail[(r % 3) * kPad];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.chunk_tail[((r + 2) % 3) * kPad] = 0;
        a.qtail[((r + 2) % 3) * kPad] = 0;
        if (!PHASED) publish_host(a.host_ring, r % kHostRing, a.stats, (nchunks != 0 || ndefer != 0) ? 1 : 0);
        else if (slot >= 0) publish_host(a.host_ring, slot % kHostRing, a.stats, ndefer != 0 ? INT_MAX : nchunks);
    }
    if (nchunks == 0 && ndefer == 0) return;
    const int total = (long long)nchunks < a.chunk_cap ? nchunks : (int)a.chunk_cap;
    const int4 *cur = (r & 1) ? a.chunks1 : a.chunks;
    const Next nx{(r & 1) ? a.queue0 : a.queue1, &a.qtail[((r + 1) % 3) * kPad], (r & 1) ? a.chunks : a.chunks1,
                  &a.chunk_tail[((r + 1) % 3) * kPad]};
    const int gw = (blockIdx.x * BLOCK + threadIdx.x) / kWave;
    const int nw = gridDim.x * (BLOCK / kWave);
    int readied = 0;
    StatAcc acc;
    if (a.want_stats && blockIdx.x == 0 && threadIdx.x == 0 && total > 0) acc.dispatches = 1;
    for (int c = gw; c < total; c += nw) {
        const int4 d = cur[c];
        const int beg = __builtin_amdgcn_readfirstlane(d.y), end = __builtin_amdgcn_readfirstlane(d.z);
        if (a.want_stats && lane_id() == 0) {
            acc.items += 1;
            acc.buffered += end - beg;
            acc.edges += end - beg;
        }
        acc.updates_buffered += release_range<true>(a, beg + lane_id(), kWave, end, r + 1, nx, readied);
    }
    const int *dq = (r & 1) ? a.queue1 : a.queue0;
    for (int i = blockIdx.x * BLOCK + threadIdx.x; i < ndefer; i += gridDim.x * BLOCK) {
        const int v = dq[i];
        const int beg = a.row_ptr[v], end = a.row_ptr[v + 1];
        if (a.want_stats) acc.edges += end - beg;
        acc.updates += release_range<true>(a, beg, 1, end, r + 1, nx, readied);
    }
    readied = wave_sum_i(readied);
    if (lane_id() == 0 && readied) (void)atomic_add_dev(a.colored, readied);
    if (a.want_stats) stat_flush(a.stats, acc);
}

// Consecutive small rounds of grid mode in one launch, by one workgroup: the
// grid-wide barrier between rounds is its own barrier.  Most rounds color a few
// dozen vertices and release some thousand edges (scale-16 graph, 775 rounds: 50
// vertices, 4,200 entries in 74 chunks at the median), less than a launch's
// worth.  The round's chunks are listed in LDS; a wave takes one, two or four of
// them at a time, and sixteen lanes list the chunks of a vertex readied here (four
// where there are many).
// The counts are kept in LDS too, 16 bits each, for the launch.  Bound by the
// round's two round trips to memory (entries, the readied vertices' ranges) and,
// beyond some thousand entries, by what one CU's LDS and issue slots take.
// Scale-16 graph, 65,536 vertices and 3.4M entries: 3.9 us a round against 6.5 of
// a launch, 5,200 -> 3,150 us in all; 1,024 and 4,096 vertices 508 and 1,043 ->
// 180 and 364 us.  Entries side by side over the threads, each finding its range
// by a search over prefixes: 5.7 us a round; the counts in memory: 6.9.
// Rule: graphs of up to kNarrowN vertices, whose counts LDS holds, and rounds of
// up to kNarrowChunks chunks (at 128, 3,400 instead of 2,420 us on 65,536
// vertices of 16 edges; at 512 the same), a launch's first of up to kNarrowEnter
// (128, 160, 192 and 256: 542, 528, 564 and 620 us on 16,384 vertices of 32 random
// neighbours, 3,605, 3,561, 3,584 and 3,575 on 65,536 of 52) and kNarrowEntries
// entries.  A launch ends before a round that it finds larger, and after one that
// readies more vertices than kNarrowChunks.
// The workgroup starts from, and where a round is larger than it takes leaves,
// the chunk buffer of the round; color_round_grid does that round (state[kWide]),
// and the next launch goes on after it.  `from` >= 0: the round to start with,
// where the rounds before were all the grid's.  A launch ends after kNarrowRounds
// rounds at the latest.  Each launch publishes the number of colored vertices when
// all is done, kNarrowOn when not, kNarrowIdle - r when it did no round itself but
// left round r, and kNarrowBad when a count would go below zero: the graph is not
// symmetric, packed counts would spill over into their neighbours, and the call is
// done again without this kernel.
constexpr int kNarrowBlock = 1024;
constexpr int kNarrowGroup = 16;     // lanes that list one vertex's chunks
constexpr int kFewLanes = 4;         // ... in a round of more than 64 vertices
constexpr int kNarrowList = 1024;    // chunks that a list holds
constexpr int kNarrowChunks = 256;   // chunks of a round that is taken here
constexpr int kNarrowEnter = 160;    // chunks and
constexpr int kNarrowEntries = 8192; // entries of a launch's first round
constexpr int kNarrowChunk = 2 * kWave;  // largest chunk
constexpr int kNarrowRounds = 4096;
constexpr int kNarrowN = 65536;
enum { kNarrowOn = -1, kNarrowBad = -2, kNarrowIdle = -16 };
// The entries of a round's chunks, U chunks a wave at a time: releases, and the
// vertices that they ready into s_ready (beyond it: a.queue0).  Each step for all
// entries before the next: a round trip a step, not one an entry.  True on a
// thread that found a count at zero.
template <int U>
__device__ __forceinline__ bool narrow_entries(const ColorArgs &a, const int2 *list, int count, int wid,
                                               unsigned int *s_wait, int *s_found, int *s_ready)
{
    constexpr int NW = kNarrowBlock / kWave;
    const int lane = lane_id();
    bool bad = false;
    for (int i0 = wid; i0 < count; i0 += NW * U) {
        int w[2 * U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * NW;
            const int2 d = i < count ? list[i] : make_int2(0, 0);
            const int e = d.x + lane;
            w[2 * u] = e < d.y ? a.rcol[e] : kNoRelease;
            w[2 * u + 1] = e + kWave < d.y ? a.rcol[e + kWave] : kNoRelease;
        }
        unsigned int old[2 * U];
#pragma unroll
        for (int u = 0; u < 2 * U; ++u)
            old[u] = w[u] >= 0 ? atomicSub(&s_wait[w[u] >> 1], 1u << 16 * (w[u] & 1)) : 0x20002u;
        int ready = 0;  // of this thread: one reservation
#pragma unroll
        for (int u = 0; u < 2 * U; ++u) {
            old[u] = old[u] >> 16 * (w[u] & 1) & 0xffffu;
            bad |= old[u] == 0;
            ready += old[u] == 1 ? 1 : 0;
        }
        if (ready) {
            int q = atomicAdd(s_found, ready);
#pragma unroll
            for (int u = 0; u < 2 * U; ++u)
                if (old[u] == 1) {
                    if (q < kNarrowBlock) s_ready[q] = w[u];
                    else if (q - kNarrowBlock < a.n) a.queue0[q - kNarrowBlock] = w[u];
                    ++q;
                }
        }
    }
    return bad;
}

// Chunks of the threads' rows side by side at `out`; their number.  The whole
// workgroup calls.
__device__ __forceinline__ int list_rows(const ColorArgs &a, int4 *out, int beg, int end, int *s_tmp)
{
    const int nch = (end - beg + a.chunk - 1) / a.chunk;
    int at, unused, tot, unused2;
    block_scan2<kNarrowBlock>(nch, 0, s_tmp, at, unused, tot, unused2);
    for (int c = 0; c < nch; ++c) {
        const int cb = beg + c * a.chunk;
        out[at + c] = make_int4(0, cb, min(end, cb + a.chunk), 0);
    }
    return tot;
}

__global__ __launch_bounds__(kNarrowBlock) void color_narrow(ColorArgs a, int slot, int from)
{
    constexpr int NW = kNarrowBlock / kWave;
    __shared__ int2 s_list[2][kNarrowList];
    __shared__ int s_ready[kNarrowBlock];
    __shared__ int s_next[2], s_entries, s_found[2];  // chunks of a list, entries of the first, vertices readied
    __shared__ int s_tmp[2 * NW], s_readied, s_spill, s_listed, s_bad;
    __shared__ unsigned int s_wait[kNarrowN / 2];
    const int tid = threadIdx.x, lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(tid / kWave);
    if (a.state[kDone]) {
        if (tid == 0) publish_host(a.host_ring, slot % kHostRing, a.stats, *a.colored);
        return;
    }
    int r = from >= 0 ? from : a.state[kRound] + a.state[kWide];  // the wide round, if there was one, is done
    const int nchunks = a.chunk_tail[(r % 3) * kPad], ndefer = a.qtail[(r % 3) * kPad];
    bool fits = ndefer == 0 && nchunks <= kNarrowEnter;
    int k = 0;  // rounds done here; the list of the current one is k & 1
    if (tid == 0) {
        s_next[0] = fits ? nchunks : 0;
        s_entries = 0;
        s_found[0] = s_readied = s_spill = s_bad = 0;
        s_listed = kNarrowList;
    }
    __syncthreads();
    if (fits && tid < nchunks) {
        const int4 d = ((r & 1) ? a.chunks1 : a.chunks)[tid];
        s_list[0][tid] = make_int2(d.y, d.z);
        atomicAdd(&s_entries, d.z - d.y);
    }
    __syncthreads();
    fits = fits && s_entries <= kNarrowEntries;
    if (fits && nchunks > 0) {
        bool large = false;
        for (int i = tid; 2 * i < a.n; i += kNarrowBlock) {
            const unsigned int lo = (unsigned int)a.wait[2 * i];
            const unsigned int hi = 2 * i + 1 < a.n ? (unsigned int)a.wait[2 * i + 1] : 0u;
            large |= (lo | hi) > 0xffffu;
            s_wait[i] = lo | hi << 16;
        }
        if (__syncthreads_or(large ? 1 : 0)) fits = false;  // multi-edges: more than 16 bits count
    }
    __syncthreads();
    int readied = 0, many = 0;  // many: vertices readied in the last round, where they are not listed
    bool below_zero = false;
    for (; fits && k < kNarrowRounds; ++k, ++r) {
        const int count = s_next[k & 1];
        if (count == 0 || count > kNarrowChunks) break;
        // the entries: releases, and the vertices that they ready
        if (tid == 0) s_next[(k + 1) & 1] = 0;
        bool bad = false;
        // more chunks a wave at once only where it has them: unused places cost issue slots
        if (count <= NW) bad |= narrow_entries<1>(a, s_list[k & 1], count, wid, s_wait, &s_found[k & 1], s_ready);
        else if (count <= 2 * NW) bad |= narrow_entries<2>(a, s_list[k & 1], count, wid, s_wait, &s_found[k & 1], s_ready);
        else bad |= narrow_entries<4>(a, s_list[k & 1], count, wid, s_wait, &s_found[k & 1], s_ready);
        if (bad) s_bad = 1;
        __syncthreads();
        // the vertices: their color, and their chunks into the next list
        const int found = s_found[k & 1];
        const bool stop = s_bad;  // set before the round's first barrier, read before its second
        if (tid == 0) s_found[(k + 1) & 1] = 0;
        if (found > kNarrowChunks && !stop) {
            many = found;
            ++k, ++r;
            break;
        }
        int2 *next = s_list[(k + 1) & 1];
        auto list_found = [&](auto group) {
            constexpr int G = decltype(group)::value;  // lanes a vertex
            const int sub = lane & (G - 1);
            for (int i = tid / G; i < found; i += kNarrowBlock / G) {
                const int v = i < kNarrowBlock ? s_ready[i] : a.queue0[min(i - kNarrowBlock, a.n - 1)];
                const int beg = a.row_ptr[v], end = a.row_ptr[v + 1];
                const int nch = (end - beg + kNarrowChunk - 1) / kNarrowChunk;
                int at = 0;
                if (sub == 0) {
                    a.color[v] = r + 1;
                    ++readied;
                    at = atomicAdd(&s_next[(k + 1) & 1], nch);
                }
                at = __shfl(at, lane & ~(G - 1), kWave);
                if (at + nch <= kNarrowList) {
                    for (int c = sub; c < nch; c += G) {
                        const int b = beg + c * kNarrowChunk;
                        next[at + c] = make_int2(b, min(end, b + kNarrowChunk));
                    }
                } else if (sub == 0) {
                    // more than the list holds (the round is too large anyway): the vertex
                    // to memory; the list ends where the first such vertex would begin
                    atomicMin(&s_listed, at);
                    const int q = atomicAdd(&s_spill, 1);
                    if (q < a.n) a.queue1[q] = v;
                }
            }
        };
        if (found <= kNarrowBlock / kNarrowGroup) list_found(std::integral_constant<int, kNarrowGroup>{});
        else list_found(std::integral_constant<int, kFewLanes>{});
        __syncthreads();
        if (stop) {
            below_zero = true;
            break;
        }
    }
    readied = wave_sum_i(readied);
    if (lane == 0 && readied) atomicAdd(&s_readied, readied);
    if (tid == 0) atomicAdd(&s_readied, many);
    if (below_zero) {
        // the launches behind this one find nothing to do
        if (tid == 0) {
            *a.colored = kNarrowBad;
            a.state[kWide] = 0;
            a.state[kDone] = 1;
            publish_host(a.host_ring, slot % kHostRing, a.stats, kNarrowBad);
        }
        return;
    }
    const int count = s_next[k & 1];
    const bool done = fits && many == 0 && count == 0;
    int chunks = 0;
    if (k > 0 && !done) {
        for (int i = tid; 2 * i < a.n; i += kNarrowBlock) {
            const unsigned int q = s_wait[i];
            a.wait[2 * i] = (int)(q & 0xffffu);
            if (2 * i + 1 < a.n) a.wait[2 * i + 1] = (int)(q >> 16);
        }
        int4 *out = (r & 1) ? a.chunks1 : a.chunks;
        if (many == 0) {
            // the list becomes the chunk buffer of its round: the chunks of each of its
            // vertices once, which the buffer holds
            chunks = min(count, s_listed);
            if (tid < chunks) out[tid] = make_int4(0, s_list[k & 1][tid].x, s_list[k & 1][tid].y, 0);
            const int spilled = min(s_spill, a.n);
            for (int i0 = 0; i0 < spilled; i0 += kNarrowBlock) {
                int beg = 0, end = 0;
                if (i0 + tid < spilled) {
                    const int v = a.queue1[i0 + tid];
                    beg = a.row_ptr[v];
                    end = a.row_ptr[v + 1];
                }
                chunks += list_rows(a, out + chunks, beg, end, s_tmp);
            }
        }
        // more vertices than their round may have chunks: a thread each, and straight
        // into the round's buffer (16,000 readied by a hub: 250 us by the list)
        for (int i0 = 0; i0 < many; i0 += kNarrowBlock) {
            const int i = i0 + tid;
            int beg = 0, end = 0;
            if (i < many) {
                const int v = i < kNarrowBlock ? s_ready[i] : a.queue0[min(i - kNarrowBlock, a.n - 1)];
                beg = a.row_ptr[v];
                end = a.row_ptr[v + 1];
                a.color[v] = r;
            }
            chunks += list_rows(a, out + chunks, beg, end, s_tmp);
        }
    }
    __syncthreads();
    if (tid != 0) return;
    if (k > 0 && !done) {
        a.chunk_tail[(r % 3) * kPad] = chunks;
        a.chunk_tail[((r + 1) % 3) * kPad] = 0;
        a.qtail[(r % 3) * kPad] = 0;
        a.qtail[((r + 1) % 3) * kPad] = 0;
    }
    const int colored = *a.colored + s_readied;
    *a.colored = colored;
    a.state[kRound] = r;
    a.state[kWide] = !done && !(fits && k == kNarrowRounds);
    a.state[kDone] = done;
    publish_host(a.host_ring, slot % kHostRing, a.stats, done ? colored : k > 0 ? kNarrowOn : kNarrowIdle - r);
}

// Clears the rings before the count pass appends to the first queue.
__global__ void color_reset(ColorArgs a)
{
    if (threadIdx.x < 3) {
        a.qtail[threadIdx.x * kPad] = 0;
        a.chunk_tail[threadIdx.x * kPad] = 0;
    }
    if (threadIdx.x == 0) *a.colored = 0;
    if (threadIdx.x < kStateInts) a.state[threadIdx.x] = 0;
}

// Grid mode: hands the number of colored vertices to the host.
__global__ void color_publish(ColorArgs a)
{
    if (threadIdx.x == 0) publish_host(a.host_ring, kHostSlotGraph, a.stats, *a.colored);
}

// Edge e of v's row toward u: does u outrank v?  Flags the edge in rcol when
// v has nothing to release along it (u outranks v, or a self-loop).
__device__ __forceinline__ bool count_edge(const ColorArgs &a, int v, uint32_t pv, int u, int e)
{
    const bool o = u != v && above(a.prio[u], u, pv, v);
    a.rcol[e] = (o || u == v) ? (u | kNoRelease) : u;
    return o;
}

// Neighbours e = first + k * stride < end of v (priority pv) that outrank v.
__device__ __forceinline__ int count_range(const ColorArgs &a, int v, uint32_t pv, int first, int stride, int end)
{
    int cnt = 0;
    for (int e0 = first; e0 < end; e0 += kUnroll * stride) {
        int u[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            const int e = e0 + k * stride;
            u[k] = e < end ? a.col[e] : v;
        }
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            const int e = e0 + k * stride;
            if (e < end) cnt += count_edge(a, v, pv, u[k], e) ? 1 : 0;
        }
    }
    return cnt;
}

template <int BLOCK>
struct CountLds {
    int v[BLOCK];
    int beg[BLOCK];
    uint32_t p[BLOCK];
    int pre[BLOCK + 1];
    int cnt[BLOCK];
    int scan_tmp[2 * (BLOCK / kWave)];
    int base;
};

// Count pass, the first irregular loop: wait[v] = neighbours that outrank v.
// A row with more than `threshold` entries is consolidated per mode (grid,
// and wave and block rows longer than one chunk: its chunks are counted by
// color_count_drain, which adds to wait[v] = 0).
template <int MODE, int BLOCK>
__global__ __launch_bounds__(BLOCK) void color_count(ColorArgs a)
{
    __shared__ CountLds<BLOCK> sb;
    const int lane = lane_id();
    for (int base = blockIdx.x * BLOCK; base < a.n; base += gridDim.x * BLOCK) {
        const int v = base + threadIdx.x;
        const bool member = v < a.n;
        int beg = 0, end = 0;
        uint32_t pv = 0;
        if (member) {
            beg = a.row_ptr[v];
            end = a.row_ptr[v + 1];
            pv = a.prio[v];
        }
        const int deg = end - beg;
        const bool heavy = MODE != WC_FLAT && deg > a.threshold;
        // wave and block modes: rows with more than one chunk go to the drain
        const bool spill = (MODE == WC_WAVE || MODE == WC_BLOCK) && heavy && deg > a.chunk;
        bool inline_count = member && !heavy;
        if constexpr (MODE == WC_WAVE || MODE == WC_BLOCK) {
            if (__ballot(spill) &&
                !spill_chunks(a, &a.chunk_tail[2 * kPad], v, beg, end, spill ? (deg + a.chunk - 1) / a.chunk : 0,
                              (int)pv))
                inline_count = true;
        }
        const bool mine = heavy && !spill;
        int cnt = 0;
        if (inline_count) cnt = count_range(a, v, pv, beg, 1, end);
        if constexpr (MODE == WC_WAVE) {
            uint64_t mask = __ballot(mine);
            while (mask) {
                const int b = __builtin_ctzll(mask);
                mask &= mask - 1;
                const int c = wave_sum_i(count_range(a, readlane(v, b), readlane_u(pv, b), readlane(beg, b) + lane,
                                                     kWave, readlane(end, b)));
                if (lane == b) cnt = c;
            }
        } else if constexpr (MODE == WC_BLOCK) {
            int k, off, nb, total;
            block_scan2<BLOCK>(mine ? 1 : 0, mine ? deg : 0, sb.scan_tmp, k, off, nb, total);
            if (mine) {
                sb.v[k] = v;
                sb.beg[k] = beg;
                sb.p[k] = pv;
                sb.pre[k] = off;
                sb.cnt[k] = 0;
            }
            if (threadIdx.x == 0) sb.pre[nb] = total;
            __syncthreads();
            int it = 0;
            for (int j = threadIdx.x; j < total; j += BLOCK) {
                while (it + 1 < nb && sb.pre[it + 1] <= j) ++it;
                const int e = sb.beg[it] + (j - sb.pre[it]);
                if (count_edge(a, sb.v[it], sb.p[it], a.col[e], e)) atomicAdd(&sb.cnt[it], 1);
            }
            __syncthreads();
            if (mine) cnt = sb.cnt[k];
            __syncthreads();  // the LDS buffer is reused by the next window
        } else if constexpr (MODE == WC_GRID) {
            if (__syncthreads_or(heavy ? 1 : 0)) {
                const int nch = heavy ? (deg + a.chunk - 1) / a.chunk : 0;
                int excl, unused, tot, unused2;
                block_scan2<BLOCK>(nch, 0, sb.scan_tmp, excl, unused, tot, unused2);
                if (threadIdx.x == 0) sb.base = tot ? atomic_add_dev(&a.chunk_tail[2 * kPad], tot) : 0;
                __syncthreads();
                const long long slot = (long long)sb.base + excl;
                const bool fits = slot + nch <= a.chunk_cap;
                if (heavy) {
                    if (fits) {
                        for (int c = 0; c < nch; ++c) {
                            const int cb = beg + c * a.chunk;
                            a.chunks[slot + c] = make_int4(v, cb, min(end, cb + a.chunk), (int)pv);
                        }
                    } else {
                        a.stats->overflowed = 1;
                        for (long long c = slot; c < slot + nch && c < a.chunk_cap; ++c)
                            a.chunks[c] = make_int4(v, 0, 0, 0);
                        cnt = count_range(a, v, pv, beg, 1, end);  // fallback: counted inline
                    }
                }
                __syncthreads();  // sb.base is rewritten by the next window
            }
        }
        if (member) a.wait[v] = cnt;
    }
}

// One wave per chunk of a buffered row (grid mode; wave and block modes: rows
// longer than one chunk) adds its count to wait[v].
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void color_count_drain(ColorArgs a)
{
    const int tail = a.chunk_tail[2 * kPad];
    const int total = (long long)tail < a.chunk_cap ? tail : (int)a.chunk_cap;
    const int gw = (blockIdx.x * BLOCK + threadIdx.x) / kWave;
    const int nw = gridDim.x * (BLOCK / kWave);
    for (int c = gw; c < total; c += nw) {
        const int4 d = a.chunks[c];
        const int v = __builtin_amdgcn_readfirstlane(d.x);
        const int cnt = wave_sum_i(count_range(a, v, (uint32_t)__builtin_amdgcn_readfirstlane(d.w),
                                               __builtin_amdgcn_readfirstlane(d.y) + lane_id(), kWave,
                                               __builtin_amdgcn_readfirstlane(d.z)));
        if (lane_id() == 0 && cnt) (void)atomic_add_dev(&a.wait[v], cnt);
    }
}

// Vertices that no neighbour outranks take color 0 and form round 0 (grid:
// their neighbour ranges are buffered as chunks); the others start
// uncolored.  One reservation per block step.
constexpr int kSeedBlock = 256;
template <bool CHUNKED>
__global__ __launch_bounds__(kSeedBlock) void color_seed(ColorArgs a)
{
    __shared__ int scan_tmp[2 * (kSeedBlock / kWave)];
    __shared__ int s_base;
    for (int base = blockIdx.x * kSeedBlock; base < a.n; base += gridDim.x * kSeedBlock) {
        const int v = base + threadIdx.x;
        const bool member = v < a.n;
        const bool first = member && a.wait[v] == 0;
        if (member) a.color[v] = first ? 0 : -1;
        if constexpr (!CHUNKED) {
            int k, unused, tot, unused2;
            block_scan2<kSeedBlock>(first ? 1 : 0, 0, scan_tmp, k, unused, tot, unused2);
            if (threadIdx.x == 0 && tot) s_base = atomic_add_dev(&a.qtail[0], tot);
            __syncthreads();
            if (first) a.queue0[s_base + k] = v;
        } else {
            int beg = 0, end = 0;
            if (first) {
                beg = a.row_ptr[v];
                end = a.row_ptr[v + 1];
            }
            const int nch = (end - beg + a.chunk - 1) / a.chunk;
            int k, unused, tot, nfirst;
            block_scan2<kSeedBlock>(nch, first ? 1 : 0, scan_tmp, k, unused, tot, nfirst);
            if (threadIdx.x == 0) {
                if (tot) s_base = atomic_add_dev(&a.chunk_tail[0], tot);
                if (nfirst) (void)atomic_add_dev(a.colored, nfirst);
            }
            __syncthreads();
            if (nch) {
                const long long slot = (long long)s_base + k;
                if (slot + nch <= a.chunk_cap) {
                    for (int c = 0; c < nch; ++c) {
                        const int cb = beg + c * a.chunk;
                        a.chunks[slot + c] = make_int4(v, cb, min(end, cb + a.chunk), (int)a.prio[v]);
                    }
                } else {
                    a.stats->overflowed = 1;
                    for (long long c = slot; c < slot + nch && c < a.chunk_cap; ++c)
                        a.chunks[c] = make_int4(v, 0, 0, 0);
                    a.queue0[atomic_add_dev(&a.qtail[0], 1)] = v;
                }
            }
        }
        __syncthreads();  // s_base is rewritten by the next step
    }
}

struct ColorKernels {
    const void *round, *count, *count_drain, *round_drain;
};

template <int BLOCK>
ColorKernels pick_block(wc_mode mode)
{
    ColorKernels k{nullptr, nullptr, reinterpret_cast<const void *>(&color_count_drain<BLOCK>),
                   reinterpret_cast<const void *>(&color_round_drain<BLOCK>)};
    switch (mode) {
    case WC_FLAT:
        k.round = reinterpret_cast<const void *>(&color_round<WC_FLAT, BLOCK>);
        k.count = reinterpret_cast<const void *>(&color_count<WC_FLAT, BLOCK>);
        break;
    case WC_WAVE:
        k.round = reinterpret_cast<const void *>(&color_round<WC_WAVE, BLOCK>);
        k.count = reinterpret_cast<const void *>(&color_count<WC_WAVE, BLOCK>);
        break;
    case WC_BLOCK:
        k.round = reinterpret_cast<const void *>(&color_round<WC_BLOCK, BLOCK>);
        k.count = reinterpret_cast<const void *>(&color_count<WC_BLOCK, BLOCK>);
        break;
    default:
        k.round = reinterpret_cast<const void *>(&color_round_grid<BLOCK, false>);
        k.count = reinterpret_cast<const void *>(&color_count<WC_GRID, BLOCK>);
        break;
    }
    return k;
}

ColorKernels pick(wc_mode mode, int block)
{
    switch (block) {
    case 64: return pick_block<64>(mode);
    case 128: return pick_block<128>(mode);
    case 512: return pick_block<512>(mode);
    case 1024: return pick_block<1024>(mode);
    default: return pick_block<256>(mode);
    }
}

}  // namespace
}  // namespace wc

using namespace wc;

extern "C" wc_status wc_color(wc_ctx *ctx, const wc_csr *g, const uint32_t *prio, int32_t *color, wc_mode mode,
                              const wc_tune *tune, hipStream_t stream, wc_stats *stats)
{
    if (!ctx || !g) return fail(WC_EINVAL, "wc_color: NULL context or graph");
    if (mode < WC_FLAT || mode > WC_GRID) return fail(WC_EINVAL, "wc_color: bad mode");
    if (g->n < 0 || g->m < 0) return fail(WC_EINVAL, "wc_color: negative size");
    if (g->n == 0) {
        if (stats) std::memset(stats, 0, sizeof(*stats));
        return WC_OK;
    }
    if (!g->row_ptr || !prio || !color || (g->m > 0 && !g->col)) return fail(WC_EINVAL, "wc_color: NULL array");
    WC_HIP(hipSetDevice(ctx->device));
    int block = (tune && tune->block_threads > 0) ? tune->block_threads : 256;
    ColorKernels ks = pick(mode, block);
    int resident = resident_blocks(ctx, ks.round, block);
    Config cfg;
    wc_status st = resolve_tune(ctx, "color", mode, tune, resident, &cfg);
    if (st != WC_OK) return st;
    if (cfg.driver != 0) return fail(WC_EINVAL, "wc_color: only the relaunch driver (driver = 0) exists");
    if (cfg.block != block) {
        ks = pick(mode, cfg.block);
        resident = resident_blocks(ctx, ks.round, cfg.block);
    }
    const long long n = g->n, m = g->m;
    const int chunk = kWave * cfg.items_per_lane;
    const bool grid_mode = mode == WC_GRID;
    // grid mode: every vertex has ceil(deg / chunk) <= deg / chunk + 1 chunks
    // in the one round that colors it (and in the count pass), so n + m / chunk
    // + 1 entries per buffer never overflow.  Wave and block modes buffer only
    // vertices with more than one chunk of neighbours (ceil(deg / chunk) <
    // 2 deg / chunk each), in the count pass or one round at a time.
    const bool spills = mode == WC_WAVE || mode == WC_BLOCK;
    const long long cap_full = grid_mode ? n + m / chunk + 1 : spills ? 2 * (m / chunk) + 1 : 1;
    const long long cap = cfg.buf_capacity > 0 && mode != WC_FLAT ? std::min(cfg.buf_capacity, cap_full) : cap_full;
    const size_t need = 3 * padded(n * 4) + padded(m * 4) + 4 * padded(3 * kPad * 4) +
                        (grid_mode ? 2 : 1) * padded(cap * 16);
    st = pool_reserve(ctx, need, stream);
    if (st != WC_OK) return st;
    ColorArgs a;
    std::memset(&a, 0, sizeof(a));
    a.row_ptr = g->row_ptr;
    a.col = g->col;
    a.prio = prio;
    a.color = color;
    a.wait = pool_take<int>(ctx, n);
    a.rcol = pool_take<int>(ctx, m);
    a.queue0 = pool_take<int>(ctx, n);
    a.queue1 = pool_take<int>(ctx, n);
    a.qtail = pool_take<int>(ctx, 3 * kPad);
    a.chunk_tail = pool_take<int>(ctx, 3 * kPad);
    a.chunks = pool_take<int4>(ctx, cap);
    a.chunks1 = grid_mode ? pool_take<int4>(ctx, cap) : nullptr;
    a.chunk_cap = cap;
    a.colored = pool_take<int>(ctx, 3 * kPad);
    a.state = pool_take<int>(ctx, 3 * kPad);
    a.n = (int)n;
    a.threshold = cfg.threshold;
    a.chunk = chunk;
    a.host_ring = ctx->host_ring_dev;
    a.stats = ctx->dstats;
    a.want_stats = stats != nullptr;
    const int grid = std::max(1, std::min<int>(std::min(cfg.grid, resident), (int)((n + cfg.block - 1) / cfg.block)));
    const int dgrid = std::max(1, std::min(cfg.grid, resident));
    st = begin_call(ctx, stream, stats);
    if (st != WC_OK) return st;
    // the counts and round 0
    auto start = [&]() -> wc_status {
        void *args[] = {&a};
        wc_status s = launch(ctx, "color_reset", reinterpret_cast<const void *>(&color_reset), dim3(1), dim3(64), args,
                             stream);
        if (s == WC_OK) s = launch(ctx, "color_count", ks.count, dim3(grid), dim3(cfg.block), args, stream);
        if (s == WC_OK && mode != WC_FLAT)
            s = launch(ctx, "color_count_drain", ks.count_drain, dim3(dgrid), dim3(cfg.block), args, stream);
        const int sg = (int)std::min<long long>((n + kSeedBlock - 1) / kSeedBlock, 4096);
        const void *seed = grid_mode ? reinterpret_cast<const void *>(&color_seed<true>)
                                     : reinterpret_cast<const void *>(&color_seed<false>);
        if (s == WC_OK) s = launch(ctx, "color_seed", seed, dim3(sg), dim3(kSeedBlock), args, stream);
        return s;
    };
    st = start();
    if (st != WC_OK) return st;
    static const char *names[] = {"color_round_flat", "color_round_wave", "color_round_block", "color_round_grid"};
    // relaunch driver: rounds kept in flight (each publishes whether it has
    // work: its queue size, or in grid mode whether chunks or vertices wait);
    // the first empty round ends the loop
    const int window = 4;
    int rounds = 0, launched = 0;
    long long colored = 0;
    // Grid mode, the launch shape, threshold and buffers the library's choice and
    // nothing counted per round: small rounds by one workgroup, many a launch, each
    // launch with a grid-wide round behind it for the one that is too large.  While
    // all rounds are too large those launches would be all loss (3 us a round), so
    // the rounds are the grid's alone, from the start where about n / (mean degree +
    // 1) vertices have no neighbour above them, and after three idle launches on end,
    // until one is small enough (16,384 vertices of 32 random neighbours 541 us a call
    // by the grid alone, 694 by a launch a round, 515 so; 50,000 vertices 787, 1,024
    // and 786; four hubs joined with 30,000 391, 821 and 391).
    constexpr int kPhasedBlock = 256;  // the library's choice
    bool narrow = grid_mode && n <= kNarrowN && chunk <= kNarrowChunk && cfg.block == kPhasedBlock && !stats &&
                  !cfg.own_shape && !(tune && tune->threshold > 0) && cfg.buf_capacity <= 0;
    bool done = false;  // with `colored`
    if (narrow) {
        bool wide = n * n / (m + n) > kNarrowChunks;
        int asked = 0, seen = 0;     // results of launches
        int next = 0, from = 0;      // the grid's next round; the first one of the next small-round launch
        int idle = 0, c = 0;
        for (long long steps = 0;; ++steps) {
            if (steps > 2 * n + 64) return fail(WC_ETIMEOUT, "wc_color: more rounds than vertices");
            for (; asked < seen + (wide ? window : 2); ++asked) {
                clear_round_slot(ctx, asked);
                int r = next, slot = asked;
                if (wide) {
                    ++next;
                } else {
                    void *nargs[] = {&a, &asked, &from};
                    st = launch(ctx, "color_narrow", reinterpret_cast<const void *>(&color_narrow), dim3(1),
                                dim3(kNarrowBlock), nargs, stream);
                    if (st != WC_OK) return st;
                    r = slot = from = -1;
                }
                void *args[] = {&a, &r, &slot};
                st = launch(ctx, names[mode], reinterpret_cast<const void *>(&color_round_grid<kPhasedBlock, true>),
                            dim3(dgrid), dim3(kPhasedBlock), args, stream);
                if (st != WC_OK) return st;
            }
            st = wait_round_count(ctx, seen++, &c);
            if (st != WC_OK) return st;
            if (wide) {
                if (c == 0) break;
                if (c <= kNarrowEnter) {
                    // behind the rounds that are enqueued already
                    wide = false;
                    from = next;
                    seen = asked;
                    idle = 0;
                }
                continue;
            }
            idle = c <= kNarrowIdle ? idle + 1 : 0;
            while (idle >= 3 && c <= kNarrowIdle && seen < asked) {
                // which round the last of the enqueued launches leaves
                st = wait_round_count(ctx, seen++, &c);
                if (st != WC_OK) return st;
            }
            if (idle >= 3 && c <= kNarrowIdle) {
                wide = true;
                next = kNarrowIdle - c + 1;  // the grid does the one it left
            }
            if (c >= 0) {
                done = true;
                colored = c;
                break;
            }
            if (c == kNarrowBad) {
                // what is enqueued behind that launch does nothing
                st = begin_call(ctx, stream, stats);
                if (st == WC_OK) st = start();
                if (st != WC_OK) return st;
                narrow = false;
                break;
            }
        }
    }
    while (!narrow) {
        while (launched < rounds + window) {
            clear_round_slot(ctx, launched);
            int no_slot = -1;
            void *args[] = {&a, &launched, &no_slot};
            st = launch(ctx, names[mode], ks.round, dim3(grid_mode ? dgrid : grid), dim3(cfg.block), args, stream);
            if (st == WC_OK && spills)
                st = launch(ctx, "color_round_drain", ks.round_drain, dim3(dgrid), dim3(cfg.block), args, stream);
            if (st != WC_OK) return st;
            ++launched;
        }
        int c = 0;
        st = wait_round_count(ctx, rounds, &c);
        if (st != WC_OK) return st;
        if (c == 0) break;
        colored += c;
        ++rounds;
        if (!grid_mode && colored > n) return fail(WC_EINVAL, "wc_color: more queued vertices than vertices");
        if (rounds > n + 1) return fail(WC_ETIMEOUT, "wc_color: more rounds than vertices");
    }
    if (grid_mode && !done) {
        // the last round with work colored the vertices of the largest color;
        // a graph without edges has one color and no round with work
        rounds = std::max(rounds, 1);
        clear_host_slot(ctx, kHostSlotGraph);
        void *args[] = {&a};
        st = launch(ctx, "color_publish", reinterpret_cast<const void *>(&color_publish), dim3(1), dim3(64), args,
                    stream);
        if (st != WC_OK) return st;
        int c = 0;
        st = wait_host_slot(ctx, kHostSlotGraph, &c);
        if (st != WC_OK) return st;
        colored = c;
    }
    st = end_call(ctx, stream, stats, rounds, cfg.fail_on_overflow);
    if (st != WC_OK) return st;
    if (colored != n)
        return fail(WC_EINVAL, "wc_color: some vertices never became ready (the graph is not symmetric)");
    return WC_OK;
}
