// Batched SSSP: many independent instances in one launch sequence.
//
// The instances' vertices are numbered consecutively (instance i owns global
// ids vbase[i] .. vbase[i+1]-1) and every round runs one parent kernel over
// the whole id range, so one grid serves all instances.  Each instance brings
// its own consolidation granularity and threshold (picked per size bucket by
// the autotuner): a heavy vertex goes to its wave's ballot buffer, its block's
// LDS buffer or the global chunk buffer, according to its instance's mode, and
// the global buffer consolidates heavy items of all grid-mode instances into
// one child (Sec. IV.A: buffering the work of many would-be child launches).
// The round kernels exit at once when no instance has a frontier, so a fixed
// number of rounds can be captured into a HIP graph and replayed as a single
// launch; the host continues with ordinary rounds if they were not enough.
#include <algorithm>
#include <cstring>
#include <vector>

#include "wc_block.h"
#include "wc_device.h"
#include "wc_internal.h"
#include "wc_stats.h"

namespace wc {
namespace {

constexpr int kPad = 32;
constexpr int kWinInst = 256;  // vertices per entry of the instance lookup table

struct Inst {
    const int *row_ptr;
    const int *col;
    const uint32_t *w;
    uint32_t *dist;
    int n;
    int mode;
    int threshold;
    int chunk;
    int src;
    int m;
};

struct BatchArgs {
    const Inst *inst;
    const int *vbase;  // [count + 1]
    const int *win_inst;  // [total / kWinInst + 1]: instance owning vertex k * kWinInst
    int count;
    int total;         // vbase[count]
    uint16_t *mark;    // [total]: the round whose frontier the vertex is in (its low 8 bits: one of an
                       // earlier round has nothing left to relax) << 8 | bound_code of its distance
    uint32_t *relaxed_at;  // [total]: the largest distance the vertex's edges were last relaxed with
    int *active;       // ring of 3 (stride kPad)
    int *chunk_tail;   // ring of 3 (stride kPad)
    int4 *chunks;      // (global u, begin, end, instance)
    long long chunk_cap;
    unsigned long long *host_ring;
    DevStats *stats;
    int want_stats;
    int has_wave, has_block, has_grid;  // which consolidation levels occur in this batch
};

// Instance owning global vertex gid: the instance owning vertex
// (gid / kWinInst) * kWinInst, from the window table, then forward.
__device__ __forceinline__ int find_inst(const BatchArgs &a, int gid)
{
    int i = a.win_inst[gid / kWinInst];
    while (gid >= a.vbase[i + 1]) ++i;
    return i;
}

__device__ __forceinline__ uint32_t add_sat(uint32_t du, uint32_t w)
{
    uint32_t s = du + w;
    return s < du ? kInf : s;
}

// The edge range of a frontier vertex, its instance's arrays along with it.
struct Range {
    gptr<const int> col;
    gptr<const uint32_t> w;
    gptr<uint32_t> dist;
    gptr<uint16_t> mark;
    int beg, end;
    uint32_t du;
    int m;  // edges of the instance
};

__device__ __forceinline__ Range make_range(const BatchArgs &a, int i)
{
    const Inst &d = a.inst[i];
    return Range{global_ptr(d.col), global_ptr(d.w), global_ptr(d.dist), global_ptr(a.mark + a.vbase[i]), 0, 0, 0u,
                 d.m};
}

// K loaded edges a lane (v[k] < 0: none), nd[k] the distances they offer.  An edge
// is dropped by the byte that bounds its target's distance (bound_code), which takes
// half the cache and which no atomic touches; the others go to the atomic without a
// look at the distance (64 graphs, block level: 1.40 ms a call with it, 1.22
// without).  The mark that a relaxation leaves carries the bound of the distance it
// offers: the vertex's own is never above any of them, whichever store comes last.
// A vertex marked by a relaxation that lowered nothing is found relaxed with its
// distance and passed over.
template <int K>
__device__ __forceinline__ bool relax_loaded(const Range *const (&t)[K], int (&v)[K], const uint32_t (&nd)[K],
                                             int next)
{
    uint32_t bound[K];
    bool any = false;
#pragma unroll
    for (int k = 0; k < K; ++k) bound[k] = v[k] >= 0 ? t[k]->mark[v[k]] & 255u : 0u;
    // all tests before the first atomic: 10 % faster than one edge after another
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = nd[k] < bound_value(bound[k]) ? v[k] : -1;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (v[k] < 0) continue;
        (void)__hip_atomic_fetch_min(&t[k]->dist[v[k]], nd[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        t[k]->mark[v[k]] = (uint16_t)(next << 8 | bound_code(nd[k]));
        any = true;
    }
    return any;
}

// four consecutive entries of a row, which starts anywhere
typedef int Quad __attribute__((ext_vector_type(4), aligned(4)));

// The four edges from e on, of a range with e < end in an instance of at least
// four edges: one load an array, moved down where it would pass the end of the
// array.  v is -1 where there is no edge.
__device__ __forceinline__ void load_quad(const Range &t, int e, int *v, uint32_t *w)
{
    const int q = min(e, t.m - 4);
    const Quad c = *(gptr<const Quad>)(t.col + q), x = *(gptr<const Quad>)(t.w + q);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = q + k >= e && q + k < t.end ? c[k] : -1;
        w[k] = (uint32_t)x[k];
    }
}

// The edges [e, t.end) of a range by a group of lanes (e: the lane's first), U
// times four consecutive edges a lane and step; a step of the group is U * stride
// edges.
template <int U>
__device__ __forceinline__ bool relax_quads(const Range &t, int e, int stride, int next)
{
    bool any = false;
    for (; e < t.end; e += U * stride) {
        int v[4 * U];
        uint32_t w[4 * U];
        const Range *range[4 * U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (e + u * stride < t.end) {
                load_quad(t, e + u * stride, v + 4 * u, w + 4 * u);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) v[4 * u + k] = -1, w[4 * u + k] = 0u;
            }
        }
#pragma unroll
        for (int k = 0; k < 4 * U; ++k) w[k] = add_sat(t.du, w[k]), range[k] = &t;
        any |= relax_loaded<4 * U>(range, v, w, next);
    }
    return any;
}

// Four consecutive edges a lane from the start of its range on, for ranges of
// different vertices (`mine`: the lane has one, of an instance of at least four
// edges).  All lanes of the wave are here, and those that share a target make one
// offer: `base` is the first global id of the lane's instance.  Without that, a
// target that very many vertices point at is offered many distances at once, and
// its atomics take turns: four graphs of 100,000 vertices joined with five hubs,
// wave level: 239 us by reading the distances, 780 by the bound alone, 135 so (64
// power-law graphs at block level 1,112 and 1,113).
__device__ __forceinline__ bool relax_lanes(const Range &t, bool mine, int base, int next)
{
    bool any = false;
    for (int e = t.beg; __any(mine && e < t.end); e += 4) {
        int v[4];
        uint32_t nd[4], bound[4];
        if (mine && e < t.end) {
            load_quad(t, e, v, nd);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = -1, nd[k] = 0u;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) bound[k] = v[k] >= 0 ? t.mark[v[k]] & 255u : 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            nd[k] = add_sat(t.du, nd[k]);
            int id = v[k] >= 0 && nd[k] < bound_value(bound[k]) ? base + v[k] : -1;
            one_of_wave(id, nd[k]);
            v[k] = id >= 0 ? v[k] : -1;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (v[k] < 0) continue;
            (void)__hip_atomic_fetch_min(&t.dist[v[k]], nd[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            t.mark[v[k]] = (uint16_t)(next << 8 | bound_code(nd[k]));
            any = true;
        }
    }
    return any;
}

// The same by one lane and edge by edge (an instance of fewer than four edges).
__device__ __forceinline__ bool relax_single(const Range &t, int next)
{
    bool any = false;
    for (int e = t.beg; e < t.end; ++e) {
        const Range *range[1] = {&t};
        int v[1] = {t.col[e]};
        const uint32_t nd[1] = {add_sat(t.du, t.w[e])};
        any |= relax_loaded<1>(range, v, nd, next);
    }
    return any;
}

__global__ void batch_init(BatchArgs a)
{
    for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < a.total; g += gridDim.x * blockDim.x) {
        const int i = find_inst(a, g);
        const Inst &d = a.inst[i];
        const int v = g - a.vbase[i];
        const bool s = v == d.src;
        d.dist[v] = s ? 0u : kInf;
        a.mark[g] = s ? 0 : 0xffff;
        a.relaxed_at[g] = kInf;
    }
    if (blockIdx.x == 0 && threadIdx.x < 3) {
        a.active[threadIdx.x * kPad] = threadIdx.x == 0 ? 1 : 0;
        a.chunk_tail[threadIdx.x * kPad] = 0;
    }
}

// Windows of BLOCK vertices whose marks a block of batch_round reads together.
constexpr int kWindowsPerStep = 4;

// Lanes of a buffered item of up to kShortItem edges, and of a longer one.
constexpr int kShortItem = 32, kShortLanes = 4, kLongLanes = 16;

// Chunks of a vertex that its own lane writes; more are written by its wave (a
// vertex of 2^20 edges, 8,192 chunks: 1.88 ms a call by its lane, 0.17 by its wave;
// the batch of 64 below 1,253 -> 1,112 us).
constexpr int kOwnChunks = 4;

template <int BLOCK>
struct BatchLds {
    int list[BLOCK * kWindowsPerStep];
    Range item[BLOCK];
    int count[3];
    int scan_tmp[2 * (BLOCK / kWave)];
    int base;
};

// The consolidated child of a wave or a block over its buffer: ns short items
// from item[0] up and nl long ones from item[cap - 1] down, by wave `wid` of nw.
__device__ __forceinline__ bool relax_buffer(const Range *item, int cap, int ns, int nl, int wid, int nw, int next)
{
    constexpr int kLongTask = kWave / kLongLanes, kShortTask = kWave / kShortLanes;
    const int short0 = (nl + kLongTask - 1) / kLongTask, tasks = short0 + (ns + kShortTask - 1) / kShortTask;
    const int lane = lane_id();
    bool any = false;
    for (int t = wid; t < tasks; t += nw) {
        const bool lng = t < short0;
        const int lanes = lng ? kLongLanes : kShortLanes;
        const int i = (lng ? t : t - short0) * (kWave / lanes) + lane / lanes;
        if (i < (lng ? nl : ns)) {
            const Range it = item[lng ? cap - 1 - i : i];
            any |= relax_quads<1>(it, it.beg + 4 * (lane & (lanes - 1)), 4 * lanes, next);
        }
    }
    return any;
}

// Round r over the vertices of all instances.  A block reads the marks of
// kWindowsPerStep windows, lists the frontier vertices among them in LDS and takes
// BLOCK of them at a time, so that a sparse round pays the chain of dependent loads
// (instance, row range, edges, distances) once a step and not once a window.
// Bound by that chain where the frontier is sparse, and by the relaxations' random
// accesses where it is dense (62M edges relaxed in a batch of 64 power-law graphs of
// 2^10 to 2^17 vertices, 16 edges each; its random reads run at about 140 G/s).
// That batch, 16 rounds: block level 1,414 -> 780 us in this kernel (thread-strided
// single edges, a window at a time, generic pointers before) and, with the long
// rows' chunks written by their wave, 1.99 -> 1.08 ms a call, wave level 2.73 ->
// 1.15 ms, grid level 1.73 -> 1.10 ms.  Lane
// groups taking adjacent edges instead of quads: 3 % slower in this kernel.  Two
// or eight windows a step: within 2 % there; 256 graphs 3 % and 1 % slower.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void batch_round(BatchArgs a, int r)
{
    __shared__ BatchLds<BLOCK> sb;
    const int act = a.active[(r % 3) * kPad];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.active[((r + 2) % 3) * kPad] = 0;
        a.chunk_tail[((r + 1) % 3) * kPad] = 0;
        publish_host(a.host_ring, r % kHostRing, a.stats, act);
    }
    if (!act) return;
    const int next = r + 1;
    const int tid = threadIdx.x, lane = lane_id(), wid = tid / kWave;
    StatAcc acc;
    bool any = false;
    constexpr int S = kWindowsPerStep;
    const int stride = gridDim.x * BLOCK;
    if (tid < 3) sb.count[tid] = 0;
    __syncthreads();
    int step = 0;
    for (long long wbase = (long long)blockIdx.x * BLOCK; wbase < a.total; wbase += (long long)S * stride) {
        int mark[S];
#pragma unroll
        for (int w = 0; w < S; ++w) {
            const long long gg = wbase + (long long)w * stride + tid;
            mark[w] = gg < a.total ? a.mark[gg] >> 8 : -1;
        }
        uint64_t mask[S];
        int mine = 0;
#pragma unroll
        for (int w = 0; w < S; ++w) {
            mask[w] = __ballot(mark[w] == (r & 255));
            mine += __builtin_popcountll(mask[w]);
        }
        if (mine) {
            int at = 0;
            if (lane == 0) at = atomicAdd(&sb.count[step], mine);
            at = readlane(at, 0);
#pragma unroll
            for (int w = 0; w < S; ++w) {
                if (mark[w] == (r & 255)) sb.list[at + rank_in(mask[w])] = (int)(wbase + (long long)w * stride) + tid;
                at += __builtin_popcountll(mask[w]);
            }
        }
        // the counter after the next one was last read two barriers ago
        const int after = step == 2 ? 0 : step + 1;
        if (tid == 0) sb.count[after] = 0;
        __syncthreads();
        const int members = sb.count[step];
        step = after;
        for (int m0 = 0; m0 < members; m0 += BLOCK) {
            const bool member = m0 + tid < members;
            int g = 0, base = 0, mode = WC_FLAT, chunk = 1, deg = 0;
            Range t = {};
            if (member) {
                g = sb.list[m0 + tid];
                const int i = find_inst(a, g);
                const Inst &d = a.inst[i];
                base = a.vbase[i];
                const int v = g - base;
                t = make_range(a, i);
                const gptr<const int> row = global_ptr(d.row_ptr);
                t.beg = row[v];
                t.end = row[v + 1];
                t.du = t.dist[v];
                chunk = d.chunk;
                // already relaxed with its present distance (it improved before its
                // own relaxations read it): nothing to do
                if (a.relaxed_at[g] == t.du) t.end = t.beg;
                deg = t.end - t.beg;
                mode = deg > d.threshold ? d.mode : WC_FLAT;
                // a wave's or block's own child keeps items of up to one chunk;
                // longer ones go to the grid-wide drain (the KC_X rule of
                // Sec. IV.E: a warp's or block's child gets many blocks), and so
                // do those of an instance of fewer than four edges, which the
                // children's loads of four would pass the ends of
                if ((mode == WC_WAVE || mode == WC_BLOCK) && (deg > chunk || t.m < 4)) mode = WC_GRID;
                // wave, block and inline work use this reading; grid chunks raise
                // the value from 0 in the drain (or it stays du on overflow)
                if (deg > 0 && mode != WC_GRID) a.relaxed_at[g] = t.du;
            }
            if (a.want_stats) {
                acc.edges += deg;
                acc.buffered += mode != WC_FLAT ? deg : 0;
                acc.items += mode != WC_FLAT ? 1 : 0;
            }
            // inline work: light vertices, four edges at a time
            const bool light = mode == WC_FLAT && deg > 0;
            any |= relax_lanes(t, light && t.m >= 4, base, next);
            if (light && t.m < 4) any |= relax_single(t, next);
            const bool lng = deg > kShortItem;
            // wave-level items: a part of the buffer of the wave's own, no barrier
            if (a.has_wave) {
                const bool it = mode == WC_WAVE;
                const uint64_t shorts = __ballot(it && !lng), longs = __ballot(it && lng);
                if (shorts | longs) {
                    if (a.want_stats && lane == 0) acc.dispatches += 1;
                    Range *const buf = sb.item + wid * kWave;
                    if (it) buf[lng ? kWave - 1 - rank_in(longs) : rank_in(shorts)] = t;
                    wave_lds_sync();
                    any |= relax_buffer(buf, kWave, __builtin_popcountll(shorts), __builtin_popcountll(longs), 0, 1,
                                        next);
                    wave_lds_sync();
                }
            }
            if (!a.has_block && !a.has_grid) continue;
            // block-level items go to the buffer in LDS, grid-level ones as chunks to
            // the global buffer, reserved with one atomic a block
            const bool bl = mode == WC_BLOCK;
            const int nch = mode == WC_GRID ? (deg + chunk - 1) / chunk : 0;
            int at, off, nb, tot;
            block_scan2<BLOCK>(bl ? (lng ? 1 << 16 : 1) : 0, nch, sb.scan_tmp, at, off, nb, tot);
            if (bl) sb.item[lng ? BLOCK - 1 - (at >> 16) : at & 0xffff] = t;
            if (tid == 0) {
                if (tot) sb.base = atomic_add_dev(&a.chunk_tail[(r % 3) * kPad], tot);
                if (a.want_stats && nb) acc.dispatches += 1;
            }
            __syncthreads();
            if (nb) any |= relax_buffer(sb.item, BLOCK, nb & 0xffff, nb >> 16, wid, BLOCK / kWave, next);
            if (tot) {
                const long long slot = (long long)sb.base + off;
                if (nch > 0) a.relaxed_at[g] = slot + nch > a.chunk_cap ? t.du : 0u;
                const int inst = nch > 0 ? find_inst(a, g) : 0;
                // a few chunks by their own lane, more by the wave
                const bool many = nch > kOwnChunks && slot + nch <= a.chunk_cap;
                for (uint64_t m = __ballot(many); m; m &= m - 1) {
                    const int b = __builtin_ctzll(m);
                    const int g0 = readlane(g, b), i0 = readlane(inst, b), n0 = readlane(nch, b), k0 = readlane(chunk, b);
                    const int from = readlane(t.beg, b), to = readlane(t.end, b);
                    int4 *const out = a.chunks + sb.base + readlane(off, b);
                    for (int c = lane; c < n0; c += kWave) {
                        const int cb = from + c * k0;
                        out[c] = make_int4(g0, cb, min(to, cb + k0), i0);
                    }
                }
                for (int c = 0; c < nch && !many; ++c) {
                    const int cb = t.beg + c * chunk, ce = min(t.end, cb + chunk);
                    if (slot + c < a.chunk_cap) {
                        a.chunks[slot + c] = make_int4(g, cb, ce, inst);
                    } else {
                        a.stats->overflowed = 1;
                        Range part = t;
                        part.beg = cb;
                        part.end = ce;
                        any |= relax_single(part, next);
                    }
                }
            }
            __syncthreads();  // the buffers' readers, before the next members
        }
        if (members) __syncthreads();  // the list's readers, before the next step
    }
    if (__ballot(any) && lane == 0) a.active[((r + 1) % 3) * kPad] = 1;
    if (a.want_stats) stat_flush(a.stats, acc);
}

// The drain's grid, in resident grids: the hardware then hands out the chunks in
// their order, so that those in flight are near each other (256 graphs at block
// level 3.64, 3.54, 3.50 ms a call at 1, 2, 4, at grid level 4.16, 4.12, 3.98; the
// batch of 64 within 3 %; 16 pays for empty blocks in the sparse rounds).
constexpr int kDrainWaves = 4;

// The chunks of round r's global buffer: a wave a chunk and two chunks at a time (of
// any instances), adjacent lanes taking adjacent edges: the columns of a row are
// sorted, so their targets share lines.  The source distances are read after the
// edges are requested; the largest one used raises relaxed_at.  606 -> 402 us in the
// batch of 64 (432 with half a wave a chunk and four consecutive edges a lane).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void batch_drain(BatchArgs a, int r)
{
    if (!a.active[(r % 3) * kPad]) return;
    const int tail = a.chunk_tail[(r % 3) * kPad];
    const int total = (long long)tail < a.chunk_cap ? tail : (int)a.chunk_cap;
    const int next = r + 1;
    const int gw = (blockIdx.x * BLOCK + threadIdx.x) / kWave;
    const int nw = gridDim.x * (BLOCK / kWave);
    if (a.want_stats && blockIdx.x == 0 && threadIdx.x == 0 && total > 0)
        atomic_add_dev(&a.stats->rep[0].dispatches, 1ull);
    bool any = false;
    constexpr int U = 2;
    int4 q[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) q[p] = load_or_zero(a.chunks, gw + (long long)p * nw, gw + (long long)p * nw < total);
    for (long long c = gw; c < total; c += 2ll * nw) {
        Range t[2];
        int src[2], gid[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            gid[p] = __builtin_amdgcn_readfirstlane(q[p].x);
            const int i = __builtin_amdgcn_readfirstlane(q[p].w);
            t[p] = make_range(a, i);
            src[p] = gid[p] - a.vbase[i];
            t[p].beg = __builtin_amdgcn_readfirstlane(q[p].y);
            t[p].end = __builtin_amdgcn_readfirstlane(q[p].z);
            const long long n = c + (2ll + p) * nw;
            q[p] = load_or_zero(a.chunks, n, n < total);
        }
        const int len = max(t[0].end - t[0].beg, t[1].end - t[1].beg);
        uint32_t used[2] = {0u, 0u};
        for (int o = 0; o < len; o += U * kWave) {
            int v[2 * U];
            uint32_t w[2 * U];
            const Range *range[2 * U];
#pragma unroll
            for (int k = 0; k < 2 * U; ++k) {
                const Range &x = t[k / U];
                const int e = x.beg + o + (k % U) * kWave + lane_id();
                v[k] = e < x.end ? x.col[e] : -1;
                w[k] = e < x.end ? x.w[e] : 0u;
                range[k] = &x;
            }
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                t[p].du = t[p].beg < t[p].end ? t[p].dist[src[p]] : 0u;
                used[p] = max(used[p], t[p].du);
            }
#pragma unroll
            for (int k = 0; k < 2 * U; ++k) w[k] = add_sat(t[k / U].du, w[k]);
            any |= relax_loaded<2 * U>(range, v, w, next);
        }
        if (lane_id() == 0) {
#pragma unroll
            for (int p = 0; p < 2; ++p)
                if (t[p].beg < t[p].end) atomic_max_dev_noret(&a.relaxed_at[gid[p]], used[p]);
        }
    }
    if (__ballot(any) && lane_id() == 0) a.active[((r + 1) % 3) * kPad] = 1;
}

// Publishes whether round r has a frontier (after the graph's last round).
__global__ void batch_publish(BatchArgs a, int r)
{
    if (threadIdx.x == 0) publish_host(a.host_ring, r % kHostRing, a.stats, a.active[(r % 3) * kPad]);
}

struct BatchKernels {
    const void *round, *drain;
};

BatchKernels pick(int block)
{
    switch (block) {
    case 64: return {reinterpret_cast<const void *>(&batch_round<64>), reinterpret_cast<const void *>(&batch_drain<64>)};
    case 128:
        return {reinterpret_cast<const void *>(&batch_round<128>), reinterpret_cast<const void *>(&batch_drain<128>)};
    case 512:
        return {reinterpret_cast<const void *>(&batch_round<512>), reinterpret_cast<const void *>(&batch_drain<512>)};
    case 1024:
        return {reinterpret_cast<const void *>(&batch_round<1024>),
                reinterpret_cast<const void *>(&batch_drain<1024>)};
    default:
        return {reinterpret_cast<const void *>(&batch_round<256>), reinterpret_cast<const void *>(&batch_drain<256>)};
    }
}

}  // namespace
}  // namespace wc

using namespace wc;

static unsigned long long fnv(unsigned long long h, const void *p, size_t n)
{
    const unsigned char *b = static_cast<const unsigned char *>(p);
    for (size_t k = 0; k < n; ++k) h = (h ^ b[k]) * 1099511628211ull;
    return h;
}

extern "C" wc_status wc_sssp_batch(wc_ctx *ctx, int32_t count, const wc_csr *graphs, const uint32_t *const *w,
                                   const int32_t *src, uint32_t *const *dist, const wc_mode *modes,
                                   const wc_tune *tunes, int32_t graph_rounds, hipStream_t stream, wc_stats *stats)
{
    if (!ctx || count < 0 || (count > 0 && (!graphs || !w || !src || !dist)))
        return fail(WC_EINVAL, "wc_sssp_batch: NULL argument");
    if (count == 0) {
        if (stats) std::memset(stats, 0, sizeof(*stats));
        return WC_OK;
    }
    if (graph_rounds < 0 || graph_rounds > 4096) return fail(WC_EINVAL, "wc_sssp_batch: graph_rounds out of range");
    WC_HIP(hipSetDevice(ctx->device));
    std::vector<Inst> inst(count);
    std::vector<int> vbase(count + 1);
    long long total = 0, cap = 1;
    int block = 256, has[4] = {0, 0, 0, 0};
    for (int i = 0; i < count; ++i) {
        const wc_csr &g = graphs[i];
        if (g.n < 1 || g.m < 0 || !g.row_ptr || !dist[i] || (g.m > 0 && (!g.col || !w[i])))
            return fail(WC_EINVAL, "wc_sssp_batch: bad instance " + std::to_string(i));
        if (src[i] < 0 || src[i] >= g.n)
            return fail(WC_EINVAL, "wc_sssp_batch: source out of range in instance " + std::to_string(i));
        const wc_mode mode = modes ? modes[i] : WC_GRID;
        if (mode < WC_FLAT || mode > WC_GRID) return fail(WC_EINVAL, "wc_sssp_batch: bad mode");
        Config cfg;
        wc_status st = resolve_tune(ctx, "sssp", mode, tunes ? &tunes[i] : nullptr, 1, &cfg);
        if (st != WC_OK) return st;
        // one workgroup size for the whole batch: the first instance's; later
        // instances that leave block_threads unset adopt it
        if (i == 0) block = cfg.block;
        else if (tunes && tunes[i].block_threads > 0 && tunes[i].block_threads != block)
            return fail(WC_EINVAL, "wc_sssp_batch: all instances must share block_threads");
        if (cfg.driver != 0) return fail(WC_EINVAL, "wc_sssp_batch: the persistent driver is disabled");
        const int chunk = kWave * cfg.items_per_lane;
        inst[i] = Inst{g.row_ptr, g.col, w[i], dist[i], g.n, (int)mode, mode == WC_FLAT ? 0x7fffffff : cfg.threshold,
                       chunk, src[i], (int)g.m};
        has[mode] = 1;
        vbase[i] = (int)total;
        total += g.n;
        if (mode == WC_GRID) cap += g.n + g.m / chunk + 1;
        // wave and block levels hand vertices with more than one chunk of edges
        // (at most 2 deg / chunk chunks each) to the grid path, and in an instance
        // of fewer than four edges the one vertex above a threshold (two edges or
        // more), a chunk
        if (mode == WC_WAVE || mode == WC_BLOCK) {
            has[WC_GRID] = 1;
            cap += 2 * (g.m / chunk) + 1;
        }
        if (total > 0x7fffffffLL) return fail(WC_EINVAL, "wc_sssp_batch: more than 2^31 vertices in one batch");
    }
    vbase[count] = (int)total;
    BatchKernels ks = pick(block);
    const int resident = resident_blocks(ctx, ks.round, block);
    const int windows = (int)((total + block - 1) / block);
    // The resident grid, or a workgroup for each window of a small batch.  With
    // wave- or block-level instances also at least a workgroup for each step of
    // kWindowsPerStep windows, so the hardware hands the steps dense with buffered
    // vertices to CUs as they free up (block level, 64 instances of 2^10 to 2^17
    // vertices: 2 % faster; 16 of 2^8 to 2^12, of 85 windows: 0.46 ms by steps
    // alone, 0.24 ms by windows); grid-level instances keep the resident grid
    // (64: even, 16: 0.26 against 0.31 ms).
    int grid = std::max(1, std::min(resident, windows));
    if (has[WC_WAVE] || has[WC_BLOCK]) grid = std::max(grid, (windows + kWindowsPerStep - 1) / kWindowsPerStep);
    const int dgrid = std::max(1, resident * kDrainWaves);
    const long long nwin = total / kWinInst + 1;
    const size_t blob = padded(sizeof(Inst) * count) + padded(4 * (count + 1)) + padded(4 * nwin);
    size_t need = blob + padded(total * 2) + padded(total * 4) + 2 * padded(3 * kPad * 4) + padded(cap * 16);
    wc_status st = pool_reserve(ctx, need, stream);
    if (st != WC_OK) return st;
    BatchArgs a;
    std::memset(&a, 0, sizeof(a));
    char *d_blob = pool_take<char>(ctx, blob);
    a.inst = reinterpret_cast<const Inst *>(d_blob);
    a.vbase = reinterpret_cast<const int *>(d_blob + padded(sizeof(Inst) * count));
    a.win_inst = reinterpret_cast<const int *>(d_blob + padded(sizeof(Inst) * count) + padded(4 * (count + 1)));
    a.count = count;
    a.total = (int)total;
    a.mark = pool_take<uint16_t>(ctx, total);
    a.relaxed_at = pool_take<uint32_t>(ctx, total);
    a.active = pool_take<int>(ctx, 3 * kPad);
    a.chunk_tail = pool_take<int>(ctx, 3 * kPad);
    a.chunks = pool_take<int4>(ctx, cap);
    a.chunk_cap = cap;
    a.host_ring = ctx->host_ring_dev;
    a.stats = ctx->dstats;
    a.want_stats = stats != nullptr;
    a.has_wave = has[WC_WAVE];
    a.has_block = has[WC_BLOCK];
    a.has_grid = has[WC_GRID];
    // descriptors (instances, then vertex offsets) in one staged upload
    std::vector<char> host_blob(blob, 0);
    std::memcpy(host_blob.data(), inst.data(), sizeof(Inst) * count);
    std::memcpy(host_blob.data() + padded(sizeof(Inst) * count), vbase.data(), 4 * (count + 1));
    {
        int *win = reinterpret_cast<int *>(host_blob.data() + padded(sizeof(Inst) * count) + padded(4 * (count + 1)));
        int i = 0;
        for (long long k = 0; k < nwin; ++k) {
            const long long v = k * kWinInst;
            while (i + 1 < count && v >= vbase[i + 1]) ++i;
            win[k] = i;
        }
    }
    st = stage_to_device(ctx, d_blob, host_blob.data(), blob, stream);
    if (st != WC_OK) return st;
    st = begin_call(ctx, stream, stats);
    if (st != WC_OK) return st;
    {
        void *args[] = {&a};
        const int ig = (int)std::min<long long>((total + 255) / 256, 8192);
        st = launch(ctx, "batch_init", reinterpret_cast<const void *>(&batch_init), dim3(ig), dim3(256), args, stream);
        if (st != WC_OK) return st;
    }
    int rounds_done = 0;
    if (graph_rounds > 0) {
        // graph_rounds rounds captured once into a graph (its kernels exit at
        // once past convergence), replayed as one launch while the arguments stay
        // the same; a final kernel publishes whether more rounds are needed
        unsigned long long key = 1469598103934665603ull;
        key = fnv(key, &a, sizeof(a));
        key = fnv(key, &graph_rounds, sizeof(graph_rounds));
        key = fnv(key, &grid, sizeof(grid));
        key = fnv(key, &dgrid, sizeof(dgrid));
        key = fnv(key, &block, sizeof(block));
        if (!ctx->graph_exec || ctx->graph_key != key) {
            if (ctx->graph_exec) {
                WC_HIP(hipStreamSynchronize(stream));
                WC_HIP(hipStreamSynchronize(ctx->capture_stream));
                (void)hipGraphExecDestroy(ctx->graph_exec);
                ctx->graph_exec = nullptr;
            }
            hipGraph_t graph = nullptr;
            WC_HIP(hipStreamBeginCapture(ctx->capture_stream, hipStreamCaptureModeThreadLocal));
            const int saved_timing = ctx->timing;
            ctx->timing = 0;  // no event records inside the captured graph
            for (int r = 0; r < graph_rounds && st == WC_OK; ++r) {
                void *args[] = {&a, &r};
                st = launch(ctx, "batch_round", ks.round, dim3(grid), dim3(block), args, ctx->capture_stream);
                if (st == WC_OK)
                    st = launch(ctx, "batch_drain", ks.drain, dim3(dgrid), dim3(block), args, ctx->capture_stream);
            }
            int rr = graph_rounds;
            void *pargs[] = {&a, &rr};
            if (st == WC_OK)
                st = launch(ctx, "batch_publish", reinterpret_cast<const void *>(&batch_publish), dim3(1), dim3(64),
                            pargs, ctx->capture_stream);
            ctx->timing = saved_timing;
            hipError_t e = hipStreamEndCapture(ctx->capture_stream, &graph);
            if (st != WC_OK) {
                if (graph) (void)hipGraphDestroy(graph);
                return st;
            }
            if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
            e = hipGraphInstantiate(&ctx->graph_exec, graph, nullptr, nullptr, 0);
            (void)hipGraphDestroy(graph);
            if (e != hipSuccess) {
                ctx->graph_exec = nullptr;
                return hip_fail(e, "hipGraphInstantiate");
            }
            ctx->graph_key = key;
        }
        for (int r = 0; r <= graph_rounds; ++r) clear_round_slot(ctx, r);
        chain_break(ctx);
        WC_HIP(hipEventRecord(ctx->graph_ready, stream));
        WC_HIP(hipStreamWaitEvent(ctx->capture_stream, ctx->graph_ready, 0));
        WC_HIP(hipGraphLaunch(ctx->graph_exec, ctx->capture_stream));
        WC_HIP(hipEventRecord(ctx->graph_done, ctx->capture_stream));
        WC_HIP(hipStreamWaitEvent(stream, ctx->graph_done, 0));
        int c = 0;
        st = wait_round_count(ctx, graph_rounds, &c);
        if (st != WC_OK) return st;
        rounds_done = graph_rounds;
        if (c == 0) return end_call(ctx, stream, stats, graph_rounds, false);
    }
    // ordinary rounds (all of them without a graph, or the ones the graph did not cover)
    const int window = 4;
    int rounds = rounds_done, launched = rounds_done;
    for (;;) {
        while (launched < rounds + window) {
            clear_round_slot(ctx, launched);
            void *args[] = {&a, &launched};
            st = launch(ctx, "batch_round", ks.round, dim3(grid), dim3(block), args, stream);
            if (st == WC_OK) st = launch(ctx, "batch_drain", ks.drain, dim3(dgrid), dim3(block), args, stream);
            if (st != WC_OK) return st;
            ++launched;
        }
        int c = 0;
        st = wait_round_count(ctx, rounds, &c);
        if (st != WC_OK) return st;
        if (c == 0) break;
        ++rounds;
        if (rounds > total + 1) return fail(WC_ETIMEOUT, "wc_sssp_batch: more rounds than vertices");
    }
    return end_call(ctx, stream, stats, rounds, false);
}
