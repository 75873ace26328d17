// SpMV with workload consolidation (irregular loop over CSR rows).
//
// One parent work item per row.  Prework reads the row's range; a row with
// more than `threshold` nonzeros is inserted into the consolidation buffer of
// its mode, a lighter row is summed inline by its lane ("work").
//   wave  - ballot-mask buffer; the wave sums its buffered rows.
//   block - LDS buffer, then the workgroup barrier; the block's waves sum the
//           buffered rows.
//   In both, the child sizes its lanes per row as grid mode does (below): g =
//   the power of two >= len / items_per_lane lanes per row, lane l of a group
//   taking elements l, l+g, ..., then a fixed butterfly over the group; the
//   rows of one g go 64 / g to a wave step.  A buffered row too long for one
//   group's child (more than one
//   chunk, 64 * items_per_lane nonzeros) is handed on as chunks to a global
//   buffer that the grid-mode drain spreads over the whole grid after the
//   parent (the KC_X rule of Sec. IV.E gives a warp's or block's child many
//   blocks); its chunk partials are combined in chunk order.
//   grid  - global buffers and a grid-wide barrier (kernel boundary).  The
//           child-work thread-count heuristic sizes the group of lanes that
//           sums one buffered row: g = the power of two >= len / items_per_lane,
//           so each lane takes about items_per_lane nonzeros.  Rows are binned by
//           g (1..64) and one wave sums 64 / g rows of a bin at once; a row
//           longer than 64 * items_per_lane is split into chunks of that size,
//           one wave each, and its chunk partials are combined in chunk order.
//           A bin's buffer holds every row, so the parent reserves places as it goes;
//           a small matrix runs in one launch (spmv_small).
//   flat  - every row is summed by its own lane.
// All sums are fp32 fused multiply-adds whose order depends only on the row
// length, the mode and the tune, so results are bitwise reproducible.  Every
// serial part of a sum (a lane's share of a row, a wave's chunk partials) goes
// through a Cascade, so no product is rounded more than ~140 times on the way
// to y for rows of up to 2^26 nonzeros in any mode; 140 * 2^-24 < 1e-5, so
// |y - y_ref| <= 1e-5 * sum |a_ij x_j| holds as a worst-case bound per row.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "wc_block.h"
#include "wc_device.h"
#include "wc_internal.h"
#include "wc_stats.h"

namespace wc {
namespace {

constexpr int kBins = 7;      // group sizes 1, 2, 4, ..., 64 lanes
constexpr int kChunkBin = 7;  // rows split into whole-wave chunks
constexpr int kUnroll = 4;    // nonzeros in flight per lane
constexpr int kMultiCol = 8;  // column of the per-block counts holding split rows
constexpr int kCols = 9;
constexpr int kPad = 32;  // the bins' counters live on separate 128-byte lines

struct SpmvArgs {
    const int *row_ptr;
    const int *col;
    const float *val;  // nullptr: every stored entry is 1 (the in-edge sums of PageRank)
    const float *x;
    float *y;
    // hot-column layout (wc_spmv_hot): column c < hot is the c-th most used
    // column, whose x value is x_hot[c]; column hot + j is column j of x
    const float *x_hot;
    const int *hot_ids;
    int hot;
    int n;
    int threshold;
    int ipl;           // items per lane
    int chunk;         // 64 * ipl
    int spill;         // wave and block modes: buffered rows longer than this go to the global chunks
    int count_drain;   // grid mode: the drain counts as the consolidated dispatch
    int windows;       // grid mode: windows of a binning step, 1 .. kWindows
    // grid mode
    int *bin_total;    // [kCols * kPad]: rows per bin 0..6, chunks, split rows; zeroed before the parent
    int *rows_buf;     // binned rows, see bin_entry
    long long bin_off[kBins + 1];
    long long rows_cap;  // driver 2: entries of `basic`
    int4 *basic;       // driver 2: (row, begin, end, 0)
    int4 *chunks;      // (what counts the chunk, begin, end, entry in multi), see put_chunk
    long long chunk_cap;
    int *groups;       // chunks still to be summed of the groups of long rows
    int4 *multi;       // (row, first chunk, chunk count, chunks or groups still to be summed)
    long long multi_cap;
    float *partials;   // one per chunk slot
    DevStats *stats;
    int want_stats;
};

// x value of stored column c.  Plain layout (hot = 0): x[c].  Hot-column
// layout: the first nlds hot values staged in LDS (xs), the other hot ones in
// x_hot, the rest in x.
__device__ __forceinline__ float load_x(const SpmvArgs &a, const float *xs, int nlds, int c)
{
    if (c < a.hot) return c < nlds ? xs[c] : a.x_hot[c];
    return a.x[c - a.hot];
}

// Sum of val[e] * x[col[e]] over e = first + k * stride (k >= 0, e < end), in
// order of k, U loads in flight; the U products of a step are fused into the
// cascade's first partial sum one after another.
template <int U>
__device__ __forceinline__ float dot_strided_u(const SpmvArgs &a, int first, int stride, int end,
                                               const float *xs = nullptr, int nlds = 0)
{
    Cascade cs;
    for (int e0 = first; e0 < end; e0 += U * stride) {
        int c[U];
        float v[U], xv[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int e = e0 + k * stride;
            const bool ok = e < end;
            c[k] = ok ? a.col[e] : -1;
            v[k] = ok ? (a.val ? a.val[e] : 1.f) : 0.f;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) xv[k] = c[k] >= 0 ? load_x(a, xs, nlds, c[k]) : 0.f;
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (c[k] >= 0) cs.s0 = fmaf(v[k], xv[k], cs.s0);
        cs.step<U>();
    }
    return cs.total();
}

__device__ __forceinline__ float dot_strided(const SpmvArgs &a, int first, int stride, int end)
{
    return dot_strided_u<kUnroll>(a, first, stride, end);
}

__device__ __forceinline__ float dot_wave(const SpmvArgs &a, int beg, int end)
{
    return wave_sum(dot_strided(a, beg + lane_id(), kWave, end));
}

// Sum over aligned groups of g lanes (g a power of two <= 64), fixed order.
__device__ __forceinline__ float group_sum(float v, int g)
{
    for (int d = g >> 1; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

// log2 of the lane group of a row of len entries: the smallest power of two g
// with g * ipl >= len.  Called with 64 * ipl >= len; counted, not divided.
__device__ __forceinline__ int bin_of(int len, int ipl)
{
    int b = 0;
#pragma unroll
    for (int k = 0; k < kBins - 1; ++k) b += len > ipl << k ? 1 : 0;
    return b;
}

// A light row (up to kLight entries, more with a larger threshold), summed by
// its lane.
constexpr int kLight = 2 * kUnroll;
__device__ __forceinline__ float light_row(const SpmvArgs &a, int beg, int end)
{
    return dot_strided_u<kLight>(a, beg, 1, end);
}

// Entry i of bin b in rows_buf: even bins grow upward, odd ones downward.
__device__ __forceinline__ long long bin_entry(const SpmvArgs &a, int b, int i)
{
    return b & 1 ? a.bin_off[b] - i : a.bin_off[b] + i;
}

// Chunks of split rows.  A row's entry in multi counts its chunks that are still
// to be summed or, for a row of more than kGroup chunks, its groups: the chunks
// with entries in one run of kGroup entries of the buffer, counted in `groups`.
// Such a row reaches beyond a run, so a run has two of them at most, one from its
// start on and one that begins later, with a count each.
constexpr int kGroup = 64;
constexpr int kGroupPad = 8;  // counts of a run (two are used): four runs a line
enum { kRow = 0, kGroupOf = 1 };  // chunks[].x: counted by the row; or by count x - kGroupOf of the run; -1: empty

// The group of a row of n chunks from `first` that has the entry `slot`: where its
// count is, and what that starts from.
__device__ __forceinline__ int group_of(int first, int slot) { return first > (slot & ~(kGroup - 1)) ? 1 : 0; }
__device__ __forceinline__ long long group_index(int slot, int which)
{
    return (long long)(slot / kGroup) * kGroupPad + which;
}
__device__ __forceinline__ int group_count(int first, int n, int slot)
{
    const long long run = slot & ~(kGroup - 1);
    return (int)(min((long long)first + n, run + kGroup) - max((long long)first, run));
}
// What the row's entry in multi counts.
__device__ __forceinline__ int row_count(int first, int n)
{
    return n <= kGroup ? n : (first + n - 1) / kGroup - first / kGroup + 1;
}

// Chunk c of a row [beg, end) of n chunks whose first has the entry `first`.
__device__ __forceinline__ void put_chunk(const SpmvArgs &a, int first, int n, int c, int beg, int end, int entry)
{
    const int slot = first + c, cb = beg + c * a.chunk;
    int by = kRow;
    if (n > kGroup) {
        const int which = group_of(first, slot);
        by = kGroupOf + which;
        if (c == 0 || slot % kGroup == 0) a.groups[group_index(slot, which)] = group_count(first, n, slot);
    }
    a.chunks[slot] = make_int4(by, cb, min(end, cb + a.chunk), entry);
}

template <int BLOCK>
struct SpmvBlockBuf {
    int row[BLOCK];  // buffered rows, laid out by bin
    int beg[BLOCK];
    int end[BLOCK];
    int cnt[kBins + 1];   // rows per bin; [kBins]: heavy rows (work counters)
    int off[kBins];       // first row of each bin
    int task[kBins + 1];  // first task of each bin; [kBins]: task count
};

__device__ __forceinline__ void count_stats(StatAcc &acc, int len, bool heavy, bool wave_dispatch)
{
    acc.edges += len;
    acc.buffered += heavy ? len : 0;
    acc.items += heavy ? 1 : 0;
    if (wave_dispatch && __ballot(heavy) && lane_id() == 0) acc.dispatches += 1;
}

// Hands the rows of the lanes with nch > 0 on as chunks of the global buffer
// (wave and block modes): one reservation per wave for the chunks and one for
// the split-row records; the wave writes each row's chunks together.  A row
// whose chunks do not all fit is summed by its own lane instead (the overflow
// fallback) and its reserved entries are marked empty.  Every lane calls this.
__device__ __forceinline__ void spill_rows(const SpmvArgs &a, int r, int beg, int end, int nch)
{
    const int slot = wave_reserve_n(nch, &a.bin_total[kChunkBin * kPad]);
    const int mslot = wave_reserve(nch > 0, &a.bin_total[kMultiCol * kPad]);
    const bool fits = nch > 0 && (long long)slot + nch <= a.chunk_cap && mslot < a.multi_cap;
    uint64_t m = __ballot(fits);
    while (m) {
        const int b = __builtin_ctzll(m);
        m &= m - 1;
        const int s0 = readlane(slot, b), n0 = readlane(nch, b), rb = readlane(beg, b), re = readlane(end, b);
        const int rm = readlane(mslot, b);
        for (int c = lane_id(); c < n0; c += kWave) put_chunk(a, s0, n0, c, rb, re, rm);
    }
    if (fits) a.multi[mslot] = make_int4(r, slot, nch, row_count(slot, nch));
    if (nch > 0 && !fits) {
        for (int c = 0; c < nch; ++c)
            if ((long long)slot + c < a.chunk_cap) a.chunks[slot + c] = make_int4(-1, 0, 0, 0);
        a.stats->overflowed = 1;
        a.y[r] = dot_strided(a, beg, 1, end);
    }
}

// Zeroes the bin totals before a parent reserves entries of its buffers.
__global__ void spmv_reset(SpmvArgs a)
{
    if (threadIdx.x < kCols) a.bin_total[threadIdx.x * kPad] = 0;
}

// Parent kernel of the flat, wave and block modes.
template <int MODE, int BLOCK>
__global__ __launch_bounds__(BLOCK) void spmv_parent(SpmvArgs a)
{
    const int lane = lane_id();
    StatAcc acc;
    for (int base = blockIdx.x * BLOCK; base < a.n; base += gridDim.x * BLOCK) {
        const int r = base + threadIdx.x;
        const bool valid = r < a.n;
        int beg = 0, end = 0;
        if (valid) {
            beg = a.row_ptr[r];
            end = a.row_ptr[r + 1];
        }
        const int len = end - beg;
        const bool heavy = MODE != WC_FLAT && len > a.threshold;
        if (a.want_stats) count_stats(acc, len, heavy, MODE == WC_WAVE);
        if (valid && !heavy) a.y[r] = dot_strided(a, beg, 1, end);
        // buffered rows too long for the group's own child go to the global chunks
        const bool spill = heavy && len > a.spill;
        if constexpr (MODE != WC_FLAT) {
            if (__ballot(spill)) spill_rows(a, r, beg, end, spill ? (len + a.chunk - 1) / a.chunk : 0);
        }
        const bool mine = heavy && !spill;

        // the child: the scope's buffered rows grouped by bin, g = 2^b lanes
        // per row (the smallest group that covers the row at items_per_lane
        // nonzeros a lane), 64 / g rows a wave step
        const int bin = mine ? bin_of(len, a.ipl) : -1;
        if constexpr (MODE == WC_WAVE) {
            const int wbase = base + (threadIdx.x & ~(kWave - 1));
            for (int b = 0; b < kBins; ++b) {
                const uint64_t m = __ballot(bin == b);
                if (!m) continue;
                // lane k learns which lane holds the bin's k-th row: the
                // members go to slots 0..cnt-1, the others after them, so the
                // permutation writes every lane once
                const int cnt = __popcll(m);
                const int to = bin == b ? rank_in(m) : cnt + rank_in(~m);
                const int src = __builtin_amdgcn_ds_permute(to << 2, lane);
                const int g = 1 << b, sub = lane & (g - 1);
                for (int i0 = 0; i0 < cnt; i0 += kWave >> b) {
                    const int i = i0 + (lane >> b);
                    const int from = __shfl(src, i < cnt ? i : 0, kWave);
                    const int rb = __shfl(beg, from, kWave), re = __shfl(end, from, kWave);
                    float s = dot_strided(a, i < cnt ? rb + sub : 0, g, i < cnt ? re : 0);
                    s = group_sum(s, g);
                    if (i < cnt && sub == 0) a.y[wbase + from] = s;
                }
            }
        } else if constexpr (MODE == WC_BLOCK) {
            __shared__ SpmvBlockBuf<BLOCK> sb;
            constexpr int NW = BLOCK / kWave;
            // per-bin insert positions: a row's sum depends only on its own
            // range and g, not on where it sits, so LDS atomics may order a bin
            if (threadIdx.x <= kBins) sb.cnt[threadIdx.x] = 0;
            __syncthreads();
            const int k = bin >= 0 ? atomicAdd(&sb.cnt[bin], 1) : 0;
            if (a.want_stats && heavy) atomicAdd(&sb.cnt[kBins], 1);
            __syncthreads();
            if (threadIdx.x == 0) {
                int o = 0, t = 0;
                for (int b = 0; b < kBins; ++b) {
                    sb.off[b] = o;
                    sb.task[b] = t;
                    o += sb.cnt[b];
                    t += (sb.cnt[b] + (kWave >> b) - 1) / (kWave >> b);
                }
                sb.task[kBins] = t;
                if (a.want_stats && sb.cnt[kBins]) acc.dispatches += 1;
            }
            __syncthreads();
            if (bin >= 0) {
                const int q = sb.off[bin] + k;
                sb.row[q] = r;
                sb.beg[q] = beg;
                sb.end[q] = end;
            }
            __syncthreads();  // the "synchronize" between inserts and the child
            // tasks of 64 / g rows of one bin, dealt round-robin to the waves
            const int total = sb.task[kBins];
            for (int t = threadIdx.x / kWave; t < total; t += NW) {
                int b = 0;
                while (b + 1 < kBins && sb.task[b + 1] <= t) ++b;
                const int g = 1 << b, sub = lane & (g - 1);
                const int i = (t - sb.task[b]) * (kWave >> b) + (lane >> b);
                const bool ok = i < sb.cnt[b];
                const int q = sb.off[b] + (ok ? i : 0);
                float s = dot_strided(a, ok ? sb.beg[q] + sub : 0, g, ok ? sb.end[q] : 0);
                s = group_sum(s, g);
                if (ok && sub == 0) a.y[sb.row[q]] = s;
            }
            __syncthreads();  // LDS buffer is reused by the next window
        }
    }
    if (a.want_stats) stat_flush(a.stats, acc);
}

// ---- grid mode --------------------------------------------------------------------------------

// Parent pass of grid mode: heavy rows into the buffers of their bins, light
// rows summed inline.  A block counts its rows of up to kWindows windows per bin
// with LDS atomics, which also give each row its place, reserves the entries
// with one atomic per bin, and sums its light rows while that is on its way.  A
// row's sum depends on its own range only, so the order in which rows get their
// places does not show in y.  Bound by latency and by the gathers of the light
// rows' x.  A count pass, a scan over all blocks and a parent took three
// launches: scale-22 graph 105 -> 80 us (about 40 of them for the light rows),
// 200,003 rows 30 -> 13 us.  Ranking the rows by ballots took 82 and 16 us; the
// light rows in workgroups of their own, or flattened over the wave's lanes, or
// in the drain gained nothing.
// STATS: the instantiation that counts work for wc_stats.
constexpr int kWindows = 4;
template <int BLOCK, bool STATS>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(8))) void spmv_parent_grid(SpmvArgs a)
{
    constexpr int kPosBits = 27;  // a block's chunks of one step: fewer than 2^31 / 64 entries
    __shared__ int s_cnt[kCols], s_base[kCols];
    __shared__ int s_where[kWindows][BLOCK];  // (bin << kPosBits) | place in the block's share of it; -1: light
    const int lane = lane_id(), tid = threadIdx.x;
    const int W = a.windows;
    StatAcc acc;
    // a block's windows lie a whole grid apart: neighbouring rows are often alike
    // (a power-law graph's hubs have small ids), and the hubs' chunks take longest
    const long long stride = (long long)gridDim.x * BLOCK;
    for (long long base = (long long)blockIdx.x * BLOCK; base < a.n; base += W * stride) {
        int len[kWindows];
#pragma unroll
        for (int w = 0; w < kWindows; ++w) {
            const long long r = base + w * stride + tid;
            len[w] = w < W && r < a.n ? a.row_ptr[r + 1] - a.row_ptr[r] : 0;
        }
        if (tid < kCols) s_cnt[tid] = 0;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kWindows; ++w) {
            if (w >= W) break;
            const bool heavy = len[w] > a.threshold;
            if (STATS) count_stats(acc, len[w], heavy, false);
            int where = -1;
            if (heavy) {
                const bool split = len[w] > a.chunk;
                const int bin = split ? kChunkBin : bin_of(len[w], a.ipl);
                where = bin << kPosBits | atomicAdd(&s_cnt[bin], split ? (len[w] + a.chunk - 1) / a.chunk : 1);
                if (split) atomicAdd(&s_cnt[kMultiCol], 1);
            }
            s_where[w][tid] = where;
        }
        __syncthreads();
        int at = 0;
        if (tid < kCols && s_cnt[tid]) at = atomic_add_dev(&a.bin_total[tid * kPad], s_cnt[tid]);
#pragma unroll 1
        for (int w = 0; w < W; ++w) {
            const long long r = base + w * stride + tid;
            if (r < a.n && s_where[w][tid] < 0) a.y[r] = light_row(a, a.row_ptr[r], a.row_ptr[r + 1]);
        }
        if (tid < kCols) s_base[tid] = at;
        __syncthreads();
#pragma unroll 1
        for (int w = 0; w < W; ++w) {
            const int where = s_where[w][tid], bin = where < 0 ? -1 : where >> kPosBits;
            const int pos = where & ((1 << kPosBits) - 1);
            const int r = (int)(base + w * stride + tid);
            if (bin >= 0 && bin < kBins) a.rows_buf[bin_entry(a, bin, s_base[bin] + pos)] = r;
            // split rows: the wave writes their chunks side by side, chunk j of the
            // wave belonging to the last row whose chunks begin at or before j
            const bool split = bin == kChunkBin;
            const uint64_t sm = __ballot(split);
            if (!sm) continue;
            const int rb = split ? a.row_ptr[r] : 0, re = split ? a.row_ptr[r + 1] : 0;
            const int nch = (re - rb + a.chunk - 1) / a.chunk;
            const int slot = s_base[kChunkBin] + pos;
            int mslot = 0;  // entries of the block's split rows, in any order
            if (split) mslot = s_base[kMultiCol] + atomicAdd(&s_cnt[kMultiCol], -1) - 1;
            const bool fits = split && (long long)slot + nch <= a.chunk_cap;
            const int take = fits ? nch : 0, incl = wave_incl_scan(take), pre = incl - take;
            const int chunks = readlane(incl, kWave - 1);
            for (int j0 = 0; j0 < chunks; j0 += kWave) {
                const int j = j0 + lane;
                int own = 0;
#pragma unroll
                for (int d = kWave / 2; d >= 1; d >>= 1) own += __shfl(pre, own + d, kWave) <= j ? d : 0;
                const int c = j - __shfl(pre, own, kWave);
                const int b0 = __shfl(rb, own, kWave), e0 = __shfl(re, own, kWave), n0 = __shfl(nch, own, kWave);
                const int s0 = __shfl(slot, own, kWave), rm = __shfl(mslot, own, kWave);
                if (j < chunks) put_chunk(a, s0, n0, c, b0, e0, rm);
            }
            if (fits) {
                a.multi[mslot] = make_int4(r, slot, nch, row_count(slot, nch));
            } else if (split) {
                // buffer full: mark the reserved slots that exist as empty and sum
                // the row inline (fallback); no chunk refers to its split-row entry
                for (int c = 0; c < nch; ++c)
                    if ((long long)slot + c < a.chunk_cap) a.chunks[slot + c] = make_int4(-1, 0, 0, 0);
                a.stats->overflowed = 1;
                a.y[r] = dot_strided(a, rb, 1, re);
            }
        }
        __syncthreads();  // the counts are cleared by the next step
    }
    if (STATS) stat_flush(a.stats, acc);
}

// Hot x values staged in LDS by the drain of the hot-column layout: 32 per
// thread, at most 16384 (64 KiB), so that four waves per SIMD stay resident.
template <int BLOCK>
constexpr int lds_hot_for() { return 32 * BLOCK < 16384 ? 32 * BLOCK : 16384; }

template <int BLOCK, bool HOT>
struct DrainLds {
    float x[HOT ? lds_hot_for<BLOCK>() : 1];
};

// Consolidated child of grid mode.  Wave tasks: first one task per chunk of the
// split rows; then, for bin b (g = 2^b lanes per row), 64 / g consecutive rows
// of the bin a task.  LIGHT: the buffers of an earlier product on the same
// matrix are still in place (PageRank's later sweeps), and the rows up to the
// threshold, which the parent sums otherwise, come last, 64 a task.
// The entry of a wave's next task is requested before the current one's
// entries.
// Post-work of split rows, by the wave whose chunk is the row's last one to be
// done: the row's partials summed in chunk order, whoever does it.  A wave's
// partials have reached memory (the wait) before it lowers the counts of their
// rows or groups; the wave that takes a group's to zero lowers the row's after
// that; and the counts go down by atomics alone, so the wave that takes a row's to
// zero finds every partial.  The counts are lowered between the wave's chunks and
// its other tasks, which hide the round trips (counting after every chunk cost
// 17 us of the scale-22 product, this 7, a kernel of its own a launch), and are
// left as they were found, for the next product on the same buffers.
// Groups, for atomics on one line take turns: with a count a row only, a product
// with six rows of 2^19 entries took 89 us in grid mode (chunks of 512) and 171 in
// wave mode (128), one row of 2^20 entries 55 and 142; now 31 and 45, 33 and 36.
// Bound by the gathers of x, a line request a lane: 62M of them in 433 us on the
// scale-22 graph, a bare gather of its 67M columns 385 us.
constexpr int kPartials = 8;  // partials of a long row in flight per lane
__device__ __forceinline__ float load_partial(const SpmvArgs &a, int k)
{
    return __hip_atomic_load(&a.partials[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// mi: the lane's split-row entry (-1: none), by: what counts its chunk, left: that
// count before it was lowered.
__device__ __forceinline__ void combine_rows(const SpmvArgs &a, int mi, int by, int left)
{
    asm volatile("" : : "v"(left) : "memory");
    bool last = left == 1;
    if (last && by != kRow) last = atomic_add_dev(&a.multi[mi].w, -1) == 1;
    for (uint64_t m = __ballot(last); m; m &= m - 1) {
        int4 *q = &a.multi[readlane(mi, __builtin_ctzll(m))];
        const int row = q->x, first = q->y, cnt = q->z;
        Cascade cs;
        int k = lane_id();
        for (; k + (kPartials - 1) * kWave < cnt; k += kPartials * kWave) {
            float v[kPartials];
#pragma unroll
            for (int u = 0; u < kPartials; ++u) v[u] = load_partial(a, first + k + u * kWave);
#pragma unroll
            for (int u = 0; u < kPartials; ++u) cs.add(v[u]);
        }
        for (; k < cnt; k += kWave) cs.add(load_partial(a, first + k));
        const float s = wave_sum(cs.total());
        const int counts = row_count(first, cnt);
        for (int g = lane_id(); cnt > kGroup && g < counts; g += kWave) {
            const int slot = max(first, (first / kGroup + g) * kGroup);
            a.groups[group_index(slot, group_of(first, slot))] = group_count(first, cnt, slot);
        }
        if (lane_id() == 0) {
            a.y[row] = s;
            q->w = counts;
        }
    }
}

template <int BLOCK, bool HOT, bool LIGHT>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(HOT ? 4 : 8))) void spmv_drain(SpmvArgs a)
{
    constexpr int kKinds = kBins + 1;  // chunks, the bins; then the light rows
    __shared__ int s_cnt[kKinds], s_task[kKinds + 2];
    __shared__ DrainLds<BLOCK, HOT> s_x;
    const int nlds = HOT ? min(a.hot, lds_hot_for<BLOCK>()) : 0;
    if (HOT)
        for (int i = threadIdx.x; i < nlds; i += BLOCK) s_x.x[i] = a.x_hot[i];
    if (threadIdx.x == 0) {
        int t = 0;
        for (int k = 0; k < kKinds; ++k) {
            int c = a.bin_total[(k ? k - 1 : kChunkBin) * kPad];
            if (k == 0) c = (long long)c < a.chunk_cap ? c : (int)a.chunk_cap;
            s_cnt[k] = c;
            s_task[k] = t;
            t += k ? (c + (kWave >> (k - 1)) - 1) / (kWave >> (k - 1)) : c;
        }
        s_task[kKinds] = t;
        if (a.want_stats && a.count_drain && blockIdx.x == 0 && t > 0)
            atomic_add_dev(&a.stats->rep[0].dispatches, 1ull);
        if (LIGHT) t += (int)(((long long)a.n + kWave - 1) / kWave);
        s_task[kKinds + 1] = t;
    }
    __syncthreads();
    // a wave's task, its kind and its position are uniform and kept so
    const int total = __builtin_amdgcn_readfirstlane(s_task[kKinds + 1]);
    const int chunks = __builtin_amdgcn_readfirstlane(s_cnt[0]);
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int gw = blockIdx.x * (BLOCK / kWave) + wid;
    const int nw = gridDim.x * (BLOCK / kWave);
    const int lane = lane_id();
    // lane k: split-row entry of the wave's k-th chunk, what counts it, and that count before it was lowered
    int t = gw, mi = -1, by = kRow, left = 0;
    while (t < chunks) {
        combine_rows(a, mi, by, left);  // a wave has more than 64 chunks
        mi = -1;
        by = kRow;
        int slot = 0;
        for (int k = 0; k < kWave && t < chunks; ++k, t += nw) {
            const int4 d = a.chunks[t];
            const int kind = __builtin_amdgcn_readfirstlane(d.x), from = __builtin_amdgcn_readfirstlane(d.y);
            const int to = __builtin_amdgcn_readfirstlane(d.z), entry = __builtin_amdgcn_readfirstlane(d.w);
            const float s = wave_sum(dot_strided_u<2 * kUnroll>(a, from + lane, kWave, to, s_x.x, nlds));
            if (lane == 0) __hip_atomic_store(&a.partials[t], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == k && kind >= 0) {
                mi = entry;
                by = kind;
                slot = t;
            }
        }
        int *count = by == kRow ? &a.multi[max(mi, 0)].w : &a.groups[group_index(slot, by - kGroupOf)];
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        left = mi >= 0 ? atomic_add_dev(count, -1) : 0;
    }
    const int bins_end = __builtin_amdgcn_readfirstlane(s_task[kKinds]);
    int kind = 1;
    // the lane's row in task t of a bin (-1: none); the kind only moves forward
    auto fetch = [&](int at) -> int {
        int r = -1;
        if (at < bins_end) {
            while (__builtin_amdgcn_readfirstlane(s_task[kind + 1]) <= at) ++kind;
            const int k = at - __builtin_amdgcn_readfirstlane(s_task[kind]);
            const int i = k * (kWave >> (kind - 1)) + (lane >> (kind - 1));
            if (i < s_cnt[kind]) r = a.rows_buf[bin_entry(a, kind - 1, i)];
        }
        return r;
    };
    int row = fetch(t);
    for (; t < bins_end; t += nw) {
        const int g = 1 << (kind - 1), sub = lane & (g - 1), dst = row;
        const int first = dst >= 0 ? a.row_ptr[dst] : 0, end = dst >= 0 ? a.row_ptr[dst + 1] : 0;
        row = fetch(t + nw);
        const float s = group_sum(dot_strided_u<2 * kUnroll>(a, first + sub, g, end, s_x.x, nlds), g);
        if (dst >= 0 && sub == 0) a.y[dst] = s;
    }
    if constexpr (LIGHT) {
        for (; t < total; t += nw) {
            const long long r = (long long)(t - bins_end) * kWave + lane;
            const int beg = r < a.n ? a.row_ptr[r] : 0, end = r < a.n ? a.row_ptr[r + 1] : 0;
            if (r < a.n && end - beg <= a.threshold) a.y[r] = light_row(a, beg, end);
        }
    }
    combine_rows(a, mi, by, left);
}

// ---- small products -----------------------------------------------------------------------------

// A whole product of grid mode in one launch, for matrices whose buffers a
// workgroup's LDS holds: a workgroup takes 8 rows, its first wave bins them,
// and its waves take the same tasks as the grid-wide child (lane groups per
// row, chunks of the split rows with their partials in LDS, the light rows one
// lane each), so every sum has the order of the general path.  A workgroup's
// rows lie a grid apart (hubs often have neighbouring ids).  Rule (small_product):
// up to kSmallNnz entries, for 8 rows fill the lane groups of seven bins worse
// than all rows of the matrix do.  R-MAT, 16 entries a row, this kernel / the
// general path: 4,096 rows 9.6 / 16.6 us (23.5 before), 16,384 rows (2^18 entries)
// 13.1 / 16.6, 32,768 rows 20.0 / 17.3, 131,072 rows 77 / 26.  Up to kSmallN rows,
// for the workgroups are as many as the rows ask, filled or not: 2^18 entries in
// 32,768 rows 12.4 / 13.4 us, in 40,000 14.0 / 13.8, in 2^20 233 / 13.  And a row
// is one workgroup's, a third of a us per thousand entries beyond the first ten
// thousand: a row of a matrix that has an entry once is no longer than n, so a
// matrix of more than n^2 entries is only taken while one row could hold them all
// (64 rows, all entries in one: 2^15 17 / 13 us, 2^16 31 / 13, 2^18 116 / 21).
// Bound by launch and memory latency.
constexpr int kSmallBlock = 512;
constexpr int kSmallRows = 8;
constexpr int kSmallNnz = 1 << 18;
constexpr int kSmallN = 1 << 15;
bool small_product(long long n, long long m)
{
    return n <= kSmallN && m <= kSmallNnz && m <= std::max<long long>(kSmallN, n * n);
}
constexpr int kSmallChunk = 512;  // smallest chunk it is used with
__global__ __launch_bounds__(kSmallBlock) void spmv_small(SpmvArgs a)
{
    constexpr int NW = kSmallBlock / kWave;
    __shared__ int s_row[kWave], s_beg[kWave], s_end[kWave];     // heavy rows by bin, then split rows
    __shared__ int s_first[kWave], s_cnt[kBins + 2], s_off[kBins + 1], s_task[kBins + 3];
    __shared__ float s_part[kSmallNnz / kSmallChunk + kWave];  // each row may end with a partly filled chunk
    const int lane = lane_id(), wid = threadIdx.x / kWave;
    const int row = lane < kSmallRows ? (int)(blockIdx.x + (long long)lane * gridDim.x) : a.n;
    int beg = 0, end = 0;
    if (row < a.n) {
        beg = a.row_ptr[row];
        end = a.row_ptr[row + 1];
    }
    const int len = end - beg;
    const bool light = len <= a.threshold;
    if (wid == 0) {
        const int bin = light ? -1 : len > a.chunk ? kChunkBin : bin_of(len, a.ipl);
        int off = 0, task = 0;
        for (int b = 0; b <= kBins; ++b) {
            const uint64_t m = __ballot(bin == b);
            const int cnt = __popcll(m);
            const int nch = b == kChunkBin && bin == b ? (len + a.chunk - 1) / a.chunk : 0;
            const int incl = b == kChunkBin && m ? wave_incl_scan(nch) : 0;
            if (bin == b) {
                const int k = off + rank_in(m);
                s_row[k] = row;
                s_beg[k] = beg;
                s_end[k] = end;
                if (b == kChunkBin) s_first[rank_in(m)] = incl - nch;
            }
            if (lane == 0) {
                s_cnt[b] = cnt;
                s_off[b] = off;
                s_task[b] = task;
            }
            off += cnt;
            task += b < kBins ? (cnt + (kWave >> b) - 1) / (kWave >> b) : readlane(incl, kWave - 1);
        }
        if (lane == 0) s_task[kBins + 1] = task;
    }
    __syncthreads();
    const int total = s_task[kBins + 1];
    // the last wave sums the light rows first, the others begin with the tasks;
    // chunks, the longest tasks, come first
    if (wid == NW - 1 && row < a.n && light) a.y[row] = light_row(a, beg, end);
    for (int t = total - 1 - wid; t >= 0; t -= NW) {
        int b = kChunkBin;
        while (s_task[b] > t) --b;
        const bool chunk = b == kChunkBin;
        const int g = chunk ? kWave : 1 << b;
        const int sub = lane & (g - 1);
        int first = 0, stop = 0, k = 0;
        bool ok = true;
        if (chunk) {
            const int c = t - s_task[kChunkBin];
            int i = 0;
            while (i + 1 < s_cnt[kChunkBin] && s_first[i + 1] <= c) ++i;
            first = s_beg[s_off[kChunkBin] + i] + (c - s_first[i]) * a.chunk;
            stop = min(s_end[s_off[kChunkBin] + i], first + a.chunk);
            first += lane;
            k = c;
        } else {
            const int i = (t - s_task[b]) * (kWave >> b) + (lane >> b);
            ok = i < s_cnt[b];
            k = s_off[b] + (ok ? i : 0);
            if (ok) {
                first = s_beg[k] + sub;
                stop = s_end[k];
            }
        }
        float s = dot_strided_u<2 * kUnroll>(a, first, g, stop);
        s = group_sum(s, g);
        if (sub == 0) {
            if (chunk) s_part[k] = s;
            else if (ok) a.y[s_row[k]] = s;
        }
    }
    if (s_cnt[kChunkBin] == 0) return;  // uniform in the block
    __syncthreads();
    for (int i = wid; i < s_cnt[kChunkBin]; i += NW) {
        const int from = s_first[i];
        const int to = i + 1 < s_cnt[kChunkBin] ? s_first[i + 1] : total - s_task[kChunkBin];
        Cascade cs;
        for (int c = from + lane; c < to; c += kWave) cs.add(s_part[c]);
        const float s = wave_sum(cs.total());
        if (lane == 0) a.y[s_row[s_off[kChunkBin] + i]] = s;
    }
}

// basic dynamic parallelism, emulated for comparison (driver 2): the parent
// sums the light rows inline and lists the heavy ones; the host then launches
// one child per listed row (no consolidation).
constexpr int kBasicBlock = 256;
__global__ __launch_bounds__(kBasicBlock) void spmv_parent_basic(SpmvArgs a)
{
    for (int base = blockIdx.x * kBasicBlock; base < a.n; base += gridDim.x * kBasicBlock) {
        const int r = base + threadIdx.x;
        const bool valid = r < a.n;
        int beg = 0, end = 0;
        if (valid) {
            beg = a.row_ptr[r];
            end = a.row_ptr[r + 1];
        }
        const bool heavy = valid && end - beg > a.threshold;
        if (valid && !heavy) a.y[r] = dot_strided(a, beg, 1, end);
        const int s = wave_reserve(heavy, &a.bin_total[0]);
        if (heavy && s < a.rows_cap) a.basic[s] = make_int4(r, beg, end, 0);
    }
}

// The child of ONE heavy row: one workgroup strides over the row, then a
// fixed-order workgroup sum.
__global__ __launch_bounds__(kBasicBlock) void spmv_child_basic(SpmvArgs a, int r, int beg, int end)
{
    __shared__ float tmp[kBasicBlock / kWave];
    const float s = block_sum<kBasicBlock>(dot_strided(a, beg + (int)threadIdx.x, kBasicBlock, end), tmp);
    if (threadIdx.x == 0) a.y[r] = s;
}

__global__ void spmv_basic_reset(SpmvArgs a)
{
    if (threadIdx.x == 0) a.bin_total[0] = 0;
}

// x_hot[k] = x[hot_ids[k]] for the hot-column layout (once per product).
__global__ __launch_bounds__(256) void spmv_gather_hot(SpmvArgs a)
{
    float *xh = const_cast<float *>(a.x_hot);
    for (int k = blockIdx.x * 256 + threadIdx.x; k < a.hot; k += gridDim.x * 256) xh[k] = a.x[a.hot_ids[k]];
}

struct SpmvKernels {
    const void *parent, *drain, *drain_light;
};

template <int BLOCK>
SpmvKernels pick_block(wc_mode mode, bool hot, bool stats)
{
    SpmvKernels k{nullptr,
                  hot ? reinterpret_cast<const void *>(&spmv_drain<BLOCK, true, false>)
                      : reinterpret_cast<const void *>(&spmv_drain<BLOCK, false, false>),
                  reinterpret_cast<const void *>(&spmv_drain<BLOCK, false, true>)};
    switch (mode) {
    case WC_FLAT: k.parent = reinterpret_cast<const void *>(&spmv_parent<WC_FLAT, BLOCK>); break;
    case WC_WAVE: k.parent = reinterpret_cast<const void *>(&spmv_parent<WC_WAVE, BLOCK>); break;
    case WC_BLOCK: k.parent = reinterpret_cast<const void *>(&spmv_parent<WC_BLOCK, BLOCK>); break;
    default:
        k.parent = stats ? reinterpret_cast<const void *>(&spmv_parent_grid<BLOCK, true>)
                         : reinterpret_cast<const void *>(&spmv_parent_grid<BLOCK, false>);
        break;
    }
    return k;
}

SpmvKernels pick(wc_mode mode, int block, bool hot, bool stats)
{
    switch (block) {
    case 64: return pick_block<64>(mode, hot, stats);
    case 128: return pick_block<128>(mode, hot, stats);
    case 512: return pick_block<512>(mode, hot, stats);
    case 1024: return pick_block<1024>(mode, hot, stats);
    default: return pick_block<256>(mode, hot, stats);
    }
}


// A planned product y = A x: the tune resolved, the kernels picked and the
// workspace laid out (plus `extra_bytes` left for the caller after it).  x and
// y may be set after planning.
struct SpmvPlan {
    SpmvArgs a;
    SpmvKernels ks;
    Config cfg;
    wc_mode mode;
    int grid, dgrid;
    bool small;  // the whole product in one launch
    long long rows, basic, cap, mcap;  // entries of the buffers
};

// Resolves the tune and the launch shapes for a device with `num_cus` compute
// units; touches no memory.
wc_status spmv_shape(int num_cus, const wc_csr *g, const float *val, wc_mode mode, const wc_tune *tune,
                     bool want_stats, SpmvPlan *p, bool hot = false)
{
    int block = (tune && tune->block_threads > 0) ? tune->block_threads : 256;
    p->mode = mode;
    p->ks = pick(mode, block, hot, want_stats);
    int resident = resident_blocks_on(num_cus, p->ks.parent, block);
    wc_status st = resolve_tune(nullptr, "spmv", mode, tune, resident, &p->cfg);
    if (st != WC_OK) return st;
    const Config &cfg = p->cfg;
    if (cfg.block != block) {
        p->ks = pick(mode, cfg.block, hot, want_stats);
        resident = resident_blocks_on(num_cus, p->ks.parent, cfg.block);
    }
    // the drain of the hot-column layout holds 64 KiB of LDS: its own residency
    if (hot) resident = std::min(resident, resident_blocks_on(num_cus, p->ks.drain, cfg.block));
    const long long n = g->n, m = g->m;
    const int chunk = kWave * cfg.items_per_lane;
    // wave and block modes hand rows longer than `spill` (one chunk) on as
    // chunks: at most m / spill such rows, each with at most one partly filled chunk
    const int spill = chunk;
    long long cap_full = n + m / chunk + 1, multi_full = n;
    if (mode == WC_WAVE || mode == WC_BLOCK) {
        cap_full = m / chunk + m / spill + 1;
        multi_full = m / spill + 1;
    }
    p->cap = mode != WC_FLAT ? (cfg.buf_capacity > 0 ? std::min(cfg.buf_capacity, cap_full) : cap_full) : 1;
    p->mcap = mode != WC_FLAT ? multi_full : 1;
    p->basic = cfg.driver == 2 ? n : 0;
    // A bin holds at most n rows and no more than m / (its shortest length);
    // bins 2k and 2k + 1 share a region, one from each end, since both together
    // hold at most n rows.
    p->rows = 0;
    long long bin_off[kBins + 1] = {};
    for (int b = 0; b < kBins && mode == WC_GRID; b += 2) {
        long long room = 0;
        for (int k = b; k < std::min(b + 2, kBins); ++k) {
            const long long shortest =
                std::max<long long>(cfg.threshold + 1LL, k ? (1LL << (k - 1)) * cfg.items_per_lane + 1 : 1);
            if (shortest <= ((long long)cfg.items_per_lane << k)) room += m / shortest;
        }
        room = std::min(n, room);
        bin_off[b] = p->rows;
        p->rows += room;
        bin_off[b + 1] = p->rows - 1;
    }
    // wave and block modes launch the parent with a thread per row (one window
    // per workgroup) unless grid_blocks caps it: the hardware hands windows to
    // CUs as they free up, which evens out the windows dense with buffered rows
    // (scale-22 graph: wave 0.92 -> 0.85 ms, block 0.93 -> 0.85 ms against the
    // resident grid)
    const long long windows = (n + cfg.block - 1) / cfg.block;
    const bool own_grid = tune && tune->grid_blocks > 0;
    p->grid = (int)std::max<long long>(1, (mode == WC_WAVE || mode == WC_BLOCK) && !own_grid
                                              ? windows
                                              : std::min<long long>(cfg.grid, windows));
    p->dgrid = std::max(1, std::min(cfg.grid, resident));
    SpmvArgs &a = p->a;
    std::memset(&a, 0, sizeof(a));
    if (mode == WC_GRID) {
        // steps of more windows once there is one for each of 1024 blocks (four a CU)
        a.windows = (int)std::min<long long>(kWindows, std::max<long long>(1, windows / 1024));
        p->grid = (int)std::min<long long>(p->grid, (windows + a.windows - 1) / a.windows);
    }
    a.row_ptr = g->row_ptr;
    a.col = g->col;
    a.val = val;
    a.n = (int)n;
    a.threshold = cfg.threshold;
    a.ipl = cfg.items_per_lane;
    a.chunk = chunk;
    a.spill = spill;
    a.count_drain = mode == WC_GRID;
    std::copy(bin_off, bin_off + kBins + 1, a.bin_off);
    a.rows_cap = p->basic;
    a.chunk_cap = p->cap;
    a.multi_cap = p->mcap;
    a.want_stats = want_stats;
    // one launch for a small matrix, where the launch shape, the threshold and
    // the buffers are the library's choice and nothing is counted
    p->small = mode == WC_GRID && !hot && !want_stats && !cfg.own_shape && !(tune && tune->threshold > 0) &&
               cfg.buf_capacity <= 0 && cfg.driver == 0 && small_product(n, m) && chunk >= kSmallChunk;
    return WC_OK;
}

// Counts of groups of chunks.
long long spmv_groups(const SpmvPlan *p)
{
    return p->mode == WC_FLAT ? 0 : (p->cap + kGroup - 1) / kGroup * kGroupPad;
}

// Bytes of workspace the planned product needs (256-byte aligned pieces).
size_t spmv_workspace_bytes(const SpmvPlan *p)
{
    return padded(kCols * kPad * 4) + padded(p->rows * 4) + padded(p->basic * 16) + padded(p->cap * 16) + padded(p->cap * 4) +
           padded(p->mcap * 16) + padded(spmv_groups(p) * 4);
}

// Lays the workspace out from `base` (256-byte aligned, spmv_workspace_bytes
// long); returns the first byte after it.
char *spmv_carve(SpmvPlan *p, char *base)
{
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *q = base + off;
        off += padded(bytes);
        return q;
    };
    SpmvArgs &a = p->a;
    a.bin_total = reinterpret_cast<int *>(take(kCols * kPad * 4));
    a.rows_buf = reinterpret_cast<int *>(take(p->rows * 4));
    a.basic = reinterpret_cast<int4 *>(take(p->basic * 16));
    a.chunks = reinterpret_cast<int4 *>(take(p->cap * 16));
    a.partials = reinterpret_cast<float *>(take(p->cap * 4));
    a.multi = reinterpret_cast<int4 *>(take(p->mcap * 16));
    a.groups = reinterpret_cast<int *>(take(spmv_groups(p) * 4));
    return base + off;
}

wc_status spmv_plan(wc_ctx *ctx, const wc_csr *g, const float *val, wc_mode mode, const wc_tune *tune,
                    size_t extra_bytes, hipStream_t stream, wc_stats *stats, SpmvPlan *p, bool hot = false)
{
    wc_status st = spmv_shape(ctx->num_cus, g, val, mode, tune, stats != nullptr, p, hot);
    if (st != WC_OK) return st;
    st = pool_reserve(ctx, spmv_workspace_bytes(p) + extra_bytes, stream);
    if (st != WC_OK) return st;
    char *end = spmv_carve(p, ctx->pool);
    ctx->pool_off = (size_t)(end - ctx->pool);
    p->a.stats = ctx->dstats;
    return WC_OK;
}

// Call bracket of the products: the device counters are cleared where something
// reads them, work counters or the overflow flag (a launch less otherwise).
wc_status begin_product(wc_ctx *ctx, const SpmvPlan &p, hipStream_t stream, wc_stats *stats)
{
    if (stats || p.cfg.fail_on_overflow) return begin_call(ctx, stream, stats);
    chain_break(ctx);
    return WC_OK;
}

// The kernels of one product: the parent, which fills the buffers, and the
// grid-wide drain of what it put there (flat mode: the parent alone; a small
// matrix: one kernel).
wc_status spmv_launch(wc_ctx *ctx, SpmvPlan *p, hipStream_t stream)
{
    const Config &cfg = p->cfg;
    void *args[] = {&p->a};
    if (p->small)
        return launch(ctx, "spmv_small", reinterpret_cast<const void *>(&spmv_small),
                      dim3((unsigned)((p->a.n + kSmallRows - 1LL) / kSmallRows)), dim3(kSmallBlock), args, stream);
    if (p->mode == WC_FLAT)
        return launch(ctx, "spmv_parent_flat", p->ks.parent, dim3(p->grid), dim3(cfg.block), args, stream);
    static const char *const names[] = {"", "spmv_parent_wave", "spmv_parent_block", "spmv_parent_grid"};
    wc_status st = launch(ctx, "spmv_reset", reinterpret_cast<const void *>(&spmv_reset), dim3(1), dim3(kWave), args,
                          stream);
    if (st == WC_OK) st = launch(ctx, names[p->mode], p->ks.parent, dim3(p->grid), dim3(cfg.block), args, stream);
    if (st == WC_OK) st = launch(ctx, "spmv_drain", p->ks.drain, dim3(p->dgrid), dim3(cfg.block), args, stream);
    return st;
}

// Grid mode, again on the same matrix with the buffers of the last spmv_launch
// of this plan still in place (full-size buffers, so nothing overflowed): the
// drain with the light rows.  Same sums, in the same order, as spmv_launch.
wc_status spmv_relaunch(wc_ctx *ctx, SpmvPlan *p, hipStream_t stream)
{
    if (p->small) return spmv_launch(ctx, p, stream);
    void *args[] = {&p->a};
    return launch(ctx, "spmv_drain", p->ks.drain_light, dim3(p->dgrid), dim3(p->cfg.block), args, stream);
}

// ---------------------------------------------------------------- PageRank

struct PrArgs {
    const int *out_degree;
    float *rank;
    float *contrib;   // rank[u] / outdeg(u), the x of the in-edge sums
    const float *sums;  // sum over the in-edges of v of contrib[u]
    const float *dpart;  // per block: rank held by vertices without out-edges, of this sweep
    float *dpart_next;   // ... of the next one
    int last;            // no sweep follows
    int nparts;
    int n;
    float base;       // (1 - d) / n
    float damping;
    float inv_n;
};

constexpr int kPrBlock = 256;

// What vertex u hands to each out-neighbour; the rank of vertices without
// out-edges goes into dang instead.
__device__ __forceinline__ float pr_give(const PrArgs &p, int u, float r, Cascade &dang)
{
    const int od = p.out_degree[u];
    dang.add(od == 0 ? r : 0.f);
    return od > 0 ? r / (float)od : 0.f;
}

// Before the first sweep: rank 1/n everywhere, its contributions and, in a
// fixed order, the rank held by each block's vertices without out-edges.
__global__ __launch_bounds__(kPrBlock) void pr_first(PrArgs p)
{
    __shared__ float red[kPrBlock / kWave];
    Cascade dang;
    for (int u = blockIdx.x * kPrBlock + threadIdx.x; u < p.n; u += gridDim.x * kPrBlock) {
        if (p.last) p.rank[u] = p.inv_n;  // no sweep follows
        else p.contrib[u] = pr_give(p, u, p.inv_n, dang);
    }
    const float held = block_sum<kPrBlock>(dang.total(), red);
    if (threadIdx.x == 0) p.dpart_next[blockIdx.x] = held;
}

// The end of a sweep and the start of the next: rank'[v] = (1 - d) / n + d *
// (sums[v] + D / n), D the sum of dpart in block order (every block computes the
// same D), and rank's contributions to the next sweep; after the last sweep the
// rank itself.  The rank of an inner sweep stays in a register.
__global__ __launch_bounds__(kPrBlock) void pr_step(PrArgs p)
{
    __shared__ float red[kPrBlock / kWave];
    Cascade part;
    for (int i = threadIdx.x; i < p.nparts; i += kPrBlock) part.add(p.dpart[i]);
    const float dsum = block_sum<kPrBlock>(part.total(), red);
    const float spread = dsum * p.inv_n;
    Cascade dang;
    for (int v = blockIdx.x * kPrBlock + threadIdx.x; v < p.n; v += gridDim.x * kPrBlock) {
        const float r = p.base + p.damping * (p.sums[v] + spread);
        if (p.last) p.rank[v] = r;
        else p.contrib[v] = pr_give(p, v, r, dang);
    }
    if (p.last) return;
    const float held = block_sum<kPrBlock>(dang.total(), red);
    if (threadIdx.x == 0) p.dpart_next[blockIdx.x] = held;
}

}  // namespace
}  // namespace wc

using namespace wc;

extern "C" wc_status wc_spmv(wc_ctx *ctx, const wc_csr *g, const float *val, const float *x, float *y, wc_mode mode,
                             const wc_tune *tune, hipStream_t stream, wc_stats *stats)
{
    if (!ctx || !g) return fail(WC_EINVAL, "wc_spmv: NULL context or matrix");
    if (mode < WC_FLAT || mode > WC_GRID) return fail(WC_EINVAL, "wc_spmv: bad mode");
    if (g->n < 0 || g->m < 0) return fail(WC_EINVAL, "wc_spmv: negative size");
    if (g->n == 0) {
        if (stats) std::memset(stats, 0, sizeof(*stats));
        return WC_OK;
    }
    if (!g->row_ptr || !x || !y || (g->m > 0 && (!g->col || !val))) return fail(WC_EINVAL, "wc_spmv: NULL array");
    WC_HIP(hipSetDevice(ctx->device));
    SpmvPlan p;
    wc_status st = spmv_plan(ctx, g, val, mode, tune, 0, stream, stats, &p);
    if (st != WC_OK) return st;
    p.a.x = x;
    p.a.y = y;
    if (p.cfg.driver == 1 || p.cfg.driver == 3 || (p.cfg.driver == 2 && mode != WC_GRID))
        return fail(WC_EINVAL, "wc_spmv: driver 2 needs grid mode; drivers 1 and 3 do not apply");
    st = begin_product(ctx, p, stream, stats);
    if (st != WC_OK) return st;
    if (p.cfg.driver == 2) {
        // Basic dynamic parallelism, emulated: the host reads the heavy rows back
        // and launches one child per row.
        void *args[] = {&p.a};
        st = launch(ctx, "spmv_basic_reset", reinterpret_cast<const void *>(&spmv_basic_reset), dim3(1), dim3(64),
                    args, stream);
        const int bgrid = (int)std::min<long long>((g->n + kBasicBlock - 1) / kBasicBlock, 4LL * ctx->num_cus);
        if (st == WC_OK)
            st = launch(ctx, "spmv_parent_basic", reinterpret_cast<const void *>(&spmv_parent_basic), dim3(bgrid),
                        dim3(kBasicBlock), args, stream);
        if (st != WC_OK) return st;
        int tail = 0;
        WC_HIP(hipMemcpyAsync(&tail, p.a.bin_total, sizeof(int), hipMemcpyDeviceToHost, stream));
        WC_HIP(hipStreamSynchronize(stream));
        const int count = (int)std::min<long long>(tail, p.a.rows_cap);
        std::vector<int4> rows((size_t)std::max(count, 1));
        if (count > 0) WC_HIP(hipMemcpy(rows.data(), p.a.basic, sizeof(int4) * (size_t)count, hipMemcpyDeviceToHost));
        chain_break(ctx);
        for (int i = 0; i < count; ++i) {
            int r = rows[i].x, beg = rows[i].y, end = rows[i].z;
            void *cargs[] = {&p.a, &r, &beg, &end};
            st = launch(ctx, "spmv_child_basic", reinterpret_cast<const void *>(&spmv_child_basic), dim3(1),
                        dim3(kBasicBlock), cargs, stream);
            if (st != WC_OK) return st;
        }
        st = end_call(ctx, stream, stats, 1, p.cfg.fail_on_overflow);
        if (stats) {
            stats->items_buffered = count;
            stats->dispatches = count;
        }
        return st;
    }
    st = spmv_launch(ctx, &p, stream);
    if (st != WC_OK) return st;
    return end_call(ctx, stream, stats, 1, p.cfg.fail_on_overflow);
}

extern "C" wc_status wc_pagerank(wc_ctx *ctx, const wc_csr *in_graph, const int32_t *out_degree, int32_t iterations,
                                 float damping, float *rank, wc_mode mode, const wc_tune *tune, hipStream_t stream,
                                 wc_stats *stats)
{
    if (!ctx || !in_graph) return fail(WC_EINVAL, "wc_pagerank: NULL context or graph");
    if (mode < WC_FLAT || mode > WC_GRID) return fail(WC_EINVAL, "wc_pagerank: bad mode");
    if (in_graph->n < 0 || in_graph->m < 0 || iterations < 0) return fail(WC_EINVAL, "wc_pagerank: negative size");
    if (!(damping >= 0.f && damping <= 1.f)) return fail(WC_EINVAL, "wc_pagerank: damping outside [0, 1]");
    if (in_graph->n == 0) {
        if (stats) std::memset(stats, 0, sizeof(*stats));
        return WC_OK;
    }
    if (!in_graph->row_ptr || !out_degree || !rank || (in_graph->m > 0 && !in_graph->col))
        return fail(WC_EINVAL, "wc_pagerank: NULL array");
    WC_HIP(hipSetDevice(ctx->device));
    const long long n = in_graph->n;
    const int pgrid = (int)std::min<long long>((n + kPrBlock - 1) / kPrBlock, 4 * (long long)ctx->num_cus);
    SpmvPlan p;
    // the contributions and the sums begin at a multiple of 64 KiB wherever the
    // workspace ends: at 256 bytes a sweep of 2^22 vertices took 423 or 441 us, one of
    // 2^20 82 or 86, by the place (421 and 83 so)
    constexpr size_t kPlace = size_t(1) << 16;
    const auto place = [&](size_t off) { return (off + kPlace - 1) / kPlace * kPlace; };
    wc_status st = spmv_plan(ctx, in_graph, nullptr, mode, tune,
                             2 * padded(n * 4) + 2 * padded((size_t)pgrid * 4) + 2 * kPlace, stream, stats, &p);
    if (st != WC_OK) return st;
    if (p.cfg.driver != 0) return fail(WC_EINVAL, "wc_pagerank: only the relaunch driver (driver = 0) applies");
    // A later sweep of the general path is one launch too (spmv_relaunch), so the
    // one-launch product, which bins its rows every time, pays in the first sweeps, the
    // more of them the fewer its workgroups.  R-MAT, one-launch / general in us: 16,384
    // vertices of 12 edges 2 sweeps 28.9 / 28.2, 3 sweeps 42 / 37; 10,547 of 9, 4 sweeps
    // 44 / 44, 5 sweeps 54 / 53; 4,096 of 16, 3 sweeps 34 / 35, 10 sweeps 104 / 92 (of 8
    // edges 85 / 94); uniform, 16,384 of 4, 2 sweeps 23 / 28, 5 sweeps 51 / 49; four
    // rows of 30,000 entries, 5 sweeps 130 / 62.
    p.small = p.small && n * iterations <= 3 << 14;
    PrArgs q;
    q.out_degree = out_degree;
    q.rank = rank;
    ctx->pool_off = place(ctx->pool_off);
    q.contrib = pool_take<float>(ctx, n);
    ctx->pool_off = place(ctx->pool_off);
    float *sums = pool_take<float>(ctx, n);
    q.sums = sums;
    float *dpart[2] = {pool_take<float>(ctx, pgrid), pool_take<float>(ctx, pgrid)};
    q.dpart = nullptr;
    q.dpart_next = dpart[0];
    q.last = iterations == 0;
    q.nparts = pgrid;
    q.n = (int)n;
    q.base = (float)((1.0 - (double)damping) / (double)n);
    q.damping = damping;
    q.inv_n = (float)(1.0 / (double)n);
    p.a.x = q.contrib;
    p.a.y = sums;
    st = begin_product(ctx, p, stream, stats);
    if (st != WC_OK) return st;
    void *args[] = {&q};
    st = launch(ctx, "pr_first", reinterpret_cast<const void *>(&pr_first), dim3(pgrid), dim3(kPrBlock), args, stream);
    // grid mode: the in-edge structure is the same every sweep, so the binned
    // rows and chunks of the first sweep serve the later ones (only when the
    // buffers are full size, so that nothing overflowed, and without work
    // counters, which count each sweep's binning)
    const bool reuse = mode == WC_GRID && !stats && !(tune && tune->buf_capacity > 0);
    for (int it = 0; it < iterations && st == WC_OK; ++it) {
        st = reuse && it > 0 ? spmv_relaunch(ctx, &p, stream) : spmv_launch(ctx, &p, stream);
        q.dpart = dpart[it & 1];
        q.dpart_next = dpart[(it + 1) & 1];
        q.last = it + 1 == iterations;
        if (st == WC_OK)
            st = launch(ctx, "pr_step", reinterpret_cast<const void *>(&pr_step), dim3(pgrid), dim3(kPrBlock), args,
                        stream);
    }
    if (st != WC_OK) return st;
    return end_call(ctx, stream, stats, iterations, p.cfg.fail_on_overflow);
}

// ---------------------------------------------------------------- hot-column layout

namespace wc {
namespace {

__global__ __launch_bounds__(256) void hot_count(const int *col, long long m, int *cnt)
{
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < m; e += (long long)gridDim.x * 256)
        atomicAdd(&cnt[col[e]], 1);
}

__global__ __launch_bounds__(256) void hot_remap(const int *col, long long m, const int *rank, int hot, int *out)
{
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < m; e += (long long)gridDim.x * 256) {
        const int c = col[e];
        const int r = rank[c];
        out[e] = r >= 0 ? r : hot + c;
    }
}

}  // namespace
}  // namespace wc

extern "C" wc_status wc_spmv_prepare(wc_ctx *ctx, const wc_csr *a, int32_t hot, int32_t *col_hot, int32_t *hot_ids,
                                     hipStream_t stream)
{
    if (!ctx || !a) return fail(WC_EINVAL, "wc_spmv_prepare: NULL context or matrix");
    if (a->n < 0 || a->m < 0) return fail(WC_EINVAL, "wc_spmv_prepare: negative size");
    if (hot < 0 || hot > a->n) return fail(WC_EINVAL, "wc_spmv_prepare: hot must be in [0, n]");
    if ((long long)a->n + hot > 0x7fffffffLL) return fail(WC_EINVAL, "wc_spmv_prepare: n + hot exceeds int32");
    if (a->n == 0) return WC_OK;
    if (!a->row_ptr || (a->m > 0 && (!a->col || !col_hot)) || (hot > 0 && !hot_ids))
        return fail(WC_EINVAL, "wc_spmv_prepare: NULL array");
    WC_HIP(hipSetDevice(ctx->device));
    const long long n = a->n, m = a->m;
    wc_status st = pool_reserve(ctx, 2 * padded(n * 4), stream);
    if (st != WC_OK) return st;
    int *cnt = pool_take<int>(ctx, n);
    int *rank = pool_take<int>(ctx, n);
    const int grid = (int)std::max<long long>(1, std::min<long long>((m + 255) / 256, 8LL * ctx->num_cus));
    chain_break(ctx);
    WC_HIP(hipMemsetAsync(cnt, 0, sizeof(int) * (size_t)n, stream));
    if (m > 0) {
        void *args[] = {const_cast<int **>(&a->col), const_cast<long long *>(&m), &cnt};
        st = launch(ctx, "hot_count", reinterpret_cast<const void *>(&hot_count), dim3(grid), dim3(256), args, stream);
        if (st != WC_OK) return st;
    }
    // the hot columns: most entries first, ties by column id
    std::vector<int> counts((size_t)n), order((size_t)n), rk((size_t)n, -1);
    WC_HIP(hipMemcpyAsync(counts.data(), cnt, sizeof(int) * (size_t)n, hipMemcpyDeviceToHost, stream));
    WC_HIP(hipStreamSynchronize(stream));
    for (long long v = 0; v < n; ++v) order[(size_t)v] = (int)v;
    auto more = [&](int u, int v) { return counts[u] != counts[v] ? counts[u] > counts[v] : u < v; };
    std::partial_sort(order.begin(), order.begin() + hot, order.end(), more);
    for (int k = 0; k < hot; ++k) rk[(size_t)order[(size_t)k]] = k;
    chain_break(ctx);
    WC_HIP(hipMemcpyAsync(rank, rk.data(), sizeof(int) * (size_t)n, hipMemcpyHostToDevice, stream));
    if (hot > 0) WC_HIP(hipMemcpyAsync(hot_ids, order.data(), sizeof(int) * (size_t)hot, hipMemcpyHostToDevice, stream));
    if (m > 0) {
        void *args[] = {const_cast<int **>(&a->col), const_cast<long long *>(&m), &rank, &hot, &col_hot};
        st = launch(ctx, "hot_remap", reinterpret_cast<const void *>(&hot_remap), dim3(grid), dim3(256), args, stream);
        if (st != WC_OK) return st;
    }
    // the host vectors above are read by the copies: wait for them
    WC_HIP(hipStreamSynchronize(stream));
    return WC_OK;
}

extern "C" wc_status wc_spmv_hot(wc_ctx *ctx, const wc_csr *a_hot, int32_t hot, const int32_t *hot_ids,
                                 const float *val, const float *x, float *y, wc_mode mode, const wc_tune *tune,
                                 hipStream_t stream, wc_stats *stats)
{
    if (!ctx || !a_hot) return fail(WC_EINVAL, "wc_spmv_hot: NULL context or matrix");
    if (mode < WC_FLAT || mode > WC_GRID) return fail(WC_EINVAL, "wc_spmv_hot: bad mode");
    if (a_hot->n < 0 || a_hot->m < 0) return fail(WC_EINVAL, "wc_spmv_hot: negative size");
    if (hot < 0 || hot > a_hot->n) return fail(WC_EINVAL, "wc_spmv_hot: hot must be in [0, n]");
    if (a_hot->n == 0) {
        if (stats) std::memset(stats, 0, sizeof(*stats));
        return WC_OK;
    }
    if (!a_hot->row_ptr || !x || !y || (a_hot->m > 0 && (!a_hot->col || !val)) || (hot > 0 && !hot_ids))
        return fail(WC_EINVAL, "wc_spmv_hot: NULL array");
    WC_HIP(hipSetDevice(ctx->device));
    SpmvPlan p;
    wc_status st = spmv_plan(ctx, a_hot, val, mode, tune, padded((size_t)std::max(hot, 1) * 4), stream, stats, &p,
                             hot > 0);
    if (st != WC_OK) return st;
    if (p.cfg.driver != 0) return fail(WC_EINVAL, "wc_spmv_hot: only the relaunch driver (driver = 0) applies");
    p.a.x = x;
    p.a.y = y;
    p.a.hot = hot;
    p.a.hot_ids = hot_ids;
    p.a.x_hot = pool_take<float>(ctx, (size_t)std::max(hot, 1));
    st = begin_product(ctx, p, stream, stats);
    if (st != WC_OK) return st;
    if (hot > 0) {
        void *args[] = {&p.a};
        const int g = (int)std::min<long long>((hot + 255) / 256, 4LL * ctx->num_cus);
        st = launch(ctx, "spmv_gather_hot", reinterpret_cast<const void *>(&spmv_gather_hot), dim3(g), dim3(256), args,
                    stream);
        if (st != WC_OK) return st;
    }
    st = spmv_launch(ctx, &p, stream);
    if (st != WC_OK) return st;
    return end_call(ctx, stream, stats, 1, p.cfg.fail_on_overflow);
}

// ---------------------------------------------------------------- SpMV without allocation
//
// wc_spmv_noalloc: the kernels of wc_spmv with their workspace in a fixed
// device array instead of a context pool.  `scratch` is a host-side stand-in
// for that array: host code only ever uses the device address that
// hipGetSymbolAddress returns for it, taken once per device on the first call
// made with that device current.

// The documented bytes, which decide what is refused, and room for the counters
// (spmv_noalloc_bound).
constexpr size_t kNoAllocScratch = (size_t)WC_SPMV_NOALLOC_SCRATCH_BYTES + (2u << 20);
static __device__ __align__(256) unsigned char scratch[kNoAllocScratch];

namespace wc {
namespace {

constexpr int kMaxDevices = 64;
struct NoAllocDevice {
    bool ready = false;
    int num_cus = 0;
    char *scratch = nullptr;  // device address of `scratch` on this device
};
std::mutex g_noalloc_mu;
NoAllocDevice g_noalloc[kMaxDevices];

// Workspace bound from n, m and the tune alone (the documented one), so oversized
// calls are refused before any HIP call is made.  Rows, chunks and split rows as
// they are documented: in grid mode 16 bytes a row for the bins, which hold row
// ids in four regions of up to n now, and 72 bytes a block.  The counters, each
// on a line of its own, are not in it: the array has room for them beside it.
size_t spmv_noalloc_bound(const wc_csr *g, const SpmvPlan *p)
{
    const size_t n = (size_t)g->n, blocks = p->mode == WC_GRID ? (n + p->cfg.block - 1) / p->cfg.block : 1;
    return 2 * padded(blocks * 36) + padded(36) + padded((p->mode == WC_GRID ? n : 1) * 16) + padded(p->cap * 16) +
           padded(p->cap * 4) + padded(p->mcap * 16) + padded(sizeof(DevStats));
}

}  // namespace
}  // namespace wc

extern "C" wc_status wc_spmv_noalloc(const wc_csr *g, const float *val, const float *x, float *y, wc_mode mode,
                                     const wc_tune *tune, hipStream_t stream)
{
    if (!g) return fail(WC_EINVAL, "wc_spmv_noalloc: NULL matrix");
    if (mode < WC_FLAT || mode > WC_GRID) return fail(WC_EINVAL, "wc_spmv_noalloc: bad mode");
    if (g->n < 0 || g->m < 0) return fail(WC_EINVAL, "wc_spmv_noalloc: negative size");
    if (g->n == 0) return WC_OK;
    if (!g->row_ptr || !x || !y || (g->m > 0 && (!g->col || !val)))
        return fail(WC_EINVAL, "wc_spmv_noalloc: NULL array");
    if (tune && tune->driver != 0)
        return fail(WC_EINVAL, "wc_spmv_noalloc: only the relaunch driver (driver = 0) applies");
    // the tune and the size limit are checked before any device memory is
    // touched; the compute-unit count only changes the drain grid, not the bound
    SpmvPlan p;
    wc_status st = spmv_shape(1, g, val, mode, tune, false, &p);
    if (st != WC_OK) return st;
    const size_t bound = spmv_noalloc_bound(g, &p);
    if (bound > (size_t)WC_SPMV_NOALLOC_SCRATCH_BYTES ||
        spmv_workspace_bytes(&p) + padded(sizeof(DevStats)) > kNoAllocScratch)  // (the second never without the first)
        return fail(WC_EINVAL, "wc_spmv_noalloc: the workspace (" + std::to_string(bound) +
                                   " bytes) exceeds the fixed scratch of " +
                                   std::to_string((size_t)WC_SPMV_NOALLOC_SCRATCH_BYTES) + " bytes");
    int dev = 0;
    WC_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(WC_EINVAL, "wc_spmv_noalloc: device index out of range");
    NoAllocDevice d;
    {
        std::lock_guard<std::mutex> lock(g_noalloc_mu);
        NoAllocDevice &slot = g_noalloc[dev];
        if (!slot.ready) {
            int cus = 0;
            WC_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
            void *ptr = nullptr;
            WC_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
            if (!ptr) return fail(WC_EHIP, "wc_spmv_noalloc: no device address for the scratch array");
            slot.num_cus = cus;
            slot.scratch = static_cast<char *>(ptr);
            slot.ready = true;
        }
        d = slot;
    }
    st = spmv_shape(d.num_cus, g, val, mode, tune, false, &p);
    if (st != WC_OK) return st;
    char *end = spmv_carve(&p, d.scratch);
    p.a.stats = reinterpret_cast<DevStats *>(end);  // written only on overflow, which a full-size buffer never has
    p.a.x = x;
    p.a.y = y;
    st = spmv_launch(nullptr, &p, stream);
    if (st != WC_OK) return st;
    WC_HIP(hipGetLastError());
    return WC_OK;
}
