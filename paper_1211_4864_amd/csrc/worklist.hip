// Work list for the pair kernels.  One item is one wave's worth of target
// particles from one unit: a run of cells (a single chaining cell, or an
// aligned pair of cells along z that holds at most 64 targets; the run rule
// is in run_of) or an RCB leaf.  Its sources are the unit's 3 x 3 x (zlen + 2)
// stencil cells.  A unit of c targets with item size T yields floor(c / T)
// items of T targets and at most two items for the remainder r = c mod T: the
// largest power of two p <= r, and r - p.  An item of t targets runs with
// k = floor_pow2(64 / t) lanes per target, each lane taking every k-th source,
// so a power-of-two item keeps all 64 lanes busy whatever its size.
//
// Item size.  T is 64 where the chip has many items, and is halved until the
// item's source steps (window / lanes per target) are at most the step limit
// of item_limit: the longest item, one wave walking its window alone, must not
// outlast the rest of the launch.  Short problems are bound by exactly that
// wave (65536 NFW particles: force 417 -> 184 us, VJP 557 -> 259 us; 343000:
// force 718 -> 537 us, VJP 1012 -> 790 us).
//
// Order of the items.  The chip has 8 XCDs, each with its own L2, and a
// kernel's workgroup k runs on XCD k mod 8.  The cells are split into 8
// spatially contiguous ranges of equal cost (columns of cells in key order),
// one per XCD, and XCD x receives the items of its range at workgroups
// x, x + 8, x + 16, ..., in decreasing cost so that the longest items start
// first.  The items of a dense cell and of its neighbours then share one L2,
// which holds their common source window.  Items beyond the shortest XCD
// list follow at the end in plain decreasing cost.  A set small enough for
// every L2 (kOneListParticles) takes one list in decreasing cost.
//
// Launches: the control words' clearing; units' windows and cost; the columns'
// XCDs (8 lists only); the histogram of the items over (list, cost) buckets; the
// items themselves, each block expanding its units' items in parallel straight
// into their final slots.  Five with 8 lists, four with one (RCB leaves of small
// sets); after a counting sort only the last is left, the others run beside the
// sort's kernels and in its clearing.  Latency-bound integer passes over the
// cells; twelve launches before (three fills, a scan in three, a separate
// item array and a one-thread bucket scan among them: 1003 particles 47 -> 16 us
// without the sharing).
//
// This replaces the tree walk that gathers leaf interaction lists in the
// paper's BG/Q code (Habib et al. 2012, Sec. III, walk minimisation and the
// paragraph on neighbour lists after Eq. 7).
#include <algorithm>

#include "worklist.h"

namespace hsr {

namespace {

constexpr int kBlock = kWorkBlock;
constexpr int kXcd = kXcds;

__global__ __launch_bounds__(kBlock) void k_windows(
    const int* __restrict__ cs, Geom g, int* __restrict__ cell_window,
    unsigned long long* __restrict__ col_cost, WorkControl* __restrict__ ctl) {
    windows_block(cs, g, cell_window, col_cost, ctl, blockIdx.x, gridDim.x);
}

// XCD of each column of cells: the columns in key order are cut into kXcd
// ranges of equal total work.  One block; the columns are split into
// contiguous chunks per thread.
__global__ __launch_bounds__(1024) void k_column_xcd(
    const unsigned long long* __restrict__ col_cost, int ncol,
    int* __restrict__ col_xcd) {
    __shared__ unsigned long long part[1024];
    const int t = threadIdx.x;
    const int per = (ncol + 1023) / 1024;
    const int a = min(ncol, t * per), b = min(ncol, a + per);
    unsigned long long sum = 0;
    for (int q = a; q < b; ++q) sum += col_cost[q];
    part[t] = sum;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {       // inclusive scan of the chunks
        const unsigned long long v = t >= d ? part[t - d] : 0ull;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    const unsigned long long total = part[1023];
    unsigned long long run = part[t] - sum;
    for (int q = a; q < b; ++q) {
        // the column goes to the XCD that holds the midpoint of its work
        const double mid = (double)run + 0.5 * (double)col_cost[q];
        int x = total ? (int)(mid * kXcd / (double)total) : 0;
        col_xcd[q] = min(kXcd - 1, max(0, x));
        run += col_cost[q];
    }
}

template <typename Units>
__global__ __launch_bounds__(kBlock) void k_items_hist(
    Units units, const int* __restrict__ cell_window, const int* __restrict__ col_xcd,
    int N, WorkControl* __restrict__ ctl) {
    items_hist_block(units, cell_window, col_xcd, N, ctl, blockIdx.x);
}

// Inclusive scan over a block of one value per thread.
__device__ __forceinline__ int block_incl_scan(int v, int* part) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int o = __shfl_up(v, d);
        if (lane >= d) v += o;
    }
    if (lane == kWave - 1) part[w] = v;
    __syncthreads();
    for (int k = 0; k < w; ++k) v += part[k];
    __syncthreads();
    return v;
}

// Writes the items at their final slots.  Every block forms the layout of the
// lists from the histogram (rank of each bucket in its list, decreasing cost;
// list lengths), reserves a range of each bucket's ranks, and expands its
// units' items (per_block units) over its threads.
template <typename Units>
__global__ __launch_bounds__(kBlock) void k_items_write(
    Units units, int per_block, const int* __restrict__ cell_window,
    const int* __restrict__ col_xcd, int N, WorkControl* __restrict__ ctl, int max_items,
    WorkItem* __restrict__ out) {
    constexpr int kPer = kOrderBuckets / kBlock;          // buckets per thread
    constexpr int kGroup = kCostBuckets / kPer;           // threads per list
    static_assert(kGroup <= kWave && kWave % kGroup == 0, "a list's threads share a wave");
    __shared__ int off[kOrderBuckets];    // first rank of a bucket in its list
    __shared__ int h[kOrderBuckets];      // this block's items of a bucket
    __shared__ int len[kXcd], tail[kXcd];
    __shared__ int part[kBlock / kWave];
    __shared__ int ends[kBlock];          // items of the block's units 0..t
    __shared__ Unit su[kBlock];
    __shared__ int sT[kBlock];
    __shared__ int4 rank[kBlock];         // final list, ranks of the pieces
    const int t = threadIdx.x;
    // Thread t holds the kPer buckets of descending cost that follow those of
    // thread t - 1 of the same list: an exclusive scan gives their ranks.
    const int list = t / kGroup, first = t % kGroup * kPer;
    int cnt[kPer], sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        cnt[j] = ctl->count[list * kCostBuckets + kCostBuckets - 1 - (first + j)];
        sum += cnt[j];
    }
    int incl = sum;
#pragma unroll
    for (int d = 1; d < kGroup; d <<= 1) {
        const int o = __shfl_up(incl, d, kGroup);
        if (t % kGroup >= d) incl += o;
    }
    int acc = incl - sum;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int b = list * kCostBuckets + kCostBuckets - 1 - (first + j);
        off[b] = acc;
        h[b] = 0;
        acc += cnt[j];
    }
    if (t % kGroup == kGroup - 1) len[list] = acc;
    __syncthreads();
    const int lists = col_xcd ? kXcd : 1;
    int shortest = len[0];
    for (int x = 1; x < lists; ++x) shortest = min(shortest, len[x]);
    if (t < kXcd) {
        int before = 0;
        for (int x = 0; x < t; ++x) before += len[x] - shortest;
        tail[t] = before;
    }
    if (blockIdx.x == 0 && t == 0) {
        int all = 0;
        for (int x = 0; x < lists; ++x) all += len[x];
        ctl->n_items = min(all, max_items);
    }
    const Mine m = my_unit(units, t < per_block ? blockIdx.x * per_block + t : units.size(),
                           item_limit(ctl->pairs), cell_window, col_xcd, N);
    // ranks inside the block's share of each bucket (any order: items write
    // only their own targets, so results do not depend on it)
    int4 r = make_int4(0, 0, 0, 0);
    __syncthreads();
    if (m.s.full) r.y = atomicAdd(&h[m.bfull], m.s.full);
    if (m.s.p) r.z = atomicAdd(&h[m.bp], 1);
    if (m.s.q) r.w = atomicAdd(&h[m.bq], 1);
    __syncthreads();
    for (int q = t; q < kOrderBuckets; q += kBlock)
        if (h[q]) off[q] += atomicAdd(&ctl->taken[q], h[q]);
    __syncthreads();
    r.x = (m.s.full ? m.bfull : m.bp) / kCostBuckets;
    r.y += off[m.bfull];
    r.z += off[m.bp];
    r.w += off[m.bq];
    su[t] = m.u;
    sT[t] = m.s.T;
    rank[t] = r;
    ends[t] = block_incl_scan(m.s.items(), part);
    __syncthreads();
    const int n_mine = ends[kBlock - 1];
    for (int q = t; q < n_mine; q += kBlock) {
        int lo = 0, hi = kBlock - 1;                 // first unit with ends > q
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (ends[mid] > q) hi = mid;
            else lo = mid + 1;
        }
        const Unit u = su[lo];
        const Pieces s = pieces_of(u.count, sT[lo]);
        const int4 rk = rank[lo];
        int j = q - (lo ? ends[lo - 1] : 0);
        int o, targets, rr;
        if (j < s.full) {
            o = j * s.T;
            targets = s.T;
            rr = rk.y + j;
        } else if (j == s.full && s.p) {
            o = s.full * s.T;
            targets = s.p;
            rr = rk.z;
        } else {
            o = s.full * s.T + s.p;
            targets = s.q;
            rr = rk.w;
        }
        // rank rr of list rk.x: workgroup rr * lists + rk.x while every list
        // still has items, then the remaining items of each list in turn
        const int slot = rr < shortest ? rr * lists + rk.x
                                       : lists * shortest + tail[rk.x] + (rr - shortest);
        WorkItem it;
        it.i_begin = u.begin + o;
        it.key = u.key;
        it.cx = (short)(u.key / N / N);
        it.cy = (short)(u.key / N % N);
        it.i_count = (unsigned char)targets;
        it.ksplit = (unsigned char)lanes_per_target(targets);
        it.zlen = (unsigned char)u.zlen;
        it.pad = 0;
        if (slot < max_items) out[slot] = it;
    }
}

inline int blocks_for(int64_t n, int per) { return (int)((n + per - 1) / per); }

// Few units can still have many items each (32768 NFW particles in 1000 cells:
// 8000 items): such sets spread their units over eight times the blocks, which
// takes 10 us there instead of 20.
constexpr int kFewUnits = 1 << 15;

// started: the windows and the histogram of the items are there already.
template <typename Units>
hipError_t order_items(const Units& units, int n_units, const int* cell_start, Geom g,
                       bool one_list, bool started, int max_items, const WorkBuffers& b,
                       WorkItem* items, hipStream_t st) {
    const int ncol = g.N * g.N;
    const int nb = std::max(1, blocks_for(n_units, kBlock));
    const int* xcd = one_list ? nullptr : b.col_xcd;
    if (!started) {
        const hipError_t e = launch_fill_i32(reinterpret_cast<int*>(b.ctl), kControlInts, 0, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_windows, dim3(window_blocks(g.N)), dim3(kBlock), 0, st, cell_start,
                           g, b.cell_window, b.col_cost, b.ctl);
        if (!one_list)
            hipLaunchKernelGGL(k_column_xcd, dim3(1), dim3(1024), 0, st,
                               (const unsigned long long*)b.col_cost, ncol, b.col_xcd);
        hipLaunchKernelGGL(k_items_hist<Units>, dim3(nb), dim3(kBlock), 0, st, units,
                           (const int*)b.cell_window, xcd, g.N, b.ctl);
    }
    const int per = n_units <= kFewUnits ? kBlock / 8 : kBlock;
    hipLaunchKernelGGL(k_items_write<Units>, dim3(std::max(1, blocks_for(n_units, per))),
                       dim3(kBlock), 0, st, units, per, (const int*)b.cell_window, xcd, g.N, b.ctl, max_items, items);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_worklist(const int* cell_start, int n, Geom g, bool started,
                           int max_items, const WorkBuffers& b, WorkItem* items,
                           hipStream_t st) {
    return order_items(CellUnits{cell_start, g}, g.N * g.N * g.N, cell_start, g,
                       n <= kOneListParticles, started, max_items, b, items, st);
}

hipError_t launch_worklist_leaves(const int* cell_start, const int* leaf_start,
                                  const int* n_leaves_dev, int n_leaves,
                                  const int* keys_sorted, int n, Geom g, int max_items,
                                  const WorkBuffers& b, WorkItem* items, hipStream_t st) {
    return order_items(LeafUnits{leaf_start, keys_sorted, n_leaves_dev, g.sbits}, n_leaves,
                       cell_start, g, n <= kOneListParticles, false, max_items, b, items, st);
}

}  // namespace hsr
