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
// Launches: units' windows and cost; the columns' XCDs (8 lists only); the
// histogram of the items over (list, cost) buckets; the items themselves,
// each block expanding its units' items in parallel straight into their final
// slots.  Latency-bound integer passes over the cells; three launches replace
// nine (a scan, a separate item array and a one-thread bucket scan among
// them: 1003 particles 47 -> 16 us).
//
// This replaces the tree walk that gathers leaf interaction lists in the
// paper's BG/Q code (Habib et al. 2012, Sec. III, walk minimisation and the
// paragraph on neighbour lists after Eq. 7).
#include <algorithm>

#include "common.h"

namespace hsr {

namespace {

constexpr int kBlock = 256;
constexpr int kXcd = kXcds;
constexpr int kOrderBuckets = kXcd * kCostBuckets;

__device__ __forceinline__ int floor_pow2(int v) {
    return v <= 0 ? 0 : (1 << (31 - __clz(v)));
}

// Unit of targets that share one source window.
struct Unit {
    int begin;     // first sorted entry
    int count;     // targets; 0: no unit
    int key;       // first cell
    int zlen;      // cells along z
};

// Run of cells that cell c heads (count 0 if c heads none).  The cells of a
// column are grouped in aligned blocks of kZRun along z; a block whose cells
// hold at most kItemI targets in all is one run (its first cell is the
// head), otherwise each cell is a run of its own.  In a periodic box a run
// leaves at least two cells of the column outside it, so its window of
// zlen + 2 cells along z has no cell twice.
__device__ __forceinline__ Unit run_of(int c, const int* __restrict__ cs, const Geom& g) {
    const int N = g.N;
    const int cz = c % N;
    const int z0 = cz - cz % kZRun;
    int zl = min(kZRun, N - z0);
    if (g.periodic) zl = min(zl, N - 2);
    if (zl >= 2 && cz < z0 + zl) {
        const int first = c - (cz - z0);
        const int total = cs[first + zl] - cs[first];
        if (total <= kItemI) return Unit{cs[c], cz == z0 ? total : 0, c, zl};
    }
    return Unit{cs[c], cs[c + 1] - cs[c], c, 1};
}

struct CellUnits {
    const int* cs;
    Geom g;
    __device__ __forceinline__ int size() const { return g.N * g.N * g.N; }
    __device__ __forceinline__ Unit get(int c) const { return run_of(c, cs, g); }
};

// Leaf l of the RCB leaf table, inside one cell.
struct LeafUnits {
    const int* leaf_start;
    const int* keys_sorted;
    const int* n_leaves;
    int sbits;
    __device__ __forceinline__ int size() const { return *n_leaves; }
    __device__ __forceinline__ Unit get(int l) const {
        const int b = leaf_start[l];
        return Unit{b, leaf_start[l + 1] - b, keys_sorted[b] >> sbits, 1};
    }
};

// Sources of a unit's window, estimated from its first cell's 27-cell window.
__device__ __forceinline__ int unit_window(const Unit& u, const int* cell_window) {
    return (int)((int64_t)cell_window[u.key] * (u.zlen + 2) / 3);
}

// Step limit of an item: the steps (64 target x source pairs) that one of the
// chip's resident waves gets, but not below kMinSteps, where an item's setup
// and staging cost as much as its steps.  Measured: a limit of half that share
// costs 2.1M particles 1% and 343000 particles 4% (more staging) and gains
// 65536 particles 8%; a floor of 128 or 512 steps costs 100003 particles 9%.
// The items this adds are bounded: a unit of c targets and window w gets at
// most c / 32 * w / limit + 2, so all units together at most
// 2 * steps / limit <= 2 * kResidentWaves more than unsplit.
__device__ __forceinline__ int item_limit(unsigned long long pairs) {
    const unsigned long long share =
        pairs / ((unsigned long long)kItemI * kResidentWaves) + 1;
    return (int)min(max(share, (unsigned long long)kMinSteps), 0x3fffffffull);
}

__device__ __forceinline__ int item_size(int window, int limit) {
    int t = kItemI;
    while (t > 1 && window > limit) {
        t >>= 1;
        limit <<= 1;
    }
    return t;
}

// Items of a unit: `full` of T targets, then one of p and one of q (0: none).
struct Pieces {
    int T, full, p, q;
    __device__ __forceinline__ int items() const { return full + (p > 0) + (q > 0); }
};

__device__ __forceinline__ Pieces pieces_of(int count, int T) {
    Pieces s;
    s.T = T;
    s.full = count / T;
    const int r = count - s.full * T;
    s.p = floor_pow2(r);
    s.q = r - s.p;
    return s;
}

__device__ __forceinline__ int lanes_per_target(int targets) {
    return floor_pow2(kItemI / targets);
}

// Quarter-octave buckets of the per-lane source count (the wave's running
// time), 0 = cheapest.
__device__ __forceinline__ int cost_bucket(int sources, int ksplit) {
    const float l = log2f(fmaxf((float)sources / (float)ksplit, 1.0f));
    return min(kCostBuckets - 1, (int)(4.0f * l));
}

// Per cell: its window size; per column (cx, cy): its pair work; in all: the
// pair work.  One wave takes a column (coalesced along z: a neighbour column
// gives a cell at most two ranges of the sorted entries).
__global__ __launch_bounds__(kBlock) void k_windows(
    const int* __restrict__ cs, Geom g, int* __restrict__ cell_window,
    unsigned long long* __restrict__ col_cost, WorkControl* __restrict__ ctl) {
    const int N = g.N, ncol = N * N;
    const int lane = threadIdx.x & (kWave - 1);
    const int waves = gridDim.x * (kBlock / kWave);
    unsigned long long sum = 0;
    for (int col = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; col < ncol;
         col += waves) {
        const int cx = col / N, cy = col % N;
        unsigned long long cost = 0;
        for (int cz = lane; cz < N; cz += kWave) {
            int w = 0;
            // the nine columns' loads are independent: all in flight at once
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                int x = cx + q / 3 - 1, y = cy + q % 3 - 1;
                bool in = true;
                if (g.periodic) {
                    x = x < 0 ? x + N : (x >= N ? x - N : x);
                    y = y < 0 ? y + N : (y >= N ? y - N : y);
                } else {
                    in = x >= 0 && x < N && y >= 0 && y < N;
                }
                const int base = in ? (x * N + y) * N : 0;
                int r = cs[base + min(cz + 2, N)] - cs[base + max(cz - 1, 0)];
                if (g.periodic) {
                    if (cz == 0) r += cs[base + N] - cs[base + N - 1];
                    if (cz == N - 1) r += cs[base + 1] - cs[base];
                }
                w += in ? r : 0;
            }
            const int c = col * N + cz;
            cell_window[c] = w;
            // at least the work of the cell's own targets, so that the bound
            // of item_limit holds for runs of cells and for leaves
            const Unit u = run_of(c, cs, g);
            const unsigned long long run =
                (unsigned long long)u.count *
                (unsigned long long)((int64_t)w * (u.zlen + 2) / 3);
            const unsigned long long own = (unsigned long long)(cs[c + 1] - cs[c]) *
                                           (unsigned long long)w;
            cost += max(run, own);
        }
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) cost += __shfl_xor(cost, o);
        if (lane == 0) col_cost[col] = cost;
        sum += cost;
    }
    __shared__ unsigned long long part[kBlock / kWave];
    if (lane == 0) part[threadIdx.x / kWave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) sum += part[w];
        if (sum) atomicAdd(&ctl->pairs, sum);
    }
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

// The unit of this thread, its pieces and their buckets (list, then cost).
struct Mine {
    Unit u;
    Pieces s;
    int bfull, bp, bq;
};

template <typename Units>
__device__ __forceinline__ Mine my_unit(const Units& units, int i, int limit,
                                        const int* __restrict__ cell_window,
                                        const int* __restrict__ col_xcd, int N) {
    Mine m{};
    if (i >= units.size()) return m;
    m.u = units.get(i);
    if (m.u.count == 0) return m;
    const int w = unit_window(m.u, cell_window);
    m.s = pieces_of(m.u.count, item_size(w, limit));
    const int list = col_xcd ? col_xcd[m.u.key / N] * kCostBuckets : 0;
    m.bfull = list + cost_bucket(w, kItemI / m.s.T);
    if (m.s.p) m.bp = list + cost_bucket(w, lanes_per_target(m.s.p));
    if (m.s.q) m.bq = list + cost_bucket(w, lanes_per_target(m.s.q));
    return m;
}

// Histogram of the items over the buckets: one block-local count in LDS, one
// global atomic per bucket and block.
template <typename Units>
__global__ __launch_bounds__(kBlock) void k_items_hist(
    Units units, const int* __restrict__ cell_window, const int* __restrict__ col_xcd,
    int N, WorkControl* __restrict__ ctl) {
    __shared__ int h[kOrderBuckets];
    for (int q = threadIdx.x; q < kOrderBuckets; q += kBlock) h[q] = 0;
    __syncthreads();
    const Mine m = my_unit(units, blockIdx.x * kBlock + threadIdx.x,
                           item_limit(ctl->pairs), cell_window, col_xcd, N);
    if (m.s.full) atomicAdd(&h[m.bfull], m.s.full);
    if (m.s.p) atomicAdd(&h[m.bp], 1);
    if (m.s.q) atomicAdd(&h[m.bq], 1);
    __syncthreads();
    for (int q = threadIdx.x; q < kOrderBuckets; q += kBlock)
        if (h[q]) atomicAdd(&ctl->count[q], h[q]);
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
// units' items over its threads.
template <typename Units>
__global__ __launch_bounds__(kBlock) void k_items_write(
    Units units, const int* __restrict__ cell_window, const int* __restrict__ col_xcd,
    int N, WorkControl* __restrict__ ctl, int max_items, WorkItem* __restrict__ out) {
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
    const Mine m = my_unit(units, blockIdx.x * kBlock + t, item_limit(ctl->pairs),
                           cell_window, col_xcd, N);
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
        it.i_count = targets;
        it.key = u.key;
        it.ksplit = (short)lanes_per_target(targets);
        it.zlen = (short)u.zlen;
        if (slot < max_items) out[slot] = it;
    }
}

inline int blocks_for(int64_t n, int per) { return (int)((n + per - 1) / per); }

template <typename Units>
hipError_t order_items(const Units& units, int n_units, const int* cell_start, Geom g,
                       bool one_list, int max_items, const WorkBuffers& b, WorkItem* items,
                       hipStream_t st) {
    const int ncol = g.N * g.N;
    hipError_t e = launch_fill_i32(reinterpret_cast<int*>(b.ctl),
                                   (int)(sizeof(WorkControl) / sizeof(int)), 0, st);
    if (e != hipSuccess) return e;
    const int nw = std::min(blocks_for(ncol, kBlock / kWave), 4096);
    hipLaunchKernelGGL(k_windows, dim3(nw), dim3(kBlock), 0, st, cell_start, g,
                       b.cell_window, b.col_cost, b.ctl);
    const int* xcd = nullptr;
    if (!one_list) {
        hipLaunchKernelGGL(k_column_xcd, dim3(1), dim3(1024), 0, st,
                           (const unsigned long long*)b.col_cost, ncol, b.col_xcd);
        xcd = b.col_xcd;
    }
    const int nb = std::max(1, blocks_for(n_units, kBlock));
    hipLaunchKernelGGL(k_items_hist<Units>, dim3(nb), dim3(kBlock), 0, st, units,
                       (const int*)b.cell_window, xcd, g.N, b.ctl);
    hipLaunchKernelGGL(k_items_write<Units>, dim3(nb), dim3(kBlock), 0, st, units,
                       (const int*)b.cell_window, xcd, g.N, b.ctl, max_items, items);
    return hipGetLastError();
}

}  // namespace

// Below this many particles the records (16 B each) fit one XCD's 4 MB L2,
// and a single list keeps the XCDs evenly loaded: no column ranges are formed.
constexpr int kOneListParticles = 1 << 18;

hipError_t launch_worklist(const int* cell_start, int n, Geom g, int max_items,
                           const WorkBuffers& b, WorkItem* items, hipStream_t st) {
    return order_items(CellUnits{cell_start, g}, g.N * g.N * g.N, cell_start, g,
                       n <= kOneListParticles, max_items, b, items, st);
}

hipError_t launch_worklist_leaves(const int* cell_start, const int* leaf_start,
                                  const int* n_leaves_dev, int n_leaves,
                                  const int* keys_sorted, int n, Geom g, int max_items,
                                  const WorkBuffers& b, WorkItem* items, hipStream_t st) {
    return order_items(LeafUnits{leaf_start, keys_sorted, n_leaves_dev, g.sbits}, n_leaves,
                       cell_start, g, n <= kOneListParticles, max_items, b, items, st);
}

}  // namespace hsr
