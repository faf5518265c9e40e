// Device side of the work list (worklist.hip) that the counting sort's kernels
// (bin.hip) also run, in blocks of their own beside theirs: the windows need
// only the cells, the histogram of the items only the windows.
#pragma once

#include "common.h"

namespace hsr {

namespace {

constexpr int kWorkBlock = 256;
constexpr int kOrderBuckets = kXcds * kCostBuckets;

__host__ __device__ __forceinline__ int floor_pow2(int v) {
    return v <= 0 ? 0 : (1 << (31 - __builtin_clz((unsigned)v)));
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
    return (int)min((int64_t)cell_window[u.key] * (u.zlen + 2) / 3, (int64_t)INT32_MAX);
}

// Step limit of an item: the steps (64 target x source pairs) that one of the
// chip's resident waves gets, but not below kMinSteps, where an item's setup
// and staging cost as much as its steps.  Measured: a limit of half that share
// costs 2.1M particles 1% and 343000 particles 4% (more staging) and gains
// 65536 particles 8%; a floor of 128 or 512 steps costs 100003 particles 9%.
// Where the chip is mostly idle that cost is nobody's, and the floor falls to
// eight shares and kFewestSteps (pair kernel of 1000 particles 24 -> 15 us,
// of 4096 24 -> 18).
// The items this adds are bounded: a unit of c targets and window w gets at
// most c / 32 * w / limit + 2, so all units together at most
// 2 * steps / limit <= 2 * kResidentWaves more than unsplit.  That needs
// limit >= share: a share that does not fit an int (pairs >= 2^50) becomes
// INT32_MAX, which no window exceeds, so that nothing is split.
__host__ __device__ __forceinline__ int item_limit(unsigned long long pairs) {
    const unsigned long long share =
        pairs / ((unsigned long long)kItemI * kResidentWaves) + 1;
    unsigned long long least = 8 * share;
    if (least < kFewestSteps) least = kFewestSteps;
    if (least > kMinSteps) least = kMinSteps;
    const unsigned long long limit = share > least ? share : least;
    return limit < INT32_MAX ? (int)limit : INT32_MAX;
}

__host__ __device__ __forceinline__ int item_size(int window, int limit) {
    int t = kItemI;
    for (int64_t steps = limit; t > 1 && window > steps; steps <<= 1) t >>= 1;
    return t;
}

// Items of a unit: `full` of T targets, then one of p and one of q (0: none).
struct Pieces {
    int T, full, p, q;
    __host__ __device__ __forceinline__ int items() const { return full + (p > 0) + (q > 0); }
};

__host__ __device__ __forceinline__ Pieces pieces_of(int count, int T) {
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
// Block `block` of `blocks`, each of kWorkBlock threads.
__device__ __forceinline__ void windows_block(
    const int* __restrict__ cs, const Geom& g, int* __restrict__ cell_window,
    unsigned long long* __restrict__ col_cost, WorkControl* __restrict__ ctl, int block,
    int blocks) {
    const int N = g.N, ncol = N * N;
    const int lane = threadIdx.x & (kWave - 1);
    const int waves = blocks * (kWorkBlock / kWave);
    unsigned long long sum = 0;
    for (int col = block * (kWorkBlock / kWave) + threadIdx.x / kWave; col < ncol;
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
    __shared__ unsigned long long part[kWorkBlock / kWave];
    if (lane == 0) part[threadIdx.x / kWave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kWorkBlock / kWave; ++w) sum += part[w];
        if (sum) atomicAdd(&ctl->pairs, sum);
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
__device__ __forceinline__ void items_hist_block(
    const Units& units, const int* __restrict__ cell_window,
    const int* __restrict__ col_xcd, int N, WorkControl* __restrict__ ctl, int block) {
    __shared__ int h[kOrderBuckets];
    for (int q = threadIdx.x; q < kOrderBuckets; q += kWorkBlock) h[q] = 0;
    __syncthreads();
    const Mine m = my_unit(units, block * kWorkBlock + threadIdx.x,
                           item_limit(ctl->pairs), cell_window, col_xcd, N);
    if (m.s.full) atomicAdd(&h[m.bfull], m.s.full);
    if (m.s.p) atomicAdd(&h[m.bp], 1);
    if (m.s.q) atomicAdd(&h[m.bq], 1);
    __syncthreads();
    for (int q = threadIdx.x; q < kOrderBuckets; q += kWorkBlock)
        if (h[q]) atomicAdd(&ctl->count[q], h[q]);
}

inline int window_blocks(int N) {
    const int b = (N * N + kWorkBlock / kWave - 1) / (kWorkBlock / kWave);
    return b < 4096 ? b : 4096;
}

}  // namespace

}  // namespace hsr
