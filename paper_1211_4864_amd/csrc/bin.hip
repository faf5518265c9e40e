// Chaining-mesh binning: cell keys and cell-relative float32 records, then for
// small sets a counting sort over the cells (its own section below), for larger
// ones stable LSD radix passes (each block orders its tile of keys in LDS and
// writes each digit's keys out as one run) and the gather of the records into
// sorted order, which also writes cell_start.  The sort key is the cell index
// followed by the Morton code of the particle's sub-cell (4^3 per cell when the
// key has room), so a cell's particles are grouped spatially and, within a
// sub-cell, keep their input order: the binning is deterministic.
//
// The chaining mesh is the cell list of the particle-particle part of a
// P^3M code (Habib et al. 2012, Sec. II); cells are at least r_cut wide so
// that all short-range partners of a particle lie in the 27 adjacent cells.
#include <algorithm>

#include "worklist.h"

namespace hsr {

namespace {

constexpr int kBlock = 256;
constexpr int kItems = 16;
constexpr int kTile = kBlock * kItems;   // 4096 elements per block

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

__device__ __forceinline__ uint64_t lanemask_lt() {
    const int l = lane_id();
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// Lanes of the wave holding the same BITS-bit value (a match over ballots).
template <int BITS>
__device__ __forceinline__ uint64_t peers(unsigned v, bool active) {
    uint64_t m = __ballot(active);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const bool bit = (v >> b) & 1u;
        const uint64_t bl = __ballot(bit && active);
        m &= bit ? bl : ~bl;
    }
    return active ? m : 0ull;
}

// Wrapped (periodic) or raw (open) coordinate and its cell index on one
// axis.  x == box after the wrap maps to 0; a non-finite coordinate lands in
// cell 0 (its record then carries the NaN and so do its accelerations).
__device__ __forceinline__ int axis_cell(double x, const Geom& g, double* xw) {
    double v = x;
    if (g.periodic) {
        v = x - g.box * floor(x / g.box);
        if (v >= g.box) v -= g.box;
    }
    const double k = floor(v / g.Lc);
    int c;
    if (!(k >= 0.0)) c = 0;
    else if (!(k <= (double)(g.N - 1))) c = g.N - 1;
    else c = (int)k;
    *xw = v;
    return c;
}

// Sub-cell index along one axis, 0..S-1, of a coordinate in its cell.
__device__ __forceinline__ int axis_sub(double xw, int c, const Geom& g, int S) {
    const double t = floor((xw - (double)c * g.Lc) / g.Lc * (double)S);
    if (!(t >= 0.0)) return 0;
    if (!(t <= (double)(S - 1))) return S - 1;
    return (int)t;
}

// How k_cell_keys counts the particles of each bucket key >> drop (counting
// sort only), leaving in vals[i] the particle's place among those of its bucket
// in order of arrival.
enum { kNoCounts = 0, kCountEach = 1, kCountBlock = 2 };

// Slots of a block's table of buckets, four per particle.
constexpr int kCountTableBits = 10;
constexpr int kCountTable = 1 << kCountTableBits;

// Sort key (cell index, then the sub-cell Morton code) and the float32
// record (position relative to the cell's lower corner, mass) of every
// particle, in input order.
// kCountEach adds every particle to its bucket's counter.  Adds on one address
// take 25 ns each in turn, so that a concentrated set is bound by them:
// kCountBlock first counts a block's particles per bucket in an LDS table (open
// addressing; it always has a free slot) and adds once per bucket and block,
// 2048 times at most instead of 524288 (all on one point: 13 ms of adds; the
// whole sort takes 0.065 now).  Also clears zero[i] where zero is given.
template <int COUNTS>
__global__ __launch_bounds__(kBlock) void k_cell_keys(
    const double* __restrict__ pos, const float* __restrict__ mass, int n,
    Geom g, int* __restrict__ keys, int* __restrict__ vals,
    float4* __restrict__ rec, int* __restrict__ counts, int drop,
    unsigned* __restrict__ zero) {
    constexpr bool kTable = COUNTS == kCountBlock;
    __shared__ int owner[kTable ? kCountTable : 1];   // bucket of a slot, -1: free
    __shared__ int held[kTable ? kCountTable : 1];    // its particles
    __shared__ int base[kTable ? kCountTable : 1];    // and the place of the first
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (kTable) {
        for (int v = threadIdx.x; v < kCountTable; v += kBlock) {
            owner[v] = -1;
            held[v] = 0;
        }
    } else if (i >= n) {
        return;
    }
    int full = 0;
    if (i < n) {
        double xw, yw, zw;
        const int cx = axis_cell(pos[3 * (int64_t)i], g, &xw);
        const int cy = axis_cell(pos[3 * (int64_t)i + 1], g, &yw);
        const int cz = axis_cell(pos[3 * (int64_t)i + 2], g, &zw);
        const int key = (cx * g.N + cy) * g.N + cz;
        int code = 0;
        const int levels = g.sbits / 3;
        if (levels > 0) {
            const int S = 1 << levels;
            const int sx = axis_sub(xw, cx, g, S);
            const int sy = axis_sub(yw, cy, g, S);
            const int sz = axis_sub(zw, cz, g, S);
            for (int b = 0; b < levels; ++b)
                code |= (((sx >> b) & 1) << (3 * b + 2)) |
                        (((sy >> b) & 1) << (3 * b + 1)) | (((sz >> b) & 1) << (3 * b));
        }
        full = (key << g.sbits) | code;
        keys[i] = full;
        if (COUNTS == kCountEach) vals[i] = atomicAdd(&counts[full >> drop], 1);
        if (zero) zero[i] = 0u;
        float4 r;
        r.x = (float)(xw - (double)cx * g.Lc);
        r.y = (float)(yw - (double)cy * g.Lc);
        r.z = (float)(zw - (double)cz * g.Lc);
        r.w = mass ? mass[i] : 0.0f;
        rec[i] = r;
    }
    if (!kTable) return;
    __syncthreads();
    const int bucket = full >> drop;
    int v = 0, place = -1;
    if (i < n) {
        // at most kBlock of the kCountTable slots are taken: the search ends
        v = (int)(((unsigned)bucket * 2654435761u) >> (32 - kCountTableBits));
        for (;;) {
            const int had = atomicCAS(&owner[v], -1, bucket);
            if (had == -1 || had == bucket) break;
            v = (v + 1) & (kCountTable - 1);
        }
        place = atomicAdd(&held[v], 1);
    }
    __syncthreads();
    if (place == 0) base[v] = atomicAdd(&counts[bucket], held[v]);
    __syncthreads();
    if (i < n) vals[i] = base[v] + place;
}

// ---------------------------------------------------------------- scan
// Exclusive prefix sum of int32: the sums of the blocks, then every block's scan
// from its carry, the sums before it, which it adds up itself.  Beyond 2048
// blocks of 4096 entries (8.4M) one block scans the sums in between; an array
// of one block takes one launch.

__device__ __forceinline__ int wave_incl_scan(int v) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int o = __shfl_up(v, d);
        if (lane_id() >= d) v += o;
    }
    return v;
}

// Block-wide exclusive scan of one value per thread; returns the prefix and
// writes the block total.
__device__ __forceinline__ int block_excl_scan(int v, int* total) {
    __shared__ int wsum[kBlock / kWave];
    const int incl = wave_incl_scan(v);
    const int w = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) wsum[w] = incl;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < kBlock / kWave; ++q) {
        const int s = wsum[q];
        if (q < w) base += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return base + incl - v;
}

template <int ITEMS>
__global__ __launch_bounds__(kBlock) void k_scan_reduce(
    const int* __restrict__ in, int n, int* __restrict__ bsum) {
    const int64_t base = (int64_t)blockIdx.x * (kBlock * ITEMS);
    int s = 0;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t e = base + it * kBlock + threadIdx.x;
        if (e < n) s += in[e];
    }
    int tot;
    block_excl_scan(s, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// One block scans an array of any length in chunks, carrying the total.
__global__ __launch_bounds__(kBlock) void k_scan_single(int* __restrict__ a,
                                                        int n) {
    int carry = 0;
    for (int64_t c0 = 0; c0 < n; c0 += kTile) {
        int v[kItems];
        int s = 0;
        const int64_t b = c0 + (int64_t)threadIdx.x * kItems;
#pragma unroll
        for (int q = 0; q < kItems; ++q) {
            v[q] = (b + q < n) ? a[b + q] : 0;
            s += v[q];
        }
        int tot;
        int pre = block_excl_scan(s, &tot) + carry;
#pragma unroll
        for (int q = 0; q < kItems; ++q) {
            if (b + q < n) a[b + q] = pre;
            pre += v[q];
        }
        carry += tot;
    }
}

// Scan of one tile plus its carry: bsum[block] when the block sums have been
// scanned, else the sum of the blocks before it, which the block adds up
// itself.  With `every`, the scan at each 2^every-th entry also goes to
// `heads` (the cells' starts among those of their sub-cells).  With `large`,
// it is set to 1 if an entry is at least `least`.
template <int ITEMS>
__global__ __launch_bounds__(kBlock) void k_scan_apply(
    const int* in, int* out, int n, const int* __restrict__ bsum, bool scanned,
    int* __restrict__ heads, int every, int* __restrict__ large, int least) {
    const int64_t b = (int64_t)blockIdx.x * (kBlock * ITEMS) + (int64_t)threadIdx.x * ITEMS;
    int v[ITEMS];
    int s = 0;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        v[q] = (b + q < n) ? in[b + q] : 0;
        s += v[q];
    }
    if (large) {
        bool any = false;
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) any = any || v[q] >= least;
        if (any) *large = 1;
    }
    int tot, carry = 0;
    if (scanned) {
        carry = bsum[blockIdx.x];
    } else if (blockIdx.x > 0) {
        int part = 0;
        for (int q = threadIdx.x; q < (int)blockIdx.x; q += kBlock) part += bsum[q];
        block_excl_scan(part, &carry);
    }
    int pre = block_excl_scan(s, &tot) + carry;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        if (b + q < n) {
            out[b + q] = pre;
            if (heads && ((b + q) & ((1 << every) - 1)) == 0) heads[(b + q) >> every] = pre;
        }
        pre += v[q];
    }
}

// ---------------------------------------------------------------- radix
// One stable counting-sort pass on a DB-bit digit of the sort key (vin null:
// the values are the entries' own indices): per
// block digit histograms, their scan (digit-major over the blocks), then the
// scatter.  This direct scatter writes each element as it is ranked; it
// serves digits of 11 bits, whose LDS-staged variant below would not fit.

// The counts are plain LDS atomics on one set of counters per wave: a sorted
// tile's equal digits meet in one wave and cost it their number in turns, less
// than finding them by ballots first (16.8M keys, 9-bit digits: 56 -> 33 us a
// pass; 2.1M, 8-bit: 13 -> 6).
template <int DB>
__global__ __launch_bounds__(kBlock) void k_radix_hist(
    const int* __restrict__ keys, int n, int shift, int* __restrict__ hist,
    int nblocks) {
    constexpr int R = 1 << DB;
    constexpr int kSets = DB <= 9 ? kBlock / kWave : 1;
    __shared__ int h[kSets][R];
    for (int q = threadIdx.x; q < R; q += kBlock)
#pragma unroll
        for (int v = 0; v < kSets; ++v) h[v][q] = 0;
    __syncthreads();
    int* mine = h[kSets > 1 ? threadIdx.x / kWave : 0];
    const int64_t base = (int64_t)blockIdx.x * kTile;
    int key[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int64_t e = base + it * kBlock + threadIdx.x;
        key[it] = e < n ? keys[e] : 0;
    }
#pragma unroll
    for (int it = 0; it < kItems; ++it)
        if (base + it * kBlock + threadIdx.x < n)
            atomicAdd(&mine[((unsigned)key[it] >> shift) & (unsigned)(R - 1)], 1);
    __syncthreads();
    for (int q = threadIdx.x; q < R; q += kBlock) {
        int sum = 0;
#pragma unroll
        for (int v = 0; v < kSets; ++v) sum += h[v][q];
        hist[(int64_t)q * nblocks + blockIdx.x] = sum;
    }
}

template <int DB>
__global__ __launch_bounds__(kBlock) void k_radix_scatter(
    const int* __restrict__ kin, const int* __restrict__ vin,
    int* __restrict__ kout, int* __restrict__ vout, int n, int shift,
    const int* __restrict__ offs, int nblocks) {
    constexpr int R = 1 << DB;
    constexpr int kW = kBlock / kWave;
    __shared__ int base_d[R];     // global offset of this block's digit d
    __shared__ int run_d[R];      // digit d entries already placed by this block
    __shared__ int wcnt[kW][R];
    for (int q = threadIdx.x; q < R; q += kBlock) {
        base_d[q] = offs[(int64_t)q * nblocks + blockIdx.x];
        run_d[q] = 0;
    }
    const int w = threadIdx.x / kWave;
    const int64_t base = (int64_t)blockIdx.x * kTile;
    for (int it = 0; it < kItems; ++it) {
        for (int q = threadIdx.x; q < R; q += kBlock)
#pragma unroll
            for (int v = 0; v < kW; ++v) wcnt[v][q] = 0;
        __syncthreads();
        const int64_t e = base + it * kBlock + threadIdx.x;
        const bool active = e < n;
        const int key = active ? kin[e] : 0;
        const int val = active ? (vin ? vin[e] : (int)e) : 0;
        const unsigned d = ((unsigned)key >> shift) & (unsigned)(R - 1);
        const uint64_t pm = peers<DB>(d, active);
        const int rank = __popcll(pm & lanemask_lt());
        if (active && rank == 0) wcnt[w][d] = __popcll(pm);
        __syncthreads();
        // each digit: exclusive prefix over the waves for these 256 keys
        for (int t = threadIdx.x; t < R; t += kBlock) {
            int acc = run_d[t];
#pragma unroll
            for (int v = 0; v < kW; ++v) {
                const int c = wcnt[v][t];
                wcnt[v][t] = acc;
                acc += c;
            }
            run_d[t] = acc;
        }
        __syncthreads();
        if (active) {
            const int dst = base_d[d] + wcnt[w][d] + rank;
            kout[dst] = key;
            vout[dst] = val;
        }
        __syncthreads();
    }
}

// The same pass with the block's keys first placed in LDS in their sorted
// order (a stable local counting sort of the 4096-key tile), then written
// out in that order: each digit's keys of the block go to consecutive
// global slots, so the writes are runs instead of one scattered element per
// lane.  Wave w ranks the keys w * 1024 .. w * 1024 + 1023 of the tile, 64 at
// a time, against its own digit counters; one prefix over the waves then
// places every key.  Needs 2^DB * (2 + 2 * kW) + 2 * 4096 ints of LDS; used
// for DB <= 10.
template <int DB>
__global__ __launch_bounds__(kBlock) void k_radix_scatter_staged(
    const int* __restrict__ kin, const int* __restrict__ vin,
    int* __restrict__ kout, int* __restrict__ vout, int n, int shift,
    const int* __restrict__ offs, int nblocks) {
    constexpr int R = 1 << DB;
    constexpr int kW = kBlock / kWave;
    constexpr int kPerW = kTile / kW / kWave;   // keys per lane
    constexpr int kPerT = R / kBlock;           // digits per thread
    static_assert(kPerT >= 1, "at least one digit per thread");
    __shared__ int base_d[R];     // global offset of this block's digit d
    __shared__ int loc_d[R];      // first tile slot of digit d in this block
    __shared__ int cw[kW][R];     // per wave: digit counts, then their prefix
    __shared__ int part[kBlock];
    __shared__ int skey[kTile];
    __shared__ int sval[kTile];
    // This block's count of each digit follows from the scanned offsets
    // (digit-major over the blocks); a block scan gives the tile slots.
    const int64_t flat = (int64_t)R * nblocks;
    int cnt[kPerT];
    int sum = 0;
#pragma unroll
    for (int j = 0; j < kPerT; ++j) {
        const int d = threadIdx.x * kPerT + j;
        const int64_t idx = (int64_t)d * nblocks + blockIdx.x;
        const int o = offs[idx];
        const int nx = idx + 1 < flat ? offs[idx + 1] : n;
        base_d[d] = o;
        cnt[j] = nx - o;
        sum += cnt[j];
#pragma unroll
        for (int v = 0; v < kW; ++v) cw[v][d] = 0;
    }
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int s = 1; s < kBlock; s <<= 1) {      // inclusive scan of the sums
        const int v = threadIdx.x >= s ? part[threadIdx.x - s] : 0;
        __syncthreads();
        part[threadIdx.x] += v;
        __syncthreads();
    }
    int acc = part[threadIdx.x] - sum;
#pragma unroll
    for (int j = 0; j < kPerT; ++j) {
        loc_d[threadIdx.x * kPerT + j] = acc;
        acc += cnt[j];
    }
    // rank of each key among the equal digits before it in this wave's keys
    const int w = threadIdx.x / kWave;
    const int64_t first = (int64_t)blockIdx.x * kTile + (int64_t)w * (kPerW * kWave) +
                          lane_id();
    int key[kPerW], val[kPerW], rk[kPerW];
#pragma unroll
    for (int r = 0; r < kPerW; ++r) {
        const int64_t e = first + r * kWave;
        const bool active = e < n;
        key[r] = active ? kin[e] : 0;
        val[r] = active ? (vin ? vin[e] : (int)e) : 0;
    }
#pragma unroll
    for (int r = 0; r < kPerW; ++r) {
        const bool active = first + r * kWave < n;
        const unsigned d = ((unsigned)key[r] >> shift) & (unsigned)(R - 1);
        const uint64_t pm = peers<DB>(d, active);
        const int rank = __popcll(pm & lanemask_lt());
        rk[r] = active ? cw[w][d] + rank : 0;
        // A wave's LDS accesses complete in program order; the barriers keep
        // the compiler from moving the counter update across the reads.
        __builtin_amdgcn_wave_barrier();
        if (active && rank == 0) cw[w][d] += __popcll(pm);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // per digit: exclusive prefix over the waves
    for (int d = threadIdx.x; d < R; d += kBlock) {
        int a = 0;
#pragma unroll
        for (int v = 0; v < kW; ++v) {
            const int c = cw[v][d];
            cw[v][d] = a;
            a += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPerW; ++r) {
        if (first + r * kWave < n) {
            const unsigned d = ((unsigned)key[r] >> shift) & (unsigned)(R - 1);
            const int slot = loc_d[d] + cw[w][d] + rk[r];
            skey[slot] = key[r];
            sval[slot] = val[r];
        }
    }
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kTile;
    const int m = (int)min((int64_t)kTile, (int64_t)n - base);
    for (int i = threadIdx.x; i < m; i += kBlock) {
        const int k = skey[i];
        const unsigned d = ((unsigned)k >> shift) & (unsigned)(R - 1);
        const int dst = base_d[d] + (i - loc_d[d]);
        kout[dst] = k;
        vout[dst] = sval[i];
    }
}

// ---------------------------------------------------------------- counting
// Counting sort for small sets, where the radix passes are a chain of
// launches that one or a few blocks run (1000 particles 33 us, 65536 67; here
// 16 and 26): the particles are counted per bucket (a cell, or its
// sub-cells where cells are well filled) as their keys are formed, placed
// in their bucket in order of arrival, and each then finds its place by
// counting the smaller entries of its bucket: sub-cell code, then input
// index, as the radix sort leaves them.  Where the work list follows, its
// windows and histogram run in the same two launches, as blocks beside the
// sort's (each launch costs 2.2 us on the host and about 2 on the GPU).
//
// Heavy buckets (heavy_least) do not count entry against entry, which is
// quadratic: the particles of one block of k_place are counted per sort key, and
// those counts added up per segment of the input, so that a particle's place
// is the keys below its own, its key's counts in the segments before, and the
// equal keys before it in its own segment.  All of it linear in n: with 524288
// particles on one point the sort takes 65 us (22.5 ms counted one by one, 91
// by radix passes), with 65536 26 (1704, 74), with a tenth of 524288 there 86
// (1567, 94); 524288 in a few cells of 100^3, where a bucket is 64 keys,
// 304 (3165, 102).

// Entry of the order array: the key bits below the bucket, then the index.
constexpr unsigned kIndexMask = (1u << kCountingIndexBits) - 1u;

// A bucket is heavy from heavy_least entries on.  Its entries of the order
// array then hold its counts, cleared by k_cell_keys: one word per sort key (all
// of its particles; unused where the bucket is one key), then per sort key a
// row of 16-bit counts, one per segment of 2^heavy_seg_bits particles of the
// input: the shortest segments, from one block of 256 particles to 16 blocks,
// whose counts fit into the bucket's entries.  A block of a longer segment
// searches the keys of those before it.
// Where it lies: counting one by one takes 1 us per 64 entries of the bucket in
// each of its waves, in turn; counting per segment 3 us where a wave has few
// keys of heavy buckets and up to 30 where it has 64, and 2.5 more per block
// that is searched, which buckets of 64 keys need sooner.
constexpr int kHeavyLeast = 1024, kHeavyLeast64 = 2048;
constexpr int kLongestSegBits = 12;      // a segment's count fits 16 bits

// Words of a sort key's row, and of all the counts.
__host__ __device__ constexpr int heavy_row(int n, int seg_bits) {
    return (((n - 1) >> seg_bits) + 2) / 2;
}
__host__ __device__ constexpr int heavy_words(int n, int drop, int seg_bits) {
    return (1 << drop) * (1 + heavy_row(n, seg_bits));
}

// For a bucket of `count` >= heavy_least entries (the search ends at kLongestSegBits).
__device__ __forceinline__ int heavy_seg_bits(int n, int drop, int count) {
    int bits = 8;
    while (bits < kLongestSegBits && heavy_words(n, drop, bits) > count) ++bits;
    return bits;
}

int heavy_least(int n, int drop) {
    return std::max(drop > 3 ? kHeavyLeast64 : kHeavyLeast,
                    heavy_words(n, drop, kLongestSegBits));
}

// Sets that are no larger have no heavy bucket and no more than that many adds
// on one counter, which cost as much as the tables of kCountBlock.
constexpr int kCountEachParticles = 1023;
static_assert(kCountEachParticles < kHeavyLeast, "small sets have no heavy bucket");

// The work list's share of a launch: blocks after the sort's `first` ones
// (none where the launch has no more).
struct BesideWork {
    CellUnits cells;
    WorkBuffers b;
    int first;
};

// The equal sort keys in a block, for its lanes with `in`: all of them, those
// of lower index, and where the first one is.  Each wave lists its keys with
// their numbers, a key in turn; its first lane of a key looks that key up in the
// other waves' lists.  Whole block.
struct Equal {
    int all, before, first;
};

struct KeyLists {
    int key[kBlock / kWave][kWave];
    int count[kBlock / kWave][kWave];
    int lane[kBlock / kWave][kWave];     // the wave's first of that key
    int len[kBlock / kWave];
};

__device__ __forceinline__ Equal equal_keys(KeyLists& s, int key, bool in) {
    constexpr int kW = kBlock / kWave;
    const int lane = lane_id(), w = (int)threadIdx.x / kWave;
    int lead = lane, same = 0, before = 0, len = 0;
    for (uint64_t left = __ballot(in); left; ++len) {
        const int l = __ffsll((unsigned long long)left) - 1;
        const int k = __shfl(key, l);
        const uint64_t m = __ballot(in && key == k);
        if (in && key == k) {
            lead = l;
            same = __popcll(m);
            before = __popcll(m & lanemask_lt());
        }
        if (lane == l) {
            s.key[w][len] = k;
            s.count[w][len] = same;
            s.lane[w][len] = l;
        }
        left &= ~m;
    }
    if (lane == 0) s.len[w] = len;
    __syncthreads();
    int all = same, lower = 0, first = w * kWave + lane;
    if (in && before == 0) {
        for (int v = kW - 1; v >= 0; --v) {
            if (v == w) continue;
            for (int j = 0; j < s.len[v]; ++j) {
                if (s.key[v][j] != key) continue;
                all += s.count[v][j];
                if (v < w) {
                    lower += s.count[v][j];
                    first = v * kWave + s.lane[v][j];
                }
            }
        }
    }
    return Equal{__shfl(all, lead), before + __shfl(lower, lead), __shfl(first, lead)};
}

__global__ __launch_bounds__(kBlock) void k_place(
    const int* __restrict__ keys, const int* __restrict__ arrival,
    const int* __restrict__ start, int n, int drop, int heavy,
    unsigned* __restrict__ order, const int* __restrict__ any_heavy, BesideWork w) {
    if ((int)blockIdx.x >= w.first) {
        windows_block(w.cells.cs, w.cells.g, w.b.cell_window, w.b.col_cost, w.b.ctl,
                      blockIdx.x - w.first, gridDim.x - w.first);
        return;
    }
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const bool live = i < n;
    const int key = live ? keys[i] : -1;
    const int b = live ? start[key >> drop] : 0;
    const unsigned low = (unsigned)key & ((1u << drop) - 1u);
    const bool any = n >= heavy && *any_heavy;        // uniform
    const int count = any && live ? start[(key >> drop) + 1] - b : 0;
    const bool is_heavy = any && count >= heavy;
    if (live && !is_heavy) order[b + arrival[i]] = (low << kCountingIndexBits) | (unsigned)i;
    if (!any || !__syncthreads_or(is_heavy)) return;
    __shared__ KeyLists lists;
    const Equal q = equal_keys(lists, key, is_heavy);
    if (!is_heavy || q.before) return;
    const int bits = heavy_seg_bits(n, drop, count);
    const int seg = i >> bits;
    if (drop) atomicAdd(&order[b + low], (unsigned)q.all);
    atomicAdd(&order[b + (1 << drop) + (int)low * heavy_row(n, bits) + (seg >> 1)],
              (unsigned)q.all << (16 * (seg & 1)));
}

// Block `block` of the input's particles: those of heavy buckets, by input index.
__device__ __forceinline__ void gather_heavy(
    int block, const unsigned* __restrict__ order, const int* __restrict__ start,
    const int* __restrict__ keys, int n, int drop, int heavy,
    const float4* __restrict__ rec_in, float4* __restrict__ rec, int* __restrict__ perm,
    int* __restrict__ keys_out) {
    __shared__ KeyLists lists;
    __shared__ int sk[kBlock];
    __shared__ int base[kBlock];        // by the first particle of a key
    __shared__ int longest;             // bits of the block's longest segment
    const int i0 = block * kBlock, i = i0 + (int)threadIdx.x;
    const bool live = i < n;
    const int key = live ? keys[i] : -1;
    const int b = live ? start[key >> drop] : 0;
    const int count = live ? start[(key >> drop) + 1] - b : 0;
    const bool is_heavy = count >= heavy;
    if (threadIdx.x == 0) longest = 0;
    if (!__syncthreads_or(is_heavy)) return;
    Equal q = equal_keys(lists, key, is_heavy);
    int bits = 0;
    if (is_heavy) {
        bits = heavy_seg_bits(n, drop, count);
        atomicMax(&longest, bits);
    }
    // the counts before each key's first particle, added up by 16 lanes, or by
    // the whole wave where it has one
    const int low = key & ((1 << drop) - 1);
    const int seg = i >> bits;
    const int lane = lane_id(), wave0 = (int)threadIdx.x - lane;
    for (uint64_t left = __ballot(is_heavy && q.before == 0); left;) {
        const int group = left & (left - 1) ? 16 : kWave;
        uint64_t mine = left;                       // the group's: first to fourth left
#pragma unroll
        for (int t = 0; t < kWave / 16; ++t) {
            if (t < lane / group) mine &= mine - 1;
            left &= left - 1;
        }
        const int l = mine ? __ffsll((unsigned long long)mine) - 1 : 0;
        const unsigned* area = order + __shfl(b, l);
        const int lw = __shfl(low, l), sg = __shfl(seg, l);
        const unsigned* row = area + (1 << drop) + lw * heavy_row(n, __shfl(bits, l));
        unsigned sum = 0u;
        if (mine) {
            for (int v = lane & (group - 1); v < lw; v += group) sum += area[v];
#pragma unroll 8
            for (int w = lane & (group - 1); w <= sg >> 1; w += group) {
                const unsigned two = row[w];
                sum += (2 * w < sg ? two & 0xffffu : 0u) + (2 * w + 1 < sg ? two >> 16 : 0u);
            }
        }
        for (int o = 1; o < group; o <<= 1) sum += (unsigned)__shfl_xor((int)sum, o);
        if (mine && (lane & (group - 1)) == 0) base[wave0 + l] = (int)sum;
    }
    __syncthreads();
    // the equal keys in the blocks before this one in its segment
    for (int s0 = i0 >> longest << longest; s0 < i0; s0 += kBlock) {
        __syncthreads();
        sk[threadIdx.x] = keys[s0 + (int)threadIdx.x];
        __syncthreads();
        if (is_heavy && s0 >= seg << bits)
            for (int j = 0; j < kBlock; ++j) q.before += sk[j] == key;
    }
    if (!is_heavy) return;
    const int at = b + base[q.first] + q.before;
    rec[at] = rec_in[i];
    perm[at] = i;
    keys_out[at] = key;
}

// A wave takes 64 consecutive entries.  Their buckets' entries are read 64 at
// a time, coalesced, and handed round through LDS as broadcast uint4 reads;
// two instructions per entry where the wave lies in one bucket.  The heavy
// buckets' particles have the first `heavy_blocks` blocks (one per block of the
// input where the set is large enough for one): beside the others, so that
// these need not wait for the flag (32768 particles: 5.2 us against 6.8).
__global__ __launch_bounds__(kBlock) void k_order_gather(
    const unsigned* __restrict__ order, const int* __restrict__ start,
    const int* __restrict__ keys, int n, int drop, int heavy, int heavy_blocks,
    const int* __restrict__ any_heavy, const float4* __restrict__ rec_in,
    float4* __restrict__ rec, int* __restrict__ perm, int* __restrict__ keys_out,
    BesideWork w_list) {
    if ((int)blockIdx.x >= w_list.first) {
        items_hist_block(w_list.cells, w_list.b.cell_window, nullptr, w_list.cells.g.N,
                         w_list.b.ctl, blockIdx.x - w_list.first);
        return;
    }
    if ((int)blockIdx.x < heavy_blocks) {
        if (*any_heavy)
            gather_heavy(blockIdx.x, order, start, keys, n, drop, heavy, rec_in, rec, perm,
                         keys_out);
        return;
    }
    __shared__ __align__(16) unsigned entries[kBlock / kWave][kWave];
    const int k = ((int)blockIdx.x - heavy_blocks) * kBlock + threadIdx.x;
    const int lane = lane_id(), w = threadIdx.x / kWave;
    if (k - lane >= n) return;
    const unsigned mine = k < n ? order[k] : 0u;
    // A heavy bucket's entries hold counts.  Whatever index they spell, it is
    // clamped, and the bucket that it leads to is heavy or does not hold k.
    const int i = min((int)(mine & kIndexMask), n - 1);
    const int key = keys[i];
    const int b = start[key >> drop], e = start[(key >> drop) + 1];
    const bool live = k < n && b <= k && k < e && e - b < heavy;
    // a heavy bucket is longer than a wave: the live lanes are consecutive
    const uint64_t lanes = __ballot(live);
    if (!lanes) return;
    const int lo = __shfl(b, __ffsll((unsigned long long)lanes) - 1);
    const int hi = __shfl(e, 63 - __clzll((long long)lanes));
    const bool one = __ballot(live && (b != lo || e != hi)) == 0ull;
    unsigned* sh = entries[w];
    int r = 0;
    for (int j0 = lo; j0 < hi; j0 += kWave) {
        const int j = j0 + lane;
        sh[lane] = j < hi ? order[j] : ~0u;
        // a wave's LDS accesses complete in program order
        __builtin_amdgcn_wave_barrier();
        if (one) {
#pragma unroll
            for (int q = 0; q < kWave / 4; ++q) {
                const unsigned* u = sh + 4 * q;
                r += (u[0] < mine) + (u[1] < mine) + (u[2] < mine) + (u[3] < mine);
            }
        } else {
#pragma unroll
            for (int q = 0; q < kWave / 4; ++q) {
                const unsigned* u = sh + 4 * q;
                const unsigned at = (unsigned)(j0 + 4 * q - b), len = (unsigned)(e - b);
                r += (u[0] < mine && at < len) + (u[1] < mine && at + 1u < len) +
                     (u[2] < mine && at + 2u < len) + (u[3] < mine && at + 3u < len);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (!live) return;
    rec[b + r] = rec_in[i];
    perm[b + r] = i;
    keys_out[b + r] = key;
}

// Empty runs of cells are written by many waves: one per kRunCells consecutive
// cells looks whether they lie in one run, and writes them.
constexpr int kRunCells = 4096;

// Wave q's cells: all with one start, or left to the entries' lanes.
__device__ __forceinline__ void fill_empty_run(const int* __restrict__ keys, int n, int sbits,
                                               int64_t q, int* __restrict__ cell_start) {
    const int c0 = (int)(q * kRunCells);
    // entries in the cells before c0: a search with 64 probes a step
    int lo = 0, hi = n;
    while (lo < hi) {
        const int step = (hi - lo - 1) / kWave + 1;
        const int64_t at = lo + (lane_id() + 1) * (int64_t)step - 1;
        const int cnt = __popcll(__ballot(at < hi && keys[at < hi ? at : lo] >> sbits < c0));
        hi = (int)min((int64_t)hi, lo + (cnt + 1) * (int64_t)step - 1);
        lo += cnt * step;
    }
    if (lo < n && keys[lo] >> sbits < c0 + kRunCells - 1) return;
    for (int c = lane_id(); c < kRunCells; c += kWave) cell_start[c0 + c] = lo;
}

// Records in sorted order, and cell_start: entry k starts every cell after its
// predecessor's up to its own (the last entry also ends the cells after its
// own).  A lane writes a short run of cells itself, its wave a longer one, but
// for whole kRunCells in it, which the first `fill_blocks` blocks write.
// Bound by the random 16-byte reads; the starts ride along (16.8M particles in
// 85^3 cells: 0.36 ms for the gather and 0.07 for a fill, an occupancy count
// and its scan, 0.38 together; 524289 in one corner of 400^3 cells: 0.15 ms
// for the whole binning, 25 with each run written by one wave).
__global__ __launch_bounds__(kBlock) void k_gather_records(
    const float4* __restrict__ rec_in, const int* __restrict__ perm,
    const int* __restrict__ keys, int n, int sbits, int ncell, int fill_blocks,
    float4* __restrict__ rec, int* __restrict__ cell_start) {
    constexpr int kShort = 4;
    if ((int)blockIdx.x < fill_blocks) {
        const int64_t q = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
        if ((q + 1) * kRunCells <= (int64_t)ncell + 1)
            fill_empty_run(keys, n, sbits, q, cell_start);
        return;
    }
    const int k = ((int)blockIdx.x - fill_blocks) * kBlock + threadIdx.x;
    const bool live = k < n;
    int from = 0, to = 0;                    // cells [from, to) start at entry k
    if (live) {
        rec[k] = rec_in[perm[k]];
        to = (keys[k] >> sbits) + 1;
        from = k ? (keys[k - 1] >> sbits) + 1 : 0;
        if (to - from <= kShort)
            for (int c = from; c < to; ++c) cell_start[c] = k;
    }
    auto run = [&](int f, int t, int v) {
        const int a = (f + kRunCells - 1) / kRunCells * kRunCells, z = t / kRunCells * kRunCells;
        const int gap = z > a ? z - a : 0;   // whole kRunCells
        for (int c = f + lane_id(); c < t - gap; c += kWave)
            cell_start[gap && c >= a ? c + gap : c] = v;
    };
    uint64_t left = __ballot(live && to - from > kShort);
    while (left) {
        const int l = __ffsll((unsigned long long)left) - 1;
        run(__shfl(from, l), __shfl(to, l), __shfl(k, l));
        left &= left - 1;
    }
    const uint64_t end = __ballot(live && k == n - 1);
    if (end) run(__shfl(to, __ffsll((unsigned long long)end) - 1), ncell + 1, n);
}

__global__ __launch_bounds__(kBlock) void k_gather_vec3(
    const float* __restrict__ v, const int* __restrict__ perm, int n,
    float4* __restrict__ out) {
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k >= n) return;
    const int64_t i = perm[k];
    out[k] = make_float4(v[3 * i], v[3 * i + 1], v[3 * i + 2], 0.0f);
}

__global__ __launch_bounds__(kBlock) void k_clear_two(int* p, int n, int* q, int m) {
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k < n) p[k] = 0;
    if (k < m) q[k] = 0;
}

__global__ __launch_bounds__(kBlock) void k_iota(int* p, int n) {
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k < n) p[k] = k;
}

__global__ __launch_bounds__(kBlock) void k_fill_i32(int* p, int n, int value) {
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k < n) p[k] = value;
}

inline int blocks_for(int64_t n, int per) { return (int)((n + per - 1) / per); }

// Block sums that every block of k_scan_apply adds up itself: eight loads per
// thread at most, less than the launch of k_scan_single.
constexpr int kOwnCarryBlocks = 2048;

}  // namespace

hipError_t launch_cell_keys(const double* pos, const float* mass, int n,
                            Geom g, int* keys, float4* rec, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cell_keys<kNoCounts>, dim3(blocks_for(n, kBlock)), dim3(kBlock),
                       0, st, pos, mass, n, g, keys, (int*)nullptr, rec, (int*)nullptr, 0,
                       (unsigned*)nullptr);
    return hipGetLastError();
}

namespace {
// Entries per thread of a scan: 16, or 4 for arrays of at most 2048 blocks of
// those, whose launches are latency-bound (74089 entries: 19 blocks of 16 per
// thread take 6 us each for the sums and for the scan, 73 blocks of 4 half).
constexpr int kFewItems = 4;
bool few_items(int n) { return blocks_for(n, kBlock * kFewItems) <= kOwnCarryBlocks; }
}  // namespace

// Room for the block sums of any array of at most n entries.
size_t scan_tmp_ints(int n) {
    return (size_t)std::max(blocks_for(n, kTile),
                            std::min(blocks_for(n, kBlock * kFewItems), kOwnCarryBlocks)) + 1;
}

namespace {
hipError_t scan_exclusive(const int* in, int* out, int n, int* tmp, int* heads, int every,
                          int* large, int least, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const dim3 block(kBlock);
    if (few_items(n)) {
        const int nb = blocks_for(n, kBlock * kFewItems);
        if (nb > 1)
            hipLaunchKernelGGL(k_scan_reduce<kFewItems>, dim3(nb), block, 0, st, in, n, tmp);
        hipLaunchKernelGGL(k_scan_apply<kFewItems>, dim3(nb), block, 0, st, in, out, n,
                           (const int*)tmp, false, heads, every, large, least);
        return hipGetLastError();
    }
    const int nb = blocks_for(n, kTile);
    const bool scanned = nb > kOwnCarryBlocks;
    hipLaunchKernelGGL(k_scan_reduce<kItems>, dim3(nb), block, 0, st, in, n, tmp);
    if (scanned) hipLaunchKernelGGL(k_scan_single, dim3(1), block, 0, st, tmp, nb);
    hipLaunchKernelGGL(k_scan_apply<kItems>, dim3(nb), block, 0, st, in, out, n,
                       (const int*)tmp, scanned, heads, every, large, least);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_scan_exclusive(const int* in, int* out, int n, int* tmp,
                                 hipStream_t st) {
    return scan_exclusive(in, out, n, tmp, nullptr, 0, nullptr, 0, st);
}

hipError_t launch_counting_sort(const double* pos, const float* mass, int n, Geom g,
                                int sub, int* keys, int* arrival, float4* rec_in,
                                int* buckets, int* cell_start, int* tmp, unsigned* order,
                                int* any_heavy, float4* rec, int* perm, int* keys_out,
                                const WorkBuffers* work, hipStream_t st) {
    static_assert(kBlock == kWorkBlock, "both shares of a launch have the same blocks");
    static_assert(kOneListParticles >= kCountingParticles, "the histogram needs no XCDs");
    if (n <= 0) return hipSuccess;
    const int drop = g.sbits - sub;
    const int ncell = g.N * g.N * g.N;
    const int nbuckets = ncell << sub;
    const int nb = blocks_for(n, kBlock);
    const int heavy = heavy_least(n, drop);
    // the work list's control words hold any_heavy
    int* words = work ? reinterpret_cast<int*>(work->ctl) : any_heavy;
    const int nwords = work ? kControlInts : 1;
    hipLaunchKernelGGL(k_clear_two, dim3(blocks_for(std::max(nbuckets + 1, nwords), kBlock)),
                       dim3(kBlock), 0, st, buckets, nbuckets + 1, words, nwords);
    unsigned* zero = n >= heavy ? order : nullptr;
    if (n <= kCountEachParticles)
        hipLaunchKernelGGL(k_cell_keys<kCountEach>, dim3(nb), dim3(kBlock), 0, st, pos, mass, n,
                           g, keys, arrival, rec_in, buckets, drop, zero);
    else
        hipLaunchKernelGGL(k_cell_keys<kCountBlock>, dim3(nb), dim3(kBlock), 0, st, pos, mass, n,
                           g, keys, arrival, rec_in, buckets, drop, zero);
    hipError_t e = scan_exclusive(buckets, buckets, nbuckets + 1, tmp,
                                  buckets == cell_start ? nullptr : cell_start, sub,
                                  n >= heavy ? any_heavy : nullptr, heavy, st);
    if (e != hipSuccess) return e;
    const int hb = n >= heavy ? nb : 0;
    const CellUnits cells{cell_start, g};
    const WorkBuffers bufs = work ? *work : WorkBuffers{};
    hipLaunchKernelGGL(k_place, dim3(nb + (work ? window_blocks(g.N) : 0)), dim3(kBlock), 0, st,
                       (const int*)keys, (const int*)arrival, (const int*)buckets, n, drop,
                       heavy, order, (const int*)any_heavy, BesideWork{cells, bufs, nb});
    hipLaunchKernelGGL(k_order_gather, dim3(hb + nb + (work ? blocks_for(ncell, kBlock) : 0)),
                       dim3(kBlock), 0, st, (const unsigned*)order, (const int*)buckets,
                       (const int*)keys, n, drop, heavy, hb, (const int*)any_heavy,
                       (const float4*)rec_in, rec, perm, keys_out,
                       BesideWork{cells, bufs, hb + nb});
    return hipGetLastError();
}

int radix_blocks(int n) { return blocks_for(n, kTile); }

namespace {
template <int DB>
hipError_t radix_pass(const int* kin, const int* vin, int* kout, int* vout,
                      int n, int shift, int* hist, int* scan_tmp,
                      hipStream_t st) {
    const int nb = radix_blocks(n);
    hipLaunchKernelGGL(k_radix_hist<DB>, dim3(nb), dim3(kBlock), 0, st, kin, n,
                       shift, hist, nb);
    hipError_t e = launch_scan_exclusive(hist, hist, (1 << DB) * nb, scan_tmp, st);
    if (e != hipSuccess) return e;
    if constexpr (DB <= 10)
        hipLaunchKernelGGL(k_radix_scatter_staged<DB>, dim3(nb), dim3(kBlock), 0, st,
                           kin, vin, kout, vout, n, shift, (const int*)hist, nb);
    else
        hipLaunchKernelGGL(k_radix_scatter<DB>, dim3(nb), dim3(kBlock), 0, st, kin,
                           vin, kout, vout, n, shift, (const int*)hist, nb);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_radix_pass(const int* kin, const int* vin, int* kout,
                             int* vout, int n, int shift, int digit_bits,
                             int* hist, int* scan_tmp, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    switch (digit_bits) {
        case 8: return radix_pass<8>(kin, vin, kout, vout, n, shift, hist, scan_tmp, st);
        case 9: return radix_pass<9>(kin, vin, kout, vout, n, shift, hist, scan_tmp, st);
        case 10: return radix_pass<10>(kin, vin, kout, vout, n, shift, hist, scan_tmp, st);
        case 11: return radix_pass<11>(kin, vin, kout, vout, n, shift, hist, scan_tmp, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gather_records(const float4* rec_in, const int* perm, const int* keys,
                                 int n, Geom g, float4* rec, int* cell_start,
                                 hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int ncell = g.N * g.N * g.N;
    const int fill = blocks_for((ncell + 1) / kRunCells, kBlock / kWave);
    hipLaunchKernelGGL(k_gather_records, dim3(fill + blocks_for(n, kBlock)), dim3(kBlock), 0,
                       st, rec_in, perm, keys, n, g.sbits, ncell, fill, rec, cell_start);
    return hipGetLastError();
}

hipError_t launch_gather_vec3(const float* v, const int* perm, int n,
                              float4* out, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_vec3, dim3(blocks_for(n, kBlock)), dim3(kBlock),
                       0, st, v, perm, n, out);
    return hipGetLastError();
}

hipError_t launch_iota(int* p, int n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_iota, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, st, p, n);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int* p, int n, int value, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0,
                       st, p, n, value);
    return hipGetLastError();
}

}  // namespace hsr
