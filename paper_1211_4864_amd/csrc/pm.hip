// Long-range spectral particle-mesh (PM) force (Habib et al. 2012, Sec. II):
// Cloud-In-Cell deposit of the masses on a periodic ng^3 grid, a forward
// 3-D FFT, the isotropising filter of Eq. 5 times the sixth-order periodic
// influence function, fourth-order spectral differencing of the potential,
// inverse FFTs and CIC interpolation back to the particles.
//
// Readings where the paper names an operator only by its order: the
// influence function is the inverse of the Fourier symbol of the
// sixth-order central-difference Laplacian,
//   K6(k) = sum_a [6 sin^2(k_a D/2) - 0.6 sin^2(k_a D) + (2/45) sin^2(3 k_a D/2)] / D^2
// (the same polynomial in cos(k_a D) as 49/18 - 3 cos + 3/10 cos 2 - 1/45
// cos 3, written without its cancelling constant); the gradient symbol is
// that of the fourth-order central difference, (4/3 sin(k_a D) -
// 1/6 sin(2 k_a D)) / D; the filter's sinc is read as
// [sin(k D/2) / (k D/2)]^n_s with k = |k|, sigma in grid cells.
//
// Layout and order of work (grids complex float32, ng^3 float2, z fastest):
//  - Deposit: each particle adds m w 2^62 / (n max|m|), rounded to int64, to
//    its 8 corners.  Integer sums do not depend on the order of the
//    additions: the whole solve is bitwise reproducible, and the two ways
//    below give the same bits.
//  - Sets whose grid stays in the caches (direct_pm) deposit and interpolate
//    straight from the positions, one thread per particle in input order.
//  - Larger sets are sorted by tiles of 8^3 cells first: one pass writes each
//    particle's lower-corner cell (tile, then cell in the tile) and a record
//    (the three CIC fractions and the mass, float32), a stable LSD radix sort
//    orders the tiles.  A block takes kChunk consecutive particles, gathers
//    their records into that order and sums the deposit of each of their tiles
//    in LDS, so that only its 9^3 sums are added to the grid.
//  - FFT: one kernel per axis.  A workgroup transforms L lines of ng points
//    as ng = R1 x R2 (the four-step method): each thread does a length-R1
//    DFT in registers, multiplies by the twiddles of the length-ng transform
//    and passes its values through LDS to the threads of a length-R2 DFT.
//    For the strided axes the L lines are adjacent in memory, so that the
//    loads and stores of a wave are contiguous over the lines.
//  - The first forward pass reads the fixed-point deposit.  The last forward
//    pass (x) applies the potential's and the gradient's symbols to its
//    lines in registers and runs the inverse x pass of the two output grids
//    at once: B = (D_y - i D_x) phi (its inverse is a_x + i a_y, both real)
//    and A = -i D_z phi (its inverse has a_z as real part).  The inverse y
//    and z passes take both grids in one launch, and one interpolation
//    kernel reads a_x, a_y and a_z at the 8 corners.  1 / ng^3 is folded
//    into the potential.
#include <algorithm>

#include "common.h"

namespace hsr {

namespace {

constexpr int kPB = 256;
constexpr float kPi = 3.14159265358979323846f;

// ---- preparation

constexpr int kMaxBlocks = 1024;

// Per-axis terms of the symbols at index m (below, with the FFT).
__device__ __forceinline__ float4 axis_symbol(int m, int ng, float d);

// Block-wide maximum of an unsigned value per thread, in every thread.
template <int THREADS>
__device__ __forceinline__ unsigned block_max(unsigned v) {
    __shared__ unsigned part[THREADS / kWave];
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) v = max(v, (unsigned)__shfl_xor((int)v, o));
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = v;
    __syncthreads();
    v = part[0];
#pragma unroll
    for (int w = 1; w < THREADS / kWave; ++w) v = max(v, part[w]);
    return v;
}

// Everything the deposit needs, in one launch: clears the fixed-point grid,
// writes tw[k] = exp(-2 pi i k / ng) and the per-axis symbol terms, and
// leaves each block's largest |mass| (as the bit pattern of a non-negative
// float, ordered like an unsigned integer) in mass_max.
__global__ __launch_bounds__(kPB) void k_pm_prepare(
    const float* __restrict__ mass, int n, int ng, float d, ulonglong2* __restrict__ grid,
    float2* __restrict__ tw, float4* __restrict__ sym, unsigned* __restrict__ mass_max) {
    const int64_t first = (int64_t)blockIdx.x * kPB + threadIdx.x;
    const int64_t all = (int64_t)gridDim.x * kPB;
    const int64_t pairs = (int64_t)ng * ng * ng / 2;
    for (int64_t k = first; k < pairs; k += all) grid[k] = make_ulonglong2(0ull, 0ull);
    for (int64_t k = first; k < ng; k += all) {
        float s, c;
        sincospif(2.0f * (float)k / (float)ng, &s, &c);
        tw[k] = make_float2(c, -s);
        sym[k] = axis_symbol((int)k, ng, d);
    }
    unsigned v = 0u;
    for (int64_t k = first; k < n; k += all) v = max(v, __float_as_uint(fabsf(mass[k])));
    v = block_max<kPB>(v);
    if (threadIdx.x == 0) mass_max[blockIdx.x] = v;
}

// The blocks' maxima of |mass|, and the largest of all, kept for the transform.
struct MassMax {
    const unsigned* of_block;
    int blocks;
    unsigned* all;
};

template <int THREADS>
__device__ __forceinline__ double largest_mass(const MassMax& m) {
    unsigned v = 0u;
    for (int k = threadIdx.x; k < m.blocks; k += THREADS) v = max(v, m.of_block[k]);
    v = block_max<THREADS>(v);
    if (blockIdx.x == 0 && threadIdx.x == 0) *m.all = v;
    return (double)__uint_as_float(v);
}

// ---- sort by tile

// Lower grid index and the CIC fraction of a coordinate (grid point g at
// g D, periodic).
__device__ __forceinline__ int cic_axis(double x, double inv_d, int ng, double* frac) {
    double u = x * inv_d;
    u -= (double)ng * floor(u / (double)ng);
    double fl = floor(u);
    int i = (int)fl;
    double f = u - fl;
    if (i >= ng) { i -= ng; }
    if (i < 0 || !(f >= 0.0 && f < 1.0)) { i = 0; f = 0.0; }   // non-finite positions
    *frac = f;
    return i;
}

__device__ __forceinline__ void cic_point(const double* __restrict__ pos, int i, double inv_d,
                                          int ng, int g0[3], double f[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) g0[a] = cic_axis(pos[3 * (int64_t)i + a], inv_d, ng, &f[a]);
}

// Tiles of kSide^3 cells: the sort key is the tile's index (x, y, z; z fastest)
// followed by the cell's in the tile.
constexpr int kSide = 8;
constexpr int kSideBits = 3;
constexpr int kCellBits = 3 * kSideBits;

__device__ __forceinline__ int tile_key(const int g0[3], int ng) {
    const int nt = ng / kSide;
    const int tile = ((g0[0] / kSide) * nt + g0[1] / kSide) * nt + g0[2] / kSide;
    const int cell = ((g0[0] % kSide) * kSide + g0[1] % kSide) * kSide + g0[2] % kSide;
    return (tile << kCellBits) | cell;
}

// Lower corner of a key's cell, and of its tile.
__device__ __forceinline__ void key_corner(int key, int ng, int g0[3], int t0[3]) {
    const int nt = ng / kSide;
    const int tile = key >> kCellBits;
    t0[2] = tile % nt * kSide;
    t0[1] = tile / nt % nt * kSide;
    t0[0] = tile / (nt * nt) * kSide;
    g0[2] = t0[2] + (key & (kSide - 1));
    g0[1] = t0[1] + ((key >> kSideBits) & (kSide - 1));
    g0[0] = t0[0] + ((key >> (2 * kSideBits)) & (kSide - 1));
}

__global__ __launch_bounds__(kPB) void k_pm_keys(const double* __restrict__ pos,
                                                 const float* __restrict__ mass, int n, int ng,
                                                 double inv_d, int* __restrict__ keys,
                                                 float4* __restrict__ rec) {
    const int i = blockIdx.x * kPB + threadIdx.x;
    if (i >= n) return;
    int g0[3];
    double f[3];
    cic_point(pos, i, inv_d, ng, g0, f);
    keys[i] = tile_key(g0, ng);
    rec[i] = make_float4((float)f[0], (float)f[1], (float)f[2], mass[i]);
}

// ---- deposit

__device__ __forceinline__ int64_t corner_index(const int g0[3], int c, int ng) {
    const int bx = c >> 2, by = (c >> 1) & 1, bz = c & 1;
    const int x = g0[0] + bx == ng ? 0 : g0[0] + bx;
    const int y = g0[1] + by == ng ? 0 : g0[1] + by;
    const int z = g0[2] + bz == ng ? 0 : g0[2] + bz;
    return ((int64_t)x * ng + y) * ng + z;
}

__device__ __forceinline__ double corner_weight(const double f[3], int c) {
    const int bx = c >> 2, by = (c >> 1) & 1, bz = c & 1;
    return (bx ? f[0] : 1.0 - f[0]) * (by ? f[1] : 1.0 - f[1]) * (bz ? f[2] : 1.0 - f[2]);
}

__device__ __forceinline__ void deposit_one(unsigned long long* grid, const int g0[3],
                                            const double f[3], double m, int ng) {
#pragma unroll
    for (int c = 0; c < 8; ++c)
        atomicAdd(&grid[corner_index(g0, c, ng)],
                  (unsigned long long)llrint(m * corner_weight(f, c)));
}

constexpr double kFixedScale = 4611686018427387904.0;      // 2^62

// Particles in input order.  Atomics of many blocks on one address take about
// 180 ns each in turn, so the dense cells of a clustered set bound this: a
// block first adds up its particles' corners in an LDS table (an entry
// belongs to the first corner that claims it; others that meet it go to
// memory) and adds each entry to the grid once.  Neighbours along z sit side by
// side in the table, so that a wave's atomics fall on fewer lines (18 G
// atomics/s on lines of their own).  50000 Plummer particles on 64^3: 54 us with
// one atomic per corner, 28 with a table of single entries, 20 with rows of 8.
// The fractions are rounded to float32 as the records of the sorted path hold
// them.
constexpr int kDB = 256;                  // threads of a block
constexpr int kDChunk = 256;              // its particles
constexpr int kTableBits = 12;
constexpr int kTable = 1 << kTableBits;   // its table, in rows of kRow neighbours along z
constexpr int kRowBits = 3;
constexpr int kRow = 1 << kRowBits;

__global__ __launch_bounds__(kDB) void k_pm_deposit_direct(
    const double* __restrict__ pos, const float* __restrict__ mass, int n, int ng,
    double inv_d, MassMax mass_max, unsigned long long* __restrict__ grid) {
    __shared__ int owner[kTable];
    __shared__ unsigned long long sum[kTable];
    for (int v = threadIdx.x; v < kTable; v += kDB) {
        owner[v] = -1;
        sum[v] = 0ull;
    }
    const double mmax = largest_mass<kDB>(mass_max);   // synchronises
    if (!(mmax > 0.0)) return;                       // uniform: nothing to deposit
    const double scale = kFixedScale / ((double)n * mmax);
    const int first = blockIdx.x * kDChunk;
    const int end = min(n, first + kDChunk);
    for (int i = first + (int)threadIdx.x; i < end; i += kDB) {
        int g0[3];
        double f[3];
        cic_point(pos, i, inv_d, ng, g0, f);
#pragma unroll
        for (int a = 0; a < 3; ++a) f[a] = (double)(float)f[a];
        const double m = (double)mass[i] * scale;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int at = (int)corner_index(g0, c, ng);
            const unsigned long long q = (unsigned long long)llrint(m * corner_weight(f, c));
            const int v = (int)((((unsigned)at / kRow) * 2654435761u) >> (32 - kTableBits + kRowBits))
                              * kRow | (at & (kRow - 1));
            const int had = atomicCAS(&owner[v], -1, at);
            if (had == -1 || had == at) atomicAdd(&sum[v], q);
            else atomicAdd(&grid[at], q);
        }
    }
    __syncthreads();
    for (int v = threadIdx.x; v < kTable; v += kDB)
        if (owner[v] >= 0 && sum[v]) atomicAdd(&grid[owner[v]], sum[v]);
}

// Particles of a block of the sorted passes, and the fewest of one tile that
// the block takes through LDS: below that, clearing and adding (or reading)
// the tile's 9^3 values costs more than the particles' own 8 corners.
constexpr int kChunk = 1024;
constexpr int kFewest = 64;
constexpr int kEdge = kSide + 1;
constexpr int kCorners = kEdge * kEdge * kEdge;

// The tiles of a block's particles: the ranges of tiles with at least kFewest
// of them (in any order), and tile[q] = -1 for the particles of the others.
struct Ranges {
    int tile[kChunk];
    int start[kChunk + 1];
    int2 full[kChunk / kFewest];
    int n_full;
    int part[kPB / kWave];
};

__device__ __forceinline__ void find_ranges(const int* __restrict__ keys, int first, int m,
                                            Ranges& r) {
    constexpr int kPer = kChunk / kPB;
    for (int q = threadIdx.x; q < m; q += kPB) r.tile[q] = keys[first + q] >> kCellBits;
    if (threadIdx.x == 0) r.n_full = 0;
    __syncthreads();
    // thread t looks at entries t * kPer ..: a scan of the counts of starts
    // gives each start its place
    bool is[kPer];
    int mine = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int q = threadIdx.x * kPer + j;
        is[j] = q < m && (q == 0 || r.tile[q] != r.tile[q - 1]);
        mine += is[j];
    }
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int incl = mine;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    if (lane == kWave - 1) r.part[w] = incl;
    __syncthreads();
    int at = incl - mine, all = 0;
#pragma unroll
    for (int k = 0; k < kPB / kWave; ++k) {
        if (k < w) at += r.part[k];
        all += r.part[k];
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (is[j]) r.start[at++] = threadIdx.x * kPer + j;
    if (threadIdx.x == 0) r.start[all] = m;
    __syncthreads();
    for (int t = threadIdx.x; t < all; t += kPB) {
        const int a = r.start[t], b = r.start[t + 1];
        if (b - a >= kFewest)
            r.full[atomicAdd(&r.n_full, 1)] = make_int2(a, b);
        else
            for (int q = a; q < b; ++q) r.tile[q] = -1;
    }
    __syncthreads();
}

// Index of corner c of a cell in its tile's 9^3 corners, and the grid index of
// corner v of a tile.
__device__ __forceinline__ int corner_in_tile(int key, int c) {
    const int x = ((key >> (2 * kSideBits)) & (kSide - 1)) + (c >> 2);
    const int y = ((key >> kSideBits) & (kSide - 1)) + ((c >> 1) & 1);
    const int z = (key & (kSide - 1)) + (c & 1);
    return (x * kEdge + y) * kEdge + z;
}

__device__ __forceinline__ int64_t tile_corner_index(const int t0[3], int v, int ng) {
    int x = t0[0] + v / (kEdge * kEdge), y = t0[1] + v / kEdge % kEdge, z = t0[2] + v % kEdge;
    x = x == ng ? 0 : x;
    y = y == ng ? 0 : y;
    z = z == ng ? 0 : z;
    return ((int64_t)x * ng + y) * ng + z;
}

// Gathers the block's records into tile order, for itself and for the
// interpolation, and deposits them.  The gather waits on random 16-byte reads
// and the deposit on LDS atomics (8 of 64 bits per particle), so that the two
// overlap between the blocks of a CU; kChunk is small for that.  The whole solve of
// 16.8M NFW particles on 256^3: 2.01 ms with the gather in a launch of its own
// (0.37 ms, and 0.28 for the deposit), 1.89 now; 262144 particles on 64^3 112 ->
// 101 us (111 with 2048 particles per block).  With every corner added in memory
// the deposit alone takes 0.78 ms.
__global__ __launch_bounds__(kPB) void k_pm_deposit(
    const int* __restrict__ keys, const int* __restrict__ vals,
    const float4* __restrict__ rec_in, float4* rec, int n, int ng, MassMax mass_max,
    unsigned long long* __restrict__ grid) {
    __shared__ Ranges r;
    __shared__ unsigned long long acc[kCorners];
    const int first = blockIdx.x * kChunk;
    const int m = min(kChunk, n - first);
    {
        constexpr int kPer = kChunk / kPB;
        int from[kPer];
        float4 p[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            from[j] = vals[first + min((int)threadIdx.x + j * kPB, m - 1)];
#pragma unroll
        for (int j = 0; j < kPer; ++j) p[j] = rec_in[from[j]];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int q = threadIdx.x + j * kPB;
            if (q < m) rec[first + q] = p[j];
        }
    }
    const double mmax = largest_mass<kPB>(mass_max);
    if (!(mmax > 0.0)) return;                       // uniform: nothing to deposit
    const double scale = kFixedScale / ((double)n * mmax);
    find_ranges(keys, first, m, r);                  // also: the block's records are written
    for (int q = threadIdx.x; q < m; q += kPB) {
        if (r.tile[q] >= 0) continue;
        const float4 p = rec[first + q];
        const double f[3] = {(double)p.x, (double)p.y, (double)p.z};
        int g0[3], t0[3];
        key_corner(keys[first + q], ng, g0, t0);
        deposit_one(grid, g0, f, (double)p.w * scale, ng);
    }
    for (int t = 0; t < r.n_full; ++t) {
        const int a = r.full[t].x, b = r.full[t].y;
        for (int v = threadIdx.x; v < kCorners; v += kPB) acc[v] = 0ull;
        __syncthreads();
        for (int q = a + (int)threadIdx.x; q < b; q += kPB) {
            const int key = keys[first + q];
            const float4 p = rec[first + q];
            const double f[3] = {(double)p.x, (double)p.y, (double)p.z};
            const double w = (double)p.w * scale;
#pragma unroll
            for (int c = 0; c < 8; ++c)
                atomicAdd(&acc[corner_in_tile(key, c)],
                          (unsigned long long)llrint(w * corner_weight(f, c)));
        }
        __syncthreads();
        int g0[3], t0[3];
        key_corner(r.tile[a] << kCellBits, ng, g0, t0);
        for (int v = threadIdx.x; v < kCorners; v += kPB)
            if (acc[v]) atomicAdd(&grid[tile_corner_index(t0, v, ng)], acc[v]);
        __syncthreads();
    }
}

// ---- FFT

// cos(2 pi j / 32), j = 0..8
__device__ constexpr float kCos32[9] = {1.0f,         0.980785251f, 0.923879504f,
                                        0.831469595f, 0.707106769f, 0.555570245f,
                                        0.382683426f, 0.195090324f, 0.0f};

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// b * exp(SIGN 2 pi i j / 32), 0 <= j < 16, j a compile-time constant after
// unrolling (so the multiplications by 1 and by +-i fold away).
template <int SIGN>
__device__ __forceinline__ float2 rot32(float2 b, int j) {
    if (j == 0) return b;
    if (j == 8) return SIGN < 0 ? make_float2(b.y, -b.x) : make_float2(-b.y, b.x);
    const float c = j <= 8 ? kCos32[j] : -kCos32[16 - j];
    const float s = j <= 8 ? kCos32[8 - j] : kCos32[j - 8];
    return cmul(b, make_float2(c, SIGN < 0 ? -s : s));
}

template <int R>
__device__ constexpr int bitrev(int i) {
    int r = 0;
    for (int b = 1; b < R; b <<= 1) {
        r = (r << 1) | (i & 1);
        i >>= 1;
    }
    return r;
}

// In-register DFT of length R (2..32), natural order in and out:
// v[k] <- sum_j v[j] exp(SIGN 2 pi i j k / R).  Radix-2 decimation in time.
template <int SIGN, int R>
__device__ __forceinline__ void dft(float2 (&v)[R]) {
    float2 t[R];
#pragma unroll
    for (int i = 0; i < R; ++i) t[i] = v[bitrev<R>(i)];
#pragma unroll
    for (int h = 1; h < R; h <<= 1) {
#pragma unroll
        for (int g = 0; g < R; g += 2 * h) {
#pragma unroll
            for (int p = 0; p < h; ++p) {
                const float2 a = t[g + p];
                const float2 b = rot32<SIGN>(t[g + p + h], p * (16 / h));
                t[g + p] = make_float2(a.x + b.x, a.y + b.y);
                t[g + p + h] = make_float2(a.x - b.x, a.y - b.y);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = t[i];
}

template <int NG>
struct Shape {
    static constexpr int R1 = NG == 8 ? 2 : NG == 16 ? 4 : NG == 32 ? 4 : NG == 64 ? 8
                            : NG == 128 ? 8 : NG == 256 ? 16 : 32;
    static constexpr int R2 = NG / R1;
    static constexpr int TPL = R1 > R2 ? R1 : R2;          // threads per line
    static constexpr int L = NG < kPB / TPL ? NG : kPB / TPL;   // lines per workgroup
    static constexpr int P = R2 + 1;                       // LDS row pitch
    static constexpr int THREADS = L * TPL;
    static constexpr int TILES = NG * NG / L;
};

enum { kPlain = 0, kFromFixed = 1, kFusedX = 2 };

struct FftArgs {
    float2* a;                         // first grid
    float2* b;                         // second grid (two-grid passes, fused output)
    const unsigned long long* q;       // fixed-point deposit (first pass)
    const float2* tw;                  // tw[k] = exp(-2 pi i k / ng)
    const float4* sym;                 // per-axis symbol terms at index m
    const unsigned* mmax_bits;
    double unit;                       // density per fixed-point unit and max|m|
    float d, sigma;
    int n_s;
};

__device__ __forceinline__ int freq(int m, int ng) { return m < ng / 2 ? m : m - ng; }

// Per-axis terms of the symbols at index m: the K6 term (times D^2), k_a^2
// and the gradient symbol D_a.
__device__ __forceinline__ float4 axis_symbol(int m, int ng, float d) {
    const float th = (float)freq(m, ng) / (float)ng;        // k_a D / (2 pi)
    const float s1 = sinpif(th), s2 = sinpif(2.0f * th), s3 = sinpif(3.0f * th);
    const float k6 = 6.0f * s1 * s1 - 0.6f * s2 * s2 + (2.0f / 45.0f) * s3 * s3;
    const float kq = 2.0f * kPi * th / d;
    const float dk = ((4.0f / 3.0f) * s2 - (1.0f / 6.0f) * sinpif(4.0f * th)) / d;
    return make_float4(k6, kq * kq, dk, 0.0f);
}

// One pass along AXIS (0: x, stride ng^2; 1: y, stride ng; 2: z,
// contiguous) over the L lines of workgroup blockIdx.x.  kPlain transforms
// grid a (blockIdx.y == 0) or b (blockIdx.y == 1) in place with sign SIGN;
// kFromFixed reads the fixed-point deposit and writes the forward transform
// of the density into a; kFusedX (AXIS 0) does the forward x transform of
// a, the symbols and the inverse x transforms into b and a.
template <int NG, int AXIS, int MODE, int SIGN>
__global__ __launch_bounds__(kPB) void k_fft(FftArgs A) {
    using S = Shape<NG>;
    constexpr int R1 = S::R1, R2 = S::R2, TPL = S::TPL, L = S::L, P = S::P;
    __shared__ float2 sm[L * R1 * P];
    const int tid = threadIdx.x;
    const int line = AXIS == 2 ? tid / TPL : tid % L;
    const int r = AXIS == 2 ? tid % TPL : tid / L;
    const int g = blockIdx.x;
    int64_t base, es;
    int ly = 0, lz = 0;                                     // the line's y and z (AXIS 0)
    if (AXIS == 2) {
        base = ((int64_t)g * L + line) * NG;
        es = 1;
    } else {
        const int outer = g / (NG / L);
        const int z = (g % (NG / L)) * L + line;
        base = AXIS == 1 ? (int64_t)outer * NG * NG + z : (int64_t)outer * NG + z;
        es = AXIS == 1 ? NG : (int64_t)NG * NG;
        ly = outer;
        lz = z;
    }
    auto li = [&](int k1, int n2) {
        return AXIS == 2 ? line * (R1 * P) + k1 * P + n2 : line + L * (k1 * P + n2);
    };
    float2* data = (MODE == kPlain && blockIdx.y == 1) ? A.b : A.a;
    double unit = 0.0;
    if (MODE == kFromFixed) unit = A.unit * (double)__uint_as_float(*A.mmax_bits);

    // stage 1: thread n2 = r, DFT over n1 of x[n2 + R2 n1], twiddle, to LDS
    constexpr int FS = MODE == kFusedX ? -1 : SIGN;
    float2 v[R1];
    if (r < R2) {
#pragma unroll
        for (int n1 = 0; n1 < R1; ++n1) {
            const int64_t at = base + (int64_t)(r + R2 * n1) * es;
            if (MODE == kFromFixed)
                v[n1] = make_float2((float)((double)(long long)A.q[at] * unit), 0.0f);
            else
                v[n1] = data[at];
        }
        dft<FS, R1>(v);
#pragma unroll
        for (int k1 = 0; k1 < R1; ++k1) {
            float2 w = A.tw[(r * k1) & (NG - 1)];
            if (FS > 0) w.y = -w.y;
            sm[li(k1, r)] = cmul(v[k1], w);
        }
    }
    __syncthreads();
    // stage 2: thread k1 = r, DFT over n2; u[k2] = X[k1 + R1 k2]
    float2 u[R2];
    if (r < R1) {
#pragma unroll
        for (int n2 = 0; n2 < R2; ++n2) u[n2] = sm[li(r, n2)];
        dft<FS, R2>(u);
    }
    if (MODE != kFusedX) {
        if (r < R1) {
#pragma unroll
            for (int k2 = 0; k2 < R2; ++k2) data[base + (int64_t)(r + R1 * k2) * es] = u[k2];
        }
        return;
    }
    // symbols: phi = -4 pi S(k) / K6(k) / ng^3 times the density's transform
    float2 bv[R2];
    if (r < R1) {
        const float4 sy = A.sym[ly], sz = A.sym[lz];
        const float norm = 1.0f / ((float)NG * (float)NG * (float)NG);
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) {
            const int mx = r + R1 * k2;
            const float4 sx = A.sym[mx];
            const float dkx = sx.z, dky = sy.z, dkz = sz.z;
            float gk = 0.0f;
            if (mx != 0 || ly != 0 || lz != 0) {
                const float k6 = (sx.x + sy.x + sz.x) / (A.d * A.d);
                const float ksq = sx.y + sy.y + sz.y;
                const float xh = 0.5f * sqrtf(ksq) * A.d;
                const float sinc = sinf(xh) / xh;
                float Sk = expf(-0.25f * ksq * A.sigma * A.sigma * A.d * A.d);
                for (int q = 0; q < A.n_s; ++q) Sk *= sinc;
                gk = -4.0f * kPi * Sk / k6 * norm;
            }
            const float2 ph = make_float2(gk * u[k2].x, gk * u[k2].y);
            bv[k2] = make_float2(dky * ph.x + dkx * ph.y, dky * ph.y - dkx * ph.x);
            u[k2] = make_float2(dkz * ph.y, -dkz * ph.x);
        }
    }
    // inverse x transforms: thread k1 = r holds X[k1 + R1 k2]; a length-R2
    // DFT over k2, the twiddles, LDS, a length-R1 DFT over k1 by thread n2
#pragma unroll
    for (int out = 0; out < 2; ++out) {
        float2* dst = out == 0 ? A.b : A.a;
        __syncthreads();                                    // LDS reads above are done
        if (r < R1) {
            if (out == 0) dft<+1, R2>(bv);
            else dft<+1, R2>(u);
#pragma unroll
            for (int n2 = 0; n2 < R2; ++n2) {
                float2 w = A.tw[(n2 * r) & (NG - 1)];
                w.y = -w.y;
                sm[li(r, n2)] = cmul(out == 0 ? bv[n2] : u[n2], w);
            }
        }
        __syncthreads();
        if (r < R2) {
#pragma unroll
            for (int k1 = 0; k1 < R1; ++k1) v[k1] = sm[li(k1, r)];
            dft<+1, R1>(v);
#pragma unroll
            for (int n1 = 0; n1 < R1; ++n1) dst[base + (int64_t)(r + R2 * n1) * es] = v[n1];
        }
    }
}

// ---- interpolation

// a_x, a_y come from the real and imaginary parts of grid b, a_z from the real
// part of grid a.
__device__ __forceinline__ void interp_one(const float2* __restrict__ gxy,
                                           const float2* __restrict__ gz, const int g0[3],
                                           const double f[3], int ng,
                                           float* __restrict__ out) {
    float ax = 0.0f, ay = 0.0f, az = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float w = (float)corner_weight(f, c);
        const int64_t at = corner_index(g0, c, ng);
        const float2 xy = gxy[at];
        ax = __builtin_fmaf(w, xy.x, ax);
        ay = __builtin_fmaf(w, xy.y, ay);
        az = __builtin_fmaf(w, gz[at].x, az);
    }
    out[0] = ax;
    out[1] = ay;
    out[2] = az;
}

__global__ __launch_bounds__(kPB) void k_pm_interp_direct(
    const double* __restrict__ pos, int n, int ng, double inv_d,
    const float2* __restrict__ gxy, const float2* __restrict__ gz, float* __restrict__ out) {
    const int i = blockIdx.x * kPB + threadIdx.x;
    if (i >= n) return;
    int g0[3];
    double f[3];
    cic_point(pos, i, inv_d, ng, g0, f);
#pragma unroll
    for (int a = 0; a < 3; ++a) f[a] = (double)(float)f[a];
    interp_one(gxy, gz, g0, f, ng, out + 3 * (int64_t)i);
}

// A block takes kIChunk particles in tile order, reads the 9^3 corners of each
// of their tiles into LDS once and interpolates from there; where they lie in
// more than kMostTiles tiles, reading those in turn takes longer than each
// particle's own corners do.
// Bound by the scattered 12-byte writes (0.23 ms of it) and the tiles' corners:
// 16.8M NFW particles on 256^3 take 0.53 ms, 0.80 with every corner read from
// memory, 0.56 and 0.66 with 512 and 2048 particles per block (0.46 with
// every corner from memory after a full sort by cell, whose third radix pass
// takes 0.16 ms).
constexpr int kIChunk = 1024;
constexpr int kMostTiles = 6;
__global__ __launch_bounds__(kPB) void k_pm_interp(
    const int* __restrict__ perm, const int* __restrict__ keys,
    const float4* __restrict__ rec, int n, int ng, const float2* __restrict__ gxy,
    const float2* __restrict__ gz, float* __restrict__ out) {
    constexpr int kPer = kIChunk / kPB;
    __shared__ float4 field[kCorners];
    __shared__ int next_tile;
    const int first = blockIdx.x * kIChunk;
    const int m = min(kIChunk, n - first);
    int key[kPer], dst[kPer];
    float4 p[kPer];
    int tiles = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int q = j * kPB + (int)threadIdx.x;
        const int k = first + min(q, m - 1);
        key[j] = q < m ? keys[k] : -1;
        p[j] = rec[k];
        dst[j] = perm[k];
        tiles += __syncthreads_count(q < m && (q == 0 || keys[k - 1] >> kCellBits !=
                                                             key[j] >> kCellBits));
    }
    if (tiles > kMostTiles) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (key[j] < 0) continue;
            const double f[3] = {(double)p[j].x, (double)p[j].y, (double)p[j].z};
            int g0[3], t0[3];
            key_corner(key[j], ng, g0, t0);
            interp_one(gxy, gz, g0, f, ng, out + 3 * (int64_t)dst[j]);
        }
        return;
    }
    int tile = keys[first] >> kCellBits;
    for (int left = tiles; left > 0; --left) {
        if (threadIdx.x == 0) next_tile = 0x7fffffff;
        int g0[3], t0[3];
        key_corner(tile << kCellBits, ng, g0, t0);
        for (int v = threadIdx.x; v < kCorners; v += kPB) {
            const int64_t at = tile_corner_index(t0, v, ng);
            const float2 xy = gxy[at];
            field[v] = make_float4(xy.x, xy.y, gz[at].x, 0.0f);
        }
        __syncthreads();
        int after = 0x7fffffff;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int tj = key[j] >> kCellBits;       // -1 for no particle
            if (tj > tile) after = min(after, tj);
            if (tj != tile) continue;
            const double f[3] = {(double)p[j].x, (double)p[j].y, (double)p[j].z};
            float ax = 0.0f, ay = 0.0f, az = 0.0f;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float w = (float)corner_weight(f, c);
                const float4 e = field[corner_in_tile(key[j], c)];
                ax = __builtin_fmaf(w, e.x, ax);
                ay = __builtin_fmaf(w, e.y, ay);
                az = __builtin_fmaf(w, e.z, az);
            }
            float* o = out + 3 * (int64_t)dst[j];
            o[0] = ax;
            o[1] = ay;
            o[2] = az;
        }
        if (after != 0x7fffffff) atomicMin(&next_tile, after);
        __syncthreads();
        tile = next_tile;
        __syncthreads();
    }
}

inline int blocks_for(int64_t n, int per) { return (int)((n + per - 1) / per); }

template <int NG>
void launch_fft_all(const FftArgs& a, hipStream_t st) {
    using S = Shape<NG>;
    const dim3 blk(S::THREADS);
    hipLaunchKernelGGL((k_fft<NG, 2, kFromFixed, -1>), dim3(S::TILES), blk, 0, st, a);
    hipLaunchKernelGGL((k_fft<NG, 1, kPlain, -1>), dim3(S::TILES, 1), blk, 0, st, a);
    hipLaunchKernelGGL((k_fft<NG, 0, kFusedX, -1>), dim3(S::TILES), blk, 0, st, a);
    hipLaunchKernelGGL((k_fft<NG, 1, kPlain, +1>), dim3(S::TILES, 2), blk, 0, st, a);
    hipLaunchKernelGGL((k_fft<NG, 2, kPlain, +1>), dim3(S::TILES, 2), blk, 0, st, a);
}

// Radix sort of the tiles: 3 log2(ng / kSide) bits in passes of 8 or 9.
void pm_sort_shape(int ng, int* passes, int* digit_bits) {
    int lg = 0;
    while ((1 << lg) < ng) ++lg;
    const int bits = 3 * (lg - kSideBits);
    *passes = (bits + 8) / 9;
    *digit_bits = *passes ? std::max(8, (bits + *passes - 1) / *passes) : 8;
}

// Whether to deposit and interpolate in input order, without the sort: its
// launches cost more than the scattered accesses to a grid (microseconds,
// direct / sorted, Plummer): 8^3 with 2048 particles 23 / 33, 131072 36 / 45;
// 16^3 16384 30 / 54, 131072 50 / 59; 32^3 32768 40 / 74, 131072 64 / 69,
// 200000 95 / 70; 64^3 65536 61 / 97, 131072 90 / 97, 262144 133 / 97; 128^3
// 131072 132 / 173, 262144 176 / 191, 524288 272 / 222; 256^3 393216 560 / 598,
// 1048576 825 / 799; 512^3 393216 5787 / 5865, 4194304 7448 / 7304.  Uniform
// sets and all particles on one point cross over later.
bool direct_pm(int ng, int64_t n) {
    return n <= (1 << 17) + std::min<int64_t>((int64_t)ng * ng * ng / 64, 1 << 18);
}

struct PmLayout {
    size_t a, b, tw, sym, mmax, block_max, keys_a, vals_a, keys_b, vals_b, rec_in, rec, hist, scan_tmp,
        total;
};

PmLayout pm_layout(int ng, int64_t n) {
    PmLayout L{};
    const size_t cells = (size_t)ng * ng * ng;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = (off + bytes + 255) & ~(size_t)255;
        return at;
    };
    int passes, db;
    pm_sort_shape(ng, &passes, &db);
    const int nn = (int)std::max<int64_t>(n, 1);
    const size_t hist_n = ((size_t)1 << db) * (size_t)radix_blocks(nn);
    const size_t ni = sizeof(int) * (size_t)nn;
    L.a = take(cells * sizeof(float2));
    L.b = take(cells * sizeof(float2));      // also the fixed-point deposit
    L.tw = take((size_t)ng * sizeof(float2));
    L.sym = take((size_t)ng * sizeof(float4));
    L.mmax = take(sizeof(unsigned));
    L.keys_a = take(ni);
    L.vals_a = take(ni);
    L.keys_b = take(ni);
    L.vals_b = take(ni);
    L.rec_in = take(sizeof(float4) * (size_t)nn);
    L.rec = take(sizeof(float4) * (size_t)nn);
    L.hist = take(sizeof(int) * hist_n);
    // until the transform writes it, grid a holds the blocks' maxima and, where
    // there is room for them, the scan's sums
    static_assert(sizeof(unsigned) * kMaxBlocks <= 8 * 8 * 8 * sizeof(float2), "fits 8^3");
    L.block_max = L.a;
    L.scan_tmp = L.a + sizeof(unsigned) * kMaxBlocks;
    const size_t tmp = sizeof(int) * scan_tmp_ints((int)hist_n);
    if (L.scan_tmp + tmp > L.b) L.scan_tmp = take(tmp);
    L.total = off;
    return L;
}

}  // namespace

size_t pm_workspace_bytes(int ng, int64_t n) { return pm_layout(ng, n).total; }

hipError_t launch_pm_accel(const double* pos, const float* mass, int n, double box, int ng,
                           float sigma, int n_s, void* ws, float* out_acc, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int64_t cells = (int64_t)ng * ng * ng;
    const PmLayout PL = pm_layout(ng, n);
    char* base = reinterpret_cast<char*>(ws);
    float2* A = reinterpret_cast<float2*>(base + PL.a);
    float2* B = reinterpret_cast<float2*>(base + PL.b);
    unsigned long long* Q = reinterpret_cast<unsigned long long*>(B);
    float2* tw = reinterpret_cast<float2*>(base + PL.tw);
    float4* sym = reinterpret_cast<float4*>(base + PL.sym);
    unsigned* mmax = reinterpret_cast<unsigned*>(base + PL.mmax);
    unsigned* block_maxima = reinterpret_cast<unsigned*>(base + PL.block_max);
    int* ka = reinterpret_cast<int*>(base + PL.keys_a);
    int* va = reinterpret_cast<int*>(base + PL.vals_a);
    int* kb = reinterpret_cast<int*>(base + PL.keys_b);
    int* vb = reinterpret_cast<int*>(base + PL.vals_b);
    float4* rec_in = reinterpret_cast<float4*>(base + PL.rec_in);
    float4* rec = reinterpret_cast<float4*>(base + PL.rec);
    int* hist = reinterpret_cast<int*>(base + PL.hist);
    int* tmp = reinterpret_cast<int*>(base + PL.scan_tmp);
    const double d = box / ng;
    const double inv_d = (double)ng / box;
    const int mb = std::min(kMaxBlocks, std::max(blocks_for(n, kPB), blocks_for(cells / 2, kPB)));
    hipLaunchKernelGGL(k_pm_prepare, dim3(mb), dim3(kPB), 0, st, mass, n, ng, (float)d,
                       reinterpret_cast<ulonglong2*>(Q), tw, sym, block_maxima);
    const MassMax mass_max{block_maxima, mb, mmax};
    const bool direct = direct_pm(ng, n);
    if (direct) {
        hipLaunchKernelGGL(k_pm_deposit_direct, dim3(blocks_for(n, kDChunk)), dim3(kDB), 0, st, pos,
                           mass, n, ng, inv_d, mass_max, Q);
    } else {
        hipLaunchKernelGGL(k_pm_keys, dim3(blocks_for(n, kPB)), dim3(kPB), 0, st, pos, mass,
                           n, ng, inv_d, ka, rec_in);
        int passes, db;
        pm_sort_shape(ng, &passes, &db);
        for (int p = 0; p < passes; ++p) {
            const hipError_t e = launch_radix_pass(ka, p ? va : nullptr, kb, vb, n, kCellBits + db * p, db,
                                                   hist, tmp, st);
            if (e != hipSuccess) return e;
            std::swap(ka, kb);
            std::swap(va, vb);
        }
        if (!passes) {                       // one tile: input order
            const hipError_t e = launch_iota(va, n, st);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(k_pm_deposit, dim3(blocks_for(n, kChunk)), dim3(kPB), 0, st,
                           (const int*)ka, (const int*)va, (const float4*)rec_in, rec, n, ng,
                           mass_max, Q);
    }
    FftArgs fa{};
    fa.a = A;
    fa.b = B;
    fa.q = Q;
    fa.tw = tw;
    fa.sym = sym;
    fa.mmax_bits = mmax;
    // density = q (n max|m| / 2^62) / D^3; k_fft multiplies by max|m|
    fa.unit = (double)n / 4611686018427387904.0 / (d * d * d);
    fa.d = (float)d;
    fa.sigma = sigma;
    fa.n_s = n_s;
    switch (ng) {
        case 8: launch_fft_all<8>(fa, st); break;
        case 16: launch_fft_all<16>(fa, st); break;
        case 32: launch_fft_all<32>(fa, st); break;
        case 64: launch_fft_all<64>(fa, st); break;
        case 128: launch_fft_all<128>(fa, st); break;
        case 256: launch_fft_all<256>(fa, st); break;
        case 512: launch_fft_all<512>(fa, st); break;
        default: return hipErrorInvalidValue;
    }
    if (direct)
        hipLaunchKernelGGL(k_pm_interp_direct, dim3(blocks_for(n, kPB)), dim3(kPB), 0, st, pos,
                           n, ng, inv_d, (const float2*)B, (const float2*)A, out_acc);
    else
        hipLaunchKernelGGL(k_pm_interp, dim3(blocks_for(n, kIChunk)), dim3(kPB), 0, st,
                           (const int*)va, (const int*)ka, (const float4*)rec, n, ng,
                           (const float2*)B, (const float2*)A, out_acc);
    return hipGetLastError();
}

}  // namespace hsr
