// Internal definitions shared by the HIP translation units of libhacc_sr.
// Not part of the public interface (include/hacc_sr.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hsr {

constexpr int kWave = 64;

// Chaining-mesh geometry: N^3 cells of side Lc = |box| / N >= r_cut.
struct Geom {
    int N;            // cells per axis
    int periodic;     // 1: periodic cube [0, box); 0: open domain [0, box)
    double box;       // |box|
    double Lc;        // cell side, float64
    float Lc_f;       // cell side rounded to float32 (frame shifts)
    int sbits;        // sub-cell bits of the sort key: 6 (4^3 sub-cells), 3 or 0
};

// Pair-kernel constants derived on the host from (r_cut, eps, poly).
// The grid-force polynomial is evaluated in t = alpha * (s + eps) + beta,
// which maps s in [0, r_cut^2] onto [-1, 1]; b[] are its coefficients in t
// db2[] those of 2 d(poly)/ds, also in t, and dq3[] = db2[] / 3.
struct PairParams {
    float alpha, beta;
    float eps;
    float rc2e;       // float32(r_cut^2 + eps): cut-off test on s + eps
    float cull2;      // float32(r_cut^2 (1 + 2^-12)): staging drops sources
                      // at least this far (squared) from the target box
    float b[6];
    float db2[5];
    float dq3[5];
};

// One unit of pair-kernel work: T = i_count target particles of one run of
// cells, processed by one wave with ksplit lanes per target (T * ksplit <= 64).
struct WorkItem {
    int i_begin;             // first sorted entry of the targets
    int key;                 // first cell of the item's run of cells
    short cx, cy;            // its column
    unsigned char i_count;   // number of targets T (1..kItemI)
    unsigned char ksplit;    // lanes per target, a power of two
    unsigned char zlen;      // cells in the run: key, key + 1, ... along z
    unsigned char pad;
};
static_assert(sizeof(WorkItem) == 16, "one 16-byte load");

// Small cells are merged into runs of up to kZRun cells along z (one item,
// one source window of 3 x 3 x (zlen + 2) cells) when a whole aligned block
// holds at most kItemI targets.
constexpr int kZRun = 2;
constexpr int kMaxSegments = 9 * (kZRun + 2);   // stencil cells of a run

constexpr int kItemI = 64;     // lanes of a wave

// ---- work list: buffers and constants

constexpr int kCostBuckets = 128;
constexpr int kXcds = 8;            // XCDs of an MI355X
// Item splitting (item_limit): waves the chip holds at 8 per SIMD, and the
// number of steps below which an item is not split, in a set that fills the
// chip and in the smallest.
constexpr int kResidentWaves = 8192;
constexpr int kMinSteps = 256;
constexpr int kFewestSteps = 16;
// Items that splitting may add (the bound is in item_limit).
constexpr int kMaxSplitItems = 2 * kResidentWaves;

struct WorkControl {
    unsigned long long pairs;             // pair work of all units
    int n_items;
    int any_heavy;                        // counting sort: a heavy bucket was met
    int count[kXcds * kCostBuckets];      // items per (list, cost bucket)
    int taken[kXcds * kCostBuckets];      // ranks handed out to blocks
};

constexpr int kControlInts = (int)(sizeof(WorkControl) / sizeof(int));

struct WorkBuffers {
    WorkControl* ctl;
    int* cell_window;
    unsigned long long* col_cost;
    int* col_xcd;
};

// ---- launch wrappers (each defined in the translation unit of its kernels)

// binning (bin.hip)
hipError_t launch_cell_keys(const double* pos, const float* mass, int n,
                            Geom g, int* keys, float4* rec, hipStream_t st);
// Largest set of the counting sort (launch_counting_sort), which beats the
// radix passes there.  Binning, this sort / radix passes in us, uniform and
// Plummer sets at a particle per mesh cell: 1000 16 / 33 and 31 / 33, 32768
// 23 / 46 and 32 / 48, 262144 47 / 79 and 55 / 80, 524288 75 / 88 and 88 / 90,
// 700000 93 / 94 and 108 / 95, 1030301 144 / 105 and 153 / 106 (random
// single-entry atomics and writes).  Concentrated sets: all on one point 65536
// 26 / 74, 524288 65 / 91; ten clumps inside cells 262144 79 / 84, 524288
// 127 / 94, and where a bucket is 64 sort keys 304 / 102 (100^3 cells).
constexpr int kCountingParticles = 1 << 19;
// Sets whose work list is a single one in decreasing cost; larger ones have
// one per XCD.
constexpr int kOneListParticles = kCountingParticles;
// The sort's entries hold the input index in their low bits.
constexpr int kCountingIndexBits = 26;
// buckets: (cells << sub) + 1 counters, cell_start itself when sub is 0.
// any_heavy: that word of the work list's control, whether or not work is given.
// work: also form the work list's windows and histogram there (or null).
hipError_t launch_counting_sort(const double* pos, const float* mass, int n, Geom g,
                                int sub, int* keys, int* arrival, float4* rec_in,
                                int* buckets, int* cell_start, int* tmp, unsigned* order,
                                int* any_heavy, float4* rec, int* perm, int* keys_out,
                                const WorkBuffers* work, hipStream_t st);
size_t scan_tmp_ints(int n);
hipError_t launch_scan_exclusive(const int* in, int* out, int n, int* tmp,
                                 hipStream_t st);
int radix_blocks(int n);
constexpr int kMaxDigitBits = 11;
// vin null: the values are the entries' indices (first pass).
hipError_t launch_radix_pass(const int* kin, const int* vin, int* kout,
                             int* vout, int n, int shift, int digit_bits,
                             int* hist, int* scan_tmp, hipStream_t st);
// Also writes cell_start from the sorted keys.
hipError_t launch_gather_records(const float4* rec_in, const int* perm, const int* keys,
                                 int n, Geom g, float4* rec, int* cell_start,
                                 hipStream_t st);
hipError_t launch_gather_vec3(const float* v, const int* perm, int n,
                              float4* out, hipStream_t st);
hipError_t launch_fill_i32(int* p, int n, int value, hipStream_t st);
hipError_t launch_iota(int* p, int n, hipStream_t st);     // p[k] = k

// work list (worklist.hip)
// started: launch_counting_sort has formed the windows and the histogram.
hipError_t launch_worklist(const int* cell_start, int n, Geom g, bool started,
                           int max_items, const WorkBuffers& b, WorkItem* items,
                           hipStream_t st);
hipError_t launch_worklist_leaves(const int* cell_start, const int* leaf_start,
                                  const int* n_leaves_dev, int n_leaves,
                                  const int* keys_sorted, int n, Geom g, int max_items,
                                  const WorkBuffers& b, WorkItem* items, hipStream_t st);

// pair kernels (pair.hip)
hipError_t launch_pair_force(const WorkItem* items, int max_items,
                             const int* n_items_dev, const float4* rec,
                             const int* cell_start, const int* perm, Geom g,
                             PairParams p, float* out_acc, hipStream_t st);
hipError_t launch_pair_count(const WorkItem* items, int max_items,
                             const int* n_items_dev, const float4* rec,
                             const int* cell_start, Geom g, PairParams p,
                             unsigned long long* counts, hipStream_t st);
hipError_t launch_pair_vjp(const WorkItem* items, int max_items,
                           const int* n_items_dev, const float4* rec,
                           const float4* gsorted, const int* cell_start,
                           const int* perm, Geom g, PairParams p,
                           double* out_grad, hipStream_t st);

// RCB fat leaves inside the chaining cells (rcb.hip)
hipError_t launch_rcb(const int* cell_start, int ncell, int n, int leaf_max,
                      int* cell_list, int* counters, float4* rec, int* perm,
                      float4* rec_tmp, int* perm_tmp, int* leafmark,
                      int4* nodes, float* split, hipStream_t st);
hipError_t launch_leaf_table(const int* leafmark, int* leafidx, int n, int* scan_tmp,
                             int* leaf_start, hipStream_t st);

// plain reference kernels (plain.hip)
hipError_t launch_force_plain(const float4* rec, const int* keys_sorted,
                              const int* cell_start, const int* perm, int n,
                              Geom g, PairParams p, float* out, hipStream_t st);
hipError_t launch_vjp_plain(const float4* rec, const float4* gsorted,
                            const int* keys_sorted, const int* cell_start,
                            const int* perm, int n, Geom g, PairParams p,
                            double* out, hipStream_t st);

// float32 VALU rate probes (probe.hip), measurement only
size_t probe_scratch_bytes();
size_t probe_clock_offset();
int probe_ops_per_iter(int kind);
hipError_t launch_valu_probe(int kind, int waves, int iters, void* scratch,
                             hipStream_t st);

// long-range spectral PM force (pm.hip)
size_t pm_workspace_bytes(int ng, int64_t n);
hipError_t launch_pm_accel(const double* pos, const float* mass, int n, double box, int ng,
                           float sigma, int n_s, void* ws, float* out_acc, hipStream_t st);

// kick / stream (integrate.hip)
hipError_t launch_kick(double* vel, const float* acc, int64_t m, double dt,
                       hipStream_t st);
hipError_t launch_stream(double* pos, const double* vel, int64_t m, double dt,
                         double box, hipStream_t st);
// vel += dt acc, then `streams` times pos += half vel (wrapped)
hipError_t launch_kick_stream(double* pos, double* vel, const float* acc, int64_t m,
                              double dt, double half, int streams, double box,
                              hipStream_t st);
hipError_t launch_kick_adjoint(const double* gv, float* ga, int64_t m,
                               double dt, hipStream_t st);

}  // namespace hsr
