// Pair kernels of the short-range force (Habib et al. 2012, Sec. III,
// Eq. 7):  a_i = sum_j m_j f(s) d,  f(s) = (s + eps)^(-3/2) - poly5(s),
// zero for s >= r_cut^2, and its vector-Jacobian product.
//
// Layout of the work: one wave (64 lanes) per work item, up to 64 targets of
// one run of cells (one cell, or two along z).  Each target lives in
// registers.  The item's sources, the 3 x 3 x (zlen + 2) stencil cells of the
// run, are staged through LDS in rounds, shifted into a frame centred on
// the item, and read back as LDS broadcasts.  Staging drops every source
// farther than r_cut from the bounding box of the item's targets (it could
// only add zeros).  An item of T targets uses k = floor_pow2(64 / T) lanes
// per target: lane t*k + r takes the sources r, r + k, r + 2k, ... and the
// k partial sums of a target are combined with wavefront shuffles at the
// end.  This is the GPU analogue of the paper's contiguous, pre-shifted
// neighbour lists shared by all particles of a leaf (Sec. III, paragraph
// after Eq. 7): equal-length lists, balanced lanes, no gathers in the inner
// loop.
//
// Arithmetic: pair terms in float32 on item-frame coordinates (within 1.5
// cell sides of the item's centre, 2 for a run, so differences of close
// pairs keep their bits); the cut-off is a branch around the pair term;
// each lane accumulates 32 sources in plain float32 and merges them into a
// Kahan-compensated float32 sum; the k lanes of a target are combined with
// float32 two-sums.  No float64 arithmetic.  The grid-force polynomial is evaluated by Horner in
// t = alpha (s + eps) + beta, in [-1, 1] over the cut-off range, whose
// coefficients the host derives in float64 from the caller's s-basis ones.
// The library is compiled without floating-point contraction; every fused
// multiply-add below is written explicitly.
#include "common.h"

namespace hsr {

namespace {

// Launch shape and loop structure, the fastest measured on MI355X for the
// 256^3 clustered workload: high occupancy hides the staging latency, and
// the LDS reads of an unrolled step are issued together before its cut-off
// branches, so that a wave waits on LDS once per step rather than per pair.
constexpr int kT = 256;            // sources per LDS tile (forward)
constexpr int kU = 2;              // sources per lane per unrolled step
constexpr int kMerge = 32;         // sources per lane between compensated merges
constexpr int kMinWaves = 8;       // forward: waves per SIMD the registers allow
constexpr int kVT = 128;           // sources per LDS tile (VJP)
constexpr int kVU = 2;             // VJP sources per lane per unrolled step
constexpr int kVMinWaves = 6;      // VJP: waves per SIMD the registers allow
constexpr int kSeg = 64;           // segment table entries (stencil cells of a run)
static_assert(kMaxSegments <= kSeg, "a run's stencil must fit the segment table");

static_assert(kItemI == kWave, "one item per wave");
static_assert(kT % (kItemI * kU) == 0, "tile must hold whole steps for any split");

__device__ __forceinline__ int wave_incl_scan(int v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int o = __shfl_up(v, d);
        if (lane >= d) v += o;
    }
    return v;
}

__device__ __forceinline__ void kahan_add(float& s, float& c, float x) {
    const float y = x - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
}

// The cut-off is a branch around the pair term rather than a select: the
// compiler moves the whole term under the test's exec mask, which the wave
// skips when a source is out of range for all its targets.  That skip is
// rare (the instruction counters show one reciprocal square root per
// candidate pair-wave); the measured gain, 7% forward and 12% VJP, comes
// from the selects the branch removes.  Bitwise the same results.

// Copy of a wave-uniform constant held in a vector register.  A VALU
// instruction reads at most one scalar register, so an FMA of two scalar
// constants needs one of them in a vector register; the compiler would
// otherwise copy it there again on every loop iteration.
__device__ __forceinline__ float in_vgpr(float s) {
    float v;
    asm("v_mov_b32 %0, %1" : "=v"(v) : "s"(s));
    return v;
}

// Wave-uniform values kept in scalar registers.
__device__ __forceinline__ float uniform(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ float4 uniform(float4 v) {
    return make_float4(uniform(v.x), uniform(v.y), uniform(v.z), uniform(v.w));
}

// Combines the compensated sums (s, c) of the k lanes of each target (lanes
// t*k .. t*k + k - 1, k a power of two) in float32: the exact rounding error
// of each pairwise sum (Knuth's two-sum) joins the compensation terms.
// Every lane of the group ends with the group's value s - c.
__device__ __forceinline__ float group_sum(float s, float c, int k) {
    for (int o = 1; o < k; o <<= 1) {
        const float s2 = __shfl_xor(s, o);
        const float c2 = __shfl_xor(c, o);
        const float t = s + s2;
        const float bb = t - s;
        const float e = (s - (t - bb)) + (s2 - bb);   // s + s2 = t + e exactly
        s = t;
        c = (c + c2) - e;
    }
    return s - c;
}

// Coordinate relative to its own cell's lower corner, shifted by `cells`
// cell sides (a multiple of 1/2) into the item frame with one rounding.
// Targets and sources go through this same expression, so a particle meets
// itself at d = 0.  The item frame is centred on the item: on its cell in x
// and y and on its run of cells in z, so coordinates stay within 1.5 cell
// sides (2 for a run of two cells) and the float32 rounding of separations
// stays small.
__device__ __forceinline__ float frame(float rel, float cells, float Lc) {
    return __builtin_fmaf(cells, Lc, rel);
}

struct Segments {
    int off[kSeg + 1];   // first tile position of each segment
    int start[kSeg];     // first sorted entry of the segment's cell
    int code[kSeg];      // (dx+1) | (dy+1) << 8 | (dz+1) << 16, relative to the
                         // run's first cell
};

// Builds the segment table of one item (one stencil cell per lane: the
// 3 x 3 x (zlen + 2) cells around the item's run of cells) and returns the
// number of sources.  *segoff receives lane q's entry off[q] (the window
// size for lanes past the stencil), a register copy of the table's offsets
// for the segment searches.  Must be called by the whole wave.
__device__ int build_segments(const WorkItem& it, const int* __restrict__ cs,
                              const Geom& g, Segments& sg, int* segoff, int* mycnt,
                              int* mycode) {
    const int lane = threadIdx.x;
    const int N = g.N;
    const int cx = it.cx, cy = it.cy, cz = it.key - (cx * N + cy) * N;
    const int zw = it.zlen + 2;          // window cells along z: 3 or 4
    int cnt = 0, start = 0, code = 0;
    if (lane < 9 * zw) {
        static_assert(kZRun == 2, "zw is 3 or 4");
        const int ab = zw == 3 ? lane / 3 : lane >> 2;
        const int a = ab / 3 - 1, b = ab % 3 - 1, c = lane - ab * zw - 1;
        int x = cx + a, y = cy + b, z = cz + c;
        bool ok = true;
        if (g.periodic) {
            x = x < 0 ? x + N : (x >= N ? x - N : x);
            y = y < 0 ? y + N : (y >= N ? y - N : y);
            z = z < 0 ? z + N : (z >= N ? z - N : z);
        } else {
            ok = x >= 0 && x < N && y >= 0 && y < N && z >= 0 && z < N;
        }
        if (ok) {
            const int key = (x * N + y) * N + z;
            start = cs[key];
            cnt = cs[key + 1] - start;
        }
        code = (a + 1) | ((b + 1) << 8) | ((c + 1) << 16);
    }
    const int incl = wave_incl_scan(cnt);
    const int total = __shfl(incl, kWave - 1);
    *segoff = incl - cnt;
    *mycnt = cnt;
    *mycode = code;
    if (lane < kSeg) {
        sg.off[lane] = incl - cnt;
        sg.start[lane] = start;
        sg.code[lane] = code;
    }
    if (lane == 0) sg.off[kSeg] = total;
    return total;
}

// Gives zero length to the stencil cells that lie wholly beyond the cull
// distance of the target box [lo, hi] and rebuilds the offsets; returns the
// new number of sources.  A cell's box in the item frame is widened by
// 1e-5 cell sides, far above the float32 rounding of a record's frame
// coordinate, so every source of a dropped cell would also fail the
// per-source cull: the kept sources and their order do not change (the
// rounds that stage them do, and with them the grouping of the float32
// partial sums).  Must be called by the whole wave, with each lane's count
// and code from build_segments.
__device__ int cull_segments(const WorkItem& it, Segments& sg, int cnt, int code, float4 lo,
                             float4 hi, float cull2, float Lc, int* segoff) {
    const int lane = threadIdx.x;
    if (cnt > 0) {
        const float a = (float)(code & 255) - 1.0f, b = (float)((code >> 8) & 255) - 1.0f;
        const float c = ((float)((code >> 16) & 255) - 1.0f) - 0.5f * (float)it.zlen;
        const float pad = 1e-5f * Lc;
        const float xl = (a - 0.5f) * Lc - pad, xh = (a + 0.5f) * Lc + pad;
        const float yl = (b - 0.5f) * Lc - pad, yh = (b + 0.5f) * Lc + pad;
        const float zl = c * Lc - pad, zh = (c + 1.0f) * Lc + pad;
        const float gx = fmaxf(fmaxf(xl - hi.x, lo.x - xh), 0.0f);
        const float gy = fmaxf(fmaxf(yl - hi.y, lo.y - yh), 0.0f);
        const float gz = fmaxf(fmaxf(zl - hi.z, lo.z - zh), 0.0f);
        if (gx * gx + gy * gy + gz * gz >= cull2) cnt = 0;
    }
    const int incl = wave_incl_scan(cnt);
    const int total = __shfl(incl, kWave - 1);
    *segoff = incl - cnt;
    if (lane < kSeg) sg.off[lane] = incl - cnt;
    if (lane == 0) sg.off[kSeg] = total;
    return total;
}

// Target record in the item frame: a target in the run's c-th cell is
// shifted as its own record is as a source (c - zlen/2 cell sides along z,
// -1/2 along x and y).  The run's cells are consecutive in key order, so
// their first entries increase along the run.
__device__ __forceinline__ float4 target_in_frame(float4 x, int ki,
                                                  const WorkItem& it,
                                                  const Segments& sg, float Lc) {
    if (ki < 0) return x;
    const int centre = 4 * (it.zlen + 2) + 1;   // segment of the run's cell 0
    int dz = 0;
    for (int c = 1; c < it.zlen; ++c)
        if (ki >= sg.start[centre + c]) dz = c;
    x.x = frame(x.x, -0.5f, Lc);
    x.y = frame(x.y, -0.5f, Lc);
    x.z = frame(x.z, (float)dz - 0.5f * (float)it.zlen, Lc);
    return x;
}

// Record shifted from its own cell into the item frame.
// zc: half the run length, the frame's centre along z in cell sides.
__device__ __forceinline__ float4 shift_into_frame(float4 r, int code, float Lc,
                                                   float zc) {
    // one byte per axis, so that each converts to float in one instruction
    return make_float4(frame(r.x, (float)(code & 255) - 1.5f, Lc),
                       frame(r.y, (float)((code >> 8) & 255) - 1.5f, Lc),
                       frame(r.z, (float)((code >> 16) & 255) - (1.0f + zc), Lc), r.w);
}

static_assert(kVT % (kItemI * kVU) == 0, "VJP tile must hold whole steps");

// Segment holding window position p (0 <= p < total): the last q with
// off[q] <= p.  The offsets do not decrease along the lanes (segoff is lane
// q's off[q]), so the lanes with segoff <= p form a prefix and the answer is
// its highest lane.
__device__ __forceinline__ int segment_of(int segoff, int p) {
    const uint64_t m = __ballot(segoff <= p);
    return 63 - __builtin_clzll(m);
}

// One tile's worth of window positions, loaded into registers: lane l holds
// positions cursor + u * 64 + l, u < TILE / 64.  seg is the segment holding
// cursor.
template <bool WithG, int TILE>
struct Round {
    static constexpr int kPer = TILE / kWave;
    float4 v[kPer];
    float4 g[WithG ? kPer : 1];
    int code[kPer];
    int k[kPer];     // sorted entry, -1 past the end of the window
};

template <bool WithG, int TILE>
__device__ __forceinline__ void load_round(const Segments& sg, int segoff, int seg,
                                           int cursor, int total,
                                           const float4* __restrict__ rec,
                                           const float4* __restrict__ gsorted,
                                           Round<WithG, TILE>& R) {
    constexpr int kPer = TILE / kWave;
    // Segment of each lane's position, slot by slot: the segments that start
    // inside a slot of 64 positions are the only ones that can change it.
    int sp[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int b = cursor + u * kWave;
        int s = seg;
        if (b < total) {
            s = segment_of(segoff, b);
            const int s1 = segment_of(segoff, min(b + kWave, total) - 1);
            for (int q = s + 1; q <= s1; ++q)
                if (b + (int)threadIdx.x >= __builtin_amdgcn_readlane(segoff, q)) s = q;
        }
        sp[u] = s;
    }
    // Every lane loads, so the round's loads issue back to back: a lane past
    // the end of the window re-reads the round's first source and is marked
    // k = -1.  (Loads under per-lane branches were each preceded by a wait
    // for the previous one.)
    const int k0 = sg.start[seg] + (cursor - sg.off[seg]);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int p = cursor + u * kWave + (int)threadIdx.x;
        const int su = sp[u];
        const bool valid = p < total;
        const int k = valid ? sg.start[su] + (p - sg.off[su]) : k0;
        R.code[u] = sg.code[su];
        R.k[u] = valid ? k : -1;
        R.v[u] = rec[k];
        if (WithG) R.g[u] = gsorted[k];
    }
}

// Squared distance from a point to the box [lo, hi].
__device__ __forceinline__ float box_gap2(float4 s, float4 lo, float4 hi) {
    const float gx = fmaxf(fmaxf(lo.x - s.x, s.x - hi.x), 0.0f);
    const float gy = fmaxf(fmaxf(lo.y - s.y, s.y - hi.y), 0.0f);
    const float gz = fmaxf(fmaxf(lo.z - s.z, s.z - hi.z), 0.0f);
    float d = gx * gx;
    d = __builtin_fmaf(gy, gy, d);
    return __builtin_fmaf(gz, gz, d);
}

// Writes the sources of a round that lie within the cull distance of the
// target box into the tile, in window order; returns their number.
// *mixed is set when a kept source's mass differs from mref.
template <bool WithG, int TILE>
__device__ __forceinline__ int compact_round(const Round<WithG, TILE>& R, float4 lo,
                                             float4 hi, float cull2, float Lc,
                                             float zc, float mref, float4* tileA,
                                             float4* tileB, int* tidx,
                                             bool* mixed) {
    constexpr int kPer = TILE / kWave;
    const uint64_t lt = threadIdx.x == 0 ? 0ull : (~0ull >> (64 - threadIdx.x));
    int fill = 0;
    bool other = false;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const float4 sv = shift_into_frame(R.v[u], R.code[u], Lc, zc);
        const bool keep = R.k[u] >= 0 && box_gap2(sv, lo, hi) < cull2;
        other |= keep && sv.w != mref;
        const uint64_t m = __ballot(keep);
        if (keep) {
            const int pos = fill + __popcll(m & lt);
            tileA[pos] = sv;
            if (WithG) tileB[pos] = R.g[u];
            if (tidx) tidx[pos] = R.k[u];
        }
        fill += __popcll(m);
    }
    *mixed = __ballot(other) != 0ull;
    return fill;
}

// Bounding box of the item's targets (lanes without a target hold none; the ks
// lanes of a target hold the same).
__device__ __forceinline__ void target_box(float4 x, bool valid, int ks, float4* lo,
                                           float4* hi) {
    const float inf = __builtin_huge_valf();
    float a = valid ? x.x : inf, b = valid ? x.y : inf, c = valid ? x.z : inf;
    float d = valid ? x.x : -inf, e = valid ? x.y : -inf, f = valid ? x.z : -inf;
    for (int o = ks; o < kWave; o <<= 1) {
        a = fminf(a, __shfl_xor(a, o));
        b = fminf(b, __shfl_xor(b, o));
        c = fminf(c, __shfl_xor(c, o));
        d = fmaxf(d, __shfl_xor(d, o));
        e = fmaxf(e, __shfl_xor(e, o));
        f = fmaxf(f, __shfl_xor(f, o));
    }
    // every lane holds the wave's result: keep it in scalar registers
    *lo = uniform(make_float4(a, b, c, 0.f));
    *hi = uniform(make_float4(d, e, f, 0.f));
}

// Padding source: zero mass, two cell sides below the target box on every
// axis, so s >= 12 Lc^2 > r_cut^2 for every target and the cut-off test
// drops it on both the general and the equal-mass paths.
__device__ __forceinline__ float4 pad_source(float4 lo, float Lc) {
    return make_float4(lo.x - 2.0f * Lc, lo.y - 2.0f * Lc, lo.z - 2.0f * Lc, 0.0f);
}

struct Lanes {
    int ks;       // lanes per target
    int r;        // this lane's residue: it takes sources r, r + ks, ...
    int ki;       // sorted index of this lane's target, -1 if none
};

__device__ __forceinline__ Lanes lane_map(const WorkItem& it) {
    Lanes L;
    L.ks = it.ksplit;
    const int lk = __ffs(L.ks) - 1;
    const int t = threadIdx.x >> lk;
    L.r = threadIdx.x & (L.ks - 1);
    L.ki = t < it.i_count ? it.i_begin + t : -1;
    return L;
}

// Tile positions [0, cntp) with cntp the source count rounded up to whole
// unrolled steps of every lane (a multiple of ks * kU, at most the tile).
__device__ __forceinline__ int padded_count(int cnt, int ks, int unroll = kU) {
    const int step = ks * unroll;
    return (cnt + step - 1) & ~(step - 1);
}

// ------------------------------------------------------------ forward

struct ForceConsts {
    float eps, rc2e, alpha, beta, b0, b1, b2, b3, b4, b5;
};

__device__ __forceinline__ ForceConsts force_consts(const PairParams& P) {
    return ForceConsts{P.eps, P.rc2e, P.alpha, P.beta, P.b[0],
                       P.b[1], P.b[2],  P.b[3], P.b[4], P.b[5]};
}

// Evaluates the tile for this lane: nit sources src[j * stride], j < nit
// (stride = KS when KS > 0, else ks), merging every kMerge partial sums
// into the compensated accumulators.  UNI: every source and target has mass
// mref, so the mass multiplies the partial sums instead of every pair.
template <int KS, bool UNI>
__device__ __forceinline__ void force_tile(const float4* __restrict__ src,
                                           int ks, int nit, float4 xi,
                                           const ForceConsts& c, float mref,
                                           float* s, float* cc) {
    const int st = KS > 0 ? KS : ks;
    const float alpha = in_vgpr(c.alpha), b5 = in_vgpr(c.b5);
    // Two instructions that each read a scalar register do not issue together
    // (4.1 cycles each against 2.4 next to one that reads none), and Horner's
    // run of them is the longest in the loop: its constants take 5 of the 16
    // vector registers that 8 waves per SIMD leave free (2.1M Plummer
    // particles: 1380 -> 1337 us).  The VJP has none to spare at 7 waves.
    const float b4 = in_vgpr(c.b4), b3 = in_vgpr(c.b3), b2 = in_vgpr(c.b2);
    const float b1 = in_vgpr(c.b1), b0 = in_vgpr(c.b0);
    for (int j0 = 0; j0 < nit; j0 += kMerge) {
        float tx = 0.f, ty = 0.f, tz = 0.f;
        const int lim = min(j0 + kMerge, nit);
        for (int jj = j0; jj < lim; jj += kU) {
            float4 cur[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) cur[u] = src[(jj + u) * st];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const float4 pj = cur[u];
                const float dx = pj.x - xi.x;
                const float dy = pj.y - xi.y;
                const float dz = pj.z - xi.z;
                float sp = __builtin_fmaf(dx, dx, c.eps);
                sp = __builtin_fmaf(dy, dy, sp);
                sp = __builtin_fmaf(dz, dz, sp);
                if (sp < c.rc2e) {
                    const float y = __builtin_amdgcn_rsqf(sp);
                    const float t = __builtin_fmaf(sp, alpha, c.beta);
                    float p = __builtin_fmaf(b5, t, b4);
                    p = __builtin_fmaf(p, t, b3);
                    p = __builtin_fmaf(p, t, b2);
                    p = __builtin_fmaf(p, t, b1);
                    p = __builtin_fmaf(p, t, b0);
                    const float y2 = y * y;
                    const float f = __builtin_fmaf(y2, y, -p);
                    const float mf = UNI ? f : pj.w * f;
                    tx = __builtin_fmaf(mf, dx, tx);
                    ty = __builtin_fmaf(mf, dy, ty);
                    tz = __builtin_fmaf(mf, dz, tz);
                }
            }
        }
        if (UNI) {
            tx *= mref;
            ty *= mref;
            tz *= mref;
        }
        kahan_add(s[0], cc[0], tx);
        kahan_add(s[1], cc[1], ty);
        kahan_add(s[2], cc[2], tz);
    }
}

__global__ __launch_bounds__(kWave, kMinWaves) void k_pair_force(
    const WorkItem* __restrict__ items, const int* __restrict__ n_items_dev,
    const float4* __restrict__ rec, const int* __restrict__ cs,
    const int* __restrict__ perm, Geom g, PairParams P,
    float* __restrict__ out_acc) {
    __shared__ Segments sg;
    __shared__ float4 tile[kT];
    if ((int)blockIdx.x >= *n_items_dev) return;
    const WorkItem it = items[blockIdx.x];
    const int lane = threadIdx.x;
    const float Lc = g.Lc_f;
    int segoff, mycnt, mycode;
    build_segments(it, cs, g, sg, &segoff, &mycnt, &mycode);
    const Lanes L = lane_map(it);
    // output slot, loaded now so that its latency overlaps the rounds
    const int dst = perm[L.ki >= 0 ? L.ki : it.i_begin];
    float4 xi = L.ki >= 0 ? rec[L.ki] : make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    xi = target_in_frame(xi, L.ki, it, sg, Lc);
    float4 lo, hi;
    target_box(xi, L.ki >= 0, L.ks, &lo, &hi);
    const int total = cull_segments(it, sg, mycnt, mycode, lo, hi, P.cull2, Lc, &segoff);
    const float mref = uniform(__shfl(xi.w, 0));
    const bool targets_equal = __ballot(L.ki >= 0 && xi.w != mref) == 0ull;
    const float4 pad = pad_source(lo, Lc);
    __syncthreads();

    const ForceConsts c = force_consts(P);
    float s[3] = {0.f, 0.f, 0.f}, cc[3] = {0.f, 0.f, 0.f};

    Round<false, kT> R;
    for (int cursor = 0; cursor < total; cursor += kT) {
        bool mixed;
        const int seg = segment_of(segoff, cursor);
        load_round(sg, segoff, seg, cursor, total, rec, rec, R);
        const int cnt = compact_round(R, lo, hi, P.cull2, Lc, 0.5f * it.zlen, mref,
                                      tile, tile,
                                      nullptr, &mixed);
        const int cntp = padded_count(cnt, L.ks);
        for (int q = cnt + lane; q < cntp; q += kWave) tile[q] = pad;
        __syncthreads();
        const int nit = cntp / L.ks;          // sources per lane in this tile
        const float4* src = tile + L.r;
        const bool uni = targets_equal && !mixed;
        if (L.ks == 1) {
            if (uni) force_tile<1, true>(src, 1, nit, xi, c, mref, s, cc);
            else force_tile<1, false>(src, 1, nit, xi, c, mref, s, cc);
        } else {
            if (uni) force_tile<0, true>(src, L.ks, nit, xi, c, mref, s, cc);
            else force_tile<0, false>(src, L.ks, nit, xi, c, mref, s, cc);
        }
        __syncthreads();
    }
    const float ax = group_sum(s[0], cc[0], L.ks);
    const float ay = group_sum(s[1], cc[1], L.ks);
    const float az = group_sum(s[2], cc[2], L.ks);
    if (L.ki >= 0 && L.r == 0) {
        const int64_t o = 3 * (int64_t)dst;
        out_acc[o] = ax;
        out_acc[o + 1] = ay;
        out_acc[o + 2] = az;
    }
}

// ------------------------------------------------------------ pair counts

// Counts the pairs the force kernel evaluates (sources that survive the
// staging cull, minus the target itself) and those inside the cut-off.
__global__ __launch_bounds__(kWave) void k_pair_count(
    const WorkItem* __restrict__ items, const int* __restrict__ n_items_dev,
    const float4* __restrict__ rec, const int* __restrict__ cs, Geom g,
    PairParams P, unsigned long long* __restrict__ counts) {
    __shared__ Segments sg;
    __shared__ float4 tile[kT];
    __shared__ int tidx[kT];
    if ((int)blockIdx.x >= *n_items_dev) return;
    const WorkItem it = items[blockIdx.x];
    const float Lc = g.Lc_f;
    int segoff, mycnt, mycode;
    const int total = build_segments(it, cs, g, sg, &segoff, &mycnt, &mycode);
    const Lanes L = lane_map(it);
    float4 xi = L.ki >= 0 ? rec[L.ki] : make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    xi = target_in_frame(xi, L.ki, it, sg, Lc);
    float4 lo, hi;
    target_box(xi, L.ki >= 0, L.ks, &lo, &hi);
    __syncthreads();
    unsigned long long inside = 0;
    int kept = 0;
    Round<false, kT> R;
    for (int cursor = 0; cursor < total; cursor += kT) {
        const int seg = segment_of(segoff, cursor);
        load_round(sg, segoff, seg, cursor, total, rec, rec, R);
        bool mixed;
        const int cnt = compact_round(R, lo, hi, P.cull2, Lc, 0.5f * it.zlen, 0.0f,
                                      tile, tile, tidx,
                                      &mixed);
        kept += cnt;
        __syncthreads();
        for (int j = L.r; j < cnt; j += L.ks) {
            const float4 pj = tile[j];
            const float dx = pj.x - xi.x, dy = pj.y - xi.y, dz = pj.z - xi.z;
            float sp = __builtin_fmaf(dx, dx, P.eps);
            sp = __builtin_fmaf(dy, dy, sp);
            sp = __builtin_fmaf(dz, dz, sp);
            inside += (L.ki >= 0 && tidx[j] != L.ki && sp < P.rc2e) ? 1ull : 0ull;
        }
        __syncthreads();
    }
    // evaluated candidates: every kept source except the target itself
    unsigned long long cand =
        (L.ki >= 0 && L.r == 0) ? (unsigned long long)(kept - 1) : 0ull;
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) {
        inside += __shfl_xor(inside, d);
        cand += __shfl_xor(cand, d);
    }
    if (threadIdx.x == 0) {
        atomicAdd(&counts[0], cand);
        atomicAdd(&counts[1], inside);
    }
}

// ------------------------------------------------------------ adjoint

struct VjpConsts {
    ForceConsts f;
    float q0, q1, q2, q3, q4;
};

// Same tile walk as force_tile for the VJP pair term
//   f w + 2 f'(s) (d.w) d,   w = m_k g_j - m_j g_k,
// with 2 f' = -3 (y^5 + q) and q = (2/3) poly'(s): the f' part is summed on
// its own, (y^5 + q)(d.w) d, and enters with the factor -3 at each merge, so
// y^5 + q is one multiply-add.
// UNI: all masses equal mref, so w = mref (g_j - g_k) and mref multiplies
// the partial sums.
template <int KS, bool UNI>
__device__ __forceinline__ void vjp_tile(const float4* __restrict__ srcA,
                                         const float4* __restrict__ srcB,
                                         int ks, int nit, float4 xk, float4 gk,
                                         const VjpConsts& v, float mref,
                                         float* s, float* cc) {
    const int st = KS > 0 ? KS : ks;
    const ForceConsts& c = v.f;
    const float alpha = in_vgpr(c.alpha), b5 = in_vgpr(c.b5), q4 = in_vgpr(v.q4);
    const float mk = xk.w;
    for (int j0 = 0; j0 < nit; j0 += kMerge) {
        float tx = 0.f, ty = 0.f, tz = 0.f;
        float ux = 0.f, uy = 0.f, uz = 0.f;
        const int lim = min(j0 + kMerge, nit);
        for (int jj = j0; jj < lim; jj += kVU) {
            float4 ca[kVU], cb[kVU];
#pragma unroll
            for (int u = 0; u < kVU; ++u) {
                ca[u] = srcA[(jj + u) * st];
                cb[u] = srcB[(jj + u) * st];
            }
#pragma unroll
            for (int u = 0; u < kVU; ++u) {
                const float4 pj = ca[u];
                const float4 gj = cb[u];
                const float dx = pj.x - xk.x;
                const float dy = pj.y - xk.y;
                const float dz = pj.z - xk.z;
                float sp = __builtin_fmaf(dx, dx, c.eps);
                sp = __builtin_fmaf(dy, dy, sp);
                sp = __builtin_fmaf(dz, dz, sp);
                if (sp < c.rc2e) {
                    const float y = __builtin_amdgcn_rsqf(sp);
                    const float t = __builtin_fmaf(sp, alpha, c.beta);
                    float p = __builtin_fmaf(b5, t, c.b4);
                    p = __builtin_fmaf(p, t, c.b3);
                    p = __builtin_fmaf(p, t, c.b2);
                    p = __builtin_fmaf(p, t, c.b1);
                    p = __builtin_fmaf(p, t, c.b0);
                    float q = __builtin_fmaf(q4, t, v.q3);
                    q = __builtin_fmaf(q, t, v.q2);
                    q = __builtin_fmaf(q, t, v.q1);
                    q = __builtin_fmaf(q, t, v.q0);
                    const float y2 = y * y;
                    const float y3 = y2 * y;
                    const float f = y3 - p;
                    const float u = __builtin_fmaf(y3, y2, q);    // y^5 + q
                    float wx, wy, wz;
                    if (UNI) {
                        wx = gj.x - gk.x;
                        wy = gj.y - gk.y;
                        wz = gj.z - gk.z;
                    } else {
                        // two separately rounded products, so that the self
                        // pair (j = k) gives w = 0 exactly
                        wx = mk * gj.x - pj.w * gk.x;
                        wy = mk * gj.y - pj.w * gk.y;
                        wz = mk * gj.z - pj.w * gk.z;
                    }
                    float dw = dx * wx;
                    dw = __builtin_fmaf(dy, wy, dw);
                    dw = __builtin_fmaf(dz, wz, dw);
                    const float cd = u * dw;
                    tx = __builtin_fmaf(f, wx, tx);
                    ty = __builtin_fmaf(f, wy, ty);
                    tz = __builtin_fmaf(f, wz, tz);
                    ux = __builtin_fmaf(cd, dx, ux);
                    uy = __builtin_fmaf(cd, dy, uy);
                    uz = __builtin_fmaf(cd, dz, uz);
                }
            }
        }
        tx = __builtin_fmaf(-3.0f, ux, tx);
        ty = __builtin_fmaf(-3.0f, uy, ty);
        tz = __builtin_fmaf(-3.0f, uz, tz);
        if (UNI) {
            tx *= mref;
            ty *= mref;
            tz *= mref;
        }
        kahan_add(s[0], cc[0], tx);
        kahan_add(s[1], cc[1], ty);
        kahan_add(s[2], cc[2], tz);
    }
}

// dL/dx_k = sum_j [f w + 2 f'(s) (d.w) d],  w = m_k g_j - m_j g_k,
// the transpose of the Jacobian of the pair term applied to the cotangents.
__global__ __launch_bounds__(kWave, kVMinWaves) void k_pair_vjp(
    const WorkItem* __restrict__ items, const int* __restrict__ n_items_dev,
    const float4* __restrict__ rec, const float4* __restrict__ gsorted,
    const int* __restrict__ cs, const int* __restrict__ perm, Geom g,
    PairParams P, double* __restrict__ out_grad) {
    __shared__ Segments sg;
    __shared__ float4 tileA[kVT];
    __shared__ float4 tileB[kVT];
    if ((int)blockIdx.x >= *n_items_dev) return;
    const WorkItem it = items[blockIdx.x];
    const int lane = threadIdx.x;
    const float Lc = g.Lc_f;
    int segoff, mycnt, mycode;
    build_segments(it, cs, g, sg, &segoff, &mycnt, &mycode);
    const Lanes L = lane_map(it);
    // output slot, loaded now so that its latency overlaps the rounds
    const int dst = perm[L.ki >= 0 ? L.ki : it.i_begin];
    float4 xk = L.ki >= 0 ? rec[L.ki] : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 gk = L.ki >= 0 ? gsorted[L.ki] : make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    xk = target_in_frame(xk, L.ki, it, sg, Lc);
    float4 lo, hi;
    target_box(xk, L.ki >= 0, L.ks, &lo, &hi);
    const int total = cull_segments(it, sg, mycnt, mycode, lo, hi, P.cull2, Lc, &segoff);
    const float mref = uniform(__shfl(xk.w, 0));
    const bool targets_equal = __ballot(L.ki >= 0 && xk.w != mref) == 0ull;
    const float4 pad = pad_source(lo, Lc);
    __syncthreads();

    const VjpConsts v{force_consts(P), P.dq3[0], P.dq3[1], P.dq3[2], P.dq3[3],
                      P.dq3[4]};
    float s[3] = {0.f, 0.f, 0.f}, cc[3] = {0.f, 0.f, 0.f};

    Round<true, kVT> R;
    for (int cursor = 0; cursor < total; cursor += kVT) {
        bool mixed;
        const int seg = segment_of(segoff, cursor);
        load_round(sg, segoff, seg, cursor, total, rec, gsorted, R);
        const int cnt = compact_round(R, lo, hi, P.cull2, Lc, 0.5f * it.zlen, mref,
                                      tileA, tileB,
                                      nullptr, &mixed);
        const int cntp = padded_count(cnt, L.ks, kVU);
        for (int q = cnt + lane; q < cntp; q += kWave) {
            tileA[q] = pad;
            tileB[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        __syncthreads();
        const int nit = cntp / L.ks;
        const float4* srcA = tileA + L.r;
        const float4* srcB = tileB + L.r;
        const bool uni = targets_equal && !mixed;
        if (L.ks == 1) {
            if (uni) vjp_tile<1, true>(srcA, srcB, 1, nit, xk, gk, v, mref, s, cc);
            else vjp_tile<1, false>(srcA, srcB, 1, nit, xk, gk, v, mref, s, cc);
        } else {
            if (uni) vjp_tile<0, true>(srcA, srcB, L.ks, nit, xk, gk, v, mref, s, cc);
            else vjp_tile<0, false>(srcA, srcB, L.ks, nit, xk, gk, v, mref, s, cc);
        }
        __syncthreads();
    }
    const float gx = group_sum(s[0], cc[0], L.ks);
    const float gy = group_sum(s[1], cc[1], L.ks);
    const float gz = group_sum(s[2], cc[2], L.ks);
    if (L.ki >= 0 && L.r == 0) {
        // float32 result stored in the float64 output (a conversion only)
        const int64_t o = 3 * (int64_t)dst;
        out_grad[o] = (double)gx;
        out_grad[o + 1] = (double)gy;
        out_grad[o + 2] = (double)gz;
    }
}

}  // namespace

hipError_t launch_pair_force(const WorkItem* items, int max_items,
                             const int* n_items_dev, const float4* rec,
                             const int* cell_start, const int* perm, Geom g,
                             PairParams p, float* out_acc, hipStream_t st) {
    if (max_items <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pair_force, dim3(max_items), dim3(kWave), 0, st, items,
                       n_items_dev, rec, cell_start, perm, g, p, out_acc);
    return hipGetLastError();
}

hipError_t launch_pair_count(const WorkItem* items, int max_items,
                             const int* n_items_dev, const float4* rec,
                             const int* cell_start, Geom g, PairParams p,
                             unsigned long long* counts, hipStream_t st) {
    if (max_items <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pair_count, dim3(max_items), dim3(kWave), 0, st, items,
                       n_items_dev, rec, cell_start, g, p, counts);
    return hipGetLastError();
}

hipError_t launch_pair_vjp(const WorkItem* items, int max_items,
                           const int* n_items_dev, const float4* rec,
                           const float4* gsorted, const int* cell_start,
                           const int* perm, Geom g, PairParams p,
                           double* out_grad, hipStream_t st) {
    if (max_items <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pair_vjp, dim3(max_items), dim3(kWave), 0, st, items,
                       n_items_dev, rec, gsorted, cell_start, perm, g, p,
                       out_grad);
    return hipGetLastError();
}

}  // namespace hsr
