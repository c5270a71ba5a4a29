// Per-agent device code of the ORCA step (gfx950), shared by the single-scene
// and the batched kernels.  One lane per agent:
//
//   kNN      exact k nearest (squared distance in FP64 without contraction,
//            ties by caller index) over the rows of the cell stencil, each row
//            one contiguous range of the cell-ordered copy
//   ORCA     one half-plane per neighbour (Fig. 1(b,c), Sec. 3.1), computed
//            without divergent branches: the arc, leg and overlap forms are
//            all evaluated and selected, so pedestrians and vehicles run the
//            same instructions (Sec. 3.1)
//   LP2      incremental closest-point LP over the half-planes and the speed
//            disc (Sec. 3)
//   LP3      least-penetration fallback when LP2 is infeasible (Sec. 3)
//   update   v' = LP result, p' = p + v' dt, written in caller order
//
// The half-planes of a lane live in LDS, one column per lane
// ([k][block] float4 = (q.x, q.y, d.x, d.y)), so the rolled LP loops index
// them dynamically without scratch memory.  Header-only: every translation
// unit instantiates the templates it launches.
#pragma once

#include "orca_internal.h"

#include <limits.h>
#include <math.h>

// Multiply-adds are fused within one expression only (C's FP_CONTRACT),
// never across statements: every instantiation of these templates (plain,
// batched, capped, adjoint recomputation) then rounds alike, which keeps
// their results equal bit for bit.
#pragma clang fp contract(on)

namespace orca {
namespace dev {

__device__ __forceinline__ float det2(float ax, float ay, float bx, float by)
{
    return ax * by - ay * bx;
}

__device__ __forceinline__ double det2(double ax, double ay, double bx, double by)
{
    return ax * by - ay * bx;
}

// The LP runs in float (LP2 over the agent's lines) or in double (LP3's
// sub-problems): these pick the operation of the scalar type.
__device__ __forceinline__ float lp_sqrt(float v) { return sqrtf(v); }
__device__ __forceinline__ double lp_sqrt(double v) { return sqrt(v); }
__device__ __forceinline__ float lp_abs(float v) { return fabsf(v); }
__device__ __forceinline__ double lp_abs(double v) { return fabs(v); }
__device__ __forceinline__ float lp_min(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ double lp_min(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ float lp_max(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double lp_max(double a, double b) { return fmax(a, b); }

template <class S>
struct LpVec;
template <>
struct LpVec<float> {
    using T = float4;
};
template <>
struct LpVec<double> {
    using T = double4;
};


// Squared distance in double from FP32 positions, each operation rounded
// separately (no fused multiply-add): the neighbour order is defined on it.
__device__ __forceinline__ double nb_key(float xi, float yi, float xj, float yj)
{
#pragma clang fp contract(off)
    const double dx = (double)xj - (double)xi;
    const double dy = (double)yj - (double)yi;
    return dx * dx + dy * dy;
}

// ---------------------------------------------------------------------------
// Exact k-nearest selection.
//
// Candidates are taken row by row from the cell stencil; each row is clipped
// to the chord of the neighbour circle at the row's nearest y (FP32, of a circle
// widened far beyond its rounding, see CellDisc), so every agent with
// key < R_n^2 is visited.
//
// Pass 1 counts the in-range candidates of the lane in kBins bins of equal
// area (bin = floor(key * kBins / R_n^2), monotone in the key); a group of
// candidates adds to 4-bit fields of one 64-bit register, which are then
// widened into the 8-bit fields of two (even and odd bins).  The first bin
// b* at which the
// running count reaches k is the threshold: every candidate of a lower bin is
// among the k nearest and the rest of the k nearest lie in bin b*.
// Pass 2 visits only the circle that holds bins <= b* and appends their
// candidates to the lane's LDS column; a sorting network over registers then
// orders them.  Buffer entries are (float(key) bits << 32 | cell-order
// position): a strict order of the FP32-rounded keys implies the same order
// of the FP64 keys (rounding is monotone); equal FP32 keys among the entries
// that decide the result are resolved by an insertion pass that recomputes
// the FP64 keys and then compares the caller indices.
// Where the bins hold more than the buffer, or the counts could overflow (> 255
// in range), a smaller circle is counted.  What kRecounts circles do not settle
// (agents at one distance) is selected by repeated minimum, exact and far slower:
// one such lane holds the whole call (131,072 agents, 2 /m^2, k 20, R_n 5 m, the
// first call on a workspace: 1950 us when all these lanes took it, 390 now).
// ---------------------------------------------------------------------------
constexpr int kBins = 16;
constexpr int kRecounts = 3;

template <int K>
struct KnnShape {
    static constexpr int kSlots = K < 8 ? 8 : K;  // 16-byte LDS slots per lane
    static constexpr int kCap = 2 * kSlots;       // buffer entries per lane
};

// Words of the sorting network for K nearest.
template <int K>
struct SortNet {
    static constexpr int N = K <= 8 ? 16 : (K <= 24 ? 32 : 64);
};

// Each agent keeps from step to step a radius that is expected to hold its K
// nearest and little more (never a part of the result: a circle that holds
// fewer is widened, one that holds too many is cut by counting).  Where the
// entries of a circle were sorted, it is the distance of the agent kMore
// places behind the K-th: a step changes who is inside by a few.  (A margin on
// the K-th distance, two speed steps, holds 32 and more in a crossing's dense
// parts: counted and scanned again there, 430 us per step over steps 10-110 of
// the 1M crossing.  By number, with kMore at 2, 3, 4 and 5: 382, 363, 362 and
// 363 us.)  Where the buffer is small for K, three sevenths of its room: more fill
// it too often, fewer are too few too often (262,144 agents walking, us per step, at
// kMore 2, 3 and 4: k 10 154, 142, 148 at 1.0 /m^2; k 12 151, 139, 136; k 8 156, 158 and 3
// the most, standing 133 and 149; k 4 115, 108, 109, standing 85, 92, 93; lists of
// those standing, k 10, at 3 and 4: 90.6 and 102.0 at 1.0 /m^2, 83.9 and 82.6 at 0.26,
// where R_n holds little more).
constexpr int kKeptMore = 4;
template <int K>
struct KeptShape {
    static constexpr int kFit = SortNet<K>::N < KnnShape<K>::kCap ? SortNet<K>::N
                                                                  : KnnShape<K>::kCap - 1;
    static constexpr int kRoom = (kFit - K - 1) * 3 / 7;
    static constexpr int kWant = K <= kBriefList ? kKeptMore - 1 : kKeptMore;
    static constexpr int kMore = kRoom < kWant ? kRoom : kWant;
};

// Hard lines of a vehicle's own motion limits: the acceleration octagon (see
// accel_line) and the two sides of the heading wedge (see turn_wedge).
constexpr int kAccLines = 8;
constexpr int kTurnLines = 2;

// Entry e of lane `tid` inside a [slot][BLOCK] float4 array viewed as u64.
// With several wavefronts per block, both entries of a 16-byte slot stay in
// the lane's own column tid: the buffer shares the LDS of the half-planes,
// and the wavefronts of a block run independently, so a lane that has
// reached its half-planes may only overwrite its own column (an
// [entry][BLOCK] layout would place a lane's entries in other lanes'
// columns, where a wavefront already writing half-planes corrupts one still
// selecting).  A block of one wavefront takes that [entry][BLOCK] layout
// (one address operation per entry instead of four): its lanes run in
// lockstep, so every lane has read its entries before any lane writes a
// half-plane, and lane_order() keeps the compiler from moving an LDS write
// across those phase boundaries.
template <int BLOCK>
__device__ __forceinline__ int buf_idx(int e, int tid)
{
    if (BLOCK == kWave) return e * BLOCK + tid;
    return (e >> 1) * (2 * BLOCK) + 2 * tid + (e & 1);
}

// Orders this lane's LDS accesses before and after it as seen by the other
// lanes of its wavefront (a compiler barrier; a one-wavefront block needs
// nothing more, its lanes execute together).
template <int BLOCK>
__device__ __forceinline__ void lane_order()
{
    if (BLOCK == kWave) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Entry = (float(key) bits << 32) | (bin << 28) | cell-order position; the
// position needs 28 bits (at most 2^28 agents), the bin field is only read
// by the single-pass selection below.
constexpr uint32_t kPosBits = 28;
constexpr uint32_t kPosMask = (1u << kPosBits) - 1u;

__device__ __forceinline__ uint64_t pack_entry(double key, uint32_t t, uint32_t bin = 0u)
{
    return ((uint64_t)__float_as_uint((float)key) << 32) | (uint64_t)((bin << kPosBits) | t);
}

__device__ __forceinline__ uint32_t entry_pos(uint64_t e) { return (uint32_t)e & kPosMask; }
__device__ __forceinline__ uint32_t entry_bin(uint64_t e) { return (uint32_t)e >> kPosBits; }

// Strict (key, caller index) order of two buffer entries.
__device__ __forceinline__ bool entry_less(uint64_t ea, uint64_t eb, const float2 *__restrict__ s0,
                                           const float4 *__restrict__ s1, float xi, float yi)
{
    const uint32_t ha = (uint32_t)(ea >> 32), hb = (uint32_t)(eb >> 32);
    if (ha != hb) return ha < hb;
    const float2 ca = s0[entry_pos(ea)];
    const float2 cb = s0[entry_pos(eb)];
    const double ka = nb_key(xi, yi, ca.x, ca.y);
    const double kb = nb_key(xi, yi, cb.x, cb.y);
    if (ka != kb) return ka < kb;
    return tag_index(s1[entry_pos(ea)].z) < tag_index(s1[entry_pos(eb)].z);
}

// Candidates loaded per group by one lane.
#ifndef ORCA_SCAN_UNROLL
#define ORCA_SCAN_UNROLL 8
#endif
constexpr int kScanUnroll = ORCA_SCAN_UNROLL;
static_assert(kScanUnroll <= kScanPad, "candidate groups may read at most kScanPad past s0");

// A group of positions, two to a 16-byte load (of 8-byte alignment).
__device__ __forceinline__ void load_group(const float2 *p, float2 (&c)[kScanUnroll])
{
    typedef float Pair __attribute__((ext_vector_type(4), aligned(8)));
    static_assert(kScanUnroll % 2 == 0, "positions are loaded in pairs");
    const Pair *pp = (const Pair *)p;
#pragma unroll
    for (int q = 0; q < kScanUnroll / 2; ++q) {
        const Pair v = pp[q];
        c[2 * q] = make_float2(v.x, v.y);
        c[2 * q + 1] = make_float2(v.z, v.w);
    }
}

struct NoGroupEnd {
    __device__ __forceinline__ void operator()() const {}
};

// A disc in cell units around a point: the cell (cx, cy) that holds the
// centre, the centre's place (fx, fy) in it, and the radius rp.  The cell and
// the place are formed in double; rp is widened by a relative 1e-6 and by
// 1e-4 cells, so that everything derived from it in FP32 (whose rounding is a
// few 1e-7 of rp, and a few 1e-7 rp^2 in a half chord squared, against the
// widening's 2e-4 rp + 2e-6 rp^2) covers the exact disc.  Which cells are
// scanned changes no result, only the test of each key does.  (Rows and
// chords in double, two conversions, a square root and two floors each,
// were a third of the scan's instructions.)
struct CellDisc {
    int cx, cy;
    float fx, fy, rp;
};

__device__ __forceinline__ CellDisc cell_disc(const GridMeta &g, double xd, double yd, double r2)
{
    CellDisc d;
    // the bounds keep every sum below in int's range, and map NaN to a bound
    const double ux = fmin(fmax((xd - (double)g.x0) * g.inv_cs, -1e9), 1e9);
    const double uy = fmin(fmax((yd - (double)g.y0) * g.inv_cs, -1e9), 1e9);
    const double cx = floor(ux), cy = floor(uy);
    d.cx = (int)cx;
    d.cy = (int)cy;
    d.fx = (float)(ux - cx);
    d.fy = (float)(uy - cy);
    d.rp = fminf((float)(sqrt(r2) * g.inv_cs) * 1.000001f + 1e-4f, 1e9f);
    return d;
}

__device__ __forceinline__ int clamp_cell(int c, int n) { return max(min(c, n - 1), 0); }

// Grid rows that can hold an agent of the disc.
__device__ __forceinline__ void row_span(const GridMeta &g, const CellDisc &d, int &ya, int &yb)
{
    ya = clamp_cell(d.cy + (int)floorf(d.fy - d.rp), g.ny);
    yb = clamp_cell(d.cy + (int)floorf(d.fy + d.rp), g.ny);
}

// Row yy's cells that meet the disc's chord, as the offsets of the two
// `start` entries that bound their range; false when the chord misses the
// row (the centre's column then).
__device__ __forceinline__ bool row_cells(const GridMeta &g, const CellDisc &d, int yy, int &ia,
                                          int &ib)
{
    const float o = (float)(yy - d.cy);
    const float dy = fmaxf(fmaxf(o - d.fy, d.fy - o - 1.0f), 0.0f);
    const float h2 = d.rp * d.rp - dy * dy;
    const bool meets = h2 > 0.0f;
    // the hardware square root: 1 ulp is far below the widening
    const float hw = meets ? __builtin_amdgcn_sqrtf(h2) : 0.0f;
    const int row = g.cell_base + yy * g.nx;
    ia = row + clamp_cell(d.cx + (int)floorf(d.fx - hw), g.nx);
    ib = row + clamp_cell(d.cx + (int)floorf(d.fx + hw), g.nx) + 1;
    return meets;
}

// Cell-order range of row yy clipped to the chord; false when empty.
__device__ __forceinline__ bool row_range(const GridMeta &g, const uint32_t *__restrict__ start,
                                          const CellDisc &d, int yy, uint32_t &a, uint32_t &b)
{
    int ia, ib;
    if (!row_cells(g, d, yy, ia, ib)) return false;
    a = start[ia];
    b = start[ib];
    if (b > g.seg_end) b = g.seg_end;  // defensive: stay inside the scene
    return a < b;
}

// Sorting network over N (a power of two) 64-bit keys held in registers,
// ascending; every index is a compile-time constant.
// Largest fixed-point sort key: 26 bits above the 6-bit buffer slot.
constexpr uint32_t kSortKeyMax = (1u << 26) - 1u;

template <int N>
__device__ __forceinline__ void cas(uint32_t (&e)[N], int i, int l)
{
    const uint32_t a = e[i], b = e[l];
    e[i] = a < b ? a : b;
    e[l] = a < b ? b : a;
}

// Batcher's odd-even merge sort (191 comparators for 32 keys against the
// bitonic network's 240); the loops run at compile time.
template <int N>
__device__ __forceinline__ void sort_network(uint32_t (&e)[N])
{
#pragma unroll
    for (int p = 1; p < N; p += p) {
#pragma unroll
        for (int k = p; k > 0; k /= 2) {
#pragma unroll
            for (int j = k % p; j + k < N; j += k + k) {
#pragma unroll
                for (int i = 0; i < k; ++i) {
                    if ((i + j) / (p + p) == (i + j + k) / (p + p)) cas<N>(e, i + j, i + j + k);
                }
            }
        }
    }
}

// Visits every candidate in the grid rows and chords of the circle of
// squared radius r2 around (xd, yd), row by row and in cell order within a
// row, in groups of kScanUnroll as group(c, t0, e): c[q] = s0[t0 + q], a
// member valid while t0 + q < e, the end of its row.  A group always loads
// all its members (the last one of a row reads up to kScanUnroll - 1
// entries past the row's end, inside s0 and its padding), so the visitor
// runs without a remainder loop and can stay branch-free.
//
// The loop runs over groups, not rows, with the memory one step ahead of
// the arithmetic: the next group -- the next one of the same row or the
// first one of the next row -- is loaded before the current one is visited,
// and a row's range is loaded from `start` one group before it is entered.
// Every lane issues both loads on every pass (a lane that stays in its row
// loads the same entries again), so the number of loads in flight is the
// same on every path and each wait covers only the data it needs.  In a
// dense crowd a row chord holds fewer candidates than one group, so a loop
// per row would wait for the memory at every row.  A row whose range turns
// out empty costs one group of invalid members.  Lanes step through their
// own rows, so a wave runs as many groups as its busiest lane.
template <class H>
__device__ __forceinline__ void scan_disc_groups(const GridMeta &g,
                                                 const uint32_t *__restrict__ start,
                                                 const float2 *__restrict__ s0, double xd,
                                                 double yd, double r2, H &&group)
{
    const CellDisc disc = cell_disc(g, xd, yd, r2);
    int yr, yb;
    row_span(g, disc, yr, yb);
    // The range of row yr is loaded into one of two register pairs while the
    // other pair, loaded a pass earlier, is consumed (the two swap roles every
    // pass, so a load never lands in a register that is still being read);
    // rm: row yr's chord meets the row; (ia, ib): its `start` offsets.
    int ia, ib;
    bool rm = row_cells(g, disc, yr, ia, ib);
    uint32_t pa[2], pb[2];
    pa[0] = start[ia];
    pb[0] = start[ib];
    // the group after [t, t + kScanUnroll) of row [.., e): the next one of
    // the row, else the first one of row yr, whose range (pair P) is then
    // consumed and row yr + 1 requested; pair 1 - P is (re)loaded with the
    // range of the row requested now; false when no row is left
    auto next_group = [&](int P, uint32_t t, uint32_t e, uint32_t &tn, uint32_t &en) -> bool {
        const bool stay = t + kScanUnroll < e;
        bool live = true;
        if (stay) {
            tn = t + kScanUnroll;
            en = e;
        } else {
            live = yr <= yb;
            tn = pa[P];
            en = pb[P] < g.seg_end ? pb[P] : g.seg_end;  // defensive: stay inside the scene
            if (!rm || !(tn < en)) en = tn;              // an empty row: no valid member
            ++yr;
            if (yr <= yb) rm = row_cells(g, disc, yr, ia, ib);
        }
        pa[1 - P] = start[ia];
        pb[1 - P] = start[ib];
        return live;
    };
    // two register groups used in turn, so no group is copied; components a
    // visitor does not read are never loaded
    float2 c[kScanUnroll], d[kScanUnroll];
    uint32_t t0 = 0, e0 = 0;
    next_group(0, 0u, 0u, t0, e0);  // row yr exists: yr <= yb here
    load_group(s0 + t0, c);
    for (;;) {
        uint32_t t1, e1;
        const bool more1 = next_group(1, t0, e0, t1, e1);
        load_group(s0 + (more1 ? t1 : t0), d);
        // keep the loads ahead of the visit (the scheduler would otherwise
        // move them next to their use)
        __builtin_amdgcn_sched_barrier(0);
        group(c, t0, e0);
        if (!more1) break;
        const bool more2 = next_group(0, t1, e1, t0, e0);
        load_group(s0 + (more2 ? t0 : t1), c);
        __builtin_amdgcn_sched_barrier(0);
        group(d, t1, e1);
        if (!more2) break;
    }
    // the loads of the last pass are read on the way out too, so that the
    // compiler keeps each prefetch where it is written instead of moving it
    // behind the exit test, next to its use
#pragma unroll
    for (int q = 0; q < kScanUnroll; ++q)
        asm volatile("" ::"v"(c[q].x), "v"(c[q].y), "v"(d[q].x), "v"(d[q].y));
}

// The same scan with a visitor per candidate: visit(c, t, valid) for each
// member of a group, then group_end().
template <class F, class G = NoGroupEnd>
__device__ __forceinline__ void scan_disc(const GridMeta &g, const uint32_t *__restrict__ start,
                                          const float2 *__restrict__ s0, double xd, double yd,
                                          double r2, F &&visit, G &&group_end = G())
{
    scan_disc_groups(g, start, s0, xd, yd, r2,
                     [&](const float2 (&c)[kScanUnroll], uint32_t t0, uint32_t e) {
#pragma unroll
                         for (int q = 0; q < kScanUnroll; ++q) visit(c[q], t0 + q, t0 + q < e);
                         group_end();
                     });
}

// Orders the `take` entries of the lane's buffer, its own agent's (position
// spos, key 0) among them, and leaves the nearest K others at least, ascending,
// in entries [0, min(take - 1, K)).
//
// A sorting network in registers when the entries fit it, over 32-bit words
// (the FP32 key in 26-bit fixed point of r2c, above the entry's buffer
// slot); the nearest entries are then gathered by slot.  The fixed-point key
// is non-decreasing in the FP32 key, which is non-decreasing in the FP64 key,
// so distinct fixed-point keys are in (FP64 key) order; a tie among the
// entries that decide the result needs the (FP64 key, caller index) order
// of entry_less, left to the insertion pass (the buffer is then untouched).
// `next` becomes the distance of the entry kMore places behind the K-th
// where there is one.  Without a tie the own entry, key 0, comes first.  Loads and stores are not
// bounded by the lane's count: the words past it sort last and in slot order
// (also behind a key of kSortKeyMax, whose slot is lower), so the first K + 1
// words name slots below kCap.
template <int K, int BLOCK>
__device__ __forceinline__ void sort_entries(const float2 *__restrict__ s0,
                                             const float4 *__restrict__ s1, float xi, float yi,
                                             uint32_t spos, uint64_t *buf, int tid, uint32_t take,
                                             double r2c, float &next)
{
    constexpr int N = SortNet<K>::N;
    constexpr int kCap = KnnShape<K>::kCap;
    static_assert(N <= 64, "buffer slots must fit six bits");
    static_assert(K + 1 <= N && K + 1 <= kCap, "room for K entries and the lane's own");
    if (take <= (uint32_t)N) {
        const float qscale = 67108864.0f / (float)r2c;  // 2^26 / r2c
        uint32_t e[N];
#pragma unroll
        for (int p = 0; p < N; ++p) {
            if (p < kCap) {
                const float fk = __uint_as_float((uint32_t)(buf[buf_idx<BLOCK>(p, tid)] >> 32));
                // clamp in the integer domain: the FP32 product reaches
                // 2^26 for keys within a few 1e-8 (relative) below r2c,
                // and 2^26 - 1 has no FP32 value to clamp to
                const uint32_t q = min((uint32_t)(fk * qscale), kSortKeyMax);
                e[p] = (p < (int)take ? q << 6 : ~63u) | (uint32_t)p;
            } else {
                e[p] = ~63u | (uint32_t)p;
            }
        }
        sort_network<N>(e);
        bool tie = false;
#pragma unroll
        for (int p = 0; p + 1 < N; ++p)
            tie = tie || (p <= K && p + 1 < (int)take && (e[p] >> 6) == (e[p + 1] >> 6));
        if (!tie) {
            uint64_t got[K];
#pragma unroll
            for (int p = 0; p < K; ++p) got[p] = buf[buf_idx<BLOCK>((int)(e[p + 1] & 63u), tid)];
            constexpr int kAt = K + KeptShape<K>::kMore;
            if (kAt < (int)take)
                next = sqrtf(__uint_as_float(
                    (uint32_t)(buf[buf_idx<BLOCK>((int)(e[kAt] & 63u), tid)] >> 32)));
#pragma unroll
            for (int p = 0; p < K; ++p) buf[buf_idx<BLOCK>(p, tid)] = got[p];
            return;
        }
    }
    // drop the own entry: those after it move up one slot
    uint32_t w = 0;
    for (uint32_t e = 0; e < take; ++e) {
        const uint64_t ent = buf[buf_idx<BLOCK>((int)e, tid)];
        buf[buf_idx<BLOCK>((int)w, tid)] = ent;
        w += entry_pos(ent) != spos ? 1u : 0u;
    }
    for (int p = 1; p < (int)take - 1; ++p) {
        const uint64_t e = buf[buf_idx<BLOCK>(p, tid)];
        int q = p - 1;
        while (q >= 0) {
            const uint64_t f = buf[buf_idx<BLOCK>(q, tid)];
            if (!entry_less(e, f, s0, s1, xi, yi)) break;
            buf[buf_idx<BLOCK>(q + 1, tid)] = f;
            --q;
        }
        buf[buf_idx<BLOCK>(q + 1, tid)] = e;
    }
    // (an estimate by number alone could hold too few, and would then be made
    // again from the same entries, call after call: 131,072 agents, 2 /m^2, k 20 and
    // R_n 5 m, 365 us a step, 252 so)
    constexpr int kAt = K + KeptShape<K>::kMore - 1;
    if (kAt < (int)take - 1)
        next = sqrtf(__uint_as_float((uint32_t)(buf[buf_idx<BLOCK>(kAt, tid)] >> 32)));
}

// Collects into the lane's buffer a set that holds its K nearest within R_n
// (or all, when there are fewer) and its own agent; returns the number of
// entries, or 0 when no such set fits the buffer, and the squared radius r2c
// that bounds their keys (then a circle that holds K at least).  rg2
// (<= R_n^2) is a guess of a squared radius that
// holds at least K candidates; with `kept` (from the previous step) it is
// expected to hold little more.  A circle that holds fewer than K is widened
// to the whole neighbour circle, so the result never depends on the guess.
//
// The lane's own agent is scanned as any other (key 0, bin 0), which keeps
// the test for it out of the loops.
template <int K, int BLOCK>
__device__ __forceinline__ uint32_t knn_collect(const GridMeta &g,
                                                const uint32_t *__restrict__ start,
                                                const float2 *__restrict__ s0, float xi, float yi,
                                                uint64_t *buf, int tid, double rg2, bool kept,
                                                double &r2c)
{
    constexpr int kCap = KnnShape<K>::kCap;
    const double xd = xi, yd = yi;
    r2c = rg2 < g.rn2 ? rg2 : g.rn2;
    // A kept circle: every candidate in range is stored, and that is the set
    // when all fit.  (The counting pass below, with a bin and two counters per
    // candidate, is needed only to cut a circle that holds too many.)
    constexpr uint32_t kFit = (uint32_t)KeptShape<K>::kFit;
    if (kept) {
        uint32_t n = 0;
        scan_disc_groups(
            g, start, s0, xd, yd, r2c,
            [&](const float2 (&c)[kScanUnroll], uint32_t t0, uint32_t e) {
                // the keys of the whole group first (independent of one
                // another, so their FP64 chains interleave), then the buffer
                // in member order
                double key[kScanUnroll];
#pragma unroll
                for (int q = 0; q < kScanUnroll; ++q) key[q] = nb_key(xi, yi, c[q].x, c[q].y);
                // branch-free, so that the candidates of a group form one
                // block: every candidate is written at the next free slot
                // and kept only when in range; once the buffer is full the
                // writes land on its last slot, the only one they can
                // overwrite
#pragma unroll
                for (int q = 0; q < kScanUnroll; ++q) {
                    const int slot = (int)min(n, (uint32_t)(kCap - 1));
                    buf[buf_idx<BLOCK>(slot, tid)] = pack_entry(key[q], t0 + q);
                    n += t0 + q < e && key[q] < r2c ? 1u : 0u;
                }
            });
        if (n <= kFit && (n > (uint32_t)K || !(r2c < g.rn2))) return n;
        // too few: a circle that should hold about half as many again as is
        // wanted, and still all of them in the buffer; all of R_n after that
        // (to R_n at once, a crowd that moves paid for it every step: 262,144
        // agents walking at 1.5 /m^2, k 8, 654 us a step, 158 so)
        constexpr int kWanted = 3 * (K + 1 + KeptShape<K>::kMore) / 2;
        constexpr int kNext = kWanted < kCap - 3 ? kWanted : kCap - 3;
        if (n <= (uint32_t)K) r2c = fmin(r2c * ((double)kNext / (double)max(n, 1u)), g.rn2);
    }
    // pass 1: per-bin counts of the keys below r2c in kBins equal-area bins,
    // and the candidates themselves while they fit the buffer; again with
    // another circle where that does not tell the nearest apart.
    double bscale;
    // Counts per bin: 4-bit counters of one group of candidates in `nib`
    // (a group adds at most kScanUnroll <= 15 to a bin), widened after each
    // group into byte counters, even bins in `hev` (byte k: bin 2k) and odd
    // bins in `hod` (byte k: bin 2k + 1), which hold up to 255 candidates.
    static_assert(kScanUnroll <= 15, "a group must fit the 4-bit counters");
    uint64_t hev, hod, nib;
    uint32_t total, take;
    int bstar;
    // circles known to hold too few, and more than needed (rounded outwards)
    float few = 0.0f, many = 0.0f;
    auto outer = [](double r2) { return (float)r2 * 1.000001f; };
    auto between = [&] { return fmin((double)(sqrtf(few) * sqrtf(many)), g.rn2); };
    for (int tries = 0;; ++tries) {
        bscale = (double)kBins / r2c;
        hev = 0;
        hod = 0;
        nib = 0;
        total = 0;
        scan_disc_groups(
            g, start, s0, xd, yd, r2c,
            [&](const float2 (&c)[kScanUnroll], uint32_t t0, uint32_t e) {
                double key[kScanUnroll];
                int bin[kScanUnroll];
                bool in[kScanUnroll];
#pragma unroll
                for (int q = 0; q < kScanUnroll; ++q) {
                    key[q] = nb_key(xi, yi, c[q].x, c[q].y);
                    in[q] = t0 + q < e && key[q] < r2c;
                    // equals min((int)(key * bscale), kBins - 1) for every
                    // key, and is defined also for the far (or invalid)
                    // candidates it is not used for
                    bin[q] = (int)fmin(key[q] * bscale, (double)(kBins - 1));
                }
#pragma unroll
                for (int q = 0; q < kScanUnroll; ++q) {
                    nib += (uint64_t)(in[q] ? 1u : 0u) << (bin[q] * 4);
                    const int slot = total < (uint32_t)(kCap - 1) ? (int)total : kCap - 1;
                    buf[buf_idx<BLOCK>(slot, tid)] = pack_entry(key[q], t0 + q, (uint32_t)bin[q]);
                    total += in[q] ? 1u : 0u;
                }
                hev += nib & 0x0F0F0F0F0F0F0F0Full;
                hod += (nib >> 4) & 0x0F0F0F0F0F0F0F0Full;
                nib = 0;
            });
        if (total <= (uint32_t)K && r2c < g.rn2) {
            few = (float)r2c;  // the guessed circle holds fewer than K: count them all
            r2c = many > 0.0f ? between() : g.rn2;
        } else if (total > 255u) {
            many = outer(r2c);  // next a circle of 64, by its share
            r2c = few > 0.0f ? between() : r2c * (64.0 / (double)total);
        } else {
            // threshold bin b*: the first bin at which the cumulative count
            // reaches K others
            uint32_t cum = 0;
            take = total;
            bstar = kBins - 1;
            bool found = false;
#pragma unroll
            for (int b = 0; b < kBins; ++b) {
                cum += (uint32_t)((((b & 1) ? hod : hev) >> ((b >> 1) * 8)) & 0xffull);
                if (!found && cum > (uint32_t)K) {
                    found = true;
                    bstar = b;
                    take = cum;
                }
            }
            if (take <= (uint32_t)kCap) break;
            // the bins are too wide: the circle up to b*, or into the last bin
            const double bin = r2c / (double)kBins;
            few = (float)((double)bstar * bin);
            many = outer(r2c);
            r2c = bstar + 1 < kBins ? (double)(bstar + 1) * bin * (1.0 + 1e-9)
                                    : between();
        }
        if (tries == kRecounts) {
            r2c = many > 0.0f ? fmin((double)many, g.rn2) : g.rn2;
            return 0;
        }
    }
    // every candidate of the circle is in the buffer, below its last slot
    const bool captured = total <= (uint32_t)(kCap - 1);
    // the circle that holds bins <= b* (with a relative margin far above the
    // rounding of key * bscale)
    const bool last = bstar + 1 >= kBins;
    const double r2 = last ? r2c : (double)(bstar + 1) * (r2c / (double)kBins) * (1.0 + 1e-9);
    if (captured) {
        // the candidates of bins <= b* are already in the buffer: keep them in
        // place.  Branch-free: each entry is written at the next kept
        // position, which never passes the one being read, and the position
        // advances only for kept entries
        uint32_t w = 0;
        for (uint32_t e = 0; e < total; ++e) {
            const uint64_t ent = buf[buf_idx<BLOCK>((int)e, tid)];
            buf[buf_idx<BLOCK>((int)w, tid)] = ent;
            w += (int)entry_bin(ent) <= bstar ? 1u : 0u;
        }
    } else {
        // pass 2: collect the candidates of bins <= b*, in scan order.  For
        // b* below the last bin, bin <= b* is exactly key * bscale < b* + 1
        // (truncation of a non-negative value), so both passes count alike.
        // Every such key is below r2, so only rows and chords of that smaller
        // circle are visited.
        const double bnext = last ? INFINITY : (double)(bstar + 1);
        uint32_t slot = 0;
        scan_disc(g, start, s0, xd, yd, r2, [&](const float2 &c, uint32_t t, bool valid) {
            const double key = nb_key(xi, yi, c.x, c.y);
            if (valid && key < r2c && key * bscale < bnext) {
                if (slot < (uint32_t)kCap)  // always true: both passes count alike
                    buf[buf_idx<BLOCK>((int)slot, tid)] = pack_entry(key, t);
                ++slot;
            }
        });
    }
    r2c = r2;
    return take;
}

// Selects the (at most K) nearest agents of the lane into entries [0, m) of
// its LDS buffer, ascending; returns m.  `keep` (nullable): the agent's kept
// radius, 0 for none; the counting pass starts from the whole neighbour
// circle then.
template <int K, int BLOCK>
__device__ int knn_select(const GridMeta &g, const uint32_t *__restrict__ start,
                          const float2 *__restrict__ s0, const float4 *__restrict__ s1, float xi,
                          float yi, uint32_t spos, uint64_t *buf, int tid, float *keep)
{
    const double xd = xi, yd = yi;
    const float last = keep ? *keep : 0.0f;
    const bool kept = last > 0.0f;
    const double rg2 = kept ? (double)last * (double)last : g.rn2;
    lane_order<BLOCK>();  // other lanes' half-planes of a previous tile are read
    double r2c;
    const uint32_t take = knn_collect<K, BLOCK>(g, start, s0, xi, yi, buf, tid, rg2, kept, r2c);
    if (take) {
        // a circle of fewer entries is widened by their share
        float next = (float)sqrt(r2c) * sqrtf((float)(K + 1 + KeptShape<K>::kMore) / (float)take);
        sort_entries<K, BLOCK>(s0, s1, xi, yi, spos, buf, tid, take, r2c, next);
        if (keep) *keep = fminf(next, g.rn);
        return (int)min(take - 1u, (uint32_t)K);
    }
    // fallback: repeated minimum over that circle, strictly above the last pick
    const CellDisc disc = cell_disc(g, xd, yd, r2c);
    int ya, yb;
    row_span(g, disc, ya, yb);
    double lk = -1.0;
    int lj = -1;
    int m = 0;
    for (; m < K; ++m) {
        double bk = INFINITY;
        int bj = INT_MAX;
        uint32_t bt = 0;
        for (int yy = ya; yy <= yb; ++yy) {
            uint32_t ra, rb;
            if (!row_range(g, start, disc, yy, ra, rb)) continue;
            for (uint32_t t = ra; t < rb; ++t) {
                const float2 c = s0[t];
                const int j = tag_index(s1[t].z);
                const double key = nb_key(xi, yi, c.x, c.y);
                const bool above = key > lk || (key == lk && j > lj);
                const bool below = key < bk || (key == bk && j < bj);
                if (key < r2c && t != spos && above && below) {
                    bk = key;
                    bj = j;
                    bt = t;
                }
            }
        }
        if (bj == INT_MAX) break;
        buf[buf_idx<BLOCK>(m, tid)] = pack_entry(bk, bt);
        lk = bk;
        lj = bj;
    }
    // the next circle, from the last pick's distance
    if (keep)
        *keep = m == K ? fminf((float)sqrt(lk) * sqrtf((float)(K + 1 + KeptShape<K>::kMore) / (float)(K + 1)),
                               g.rn)
                       : g.rn;
    return m;
}

// |P|^2 - R^2 of two agents, in double from their FP32 positions and radii
// (the differences and the sum are exact there, the products nearly so): the
// contact test |P| > R and the length of the legs' tangent, sqrt(|P|^2 - R^2),
// which FP32 would form with a cancellation of its own rounding error when
// the two discs almost touch.
__device__ __forceinline__ double clearance2(float pax, float pay, float ra, float pbx, float pby,
                                             float rb)
{
    const double px = (double)pbx - (double)pax, py = (double)pby - (double)pay;
    const double r = (double)ra + (double)rb;
    return px * px + py * py - r * r;
}

// ORCA_{A|B} as (q.x, q.y, d.x, d.y); permitted side det(d, v - q) >= 0.
// P = p_B - p_A, V = v_A - v_B, R = r_A + r_B.
//  - not overlapping: w = V - P/tau; the cutoff arc is nearest when the angle
//    between w and -P is below arccos(R/|P|), else the left leg (det(P,w) > 0)
//    or the right leg; u is the shortest vector from V to the boundary and n
//    the outward normal there.
//  - overlapping (|P| <= R): the horizon becomes dt and only the disc is used;
//    w = 0 takes the normal (+1, 0) if A's caller index is the smaller one,
//    else (-1, 0).
//  - q = v_A + f u, d = (n.y, -n.x).  q is kept as this sum: with f = 0 all
//    of an agent's lines then pass exactly through v_A, so a feasible set that
//    has shrunk to that single point stays feasible in FP32.
__device__ __forceinline__ float4 halfplane(float pax, float pay, float vax, float vay, float ra,
                                            float pbx, float pby, float vbx, float vby, float rb,
                                            float f, float inv_tau, float inv_dt, bool a_first)
{
    const float Px = pbx - pax, Py = pby - pay;
    const float Vx = vax - vbx, Vy = vay - vby;
    const float R = ra + rb;
    const float dist2 = Px * Px + Py * Py;
    const float R2 = R * R;
    const double c2 = clearance2(pax, pay, ra, pbx, pby, rb);
    const bool overlap = !(c2 > 0.0);
    const float it = overlap ? inv_dt : inv_tau;
    const float wx = Vx - Px * it, wy = Vy - Py * it;
    const float w2 = wx * wx + wy * wy;
    const float wp = wx * Px + wy * Py;
    const bool arc = overlap || (wp < 0.0f && wp * wp > R2 * w2);
    // disc (cutoff arc / overlap) form
    const bool wz = !(w2 > 0.0f);
    const float wl = sqrtf(w2);
    const float iwl = wz ? 0.0f : 1.0f / wl;
    const float anx = wz ? (a_first ? 1.0f : -1.0f) : wx * iwl;
    const float any = wz ? 0.0f : wy * iwl;
    const float ul = R * it - wl;
    float nx = anx, ny = any, ux = ul * anx, uy = ul * any;
    // leg form, only where a lane of the wavefront needs it (in dense flows
    // most half-planes take the cutoff arc: relative velocities are small)
    if (__any(!arc)) {
        const float leg = sqrtf(fmaxf((float)c2, 0.0f));
        const float id2 = overlap ? 0.0f : 1.0f / dist2;
        const bool left = det2(Px, Py, wx, wy) > 0.0f;
        const float sR = left ? R : -R;
        const float ex = (Px * leg - Py * sR) * id2;
        const float ey = (Px * sR + Py * leg) * id2;
        const float lnx = left ? -ey : ey;
        const float lny = left ? ex : -ex;
        const float s = Vx * ex + Vy * ey;
        nx = arc ? nx : lnx;
        ny = arc ? ny : lny;
        ux = arc ? ux : s * ex - Vx;
        uy = arc ? uy : s * ey - Vy;
    }
    return make_float4(vax + f * ux, vay + f * uy, ny, -nx);
}

// Acceleration limit (Sec. 5: acceleration-limited vehicles add linear
// constraints of their own motion to the same LP).  Within one step the
// velocity may change by at most a dt: the new velocity must lie in the
// regular octagon inscribed in the disc of radius a dt about c, the current
// velocity scaled onto the speed circle when it lies outside it (so the
// octagon and the speed disc always meet).  Edge k has outward normal n_k at
// angle k pi/4 at distance h = a dt cos(pi/8) from c; as a line,
// q = c + h n_k, d = (-n_k.y, n_k.x).  The lines are hard constraints: they
// precede the ORCA lines in LP2 and LP3 never relaxes them.
__device__ __forceinline__ void accel_centre(float vx, float vy, float vmax, float &cx, float &cy)
{
    const float v2 = vx * vx + vy * vy;
    const float sc = v2 > vmax * vmax ? vmax / sqrtf(v2) : 1.0f;
    cx = vx * sc;
    cy = vy * sc;
}

// Distance of the octagon's edges from its centre, a dt cos(pi/8).
__device__ __forceinline__ float accel_half_width(float acc, float dt)
{
    return acc * dt * 0.92387953f;
}

// cos(k pi/4) for k in 0..7, exactly 0, +-1 or +-0.70710678f.
__device__ __forceinline__ float cos_quarter(int k)
{
    const int m = k & 7;
    const float mag = (m & 1) ? 0.70710678f : ((m & 2) ? 0.0f : 1.0f);
    return (m >= 3 && m <= 5) ? -mag : mag;
}

// Acceleration line k, generated where it is read (no LDS): q = c + h n_k
// with single-rounding fmaf, so every read of a line gives the same bits.
__device__ __forceinline__ float4 accel_line(int k, float cx, float cy, float h)
{
    const float nx = cos_quarter(k), ny = cos_quarter(k + 6);  // sin(x) = cos(x - pi/2)
    return make_float4(fmaf(h, nx, cx), fmaf(h, ny, cy), -ny, nx);
}

// Turn-rate limit (the non-holonomic half of the same Sec. 5 extension): a
// vehicle moves along its heading, the direction of its current velocity,
// and turns it by at most w dt per step, so the new velocity lies in the
// wedge of half-angle phi = min(w dt, pi/2) about the heading, apex at the
// origin.  Its sides are the lines through the origin with directions
// r_R = R(-phi) h and -r_L = -R(phi) h (permitted side on the left), hard
// constraints after any acceleration lines.  Returns false at rest (no
// heading, no wedge).  The heading is formed in double, so that a speed
// whose square underflows FP32 still has one.
// The heading h = v/|v| and the wedge's cos(phi), sin(phi); false at rest.
// `speed` is |v| (for the adjoint's Jacobian of h).
__device__ __forceinline__ bool turn_basis(float vx, float vy, float turn, float dt, float &hx,
                                           float &hy, float &cs, float &sn, float &speed)
{
    const double v2 = (double)vx * vx + (double)vy * vy;
    if (!(turn > 0.0f) || !(v2 > 0.0)) return false;
    const double sp = sqrt(v2);
    const double inv = 1.0 / sp;
    hx = (float)(vx * inv);
    hy = (float)(vy * inv);
    speed = (float)sp;
    const float phi = fminf(turn * dt, 1.57079633f);
    sincosf(phi, &sn, &cs);
    return true;
}

__device__ __forceinline__ bool turn_wedge(float vx, float vy, float turn, float dt, float &rx,
                                           float &ry, float &lx, float &ly)
{
    float hx, hy, cs, sn, speed;
    if (!turn_basis(vx, vy, turn, dt, hx, hy, cs, sn, speed)) return false;
    rx = hx * cs + hy * sn;
    ry = hy * cs - hx * sn;
    lx = -(hx * cs - hy * sn);
    ly = -(hy * cs + hx * sn);
    return true;
}

// The lines of this lane's LP: with ACC the first nh are hard -- nacc
// acceleration lines (generated from the centre (cx, cy) and half-width h),
// then the wedge sides (through the origin, directions (rx, ry), (lx, ly))
// -- followed by the half-planes, stored in LDS column `tid`.
template <int BLOCK, bool ACC = false>
struct LdsLines {
    const float4 *L;
    int tid;
    int nh = 0;
    float cx = 0.0f, cy = 0.0f, h = 0.0f;
    int nacc = kAccLines;
    float rx = 0.0f, ry = 0.0f, lx = 0.0f, ly = 0.0f;
    __device__ __forceinline__ float4 line(int j) const
    {
        if (!ACC) return L[j * BLOCK + tid];
        // a select, not a branch: the LP code around keeps the control flow
        // (and so the multiply-add fusion) of the kernel without caps, and an
        // agent without a cap gets the same bits from both kernels
        const float4 s = L[(j >= nh ? j - nh : 0) * BLOCK + tid];
        const float4 a = accel_line(j, cx, cy, h);
        const bool right = j == nacc;
        const float wx = right ? rx : lx, wy = right ? ry : ly;
        const bool hard = j < nh, oct = j < nacc;
        return make_float4(hard ? (oct ? a.x : 0.0f) : s.x, hard ? (oct ? a.y : 0.0f) : s.y,
                           hard ? (oct ? a.z : wx) : s.z, hard ? (oct ? a.w : wy) : s.w);
    }
    __device__ __forceinline__ bool get(int j, float4 &l) const
    {
        l = line(j);
        return true;
    }
};

// Boundaries of "delta_j(v) <= delta_i(v)" for j < i (least-penetration
// sub-problem), recomputed on demand from lines i and j.  Lines parallel to i
// and pointing the same way are not constraints (invalid).  With ACC the
// first nh lines are hard (acceleration lines) and are passed on unchanged.
// Since delta_j(v) - delta_i(v) = c - det(e, v) with e = d_j - d_i and
// c = det(d_j, q_j) - det(d_i, q_i), the boundary is det(e/|e|, v) = c/|e|;
// it is stored through its point nearest the origin, (c/|e|) (-e_y, e_x)/|e|.
// This is the same line as the one through the intersection of lines i and j
// (or the midpoint of q_i, q_j for antiparallel lines), but stays well
// scaled in FP32 when the two lines are nearly parallel and intersect far
// away from the speed disc.  Two lines with the same point q pass through it
// together, and so does their boundary: it keeps q itself as its point.
template <int BLOCK, bool ACC = false>
struct ProjLines {
    const LdsLines<BLOCK, ACC> &ls;
    float4 li;
    float ci;    // det(d_i, q_i)
    float eps;
    // Computes the boundary without a branch on the line; returns false when
    // it is not a constraint (its components are then meaningless).
    __device__ __forceinline__ bool get(int j, float4 &out) const
    {
        return make(j, ls.line(j), out);
    }
    __device__ __forceinline__ bool make(int j, float4 lj, float4 &out) const
    {
        if (ACC && j < ls.nh) {
            out = lj;
            return true;
        }
        const float dij = det2(li.z, li.w, lj.z, lj.w);
        const bool same = fabsf(dij) <= eps && li.z * lj.z + li.w * lj.w > 0.0f;
        const float ex = lj.z - li.z, ey = lj.w - li.w;
        const float il = 1.0f / sqrtf(ex * ex + ey * ey);
        const float dx = ex * il, dy = ey * il;
        const float off = (det2(lj.z, lj.w, lj.x, lj.y) - ci) * il;
        // Lines through one point (the f = 0 lines of an agent all pass
        // exactly through its velocity) have their boundary through that same
        // point: it is kept exactly, so that an LP whose feasible region is a
        // cone with its apex there (or that apex alone) decides feasibility
        // at the apex exactly, as the oracle's intersection form does.
        const bool common = lj.x == li.x && lj.y == li.y;
        out = make_float4(common ? li.x : -dy * off, common ? li.y : dx * off, dx, dy);
        return !same;
    }
};


// The same boundaries in double, for a sub-problem that failed in FP32: the
// boundary passes through the intersection of lines i and j (the midpoint
// of q_i and q_j when they are antiparallel) with direction
// (d_j - d_i) / |d_j - d_i|.  Such a sub-problem always has a solution in
// exact arithmetic (the current point lies in its region), so its failure
// means a feasible set thinner than FP32 resolves: several lines through
// one vertex, the f = 0 lines that all meet at the agent's own velocity, an
// apex on the speed circle.  In double it is decided as the oracle decides.
template <int BLOCK, bool ACC = false>
struct ProjLinesD {
    const LdsLines<BLOCK, ACC> &ls;
    double4 li;
    double eps;
    // Computes the boundary without a branch on the line; returns false when
    // it is not a constraint (its components are then meaningless).
    __device__ __forceinline__ bool get(int j, double4 &out) const
    {
        const float4 l = ls.line(j);
        const double4 lj = make_double4(l.x, l.y, l.z, l.w);
        if (ACC && j < ls.nh) {
            out = lj;
            return true;
        }
        const double dij = det2(li.z, li.w, lj.z, lj.w);
        const bool par = fabs(dij) <= eps;
        const bool same = par && li.z * lj.z + li.w * lj.w > 0.0;
        const double t = det2(lj.z, lj.w, li.x - lj.x, li.y - lj.y) / dij;
        const double px = par ? 0.5 * (li.x + lj.x) : li.x + t * li.z;
        const double py = par ? 0.5 * (li.y + lj.y) : li.y + t * li.w;
        const double ex = lj.z - li.z, ey = lj.w - li.w;
        const double il = 1.0 / sqrt(ex * ex + ey * ey);
        out = make_double4(px, py, ex * il, ey * il);
        return !same;
    }
};

// The constraints that define an LP result (its active set), recorded by
// the adjoint's recomputation of the step.  LP2 results: kFree (v = v_pref),
// kDisc (v_pref scaled onto the speed circle), kLine (projection of v_pref
// onto line a), kLineLine (intersection of lines a and b), kLineDisc (line a
// on the speed circle).  LP3 results, for the line i3 whose penetration was
// minimised last: kDir (v_max times i3's inward normal), kProjDisc (the
// equal-penetration boundary of a and i3 on the circle), kProjProj (the
// point of equal penetration of a, b and i3), kTie (v_pref projected onto
// the boundary of a and i3); with acceleration lines, a or b below their
// count stands for that hard line itself instead of a boundary.  kCentre:
// the acceleration octagon's centre (LP2 failed on a hard line).
enum ActiveKind {
    kFree = 0,
    kDisc,
    kLine,
    kLineLine,
    kLineDisc,
    kDir,
    kProjDisc,
    kProjProj,
    kTie,
    kCentre
};

struct ActiveSet {
    int kind;
    int i3;
    int a, b;
};

// What the LP's scalar type resolves in a velocity, relative to v_max (about
// 16 ulps): the slack of lp1's interval test and the least excess over
// LP3's level that makes a line be re-solved.
template <class S>
struct FeasSlack;
template <>
struct FeasSlack<float> {
    static constexpr float v = 0x1p-20f;
};
template <>
struct FeasSlack<double> {
    static constexpr double v = 0x1p-49;
};

// One-dimensional sub-problem on line li (index i): the parameter interval
// inside the speed disc (lp1_disc) and on the permitted side of every valid
// line j < i (lp1_cut), then the point of it that the objective takes
// (lp1_point).  The parts are shared by the form that walks the lines in one
// lane and the one that spreads them over four.
//
// The line meets the speed circle at t^2 + 2 dot t + c = 0, c = |q|^2 -
// v_max^2.  c is formed in double (exact products), so its sign -- whether
// q itself lies in the disc -- is exact; the root near q is taken as c
// over the other root, which has no cancellation, so q stays inside the
// interval exactly when it lies in the disc (the f = 0 lines of an agent
// pass through its own velocity, which the grid build puts inside the
// disc: that apex is then a feasible point, as it is exactly).
template <class S, class V4>
__device__ __forceinline__ bool lp1_disc(V4 li, S vmax, S &tl, S &tr)
{
    const S dot = li.x * li.z + li.y * li.w;
    const double cd = (double)li.x * (double)li.x + (double)li.y * (double)li.y -
                      (double)vmax * (double)vmax;
    const S c = (S)cd;
    const S disc = dot * dot - c;
    if (disc < (S)0) return false;
    const S sq = lp_sqrt(disc);
    const S far = dot > (S)0 ? -dot - sq : -dot + sq;
    const S near = far != (S)0 ? c / far : (S)0;
    tl = lp_min(far, near);
    tr = lp_max(far, near);
    return true;
}

// Line j's cut of the interval [tl, tr] (whose ends lines sl and sr set).
// Branch-free: the lanes of a wavefront meet different cases (parallel,
// lower or upper bound) at the same j, so every case is a select.  Lines
// parallel within eps are one line when line i is offset to j's forbidden
// side by no more than 2^-20 v_max (far below what the FP32 positions
// resolve), else disjoint (`apart`); the same offset in either precision and
// in the FP64 reference.
template <class S, class V4>
__device__ __forceinline__ void lp1_cut(int j, V4 lj, bool valid, V4 li, S eps, S pslack, S &tl,
                                        S &tr, int &sl, int &sr, bool &apart)
{
    const S a = det2(lj.z, lj.w, li.z, li.w);
    const S b = det2(lj.z, lj.w, li.x - lj.x, li.y - lj.y);
    const bool par = lp_abs(a) <= eps;
    const S t = -b / a;
    const bool cut = valid && !par;
    const bool lo = cut && a > (S)0 && t > tl;
    const bool hi = cut && !(a > (S)0) && t < tr;
    tl = lo ? t : tl;
    sl = lo ? j : sl;
    tr = hi ? t : tr;
    sr = hi ? j : sr;
    apart = apart || (valid && par && b < -pslack);
}

// mode 0: closest point to (ox, oy); mode 1: extreme along unit (ox, oy), or,
// when the line is orthogonal to it, the point closest to (tx, ty).
// `how` reports what fixed the result: 0 projection, 1 / 2 the lower / upper
// end of the interval (bounded by line `src`, or by the disc when src < 0),
// 3 the tie projection.
template <class S, class V4>
__device__ __forceinline__ void lp1_point(V4 li, int mode, S ox, S oy, S tx, S ty, S eps, S tl,
                                          S tr, int sl, int sr, S &x, S &y, int &how, int &bound)
{
    S t;
    if (mode == 0) {
        t = li.z * (ox - li.x) + li.w * (oy - li.y);
        how = 0;
    } else {
        const S sd = ox * li.z + oy * li.w;
        if (lp_abs(sd) <= eps) {
            t = li.z * (tx - li.x) + li.w * (ty - li.y);
            how = 3;
        } else {
            t = sd > (S)0 ? tr : tl;
            how = sd > (S)0 ? 2 : 1;
        }
    }
    if (t < tl) {
        t = tl;
        how = 1;
    }
    if (t > tr) {
        t = tr;
        how = 2;
    }
    bound = how == 1 ? sl : (how == 2 ? sr : -1);
    x = li.x + t * li.z;
    y = li.y + t * li.w;
}

template <class S, class Src>
__device__ __forceinline__ bool lp1(const Src &src, int i, typename LpVec<S>::T li, S vmax,
                                    int mode, S ox, S oy, S tx, S ty, S eps, S &x, S &y, int &how,
                                    int &bound)
{
    using V4 = typename LpVec<S>::T;
    S tl, tr;
    if (!lp1_disc<S>(li, vmax, tl, tr)) return false;
    int sl = -1, sr = -1;
    // An interval empty by less than the scalar type resolves at this
    // velocity scale (FeasSlack v_max) counts as one point: a feasible set
    // that thin --
    // several lines through one vertex, an apex on the speed circle -- is
    // empty or not by rounding alone, and the point found then violates a
    // constraint by no more than that.  The interval only shrinks, so a
    // failure at some j is a failure at the end.
    const S slack = vmax * FeasSlack<S>::v;
    const S pslack = vmax * (S)0x1p-20;
    bool apart = false;
    for (int j = 0; j < i; ++j) {
        V4 lj;
        const bool valid = src.get(j, lj);
        lp1_cut<S>(j, lj, valid, li, eps, pslack, tl, tr, sl, sr, apart);
    }
    if (apart || tl > tr + slack) return false;
    lp1_point<S>(li, mode, ox, oy, tx, ty, eps, tl, tr, sl, sr, x, y, how, bound);
    return true;
}

// The LP's answer without any line: in the direction (ox, oy) on the speed
// circle (mode 1), or the point (ox, oy) itself, scaled onto the circle when
// it lies outside.
template <bool REC, class S>
__device__ __forceinline__ void lp2_start(S vmax, int mode, S ox, S oy, S &x, S &y, ActiveSet *rec)
{
    if (mode == 1) {
        x = ox * vmax;
        y = oy * vmax;
        if (REC) rec->kind = kDir;
    } else {
        const S o2 = ox * ox + oy * oy;
        if (o2 > vmax * vmax) {
            const S sc = vmax / lp_sqrt(o2);
            x = ox * sc;
            y = oy * sc;
            if (REC) rec->kind = kDisc;
        } else {
            x = ox;
            y = oy;
            if (REC) rec->kind = kFree;
        }
    }
}

// Line i was re-solved (lp1_point's `how` and bounding line).
__device__ __forceinline__ void lp2_record(int i, int bound, int mode, int how, ActiveSet *rec)
{
    rec->a = i;
    rec->b = bound;
    if (mode == 0)
        rec->kind = how == 0 ? kLine : (bound >= 0 ? kLineLine : kLineDisc);
    else
        rec->kind = how == 3 ? kTie : (bound >= 0 ? kProjProj : kProjDisc);
}

// Incremental 2D LP over lines 0..m-1 of `src` and the disc |v| <= vmax.
// Returns the first infeasible line, or m; v keeps its pre-failure value.
// With REC the active set of the result is written to *rec.
template <bool REC, class S, class Src>
__device__ __forceinline__ int lp2(const Src &src, int m, S vmax, int mode, S ox, S oy, S tx,
                                   S ty, S eps, S &vx, S &vy, ActiveSet *rec)
{
    S x, y;
    lp2_start<REC>(vmax, mode, ox, oy, x, y, rec);
    for (int i = 0; i < m; ++i) {
        typename LpVec<S>::T li;
        const bool valid = src.get(i, li);
        if (valid && det2(li.z, li.w, li.x - x, li.y - y) > (S)0) {
            S nx = x, ny = y;
            int how, bound;
            if (!lp1<S>(src, i, li, vmax, mode, ox, oy, tx, ty, eps, nx, ny, how, bound)) {
                vx = x;
                vy = y;
                return i;
            }
            x = nx;
            y = ny;
            if (REC) lp2_record(i, bound, mode, how, rec);
        }
    }
    vx = x;
    vy = y;
    return m;
}


// Least penetration (Sec. 3): from LP2's partial result at line `fail`, each
// later line i whose penetration exceeds the current level re-solves v in the
// region where no earlier line penetrates more than line i, as deep into line
// i's permitted side as possible.  With ACC the first nh lines are hard: never
// relaxed, they bound every re-solve as they are.
template <bool REC, int BLOCK, bool ACC = false>
__device__ __forceinline__ void lp3(const LdsLines<BLOCK, ACC> &ls, int m, int fail, float vmax,
                                    float tx, float ty, float eps, float &vx, float &vy,
                                    ActiveSet *rec)
{
    float level = 0.0f;
    float x = vx, y = vy;
    const int nhard = ACC ? ls.nh : 0;
    // a line is re-solved only when it exceeds the level by more than FP32
    // resolves in a penetration (about 2^-20 v_max): at a point where several
    // lines are penetrated equally, FP32 rounding alone would otherwise
    // decide whether a later tied line triggers a re-solve, and the re-solve
    // then jumps to another vertex of the tie
    const float tol = vmax * FeasSlack<float>::v;
    // as in lp2: each lane steps on to its own next line above the level, and
    // the lanes re-solve together
    int i = fail > nhard ? fail : nhard;
    for (;;) {
        float4 li;
        for (; i < m; ++i) {
            li = ls.line(i);
            if (det2(li.z, li.w, li.x - x, li.y - y) > level + tol) break;
        }
        if (i >= m) break;
        ProjLines<BLOCK, ACC> src{ls, li, det2(li.z, li.w, li.x, li.y), eps};
        float nx = x, ny = y;
        ActiveSet inner;
        bool solved = lp2<REC, float>(src, i, vmax, 1, -li.w, li.z, tx, ty, eps, nx, ny,
                                      &inner) == i;
        if (!solved) {
            // failed in FP32 only: solve it again in double (ProjLinesD)
            const double4 lid = make_double4(li.x, li.y, li.z, li.w);
            ProjLinesD<BLOCK, ACC> srcd{ls, lid, (double)eps};
            double dx = x, dy = y;
            solved = lp2<REC, double>(srcd, i, (double)vmax, 1, -lid.w, lid.z, (double)tx,
                                      (double)ty, (double)eps, dx, dy, &inner) == i;
            nx = (float)dx;
            ny = (float)dy;
        }
        if (solved) {
            x = nx;
            y = ny;
            if (REC) {
                *rec = inner;
                rec->i3 = i;
            }
        }
        level = det2(li.z, li.w, li.x - x, li.y - y);
        ++i;
    }
    vx = x;
    vy = y;
}

// ---------------------------------------------------------------------------
// Least penetration (Sec. 3), by a group of lanes per agent: from LP2's
// partial result at line `fail`, each later line i whose penetration exceeds
// the current level re-solves v in the region where no earlier line penetrates
// more than line i, as deep into line i's permitted side as possible.  Hard
// lines are never relaxed; they bound every re-solve as they are.
//
// What bounds it is the serial walk over lines inside lines inside lines, and
// the lanes that wait for it: a wavefront has few lanes in LP3 (a quarter in a
// dense crossing, an eighth in a mixed crowd), so a walk by the lane itself
// runs at that share of the SIMD.  Here the failed agents of the wavefront, 16
// at a time, are taken over by its 16 groups of G = 4 lanes: lane c of a group
// holds lines c, c + G, c + 2 G, ... of its agent, so the boundaries, the test
// for the next violated line and the cuts of an interval each take a fourth
// of the walk (one pass over the lane's registers and two DPP steps), and each
// boundary is formed once for a sub-problem.
// The result is the serial one bit for bit: the first violated line is the
// least index over the group, an interval's ends are an exact maximum and
// minimum (the first line that attains one is kept, as in the walk), and
// every value is formed by the same expressions.
//
// Against the walk per lane, whole steps: 1M dense crossing (24 % of agents in
// LP3) 452 -> 394 us, 66,560 mixed (12 %) 148 -> 96 us, 4,999 mixed 121 -> 92
// us, 512 scenes (44 %) 4.03 -> 3.56 ms.  G = 8 and 16: 407 and 452 us on the
// crossing against 384 us; with hard lines, up to ten more per agent, 8 is the
// best (200,003 capped: 240, 208 and 226 us at 4, 8 and 16; 278 us by the walk).
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ int dpp(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}

// Reductions over the G lanes of a group (4, 8 or 16), the result in each:
// lanes 1,0,3,2 and 2,3,0,1 of each quad, then the lanes of each half row and
// of each row in reverse.
template <int G, class F>
__device__ __forceinline__ int group_reduce(int v, F f)
{
    v = f(v, dpp<0xB1>(v));
    v = f(v, dpp<0x4E>(v));
    if (G >= 8) v = f(v, dpp<0x141>(v));
    if (G >= 16) v = f(v, dpp<0x140>(v));
    return v;
}
template <int G>
__device__ __forceinline__ int group_min(int v)
{
    return group_reduce<G>(v, [](int a, int b) { return min(a, b); });
}
template <int G>
__device__ __forceinline__ bool group_any(bool p)
{
    return group_reduce<G>(p ? 1 : 0, [](int a, int b) { return a | b; }) != 0;
}
template <int G>
__device__ __forceinline__ float group_max(float v)
{
    return __int_as_float(group_reduce<G>(__float_as_int(v), [](int a, int b) {
        return __float_as_int(fmaxf(__int_as_float(a), __int_as_float(b)));
    }));
}
template <int G>
__device__ __forceinline__ float group_min(float v)
{
    return __int_as_float(group_reduce<G>(__float_as_int(v), [](int a, int b) {
        return __float_as_int(fminf(__int_as_float(a), __int_as_float(b)));
    }));
}

// Line k of the group's (the same k in its lanes), from register k / G of
// lane k % G.
template <int G, int NL>
__device__ __forceinline__ float4 group_line(const float4 (&l)[NL], int k)
{
    float4 v = l[0];
#pragma unroll
    for (int r = 1; r < NL; ++r) {
        const bool is = k / G == r;
        v = make_float4(is ? l[r].x : v.x, is ? l[r].y : v.y, is ? l[r].z : v.z,
                        is ? l[r].w : v.w);
    }
    return make_float4(__shfl(v.x, k % G, G), __shfl(v.y, k % G, G), __shfl(v.z, k % G, G),
                       __shfl(v.w, k % G, G));
}

// lp2 by the group: lane c holds lines c, c + G, ... of the m in ln, valid where
// bit r of `valid` is set (only below m).
template <bool REC, int G, int NL>
__device__ __forceinline__ int group_lp2(const float4 (&ln)[NL], uint32_t valid, int c, int m,
                                         float vmax, int mode, float ox, float oy, float tx,
                                         float ty, float eps, float &vx, float &vy, ActiveSet *rec)
{
    const float slack = vmax * FeasSlack<float>::v;
    const float pslack = vmax * 0x1p-20f;
    lp2_start<REC>(vmax, mode, ox, oy, vx, vy, rec);
    for (int k = 0;; ++k) {
        // the next violated line
        int next = m;
#pragma unroll
        for (int r = NL - 1; r >= 0; --r) {
            const int j = c + G * r;
            if (G * r < m) {  // the same in the whole group
                const bool out = det2(ln[r].z, ln[r].w, ln[r].x - vx, ln[r].y - vy) > 0.0f;
                next = ((valid >> r) & 1u) && j >= k && out ? j : next;
            }
        }
        k = group_min<G>(next);
        if (k >= m) return m;
        const float4 lk = group_line<G>(ln, k);
        float tl, tr;
        if (!lp1_disc<float>(lk, vmax, tl, tr)) return k;
        const float tl0 = tl, tr0 = tr;
        int sl = -1, sr = -1;
        bool apart = false;
#pragma unroll
        for (int r = 0; r < NL; ++r) {
            const int j = c + G * r;
            if (G * r < k)
                lp1_cut<float>(j, ln[r], ((valid >> r) & 1u) && j < k, lk, eps, pslack, tl, tr, sl,
                               sr, apart);
        }
        const float gl = group_max<G>(tl), gr = group_min<G>(tr);
        if (REC) {
            // the first line that sets each end
            const int fl = group_min<G>(sl >= 0 && tl == gl ? sl : INT_MAX);
            const int fr = group_min<G>(sr >= 0 && tr == gr ? sr : INT_MAX);
            sl = gl > tl0 && fl != INT_MAX ? fl : -1;
            sr = gr < tr0 && fr != INT_MAX ? fr : -1;
        }
        if (group_any<G>(apart) || gl > gr + slack) return k;
        int how, bound;
        lp1_point<float>(lk, mode, ox, oy, tx, ty, eps, gl, gr, sl, sr, vx, vy, how, bound);
        if (REC) lp2_record(k, bound, mode, how, rec);
    }
}

// LP3 of one agent by the group this lane belongs to (c = its lane there); all
// arguments are the same in the group's lanes.  ls reads the agent's lines.  NL:
// lines per lane.
template <bool REC, int BLOCK, bool ACC, int G, int NL>
__device__ __forceinline__ void group_lp3(const LdsLines<BLOCK, ACC> &ls, int c, int m, int fail,
                                         float vmax, float tx, float ty, float eps, float &vx,
                                         float &vy, ActiveSet *rec)
{
    float level = 0.0f;
    float x = vx, y = vy;
    const int nhard = ACC ? ls.nh : 0;
    // a line is re-solved only when it exceeds the level by more than FP32
    // resolves in a penetration (about 2^-20 v_max): at a point where several
    // lines are penetrated equally, FP32 rounding alone would otherwise
    // decide whether a later tied line triggers a re-solve, and the re-solve
    // then jumps to another vertex of the tie
    const float tol = vmax * FeasSlack<float>::v;
    float4 ln[NL];
#pragma unroll
    for (int r = 0; r < NL; ++r) ln[r] = ls.line(min(c + G * r, m - 1));
    int i = fail > nhard ? fail : nhard;
    for (;;) {
        // the next line above the level
        int first = m;
#pragma unroll
        for (int r = NL - 1; r >= 0; --r) {
            const int j = c + G * r;
            const bool above = det2(ln[r].z, ln[r].w, ln[r].x - x, ln[r].y - y) > level + tol;
            first = j >= i && j < m && above ? j : first;
        }
        i = group_min<G>(first);
        if (i >= m) break;
        const float4 li = ls.line(i);
        const ProjLines<BLOCK, ACC> src{ls, li, det2(li.z, li.w, li.x, li.y), eps};
        float4 bd[NL];
        uint32_t valid = 0;
#pragma unroll
        for (int r = 0; r < NL; ++r) {
            const int j = c + G * r;
            if (G * r < i) {  // the same in the whole group
                const bool is = src.make(j, ln[r], bd[r]) && j < i;
                valid |= (is ? 1u : 0u) << r;
            }
        }
        // LP2 over the boundaries, objective: deepest into line i
        float nx, ny;
        ActiveSet inner;
        bool solved = group_lp2<REC, G>(bd, valid, c, i, vmax, 1, -li.w, li.z, tx, ty, eps, nx, ny,
                                        &inner) == i;
        if (!solved) {
            // failed in FP32 only: solve it again in double (ProjLinesD), the
            // same walk in each of the group's lanes
            const double4 lid = make_double4(li.x, li.y, li.z, li.w);
            ProjLinesD<BLOCK, ACC> srcd{ls, lid, (double)eps};
            double dx = x, dy = y;
            solved = lp2<REC, double>(srcd, i, (double)vmax, 1, -lid.w, lid.z, (double)tx,
                                      (double)ty, (double)eps, dx, dy, &inner) == i;
            nx = (float)dx;
            ny = (float)dy;
        }
        if (solved) {
            x = nx;
            y = ny;
            if (REC) {
                *rec = inner;
                rec->i3 = i;
            }
        }
        level = det2(li.z, li.w, li.x - x, li.y - y);
        ++i;
    }
    vx = x;
    vy = y;
}

// LP3 of every lane of the wavefront with `need` (its LP2 stopped at line
// fail < m), all 64 lanes taking part: by groups of lanes, or by each lane
// itself (lp3) where most of the wavefront needs it and the walk keeps its
// lanes busy.  The line at 24, 32, 40 and 48 lanes and groups alone: the 1M
// crossing simulated over steps 10-110 403, 403, 407, 410 and 419 us per step
// (419 us by the walk alone), 512 scenes at 32, 40 and groups alone 3.68, 3.57
// and 3.56 ms, 200,003 capped at 24 to 48 253, 238, 211 and 212 us; small
// crowds are the same down to 32 and lose at 24 (4,999 mixed: 92 and 112 us).
// WALK: the lanes in any case.  Groups that record the active set take the registers
// of a wavefront or two per SIMD, which large crowds feel and small ones do not (whole
// adjoints in us, groups / walk, at 0.05 and 0.45 /m^2: k 10 131,072 agents 83 / 85, 151 /
// 148, 200,000 121 / 101, 227 / 180, 1M 497 / 468, 765 / 592; with hard lines k 8 131,072 113 /
// 139, 193 / 188, 200,000 169 / 166, 306 / 262, 1M 592 / 514, 1107 / 816): the adjoint up to k
// 12, above kWalkAgents.  Lists of up to kBriefList are walked by all kernels without hard
// lines (step, 66,560 agents at 0.5 /m^2, 65 / 62 us).
template <bool REC, int K, int BLOCK, bool ACC, bool WALK>
__device__ __forceinline__ void wave_lp3(const LdsLines<BLOCK, ACC> &ls, int tid, bool need, int m,
                                         int fail, float vmax, float tx, float ty, float eps,
                                         float &vx, float &vy, ActiveSet *rec)
{
    constexpr int G = ACC ? 8 : 4;
    constexpr int NL = (K + (ACC ? kAccLines + kTurnLines : 0) + G - 1) / G;
    constexpr int kGroups = kWave / G;
    const uint64_t needm = __ballot(need);
    const int nf = __popcll(needm);
    if (WALK || nf > (ACC ? 48 : 40)) {
        if (need) lp3<REC, BLOCK, ACC>(ls, m, fail, vmax, tx, ty, eps, vx, vy, rec);
        return;
    }
    const int lane = tid & (kWave - 1);
    const int rank = __popcll(needm & ((1ull << lane) - 1ull));
    lane_order<kWave>();  // the groups read other lanes' lines
    for (int base = 0; base < nf; base += kGroups) {
        const bool mine = need && rank >= base && rank < base + kGroups;
        const int slot = (rank - base) * G;
        // each group learns whose agent it takes (a lane without one sends to
        // lane 1, which nobody reads)
        const int from = __shfl(__builtin_amdgcn_ds_permute((mine ? slot : 1) * 4, lane), 0, G);
        const bool busy = lane / G < nf - base;
        const int src = busy ? from : lane;
        float qx = __shfl(vx, src, kWave), qy = __shfl(vy, src, kWave);
        const float qvm = __shfl(vmax, src, kWave), qtx = __shfl(tx, src, kWave),
                    qty = __shfl(ty, src, kWave), qeps = __shfl(eps, src, kWave);
        const int qm = __shfl(m, src, kWave), qfail = __shfl(fail, src, kWave);
        LdsLines<BLOCK, ACC> ql{ls.L, (tid - lane) + src};
        if (ACC) {
            ql.nh = __shfl(ls.nh, src, kWave);
            ql.nacc = __shfl(ls.nacc, src, kWave);
            ql.cx = __shfl(ls.cx, src, kWave);
            ql.cy = __shfl(ls.cy, src, kWave);
            ql.h = __shfl(ls.h, src, kWave);
            ql.rx = __shfl(ls.rx, src, kWave);
            ql.ry = __shfl(ls.ry, src, kWave);
            ql.lx = __shfl(ls.lx, src, kWave);
            ql.ly = __shfl(ls.ly, src, kWave);
        }
        ActiveSet r{kFree, -1, -1, -1};
        if (REC) r = ActiveSet{__shfl(rec->kind, src, kWave), __shfl(rec->i3, src, kWave),
                               __shfl(rec->a, src, kWave), __shfl(rec->b, src, kWave)};
        if (busy)
            group_lp3<REC, BLOCK, ACC, G, NL>(ql, lane % G, qm, qfail, qvm, qtx, qty, qeps, qx,
                                              qy, &r);
        const int back = mine ? slot : lane;
        const float gx = __shfl(qx, back, kWave), gy = __shfl(qy, back, kWave);
        vx = mine ? gx : vx;
        vy = mine ? gy : vy;
        if (REC) {
            const ActiveSet g{__shfl(r.kind, back, kWave), __shfl(r.i3, back, kWave),
                              __shfl(r.a, back, kWave), __shfl(r.b, back, kWave)};
            if (mine) *rec = g;
        }
    }
}

// Scalar parameters of the scene an agent belongs to, in the form the
// per-agent step uses.
struct SceneP {
    float dt, inv_dt, inv_tau, eps;
    int k;
    int pref_is_goal;
    float f00, f01, f10, f11;
    float acc0, acc1;    // acceleration cap per class (0: none)
    float turn0, turn1;  // turn-rate cap per class (0: none)
};

__device__ __host__ __forceinline__ SceneP scene_params(const orca_params &p)
{
    SceneP s;
    s.dt = p.dt;
    s.inv_dt = 1.0f / p.dt;
    s.inv_tau = 1.0f / p.time_horizon;
    s.eps = p.par_eps;
    s.k = p.max_neighbors;
    s.pref_is_goal = p.pref_is_goal;
    s.f00 = p.f[0][0];
    s.f01 = p.f[0][1];
    s.f10 = p.f[1][0];
    s.f11 = p.f[1][1];
    s.acc0 = p.accel[0];
    s.acc1 = p.accel[1];
    s.turn0 = p.turn[0];
    s.turn1 = p.turn[1];
    return s;
}

// The half-planes of the agent's m neighbours into its LDS column.
// Neighbour states are loaded a group at a time without a branch (unused
// slots read position 0, a valid entry) so the loads of a group are in
// flight together; the half-planes of the group follow.
template <int K, int BLOCK>
__device__ __forceinline__ void build_halfplanes(const uint32_t (&pos)[K], int m,
                                                 const float2 *__restrict__ s0,
                                                 const float4 *__restrict__ s1, float xi,
                                                 float yi, float vxi, float vyi, float ri, int i,
                                                 int ci, const SceneP &p, float4 *lines, int tid)
{
    const float fa = ci ? p.f10 : p.f00;  // f[ci][0]
    const float fb = ci ? p.f11 : p.f01;  // f[ci][1]
    constexpr int kHpGroup = 4;
    lane_order<BLOCK>();  // every lane's selection entries are read
#pragma unroll
    for (int q0 = 0; q0 < K; q0 += kHpGroup) {
        float2 b0[kHpGroup];
        float4 b1[kHpGroup];
#pragma unroll
        for (int u = 0; u < kHpGroup; ++u) {
            if (q0 + u < K) {
                b0[u] = s0[pos[q0 + u]];
                b1[u] = s1[pos[q0 + u]];
            }
        }
#pragma unroll
        for (int u = 0; u < kHpGroup; ++u) {
            const int q = q0 + u;
            if (q < K && q < m) {
                const float f = tag_class(b1[u].z) ? fb : fa;
                lines[q * BLOCK + tid] =
                    halfplane(xi, yi, vxi, vyi, ri, b0[u].x, b0[u].y, b1[u].x, b1[u].y, b1[u].w,
                              f, p.inv_tau, p.inv_dt, i < tag_index(b1[u].z));
            }
        }
    }
}

// Goal mode: the pref input (the goal) becomes the desired velocity
// (g - p) min(v_max / |g - p|, 1/dt), zero at the goal.
__device__ __forceinline__ void desired_velocity(const SceneP &p, float xi, float yi, float vmax,
                                                 float &prx, float &pry)
{
    if (p.pref_is_goal) {
        const float gx = prx - xi, gy = pry - yi;
        const float d2 = gx * gx + gy * gy;
        const float sc = d2 > 0.0f ? fminf(vmax / sqrtf(d2), p.inv_dt) : 0.0f;
        prx = gx * sc;
        pry = gy * sc;
    }
}

// One whole ORCA step of the agent at cell-order position s: neighbours,
// half-planes (into the lane's LDS column), LP2, LP3 if needed, update.
// `lines` is a [KnnShape<K>::kSlots][BLOCK] float4 array; lane `tid` owns
// column tid.  `guess` (caller order, nullable) keeps each agent's radius of
// the neighbour scan between steps (0: none).  ACC compiles the acceleration lines in (used for agents whose class
// has a cap).  EXPORT also writes the neighbour list the step used (caller
// indices, ascending, -1 padded) to nbr[i * kout ..] and its length to
// cnt[i] (either nullable); the step itself is unchanged.  All 64 lanes of a
// wavefront call it; one that is not `live` repeats an agent of another lane
// and writes nothing (its lanes serve LP3).
template <int K, int BLOCK, bool ACC = false, bool EXPORT = false>
__device__ __forceinline__ void step_agent(bool live, int s, const GridMeta &g, const SceneP &p,
                                           const orca_agents_in &in, const orca_agents_out &out,
                                           const uint32_t *__restrict__ start,
                                           const float2 *__restrict__ s0,
                                           const float4 *__restrict__ s1, float4 *lines, int tid,
                                           float *__restrict__ guess, int32_t *nbr = nullptr,
                                           int32_t *cnt = nullptr, int kout = 0)
{
    const float2 me0 = s0[s];
    const float4 me1 = s1[s];
    const int i = tag_index(me1.z);
    const float xi = me0.x, yi = me0.y, ri = me1.w, vxi = me1.x, vyi = me1.y;
    const int ci = tag_class(me1.z);
    const float vmax = in.max_speed[i];

    uint64_t *buf = reinterpret_cast<uint64_t *>(lines);
    float kept = guess ? guess[i] : 0.0f;
    const int found = knn_select<K, BLOCK>(g, start, s0, s1, xi, yi, (uint32_t)s, buf, tid, &kept);
    if (guess && live) guess[i] = kept;
    const int kk = p.k < K ? p.k : K;
    const int m = found < kk ? found : kk;
    uint32_t pos[K];
#pragma unroll
    for (int q = 0; q < K; ++q) pos[q] = q < m ? entry_pos(buf[buf_idx<BLOCK>(q, tid)]) : 0u;
    if (EXPORT && live) {
        if (nbr) {
            int32_t *row = nbr + (int64_t)i * kout;
            for (int q = 0; q < kout; ++q)
                row[q] = q < m ? tag_index(s1[entry_pos(buf[buf_idx<BLOCK>(q, tid)])].z) : -1;
        }
        if (cnt) cnt[i] = m;
    }

    float prx = in.pref_x[i], pry = in.pref_y[i];
    const float acc = ACC ? (ci ? p.acc1 : p.acc0) : 0.0f;
    const float turn = ACC ? (ci ? p.turn1 : p.turn0) : 0.0f;
    const int nacc = (ACC && acc > 0.0f) ? kAccLines : 0;
    float rx = 0.0f, ry = 0.0f, lx = 0.0f, ly = 0.0f;
    const int nh = nacc + ((ACC && turn_wedge(vxi, vyi, turn, p.dt, rx, ry, lx, ly))
                               ? kTurnLines : 0);
    build_halfplanes<K, BLOCK>(pos, m, s0, s1, xi, yi, vxi, vyi, ri, i, ci, p, lines, tid);
    float cx = 0.0f, cy = 0.0f;
    if (ACC && nh) accel_centre(vxi, vyi, vmax, cx, cy);
    desired_velocity(p, xi, yi, vmax, prx, pry);

    const LdsLines<BLOCK, ACC> src{lines, tid, nh, cx, cy,
                                   ACC && nacc ? accel_half_width(acc, p.dt) : 0.0f,
                                   nacc, rx, ry, lx, ly};
    const int mt = nh + m;
    float vx, vy;
    int fail = lp2<false, float>(src, mt, vmax, 0, prx, pry, 0.0f, 0.0f, p.eps, vx, vy, nullptr);
    uint8_t st = 0;
    if (ACC && fail < nh) {
        // the centre (the current velocity scaled into the speed disc) lies
        // in the octagon and on the wedge's axis, so only rounding can get
        // here: take the centre and let LP3 start from it
        vx = cx;
        vy = cy;
        fail = nh;
        st = 1;
    }
    const bool infeasible = fail < mt;
    wave_lp3<false, K, BLOCK, ACC, (!ACC && K <= kBriefList)>(src, tid, live && infeasible, mt, fail, vmax, prx, pry, p.eps,
                                   vx, vy, nullptr);
    if (infeasible) st = 1;
    if (!live) return;
    out.vx[i] = vx;
    out.vy[i] = vy;
    out.px[i] = xi + vx * p.dt;
    out.py[i] = yi + vy * p.dt;
    if (out.status) out.status[i] = st;
}

}  // namespace dev
}  // namespace orca
