// Internal declarations shared by the HIP translation units of liborca.so.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/orca.h"

namespace orca {

constexpr int kWave = 64;
constexpr int kBboxBlocks = 1024;   // partial bounding boxes per scene (max)
constexpr int kBboxSplit = 8;      // blocks (partial boxes) per scene of a batch
constexpr int kScanTile = 2048;     // cells per scan tile (256 threads x 8)
constexpr int kAlign = 256;
constexpr int kScanPad = 16;        // entries after the cell-ordered copy s0,
                                    // so candidate groups may read past its end

// Uniform grid of one scene, computed on the device from its bounding box.
struct GridMeta {
    float x0, y0;      // origin (bounding-box minimum)
    float cs;          // effective cell size (>= neighbour distance / m)
    float rn;          // neighbour distance
    int nx, ny;        // cells per axis
    int m;             // stencil radius in cells: in-range pairs are <= m cells apart
    int n_cells;       // nx * ny
    double inv_cs;     // 1 / cs, for the FP64 cell coordinates
    double rn2;        // rn * rn in double (exact)
    int cell_base;     // first global cell id of this scene (batched form)
    int agent_base;    // first agent (caller order) of this scene
    int n;             // agents in this scene
    uint32_t seg_end;  // one past the scene's last cell-order position
};

// Caller index (28 bits at most) and class of an agent in one word.
__host__ __device__ inline int agent_tag(int i, int cls) { return (i << 1) | (cls & 1); }
__device__ __forceinline__ int tag_index(float z) { return (int)(__float_as_uint(z) >> 1); }
__device__ __forceinline__ int tag_class(float z) { return __float_as_int(z) & 1; }

// A velocity within the speed cap: (vx, vy) itself when |v| <= v_max (the
// test in double from the FP32 values, products exact), else scaled onto the
// cap and rounded to FP32, then moved toward zero one ulp at a time until the
// test holds.  The ORCA lines an agent takes no responsibility for (f = 0)
// all pass through its own velocity; a velocity the previous step left on
// the speed circle lies outside it by a few FP32 ulps half of the time, and
// the LP's feasible set around that apex would then be thinner than FP32
// resolves.  Inside the cap, the apex is a feasible point exactly.
__device__ __forceinline__ void cap_velocity(float &vx, float &vy, float vmax)
{
    const double vm2 = (double)vmax * (double)vmax;
    const double d = (double)vx * (double)vx + (double)vy * (double)vy;
    if (!(d > vm2)) return;
    const double s = (double)vmax / sqrt(d);
    float x = (float)((double)vx * s), y = (float)((double)vy * s);
    for (int it = 0; it < 16 && (double)x * (double)x + (double)y * (double)y > vm2; ++it) {
        if (fabsf(x) >= fabsf(y))
            x = nextafterf(x, 0.0f);
        else
            y = nextafterf(y, 0.0f);
    }
    vx = x;
    vy = y;
}

// Agent i's scan position and record at place `pos` of the cell-ordered copies;
// velocities taken within the speed cap.
__device__ __forceinline__ void write_record(const orca_agents_in &in, int i, uint32_t pos,
                                             float2 *__restrict__ s0, float4 *__restrict__ s1)
{
    s0[pos] = make_float2(in.px[i], in.py[i]);
    float vx = in.vx[i], vy = in.vy[i];
    cap_velocity(vx, vy, in.max_speed[i]);
    s1[pos] = make_float4(vx, vy, __int_as_float(agent_tag(i, (int)in.cls[i])), in.radius[i]);
}

// Byte offsets of the workspace regions (all 256-byte aligned).
struct Layout {
    size_t meta, partial, cell, rank, count, start, tiles, s0, s1, guess, total;
    int64_t n, n_scenes, max_cells, n_tiles;
};

// Cells of the batched form: 2 per agent + 64 per scene.
__host__ __device__ inline int64_t batched_cells(int64_t n, int64_t n_scenes) { return 2 * n + 64 * n_scenes; }

// Cell coordinate along one axis, in FP64, clamped to [0, ncell - 1]
// (fmax/fmin also map NaN to 0).  Shared by the grid build and the
// neighbour query so that both see identical cells.
__device__ __forceinline__ int cell_axis(float v, float v0, double inv_cs, int ncell)
{
    double c = floor(((double)v - (double)v0) * inv_cs);
    c = fmin(fmax(c, 0.0), (double)(ncell - 1));
    return (int)c;
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  Remapping dispatch index b to a logical tile so that every XCD works
// on one contiguous range of tiles keeps neighbouring agents (which read each
// other's state) inside one L2.  Bijective on [0, nb).
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_tile(int b, int nb)
{
    const int q = nb / kXcds, r = nb % kXcds;
    const int x = b % kXcds;
    return x * q + (x < r ? x : r) + b / kXcds;
}

// The same with the tiles dealt to the XCDs in chunks, for work that is uneven
// from one end of the tiles to the other (see launch_step_batched_b).  Each round of
// eight chunks starts at another XCD, so that work that recurs every so many
// tiles does not fall to the same one.
__device__ __forceinline__ int xcd_chunk_tile(int b, int nb, int chunk)
{
    const int whole = nb / (kXcds * chunk) * (kXcds * chunk);
    if (b >= whole) return whole + xcd_tile(b - whole, nb - whole);
    const int l = b / kXcds, round = l / chunk;
    const int x = (b + round + round / kXcds + round / (kXcds * kXcds)) % kXcds;
    return (round * kXcds + x) * chunk + l % chunk;
}

// Rank of this lane's agent in cell c, counted into count[c]: neighbouring lanes
// of one cell (a caller whose order follows the places) count together, by the
// first of them.  Called by all lanes that have an agent, in index order.
__device__ __forceinline__ uint32_t count_run(uint32_t c, uint32_t *__restrict__ count)
{
    const int lane = threadIdx.x % kWave;
    const uint32_t before = (uint32_t)__shfl_up((int)c, 1, kWave);
    const uint64_t heads = __ballot(lane == 0 || before != c);
    const uint64_t live = __ballot(true);
    const int head = 63 - __clzll((long long)(heads & (~0ull >> (63 - lane))));
    const uint64_t after = head < 63 ? (heads >> (head + 1)) << (head + 1) : 0ull;
    const int end = after ? __ffsll((long long)after) - 1 : __popcll(live);
    uint32_t base = 0;
    if (lane == head) base = atomicAdd(&count[c], (uint32_t)(end - head));
    return (uint32_t)__shfl((int)base, head, kWave) + (uint32_t)(lane - head);
}

__device__ __forceinline__ float wave_min(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, kWave));
    return v;
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

// Inclusive prefix sum over the 64 lanes of a wavefront.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    const int lane = threadIdx.x % kWave;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive block scan of one value per thread; returns the exclusive prefix
// and writes the block total to *total (all threads).
template <int BLOCK>
__device__ uint32_t block_excl_scan(uint32_t v, uint32_t *total)
{
    __shared__ uint32_t wsum[BLOCK / kWave];
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    const uint32_t inc = wave_incl_scan(v);
    if (lane == kWave - 1) wsum[wid] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < BLOCK / kWave; ++k) {
        if (k < wid) base += wsum[k];
        tot += wsum[k];
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

// Block-wide (min x, min y, max x, max y).  Result valid in thread 0.
template <int kBlock>
__device__ float4 block_bbox(float4 b)
{
    __shared__ float4 red[kBlock / kWave];
    b.x = wave_min(b.x);
    b.y = wave_min(b.y);
    b.z = wave_max(b.z);
    b.w = wave_max(b.w);
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    if (lane == 0) red[wid] = b;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < kBlock / kWave; ++k) {
            b.x = fminf(b.x, red[k].x);
            b.y = fminf(b.y, red[k].y);
            b.z = fmaxf(b.z, red[k].z);
            b.w = fmaxf(b.w, red[k].w);
        }
    }
    return b;
}

// Grid geometry of one scene from its bounding box b = (min x, min y,
// max x, max y):
//   m  = stencil radius in cells, ceil(R_n / requested cell size)
//   cs = max(requested, R_n / m) * (1 + 1e-5), so that m * cs > R_n with a
//        margin far above the rounding of the FP64 cell coordinates
//   the cell size grows (and m is re-derived) until nx * ny <= max_cells;
//   non-finite boxes (NaN/Inf positions) collapse to a single cell.
// few_cells > 0 asks for so few cells where that costs nothing: those finer than
// R_n in any case, others up to kStretch R_n (see k_scan_scatter).
// Fills every field except cell_base, agent_base, n and seg_end.
constexpr double kStretch = 1.6;
__device__ __forceinline__ void grid_geometry(float4 b, float rn, float cs_req, int max_cells,
                                              GridMeta &g, int few_cells = 0)
{
    const bool finite = isfinite(b.x) && isfinite(b.y) && isfinite(b.z) && isfinite(b.w);
    const double w = finite ? (double)b.z - (double)b.x : 0.0;
    const double h = finite ? (double)b.w - (double)b.y : 0.0;
    const double c0 = cs_req > 0.0f ? (double)cs_req : (double)rn;
    int m = 1;
    double cs = c0, fx = 0.0, fy = 0.0;
    auto cells_of = [&](double c) {
        m = (int)ceil((double)rn / c - 1e-6);
        if (m < 1) m = 1;
        cs = fmax(c, (double)rn / m) * (1.0 + 1e-5);
        fx = floor(w / cs) + 1.0;
        fy = floor(h / cs) + 1.0;
        return fx * fy;
    };
    bool few = few_cells > 0;
    double limit = few && few_cells < max_cells ? few_cells : max_cells;
    double c = c0;
    for (int it = 0; it < 264; ++it) {
        if (few && (it == 64 || !(c <= kStretch * (double)rn))) {
            few = false;
            limit = max_cells;
            c = fmax(c0, (double)rn);
        }
        if (cells_of(c) <= limit) break;
        c *= 1.25;
    }
    if (!(fx * fy <= (double)max_cells) || !(cs > 0.0)) {
        // only for extents beyond ~1e19 cells or non-positive sizes: one
        // cell holding everything is slow but still exact
        m = 1;
        fx = 1.0;
        fy = 1.0;
        cs = fmax(w, h) + fabs((double)rn) + 1.0;
    }
    g.x0 = finite ? b.x : 0.0f;
    g.y0 = finite ? b.y : 0.0f;
    g.cs = (float)cs;
    g.rn = rn;
    g.nx = (int)fx;
    g.ny = (int)fy;
    g.m = m;
    g.n_cells = g.nx * g.ny;
    g.inv_cs = 1.0 / cs;
    g.rn2 = (double)rn * (double)rn;
}

Layout make_layout(int64_t n, int64_t n_scenes, int64_t max_cells);

inline int64_t default_max_cells(int64_t n) { return n * 2 > 4096 ? n * 2 : 4096; }

// Device pointers into one workspace.
struct Work {
    GridMeta *meta;
    float4 *partial;
    uint32_t *cell;
    uint32_t *rank;
    uint32_t *count;
    uint32_t *start;
    uint32_t *tiles;
    float2 *s0;   // cell order: position (what the neighbour scan reads)
    float4 *s1;   // cell order: (vx, vy, bits(tag), radius), see agent_tag
    float *guess; // caller order: radius of the neighbour scan kept from the last call (0: none)
};

Work bind(const Layout &L, void *ws);

// Grid build for one scene: bounding box, cell keys, counting sort, SoA
// gather into cell order.  Returns hipSuccess or the launch error.
// `clear` (nullable): clear_len words to be set to zero on the way.
hipError_t launch_grid_build(const orca_agents_in &in, int n, const orca_params &p,
                             const Layout &L, const Work &w, hipStream_t stream,
                             uint32_t *clear = nullptr, int64_t clear_len = 0);

// The same for a neighbour distance and a cell size; fine: a short distance, which
// takes many cells for the agents there are.
hipError_t launch_grid_build_rn(const orca_agents_in &in, int n, float rn, float cell_size,
                                const Layout &L, const Work &w, hipStream_t stream,
                                uint32_t *clear = nullptr, int64_t clear_len = 0, bool fine = false);

// Histogram scan and scatter into cell order; scan_meta supplies the number
// of cells (n_cells) and of agents (n) of the whole cell space.
hipError_t launch_scan_scatter(const orca_agents_in &in, int n, const Layout &L, const Work &w,
                               const GridMeta *scan_meta, hipStream_t stream);

// Batched form: many independent scenes, scene s owning caller indices
// [off[s], off[s+1]) and cells [2 off[s] + 64 s, 2 off[s+1] + 64 (s + 1)).
hipError_t launch_batched(const orca_agents_in &in, const orca_agents_out &out, int n,
                          const int32_t *scene_off, int n_scenes, const orca_params *params,
                          int k_max, bool acc, int block, const Layout &L, const Work &w,
                          int32_t *error_flag, const orca_step_events *ev,
                          hipStream_t stream);

// What the batched step kernels read.
struct BatchArgs {
    orca_agents_in in;
    orca_agents_out out;
    const GridMeta *meta;
    const orca_params *prm;
    const int32_t *off;
    int S;
    int n;
    const uint32_t *start;
    const float2 *s0;
    const float4 *s1;
    float *guess;  // per-agent radius of the neighbour scan kept between steps
};

// Scene of caller index i: the largest s with off[s] <= i (off ascending).
__device__ __forceinline__ int scene_of(const int32_t *__restrict__ off, int S, int i)
{
    int lo = 0, hi = S - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Scene of caller index i given the scene s0 of an index <= i (off
// ascending): a walk forward from s0, a step or two for the indices of one
// tile, instead of a binary search per index.
__device__ __forceinline__ int scene_from(const int32_t *__restrict__ off, int S, int s0, int i)
{
    int s = s0;
    while (s + 1 < S && off[s + 1] <= i) ++s;
    return s;
}

// Fused neighbour search + half-planes + LP + update for one scene; with
// nbr / cnt (nullable) also the neighbour lists the step used.
hipError_t launch_step(const orca_agents_in &in, const orca_agents_out &out, int n,
                       const orca_params &p, const Layout &L, const Work &w, int32_t *nbr,
                       int32_t *cnt, hipStream_t stream);

// Small crowds: a group of lanes per agent, over the grid or (whole) over the
// copies that launch_pack makes in caller order.  A lane per agent is one wavefront
// per SIMD up to 65,536 agents and takes a wavefront's latency however few they are;
// a group of 16 does the same work in more instructions, the fewer the more work
// an agent has.  The largest crowd that takes the form, by whole calls in us, group /
// lane, R_n 5 m (density and k decide; the density is not known where the form is
// chosen):
//   step          50,000: 0.05 /m^2, k 10 56 / 52; 0.25, k 10 71 / 92; 1.0, k 10 81 / 129;
//                 66,560: 61 / 54, 84 / 97, 99 / 131, but 51 / 43 at 0.01; 100,000 (k 20,
//                 2 /m^2) 308 / 279
//   k up to 4     16,384: 0.02 33 / 34, 0.5 34 / 37; 32,769: 41 / 36, 50 / 46
//   hard lines    98,304: 0.05, k 20 105 / 96; 0.35, k 16 151 / 181; 131,072: 131 / 95, 186
//                 / 230, 0.01, k 10 110 / 77
//                 k up to 4: 66,560 0.02 73 / 79, 0.5 102 / 103; 98,304 93 / 83, 132 / 112
//   adjoint       32,769: 0.05, k 10 66 / 72, 1.0 106 / 147; 50,000 74 / 73, 165 / 152
//   hard lines    66,560: 0.05, k 10 122 / 114, 0.25 158 / 176, 2 /m^2, k 20 199 / 272
//                 k up to 4: 66,560 0.02 113 / 93, 0.5 156 / 122
//   lists         50,000: 0.05, k 8 38 / 33, 0.35, k 16 45 / 41, 1.0, k 10 46 / 66, one agent 7
//                 km away 75 / 188; k 32 (a network of 64) 200,000 146 / 158, 300,000 203 / 217
//                 k up to 4: 50,000 0.02 37 / 33, 0.5 40 / 36
//   batched step  see launch_batched
// Without a grid, each agent scanning the whole crowd: 1,500 agents 31 / 34, 2,500
// 40 / 35 (256 agents: 15 us, bound by the host).
constexpr int kGroup = 16;  // lanes per agent
constexpr int kWholeMax = 2048;
constexpr int kGroupStepMax = 72000, kGroupStepMaxHard = 98304;
constexpr int kGroupAdjointMax = 49152, kGroupAdjointMaxHard = 72000;
constexpr int kBriefList = 4;  // lists so short that a lane has little to do
constexpr int kGroupStepMaxBrief = 16384, kGroupStepMaxBriefHard = 72000;
constexpr int kGroupAdjointMaxBriefHard = 49152;
constexpr int kGroupListMax = 65536, kGroupListMaxLarge = 262144, kGroupListMaxBrief = 49152;
constexpr int kGroupBatchMax = 98304;
// The adjoint of more agents, two wavefronts per SIMD, walks LP3 by the lane where the
// lists are short (see wave_lp3).
constexpr int kWalkAgents = 131072;
inline bool has_hard_lines(const orca_params &p)
{
    return p.accel[0] > 0.0f || p.accel[1] > 0.0f || p.turn[0] > 0.0f || p.turn[1] > 0.0f;
}
inline int group_step_max(const orca_params &p)
{
    const bool brief = p.max_neighbors <= kBriefList;
    if (has_hard_lines(p)) return brief ? kGroupStepMaxBriefHard : kGroupStepMaxHard;
    return brief ? kGroupStepMaxBrief : kGroupStepMax;
}
inline int group_adjoint_max(const orca_params &p)
{
    if (!has_hard_lines(p)) return kGroupAdjointMax;
    return p.max_neighbors <= kBriefList ? kGroupAdjointMaxBriefHard : kGroupAdjointMaxHard;
}
inline int group_list_max(const orca_params &p)
{
    return p.max_neighbors <= kBriefList ? kGroupListMaxBrief
           : p.max_neighbors > 24        ? kGroupListMaxLarge
                                         : kGroupListMax;
}
// What a scan of the whole crowd needs of a grid.
__device__ __forceinline__ GridMeta whole_crowd(int n, float rn)
{
    GridMeta g{};
    g.rn = rn;
    g.rn2 = (double)rn * (double)rn;
    g.n = n;
    g.seg_end = (uint32_t)n;
    return g;
}
hipError_t launch_pack(const orca_agents_in &in, int n, const Work &w, hipStream_t stream,
                       uint32_t *clear = nullptr, int64_t clear_len = 0);
hipError_t launch_step_group(const orca_agents_in &in, const orca_agents_out &out, int n,
                             const orca_params &prm, const Work &w, bool whole, int32_t *nbr,
                             int32_t *cnt, hipStream_t stream);

// Neighbour lists by groups of lanes; the batched step by groups of lanes.
hipError_t launch_list_group(int n, const orca_params &prm, const Work &w, int32_t *nbr,
                             int32_t *cnt, hipStream_t stream);
hipError_t launch_batched_group(const BatchArgs &a, int k_max, bool acc, hipStream_t stream);

// Neighbour lists only (caller order), for orca_build_grid.
hipError_t launch_knn_export(const orca_agents_in &in, int n, const orca_params &p,
                             const Layout &L, const Work &w, int32_t *nbr, int32_t *cnt,
                             hipStream_t stream);

hipError_t launch_fill_zero(void *ws, size_t bytes, hipStream_t stream);

// Agent lifecycle (leaving at the goal, entering at clear spawn points).
size_t lifecycle_bytes(int64_t n, int64_t n_cand);
hipError_t launch_remove_arrived(const orca_agents_in &in, const orca_agents_buf &out, int n,
                                 int32_t *n_alive, int32_t *old_to_new, void *extra,
                                 hipStream_t stream);
size_t overlap_extra_bytes(int64_t n);
hipError_t launch_overlap_stats(const orca_agents_in &in, int n, float reach, double *out,
                                const Layout &L, const Work &w, void *extra, hipStream_t stream);
hipError_t launch_spawn(const orca_agents_buf &state, int n, const orca_agents_in &cand,
                        int n_cand, float t_clear, int32_t *n_total, uint8_t *accepted, void *extra,
                        hipStream_t stream);

// Extra workspace of the adjoint: per-agent tau contributions and the edge
// list (3 per agent) of contributions to neighbours, found again by target.
constexpr int kEdgeSlots = 8;  // edges of a target found directly
struct AdjointBufs {
    float *tau_part;     // n
    float4 *e_val;       // 3n: (gp.x, gp.y, gv.x, gv.y) for the edge's target
    uint32_t *e_list;    // kEdgeSlots n: each target's first edges
    uint32_t *e_next;    // 3n: edge before this one (+ 1) in its target's chain
    uint32_t *e_cnt;     // n: edges of each target } cleared by the
    uint32_t *e_head;    // n: end of its chain + 1 } kernels before the adjoint
    double *tau_blocks;  // partial sums of the tau contributions
};

size_t adjoint_extra_bytes(int64_t n);
AdjointBufs bind_adjoint(int64_t n, void *base);

hipError_t launch_adjoint(const orca_agents_in &in, int n, const orca_params &prm,
                          const Layout &L, const Work &w, const AdjointBufs &b,
                          const float *gpx1, const float *gpy1, const float *gvx1,
                          const float *gvy1, float *gpx0, float *gpy0, float *gvx0, float *gvy0,
                          float *gprx, float *gpry, float *g_tau, const orca_step_events *ev,
                          hipStream_t stream);

}  // namespace orca
