// Batched ORCA step: many independent scenes of uneven sizes advanced by one
// set of launches per step (batched form; not in the paper, which simulates
// one scene).
//
// Scene s owns caller indices [off[s], off[s+1]) and the cells
// [2 off[s] + 64 s, 2 off[s+1] + 64 (s+1)) of one global cell space, so a
// single histogram, scan and scatter order every scene at once and each scene
// stays contiguous in cell order (its agents fill exactly the positions
// [off[s], off[s+1])).  Agents of different scenes never share a cell and so
// never see each other.
//
// The step kernel takes one 64-agent tile per wavefront in an XCD-aware order
// (neighbouring tiles stay in one L2), small batches a group of lanes per agent.
#include "orca_device.h"

namespace orca {
namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ int clamp_off(int v, int n) { return v < 0 ? 0 : (v > n ? n : v); }

// (1) kBboxSplit blocks per scene: partial bounding boxes of its agents (a
// block per scene left the largest scenes to one block each).  All blocks
// also clear the histogram; scene offsets and
// parameters are checked and any violation is flagged (the kernels stay in
// bounds regardless: offsets are clamped to [0, n]).
__global__ __launch_bounds__(kBlock) void k_batch_bbox(const float *__restrict__ px,
                                                       const float *__restrict__ py, int n,
                                                       const int32_t *__restrict__ off, int S,
                                                       const orca_params *__restrict__ prm,
                                                       float4 *__restrict__ partial,
                                                       uint32_t *__restrict__ count, int count_len,
                                                       int32_t *__restrict__ error_flag,
                                                       int has_accel)
{
    const int s = blockIdx.x / kBboxSplit, part = blockIdx.x % kBboxSplit;
    const int a = clamp_off(off[s], n), b = clamp_off(off[s + 1], n);
    float4 bb = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
    for (int i = a + part * kBlock + threadIdx.x; i < b; i += kBlock * kBboxSplit) {
        const float x = px[i], y = py[i];
        bb.x = fminf(bb.x, x);
        bb.y = fminf(bb.y, y);
        bb.z = fmaxf(bb.z, x);
        bb.w = fmaxf(bb.w, y);
    }
    const int stride = gridDim.x * kBlock;
    for (int c = blockIdx.x * kBlock + threadIdx.x; c < count_len; c += stride) count[c] = 0u;
    bb = block_bbox<kBlock>(bb);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = bb;
        if (error_flag && part == 0) {
            const orca_params p = prm[s];
            bool bad = off[s] > off[s + 1] || off[s] < 0 || off[s + 1] > n;
            if (s == 0) bad = bad || off[0] != 0;
            if (s == S - 1) bad = bad || off[S] != n;
            bad = bad || !(p.dt > 0.0f) || !(p.time_horizon > 0.0f) ||
                  !(p.neighbor_dist > 0.0f) || !(p.cell_size >= 0.0f) ||
                  p.max_neighbors < 1 || p.max_neighbors > ORCA_K_MAX ||
                  (p.pref_is_goal != 0 && p.pref_is_goal != 1) ||
                  !(p.accel[0] >= 0.0f) || !(p.accel[1] >= 0.0f) ||
                  !isfinite(p.accel[0]) || !isfinite(p.accel[1]) ||
                  !(p.turn[0] >= 0.0f) || !(p.turn[1] >= 0.0f) ||
                  !isfinite(p.turn[0]) || !isfinite(p.turn[1]) ||
                  (!has_accel && (p.accel[0] > 0.0f || p.accel[1] > 0.0f ||
                                  p.turn[0] > 0.0f || p.turn[1] > 0.0f));
            if (bad) atomicOr(error_flag, 1);
        }
    }
}

// (2) one thread per scene: grid geometry within the scene's cell budget.
// meta[S] describes the whole cell space for the scan.
__global__ __launch_bounds__(kBlock) void k_batch_setup(const float4 *__restrict__ partial,
                                                        const int32_t *__restrict__ off, int S,
                                                        int n, const orca_params *__restrict__ prm,
                                                        GridMeta *__restrict__ meta)
{
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s == 0) {
        GridMeta g{};
        g.n_cells = (int)batched_cells(n, S);
        g.n = n;
        g.seg_end = (uint32_t)n;
        meta[S] = g;
    }
    if (s >= S) return;
    const int a = clamp_off(off[s], n);
    const int b = max(clamp_off(off[s + 1], n), a);
    const int budget = 2 * (b - a) + 64;
    float4 bb = partial[s * kBboxSplit];
    for (int q = 1; q < kBboxSplit; ++q) {
        const float4 p = partial[s * kBboxSplit + q];
        bb = make_float4(fminf(bb.x, p.x), fminf(bb.y, p.y), fmaxf(bb.z, p.z), fmaxf(bb.w, p.w));
    }
    GridMeta g;
    grid_geometry(bb, prm[s].neighbor_dist, prm[s].cell_size, budget, g);
    // a budget is 2 cells per agent plus 64; the cell ranges of consecutive
    // scenes tile the global cell space when offsets are valid and stay
    // inside it otherwise
    g.cell_base = 2 * a + 64 * s;
    g.agent_base = a;
    g.n = b - a;
    g.seg_end = (uint32_t)b;
    meta[s] = g;
}

// (3) scene, cell and rank inside the cell.
__global__ __launch_bounds__(kBlock) void k_batch_count(const float *__restrict__ px,
                                                        const float *__restrict__ py, int n,
                                                        const int32_t *__restrict__ off, int S,
                                                        const GridMeta *__restrict__ meta,
                                                        uint32_t *__restrict__ cell,
                                                        uint32_t *__restrict__ rank,
                                                        uint32_t *__restrict__ count)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const GridMeta g = meta[scene_of(off, S, i)];
    const int cx = cell_axis(px[i], g.x0, g.inv_cs, g.nx);
    const int cy = cell_axis(py[i], g.y0, g.inv_cs, g.ny);
    const uint32_t c = (uint32_t)(g.cell_base + cx + g.nx * cy);
    cell[i] = c;
    rank[i] = count_run(c, count);
}

// The agent at cell-order position s (all lanes of the wavefront call it; one
// past the last agent takes part without an agent of its own).
template <int K, int BLOCK, bool ACC>
__device__ __forceinline__ void batch_agent(const BatchArgs &a, int s, int first, float4 *lines,
                                            int tid)
{
    const bool live = s < a.n;
    s = min(s, a.n - 1);
    const int sc = scene_from(a.off, a.S, first, s);
    const GridMeta g = a.meta[sc];
    const dev::SceneP p = dev::scene_params(a.prm[sc]);
    dev::step_agent<K, BLOCK, ACC>(live, s, g, p, a.in, a.out, a.start, a.s0, a.s1, lines, tid,
                                   a.guess);
}

// The step: one 64-agent tile per wavefront, XCD-aware order.
template <int K, int BLOCK, bool ACC>
__global__ __launch_bounds__(BLOCK) void k_step_batched_flat(BatchArgs a, int chunk)
{
    __shared__ float4 lines[dev::KnnShape<K>::kSlots * BLOCK];
    const int tid = threadIdx.x;
    const int s0 = xcd_chunk_tile(blockIdx.x, gridDim.x, chunk) * BLOCK;
    batch_agent<K, BLOCK, ACC>(a, s0 + tid, scene_of(a.off, a.S, s0), lines, tid);
}

// Tiles that an XCD takes in one piece: the scenes of a batch can be far from
// alike, and with an eighth of the whole in one piece the XCD that has the dense
// ones ends last (kernel in us, in eighths / in chunks: 64 scenes of 16,384 agents,
// the first eight dense 912 / 320, dense ones spread over it 326 / 430, by how late
// the last of them starts; 6 scenes, 1M agents, all vehicles in the first, k 32
// 1473 / 1030).  Where all scenes are alike an eighth in one piece finds more of
// what the scatter wrote in its own L2, so the chunks are as large as eight for
// each XCD allow (8 scenes, 1M agents, 0.3 /m^2: 431 / 438 us a call, 512 scenes of
// all sizes 2628 / 2640), and batches whose tiles are all under way at once keep the
// eighths (8 scenes, 131,072 agents, 0.02 /m^2: 45 / 51).
constexpr int kChunkMax = 1024;
constexpr int kChunkAgents = 262144;  // batches of more agents


template <int K, int BLOCK>
hipError_t launch_step_batched_b(const BatchArgs &a, bool acc, hipStream_t stream)
{
    const int nb = (a.n + BLOCK - 1) / BLOCK;
    int chunk = nb;  // eighths: no whole round of chunks
    if (a.n > kChunkAgents) chunk = nb / (8 * kXcds) < kChunkMax ? nb / (8 * kXcds) : kChunkMax;
    if (acc)
        hipLaunchKernelGGL((k_step_batched_flat<K, BLOCK, true>), dim3(nb), dim3(BLOCK), 0, stream,
                           a, chunk);
    else
        hipLaunchKernelGGL((k_step_batched_flat<K, BLOCK, false>), dim3(nb), dim3(BLOCK), 0, stream,
                           a, chunk);
    return hipGetLastError();
}

// Workgroup size: one wavefront, whose LDS is free again as soon as it ends,
// unless the caller asks for 128 or 256 lanes.  512 scenes, 5.56M agents: 3.17
// ms at 64 lanes, 3.69 at 128, 3.87 at 256.  (Wavefronts that stay and pop tiles
// from a queue per XCD took 3.54 ms: the pops, and each wavefront's look at every
// queue at the end, are atomics on one line, 9 ns each; 3.41 ms with a line per
// queue.  The hardware's own dispatch balances as well and costs nothing.)
template <int K>
hipError_t launch_step_batched_k(const BatchArgs &a, bool acc, int block, hipStream_t stream)
{
    if (block == 128) return launch_step_batched_b<K, 128>(a, acc, stream);
    if (block == 256) return launch_step_batched_b<K, 256>(a, acc, stream);
    return launch_step_batched_b<K, 64>(a, acc, stream);
}

}  // namespace

hipError_t launch_batched(const orca_agents_in &in, const orca_agents_out &out, int n,
                          const int32_t *scene_off, int n_scenes, const orca_params *params,
                          int k_max, bool acc, int block, const Layout &L, const Work &w,
                          int32_t *error_flag, const orca_step_events *ev,
                          hipStream_t stream)
{
    const int S = n_scenes;
    const int nb = (n + kBlock - 1) / kBlock;
    if (ev && ev->grid_begin && hipEventRecord(ev->grid_begin, stream) != hipSuccess)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_batch_bbox, dim3(S * kBboxSplit), dim3(kBlock), 0, stream, in.px, in.py,
                       n, scene_off,
                       S, params, w.partial, w.count, (int)L.max_cells, error_flag,
                       acc ? 1 : 0);
    hipLaunchKernelGGL(k_batch_setup, dim3((S + kBlock - 1) / kBlock), dim3(kBlock), 0, stream,
                       w.partial, scene_off, S, n, params, w.meta);
    hipLaunchKernelGGL(k_batch_count, dim3(nb), dim3(kBlock), 0, stream, in.px, in.py, n,
                       scene_off, S, w.meta, w.cell, w.rank, w.count);
    hipError_t e = launch_scan_scatter(in, n, L, w, w.meta + S, stream);
    if (e != hipSuccess) return e;
    BatchArgs a;
    a.in = in;
    a.out = out;
    a.meta = w.meta;
    a.prm = params;
    a.off = scene_off;
    a.S = S;
    a.n = n;
    a.start = w.start;
    a.s0 = w.s0;
    a.s1 = w.s1;
    a.guess = w.guess;
    if (ev && ev->step_begin && hipEventRecord(ev->step_begin, stream) != hipSuccess)
        return hipErrorInvalidValue;
    // (8 scenes with vehicles, group / lane per agent: 72,000 agents 95 / 140 us,
    // 100,000 124 / 147, 150,000 158 / 155; pedestrians alone, k 10: 72,000 78 /
    // 78, 100,000 98 / 81)
    if (n <= kGroupBatchMax)
        e = launch_batched_group(a, k_max, acc, stream);
    else if (k_max <= 4)
        e = launch_step_batched_k<4>(a, acc, block, stream);
    else if (k_max <= 8)
        e = launch_step_batched_k<8>(a, acc, block, stream);
    else if (k_max <= 10)
        e = launch_step_batched_k<10>(a, acc, block, stream);
    else if (k_max <= 12)
        e = launch_step_batched_k<12>(a, acc, block, stream);
    else if (k_max <= 16)
        e = launch_step_batched_k<16>(a, acc, block, stream);
    else if (k_max <= 20)
        e = launch_step_batched_k<20>(a, acc, block, stream);
    else if (k_max <= 24)
        e = launch_step_batched_k<24>(a, acc, block, stream);
    else
        e = launch_step_batched_k<32>(a, acc, block, stream);
    if (e != hipSuccess) return e;
    if (ev && ev->step_end && hipEventRecord(ev->step_end, stream) != hipSuccess)
        return hipErrorInvalidValue;
    return hipSuccess;
}

}  // namespace orca
