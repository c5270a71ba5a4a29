// Uniform-grid build for one scene: bounding box -> cell keys -> counting sort
// -> cell-ordered SoA copy.  The grid only bounds which agents are examined as
// neighbour candidates (Sec. 1 and Sec. 3 use a grid spatial partition for
// the "nearby agents" query); the neighbour set itself is defined exactly
// and does not depend on the cell size.
#include "orca_internal.h"

#include <math.h>

namespace orca {

namespace {

constexpr int kBlock = 256;
// Crowds whose bounding box takes at most this many blocks of (1) form the
// grid geometry inside (3) (see k_cell_count).
constexpr int kFusedParts = 128;

// (1) partial bounding boxes; also clears the cell histogram for (3), and what
// else the caller wants cleared.
__global__ __launch_bounds__(kBlock) void k_bbox_partial(const float *__restrict__ px,
                                                         const float *__restrict__ py, int n,
                                                         float4 *__restrict__ partial,
                                                         uint32_t *__restrict__ count,
                                                         int count_len,
                                                         uint32_t *__restrict__ clear,
                                                         int64_t clear_len)
{
    float4 b = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
    const int stride = gridDim.x * kBlock;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
        const float x = px[i], y = py[i];
        b.x = fminf(b.x, x);
        b.y = fminf(b.y, y);
        b.z = fmaxf(b.z, x);
        b.w = fmaxf(b.w, y);
    }
    for (int c = blockIdx.x * kBlock + threadIdx.x; c < count_len; c += stride) count[c] = 0u;
    for (int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x; c < clear_len; c += stride)
        clear[c] = 0u;
    b = block_bbox<kBlock>(b);
    if (threadIdx.x == 0) partial[blockIdx.x] = b;
}

// (2) one block: final bounding box and grid geometry (grid_geometry).
__global__ __launch_bounds__(kBlock) void k_grid_setup(const float4 *__restrict__ partial,
                                                       int n_partial, float rn, float cs_req,
                                                       int max_cells, int n,
                                                       GridMeta *__restrict__ meta)
{
    float4 b = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
    for (int k = threadIdx.x; k < n_partial; k += kBlock) {
        const float4 q = partial[k];
        b.x = fminf(b.x, q.x);
        b.y = fminf(b.y, q.y);
        b.z = fmaxf(b.z, q.z);
        b.w = fmaxf(b.w, q.w);
    }
    b = block_bbox<kBlock>(b);
    if (threadIdx.x != 0) return;
    GridMeta g;
    grid_geometry(b, rn, cs_req, max_cells, g);
    g.cell_base = 0;
    g.agent_base = 0;
    g.n = n;
    g.seg_end = (uint32_t)n;
    *meta = g;
}

// (3) cell key and rank inside the cell (atomic counting).  With `partial`
// (small crowds, at most kFusedParts boxes from (1)) every block also does
// (2) itself: it combines the boxes and forms the geometry (grid_geometry,
// the same bits in every block), and block 0 stores it for the kernels
// after this one; a crowd of 16,384 agents then saves the one-block launch.
// Without it (large crowds, whose (1) runs many more blocks than a block of
// (3) could combine cheaply) the geometry comes from (2) through `meta`.
__global__ __launch_bounds__(kBlock) void k_cell_count(const float *__restrict__ px,
                                                       const float *__restrict__ py, int n,
                                                       const float4 *__restrict__ partial,
                                                       int n_partial, float rn, float cs_req,
                                                       int max_cells, int few_cells,
                                                       GridMeta *__restrict__ meta,
                                                       uint32_t *__restrict__ cell,
                                                       uint32_t *__restrict__ rank,
                                                       uint32_t *__restrict__ count)
{
    GridMeta g;
    if (partial) {
        __shared__ GridMeta gs;
        float4 b = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
        for (int k = threadIdx.x; k < n_partial; k += kBlock) {
            const float4 q = partial[k];
            b.x = fminf(b.x, q.x);
            b.y = fminf(b.y, q.y);
            b.z = fmaxf(b.z, q.z);
            b.w = fmaxf(b.w, q.w);
        }
        b = block_bbox<kBlock>(b);
        if (threadIdx.x == 0) {
            GridMeta h;
            grid_geometry(b, rn, cs_req, max_cells, h, few_cells);
            h.cell_base = 0;
            h.agent_base = 0;
            h.n = n;
            h.seg_end = (uint32_t)n;
            gs = h;
            if (blockIdx.x == 0) *meta = h;
        }
        __syncthreads();
        g = gs;
    } else {
        g = *meta;
    }
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const int cx = cell_axis(px[i], g.x0, g.inv_cs, g.nx);
    const int cy = cell_axis(py[i], g.y0, g.inv_cs, g.ny);
    const uint32_t c = (uint32_t)(cx + g.nx * cy);
    cell[i] = c;
    rank[i] = count_run(c, count);
}

constexpr int kPer = kScanTile / kBlock;  // 8 cells per thread

// (4a) per-tile sums of the histogram.
__global__ __launch_bounds__(kBlock) void k_scan_reduce(const uint32_t *__restrict__ count,
                                                        const GridMeta *__restrict__ meta,
                                                        uint32_t *__restrict__ tiles)
{
    const int n_cells = meta->n_cells;
    const int base = blockIdx.x * kScanTile;
    if (base >= n_cells) return;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int c = base + threadIdx.x * kPer + k;
        if (c < n_cells) s += count[c];
    }
    uint32_t tot;
    block_excl_scan<kBlock>(s, &tot);
    if (threadIdx.x == 0) tiles[blockIdx.x] = tot;
}

// (4b) exclusive scan inside each tile, offset by the tile's prefix: the sum
// of the tile sums of (4a) before it, which every block adds up itself (at
// most a few thousand words from L2, in place of a one-block scan kernel
// between the two).
__global__ __launch_bounds__(kBlock) void k_scan_apply(const uint32_t *__restrict__ count,
                                                       const uint32_t *__restrict__ tiles,
                                                       const GridMeta *__restrict__ meta,
                                                       uint32_t *__restrict__ start)
{
    const GridMeta g = *meta;
    const int base = blockIdx.x * kScanTile;
    if (base >= g.n_cells) return;
    uint32_t before = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += kBlock) before += tiles[t];
    uint32_t prefix;
    block_excl_scan<kBlock>(before, &prefix);
    uint32_t v[kPer];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int c = base + threadIdx.x * kPer + k;
        v[k] = c < g.n_cells ? count[c] : 0u;
        s += v[k];
    }
    uint32_t tot;
    uint32_t run = prefix + block_excl_scan<kBlock>(s, &tot);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int c = base + threadIdx.x * kPer + k;
        if (c < g.n_cells) start[c] = run;
        run += v[k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) start[g.n_cells] = (uint32_t)g.n;
}

// (5) scatter into cell order: position = start[cell] + rank.
// What bounds it is the writes: two small records per agent to scattered
// positions, lines of which a block of another XCD also writes parts.  Each XCD
// therefore takes a contiguous range of agents (xcd_tile): where callers hold
// neighbours together, as the scenes of a batch are, its L2 then has the whole
// line before it writes it back (512 scenes, 5.6M agents: 201 -> 140 us,
// the whole step 3.17 -> 3.11 ms; 1M agents in random order: 10.5 us either way).
__global__ __launch_bounds__(kBlock) void k_scatter(orca_agents_in in, int n,
                                                    const uint32_t *__restrict__ cell,
                                                    const uint32_t *__restrict__ rank,
                                                    const uint32_t *__restrict__ start,
                                                    float2 *__restrict__ s0,
                                                    float4 *__restrict__ s1)
{
    const int i = xcd_tile(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    if (i >= n) return;
    const uint32_t pos = start[cell[i]] + rank[i];
    if (pos >= (uint32_t)n) return;  // cannot happen for a consistent histogram
    write_record(in, i, pos, s0, s1);
}

// (4 + 5) for a small crowd, which spends its time on launches: two fewer.  Every
// block has the whole histogram to go through, so blocks are as large as they
// can be, and each loads its share at once.
//   up to kTable cells: scanned into a table in LDS, an agent reads its start there;
//   more: summed by runs of kSub cells (8 lanes a run), the sums scanned in LDS;
//         an agent's start is its run's prefix and what the run holds before its
//         cell.
// The starts are also stored for the kernels after this one, each block a part of
// them.  Whole builds in us, five launches / this: 16,384 agents in 2,304 cells 19.1
// / 14.2, 20,000 in 28,390 cells 28.1 / 23.6, 32,768 in them 21.5 / 23.9.  The
// geometry therefore asks for kTable cells where larger ones cost nothing (the
// group kernels take a row's candidates 16 at a time).  (With kTable as the limit a
// crowd spread wide had far larger cells than it asked for: 30,000 agents, one of
// them 7 km away, 2^20 cells allowed, lists 61 us in five launches, 206 with the
// limit, 42 now.)
constexpr int kTable = 8192;
constexpr int kSub = 32;
constexpr int kSmallCells = 131072 + kSub;  // workspaces of up to 65,536 agents by default
constexpr int kSubs = kSmallCells / kSub;
static_assert(kSubs <= kTable, "run sums take the table's place");

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_scan_scatter(orca_agents_in in, int n,
                                                        const uint32_t *__restrict__ cell,
                                                        const uint32_t *__restrict__ rank,
                                                        const uint32_t *__restrict__ count,
                                                        const GridMeta *__restrict__ meta,
                                                        uint32_t *__restrict__ start,
                                                        float2 *__restrict__ s0,
                                                        float4 *__restrict__ s1)
{
    __shared__ uint32_t table[kTable];
    const int n_cells = min(meta->n_cells, kSmallCells);
    const int tid = threadIdx.x;
    const int i = blockIdx.x * BLOCK + tid;
    const uint32_t mine = i < n ? min(cell[i], (uint32_t)n_cells - 1u) : 0u;
    uint32_t pos = i < n ? rank[i] : 0u;
    // (the count's region is a multiple of a run long; past the cells in use it is
    // not read into a sum)
    const uint4 *four = (const uint4 *)count;
    const int last = (n_cells - 1) / 4;
    auto cells4 = [&](int c) {  // counts of cells c .. c + 3, 0 past the last one
        uint4 v = four[min(c / 4, last)];
        v.x = c < n_cells ? v.x : 0u;
        v.y = c + 1 < n_cells ? v.y : 0u;
        v.z = c + 2 < n_cells ? v.z : 0u;
        v.w = c + 3 < n_cells ? v.w : 0u;
        return v;
    };
    uint32_t tot;
    if (n_cells <= kTable) {
        uint32_t before = 0;
        for (int c0 = tid * 8; c0 - tid * 8 < n_cells; c0 += BLOCK * 8) {
            const uint4 a = cells4(c0), b = cells4(c0 + 4);
            const uint32_t v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            uint32_t s = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) s += v[k];
            uint32_t run = before + block_excl_scan<BLOCK>(s, &tot);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (c0 + k < n_cells) {
                    table[c0 + k] = run;
                    if (blockIdx.x == 0) start[c0 + k] = run;
                }
                run += v[k];
            }
            before += tot;
        }
        __syncthreads();
        pos += table[mine];
    } else {
        const int n_sub = (n_cells + kSub - 1) / kSub;
        constexpr int kLanes = kSub / 4, kGroups = BLOCK / kLanes, kLoads = 16;
        for (int q0 = tid / kLanes; q0 < n_sub; q0 += kLoads * kGroups) {
            uint4 v[kLoads];
#pragma unroll
            for (int u = 0; u < kLoads; ++u)
                v[u] = cells4((q0 + u * kGroups) * kSub + tid % kLanes * 4);
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                uint32_t t = v[u].x + v[u].y + v[u].z + v[u].w;
#pragma unroll
                for (int o = kLanes / 2; o > 0; o >>= 1) t += (uint32_t)__shfl_xor((int)t, o, kLanes);
                if (tid % kLanes == 0 && q0 + u * kGroups < n_sub) table[q0 + u * kGroups] = t;
            }
        }
        __syncthreads();
        constexpr int kPerThread = (kSubs + BLOCK - 1) / BLOCK;
        uint32_t v[kPerThread], s = 0;
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int q = tid * kPerThread + k;
            v[k] = q < n_sub ? table[q] : 0u;
            s += v[k];
        }
        uint32_t run = block_excl_scan<BLOCK>(s, &tot);
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int q = tid * kPerThread + k;
            if (q < n_sub) table[q] = run;
            run += v[k];
        }
        __syncthreads();
        for (int q = blockIdx.x * (BLOCK / kSub) + tid / kSub; q < n_sub;
             q += gridDim.x * (BLOCK / kSub)) {
            const int c = q * kSub + tid % kSub;
            uint32_t before = c < n_cells ? count[c] : 0u;
            const uint32_t have = before;
#pragma unroll
            for (int o = 1; o < kSub; o <<= 1) {
                const uint32_t t = (uint32_t)__shfl_up((int)before, o, kSub);
                before += tid % kSub >= o ? t : 0u;
            }
            if (c < n_cells) start[c] = table[q] + before - have;
        }
        if (i < n) {
            const int in_run = (int)mine % kSub, c0 = (int)mine - in_run;
            pos += table[c0 / kSub];
            for (int q0 = 0; q0 < in_run; q0 += 16) {
                uint4 h[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) h[u] = cells4(c0 + q0 + 4 * u);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int q = q0 + 4 * u;
                    pos += (q < in_run ? h[u].x : 0u) + (q + 1 < in_run ? h[u].y : 0u) +
                           (q + 2 < in_run ? h[u].z : 0u) + (q + 3 < in_run ? h[u].w : 0u);
                }
            }
        }
    }
    if (blockIdx.x == 0 && tid == 0) start[n_cells] = (uint32_t)n;
    if (i >= n || pos >= (uint32_t)n) return;  // the latter cannot happen for a consistent histogram
    write_record(in, i, pos, s0, s1);
}

__global__ void k_fill_zero(uint4 *p, size_t n16)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n16; k += stride)
        p[k] = make_uint4(0, 0, 0, 0);
}

}  // namespace

namespace {

// (1) to (3), with at most max_cells cells (few_cells: see grid_geometry; of crowds
// whose geometry is formed in (3)).
void launch_count(const orca_agents_in &in, int n, float rn, float cell_size, int max_cells,
                  int few_cells, const Work &w, hipStream_t stream, uint32_t *clear,
                  int64_t clear_len)
{
    const int nb = (int)((n + kBlock - 1) / kBlock);
    const int nbb = nb < kBboxBlocks ? nb : kBboxBlocks;
    hipLaunchKernelGGL(k_bbox_partial, dim3(nbb), dim3(kBlock), 0, stream, in.px, in.py, n,
                       w.partial, w.count, max_cells, clear, clear_len);
    const bool fused = nbb <= kFusedParts;
    if (!fused)
        hipLaunchKernelGGL(k_grid_setup, dim3(1), dim3(kBlock), 0, stream, w.partial, nbb, rn,
                           cell_size, max_cells, n, w.meta);
    hipLaunchKernelGGL(k_cell_count, dim3(nb), dim3(kBlock), 0, stream, in.px, in.py, n,
                       fused ? w.partial : nullptr, nbb, rn, cell_size, max_cells, few_cells,
                       w.meta, w.cell, w.rank, w.count);
}
}  // namespace

hipError_t launch_grid_build(const orca_agents_in &in, int n, const orca_params &p,
                             const Layout &L, const Work &w, hipStream_t stream, uint32_t *clear,
                             int64_t clear_len)
{
    return launch_grid_build_rn(in, n, p.neighbor_dist, p.cell_size, L, w, stream, clear, clear_len);
}

hipError_t launch_grid_build_rn(const orca_agents_in &in, int n, float rn, float cell_size,
                                const Layout &L, const Work &w, hipStream_t stream, uint32_t *clear,
                                int64_t clear_len, bool fine)
{
    const int nb = (int)((n + kBlock - 1) / kBlock);
    // (a workspace that allows more cells is used as it asks: how many the crowd
    // needs is known on the device only; a short reach needs many: overlap statistics
    // of 16,384 agents at 0.5 /m^2 within 1.5 m 27.4 us in five launches, 28.9 in three,
    // 5,000 26.6 and 24.7)
    const bool small = nb <= kFusedParts && L.max_cells <= (fine ? 2 * kTable : kSmallCells);
    launch_count(in, n, rn, cell_size, (int)L.max_cells, small ? kTable : 0, w, stream, clear,
                 clear_len);
    if (!small) return launch_scan_scatter(in, n, L, w, w.meta, stream);
    // (4,999 agents in 770 cells: 4.2 us at 256 lanes, 5.2 at 1,024)
    if (L.max_cells <= 2 * kTable)
        hipLaunchKernelGGL((k_scan_scatter<kBlock>), dim3(nb), dim3(kBlock), 0, stream, in, n, w.cell,
                           w.rank, w.count, w.meta, w.start, w.s0, w.s1);
    else
        hipLaunchKernelGGL((k_scan_scatter<1024>), dim3((n + 1023) / 1024), dim3(1024), 0, stream, in,
                           n, w.cell, w.rank, w.count, w.meta, w.start, w.s0, w.s1);
    return hipGetLastError();
}

hipError_t launch_scan_scatter(const orca_agents_in &in, int n, const Layout &L, const Work &w,
                               const GridMeta *scan_meta, hipStream_t stream)
{
    const int nb = (int)((n + kBlock - 1) / kBlock);
    const int nt = (int)L.n_tiles;
    hipLaunchKernelGGL(k_scan_reduce, dim3(nt), dim3(kBlock), 0, stream, w.count, scan_meta,
                       w.tiles);
    hipLaunchKernelGGL(k_scan_apply, dim3(nt), dim3(kBlock), 0, stream, w.count, w.tiles,
                       scan_meta, w.start);
    hipLaunchKernelGGL(k_scatter, dim3(nb), dim3(kBlock), 0, stream, in, n, w.cell, w.rank,
                       w.start, w.s0, w.s1);
    return hipGetLastError();
}

hipError_t launch_fill_zero(void *ws, size_t bytes, hipStream_t stream)
{
    const size_t n16 = bytes / 16;
    if (n16) {
        size_t blocks = (n16 + 255) / 256;
        if (blocks > 4096) blocks = 4096;
        hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, stream, (uint4 *)ws,
                           n16);
    }
    return hipGetLastError();
}

}  // namespace orca
