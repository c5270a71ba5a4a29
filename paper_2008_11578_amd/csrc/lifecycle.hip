// Agent lifecycle of the crossing experiments (Sec. 4, first experiment):
// agents leave once they reach their goal, and new agents enter at spawn
// points that keep clear of everyone for a time window.
//
//  - leaving: a stable compaction (per-block counts, one scan block, move),
//    with the arrival test evaluated in double without fused multiply-add so
//    that the decision is exactly reproducible;
//  - entering: the candidates (a few thousand, in the start regions) are put
//    into a grid whose cells are as large as the widest clearance, computed on
//    the device from the largest radii and speed caps.  Every agent looks up
//    the candidates around it and blocks those too close; every candidate
//    lists the earlier candidates it conflicts with; and one workgroup
//    settles the first-come decisions in rounds (a candidate enters once all
//    its earlier conflicts are rejected, and is rejected as soon as one of
//    them enters), which equals taking the candidates one by one in order.
#include "orca_device.h"

#include <math.h>

namespace orca {
namespace {

constexpr int kBlock = 256;
constexpr int kScanThreads = 1024;
constexpr int kConfCap = 16;  // earlier conflicts listed per candidate
constexpr int kUndecided = 0, kAccepted = 1, kRejected = 2;
constexpr int kBoundBlocksMax = 1024;

// Grid over the spawn candidates.
constexpr int kCandCells = 8192;  // histogram of 32 KB in one workgroup's LDS
struct CandGrid {
    double x0, y0, inv;  // origin and 1 / cell size
    int nx, ny;
};

struct LifeBufs {
    uint32_t *block_count;  // leaving: survivors per block, then their offsets
    float4 *partial;        // entering: per-block maxima
    float4 *box;            // entering: per-block bounding boxes of the candidates
    CandGrid *grid;
    uint32_t *start;        // entering: first candidate of each cell (+ 1 entry)
    float4 *cand;           // entering: candidates in cell order (x, y, radius, speed cap)
    int32_t *index;         // entering: their places in the caller's order
    uint8_t *blocked;       // entering, in cell order: blocked by a current agent
    int32_t *decision;      // entering: places in cell order; then kUndecided, kAccepted or
                            // kRejected; then the place of an accepted candidate or -1
    int32_t *conf_count;    // entering: earlier conflicting candidates (may exceed the cap)
    int32_t *conf;          // entering: their indices, kConfCap per candidate
};

size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

LifeBufs bind_life(int64_t n, int64_t n_cand, void *base, size_t *bytes = nullptr)
{
    char *b = (char *)base;
    LifeBufs r;
    size_t o = 0;
    auto take = [&](size_t len) {
        char *p = b + o;
        o += a256(len);
        return p;
    };
    const size_t nc = (size_t)n_cand;
    r.block_count = (uint32_t *)take(sizeof(uint32_t) * (size_t)((n + kBlock - 1) / kBlock + 1));
    r.partial = (float4 *)take(sizeof(float4) * kBoundBlocksMax);
    r.box = (float4 *)take(sizeof(float4) * kBoundBlocksMax);
    r.grid = (CandGrid *)take(sizeof(CandGrid));
    r.start = (uint32_t *)take(sizeof(uint32_t) * (kCandCells + 1));
    r.cand = (float4 *)take(sizeof(float4) * nc);
    r.index = (int32_t *)take(sizeof(int32_t) * nc);
    r.blocked = (uint8_t *)take(nc);
    r.decision = (int32_t *)take(sizeof(int32_t) * nc);
    r.conf_count = (int32_t *)take(sizeof(int32_t) * nc);
    r.conf = (int32_t *)take(sizeof(int32_t) * kConfCap * nc);
    if (bytes) *bytes = o;
    return r;
}

// Reaching the goal: |g - p|^2 <= r^2 in double, operations rounded
// separately (the same expression as the oracle's).
__device__ __forceinline__ bool arrived(float px, float py, float gx, float gy, float r)
{
#pragma clang fp contract(off)
    const double dx = (double)gx - (double)px;
    const double dy = (double)gy - (double)py;
    const double rr = (double)r;
    return dx * dx + dy * dy <= rr * rr;
}

// Two discs that could touch within t seconds at full speed.
__device__ __forceinline__ bool too_close(float ax, float ay, float ar, float as, float bx, float by,
                                          float br, float bs, double t)
{
#pragma clang fp contract(off)
    const double dx = (double)bx - (double)ax;
    const double dy = (double)by - (double)ay;
    const double d = ((double)ar + (double)br) + t * ((double)as + (double)bs);
    return dx * dx + dy * dy < d * d;
}

// (leaving 1) survivors per block
__global__ __launch_bounds__(kBlock) void k_arrive_count(orca_agents_in in, int n,
                                                          uint32_t *__restrict__ block_count)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    bool keep = false;
    if (i < n) keep = !arrived(in.px[i], in.py[i], in.pref_x[i], in.pref_y[i], in.radius[i]);
    const int c = __syncthreads_count(keep);
    if (threadIdx.x == 0) block_count[blockIdx.x] = (uint32_t)c;
}

// Exclusive scan of `count[0 .. m)` in place by one block; total to *sum.
__device__ void block_exclusive_scan(uint32_t *count, int m, uint32_t *sum)
{
    __shared__ uint32_t part[kScanThreads];
    const int tid = threadIdx.x;
    const int per = (m + kScanThreads - 1) / kScanThreads;
    const int a = tid * per, b = min(a + per, m);
    uint32_t s = 0;
    for (int k = a; k < b; ++k) s += count[k];
    part[tid] = s;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        const uint32_t v = tid >= off ? part[tid - off] : 0u;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    uint32_t run = tid ? part[tid - 1] : 0u;
    for (int k = a; k < b; ++k) {
        const uint32_t c = count[k];
        count[k] = run;
        run += c;
    }
    if (tid == kScanThreads - 1) *sum = part[tid];
}

// (leaving 2) block offsets and the survivor count
__global__ __launch_bounds__(kScanThreads) void k_arrive_scan(uint32_t *__restrict__ block_count,
                                                              int nb, int32_t *__restrict__ n_alive)
{
    __shared__ uint32_t total;
    block_exclusive_scan(block_count, nb, &total);
    __syncthreads();
    if (threadIdx.x == 0) *n_alive = (int32_t)total;
}

// (leaving 3) move the survivors, keeping their order
__global__ __launch_bounds__(kBlock) void k_arrive_move(orca_agents_in in, orca_agents_buf out,
                                                         int n,
                                                         const uint32_t *__restrict__ block_off,
                                                         int32_t *__restrict__ old_to_new)
{
    __shared__ uint32_t wave_base[kBlock / kWave];
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    bool keep = false;
    if (i < n) keep = !arrived(in.px[i], in.py[i], in.pref_x[i], in.pref_y[i], in.radius[i]);
    const uint64_t mask = __ballot(keep);
    if (lane == 0) wave_base[wid] = (uint32_t)__popcll(mask);
    __syncthreads();
    uint32_t base = block_off[blockIdx.x];
    for (int w = 0; w < wid; ++w) base += wave_base[w];
    const uint32_t rank = base + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
    if (i >= n) return;
    if (keep) {
        out.px[rank] = in.px[i];
        out.py[rank] = in.py[i];
        out.vx[rank] = in.vx[i];
        out.vy[rank] = in.vy[i];
        out.pref_x[rank] = in.pref_x[i];
        out.pref_y[rank] = in.pref_y[i];
        out.radius[rank] = in.radius[i];
        out.max_speed[rank] = in.max_speed[i];
        out.cls[rank] = in.cls[i];
    }
    if (old_to_new) old_to_new[i] = keep ? (int32_t)rank : -1;
}

// (entering 1) per block: largest radius and speed cap of the agents and of
// the candidates, and the candidates' bounding box
__global__ __launch_bounds__(kBlock) void k_spawn_bounds(const float *__restrict__ r_a,
                                                          const float *__restrict__ s_a, int n,
                                                          orca_agents_in cand, int nc,
                                                          float4 *__restrict__ partial,
                                                          float4 *__restrict__ box)
{
    float4 m = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    float4 b = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
    const int stride = gridDim.x * kBlock;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
        m.x = fmaxf(m.x, r_a[i]);
        m.y = fmaxf(m.y, s_a[i]);
    }
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < nc; i += stride) {
        m.z = fmaxf(m.z, cand.radius[i]);
        m.w = fmaxf(m.w, cand.max_speed[i]);
        const float x = cand.px[i], y = cand.py[i];
        b = make_float4(fminf(b.x, x), fminf(b.y, y), fmaxf(b.z, x), fmaxf(b.w, y));
    }
    // the bounding-box reduction's (min, min, max, max) applied to (-x, -y, z, w)
    float4 q = block_bbox<kBlock>(make_float4(-m.x, -m.y, m.z, m.w));
    if (threadIdx.x == 0) partial[blockIdx.x] = make_float4(-q.x, -q.y, q.z, q.w);
    __syncthreads();  // the reduction's LDS is used again
    b = block_bbox<kBlock>(b);
    if (threadIdx.x == 0) box[blockIdx.x] = b;
}

// Cell of a place along one axis, -2 or n + 1 for places with no cell beside them
// (and for NaN).  Without a finite box (inv 0) every place is in cell 0.
__device__ __forceinline__ int cand_axis(float v, double v0, double inv, int n)
{
    if (inv == 0.0) return 0;
    return (int)fmin(fmax(floor(((double)v - v0) * inv), -2.0), (double)(n + 1));
}

// (entering 2) one workgroup: the widest clearance D_max, a grid over the
// candidates with cells at least that large (so whoever is too close to a
// candidate stands in the 3 x 3 cells around it), and each candidate's place in
// cell order.  The rounding of the cell coordinates is covered by the cells' margin
// of 1e-6.
__global__ __launch_bounds__(kScanThreads) void k_spawn_grid(
    orca_agents_in cand, int nc, float t_clear, const float4 *__restrict__ partial,
    const float4 *__restrict__ box, int np, CandGrid *__restrict__ grid,
    uint32_t *__restrict__ start, int32_t *__restrict__ place)
{
    __shared__ uint32_t count[kCandCells];
    __shared__ CandGrid gs;
    float4 m = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    float4 b = make_float4(INFINITY, INFINITY, -INFINITY, -INFINITY);
    for (int k = threadIdx.x; k < np; k += kScanThreads) {
        const float4 v = partial[k], w = box[k];
        m = make_float4(fmaxf(m.x, v.x), fmaxf(m.y, v.y), fmaxf(m.z, v.z), fmaxf(m.w, v.w));
        b = make_float4(fminf(b.x, w.x), fminf(b.y, w.y), fmaxf(b.z, w.z), fmaxf(b.w, w.w));
    }
    for (int k = threadIdx.x; k < kCandCells; k += kScanThreads) count[k] = 0u;
    const float4 q = block_bbox<kScanThreads>(make_float4(-m.x, -m.y, m.z, m.w));
    __syncthreads();
    b = block_bbox<kScanThreads>(b);
    if (threadIdx.x == 0) {
        // clearance of the largest radii and speed caps, of a candidate beside
        // an agent or another candidate
        const double r = fmax(-(double)q.x, (double)q.z), s = fmax(-(double)q.y, (double)q.w);
        const double d = ((double)q.z + r) + (double)t_clear * ((double)q.w + s);
        const bool finite = isfinite(b.x) && isfinite(b.y) && isfinite(b.z) && isfinite(b.w) &&
                            isfinite(d);
        const double w = finite ? (double)b.z - (double)b.x : 0.0;
        const double h = finite ? (double)b.w - (double)b.y : 0.0;
        // a positive size even when everything is a point at rest; larger where
        // the box would need more cells (or one cell, by its size, for all)
        double c = fmax(d * (1.0 + 1e-6), fmax(1e-3, fmax(w, h) * 1e-6));
        // the cell counts as they are used below: at the limit a quotient here
        // and a product there can round to either side of a whole number
        double inv = 1.0 / c, fx = floor(w * inv) + 1.0, fy = floor(h * inv) + 1.0;
        while (fx * fy > (double)kCandCells) {
            c *= 1.125;
            inv = 1.0 / c;
            fx = floor(w * inv) + 1.0;
            fy = floor(h * inv) + 1.0;
        }
        gs.x0 = finite ? (double)b.x : 0.0;
        gs.y0 = finite ? (double)b.y : 0.0;
        gs.inv = finite ? inv : 0.0;
        gs.nx = (int)fx;
        gs.ny = (int)fy;
        *grid = gs;
    }
    __syncthreads();
    const CandGrid g = gs;
    // a thread's candidates are loaded together (their latencies overlap); an
    // index past the last candidate repeats it and is not used
    constexpr int kMine = ORCA_SPAWN_MAX / kScanThreads;
    float px[kMine], py[kMine];
    uint32_t at[kMine];  // cell (13 bits and more) and rank inside it
#pragma unroll
    for (int k = 0; k < kMine; ++k) {
        const int c = min(k * kScanThreads + (int)threadIdx.x, nc - 1);
        px[k] = cand.px[c];
        py[k] = cand.py[c];
    }
#pragma unroll
    for (int k = 0; k < kMine; ++k) {
        const int cx = min(max(cand_axis(px[k], g.x0, g.inv, g.nx), 0), g.nx - 1);
        const int cy = min(max(cand_axis(py[k], g.y0, g.inv, g.ny), 0), g.ny - 1);
        at[k] = (uint32_t)(cx + g.nx * cy);
        if (k * kScanThreads + (int)threadIdx.x < nc) at[k] |= atomicAdd(&count[at[k]], 1u) << 14;
    }
    __syncthreads();
    // exclusive scan of the histogram, kCandCells / kScanThreads cells a thread
    constexpr int kPer = kCandCells / kScanThreads;
    uint32_t v[kPer], sum = 0, tot;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        v[k] = count[threadIdx.x * kPer + k];
        sum += v[k];
    }
    uint32_t run = block_excl_scan<kScanThreads>(sum, &tot);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        count[threadIdx.x * kPer + k] = run;
        start[threadIdx.x * kPer + k] = run;
        run += v[k];
    }
    if (threadIdx.x == 0) start[kCandCells] = (uint32_t)nc;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kMine; ++k) {
        const int c = k * kScanThreads + threadIdx.x;
        if (c < nc) place[c] = (int32_t)(count[at[k] & 16383u] + (at[k] >> 14));
    }
}
static_assert(kCandCells <= 1 << 14 && ORCA_SPAWN_MAX <= 1 << 18, "a cell and a rank share a word");

// (entering 3) the candidates in cell order
__global__ __launch_bounds__(kBlock) void k_spawn_sort(orca_agents_in cand, int nc,
                                                        const int32_t *__restrict__ place,
                                                        float4 *__restrict__ sorted,
                                                        int32_t *__restrict__ index,
                                                        uint8_t *__restrict__ blocked)
{
    const int c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= nc) return;
    const int to = place[c];
    sorted[to] = make_float4(cand.px[c], cand.py[c], cand.radius[c], cand.max_speed[c]);
    index[to] = c;
    blocked[to] = 0;
}

// Visits the candidates in the 3 x 3 cells around (x, y), a row of cells (one
// range of the cell order) at a time and four candidates together: visit(t, e)
// for positions t .. t + 3 below e.
constexpr int kAhead = 4;

template <class F>
__device__ __forceinline__ void near_candidates(const CandGrid &g, const uint32_t *__restrict__ start,
                                                float x, float y, F &&visit)
{
    const int cx = cand_axis(x, g.x0, g.inv, g.nx), cy = cand_axis(y, g.y0, g.inv, g.ny);
    const int xa = max(cx - 1, 0), xb = min(cx + 1, g.nx - 1);
    for (int yy = max(cy - 1, 0); yy <= min(cy + 1, g.ny - 1); ++yy) {
        const uint32_t e = start[yy * g.nx + xb + 1];
        for (uint32_t t = start[yy * g.nx + xa]; t < e; t += kAhead) visit(t, e);
    }
}

// (entering 4) every agent blocks the candidates it is too close to.  One pass
// over the positions: only agents beside a candidate read more.  (A grid over
// the agents and a look from each candidate: 1M agents and 16,384 candidates
// 125 us, most of it the counting atomics of cells as wide as the clearance.)
//
// A wavefront looks at `per` agents.  Those beside candidates then go through
// their candidates lane by lane, four at a time, or the wavefront takes one agent
// after the other, 64 candidates at a time: whichever is fewer passes.  Callers
// whose order follows the places have whole wavefronts of agents beside few
// candidates each (1M agents, 16,384 candidates in rows: 5.6 us by lanes); with a
// wide clearance, or an order without places, few lanes would walk long ranges
// alone (1M agents, 16,384 candidates, 62 m: 8200 us by lanes alone, 320 now; 262,144
// and 2,000: 280 and 13 us).
__global__ __launch_bounds__(kBlock) void k_spawn_block(const float *__restrict__ px,
                                                         const float *__restrict__ py,
                                                         const float *__restrict__ radius,
                                                         const float *__restrict__ max_speed, int n,
                                                         int per, float t_clear,
                                                         const CandGrid *__restrict__ grid,
                                                         const uint32_t *__restrict__ start,
                                                         const float4 *__restrict__ sorted,
                                                         uint8_t *__restrict__ blocked)
{
    const int lane = threadIdx.x % kWave;
    const int wave = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    const int64_t i = (int64_t)wave * per + lane;
    const bool have = lane < per && i < n;
    const CandGrid g = *grid;
    const double t = (double)t_clear;
    const float x = have ? px[i] : 0.0f, y = have ? py[i] : 0.0f;
    const int cx = cand_axis(x, g.x0, g.inv, g.nx), cy = cand_axis(y, g.y0, g.inv, g.ny);
    const int xa = max(cx - 1, 0), xb = min(cx + 1, g.nx - 1);
    // the agent's candidates: one range per row of cells
    uint32_t ra[3], rb[3], by_lane = 0, by_wave = 0;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int yy = cy - 1 + q;
        const bool row = have && yy >= 0 && yy < g.ny;
        ra[q] = row ? start[yy * g.nx + xa] : 0u;
        rb[q] = row ? start[yy * g.nx + xb + 1] : 0u;
        by_lane += (rb[q] - ra[q] + kAhead - 1) / kAhead;
        by_wave += (rb[q] - ra[q] + kWave - 1) / kWave;
    }
    uint64_t busy = __ballot(by_lane != 0u);
    if (!busy) return;
    const float r = by_lane ? radius[i] : 0.0f, v = by_lane ? max_speed[i] : 0.0f;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        by_lane = max(by_lane, (uint32_t)__shfl_xor((int)by_lane, o, kWave));
        by_wave += (uint32_t)__shfl_xor((int)by_wave, o, kWave);
    }
    if (by_lane <= by_wave) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            for (uint32_t k = ra[q]; k < rb[q]; k += kAhead) {
                float4 c[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) c[u] = sorted[min(k + u, rb[q] - 1u)];
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
                    if (k + u < rb[q] && too_close(c[u].x, c[u].y, c[u].z, c[u].w, x, y, r, v, t))
                        blocked[k + u] = 1;  // every writer writes the same
            }
        }
        return;
    }
    for (; busy; busy &= busy - 1) {
        const int who = __ffsll((long long)busy) - 1;
        const float wx = __shfl(x, who, kWave), wy = __shfl(y, who, kWave);
        const float wr = __shfl(r, who, kWave), wv = __shfl(v, who, kWave);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const uint32_t e = (uint32_t)__shfl((int)rb[q], who, kWave);
            for (uint32_t k = (uint32_t)__shfl((int)ra[q], who, kWave) + lane; k < e; k += kWave) {
                const float4 c = sorted[k];
                if (too_close(c.x, c.y, c.z, c.w, wx, wy, wr, wv, t)) blocked[k] = 1;
            }
        }
    }
}

// Agents per wavefront of (4): 64 where that fills the chip, fewer (4 at least)
// for smaller crowds, whose wavefronts then have shorter walks (5,000 agents and
// 500 candidates 8 m wide: 60 us at 64, 6 at 4).
int spawn_block_agents(int n)
{
    int per = kWave;
    while (per > 4 && n / per < 4096) per /= 2;
    return per;
}

// (entering 5) each candidate's earlier conflicting candidates.  A candidate
// blocked by the agents is rejected whatever else happens, so lists are built
// for the unblocked ones and hold unblocked candidates only.  The decision
// rounds read a list as a set, and one that overflows sends its candidate to
// the exhaustive test, so the order of the entries does not matter.
__global__ __launch_bounds__(kBlock) void k_spawn_pairs(int nc, float t_clear,
                                                         const CandGrid *__restrict__ grid,
                                                         const uint32_t *__restrict__ start,
                                                         const float4 *__restrict__ sorted,
                                                         const int32_t *__restrict__ index,
                                                         const uint8_t *__restrict__ blocked,
                                                         int32_t *__restrict__ decision,
                                                         int32_t *__restrict__ conf_count,
                                                         int32_t *__restrict__ conf)
{
    const int s = blockIdx.x * kBlock + threadIdx.x;
    if (s >= nc) return;
    const int c = index[s];
    const bool free = !blocked[s];
    int found = 0;
    if (free) {
        const CandGrid g = *grid;
        const float4 me = sorted[s];
        near_candidates(g, start, me.x, me.y, [&](uint32_t t, uint32_t e) {
            float4 o[kAhead];
            int other[kAhead];
            bool out[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const uint32_t p = min(t + u, e - 1u);
                o[u] = sorted[p];
                other[u] = index[p];
                out[u] = blocked[p] != 0;
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (t + u >= e || other[u] >= c || out[u] ||
                    !too_close(me.x, me.y, me.z, me.w, o[u].x, o[u].y, o[u].z, o[u].w,
                               (double)t_clear))
                    continue;
                if (found < kConfCap) conf[(int64_t)c * kConfCap + found] = other[u];
                ++found;
            }
        });
    }
    conf_count[c] = found;
    decision[c] = !free ? kRejected : (found ? kUndecided : kAccepted);
}

// The decision of an undecided candidate from those of its conflicts, kUndecided
// while an earlier one that is open could still enter.
template <class Get>
__device__ __forceinline__ int decide(int cnt, const int32_t *__restrict__ list, Get &&get)
{
    bool any_open = false;
    for (int q = 0; q < cnt; ++q) {
        const int d = get(list[q]);
        if (d == kAccepted) return kRejected;
        any_open = any_open || d == kUndecided;
    }
    return any_open ? kUndecided : kAccepted;
}

// (entering 6) a few rounds of first-come decisions by all candidates at once.  A
// decision never changes once taken, so it does not matter which of the others'
// a thread sees already; what stays open is left to (7), one workgroup, whose
// rounds over all 16,384 candidates took 80 us.
constexpr int kOpenRounds = 4;

__global__ __launch_bounds__(kBlock) void k_spawn_decide(int nc, int32_t *__restrict__ decision,
                                                          const int32_t *__restrict__ conf_count,
                                                          const int32_t *__restrict__ conf)
{
    const int c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= nc || decision[c] != kUndecided) return;
    const int cnt = conf_count[c];
    if (cnt > kConfCap) return;
    for (int round = 0; round < kOpenRounds; ++round) {
        const int d = decide(cnt, conf + (int64_t)c * kConfCap, [&](int e) {
            return __hip_atomic_load(&decision[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        });
        if (d != kUndecided) {
            __hip_atomic_store(&decision[c], d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
    }
}

// (entering 7) one workgroup: the decisions still open, in rounds, and the places
// of the accepted candidates.
__global__ __launch_bounds__(kScanThreads) void k_spawn_resolve(
    orca_agents_in cand, int nc, float t_clear, int32_t *__restrict__ decision,
    const int32_t *__restrict__ conf_count, const int32_t *__restrict__ conf, int n,
    int32_t *__restrict__ n_total)
{
    __shared__ uint8_t st[ORCA_SPAWN_MAX];
    __shared__ uint16_t todo[ORCA_SPAWN_MAX];
    __shared__ uint32_t n_todo;
    static_assert(ORCA_SPAWN_MAX <= 65536, "candidates fit 16 bits");
    const int tid = threadIdx.x;
    const double t = (double)t_clear;
    if (tid == 0) n_todo = 0u;
    __syncthreads();
#pragma unroll 4
    for (int c = tid; c < nc; c += kScanThreads) {
        const int d = decision[c];
        st[c] = (uint8_t)d;
        if (d == kUndecided) todo[atomicAdd(&n_todo, 1u)] = (uint16_t)c;
    }
    __syncthreads();
    // every round decides at least the first undecided candidate, so at most
    // nc rounds
    const uint32_t open_at_first = n_todo;
    for (int round = 0; round <= nc; ++round) {
        int open = 0;
        for (uint32_t w = tid; w < open_at_first; w += kScanThreads) {
            const int c = todo[w];
            if (st[c] != kUndecided) continue;
            const int cnt = conf_count[c];
            int d;
            if (cnt <= kConfCap) {
                d = decide(cnt, conf + (int64_t)c * kConfCap, [&](int e) { return (int)st[e]; });
            } else {
                // more conflicts than listed: test every earlier candidate
                const float cx = cand.px[c], cy = cand.py[c], cr = cand.radius[c],
                            cs = cand.max_speed[c];
                bool any_acc = false, any_open = false;
                for (int e = 0; e < c; ++e) {
                    const int s = st[e];
                    if (s == kRejected) continue;
                    if (too_close(cx, cy, cr, cs, cand.px[e], cand.py[e], cand.radius[e],
                                  cand.max_speed[e], t)) {
                        any_acc = any_acc || s == kAccepted;
                        any_open = any_open || s == kUndecided;
                    }
                }
                d = any_acc ? kRejected : (any_open ? kUndecided : kAccepted);
            }
            if (d != kUndecided)
                st[c] = (uint8_t)d;
            else
                open = 1;
        }
        if (!__syncthreads_or(open)) break;
    }
    // places of the accepted candidates (exclusive scan over thread chunks)
    const int per = (nc + kScanThreads - 1) / kScanThreads;
    const int a = tid * per, b = min(a + per, nc);
    uint32_t s = 0, tot;
    for (int c = a; c < b; ++c) s += st[c] == kAccepted ? 1u : 0u;
    uint32_t rank = (uint32_t)n + block_excl_scan<kScanThreads>(s, &tot);
    for (int c = a; c < b; ++c) decision[c] = st[c] == kAccepted ? (int32_t)rank++ : -1;
    if (tid == 0) *n_total = (int32_t)((uint32_t)n + tot);
}

// (entering 8) the accepted candidates appended in order
__global__ __launch_bounds__(kBlock) void k_spawn_append(orca_agents_in cand, int nc,
                                                          const int32_t *__restrict__ place,
                                                          orca_agents_buf state,
                                                          uint8_t *__restrict__ accepted)
{
    const int c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= nc) return;
    const int to = place[c];
    if (accepted) accepted[c] = to >= 0 ? 1 : 0;
    if (to < 0) return;
    state.px[to] = cand.px[c];
    state.py[to] = cand.py[c];
    state.vx[to] = cand.vx[c];
    state.vy[to] = cand.vy[c];
    state.pref_x[to] = cand.pref_x[c];
    state.pref_y[to] = cand.pref_y[c];
    state.radius[to] = cand.radius[c];
    state.max_speed[to] = cand.max_speed[c];
    state.cls[to] = cand.cls[c];
}

// Overlap statistics, per block: pairs counted from both ends, agents in
// an overlap, and the smallest clearance over pairs closer than the grid's
// neighbour distance.  One lane per agent in cell order.
struct OverlapPart {
    double gap;
    uint32_t pairs2;  // overlapping pairs, each counted by both agents
    uint32_t agents;
};

__global__ __launch_bounds__(kBlock) void k_overlap(const GridMeta *__restrict__ meta,
                                                     const uint32_t *__restrict__ start,
                                                     const float2 *__restrict__ s0,
                                                     const float4 *__restrict__ s1, int n,
                                                     OverlapPart *__restrict__ part)
{
    const int s = blockIdx.x * kBlock + threadIdx.x;
    uint32_t cnt = 0;
    double gap = INFINITY;
    if (s < n) {
        const GridMeta g = *meta;
        const float2 me = s0[s];
        const double r = (double)s1[s].w;
        // the radii of a group's agents in range are asked for together
        dev::scan_disc_groups(
            g, start, s0, (double)me.x, (double)me.y, g.rn2,
            [&](const float2 (&a)[dev::kScanUnroll], uint32_t t0, uint32_t e) {
                double d2[dev::kScanUnroll];
                float other[dev::kScanUnroll];
                bool in[dev::kScanUnroll];
#pragma unroll
                for (int q = 0; q < dev::kScanUnroll; ++q) {
                    d2[q] = dev::nb_key(me.x, me.y, a[q].x, a[q].y);
                    in[q] = t0 + q < e && d2[q] < g.rn2 && t0 + q != (uint32_t)s;
                    other[q] = 0.0f;
                    if (in[q]) other[q] = s1[t0 + q].w;
                }
#pragma unroll
                for (int q = 0; q < dev::kScanUnroll; ++q) {
                    if (in[q]) {
                        const double rr = r + (double)other[q];
                        cnt += d2[q] < rr * rr ? 1u : 0u;
                        gap = fmin(gap, sqrt(d2[q]) - rr);
                    }
                }
            });
    }
    __shared__ double sg[kBlock / kWave];
    __shared__ uint32_t sp[kBlock / kWave], sa[kBlock / kWave];
    double wg = gap;
    uint32_t wp = cnt, wa = cnt > 0 ? 1u : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        wg = fmin(wg, __shfl_xor(wg, o, kWave));
        wp += __shfl_xor(wp, o, kWave);
        wa += __shfl_xor(wa, o, kWave);
    }
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    if (lane == 0) {
        sg[wid] = wg;
        sp[wid] = wp;
        sa[wid] = wa;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        OverlapPart r{INFINITY, 0u, 0u};
        for (int w = 0; w < kBlock / kWave; ++w) {
            r.gap = fmin(r.gap, sg[w]);
            r.pairs2 += sp[w];
            r.agents += sa[w];
        }
        part[blockIdx.x] = r;
    }
}

__global__ __launch_bounds__(kBlock) void k_overlap_final(const OverlapPart *__restrict__ part,
                                                           int np, double *__restrict__ out)
{
    __shared__ double sg[kBlock];
    __shared__ unsigned long long sp[kBlock], sa[kBlock];
    double g = INFINITY;
    unsigned long long p = 0, a = 0;
    for (int k = threadIdx.x; k < np; k += kBlock) {
        g = fmin(g, part[k].gap);
        p += part[k].pairs2;
        a += part[k].agents;
    }
    sg[threadIdx.x] = g;
    sp[threadIdx.x] = p;
    sa[threadIdx.x] = a;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) {
            sg[threadIdx.x] = fmin(sg[threadIdx.x], sg[threadIdx.x + o]);
            sp[threadIdx.x] += sp[threadIdx.x + o];
            sa[threadIdx.x] += sa[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = (double)(sp[0] / 2);
        out[1] = (double)sa[0];
        out[2] = sg[0];
    }
}

}  // namespace

size_t lifecycle_bytes(int64_t n, int64_t n_cand)
{
    size_t bytes;
    bind_life(n, n_cand, nullptr, &bytes);
    return bytes;
}

hipError_t launch_remove_arrived(const orca_agents_in &in, const orca_agents_buf &out, int n,
                                 int32_t *n_alive, int32_t *old_to_new, void *extra,
                                 hipStream_t stream)
{
    const LifeBufs b = bind_life(n, 0, extra);
    const int nb = (n + kBlock - 1) / kBlock;
    if (nb > 0)
        hipLaunchKernelGGL(k_arrive_count, dim3(nb), dim3(kBlock), 0, stream, in, n,
                           b.block_count);
    hipLaunchKernelGGL(k_arrive_scan, dim3(1), dim3(kScanThreads), 0, stream, b.block_count, nb,
                       n_alive);
    if (nb > 0)
        hipLaunchKernelGGL(k_arrive_move, dim3(nb), dim3(kBlock), 0, stream, in, out, n,
                           b.block_count, old_to_new);
    return hipGetLastError();
}

hipError_t launch_spawn(const orca_agents_buf &state, int n, const orca_agents_in &cand,
                        int n_cand, float t_clear, int32_t *n_total, uint8_t *accepted, void *extra,
                        hipStream_t stream)
{
    const LifeBufs b = bind_life(n, n_cand, extra);
    const int m = n > n_cand ? n : n_cand;
    int nbb = (m + kBlock - 1) / kBlock;
    nbb = nbb < 1 ? 1 : (nbb > kBoundBlocksMax ? kBoundBlocksMax : nbb);
    const int ncb = (n_cand + kBlock - 1) / kBlock;
    if (ncb > 0) {
        hipLaunchKernelGGL(k_spawn_bounds, dim3(nbb), dim3(kBlock), 0, stream, state.radius,
                           state.max_speed, n, cand, n_cand, b.partial, b.box);
        hipLaunchKernelGGL(k_spawn_grid, dim3(1), dim3(kScanThreads), 0, stream, cand, n_cand,
                           t_clear, b.partial, b.box, nbb, b.grid, b.start, b.decision);
        hipLaunchKernelGGL(k_spawn_sort, dim3(ncb), dim3(kBlock), 0, stream, cand, n_cand, b.decision,
                           b.cand, b.index, b.blocked);
        if (n > 0) {
            const int per = spawn_block_agents(n), block = per * (kBlock / kWave);
            hipLaunchKernelGGL(k_spawn_block, dim3((n + block - 1) / block), dim3(kBlock), 0, stream,
                               (const float *)state.px, (const float *)state.py,
                               (const float *)state.radius, (const float *)state.max_speed, n, per,
                               t_clear, b.grid, b.start, b.cand, b.blocked);
        }
        hipLaunchKernelGGL(k_spawn_pairs, dim3(ncb), dim3(kBlock), 0, stream, n_cand, t_clear, b.grid,
                           b.start, b.cand, b.index, b.blocked, b.decision, b.conf_count, b.conf);
        hipLaunchKernelGGL(k_spawn_decide, dim3(ncb), dim3(kBlock), 0, stream, n_cand, b.decision,
                           b.conf_count, b.conf);
    }
    hipLaunchKernelGGL(k_spawn_resolve, dim3(1), dim3(kScanThreads), 0, stream, cand, n_cand,
                       t_clear, b.decision, b.conf_count, b.conf, n, n_total);
    if (ncb > 0)
        hipLaunchKernelGGL(k_spawn_append, dim3(ncb), dim3(kBlock), 0, stream, cand, n_cand,
                           b.decision, state, accepted);
    return hipGetLastError();
}

}  // namespace orca

namespace orca {

size_t overlap_extra_bytes(int64_t n)
{
    return a256(sizeof(OverlapPart) * (size_t)((n + kBlock - 1) / kBlock + 1));
}

hipError_t launch_overlap_stats(const orca_agents_in &in, int n, float reach, double *out,
                                const Layout &L, const Work &w, void *extra, hipStream_t stream)
{
    OverlapPart *part = (OverlapPart *)extra;
    const int nb = (n + kBlock - 1) / kBlock;
    if (n > 0) {
        const hipError_t e = launch_grid_build_rn(in, n, reach, 0.0f, L, w, stream, nullptr, 0, true);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_overlap, dim3(nb), dim3(kBlock), 0, stream, w.meta, w.start, w.s0,
                           w.s1, n, part);
    }
    hipLaunchKernelGGL(k_overlap_final, dim3(1), dim3(kBlock), 0, stream, part, nb, out);
    return hipGetLastError();
}

}  // namespace orca
