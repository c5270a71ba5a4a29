// The step of a small crowd: a group of lanes per agent (orca_group.h), and for
// the smallest crowds no grid at all.
#include "orca_group.h"

namespace orca {
namespace {

constexpr int kBlock = 256;

struct GroupArgs {
    orca_agents_in in;
    orca_agents_out out;
    const GridMeta *meta;
    const uint32_t *start;
    const float2 *s0;
    const float4 *s1;
    float *guess;  // per-agent radius of the neighbour scan kept between steps
    int32_t *nbr;  // export only
    int32_t *cnt;
    int n, k;
    float rn;
};

// The cell-ordered copies in caller order, for a scan of the whole crowd.
__global__ __launch_bounds__(kBlock) void k_pack(orca_agents_in in, int n, float2 *__restrict__ s0,
                                                 float4 *__restrict__ s1,
                                                 uint32_t *__restrict__ clear, int64_t clear_len)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) write_record(in, i, (uint32_t)i, s0, s1);
    for (int64_t c = i; c < clear_len; c += (int64_t)gridDim.x * kBlock) clear[c] = 0u;
}

template <int K, int G, bool ACC, bool WHOLE, bool EXPORT>
__global__ __launch_bounds__(kWave) void k_step_group(GroupArgs a, dev::SceneP p)
{
    __shared__ dev::GroupLds<K, G> lds;
    constexpr int A = kWave / G;
    const int who = threadIdx.x / G;
    const int s = xcd_tile(blockIdx.x, gridDim.x) * A + who;
    const GridMeta g = WHOLE ? whole_crowd(a.n, a.rn) : *a.meta;
    dev::group_step_write<K, G, ACC, WHOLE, EXPORT>(s < a.n, min(s, a.n - 1), g, p, a.in, a.out,
                                                    a.start, a.s0, a.s1, lds, who, threadIdx.x % G,
                                                    a.guess, a.nbr, a.cnt, a.k);
}

// The lists alone.
template <int K, int G>
__global__ __launch_bounds__(kWave) void k_list_group(GroupArgs a)
{
    __shared__ dev::GroupLds<K, G> lds;
    constexpr int A = kWave / G;
    const int who = threadIdx.x / G, c = threadIdx.x % G;
    const int at = xcd_tile(blockIdx.x, gridDim.x) * A + who;
    const int s = min(at, a.n - 1);
    const GridMeta g = *a.meta;
    const float2 p = a.s0[s];
    const int i = tag_index(a.s1[s].z);
    float keep = a.guess[i];
    const int m = dev::group_knn<K, G, false>(g, a.start, a.s0, a.s1, p.x, p.y, (uint32_t)s, a.k,
                                              lds, who, c, keep);
    if (at >= a.n) return;
    if (c == 0) a.guess[i] = keep;
    if (a.nbr)
        for (int q = c; q < a.k; q += G)
            a.nbr[(int64_t)i * a.k + q] = q < m ? tag_index(a.s1[lds.nbr[who][q]].z) : -1;
    if (a.cnt && c == 0) a.cnt[i] = m;
}

// One step of every scene of a small batch (the scenes' grids are built).
template <int K, int G, bool ACC>
__global__ __launch_bounds__(kWave) void k_step_batched_group(BatchArgs a)
{
    __shared__ dev::GroupLds<K, G> lds;
    constexpr int A = kWave / G;
    const int who = threadIdx.x / G;
    const int s0 = xcd_tile(blockIdx.x, gridDim.x) * A;
    const int s = min(s0 + who, a.n - 1);
    const int sc = scene_from(a.off, a.S, scene_of(a.off, a.S, s0), s);
    const GridMeta g = a.meta[sc];
    const dev::SceneP p = dev::scene_params(a.prm[sc]);
    dev::group_step_write<K, G, ACC, false, false>(s0 + who < a.n, s, g, p, a.in, a.out, a.start,
                                                   a.s0, a.s1, lds, who, threadIdx.x % G, a.guess,
                                                   nullptr, nullptr, 0);
}

template <int K, int G, bool ACC, bool WHOLE>
void launch_group_v(const GroupArgs &a, const dev::SceneP &p, hipStream_t stream)
{
    const int nb = (a.n + kWave / G - 1) / (kWave / G);
    if (a.nbr || a.cnt)
        hipLaunchKernelGGL((k_step_group<K, G, ACC, WHOLE, true>), dim3(nb), dim3(kWave), 0, stream,
                           a, p);
    else
        hipLaunchKernelGGL((k_step_group<K, G, ACC, WHOLE, false>), dim3(nb), dim3(kWave), 0,
                           stream, a, p);
}

template <int K, int G, bool WHOLE>
void launch_group_k(const GroupArgs &a, const dev::SceneP &p, hipStream_t stream)
{
    if (p.acc0 > 0.0f || p.acc1 > 0.0f || p.turn0 > 0.0f || p.turn1 > 0.0f)
        launch_group_v<K, G, true, WHOLE>(a, p, stream);
    else
        launch_group_v<K, G, false, WHOLE>(a, p, stream);
}

}  // namespace

hipError_t launch_pack(const orca_agents_in &in, int n, const Work &w, hipStream_t stream,
                       uint32_t *clear, int64_t clear_len)
{
    hipLaunchKernelGGL(k_pack, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, stream, in, n, w.s0,
                       w.s1, clear, clear_len);
    return hipGetLastError();
}

hipError_t launch_step_group(const orca_agents_in &in, const orca_agents_out &out, int n,
                             const orca_params &prm, const Work &w, bool whole, int32_t *nbr,
                             int32_t *cnt, hipStream_t stream)
{
    const GroupArgs a{in, out, w.meta, w.start, w.s0, w.s1, w.guess, nbr, cnt, n, prm.max_neighbors,
                      prm.neighbor_dist};
    const dev::SceneP p = dev::scene_params(prm);
    if (prm.max_neighbors <= 16) {
        if (whole)
            launch_group_k<16, kGroup, true>(a, p, stream);
        else
            launch_group_k<16, kGroup, false>(a, p, stream);
    } else {
        if (whole)
            launch_group_k<32, kGroup, true>(a, p, stream);
        else
            launch_group_k<32, kGroup, false>(a, p, stream);
    }
    return hipGetLastError();
}

hipError_t launch_list_group(int n, const orca_params &prm, const Work &w, int32_t *nbr,
                             int32_t *cnt, hipStream_t stream)
{
    const GroupArgs a{{}, {}, w.meta, w.start, w.s0, w.s1, w.guess, nbr, cnt, n, prm.max_neighbors,
                      prm.neighbor_dist};
    const int nb = (n + kWave / kGroup - 1) / (kWave / kGroup);
    if (prm.max_neighbors <= 16)
        hipLaunchKernelGGL((k_list_group<16, kGroup>), dim3(nb), dim3(kWave), 0, stream, a);
    else
        hipLaunchKernelGGL((k_list_group<32, kGroup>), dim3(nb), dim3(kWave), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_batched_group(const BatchArgs &a, int k_max, bool acc, hipStream_t stream)
{
    const dim3 nb((a.n + kWave / kGroup - 1) / (kWave / kGroup));
    if (k_max <= 16) {
        if (acc)
            hipLaunchKernelGGL((k_step_batched_group<16, kGroup, true>), nb, dim3(kWave), 0, stream,
                               a);
        else
            hipLaunchKernelGGL((k_step_batched_group<16, kGroup, false>), nb, dim3(kWave), 0, stream,
                               a);
    } else {
        if (acc)
            hipLaunchKernelGGL((k_step_batched_group<32, kGroup, true>), nb, dim3(kWave), 0, stream,
                               a);
        else
            hipLaunchKernelGGL((k_step_batched_group<32, kGroup, false>), nb, dim3(kWave), 0, stream,
                               a);
    }
    return hipGetLastError();
}

}  // namespace orca
