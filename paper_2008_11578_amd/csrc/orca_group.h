// The ORCA step of one agent by a group of G lanes, for crowds too small to
// fill the chip with a lane per agent (gfx950).
//
// A lane per agent gives a crowd of 66,560 one wavefront per SIMD and a crowd
// of 256 four wavefronts in all: the step then takes as long as one wavefront's
// chain of dependent loads, sorts and line walks, 30-100 us, however idle the
// chip is.  Here a wavefront takes 64 / G agents.  Each phase is split over the
// group's lanes:
//
//   scan    a row's cells by one lane each, then G candidates at a time
//   order   each lane ranks its share of the entries by counting the smaller
//           ones (exact keys and caller indices: no network, no tie pass)
//   lines   one half-plane per lane and pass
//   LP      group_lp2 and group_lp3: lines over the lanes
//
// All values are formed by the expressions of the lane-per-agent step, and the
// neighbour order is defined by exact keys, so the results are its bit for bit.
#pragma once

#include "orca_device.h"

#pragma clang fp contract(on)

namespace orca {
namespace dev {

// Entries of one agent's neighbour buffer; a circle that holds more is cut.
constexpr int kGroupCap = 64;
constexpr int kGroupChunks = 32;  // scan chunks listed at a time
constexpr int kGroupBins = 64;    // equal-area bins that cut a full circle

// LDS of one wavefront of 64 / G agents, at most K lines each.
template <int K, int G>
struct GroupLds {
    static constexpr int A = kWave / G;
    struct Entry {
        double key;
        uint32_t pos, pad;
    };
    Entry ent[A][kGroupCap + 1];  // + 1: the agents' entries start in other banks
    uint2 chunk[A][kGroupChunks];
    uint32_t bins[A][kGroupBins];
    uint32_t nbr[A][K];
    float4 lines[K][A];
};

// Bits of the group's lanes (agent a of the wavefront) in a wavefront mask.
template <int G>
__device__ __forceinline__ uint32_t group_bits(uint64_t mask, int a)
{
    return (uint32_t)(mask >> (a * G)) & ((1u << G) - 1u);
}

// Visits the candidates of the disc by the group: visit(t, xy, valid) for G
// consecutive positions at a time, the lanes together.  WHOLE: every agent of
// the scene (positions [first, g.seg_end)) instead, without a grid.
template <int K, int G, bool WHOLE, class F>
__device__ __forceinline__ void group_scan(const GridMeta &g, const uint32_t *__restrict__ start,
                                           const float2 *__restrict__ s0, double xd, double yd,
                                           double r2, GroupLds<K, G> &lds, int a, int c, F &&visit)
{
    constexpr int kAhead = 4;  // loads in flight
    if (WHOLE) {
        const uint32_t e = g.seg_end;
        for (uint32_t t0 = (uint32_t)g.agent_base; t0 < e; t0 += kAhead * G) {
            float2 p[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) p[u] = s0[min(t0 + u * G + c, e - 1u)];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const uint32_t t = t0 + u * G + c;
                visit(t, p[u], t < e);
            }
        }
        return;
    }
    const CellDisc disc = cell_disc(g, xd, yd, r2);
    int ya, yb;
    row_span(g, disc, ya, yb);
    for (int y0 = ya; y0 <= yb; y0 += G) {
        // each lane finds one row's range and its number of chunks
        uint32_t ra = 0, rb = 0;
        if (y0 + c <= yb && !row_range(g, start, disc, y0 + c, ra, rb)) rb = ra;
        const int mine = (int)((rb - ra + (G - 1)) / G);
        int upto = mine;
#pragma unroll
        for (int o = 1; o < G; o <<= 1) {
            const int v = __shfl_up(upto, o, G);
            upto += c >= o ? v : 0;
        }
        const int all = __shfl(upto, G - 1, G);
        for (int w = 0; w < all; w += kGroupChunks) {
            lane_order<kWave>();  // the last window's list is read
            for (int q = max(w - (upto - mine), 0); q < mine; ++q) {
                const int at = upto - mine + q - w;
                if (at >= kGroupChunks) break;
                lds.chunk[a][at] = make_uint2(ra + (uint32_t)(q * G), rb);
            }
            lane_order<kWave>();
            const int m = min(all - w, kGroupChunks);
            for (int d = 0; d < m; d += kAhead) {
                uint2 ch[kAhead];
                float2 p[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    ch[u] = lds.chunk[a][min(d + u, m - 1)];
                    p[u] = s0[ch[u].x + (uint32_t)c];  // at most G - 1 past the row: s0's padding
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const uint32_t t = ch[u].x + (uint32_t)c;
                    visit(t, p[u], d + u < m && t < ch[u].y);
                }
            }
        }
    }
}
static_assert(16 <= kScanPad, "a chunk may read a group's lanes past a row");

// The candidates with key < r2 (the own agent, position spos, left out) into
// the agent's entries; returns how many there are, also beyond the capacity.
template <int K, int G, bool WHOLE>
__device__ __forceinline__ int group_collect(const GridMeta &g, const uint32_t *__restrict__ start,
                                             const float2 *__restrict__ s0, float xi, float yi,
                                             uint32_t spos, double r2, GroupLds<K, G> &lds, int a,
                                             int c)
{
    int total = 0;
    lane_order<kWave>();  // earlier entries are read
    group_scan<K, G, WHOLE>(
        g, start, s0, (double)xi, (double)yi, r2, lds, a, c, [&](uint32_t t, float2 p, bool valid) {
            const double key = nb_key(xi, yi, p.x, p.y);
            const bool in = valid && key < r2 && t != spos;
            const uint32_t bits = group_bits<G>(__ballot(in), a);
            const int at = total + __popc(bits & ((1u << c) - 1u));
            if (in && at < kGroupCap) lds.ent[a][at] = {key, t, 0u};
            total += __popc(bits);
        });
    lane_order<kWave>();
    return total;
}

// The (at most k) nearest agents, ascending, as positions in lds.nbr[a]; returns
// their number.  keep: the kept scan radius (0: none) and, on return, the next.
template <int K, int G, bool WHOLE>
__device__ __forceinline__ int group_knn(const GridMeta &g, const uint32_t *__restrict__ start,
                                         const float2 *__restrict__ s0,
                                         const float4 *__restrict__ s1, float xi, float yi,
                                         uint32_t spos, int k, GroupLds<K, G> &lds, int a, int c,
                                         float &keep)
{
    double r2 = keep > 0.0f ? fmin((double)keep * (double)keep, g.rn2) : g.rn2;
    int total = group_collect<K, G, WHOLE>(g, start, s0, xi, yi, spos, r2, lds, a, c);
    if (total < k && r2 < g.rn2) {
        r2 = g.rn2;  // the kept circle holds too few
        total = group_collect<K, G, WHOLE>(g, start, s0, xi, yi, spos, r2, lds, a, c);
    }
    if (total > kGroupCap) {
        // cut the circle at the first equal-area bin that completes k
        const double scale = (double)kGroupBins / r2;
        for (int b = c; b < kGroupBins; b += G) lds.bins[a][b] = 0u;
        lane_order<kWave>();
        group_scan<K, G, WHOLE>(g, start, s0, (double)xi, (double)yi, r2, lds, a, c,
                                [&](uint32_t t, float2 p, bool valid) {
                                    const double key = nb_key(xi, yi, p.x, p.y);
                                    if (valid && key < r2 && t != spos)
                                        atomicAdd(&lds.bins[a][min((int)(key * scale), kGroupBins - 1)],
                                                  1u);
                                });
        lane_order<kWave>();
        int cut = 0;
        for (uint32_t cum = 0; cut < kGroupBins; ++cut) {
            cum += lds.bins[a][cut];
            if (cum >= (uint32_t)k) break;
        }
        r2 = fmin((double)(cut + 1) * (r2 / (double)kGroupBins) * (1.0 + 1e-9), r2);
        total = group_collect<K, G, WHOLE>(g, start, s0, xi, yi, spos, r2, lds, a, c);
    }
    if (total <= kGroupCap && (total >= k || !(r2 < g.rn2))) {
        // a circle of few entries is widened by their share
        constexpr int kMore = kKeptMore;
        float next = (float)sqrt(r2) * sqrtf((float)(k + kMore + 1) / (float)(total + 1));
        bool at_next = false;
        for (int e = c; e < total; e += G) {
            const double ke = lds.ent[a][e].key;
            int rank = 0, same = 0;
#pragma unroll 4
            for (int f = 0; f < total; ++f) {
                const double kf = lds.ent[a][f].key;
                rank += kf < ke ? 1 : 0;
                same += kf == ke ? 1 : 0;
            }
            const uint32_t pos = lds.ent[a][e].pos;
            if (same > 1) {
                // equal keys: the smaller caller index first
                const int i = tag_index(s1[pos].z);
                for (int f = 0; f < total; ++f)
                    if (lds.ent[a][f].key == ke && tag_index(s1[lds.ent[a][f].pos].z) < i) ++rank;
            }
            if (rank < k) lds.nbr[a][rank] = pos;
            if (rank == k - 1 + kMore) {
                next = sqrtf((float)ke);
                at_next = true;
            }
        }
        // the lane that holds that entry tells the group
        const uint32_t holds = group_bits<G>(__ballot(at_next), a);
        next = __shfl(next, holds ? __ffs((int)holds) - 1 : 0, G);
        keep = fminf(next, g.rn);
        lane_order<kWave>();
        return min(total, k);
    }
    // crowded beyond the bins: repeated minimum, strictly above the last pick
    double lk = -1.0;
    int lj = -1, m = 0;
    for (; m < k; ++m) {
        double bk = INFINITY;
        int bj = INT_MAX;
        uint32_t bt = 0;
        group_scan<K, G, WHOLE>(
            g, start, s0, (double)xi, (double)yi, g.rn2, lds, a, c,
            [&](uint32_t t, float2 p, bool valid) {
                const double key = nb_key(xi, yi, p.x, p.y);
                if (!(valid && key < g.rn2 && t != spos && key >= lk && key <= bk)) return;
                const int j = tag_index(s1[t].z);
                if ((key > lk || j > lj) && (key < bk || j < bj)) {
                    bk = key;
                    bj = j;
                    bt = t;
                }
            });
#pragma unroll
        for (int o = 1; o < G; o <<= 1) {
            const double ok = __shfl_xor(bk, o, G);
            const int oj = __shfl_xor(bj, o, G);
            const uint32_t ot = __shfl_xor(bt, o, G);
            if (ok < bk || (ok == bk && oj < bj)) {
                bk = ok;
                bj = oj;
                bt = ot;
            }
        }
        if (bj == INT_MAX) break;
        if (c == 0) lds.nbr[a][m] = bt;
        lk = bk;
        lj = bj;
    }
    lane_order<kWave>();
    // the next circle, from the last pick's distance
    keep = m == k ? fminf((float)sqrt(lk) * sqrtf((float)(k + kKeptMore + 1) / (float)(k + 1)), g.rn)
                  : g.rn;
    return m;
}

// The state of an agent after its step, the same in every lane of its group.
template <int K, int G, bool ACC>
struct GroupAgent {
    int i, m, nh, nacc;  // caller index, neighbours, hard lines, octagon lines
    float2 p;
    float4 s;  // cell-order record (velocity, tag, radius)
    float vmax, prx, pry, cx, cy;
    float vx, vy;
    uint8_t status;
    LdsLines<kWave / G, ACC> lines;
};

// One step of the agent at position s up to its new velocity (step_agent by a
// group).  REC records the active set.
template <bool REC, int K, int G, bool ACC, bool WHOLE>
__device__ __forceinline__ GroupAgent<K, G, ACC>
group_step(int s, const GridMeta &g, const SceneP &p, const orca_agents_in &in,
           const uint32_t *__restrict__ start, const float2 *__restrict__ s0,
           const float4 *__restrict__ s1, GroupLds<K, G> &lds, int a, int c, bool live,
           float *__restrict__ guess, ActiveSet *rec)
{
    constexpr int A = kWave / G;
    constexpr int NL = (K + (ACC ? kAccLines + kTurnLines : 0) + G - 1) / G;
    GroupAgent<K, G, ACC> r;
    r.p = s0[s];
    r.s = s1[s];
    r.i = tag_index(r.s.z);
    const int ci = tag_class(r.s.z);
    r.vmax = in.max_speed[r.i];
    r.prx = in.pref_x[r.i];
    r.pry = in.pref_y[r.i];
    float keep = guess[r.i];
    r.m = group_knn<K, G, WHOLE>(g, start, s0, s1, r.p.x, r.p.y, (uint32_t)s, min(p.k, K), lds, a, c,
                                 keep);
    if (live && c == 0) guess[r.i] = keep;

    const float acc = ACC ? (ci ? p.acc1 : p.acc0) : 0.0f;
    const float turn = ACC ? (ci ? p.turn1 : p.turn0) : 0.0f;
    r.nacc = (ACC && acc > 0.0f) ? kAccLines : 0;
    float rx = 0.0f, ry = 0.0f, lx = 0.0f, ly = 0.0f;
    r.nh = r.nacc + ((ACC && turn_wedge(r.s.x, r.s.y, turn, p.dt, rx, ry, lx, ly)) ? kTurnLines : 0);
    const float fa = ci ? p.f10 : p.f00;  // f[ci][0]
    const float fb = ci ? p.f11 : p.f01;  // f[ci][1]
#pragma unroll
    for (int q0 = 0; q0 < K; q0 += G) {
        const int q = q0 + c;
        if (q < r.m) {
            const uint32_t pos = lds.nbr[a][q];
            const float2 b0 = s0[pos];
            const float4 b1 = s1[pos];
            lds.lines[q][a] =
                halfplane(r.p.x, r.p.y, r.s.x, r.s.y, r.s.w, b0.x, b0.y, b1.x, b1.y, b1.w,
                          tag_class(b1.z) ? fb : fa, p.inv_tau, p.inv_dt, r.i < tag_index(b1.z));
        }
    }
    lane_order<kWave>();
    r.cx = r.cy = 0.0f;
    if (ACC && r.nh) accel_centre(r.s.x, r.s.y, r.vmax, r.cx, r.cy);
    desired_velocity(p, r.p.x, r.p.y, r.vmax, r.prx, r.pry);
    r.lines = LdsLines<A, ACC>{&lds.lines[0][0], a, r.nh, r.cx, r.cy,
                               ACC && r.nacc ? accel_half_width(acc, p.dt) : 0.0f,
                               r.nacc, rx, ry, lx, ly};
    const int mt = r.nh + r.m;
    float4 ln[NL];
    uint32_t valid = 0;
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const int j = c + G * q;
        if (G * q < mt) {  // the same in the whole group
            ln[q] = r.lines.line(min(j, mt - 1));
            valid |= (j < mt ? 1u : 0u) << q;
        }
    }
    int fail = group_lp2<REC, G>(ln, valid, c, mt, r.vmax, 0, r.prx, r.pry, 0.0f, 0.0f, p.eps, r.vx,
                                 r.vy, rec);
    r.status = 0;
    if (ACC && fail < r.nh) {
        // only rounding gets here: the centre, and LP3 from it (step_agent)
        r.vx = r.cx;
        r.vy = r.cy;
        fail = r.nh;
        r.status = 1;
        if (REC) rec->kind = kCentre;
    }
    if (fail < mt) {
        group_lp3<REC, A, ACC, G, NL>(r.lines, c, mt, fail, r.vmax, r.prx, r.pry, p.eps, r.vx, r.vy,
                                      rec);
        r.status = 1;
    }
    return r;
}

// The same with the results written by the group's first lane.
template <int K, int G, bool ACC, bool WHOLE, bool EXPORT>
__device__ __forceinline__ void group_step_write(bool live, int s, const GridMeta &g,
                                                 const SceneP &p, const orca_agents_in &in,
                                                 const orca_agents_out &out,
                                                 const uint32_t *__restrict__ start,
                                                 const float2 *__restrict__ s0,
                                                 const float4 *__restrict__ s1,
                                                 GroupLds<K, G> &lds, int a, int c,
                                                 float *__restrict__ guess, int32_t *nbr,
                                                 int32_t *cnt, int kout)
{
    const GroupAgent<K, G, ACC> r = group_step<false, K, G, ACC, WHOLE>(
        s, g, p, in, start, s0, s1, lds, a, c, live, guess, nullptr);
    if (!live) return;
    if (EXPORT) {
        if (nbr)
            for (int q = c; q < kout; q += G)
                nbr[(int64_t)r.i * kout + q] = q < r.m ? tag_index(s1[lds.nbr[a][q]].z) : -1;
        if (cnt && c == 0) cnt[r.i] = r.m;
    }
    if (c != 0) return;
    out.vx[r.i] = r.vx;
    out.vy[r.i] = r.vy;
    out.px[r.i] = r.p.x + r.vx * p.dt;
    out.py[r.i] = r.p.y + r.vy * p.dt;
    if (out.status) out.status[r.i] = r.status;
}

}  // namespace dev
}  // namespace orca
