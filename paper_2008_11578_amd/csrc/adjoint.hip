// Adjoint of one ORCA step (the differentiable form; not in the paper).
//
// Given the cotangents (gp1, gv1) of the step's outputs p' = p + v' dt and v',
// the kernels below produce the cotangents of the step-t positions and
// velocities, accumulate those of the pref input (desired velocity, or goal in
// goal mode) and of the look-ahead tau:
//
//   k_adjoint       one lane per agent: recompute the agent's step exactly as
//                   the forward kernel does (same neighbours, half-planes, LP),
//                   recording the LP's active set; then differentiate:
//                     LP   implicit differentiation of the active equalities
//                          (a line, two lines, a line on the speed circle, or
//                          the equal-penetration boundaries of LP3),
//                     ORCA each involved half-plane through its branch (cutoff
//                          arc, leg, overlap) to P = p_B - p_A, V = v_A - v_B
//                          and 1/tau,
//                     caps an involved acceleration line (q = c + h n_k)
//                          through its centre c to the agent's own velocity
//                          (c = v, or v scaled onto the speed circle),
//                   writing the agent's own cotangents and up to three
//                   contributions to neighbours into an edge list;
//                   the edge also goes to its target's list, by an atomic count;
//   k_edge_gather   each target sums its edges in source order (no
//                   floating-point atomics, so results are bit-reproducible);
//                   also the tau contributions of the block's agents, in double
//                   and in a fixed order;
//   k_tau_final     one block adds the block sums.
// Neighbour sets and branches are held fixed (they are piecewise constant).
#include "orca_group.h"

namespace orca {
namespace {

constexpr int kAdjBlock = 64;
constexpr int kBlock = 256;
constexpr int kEdges = 3;  // at most three lines define an LP result

struct AdjArgs {
    orca_agents_in in;
    int n;
    const GridMeta *meta;
    const uint32_t *start;
    const float2 *s0;
    const float4 *s1;
    float *guess;  // per-agent radius of the neighbour scan kept between calls
    dev::SceneP p;
    const float *gpx1, *gpy1, *gvx1, *gvy1;
    float *gpx0, *gpy0, *gvx0, *gvy0, *gprx, *gpry;
    AdjointBufs b;
};

// Cotangents of the (at most three) lines (q, n) that define the LP result:
// slot e holds line idx[e] (neighbour slot, -1 = unused).
struct LineBars {
    int idx[kEdges];
    float qx[kEdges], qy[kEdges], nx[kEdges], ny[kEdges];
};

__device__ __forceinline__ void add_line(LineBars &lb, int idx, float qx, float qy, float nx,
                                         float ny)
{
    // slot of line idx, or the first free one (static indices only, so the
    // arrays stay in registers)
    int slot = -1;
#pragma unroll
    for (int e = 0; e < kEdges; ++e)
        if (slot < 0 && lb.idx[e] == idx) slot = e;
#pragma unroll
    for (int e = 0; e < kEdges; ++e) {
        if (slot < 0 && lb.idx[e] < 0) {
            slot = e;
            lb.idx[e] = idx;
        }
    }
#pragma unroll
    for (int e = 0; e < kEdges; ++e) {
        if (e == slot) {
            lb.qx[e] += qx;
            lb.qy[e] += qy;
            lb.nx[e] += nx;
            lb.ny[e] += ny;
        }
    }
}

// VJP of ORCA_{A|B} (see dev::halfplane) given the cotangents of its point q
// and normal n.  Returns the cotangents of P = p_B - p_A, V = v_A - v_B, of
// the horizon's reciprocal (only when not overlapping), and q's direct
// dependence on v_A is left to the caller (q = v_A + f u).
__device__ __forceinline__ void halfplane_vjp(float pax, float pay, float vax, float vay, float ra,
                                              float pbx, float pby, float vbx, float vby, float rb,
                                              float f, float inv_tau, float inv_dt, bool a_first,
                                              float qbx, float qby, float nbx, float nby,
                                              float &Pbx, float &Pby, float &Vbx, float &Vby,
                                              float &itb, bool &uses_tau)
{
    const float Px = pbx - pax, Py = pby - pay;
    const float Vx = vax - vbx, Vy = vay - vby;
    const float R = ra + rb;
    const float dist2 = Px * Px + Py * Py;
    const float R2 = R * R;
    const double c2 = dev::clearance2(pax, pay, ra, pbx, pby, rb);
    const bool overlap = !(c2 > 0.0);
    const float it = overlap ? inv_dt : inv_tau;
    const float wx = Vx - Px * it, wy = Vy - Py * it;
    const float w2 = wx * wx + wy * wy;
    const float wp = wx * Px + wy * Py;
    const bool arc = overlap || (wp < 0.0f && wp * wp > R2 * w2);
    const float ubx = f * qbx, uby = f * qby;
    uses_tau = !overlap && arc;
    if (arc) {
        const bool wz = !(w2 > 0.0f);
        const float wl = sqrtf(w2);
        const float iwl = wz ? 0.0f : 1.0f / wl;
        const float nx = wz ? (a_first ? 1.0f : -1.0f) : wx * iwl;
        const float ny = wz ? 0.0f : wy * iwl;
        const float ul = R * it - wl;
        const float ulb = ubx * nx + uby * ny;
        const float tx = nbx + ul * ubx, ty = nby + ul * uby;
        const float nt = nx * tx + ny * ty;
        const float wbx = wz ? 0.0f : (tx - nx * nt) * iwl - ulb * nx;
        const float wby = wz ? 0.0f : (ty - ny * nt) * iwl - ulb * ny;
        itb = ulb * R - (wbx * Px + wby * Py);
        Vbx = wbx;
        Vby = wby;
        Pbx = -wbx * it;
        Pby = -wby * it;
        return;
    }
    // leg: e = (leg P + sigma R P_perp) / |P|^2, n = sigma (-e.y, e.x), u = (V.e) e - V
    const float leg = sqrtf(fmaxf((float)c2, 0.0f));
    const float id2 = 1.0f / dist2;
    const bool left = dev::det2(Px, Py, wx, wy) > 0.0f;
    const float sR = left ? R : -R;
    const float ex = (Px * leg - Py * sR) * id2;
    const float ey = (Px * sR + Py * leg) * id2;
    const float s = Vx * ex + Vy * ey;
    const float eu = ex * ubx + ey * uby;
    Vbx = ex * eu - ubx;
    Vby = ey * eu - uby;
    float ebx = s * ubx + eu * Vx;
    float eby = s * uby + eu * Vy;
    ebx += left ? nby : -nby;
    eby += left ? -nbx : nbx;
    const float abx = ebx * id2, aby = eby * id2;
    float Db = -(ebx * ex + eby * ey) * id2;
    Pbx = leg * abx + sR * aby;
    Pby = -sR * abx + leg * aby;
    const float legb = abx * Px + aby * Py;
    Db += leg > 0.0f ? legb / (2.0f * leg) : 0.0f;
    Pbx += 2.0f * Db * Px;
    Pby += 2.0f * Db * Py;
    itb = 0.0f;
}

// Solves mu_1 g1 + mu_2 g2 = w (2x2); zero when singular.
__device__ __forceinline__ void solve2(float g1x, float g1y, float g2x, float g2y, float wx,
                                       float wy, float &m1, float &m2)
{
    const float det = g1x * g2y - g1y * g2x;
    if (!(fabsf(det) > 1e-20f)) {
        m1 = 0.0f;
        m2 = 0.0f;
        return;
    }
    const float id = 1.0f / det;
    m1 = (wx * g2y - wy * g2x) * id;
    m2 = (g1x * wy - g1y * wx) * id;
}

// Edge e's contribution to agent j: into the first free slot of j's list, past
// them onto its chain.  (Slots found by a count, a scan over all targets and a
// pass that places every edge: four more launches, 42 of 519 us at 1M agents and
// 16 of 80 us at 16,384.)
__device__ __forceinline__ void add_edge(const AdjointBufs &b, uint32_t e, uint32_t j, float4 val)
{
    b.e_val[e] = val;
    const uint32_t slot = atomicAdd(&b.e_cnt[j], 1u);
    if (slot < (uint32_t)kEdgeSlots)
        b.e_list[(int64_t)j * kEdgeSlots + slot] = e;
    else
        b.e_next[e] = atomicExch(&b.e_head[j], e + 1u);
}

// One agent's step as the adjoint needs it: what its forward recomputation
// found, the same whichever kernel form ran it.
template <int BLOCK, bool ACC>
struct AdjAgent {
    int i, ci;
    float xi, yi, ri, vxi, vyi, vmax;  // state of the step
    float prx, pry;                    // desired velocity
    float vx, vy;                      // new velocity
    int nh, nacc;                      // hard lines, octagon lines among them
    dev::LdsLines<BLOCK, ACC> src;
    dev::ActiveSet rec;
};

// The VJP of an agent's step; pos_of(q): cell-order position of neighbour q.
template <int BLOCK, bool ACC, class PosOf>
__device__ __forceinline__ void adjoint_vjp(const AdjArgs &a, const AdjAgent<BLOCK, ACC> &f,
                                            PosOf &&pos_of)
{
    const dev::SceneP &p = a.p;
    const int i = f.i, ci = f.ci, nh = f.nh, nacc = f.nacc;
    const float xi = f.xi, yi = f.yi, ri = f.ri, vxi = f.vxi, vyi = f.vyi, vmax = f.vmax;
    const float prx = f.prx, pry = f.pry, vx = f.vx, vy = f.vy;
    const dev::LdsLines<BLOCK, ACC> &src = f.src;
    const dev::ActiveSet &rec = f.rec;
    const float turn = ACC ? (ci ? p.turn1 : p.turn0) : 0.0f;
    // the goal-mode quantities the desired velocity was formed from
    float gxg = 0.0f, gyg = 0.0f, d2g = 0.0f;
    if (p.pref_is_goal) {
        gxg = a.in.pref_x[i] - xi;
        gyg = a.in.pref_y[i] - yi;
        d2g = gxg * gxg + gyg * gyg;
    }

    // -- cotangent of the new velocity: v' directly and through p' = p + v' dt --
    const float gpx = a.gpx1[i], gpy = a.gpy1[i];
    const float wx = a.gvx1[i] + gpx * p.dt, wy = a.gvy1[i] + gpy * p.dt;

    // -- LP: active-set VJP --
    LineBars lb;
#pragma unroll
    for (int e = 0; e < kEdges; ++e) {
        lb.idx[e] = -1;
        lb.qx[e] = lb.qy[e] = lb.nx[e] = lb.ny[e] = 0.0f;
    }
    float pbx = 0.0f, pby = 0.0f;  // cotangent of the desired velocity
    float cbx = 0.0f, cby = 0.0f;  // cotangent of the acceleration octagon's centre
    float hbx = 0.0f, hby = 0.0f;  // cotangent of the heading (turn wedge)
    auto Lq = [&](int idx) { return src.line(idx); };
    // Rows of an LP3 sub-problem: line j < nh is a hard line, g = n_j,
    // r = n_j . q_j; otherwise the equal-penetration boundary of j and i3,
    // g = n_i3 - n_j, r = n_i3 . q_i3 - n_j . q_j.  For v = G^-1 r the
    // cotangents are r-bar = mu, g-bar = -mu v with mu = G^-T w; row_bar
    // scatters them to the lines and returns the share that goes to i3.
    auto row_g = [&](int j, float nix, float niy, float &gx, float &gy) {
        const float4 lj = Lq(j);
        if (ACC && j < nh) {
            gx = -lj.w;
            gy = lj.z;
        } else {
            gx = nix - (-lj.w);
            gy = niy - lj.z;
        }
    };
    auto row_bar = [&](int j, float mu) -> float {
        const float4 lj = Lq(j);
        const float njx = -lj.w, njy = lj.z;
        if (ACC && j < nh) {
            add_line(lb, j, mu * njx, mu * njy, mu * (lj.x - vx), mu * (lj.y - vy));
            return 0.0f;
        }
        add_line(lb, j, -mu * njx, -mu * njy, -mu * (lj.x - vx), -mu * (lj.y - vy));
        return mu;
    };
    switch (rec.kind) {
    case dev::kFree:
        pbx = wx;
        pby = wy;
        break;
    case dev::kDisc: {
        const float ol = sqrtf(prx * prx + pry * pry);
        const float ux = prx / ol, uy = pry / ol;
        const float uw = ux * wx + uy * wy;
        pbx = vmax / ol * (wx - ux * uw);
        pby = vmax / ol * (wy - uy * uw);
        break;
    }
    case dev::kLine: {
        const float4 l = Lq(rec.a);
        const float rx = prx - l.x, ry = pry - l.y;
        const float t = rx * l.z + ry * l.w;
        const float c = wx * l.z + wy * l.w;
        pbx = c * l.z;
        pby = c * l.w;
        // d-bar = t w + c r; n = (-d.y, d.x) so n-bar = (-dbar.y, dbar.x)
        const float dbx = t * wx + c * rx, dby = t * wy + c * ry;
        add_line(lb, rec.a, wx - c * l.z, wy - c * l.w, -dby, dbx);
        break;
    }
    case dev::kLineLine: {
        const float4 la = Lq(rec.a), lc = Lq(rec.b);
        const float nax = -la.w, nay = la.z, ncx = -lc.w, ncy = lc.z;
        float ma, mc;
        solve2(nax, nay, ncx, ncy, wx, wy, ma, mc);
        add_line(lb, rec.a, ma * nax, ma * nay, -ma * (vx - la.x), -ma * (vy - la.y));
        add_line(lb, rec.b, mc * ncx, mc * ncy, -mc * (vx - lc.x), -mc * (vy - lc.y));
        break;
    }
    case dev::kLineDisc: {
        const float4 la = Lq(rec.a);
        const float nax = -la.w, nay = la.z;
        float m1, m2;
        solve2(nax, nay, vx, vy, wx, wy, m1, m2);
        add_line(lb, rec.a, m1 * nax, m1 * nay, -m1 * (vx - la.x), -m1 * (vy - la.y));
        break;
    }
    case dev::kDir:
        add_line(lb, rec.i3, 0.0f, 0.0f, vmax * wx, vmax * wy);
        break;
    case dev::kProjDisc: {
        const float4 li = Lq(rec.i3);
        const float nix = -li.w, niy = li.z;
        float gax, gay, m1, m2;
        row_g(rec.a, nix, niy, gax, gay);
        solve2(gax, gay, vx, vy, wx, wy, m1, m2);
        const float ms = row_bar(rec.a, m1);
        if (!ACC || ms != 0.0f)
            add_line(lb, rec.i3, ms * nix, ms * niy, ms * (li.x - vx), ms * (li.y - vy));
        break;
    }
    case dev::kProjProj: {
        const float4 li = Lq(rec.i3);
        const float nix = -li.w, niy = li.z;
        float gax, gay, gcx, gcy, ma, mc;
        row_g(rec.a, nix, niy, gax, gay);
        row_g(rec.b, nix, niy, gcx, gcy);
        solve2(gax, gay, gcx, gcy, wx, wy, ma, mc);
        const float msa = row_bar(rec.a, ma);
        const float ms = msa + row_bar(rec.b, mc);
        if (!ACC || ms != 0.0f)
            add_line(lb, rec.i3, ms * nix, ms * niy, ms * (li.x - vx), ms * (li.y - vy));
        break;
    }
    case dev::kTie: {
        const float4 li = Lq(rec.i3), la = Lq(rec.a);
        const float nix = -li.w, niy = li.z, nax = -la.w, nay = la.z;
        const bool hard = ACC && rec.a < nh;
        float gx, gy;
        row_g(rec.a, nix, niy, gx, gy);
        const float G = gx * gx + gy * gy;
        const float h = hard ? nax * la.x + nay * la.y
                             : nix * li.x + niy * li.y - (nax * la.x + nay * la.y);
        const float sv = (gx * prx + gy * pry - h) / G;
        const float c = wx * gx + wy * gy;
        pbx = wx - c / G * gx;
        pby = wy - c / G * gy;
        const float hb = c / G;
        const float gbx = -(c / G) * (prx - 2.0f * sv * gx) - sv * wx;
        const float gby = -(c / G) * (pry - 2.0f * sv * gy) - sv * wy;
        if (hard) {
            add_line(lb, rec.a, hb * nax, hb * nay, gbx + hb * la.x, gby + hb * la.y);
        } else {
            add_line(lb, rec.i3, hb * nix, hb * niy, gbx + hb * li.x, gby + hb * li.y);
            add_line(lb, rec.a, -hb * nax, -hb * nay, -gbx - hb * la.x, -gby - hb * la.y);
        }
        break;
    }
    case dev::kCentre:
        cbx = wx;
        cby = wy;
        break;
    default:
        break;
    }

    // -- ORCA half-planes of the involved lines --
    const float fa = ci ? p.f10 : p.f00;  // f[ci][0]
    const float fb = ci ? p.f11 : p.f01;  // f[ci][1]
    float spx = 0.0f, spy = 0.0f, svx = 0.0f, svy = 0.0f, taub = 0.0f;
#pragma unroll
    for (int e = 0; e < kEdges; ++e) {
        if (ACC && lb.idx[e] >= 0 && lb.idx[e] < nacc) {
            // acceleration line: q = c + h n_k with a constant normal
            cbx += lb.qx[e];
            cby += lb.qy[e];
        } else if (ACC && lb.idx[e] >= nacc && lb.idx[e] < nh) {
            // wedge side: q = 0, d = R(-phi) h (right) or -R(phi) h (left);
            // n = (-d.y, d.x), so d-bar = (n-bar.y, -n-bar.x), and h-bar =
            // R(phi) d-bar (right) or -R(-phi) d-bar (left)
            float hx, hy, cs, sn, speed;
            dev::turn_basis(vxi, vyi, turn, p.dt, hx, hy, cs, sn, speed);
            const float dbx = lb.ny[e], dby = -lb.nx[e];
            if (lb.idx[e] == nacc) {
                hbx += cs * dbx - sn * dby;
                hby += sn * dbx + cs * dby;
            } else {
                hbx -= cs * dbx + sn * dby;
                hby -= -sn * dbx + cs * dby;
            }
        } else if (lb.idx[e] >= 0) {
            const uint32_t pj = pos_of(lb.idx[e] - nh);
            const float2 b0 = a.s0[pj];
            const float4 b1 = a.s1[pj];
            const int j = tag_index(b1.z);
            const float f = tag_class(b1.z) ? fb : fa;
            float Pbx, Pby, Vbx, Vby, itb;
            bool uses_tau;
            halfplane_vjp(xi, yi, vxi, vyi, ri, b0.x, b0.y, b1.x, b1.y, b1.w, f, p.inv_tau,
                          p.inv_dt, i < j, lb.qx[e], lb.qy[e], lb.nx[e], lb.ny[e], Pbx, Pby, Vbx,
                          Vby, itb, uses_tau);
            spx -= Pbx;
            spy -= Pby;
            svx += Vbx + lb.qx[e];
            svy += Vby + lb.qy[e];
            if (uses_tau) taub -= itb * p.inv_tau * p.inv_tau;
            add_edge(a.b, (uint32_t)(kEdges * i + e), (uint32_t)j,
                     make_float4(Pbx, Pby, -Vbx, -Vby));
        }
    }
    if (ACC && nh > nacc) {
        // h = v / |v|: Jacobian (I - h h^T) / |v|
        float hx, hy, cs, sn, speed;
        dev::turn_basis(vxi, vyi, turn, p.dt, hx, hy, cs, sn, speed);
        const float hh = hx * hbx + hy * hby;
        svx += (hbx - hx * hh) / speed;
        svy += (hby - hy * hh) / speed;
    }
    if (ACC && nh) {
        // c = v, or v (v_max / |v|) when |v| > v_max: Jacobian (v_max/|v|)(I - u u^T)
        const float v2 = vxi * vxi + vyi * vyi;
        if (v2 > vmax * vmax) {
            const float l = sqrtf(v2);
            const float ux = vxi / l, uy = vyi / l, sc = vmax / l;
            const float uc = ux * cbx + uy * cby;
            svx += sc * (cbx - ux * uc);
            svy += sc * (cby - uy * uc);
        } else {
            svx += cbx;
            svy += cby;
        }
    }

    // -- desired velocity: the pref input itself, or the goal --
    float grx = pbx, gry = pby;
    if (p.pref_is_goal) {
        grx = 0.0f;
        gry = 0.0f;
        if (d2g > 0.0f) {
            const float d = sqrtf(d2g);
            if (p.inv_dt < vmax / d) {
                grx = pbx * p.inv_dt;
                gry = pby * p.inv_dt;
            } else {
                const float ux = gxg / d, uy = gyg / d;
                const float up = ux * pbx + uy * pby;
                grx = vmax / d * (pbx - ux * up);
                gry = vmax / d * (pby - uy * up);
            }
        }
        spx -= grx;
        spy -= gry;
    }
    a.gprx[i] += grx;
    a.gpry[i] += gry;
    a.gpx0[i] = gpx + spx;
    a.gpy0[i] = gpy + spy;
    a.gvx0[i] = svx;
    a.gvy0[i] = svy;
    a.b.tau_part[i] = taub;
}

template <int K, int BLOCK, bool ACC, bool WALK>
__device__ __forceinline__ void adjoint_agent(bool live, int s, const AdjArgs &a, const GridMeta &g,
                                              float4 *lines, int tid)
{
    const dev::SceneP &p = a.p;
    const float2 me0 = a.s0[s];
    const float4 me1 = a.s1[s];
    AdjAgent<BLOCK, ACC> f;
    f.i = tag_index(me1.z);
    f.ci = tag_class(me1.z);
    f.xi = me0.x;
    f.yi = me0.y;
    f.ri = me1.w;
    f.vxi = me1.x;
    f.vyi = me1.y;

    // -- forward recomputation (identical to dev::step_agent) --
    uint64_t *buf = reinterpret_cast<uint64_t *>(lines);
    float kept = a.guess[f.i];
    const int found = dev::knn_select<K, BLOCK>(g, a.start, a.s0, a.s1, f.xi, f.yi, (uint32_t)s, buf,
                                                tid, &kept);
    if (live) a.guess[f.i] = kept;
    const int kk = p.k < K ? p.k : K;
    const int m = found < kk ? found : kk;
    uint32_t pos[K];
#pragma unroll
    for (int q = 0; q < K; ++q)
        pos[q] = q < m ? dev::entry_pos(buf[dev::buf_idx<BLOCK>(q, tid)]) : 0u;
    f.vmax = a.in.max_speed[f.i];
    const float acc = ACC ? (f.ci ? p.acc1 : p.acc0) : 0.0f;
    const float turn = ACC ? (f.ci ? p.turn1 : p.turn0) : 0.0f;
    f.nacc = (ACC && acc > 0.0f) ? dev::kAccLines : 0;
    float rx = 0.0f, ry = 0.0f, lx = 0.0f, ly = 0.0f;
    f.nh = f.nacc + ((ACC && dev::turn_wedge(f.vxi, f.vyi, turn, p.dt, rx, ry, lx, ly))
                         ? dev::kTurnLines : 0);
    dev::build_halfplanes<K, BLOCK>(pos, m, a.s0, a.s1, f.xi, f.yi, f.vxi, f.vyi, f.ri, f.i, f.ci, p,
                                    lines, tid);
    float cx = 0.0f, cy = 0.0f;
    if (ACC && f.nh) dev::accel_centre(f.vxi, f.vyi, f.vmax, cx, cy);
    f.prx = a.in.pref_x[f.i];
    f.pry = a.in.pref_y[f.i];
    dev::desired_velocity(p, f.xi, f.yi, f.vmax, f.prx, f.pry);
    f.src = dev::LdsLines<BLOCK, ACC>{lines, tid, f.nh, cx, cy,
                                      ACC && f.nacc ? dev::accel_half_width(acc, p.dt) : 0.0f,
                                      f.nacc, rx, ry, lx, ly};
    f.rec = dev::ActiveSet{dev::kFree, -1, -1, -1};
    const int mt = f.nh + m;
    int fail = dev::lp2<true, float>(f.src, mt, f.vmax, 0, f.prx, f.pry, 0.0f, 0.0f, p.eps, f.vx,
                                     f.vy, &f.rec);
    if (ACC && fail < f.nh) {
        f.vx = cx;
        f.vy = cy;
        fail = f.nh;
        f.rec.kind = dev::kCentre;
    }
    dev::wave_lp3<true, K, BLOCK, ACC, WALK>(f.src, tid, live && fail < mt, mt, fail, f.vmax, f.prx, f.pry,
                                       p.eps, f.vx, f.vy, &f.rec);
    if (!live) return;
    adjoint_vjp(a, f, [&](int qn) {
        uint32_t pj = 0u;
#pragma unroll
        for (int q = 0; q < K; ++q)
            if (q == qn) pj = pos[q];
        return pj;
    });
}

// (four wavefronts per SIMD up to K 10, as the LDS allows: one register too many
// without the bound)
template <int K, int BLOCK, bool ACC, bool WALK>
__global__ __launch_bounds__(BLOCK, K <= 10 && !ACC && WALK ? 4 : 1) void k_adjoint(AdjArgs a)
{
    __shared__ float4 lines[dev::KnnShape<K>::kSlots * BLOCK];
    const int tid = threadIdx.x;
    const int s = xcd_tile(blockIdx.x, gridDim.x) * BLOCK + tid;
    const GridMeta g = *a.meta;
    // every lane of the last wavefront takes part (LP3 is solved by quads)
    adjoint_agent<K, BLOCK, ACC, WALK>(s < a.n, min(s, a.n - 1), a, g, lines, tid);
}

// The same for a small crowd: a group of lanes per agent (orca_group.h), the
// VJP by its first lane.
template <int K, int G, bool ACC, bool WHOLE>
__global__ __launch_bounds__(kWave) void k_adjoint_group(AdjArgs a, float rn)
{
    __shared__ dev::GroupLds<K, G> lds;
    constexpr int A = kWave / G;
    const int who = threadIdx.x / G, c = threadIdx.x % G;
    const int at = xcd_tile(blockIdx.x, gridDim.x) * A + who;
    const bool live = at < a.n;
    const GridMeta g = WHOLE ? whole_crowd(a.n, rn) : *a.meta;
    AdjAgent<A, ACC> f;
    f.rec = dev::ActiveSet{dev::kFree, -1, -1, -1};
    const dev::GroupAgent<K, G, ACC> r = dev::group_step<true, K, G, ACC, WHOLE>(
        min(at, a.n - 1), g, a.p, a.in, a.start, a.s0, a.s1, lds, who, c, live, a.guess, &f.rec);
    if (!live || c != 0) return;
    f.i = r.i;
    f.ci = tag_class(r.s.z);
    f.xi = r.p.x;
    f.yi = r.p.y;
    f.ri = r.s.w;
    f.vxi = r.s.x;
    f.vyi = r.s.y;
    f.vmax = r.vmax;
    f.prx = r.prx;
    f.pry = r.pry;
    f.vx = r.vx;
    f.vy = r.vy;
    f.nh = r.nh;
    f.nacc = r.nacc;
    f.src = r.lines;
    adjoint_vjp(a, f, [&](int q) { return lds.nbr[who][q]; });
}

// Targets of more edges than a list holds are ordered by their own lane up to
// kHubLane, in a column of the wavefront's LDS (kHubCols lanes at a time), up to
// kHubWave by the wavefront there, and beyond as linked lists in place.
// (A column of 32 and not of 16 or 24: a vehicle among pedestrians has about k
// edges, and vehicles lie together in many orders; 5,000 agents, 50 of them with
// discs of 2.5 m, k 20: 202 us at 16, 100 at 24 and 32; k 32 260 at 24, 171 at 32.
// A column for every lane held the SIMDs to five wavefronts: 1M crossing 479 us, 472
// so.)
constexpr int kHubLane = 32;
constexpr int kHubCols = 32;
constexpr int kHubWords = kHubLane * kHubCols;  // of a wavefront
constexpr int kHubWave = kHubWords / 2;
constexpr int kHubBins = kHubWords / kWave;

// Two chains (edge index + 1, ended by 0), each ascending, into one.
__device__ uint32_t merge_chains(uint32_t *__restrict__ next, uint32_t x, uint32_t y)
{
    if (!x || !y) return x ? x : y;
    uint32_t head = 0, last = 0;
    while (x && y) {
        const uint32_t take = x < y ? x : y;
        (x < y ? x : y) = next[take - 1u];
        if (last)
            next[last - 1u] = take;
        else
            head = take;
        last = take;
    }
    next[last - 1u] = x ? x : y;
    return head;
}

// A chain of m edges beyond the LDS (agents at one place, which all look at the
// same few) and the target's list, as one ascending chain: every lane orders a
// 64th of it, one edge after another into chains of doubling lengths (`bins`, the
// lane's column), and the lanes' chains are merged pair by pair.
__device__ uint32_t sort_chain(const AdjointBufs &b, int64_t j, uint32_t m, uint32_t *bins, int lane)
{
    uint32_t *next = b.e_next;
    const uint32_t rest = m - (uint32_t)kEdgeSlots, share = (rest + kWave - 1) / kWave;
    uint32_t first = 0, h = b.e_head[j];
    for (uint32_t at = 0; at < rest && h; ++at) {
        if (at == (uint32_t)lane * share) first = h;
        h = next[h - 1u];
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    for (int k = 0; k < kHubBins; ++k) bins[k * kWave] = 0u;
    const uint32_t from = (uint32_t)lane * share;
    uint32_t left = from < rest ? min(share, rest - from) : 0u;
    uint32_t mine = lane < kEdgeSlots ? b.e_list[j * kEdgeSlots + lane] + 1u : 0u;
    while (mine || left) {
        uint32_t chain = mine;
        if (!chain) {
            chain = first;
            first = next[chain - 1u];
            --left;
        }
        mine = 0u;
        next[chain - 1u] = 0u;
        for (int k = 0;; ++k) {
            const uint32_t have = bins[k * kWave];
            bins[k * kWave] = 0u;
            chain = merge_chains(next, have, chain);
            if (!have || k == kHubBins - 1) {
                bins[k * kWave] = chain;
                break;
            }
        }
    }
    uint32_t chain = 0;
    for (int k = 0; k < kHubBins; ++k) chain = merge_chains(next, bins[k * kWave], chain);
    for (int o = 1; o < kWave; o <<= 1) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        const uint32_t other = (uint32_t)__shfl_down((int)chain, o, kWave);
        if (lane % (2 * o) == 0) chain = merge_chains(next, chain, other);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    return (uint32_t)__shfl((int)chain, 0, kWave);
}

// The sum of the m > kHubLane edges of target j, by a wavefront, in increasing edge
// index.  `lds`: the wavefront's.
__device__ float4 hub_sum(const AdjointBufs &b, int64_t j, uint32_t m, uint32_t *lds, int lane)
{
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    auto add = [&](const float4 &v) {
        s.x += v.x;
        s.y += v.y;
        s.z += v.z;
        s.w += v.w;
    };
    dev::lane_order<kWave>();  // the lanes' own columns are read
    if (m > (uint32_t)kHubWave) {
        for (uint32_t h = sort_chain(b, j, m, lds + lane, lane); h; h = b.e_next[h - 1u])
            add(b.e_val[h - 1u]);
        return s;
    }
    uint32_t *sorted = lds + kHubWave;
    if (lane < kEdgeSlots) lds[lane] = b.e_list[j * kEdgeSlots + lane];
    uint32_t h = b.e_head[j];
    for (uint32_t q = kEdgeSlots; q < m && h; ++q) {
        if (lane == 0) lds[q] = h - 1u;
        h = b.e_next[h - 1u];
    }
    dev::lane_order<kWave>();
    for (uint32_t q = lane; q < m; q += kWave) {
        const uint32_t e = lds[q];
        uint32_t rank = 0;
#pragma unroll 4
        for (uint32_t r = 0; r < m; ++r) rank += lds[r] < e ? 1u : 0u;
        sorted[rank] = e;
    }
    dev::lane_order<kWave>();
    for (uint32_t q = 0; q < m; q += kWave) {
        const float4 v = b.e_val[sorted[min(q + (uint32_t)lane, m - 1u)]];
        auto lane_of = [](float x, int r) {
            return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), r));
        };
        for (int r = 0; r < min((int)(m - q), kWave); ++r)
            add(make_float4(lane_of(v.x, r), lane_of(v.y, r), lane_of(v.z, r), lane_of(v.w, r)));
    }
    return s;
}

// Each target sums its edges in increasing edge index (= source agent, slot):
// those of its list ordered in registers, more of them as above.  (One walk over
// the chain for each edge summed cost a lane c (c - 8) dependent loads for c edges:
// 600 agents at one place among 5,000, k 10: 4640 us a call, 540 so.)  TAU: the block's
// tau contributions too (a fixed order: lanes, then wavefronts).
template <bool TAU>
__global__ __launch_bounds__(kBlock) void k_edge_gather(int n, AdjointBufs b, float *gpx0, float *gpy0,
                                                        float *gvx0, float *gvy0)
{
    __shared__ uint32_t order[kBlock / kWave][kHubWords];
    const int lane = threadIdx.x % kWave;
    uint32_t *lds = order[threadIdx.x / kWave];
    const int j = blockIdx.x * kBlock + threadIdx.x;
    const uint32_t c = j < n ? b.e_cnt[j] : 0u;
    float sx = 0.0f, sy = 0.0f, tx = 0.0f, ty = 0.0f;
    auto add = [&](const float4 &v) {
        sx += v.x;
        sy += v.y;
        tx += v.z;
        ty += v.w;
    };
    const bool hub = c > (uint32_t)kEdgeSlots && c <= (uint32_t)kHubLane;
    const uint64_t own = __ballot(hub);
    const int rank = __popcll(own & ((1ull << lane) - 1ull));
    uint32_t e[kEdgeSlots];
    if (c <= (uint32_t)kHubLane) {
        static_assert(kEdgeSlots == 8, "two loads and a network of eight");
        const uint4 *l = (const uint4 *)(b.e_list + (int64_t)min(j, n - 1) * kEdgeSlots);
        const uint4 p = l[0], q = c > 4u ? l[1] : make_uint4(~0u, ~0u, ~0u, ~0u);
        e[0] = c > 0u ? p.x : ~0u;
        e[1] = c > 1u ? p.y : ~0u;
        e[2] = c > 2u ? p.z : ~0u;
        e[3] = c > 3u ? p.w : ~0u;
        e[4] = c > 4u ? q.x : ~0u;
        e[5] = c > 5u ? q.y : ~0u;
        e[6] = c > 6u ? q.z : ~0u;
        e[7] = c > 7u ? q.w : ~0u;
        dev::sort_network<kEdgeSlots>(e);
        if (!hub) {
#pragma unroll
            for (int k = 0; k < kEdgeSlots; ++k)
                if ((uint32_t)k < c) add(b.e_val[e[k]]);
        }
    }
    for (int first = 0; first < __popcll(own); first += kHubCols) {
        dev::lane_order<kWave>();  // the columns of the lanes before are read
        if (hub && rank >= first && rank < first + kHubCols) {
            uint32_t *col = lds + (rank - first);
#pragma unroll
            for (int k = 0; k < kEdgeSlots; ++k) col[k * kHubCols] = e[k];
            uint32_t h = b.e_head[j];
            for (int k = kEdgeSlots; k < (int)c && h; ++k) {
                int at = k;
                for (; at > 0 && col[(at - 1) * kHubCols] > h - 1u; --at)
                    col[at * kHubCols] = col[(at - 1) * kHubCols];
                col[at * kHubCols] = h - 1u;
                h = b.e_next[h - 1u];
            }
            for (uint32_t k = 0; k < c; ++k) add(b.e_val[col[k * kHubCols]]);
        }
    }
    for (uint64_t hubs = __ballot(c > (uint32_t)kHubLane); hubs; hubs &= hubs - 1) {
        const int who = __ffsll((long long)hubs) - 1;
        const float4 v = hub_sum(b, (int64_t)(j - lane + who), (uint32_t)__shfl((int)c, who, kWave),
                                 lds, lane);
        if (lane == who) add(v);
    }
    if (j < n) {
        gpx0[j] += sx;
        gpy0[j] += sy;
        gvx0[j] += tx;
        gvy0[j] += ty;
    }
    if (TAU) {
        __shared__ double red[kBlock / kWave];
        double t = j < n ? (double)b.tau_part[j] : 0.0;
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) t += __shfl_xor(t, o, kWave);
        if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = t;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kBlock / kWave; ++w) t += red[w];
            b.tau_blocks[blockIdx.x] = t;
        }
    }
}

// g_tau += the sum of the block sums, in a fixed order.
__global__ __launch_bounds__(kBlock) void k_tau_final(const double *__restrict__ blocks, int nb,
                                                      float *g_tau)
{
    __shared__ double red[kBlock];
    double s = 0.0;
    for (int k = threadIdx.x; k < nb; k += kBlock) s += blocks[k];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) *g_tau += (float)red[0];
}

template <int K, bool ACC>
void launch_adjoint_v(const AdjArgs &a, hipStream_t stream)
{
    const int nb = (a.n + kAdjBlock - 1) / kAdjBlock;
    if (K <= 12 && a.n > kWalkAgents)
        hipLaunchKernelGGL((k_adjoint<K, kAdjBlock, ACC, K <= 12>), dim3(nb), dim3(kAdjBlock), 0, stream,
                           a);
    else
        hipLaunchKernelGGL((k_adjoint<K, kAdjBlock, ACC, K <= kBriefList>), dim3(nb), dim3(kAdjBlock), 0,
                           stream, a);
}

template <int K>
void launch_adjoint_k(const AdjArgs &a, hipStream_t stream)
{
    if (a.p.acc0 > 0.0f || a.p.acc1 > 0.0f || a.p.turn0 > 0.0f || a.p.turn1 > 0.0f)
        launch_adjoint_v<K, true>(a, stream);
    else
        launch_adjoint_v<K, false>(a, stream);
}

template <int K, bool ACC>
void launch_adjoint_group_k(const AdjArgs &a, bool whole, float rn, hipStream_t stream)
{
    const int nb = (a.n + kWave / kGroup - 1) / (kWave / kGroup);
    if (whole)
        hipLaunchKernelGGL((k_adjoint_group<K, kGroup, ACC, true>), dim3(nb), dim3(kWave), 0, stream,
                           a, rn);
    else
        hipLaunchKernelGGL((k_adjoint_group<K, kGroup, ACC, false>), dim3(nb), dim3(kWave), 0,
                           stream, a, rn);
}

void launch_adjoint_group(const AdjArgs &a, bool whole, float rn, hipStream_t stream)
{
    const bool acc = a.p.acc0 > 0.0f || a.p.acc1 > 0.0f || a.p.turn0 > 0.0f || a.p.turn1 > 0.0f;
    if (a.p.k <= 16)
        acc ? launch_adjoint_group_k<16, true>(a, whole, rn, stream)
            : launch_adjoint_group_k<16, false>(a, whole, rn, stream);
    else
        acc ? launch_adjoint_group_k<32, true>(a, whole, rn, stream)
            : launch_adjoint_group_k<32, false>(a, whole, rn, stream);
}

}  // namespace

hipError_t launch_adjoint(const orca_agents_in &in, int n, const orca_params &prm,
                          const Layout &L, const Work &w, const AdjointBufs &b,
                          const float *gpx1, const float *gpy1, const float *gvx1,
                          const float *gvy1, float *gpx0, float *gpy0, float *gvx0, float *gvy0,
                          float *gprx, float *gpry, float *g_tau, const orca_step_events *ev,
                          hipStream_t stream)
{
    (void)L;
    AdjArgs a;
    a.in = in;
    a.n = n;
    a.meta = w.meta;
    a.start = w.start;
    a.s0 = w.s0;
    a.s1 = w.s1;
    a.guess = w.guess;
    a.p = dev::scene_params(prm);
    a.gpx1 = gpx1;
    a.gpy1 = gpy1;
    a.gvx1 = gvx1;
    a.gvy1 = gvy1;
    a.gpx0 = gpx0;
    a.gpy0 = gpy0;
    a.gvx0 = gvx0;
    a.gvy0 = gvy0;
    a.gprx = gprx;
    a.gpry = gpry;
    a.b = b;
    const int k = prm.max_neighbors;
    if (ev && ev->step_begin && hipEventRecord(ev->step_begin, stream) != hipSuccess)
        return hipErrorInvalidValue;
    if (n <= group_adjoint_max(prm))
        launch_adjoint_group(a, n <= kWholeMax, prm.neighbor_dist, stream);
    else if (k <= 4)
        launch_adjoint_k<4>(a, stream);
    else if (k <= 8)
        launch_adjoint_k<8>(a, stream);
    else if (k <= 10)
        launch_adjoint_k<10>(a, stream);
    else if (k <= 12)
        launch_adjoint_k<12>(a, stream);
    else if (k <= 16)
        launch_adjoint_k<16>(a, stream);
    else if (k <= 20)
        launch_adjoint_k<20>(a, stream);
    else if (k <= 24)
        launch_adjoint_k<24>(a, stream);
    else
        launch_adjoint_k<32>(a, stream);
    if (ev && ev->step_end && hipEventRecord(ev->step_end, stream) != hipSuccess)
        return hipErrorInvalidValue;
    const int nb = (n + kBlock - 1) / kBlock;
    if (g_tau) {
        hipLaunchKernelGGL((k_edge_gather<true>), dim3(nb), dim3(kBlock), 0, stream, n, b, gpx0, gpy0,
                           gvx0, gvy0);
        hipLaunchKernelGGL(k_tau_final, dim3(1), dim3(kBlock), 0, stream, b.tau_blocks, nb, g_tau);
    } else {
        hipLaunchKernelGGL((k_edge_gather<false>), dim3(nb), dim3(kBlock), 0, stream, n, b, gpx0,
                           gpy0, gvx0, gvy0);
    }
    return hipGetLastError();
}

}  // namespace orca
