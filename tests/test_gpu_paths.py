"""Which kernel runs is chosen by sizes alone and changes no result: on both
sides of each such line, the two forms agree bit for bit."""
import numpy as np
import pytest

from paper_2008_11578_amd import scenarios

pytestmark = pytest.mark.gpu

FIELDS = ("px", "py", "vx", "vy")


def _scenes(total, params, seed):
    """Uneven scenes with `total` agents together."""
    sizes = [total // 2 + 1, 1, total // 3, 63]
    sizes.append(total - sum(sizes))
    parts = [scenarios.random_state(n, max(np.sqrt(n / 0.5), 5.0), seed=seed + s, n_vehicles=n // 20,
                                    params=params) for s, n in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    return off, {k: np.concatenate([getattr(p, k) for p in parts]) for k in parts[0].arrays()}


@pytest.mark.parametrize("total", [98304, 98305])
def test_batch_by_groups_of_lanes_equals_a_lane_per_agent(total):
    """Batches of up to 98,304 agents are stepped by groups of lanes, larger
    ones by a lane per agent: every scene equals its plain step (itself by
    groups up to 72,000 agents), and a workgroup size of 256 lanes with a
    capacity of 32 neighbours gives the same."""
    import torch
    from paper_2008_11578_amd import orca
    p = scenarios.Params(dt=0.05, neighbor_dist=5.0, max_neighbors=16)
    off, cat = _scenes(total, p, seed=70)
    st = orca.State.from_arrays(cat)
    got = []
    for mode, block, k_tile in ((0, 0, 0), (1, 256, 32)):
        b = orca.Batch(off, [p] * (len(off) - 1), mode=mode, block=block, k_tile=k_tile)
        status = torch.zeros(st.n, dtype=torch.uint8, device="cuda")
        out = orca.step_batched(st, b, orca.Workspace(st.n, n_scenes=len(off) - 1), status=status)
        torch.cuda.synchronize()
        assert int(b.error.item()) == 0
        got.append([getattr(out, k) for k in FIELDS] + [status])
    for a, b in zip(*got):
        assert torch.equal(a, b)
    for a, z in zip(off[:-1], off[1:]):
        part = orca.State(**{k: getattr(st, k)[a:z].clone() for k in orca.STATE_FIELDS})
        o1 = orca.step(part, p, orca.Workspace(part.n))
        torch.cuda.synchronize()
        for k, v in zip(FIELDS, got[0]):
            assert torch.equal(v[a:z], getattr(o1, k)), (a, k)


@pytest.mark.parametrize("k", [1, 4, 5, 16, 20, 32])
@pytest.mark.parametrize("jam,free,caps", [(15, 49, False), (17, 47, False), (33, 30, False),
                                           (64, 0, False), (65, 1, False), (9, 40, True),
                                           (64, 0, True)])
def test_least_penetration_by_groups_of_lanes(k, jam, free, caps):
    """A wavefront's agents in LP3 are solved 16 (8 with hard lines) at a
    time: jammed agents on either side of that, up to whole wavefronts, among
    free ones in caller order, and the last wavefront partly empty."""
    from parity import compare_step
    rng = np.random.Generator(np.random.PCG64(1000 + 7 * jam + k))
    p = scenarios.Params(dt=0.1, neighbor_dist=6.0, max_neighbors=k, pref_is_goal=0,
                         accel=(2.0, 1.0) if caps else (0.0, 0.0),
                         turn=(0.0, 1.0) if caps else (0.0, 0.0))
    n = jam + free
    order = rng.permutation(n)
    x = np.where(np.arange(n) < jam, rng.uniform(0.0, 2.5, n), 50.0 + 20.0 * np.arange(n))[order]
    y = np.where(np.arange(n) < jam, rng.uniform(0.0, 2.5, n), 10.0)[order]
    veh = rng.random(n) < 0.2
    f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32)  # noqa: E731
    ang, sp = rng.uniform(0.0, 2.0 * np.pi, n), np.where(veh, 6.0, 1.5)
    st = {"px": f32(x), "py": f32(y), "vx": f32(0.9 * sp * np.cos(ang)),
          "vy": f32(0.9 * sp * np.sin(ang)), "pref_x": f32(0.9 * sp * np.sin(ang)),
          "pref_y": f32(0.9 * sp * np.cos(ang)), "radius": f32(np.where(veh, 0.8, 0.3)),
          "max_speed": f32(sp), "cls": veh.astype(np.uint8)}
    rep, g, o = compare_step(st, p, max_ill_frac=1.0)
    assert rep["n_bad"] <= max(2, n // 20), rep
    if k >= 4:
        assert rep["lp3_oracle"] >= jam // 3, rep


@pytest.mark.parametrize("k", [1, 4, 8, 10, 12, 16, 20, 24, 32])
def test_kept_scan_radius_changes_no_result(k):
    """Each agent keeps the radius of its neighbour scan in the workspace.  A
    circle kept from another crowd holds too few (sparse after dense), more
    than the sorting network takes, more than the buffer, more than the
    byte counters (300 agents within it), agents at one place (ties and keys
    of zero beside the own), or no agent but the own: lists and velocities
    equal those of a fresh workspace bit for bit, call after call."""
    import torch
    from paper_2008_11578_amd import orca
    n = 331
    rng = np.random.Generator(np.random.PCG64(500 + k))
    p = scenarios.Params(dt=0.1, neighbor_dist=4.0, max_neighbors=k)
    sides = [3.0, 8.0, 14.0, 20.0, 60.0, 2000.0, 8.0, 20.0]
    ws, wsb = orca.Workspace(n), orca.Workspace(n, backward=True)
    g = [torch.randn(n, device="cuda", generator=torch.Generator("cuda").manual_seed(j))
         for j in range(4)]

    def backward(st, w):
        acc = [torch.zeros(n, device="cuda") for _ in range(2)] + [torch.zeros(1, device="cuda")]
        return list(orca.step_backward(st, p, w, *g, *acc)) + acc

    for rep, side in enumerate(sides):
        sc = scenarios.random_state(n, side, seed=600 + 31 * rep + k, n_vehicles=8, params=p)
        if rep % 2:  # lattice places: ties in distance, and agents at one place
            sc.px = np.round(sc.px * 2.0).astype(np.float32) / 2
            sc.py = np.round(sc.py * 2.0).astype(np.float32) / 2
        sc.px[rng.integers(0, n, 9)] = sc.px[0]
        st = orca.State.from_arrays(sc)
        for again in range(2):
            out, nbr, cnt = orca.step_nbr(st, p, ws)
            ref, rnbr, rcnt = orca.step_nbr(st, p, orca.Workspace(n))
            lnbr, lcnt = orca.build_grid(st, p, ws)
            fnbr, fcnt = orca.build_grid(st, p, orca.Workspace(n))
            torch.cuda.synchronize()
            for a, b in ((nbr, rnbr), (cnt, rcnt), (lnbr, fnbr), (lcnt, fcnt), (nbr, fnbr),
                         *[(getattr(out, f), getattr(ref, f)) for f in FIELDS]):
                assert torch.equal(a, b), (rep, again)
            for a, b in zip(backward(st, wsb), backward(st, orca.Workspace(n, backward=True))):
                assert torch.equal(a, b), (rep, again)


@pytest.mark.parametrize("caps", [False, True])
@pytest.mark.parametrize("n,k,side", [(1, 4, 1.0), (2, 1, 1.0), (5, 32, 2.0), (66, 16, 4.0),
                                      (257, 10, 30.0), (300, 17, 2.0), (2048, 20, 40.0),
                                      (2049, 20, 40.0), (5003, 16, 100.0), (4000, 24, 12.0)])
def test_small_crowd_by_groups_of_lanes_equals_a_lane_per_agent(n, k, side, caps):
    """The same crowd alone (a group of lanes per agent; without a grid up to
    2,048 agents) and with 140,000 agents standing far away, which makes the
    call take a lane per agent: velocities, lists and the VJP agree bit for bit.
    300 agents within 2 m and 4,000 within 12 m hold more than a group's
    buffer (64) in every circle; a hundred stand at one place, more than fit
    any cut of it."""
    import torch
    from paper_2008_11578_amd import orca
    p = scenarios.Params(dt=0.1, neighbor_dist=4.0, max_neighbors=k, pref_is_goal=k % 2,
                         accel=(2.0, 1.0) if caps else (0.0, 0.0),
                         turn=(0.0, 1.0) if caps else (0.0, 0.0))
    sc = scenarios.random_state(n, side, seed=40 + n + k, n_vehicles=n // 10, params=p)
    if n == 300:
        sc.px[100:200], sc.py[100:200] = sc.px[0], sc.py[0]
    m = 140000
    far = {f: np.zeros(m, v.dtype) for f, v in sc.arrays().items()}
    far["px"] = (1000.0 + 10.0 * (np.arange(m) % 400)).astype(np.float32)
    far["py"] = (1000.0 + 10.0 * (np.arange(m) // 400)).astype(np.float32)
    far["pref_x"], far["pref_y"] = far["px"].copy(), far["py"].copy()
    far["radius"] += np.float32(0.3)
    far["max_speed"] += np.float32(1.5)
    both = {f: np.concatenate([v, far[f]]) for f, v in sc.arrays().items()}
    gen = np.random.Generator(np.random.PCG64(9))
    cot = [gen.standard_normal(n).astype(np.float32) for _ in range(4)]
    got = []
    for arrays in (sc.arrays(), both):
        st = orca.State.from_arrays(arrays)
        ws, wsb = orca.Workspace(st.n), orca.Workspace(st.n, backward=True)
        for again in range(2):  # the second call from the kept radii
            out, nbr, cnt = orca.step_nbr(st, p, ws)
            g = [torch.cat([torch.from_numpy(c), torch.zeros(st.n - n)]).cuda() for c in cot]
            acc = [torch.zeros(st.n, device="cuda") for _ in range(2)]
            b = orca.step_backward(st, p, wsb, *g, *acc, torch.zeros(1, device="cuda"))
            torch.cuda.synchronize()
            got.append([t[:n] for t in (*[getattr(out, f) for f in FIELDS], nbr, cnt, *b, *acc)])
    for other in got[1:]:
        for q, (a, b) in enumerate(zip(got[0], other)):
            assert torch.equal(a, b), q


@pytest.mark.parametrize("n,nc,spread,agents,t_clear", [
    (3, 1, 1.0, 5.0, 1.0), (4000, 700, 20000.0, 30000.0, 0.5), (4000, 1500, 3.0, 40.0, 0.0),
    (2500, 1025, 60.0, 4000.0, 0.25), (500, 16384, 500.0, 100.0, 0.02), (300, 200, 0.0, 30.0, 0.5)])
@pytest.mark.parametrize("odd", ["", "nan", "inf"])
def test_spawn_grid_over_the_candidates(n, nc, spread, agents, t_clear, odd):
    """The candidates' grid: boxes that would need more cells than it has, all
    candidates in one cell or at one place, agents far outside the box, and
    places that are not finite (no box: one cell holds everyone).  Decisions
    equal the oracle's, taken one by one in order."""
    import oracle
    import torch
    from paper_2008_11578_amd import orca
    rng = np.random.default_rng(n + nc)

    def crowd(m, side, shift):
        f = {k: np.zeros(m, np.float32) for k in ("vx", "vy", "pref_x", "pref_y")}
        f["px"] = (shift + rng.uniform(0, max(side, 1e-9), m)).astype(np.float32)
        f["py"] = (shift + rng.uniform(0, max(side, 1e-9), m)).astype(np.float32)
        f["radius"] = rng.uniform(0.2, 0.6, m).astype(np.float32)
        f["max_speed"] = rng.uniform(0.5, 6.0, m).astype(np.float32)
        return dict(f, cls=np.zeros(m, np.uint8))

    a, c = crowd(n, agents, -agents / 3), crowd(nc, spread, 7.0)
    if odd:
        c["px"][nc // 2] = a["py"][n // 2] = np.float32(odd)
    room = {k: np.concatenate([v, c[k]]) for k, v in a.items()}
    acc = torch.empty(nc, dtype=torch.uint8, device="cuda")
    tot = orca.spawn(orca.State.from_arrays(room), n, orca.State.from_arrays(c), t_clear,
                     orca.LifecycleWorkspace(n, nc), accepted=acc)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        want = oracle.spawn(a, c, t_clear)
    np.testing.assert_array_equal(acc.cpu().numpy(), want)
    assert int(tot.item()) == n + int(want.sum())


def _hub(m, n):
    """A disc and a ring of m agents walking into it, and agents far away."""
    ang = 2.0 * np.pi * (np.arange(m) + 0.25) / m
    far = 0.5 * m / np.pi + 4.0
    f = {k: np.zeros(n, np.float32) for k in ("px", "py", "vx", "vy", "pref_x", "pref_y", "radius",
                                              "max_speed")}
    f["px"][1:m + 1], f["py"][1:m + 1] = far * np.cos(ang), far * np.sin(ang)
    f["px"][m + 1:] = 1000.0 + 40.0 * (np.arange(n - m - 1) % 250)
    f["py"][m + 1:] = 1000.0 + 40.0 * (np.arange(n - m - 1) // 250)
    for k, wave in (("vx", np.cos), ("pref_x", np.cos), ("vy", np.sin), ("pref_y", np.sin)):
        f[k][1:m + 1] = -1.2 * wave(ang + 0.05)
    f["radius"][:] = 0.3
    f["radius"][0] = far - 2.0
    f["max_speed"][:] = 1.5
    return dict(f, cls=np.zeros(n, np.uint8))


@pytest.mark.parametrize("m", [6, 8, 9, 40])
@pytest.mark.parametrize("filler", [0, 60000])
def test_adjoint_sums_every_contribution_to_an_agent(m, filler):
    """Every agent around a hub avoids it, so the hub receives about m
    contributions: as many as its list holds, one more, and many more.  The VJP
    is linear in the cotangents, so the hub's answer to all of them together is
    the sum of its answers to a third of the agents at a time, and those to one
    agent at a time (three contributions at most), but for the rounding of m
    FP32 additions; and call after call gives the same bits.  With 60,000
    agents far away the call takes a lane per agent."""
    import torch
    from paper_2008_11578_amd import orca
    n = m + 1 + filler
    p = scenarios.Params(dt=0.1, neighbor_dist=120.0, max_neighbors=min(m, 32), pref_is_goal=0)
    st = orca.State.from_arrays(_hub(m, n))
    ws = orca.Workspace(n, backward=True)
    gen = torch.Generator().manual_seed(m)
    cot = [torch.zeros(n) for _ in range(4)]
    for c in cot:
        c[1:m + 1] = torch.randn(m, generator=gen)

    def hub(mask):
        g = [(c * mask).cuda() for c in cot]
        acc = [torch.zeros(n, device="cuda") for _ in range(2)] + [torch.zeros(1, device="cuda")]
        out = orca.step_backward(st, p, ws, *g, *acc)
        return torch.stack([t[0] for t in (*out, acc[2])]).double().cpu().numpy()

    whole = hub(torch.ones(n))
    np.testing.assert_array_equal(whole, hub(torch.ones(n)))
    assert np.abs(whole).sum() > 1e-3
    ones = [hub((torch.arange(n) == i).float()) for i in range(1, m + 1)]
    thirds = [hub((torch.arange(n) % 3 == r).float()) for r in range(3)]
    for parts in (ones, thirds):
        size = np.sum(np.abs(ones), axis=0)
        assert (np.abs(whole - np.sum(parts, axis=0)) <= 4 * m * 2.0 ** -24 * size + 1e-30).all()
    assert sum(np.abs(o[:4]).sum() > 0 for o in ones) > min(m, 32) * 0.6  # the hub is in most ways


@pytest.mark.parametrize("n", [2049, 32768, 32769])
@pytest.mark.parametrize("cell", [0.0, 0.07, 300.0])
def test_small_crowd_grid_lists_match_oracle(n, cell):
    """Crowds of up to 32,768 agents bound their grid at 8,192 cells and scan
    and scatter in one kernel: neighbour lists equal the oracle's on both
    sides of the line, with cells that would be far more, the default, and one
    cell for all; also of a crowd on a line (cells along one axis only)."""
    import oracle
    from parity import gpu_neighbors
    p = scenarios.Params(neighbor_dist=3.0, max_neighbors=10, cell_size=cell)
    sc = scenarios.random_state(n, np.sqrt(n / (0.5 if cell < 200 else 40.0)), seed=n, params=p)
    lists = [sc]
    if cell < 200:
        line = sc.copy()
        line.px, line.py = (line.px * 300.0).astype(np.float32), (line.py * 0.0).astype(np.float32)
        lists.append(line)
    for s in lists:
        nbr, cnt = gpu_neighbors(s, p)
        ref = oracle.step(s, p, want_neighbors=True)
        np.testing.assert_array_equal(nbr, ref["nbr"])


def test_rollout_of_a_state_held_in_columns():
    """A state's arrays may have any shape of n elements: positions in columns
    give the trajectory and gradients of flat ones, and keep their shape."""
    import torch
    from paper_2008_11578_amd import orca, rollout
    sc = scenarios.c5_rollout(n=300, side=30.0)
    got = []
    for shape in ((300,), (300, 1)):
        st = orca.State.from_arrays(sc.arrays())
        prx, pry = st.pref_x.clone().requires_grad_(), st.pref_y.clone().requires_grad_()
        for k in FIELDS:
            setattr(st, k, getattr(st, k).reshape(shape))
        tau = torch.tensor(2.0, device="cuda", requires_grad=True)
        px, py = rollout.rollout(prx, pry, tau, st, sc.params, 7, 3)
        assert px.shape == shape and py.shape == shape
        (px.square().mean() + py.square().mean()).backward()
        got.append((px.detach().reshape(-1), py.detach().reshape(-1), prx.grad, pry.grad, tau.grad))
    for a, b in zip(*got):
        assert torch.equal(a, b)
