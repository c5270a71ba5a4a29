"""The kernels that take a lane per agent, on crowds small enough to be checked in
every detail: agents standing far away lift the call above the sizes that are
stepped by groups of lanes, and the answers of the crowd proper equal those it has
alone (by groups, which other tests hold against the oracle) bit for bit."""
import numpy as np
import pytest

from paper_2008_11578_amd import scenarios

pytestmark = pytest.mark.gpu

FIELDS = ("px", "py", "vx", "vy")
FAR = 140000        # above every line of the step and the adjoint, and of the lists up to k 24
FAR_LISTS = 270000  # above the line of longer lists


def _params(k, caps=False, goal=0, rn=4.0):
    return scenarios.Params(dt=0.1, neighbor_dist=rn, max_neighbors=k, pref_is_goal=goal,
                            accel=(2.0, 1.0) if caps else (0.0, 0.0),
                            turn=(0.0, 1.0) if caps else (0.0, 0.0))


def _among(arrays, m):
    """The crowd with m agents standing far away, one to a cell."""
    far = {f: np.zeros(m, v.dtype) for f, v in arrays.items()}
    far["px"] = (1000.0 + 10.0 * (np.arange(m) % 600)).astype(np.float32)
    far["py"] = (1000.0 + 10.0 * (np.arange(m) // 600)).astype(np.float32)
    far["pref_x"], far["pref_y"] = far["px"].copy(), far["py"].copy()
    far["radius"] += np.float32(0.3)
    far["max_speed"] += np.float32(1.5)
    return {f: np.concatenate([v, far[f]]) for f, v in arrays.items()}


def _cotangents(n, total, seed=9):
    import torch
    gen = np.random.Generator(np.random.PCG64(seed))
    return [torch.cat([torch.from_numpy(gen.standard_normal(n).astype(np.float32)),
                       torch.zeros(total - n)]).cuda() for _ in range(4)]


def _answers(st, p, n, ws, wsb, cot, lists=True):
    """Everything a call gives for the first n agents."""
    import torch
    from paper_2008_11578_amd import orca
    status = torch.zeros(st.n, dtype=torch.uint8, device="cuda")
    out, nbr, cnt = orca.step_nbr(st, p, ws, status=status)
    acc = [torch.zeros(st.n, device="cuda") for _ in range(2)]
    back = orca.step_backward(st, p, wsb, *cot, *acc, torch.zeros(1, device="cuda"))
    got = [*[getattr(out, f) for f in FIELDS], status, nbr, cnt, *back, *acc]
    if lists:
        got += list(orca.build_grid(st, p, ws))
    torch.cuda.synchronize()
    return [t[:n] for t in got]


def _same(a, b, what):
    import torch
    for q, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x, y), (what, q)


@pytest.mark.parametrize("caps", [False, True])
@pytest.mark.parametrize("k", [1, 3, 4, 6, 8, 9, 11, 12, 14, 18, 22, 28, 32])
def test_every_capacity_equals_the_groups(k, caps):
    """Each compiled capacity with and without hard lines: step, lists, VJP."""
    from paper_2008_11578_amd import orca
    n = 3001
    p = _params(k, caps, goal=k % 2)
    sc = scenarios.random_state(n, 70.0, seed=80 + k, n_vehicles=n // 10, params=p)
    got = []
    for arrays in (sc.arrays(), _among(sc.arrays(), FAR if k <= 24 else FAR_LISTS)):
        st = orca.State.from_arrays(arrays)
        ws, wsb = orca.Workspace(st.n), orca.Workspace(st.n, backward=True)
        for again in range(2):
            got.append(_answers(st, p, n, ws, wsb, _cotangents(n, st.n)))
    for other in got[1:]:
        _same(got[0], other, k)


@pytest.mark.parametrize("caps", [False, True])
@pytest.mark.parametrize("k", [4, 8, 10, 12, 16, 20, 24, 32])
def test_radius_kept_from_another_crowd_changes_no_result(k, caps):
    """A circle kept from another crowd: too few within it, more than the sorting
    network takes, than the buffer, than the counters (300 agents), agents at
    one place, none but the own.  Lists, velocities and the VJP equal those of
    a fresh workspace, call after call."""
    from paper_2008_11578_amd import orca
    n = 331
    rng = np.random.Generator(np.random.PCG64(700 + k))
    p = _params(k, caps)
    m = FAR if k <= 24 else FAR_LISTS
    ws, wsb = orca.Workspace(n + m), orca.Workspace(n + m, backward=True)
    cot = _cotangents(n, n + m, seed=k)
    for rep, side in enumerate([3.0, 8.0, 14.0, 20.0, 60.0, 900.0, 8.0, 20.0]):
        sc = scenarios.random_state(n, side, seed=600 + 31 * rep + k, n_vehicles=8, params=p)
        if rep % 2:  # lattice places: ties in distance, and agents at one place
            sc.px = np.round(sc.px * 2.0).astype(np.float32) / 2
            sc.py = np.round(sc.py * 2.0).astype(np.float32) / 2
        sc.px[rng.integers(0, n, 9)] = sc.px[0]
        st = orca.State.from_arrays(_among(sc.arrays(), m))
        fresh = _answers(st, p, n, orca.Workspace(st.n), orca.Workspace(st.n, backward=True), cot)
        for again in range(2):
            _same(fresh, _answers(st, p, n, ws, wsb, cot), (rep, again))


@pytest.mark.parametrize("caps", [False, True])
@pytest.mark.parametrize("k", [4, 5, 10, 12, 16, 20, 32])
@pytest.mark.parametrize("jam", [7, 9, 15, 17, 33, 39, 40, 41, 42, 47, 48, 49, 50, 63, 64, 90])
def test_least_penetration_in_a_wavefront_of_agents(jam, k, caps):
    """Jammed agents, one beside the other in cell order, on either side of the
    counts at which LP3 takes another round of groups (16, 8 with hard lines) or
    is walked by the lanes (40, 48): velocities, active sets (through the VJP)
    and status as by groups."""
    from paper_2008_11578_amd import orca
    rng = np.random.Generator(np.random.PCG64(1000 + 7 * jam + k))
    p = _params(k, caps, rn=6.0)
    n = jam + 5
    order = rng.permutation(n)
    x = np.where(np.arange(n) < jam, rng.uniform(0.0, 2.5, n), 50.0 + 20.0 * np.arange(n))[order]
    y = np.where(np.arange(n) < jam, rng.uniform(0.0, 2.5, n), 10.0)[order]
    veh = rng.random(n) < 0.2
    f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32)  # noqa: E731
    ang, sp = rng.uniform(0.0, 2.0 * np.pi, n), np.where(veh, 6.0, 1.5)
    arrays = {"px": f32(x), "py": f32(y), "vx": f32(0.9 * sp * np.cos(ang)),
              "vy": f32(0.9 * sp * np.sin(ang)), "pref_x": f32(0.9 * sp * np.sin(ang)),
              "pref_y": f32(0.9 * sp * np.cos(ang)), "radius": f32(np.where(veh, 0.8, 0.3)),
              "max_speed": f32(sp), "cls": veh.astype(np.uint8)}
    got = []
    for a in (arrays, _among(arrays, FAR)):
        st = orca.State.from_arrays(a)
        got.append(_answers(st, p, n, orca.Workspace(st.n), orca.Workspace(st.n, backward=True),
                            _cotangents(n, st.n), lists=False))
    _same(got[0], got[1], jam)
    if k >= 10:
        assert int(got[0][4].sum()) >= jam // 2  # in LP3


@pytest.mark.parametrize("caps", [False, True])
@pytest.mark.parametrize("block,k_tile", [(64, 0), (128, 0), (256, 0), (128, 24), (256, 32), (64, 32)])
def test_large_batch_scenes_equal_their_plain_steps(block, k_tile, caps):
    """A batch of more agents than the groups take, in every workgroup size and
    with larger capacities, jammed, sparse and tiny scenes: each equals its plain
    step, which runs by groups."""
    import torch
    from paper_2008_11578_amd import orca
    sizes = [(3000, 3.0), (1500, 0.05), (2200, 0.6), (1, 1.0), (64, 2.0), (98400, 0.1), (129, 0.5)]
    ks = [16, 10, 16, 4, 12, 8, 16]
    parts, prm = [], []
    for s, ((n, density), k) in enumerate(zip(sizes, ks)):
        p = _params(k, caps and s % 3 != 1, rn=5.0)
        prm.append(p)
        parts.append(scenarios.random_state(n, float(np.sqrt(n / density)), seed=900 + s,
                                            n_vehicles=n // 20, params=p))
    off = np.concatenate([[0], np.cumsum([q.n for q in parts])]).astype(np.int32)
    st = orca.State.from_arrays({f: np.concatenate([getattr(q, f) for q in parts])
                                 for f in parts[0].arrays()})
    b = orca.Batch(off, prm, mode=1, block=block, k_tile=k_tile)
    ws = orca.Workspace(st.n, n_scenes=len(parts))
    for again in range(2):
        status = torch.zeros(st.n, dtype=torch.uint8, device="cuda")
        out = orca.step_batched(st, b, ws, status=status)
        torch.cuda.synchronize()
        assert int(b.error.item()) == 0
        for s, q in enumerate(parts):
            status1 = torch.zeros(q.n, dtype=torch.uint8, device="cuda")
            one = orca.step(orca.State.from_arrays(q), prm[s], orca.Workspace(q.n), status=status1)
            torch.cuda.synchronize()
            a, z = off[s], off[s + 1]
            for f in FIELDS:
                assert torch.equal(getattr(out, f)[a:z], getattr(one, f)), (s, f)
            assert torch.equal(status[a:z], status1), s


def test_full_batch_in_every_workgroup_size():
    """All 512 scenes (5,559,168 agents): 128 and 256 lanes give what 64 give."""
    import torch
    from paper_2008_11578_amd import orca
    sc = scenarios.c4_batched()
    st = orca.State.from_arrays(sc)
    got = []
    for mode, block in ((0, 0), (1, 64), (1, 128), (1, 256)):
        b = orca.Batch(sc.scene_off, sc.scene_params, mode=mode, block=block)
        status = torch.zeros(st.n, dtype=torch.uint8, device="cuda")
        out = orca.step_batched(st, b, orca.Workspace(st.n, n_scenes=len(sc.scene_params)), status=status)
        torch.cuda.synchronize()
        assert int(b.error.item()) == 0
        got.append([*[getattr(out, f) for f in FIELDS], status])
    for other in got[1:]:
        _same(got[0], other, "block")
