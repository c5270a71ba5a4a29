"""The grid over the spawn candidates at the largest number of cells it may have."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CELLS = 8192


def _box_at_the_limit():
    """A radius, a speed cap and two places on a line so that the candidates'
    box holds just under CELLS cells by the quotient of its length and the
    cell, and CELLS by the product with the cell's reciprocal."""
    rng = np.random.default_rng(0)
    f = np.float32
    while True:
        r, s = f(rng.uniform(0.2, 0.6)), f(rng.uniform(0.5, 3.0))
        cell = ((float(r) + float(r)) + (float(s) + float(s))) * (1.0 + 1e-6)
        w = CELLS * cell
        for _ in range(4):
            hi = f(w)
            lo = f(float(hi) - w)
            if (float(hi) - float(lo) == w and np.floor(w / cell) == CELLS - 1
                    and np.floor(w * (1.0 / cell)) == CELLS):
                return r, s, lo, hi
            w = float(np.nextafter(w, 0.0))


def test_spawn_where_the_box_fills_the_grid_by_rounding_alone():
    """Candidates along a line, some beside another or beside an agent: the
    decisions equal the oracle's, taken one by one in order, all along it."""
    import oracle
    import torch
    from paper_2008_11578_amd import orca
    r, s, lo, hi = _box_at_the_limit()
    mid = np.linspace(50.0, float(hi) - 50.0, 60).astype(np.float32)
    crowds = []
    for x in (mid[::3] + np.float32(1.0), np.concatenate([[lo, hi], mid, mid + np.float32(0.5)])):
        z = np.zeros(x.size, np.float32)
        crowds.append({"px": x.astype(np.float32), "py": z, "vx": z, "vy": z, "pref_x": z,
                       "pref_y": z, "radius": z + r, "max_speed": z + s,
                       "cls": np.zeros(x.size, np.uint8)})
    a, c = crowds
    n, nc = a["px"].size, c["px"].size
    room = orca.State.from_arrays({k: np.concatenate([v, c[k]]) for k, v in a.items()})
    acc = torch.empty(nc, dtype=torch.uint8, device="cuda")
    total = orca.spawn(room, n, orca.State.from_arrays(c), 1.0, orca.LifecycleWorkspace(n, nc),
                       accepted=acc)
    torch.cuda.synchronize()
    want = oracle.spawn(a, c, 1.0)
    assert 0 < want.sum() < nc
    np.testing.assert_array_equal(acc.cpu().numpy(), want)
    assert int(total.item()) == n + int(want.sum())


def _crowd(rng, m, side, in_places):
    x, y = rng.uniform(0.0, side, m), rng.uniform(0.0, side, m)
    if in_places:  # the caller's order follows the places, in rows 10 m wide
        o = np.lexsort((x, np.floor(y / 10.0)))
        x, y = x[o], y[o]
    z = np.zeros(m, np.float32)
    return {"px": x.astype(np.float32), "py": y.astype(np.float32), "vx": z, "vy": z, "pref_x": z,
            "pref_y": z, "radius": rng.uniform(0.2, 0.6, m).astype(np.float32),
            "max_speed": rng.uniform(0.5, 2.0, m).astype(np.float32), "cls": np.zeros(m, np.uint8)}


def _spawn(a, c, t_clear):
    import torch
    from paper_2008_11578_amd import orca
    n, nc = a["px"].size, c["px"].size
    room = orca.State.from_arrays({k: np.concatenate([v, c[k]]) for k, v in a.items()})
    cand, ws = orca.State.from_arrays(c), orca.LifecycleWorkspace(n, nc)
    acc = torch.empty(nc, dtype=torch.uint8, device="cuda")
    return lambda: (orca.spawn(room, n, cand, t_clear, ws, accepted=acc), acc)


@pytest.mark.parametrize("in_places", [False, True])
@pytest.mark.parametrize("n,nc,side,t_clear", [
    (1, 3, 4.0, 0.5), (5, 70, 9.0, 0.0), (16383, 300, 400.0, 0.3), (32769, 900, 600.0, 2.0),
    (262143, 400, 3000.0, 1.0), (262144, 2000, 3000.0, 0.0), (300007, 500, 3000.0, 12.0)])
def test_agents_beside_few_and_beside_many_candidates(n, nc, side, t_clear, in_places):
    """Agents look through the candidates beside them by lanes or by whole
    wavefronts, and small crowds with few agents in a wavefront: decisions
    equal the oracle's for short and long ranges and both kinds of order."""
    import oracle
    import torch
    rng = np.random.default_rng(n + nc)
    a, c = _crowd(rng, n, side, in_places), _crowd(rng, nc, side / 4.0, in_places)
    total, acc = _spawn(a, c, t_clear)()
    torch.cuda.synchronize()
    want = oracle.spawn(a, c, t_clear)
    np.testing.assert_array_equal(acc.cpu().numpy(), want)
    assert int(total.item()) == n + int(want.sum())


def test_a_wide_clearance_among_agents_in_any_order_stays_cheap():
    """A million agents in random order, a few in a hundred of them within the
    clearance of all 16,384 candidates: no wavefront walks the candidates for
    one or two of its lanes alone (84 times the narrow clearance's time, 4.5 now)."""
    import torch
    rng = np.random.default_rng(7)
    a, c = _crowd(rng, 1 << 20, 1448.0, False), _crowd(rng, 16384, 181.0, False)
    took = []
    for t_clear in (0.0, 15.0):
        go = _spawn(a, c, t_clear)
        go()
        best = float("inf")
        for _ in range(5):
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            begin.record()
            go()
            end.record()
            torch.cuda.synchronize()
            best = min(best, begin.elapsed_time(end))
        took.append(best)
    print("narrow %.3f ms, wide %.3f ms" % tuple(took))
    assert took[1] < 40.0 * took[0]
