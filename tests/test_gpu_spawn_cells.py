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
