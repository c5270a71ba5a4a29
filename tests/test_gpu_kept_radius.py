"""The radius of the neighbour scan that a workspace keeps for each agent: it
changes no result, but a poor one makes a call scan again and again."""
import numpy as np
import pytest

from paper_2008_11578_amd import scenarios

pytestmark = pytest.mark.gpu

N = 140000  # a lane per agent, whichever the options


def _crowd(density, k, rn=5.0, n=N):
    p = scenarios.Params(dt=0.05, neighbor_dist=rn, max_neighbors=k)
    return scenarios.random_state(n, float(np.sqrt(n / density)), seed=11, params=p), p


def _kept(ws, n):
    """The radii, the last region of the workspace (float32, caller order)."""
    import torch
    at = ws.nbytes - (4 * n + 255) // 256 * 256
    return ws.buf[at:at + 4 * n].view(torch.float32).double().cpu().numpy()


def _kth_distance(sc, nbr, k):
    """Distance of the k-th neighbour, NaN where there are fewer."""
    j = nbr.cpu().numpy()[:, k - 1]
    x, y = sc.px.astype(np.float64), sc.py.astype(np.float64)
    return np.where(j >= 0, np.hypot(x[j] - x, y[j] - y), np.nan)


@pytest.mark.parametrize("density,k", [(2.0, 20), (1.0, 10), (2.0, 16), (0.6, 32), (0.5, 8)])
def test_kept_circle_holds_the_nearest(density, k):
    """After two steps of a crowd at rest in its places the kept circle of every
    agent with k neighbours in range holds them, so the third scans no circle
    twice."""
    import torch
    from paper_2008_11578_amd import orca
    sc, p = _crowd(density, k)
    st, ws = orca.State.from_arrays(sc), orca.Workspace(N)
    out = st.clone()
    for _ in range(2):
        orca.step(st, p, ws, out=out)
    nbr, _ = orca.build_grid(st, p, orca.Workspace(N))
    torch.cuda.synchronize()
    kept, dk = _kept(ws, N), _kth_distance(sc, nbr, k)
    full = ~np.isnan(dk)
    assert full.mean() > 0.9
    assert (kept[full] > 0).all()
    assert int((kept[full] <= dk[full]).sum()) == 0
