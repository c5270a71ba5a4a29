"""The adjoint's sum over the contributions to one agent, for agents that very many
others look at: agents at one place all take the same few of them (the lowest in
the caller's order) as their nearest."""
import numpy as np
import pytest

from paper_2008_11578_amd import scenarios

pytestmark = pytest.mark.gpu


def _crowd(m, n, k, seed):
    """m agents at one place (the first in the caller's order), n - m around them."""
    p = scenarios.Params(dt=0.1, neighbor_dist=5.0, max_neighbors=k, pref_is_goal=0)
    sc = scenarios.random_state(n, float(np.sqrt(n / 0.3)), seed=seed, params=p)
    sc.px[:m], sc.py[:m] = sc.px[0], sc.py[0]
    return sc, p


def _backward(sc, p):
    import torch
    from paper_2008_11578_amd import orca
    st = orca.State.from_arrays(sc.arrays())
    n = st.n
    ws = orca.Workspace(n, backward=True)

    def go(cot):
        acc = [torch.zeros(n, device="cuda") for _ in range(2)] + [torch.zeros(1, device="cuda")]
        return torch.stack(orca.step_backward(st, p, ws, *cot, *acc))

    return go


@pytest.mark.parametrize("filler", [0, 60000])  # by groups of lanes, by a lane per agent
@pytest.mark.parametrize("m,k", [(14, 4), (26, 4), (30, 10), (56, 4), (80, 4), (300, 4), (1300, 4),
                                 (1900, 4)])
def test_contributions_are_summed_in_the_order_of_their_sources(m, k, filler):
    """A source's contribution does not depend on the other agents' cotangents, so
    calls with one source at a time give every term, and the sum of all of them,
    in FP32 and in the order of the sources, is the whole call's answer bit for
    bit: for as many terms as a list, a lane, a wavefront's LDS holds, and more."""
    import torch
    n = m + 40 + filler
    go = _backward(*_crowd(m, n, k, seed=m))
    gen = torch.Generator().manual_seed(m)
    hubs = list(range(k + 1))
    cot = [torch.zeros(n) for _ in range(4)]
    for c in cot:
        c[k + 1:m] = torch.randn(m - k - 1, generator=gen)  # none of the hubs' own
    whole = go([c.cuda() for c in cot])[:, hubs].cpu().numpy()
    one = [torch.zeros(n, device="cuda") for _ in range(4)]
    terms = []
    for i in range(k + 1, m):
        for o, c in zip(one, cot):
            o[i] = c[i]
        terms.append(go(one)[:, hubs].clone())
        for o in one:
            o[i] = 0.0
    terms = torch.stack(terms).cpu().numpy()
    total = np.zeros_like(whole)
    for t in terms:
        total += t
    count = (np.abs(terms).sum(axis=1) > 0).sum(axis=0)
    print("terms of each:", count)
    np.testing.assert_array_equal(whole, total)
    np.testing.assert_array_equal(whole, go([c.cuda() for c in cot])[:, hubs].cpu().numpy())
    assert count.max() > 0.4 * m * 3 / max(k, 3) - 6


@pytest.mark.parametrize("m", [4000, 20000])
def test_thousands_at_one_place_stay_cheap(m):
    """The terms are ordered once, not found again for each (4,000 agents at one
    place: 690 ms when they were)."""
    import torch
    n = m + 1000
    go = _backward(*_crowd(m, n, 4, seed=3))
    cot = [torch.randn(n, device="cuda") for _ in range(4)]
    first = go(cot)
    best = float("inf")
    for _ in range(3):
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        begin.record()
        again = go(cot)
        end.record()
        torch.cuda.synchronize()
        best = min(best, begin.elapsed_time(end))
    print(f"{m} at one place: {best:.2f} ms")
    assert torch.equal(first, again)
    assert best < 25.0 * m / 1000.0


@pytest.mark.parametrize("filler", [0, 60000])
@pytest.mark.parametrize("vehicles,ring", [(70, 14), (64, 20), (33, 12), (30, 38)])
def test_a_wavefront_of_vehicles_that_everyone_avoids(vehicles, ring, filler):
    """Vehicles lie together in the caller's order, each in a ring of pedestrians
    who walk towards it, so most lanes of a wavefront have more terms than a list
    holds: each vehicle's sum is the FP32 sum of its terms in the order of the
    sources."""
    import torch
    n = vehicles * (ring + 1)
    p = scenarios.Params(dt=0.1, neighbor_dist=8.0, max_neighbors=16, pref_is_goal=0,
                         f=((0.5, 1.0), (0.0, 0.5)))
    rng = np.random.default_rng(ring)
    side = 0.12 * ring + 0.6  # radius of the ring
    at = np.stack([np.arange(vehicles) % 9, np.arange(vehicles) // 9], 1) * (2.0 * side + 9.0)
    ang = 2.0 * np.pi * (np.arange(ring)[None] + rng.uniform(0, 0.3, (vehicles, ring))) / ring
    out = np.stack([np.cos(ang), np.sin(ang)], 2)
    arrays = {f: np.zeros(n, np.float32) for f in ("px", "py", "vx", "vy", "pref_x", "pref_y",
                                                  "radius", "max_speed")}
    for c, f in enumerate(("px", "py")):
        arrays[f][:vehicles] = at[:, c]
        arrays[f][vehicles:] = (at[:, None, c] + side * out[:, :, c]).ravel()
    for c, (f, g) in enumerate((("vx", "pref_x"), ("vy", "pref_y"))):
        arrays[f][vehicles:] = arrays[g][vehicles:] = (-1.2 * out[:, :, c]).ravel()
    arrays["radius"][:] = 0.2
    arrays["radius"][:vehicles] = side - 0.5
    arrays["max_speed"][:] = 1.5
    arrays["cls"] = (np.arange(n) < vehicles).astype(np.uint8)
    if filler:
        far = {f: np.zeros(filler, v.dtype) for f, v in arrays.items()}
        far["px"] = (1000.0 + 20.0 * (np.arange(filler) % 250)).astype(np.float32)
        far["py"] = (1000.0 + 20.0 * (np.arange(filler) // 250)).astype(np.float32)
        far["radius"] += np.float32(0.3)
        far["max_speed"] += np.float32(1.5)
        arrays = {f: np.concatenate([v, far[f]]) for f, v in arrays.items()}

    class Crowd:
        pass

    crowd = Crowd()
    crowd.arrays = lambda: arrays
    go = _backward(crowd, p)
    total = n + filler
    gen = torch.Generator().manual_seed(ring)
    cot = [torch.zeros(total) for _ in range(4)]
    for c in cot:
        c[vehicles:n] = torch.randn(n - vehicles, generator=gen)
    whole = go([c.cuda() for c in cot])[:, :vehicles].cpu().numpy()
    one = [torch.zeros(total, device="cuda") for _ in range(4)]
    terms = []
    for i in range(vehicles, n):
        for o, c in zip(one, cot):
            o[i] = c[i]
        terms.append(go(one)[:, :vehicles].clone())
        for o in one:
            o[i] = 0.0
    terms = torch.stack(terms).cpu().numpy()
    sums = np.zeros_like(whole)
    for t in terms:
        sums += t
    count = (np.abs(terms).sum(axis=1) > 0).sum(axis=0)
    print("terms of each vehicle: %d to %d, %d of %d more than 8" %
          (count.min(), count.max(), (count > 8).sum(), vehicles))
    assert (count > min(8, ring - 2)).mean() > 0.7
    np.testing.assert_array_equal(whole, sums)
