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
