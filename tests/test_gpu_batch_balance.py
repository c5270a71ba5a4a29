"""Scenes of one batch that cost far from alike."""
import numpy as np
import pytest

from paper_2008_11578_amd import scenarios

pytestmark = pytest.mark.gpu

FIELDS = ("px", "py", "vx", "vy")


def _batch(dense, sizes, k=16):
    import torch  # noqa: F401
    from paper_2008_11578_amd import orca
    p = scenarios.Params(dt=0.05, neighbor_dist=5.0, max_neighbors=k)
    parts = [scenarios.random_state(n, float(np.sqrt(n / (2.0 if d else 0.1))), seed=s, params=p)
             for s, (d, n) in enumerate(zip(dense, sizes))]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    st = orca.State.from_arrays({f: np.concatenate([getattr(q, f) for q in parts])
                                 for f in parts[0].arrays()})
    return st, p, off, parts


def test_order_of_dense_scenes_does_not_set_the_time():
    """Eight dense scenes among sixty-four of 16,384 agents take about the same time
    at the head or the end of the batch as spread over it (two and a half times as
    long when each XCD had its eighth of the batch in one piece)."""
    import torch
    from paper_2008_11578_amd import orca
    took = []
    for dense in ([s < 8 for s in range(64)], [s >= 56 for s in range(64)],
                  [s % 8 == 0 for s in range(64)], [s % 8 == 3 for s in range(64)]):
        st, p, off, _ = _batch(dense, [16384] * 64)
        b, ws, out = orca.Batch(off, [p] * 64), orca.Workspace(st.n, n_scenes=64), st.clone()
        best = float("inf")
        for _ in range(6):
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            begin.record()
            orca.step_batched(st, b, ws, out=out)
            end.record()
            torch.cuda.synchronize()
            best = min(best, begin.elapsed_time(end))
        took.append(best)
    print(["%.3f" % t for t in took])
    assert max(took) < 1.5 * min(took)


@pytest.mark.parametrize("sizes", [[98305], [49152, 49153 + 64 * 8 - 1], [100000, 1, 37000],
                                   [64 * 128 * 8 * 2, 64 * 100 + 1], [262144, 1], [262080, 64],
                                   [64 * 8 * 130 * 8 + 63]])
@pytest.mark.parametrize("block", [64, 128, 256])
def test_every_tile_is_stepped_once(sizes, block):
    """Tile counts on, below and above whole rounds of chunks, in each workgroup
    size: every scene equals its plain step and nothing is left out."""
    import torch
    from paper_2008_11578_amd import orca
    st, p, off, parts = _batch([False] * len(sizes), sizes, k=4)
    out = st.clone()
    for k in FIELDS:
        getattr(out, k).fill_(float("nan"))
    orca.step_batched(st, orca.Batch(off, [p] * len(sizes), mode=1, block=block),
                      orca.Workspace(st.n, n_scenes=len(sizes)), out=out)
    for q, a, z in zip(parts, off[:-1], off[1:]):
        one = orca.step(orca.State.from_arrays(q), p, orca.Workspace(q.n))
        torch.cuda.synchronize()
        for k in FIELDS:
            assert torch.equal(getattr(out, k)[a:z], getattr(one, k)), (k, a)
