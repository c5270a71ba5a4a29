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


@pytest.mark.parametrize("total", [65536, 65537])
def test_batch_that_fits_the_device_at_once_equals_the_queued_form(total):
    """Neighbour capacity 32 at 256 lanes takes 128 KB of LDS, so one workgroup
    per CU: 256 of them hold 65,536 agents, one more agent goes to the
    queues; the flat launch form never queues."""
    import torch
    from paper_2008_11578_amd import orca
    p = scenarios.Params(dt=0.05, neighbor_dist=5.0, max_neighbors=16)
    off, cat = _scenes(total, p, seed=70)
    st = orca.State.from_arrays(cat)
    got = []
    for mode in (0, 1):
        b = orca.Batch(off, [p] * (len(off) - 1), mode=mode, block=256, k_tile=32)
        status = torch.zeros(st.n, dtype=torch.uint8, device="cuda")
        out = orca.step_batched(st, b, orca.Workspace(st.n, n_scenes=len(off) - 1), status=status)
        torch.cuda.synchronize()
        assert int(b.error.item()) == 0
        got.append([getattr(out, k) for k in FIELDS] + [status])
    for a, b in zip(*got):
        assert torch.equal(a, b)
