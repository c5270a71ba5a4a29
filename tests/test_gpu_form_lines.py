"""Which form of a kernel runs is chosen by sizes: a call just below such a line
does not take much longer than one just above it, with little work for each agent
or much."""
import numpy as np
import pytest

from paper_2008_11578_amd import scenarios

pytestmark = pytest.mark.gpu


def _time(call):
    import torch
    for _ in range(3):
        call()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(8):
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        begin.record()
        for _ in range(10):
            call()
        end.record()
        torch.cuda.synchronize()
        best = min(best, begin.elapsed_time(end) * 100.0)
    return best


def _took(what, n, density, k, caps):
    import torch
    from paper_2008_11578_amd import orca
    p = scenarios.Params(dt=0.05, neighbor_dist=5.0, max_neighbors=k,
                         accel=(2.0, 1.0) if caps else (0.0, 0.0), turn=(0.0, 1.0) if caps else (0.0, 0.0))
    sc = scenarios.random_state(n, float(np.sqrt(n / density)), seed=5, n_vehicles=n // 20, params=p)
    st = orca.State.from_arrays(sc)
    prm, out = orca.make_params(p), st.clone()
    ws = orca.Workspace(n, backward=what == "adjoint")
    g = [torch.ones(n, device="cuda") for _ in range(4)]
    acc = [torch.zeros(n, device="cuda") for _ in range(2)] + [torch.zeros(1, device="cuda")]
    to = tuple(torch.empty_like(t) for t in g)
    return _time({"step": lambda: orca.step(st, prm, ws, out=out),
                  "lists": lambda: orca.build_grid(st, prm, ws),
                  "adjoint": lambda: orca.step_backward(st, prm, ws, *g, *acc, out=to)}[what])


@pytest.mark.parametrize("what,line,k,caps", [
    ("step", 16384, 4, False), ("step", 72000, 4, False), ("step", 72000, 10, False),
    ("step", 72000, 4, True), ("step", 98304, 16, True), ("step", 131072, 4, True),
    ("step", 131072, 20, True), ("adjoint", 49152, 10, False), ("adjoint", 49152, 4, True),
    ("adjoint", 72000, 4, True), ("lists", 65536, 10, False),
    ("lists", 49152, 4, False), ("step", 131072, 8, True), ("adjoint", 131072, 10, False)])
def test_both_sides_of_a_line_take_about_as_long(what, line, k, caps):
    for density in (0.05, 0.3):
        below, above = (_took(what, n, density, k, caps) for n in (line, line + 1))
        print(f"{what} {line} k {k} caps {caps} {density} /m^2: {below:.1f} / {above:.1f} us")
        assert below < 1.28 * above, density
