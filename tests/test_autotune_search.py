"""The autotuner's search on the CPU, with the timing replaced: it times only
configurations that run differently, and a choice found for one form of the
kernels is not used for another."""
import os
import re

import pytest
import torch

from paper_2008_11578_amd import autotune, orca, scenarios

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class FakeBatch:
    def __init__(self, off, params, mode=0, block=0, k_tile=0):
        self.cell = params[0].cell_size / params[0].neighbor_dist
        self.shape = (mode, block, k_tile)


def effect(n, batch):
    """What the library runs for a batch of n agents."""
    mode, block, k_tile = batch.shape
    if n <= autotune.GROUP_BATCH_MAX:
        return batch.cell, 16 if k_tile <= 16 else 32
    return batch.cell, block if mode == 1 and block else 64, k_tile


@pytest.fixture
def search(monkeypatch, tmp_path):
    monkeypatch.setenv("ORCA_AUTOTUNE_CACHE", str(tmp_path / "tune.json"))
    monkeypatch.setattr(orca, "Batch", FakeBatch)

    def run(n, k, cost=lambda e: 1.0, **kw):
        z = torch.zeros(n)
        st = orca.State(*([torch.linspace(0.0, 100.0, n)] * 2 + [z] * 7))
        now = []
        monkeypatch.setattr(orca, "step_batched", lambda s, b, ws, out: now.append(effect(n, b)))

        def timed(fn, reps):
            fn()
            return cost(now[-1])

        monkeypatch.setattr(autotune, "_time_ms", timed)
        p = scenarios.Params(neighbor_dist=5.0, max_neighbors=k)
        r = autotune.tune_batched(st, [0, n], [p], None, **kw)
        return r, list(now)

    return run


@pytest.mark.parametrize("n", [5000, 98304, 98305, 400000])
@pytest.mark.parametrize("k", [4, 10, 16, 20, 32])
def test_no_stage_times_one_kernel_twice(search, n, k):
    r, ran = search(n, k)
    cells, shapes, tiles = ({e[q] for e in ran} for q in (0, 1, -1))
    assert cells == set(autotune.FACTORS)
    stages = [len(autotune.FACTORS)]
    if n > autotune.GROUP_BATCH_MAX:
        assert shapes == set(autotune.BLOCKS)
        stages += [3, len([t for t in autotune.K_TILES if t >= k][:3])]
    else:
        stages += [2 if k <= 16 else 1]
    assert len(ran) == sum(stages)
    at = 0
    for s in stages:
        assert len(set(ran[at:at + s])) == s, ran[at:at + s]
        at += s
    assert r["mode"] in autotune.MODES and r["block"] in autotune.BLOCKS and r["k_tile"] >= k


def test_lanes_are_found_where_there_is_a_choice(search):
    r, _ = search(400000, 10, cost=lambda e: 1.0 if e[1] == 256 else 2.0)
    assert (r["mode"], r["block"]) == (1, 256)
    r, _ = search(400000, 10, cost=lambda e: 1.0 if e[1] == 64 else 2.0, use_cache=False)
    assert (r["mode"], r["block"]) == (0, 64)


def test_choice_is_not_shared_between_kernel_forms(search):
    r, _ = search(98304, 10, cost=lambda e: 1.0 if e[1] == 32 else 2.0)
    assert r["k_tile"] == 32 and not r["cached"]
    assert search(98304, 10)[0]["cached"]
    assert not search(98305, 10)[0]["cached"]


def test_key_names_the_kernels_generation(monkeypatch):
    a = autotune.cache_key("plain", 1000, 1.0, 10)
    monkeypatch.setattr(autotune, "KERNELS", autotune.KERNELS + 1)
    assert autotune.cache_key("plain", 1000, 1.0, 10) != a


def test_lines_are_the_library_s():
    src = open(os.path.join(ROOT, "paper_2008_11578_amd", "csrc", "orca_internal.h")).read()
    for name, value in (("kWholeMax", autotune.WHOLE_MAX), ("kGroupBatchMax", autotune.GROUP_BATCH_MAX)):
        assert int(re.search(name + r" = (\d+);", src).group(1)) == value
