"""autotune_batch on a batch that ordinary calls run on the members' sectors:
its candidates of tiles and work items run on the full vectors, which they
shape, and the stored lanes are the ordinary calls' best.  Watches which of the
two a timed call runs by the members' timing switch."""
import numpy as np
import pytest
import torch

from paper_2408_00836_amd import abi, tune, workloads as W
from paper_2408_00836_amd.model import Batch, Hubbard

pytestmark = pytest.mark.gpu


def test_candidates_run_where_they_count(gpu, tmp_path, monkeypatch):
    wl = W.batch(6)
    monkeypatch.setenv("HUBVQE_TUNE_CACHE", str(tmp_path / "t.json"))
    models = [Hubbard(w.nx, w.ny, **w.kwargs()) for w in wl]
    b = Batch(models, [w.layers for w in wl])
    theta = torch.tensor(np.concatenate([w.theta for w in wl]), device=gpu)
    on, timed = set(), []
    switch, run = abi.hubbard_set_timing, b.energy_grad

    def set_timing(h, enable):
        (on.add if enable else on.discard)(h)
        switch(h, enable)

    def energy_grad(th):
        assert len(on) in (0, len(models))
        timed.append((bool(on), b.config, b.member_tiles))
        return run(th)
    monkeypatch.setattr(abi, "hubbard_set_timing", set_timing)
    monkeypatch.setattr(b, "energy_grad", energy_grad)
    ent = tune.autotune_batch(b, theta, reps=1)
    assert not on
    full = {(tuple(c), t) for f, c, t in timed if f}
    assert full == {((i, l), t) for t in tune.BATCH_TILES for i in tune.BATCH_ITEMS
                    for l in tune.BATCH_LANES}
    ordinary = {(tuple(c), t) for f, c, t in timed if not f}
    items, lanes, tiles = ent["best"]
    assert ordinary == {((items, l), tiles) for l in tune.BATCH_LANES}
    assert lanes == min(ent["lane_table"], key=lambda r: r["ms"])["lanes"]
    best = min(ent["table"], key=lambda r: r["ms"])
    assert (best["items"], best["tiles"]) == (items, tiles)
    abi.hubbard_batch_set_config(32, 4)
