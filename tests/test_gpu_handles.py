"""GPU tests of what a handle takes and gives back: making and destroying one waits for no other work on the device, and handles
beyond the pinned blocks that the library keeps, or on blocks that others have used, read the same statistics."""
import numpy as np
import pytest

from paper_2602_02987_amd import workloads as W
from parity import assert_stats_equal
from test_gpu_parity import B  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def test_destroying_a_handle_waits_for_no_other_work(B):
    import torch
    busy, other = B.Sim(W.config(3, replications=256)), B.Sim(W.config(1))
    other.run(10)
    other.stats()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):   # work of another handle on another stream, a third of a second
        busy.run(40_000)
        end = torch.cuda.Event()
        end.record()
    assert not end.query()
    other.close()
    assert not end.query()
    side.synchronize()
    busy.close()


def test_many_handles_and_used_blocks(B, oracle_mod):
    small = W.config(1, N=8, replications=2)
    wide = W.config(4, N=64, replications=2)
    expect = {}
    for cfg in (small, wide):
        orc = oracle_mod.Oracle(cfg)
        orc.run(300)
        expect[cfg.K] = orc.stats()
    for cfg in (wide, small, wide):   # (totals of other classes than the ones that a block held before)
        sims = [B.Sim(cfg) for _ in range(40)]
        for sim in sims:
            sim.run(300)
        for sim in reversed(sims):
            assert_stats_equal(sim.stats(), expect[cfg.K])
        assert np.array_equal(sims[0].stats()["tally"], sims[-1].stats()["tally"])
        for sim in sims:
            sim.close()
