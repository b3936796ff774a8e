"""The statistics' totals over replications equal the sum of the replications' own tallies and histograms, for numbers of
replications on both sides of every step of the summation: one wave, several waves with a remainder, all sixteen waves with
whole rounds and with rows left over."""
import numpy as np
import pytest

from paper_2602_02987_amd import workloads as W
from test_gpu_parity import B  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _quantile_bin(hist, percent):
    """The bin that holds the entry of rank ceil(total * percent / 100)."""
    need = (int(hist.sum()) * percent + 99) // 100
    return int(np.searchsorted(np.cumsum(hist), need))


@pytest.mark.parametrize("reps", [1, 7, 8, 9, 17, 120, 127, 128, 129, 300])
def test_totals_over_replications(B, reps):
    cfg = W.config(1, replications=reps)
    sim = B.Sim(cfg)
    sim.run(3000)
    st = sim.stats()
    parts = [sim.tallies(r) for r in range(reps)]
    assert np.array_equal(st["tally"][:cfg.K], np.sum([p[0] for p in parts], axis=0, dtype=np.uint64))
    assert np.array_equal(st["glob"][:5], np.sum([p[1][:5] for p in parts], axis=0, dtype=np.uint64))
    tbt = np.sum([sim.hist(r, 2) for r in range(reps)], axis=0, dtype=np.uint64)
    assert (tbt.sum(axis=1) > 100).all()
    for k in range(cfg.K):   # a percentile is reported as the lower edge of its bin (16 bins per octave, exact below 16)
        for percent, name in ((50, "tbt_p50"), (95, "tbt_p95"), (99, "tbt_p99")):
            b = _quantile_bin(tbt[k], percent)
            low = b if b < 16 else (16 + b % 16) << (b // 16 - 1)
            assert abs(st[name][k] - low * 1e-9) < 1e-15, (k, name, b, st[name][k])
