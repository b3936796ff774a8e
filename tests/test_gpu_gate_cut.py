"""GPU parity of the occupancy gate where its short cuts decide: queues much longer than a step's admissions (the classes are cut
before the ranking), targets whose estimate is exact, lies next to a whole number (equal targets, ties down to the class
index), is not used (terms of a million and more), or nothing may be cut (a milliard and more), and a burst of idle slots after
a move of the split."""
from dataclasses import replace

import pytest

from paper_2602_02987_amd import workloads as W
from parity import assert_replication_equal, assert_stats_equal
from test_gpu_parity import B, _limits_cfg, _limits_class  # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

_TARGETS = {
    "distinct": lambda k: 0.013 + 0.0171 * k,
    "equal": lambda k: 0.0625,
    "some_equal": lambda k: (0.05, 0.025, 0.1)[k % 3],
    "one_zero": lambda k: 0.0 if k == 1 else 0.03 + 0.011 * k,
    "huge": lambda k: 1e6 * (1 + k),
    "huge_and_tiny": lambda k: 1e9 if k % 2 else 1e-9,
    # a request more or less is lost in the rounding of these
    "beyond_rounding": lambda k: (0.03, 1e16, 1e300)[k % 3] * (1 + 0.1 * k),
    "all_beyond": lambda k: 1e200 * (1 + k),
    "tiny": lambda k: 1e-12 * (1 + 0.37 * k),
}


@pytest.mark.parametrize("targets", list(_TARGETS))
# servers, replications the handle is laid out for, waves a workgroup then has (from four on a lane takes a candidate and goes
# through the classes, below that the classes have a lane each), classes, patience rate
@pytest.mark.parametrize("N,laid_out,waves,K,theta", [
    (2000, 2500, 2, 8, 0.0), (2000, 2500, 2, 3, 0.0), (600, 8, 8, 6, 0.2), (700, 8, 8, 2, 0.0),
    (1000, 2100, 1, 5, 0.0), (1500, 600, 4, 8, 0.0), (1500, 600, 4, 3, 0.2), (700, 8, 8, 8, 0.0), (2000, 4, 16, 8, 0.2), (2000, 4, 16, 7, 0.0),
])
def test_long_queues(B, oracle_mod, targets, N, laid_out, waves, K, theta):
    # more arrivals than the mixed group can take; constant prompts, so that many slots fall free together
    cls = [_limits_class(lam=3.0 * (k + 1) / (K * (K + 1) / 2), in_p0=250.0 + 250.0 * (k % 2), out_p0=3.0, theta=theta) for k in range(K)]
    cfg = _limits_cfg("cut", cls, N=N, M=N // 60, B=6, steps=0, x_star=[_TARGETS[targets](k) for k in range(K)],
                      queue_cap=4096, dbuf_cap=2048)
    cfg = replace(cfg, qp_star=[0.01 * (k % 3) for k in range(K)])
    assert B.sim_launch_plan(cfg, laid_out)[0] == 64 * waves
    sim, orc = B.Sim(cfg, max_replications=laid_out), oracle_mod.Oracle(cfg)
    for M, n in ((N // 60, 120), (N // 5, 1), (N // 5, 40), (N // 20, 60)):
        for e in (sim, orc):
            e.set_split(M)
        sim.run(n, cfg.replications)
        orc.run(n)
        for r in range(cfg.replications):
            assert_replication_equal(sim, orc, r, what=f"{targets} N={N} K={K} after {orc.steps_done()} steps")
    assert_stats_equal(sim.stats(), orc.stats())
    t = orc.stats()["tally"]
    assert t[:, 2].sum() < 0.9 * t[:, 0].sum()   # queues have grown
