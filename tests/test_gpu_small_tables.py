"""One- and two-wave workgroups, whose tables are small (64 admissions and 64 staged requests a pass, 96 queued servers a
wave) and whose ranks of completions share space with those of the routing levels: against the oracle with a few and with
many words, several gate passes and several levels a step."""
from dataclasses import replace

import pytest

from paper_2602_02987_amd import workloads as W
from parity import assert_replication_equal, assert_stats_equal
from test_gpu_parity import B, _limits_cfg, _limits_class  # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

_GATE = {"occupancy": W.GATE_OCCUPANCY, "fcfs": W.GATE_FCFS}
_ROUTE = {"solo": W.ROUTE_SOLO_FIRST, "random": W.ROUTE_RANDOM_SPLIT, "weighted": W.ROUTE_WEIGHTED_SPLIT, "immediate": W.ROUTE_IMMEDIATE}


# servers, replications the handle is laid out for, waves a workgroup then has, classes, gate, router, patience rate
@pytest.mark.parametrize("N,laid_out,waves,K,gate,route,theta", [
    (33, 4, 1, 8, "occupancy", "random", 0.0),
    (64, 4, 1, 3, "occupancy", "weighted", 0.3),
    (1000, 4096, 1, 8, "occupancy", "solo", 0.0),
    (1000, 4096, 1, 5, "fcfs", "solo", 0.3),
    (1000, 4096, 1, 8, "occupancy", "random", 0.0),
    (1000, 4096, 2, 8, "occupancy", "weighted", 0.3),
    (1100, 2048, 1, 2, "fcfs", "immediate", 0.0),
    (2500, 700, 2, 8, "occupancy", "weighted", 0.3),
    (150, 600, 2, 8, "occupancy", "solo", 0.0),
    (3700, 700, 2, 8, "occupancy", "solo", 0.0),
    (3500, 700, 2, 8, "occupancy", "random", 0.3),
])
def test_small_tables(B, oracle_mod, N, laid_out, waves, K, gate, route, theta):
    cls = [_limits_class(lam=4.0 * (k + 1) / (K * (K + 1) / 2), in_p0=60.0 + 40.0 * k, out_p0=3.0 + 2.0 * k, theta=theta)
           for k in range(K)]
    cfg = _limits_cfg("small tables", cls, N=N, M=max(1, 3 * N // 5), B=6, steps=0, queue_cap=1024, dbuf_cap=1024,
                      x_star=[0.05 + 0.1 * (k % 3) / K for k in range(K)])
    cfg = replace(cfg, gate_mode=_GATE[gate], route_mode=_ROUTE[route], p_solo=[0.3 + 0.4 * (k % 2) for k in range(K)],
                  w_solo=[(1.0 + k) / K for k in range(K)], w_mixed=[0.5 + 0.5 * (k % 2) for k in range(K)])
    assert B.sim_launch_plan(cfg, laid_out)[0] == 64 * waves
    sim, orc = B.Sim(cfg, max_replications=laid_out), oracle_mod.Oracle(cfg)
    for n in (30, 1, 200):
        sim.run(n, cfg.replications)
        orc.run(n)
        for r in range(cfg.replications):
            assert_replication_equal(sim, orc, r, what=f"N={N} K={K} {gate} {route} after {orc.steps_done()} steps")
    assert_stats_equal(sim.stats(), orc.stats())
    assert orc.stats()["tally"][:, 6:8].sum() > N // 8   # decodes have ended
