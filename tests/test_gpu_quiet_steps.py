"""GPU parity of small systems, where most steps bring neither an arrival nor an event and are passed over: numbers of servers
on both sides of every power of two up to the last that is searched and one beyond, arrivals that vary in time with a period
shorter than one draw ahead and longer than a run, every router and gate, requests that leave, runs that begin and end anywhere,
and a split and targets that move between runs."""
from dataclasses import replace

import pytest

from paper_2602_02987_amd import workloads as W
from parity import assert_replication_equal, assert_stats_equal
from test_gpu_parity import B, _limits_cfg, _limits_class  # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu


# servers, arrivals per step, gate, router, patience rate, modulation period
@pytest.mark.parametrize("N,per_step,gate,route,theta,period", [
    (1, 0.02, W.GATE_OCCUPANCY, W.ROUTE_SOLO_FIRST, 0.0, 0),
    (1, 0.01, W.GATE_FCFS, W.ROUTE_IMMEDIATE, 0.2, 7),
    (2, 0.03, W.GATE_FCFS, W.ROUTE_SOLO_FIRST, 0.4, 0),
    (3, 0.02, W.GATE_PRIORITY, W.ROUTE_RANDOM_SPLIT, 0.0, 5),
    (4, 0.03, W.GATE_OCCUPANCY, W.ROUTE_WEIGHTED_SPLIT, 0.2, 13),
    (5, 0.04, W.GATE_OCCUPANCY, W.ROUTE_SOLO_FIRST, 0.0, 9),
    (8, 0.07, W.GATE_OCCUPANCY, W.ROUTE_SOLO_FIRST, 0.0, 400),
    (8, 0.10, W.GATE_OCCUPANCY, W.ROUTE_RANDOM_SPLIT, 0.3, 0),
    (9, 0.10, W.GATE_OCCUPANCY, W.ROUTE_WEIGHTED_SPLIT, 0.0, 3),
    (16, 0.05, W.GATE_FCFS, W.ROUTE_IMMEDIATE, 0.0, 0),
    (17, 0.08, W.GATE_PRIORITY, W.ROUTE_WEIGHTED_SPLIT, 0.3, 100000),
    (32, 0.02, W.GATE_OCCUPANCY, W.ROUTE_SOLO_FIRST, 0.1, 11),
    (33, 0.02, W.GATE_OCCUPANCY, W.ROUTE_SOLO_FIRST, 0.0, 11),
])
def test_quiet_steps(B, oracle_mod, N, per_step, gate, route, theta, period):
    K = 1 if N == 1 else 2
    lam = per_step / (0.01 * N * K)
    cls = [_limits_class(lam=lam, in_p0=300.0 + 400.0 * k, out_p0=12.0 + 30.0 * k, theta=theta, priority=float(k)) for k in range(K)]
    cfg = _limits_cfg("quiet", cls, N=N, M=max(1, N // 3), B=4, steps=0, replications=3)
    over = dict(gate_mode=gate, route_mode=route)
    if period:
        over.update(mod_amp=0.8, mod_period=period)
    if route in (W.ROUTE_RANDOM_SPLIT, W.ROUTE_WEIGHTED_SPLIT):
        over["p_solo"] = [0.5] * K
    if route == W.ROUTE_WEIGHTED_SPLIT:
        over.update(w_solo=[0.5] * K, w_mixed=[1.0] * K)
    cfg = replace(cfg, **over)
    sim, orc = B.Sim(cfg), oracle_mod.Oracle(cfg)
    for i, n in enumerate((1, 700, 2, 63, 64, 65, 1, 2500)):
        if i in (3, 5):   # the first step after such a change may admit or place what waited
            M = max(1, N // 2) if i == 3 else max(1, N // 4)
            for e in (sim, orc):
                e.set_split(M)
                e.set_targets([0.2 + 0.1 * k for k in range(K)], [0.05] * K)
        sim.run(n)
        orc.run(n)
        for r in range(cfg.replications):
            assert_replication_equal(sim, orc, r, what=f"N={N} gate {gate} route {route} after {orc.steps_done()} steps")
    assert_stats_equal(sim.stats(), orc.stats())
    assert orc.stats()["tally"][:, 6:8].sum() > 10   # decodes have ended
