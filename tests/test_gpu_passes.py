"""GPU parity where the gate's ranking and the routing pass change form: one to eight classes (two, four or eight lanes to
a candidate), every gate, all routers, workgroups of two waves that own many words and queue more servers in a pass than
the queue holds, and of several waves with a ragged last word; and where the groups of servers end inside or on the border of
the sixteen servers that a lane of the level pass looks at."""
from dataclasses import replace

import pytest

from paper_2602_02987_amd import workloads as W
from parity import assert_replication_equal, assert_stats_equal
from test_gpu_parity import B, _limits_cfg, _limits_class  # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

_GATE = {"occupancy": W.GATE_OCCUPANCY, "priority": W.GATE_PRIORITY, "fcfs": W.GATE_FCFS}
_ROUTE = {"solo": W.ROUTE_SOLO_FIRST, "random": W.ROUTE_RANDOM_SPLIT, "weighted": W.ROUTE_WEIGHTED_SPLIT, "immediate": W.ROUTE_IMMEDIATE}


# servers, replications the handle is laid out for (many: small workgroups), classes, gate, router, patience rate
@pytest.mark.parametrize("N,laid_out,K,gate,route,theta", [
    (2500, 3000, 1, "occupancy", "solo", 0.0),
    (2500, 3000, 3, "occupancy", "solo", 0.0),
    (2500, 3000, 8, "priority", "random", 0.0),
    (1100, 8, 5, "occupancy", "random", 0.3),
    (1100, 8, 8, "fcfs", "solo", 0.0),
    (700, 300, 4, "fcfs", "solo", 0.3),
    (700, 300, 6, "priority", "weighted", 0.3),
    (449, 4, 2, "priority", "immediate", 0.0),
    (449, 4, 7, "occupancy", "weighted", 0.0),
    (65, 4, 8, "occupancy", "solo", 0.3),
])
def test_pass_shapes(B, oracle_mod, N, laid_out, K, gate, route, theta):
    # arrivals near the highest rate accepted (a request for every 25 servers and step), prompts and outputs that keep
    # most servers changing, and targets of which some are exceeded and one is zero where there are several classes
    cls = [_limits_class(lam=4.0 * (k + 1) / (K * (K + 1) / 2), in_p0=60.0 + 55.0 * k, out_p0=3.0 + 2.0 * k, theta=theta,
                         priority=float((k * 3) % 5)) for k in range(K)]
    x = [0.05 + 0.1 * (k % 3) / K for k in range(K)]
    if K > 3 and gate == "occupancy":
        x[1] = 0.0
    cfg = _limits_cfg("passes", cls, N=N, M=max(1, 3 * N // 5), B=6, steps=0, x_star=x,
                      queue_cap=2048, dbuf_cap=2048)
    over = dict(gate_mode=_GATE[gate], route_mode=_ROUTE[route], qp_star=[0.01 * k for k in range(K)])
    if route in ("random", "weighted"):
        over["p_solo"] = [0.3 + 0.4 * (k % 2) for k in range(K)]
    if route == "weighted":
        over.update(w_solo=[(1.0 + k) / K for k in range(K)], w_mixed=[0.5 + 0.5 * (k % 2) for k in range(K)])
    cfg = replace(cfg, **over)
    sim, orc = B.Sim(cfg, max_replications=laid_out), oracle_mod.Oracle(cfg)
    for n in (40, 1, 260):
        sim.run(n, cfg.replications)
        orc.run(n)
        for r in range(cfg.replications):
            assert_replication_equal(sim, orc, r, what=f"N={N} K={K} {gate} {route} after {orc.steps_done()} steps")
    assert_stats_equal(sim.stats(), orc.stats())
    assert orc.stats()["tally"][:, 6:8].sum() > N // 8   # decodes have ended


# Both groups take jobs on several levels until no slot is left. Split and end of the servers on, before and behind a border of
# sixteen servers and of a word; one wave and (N > 64) several.
@pytest.mark.parametrize("laid_out", [4, 4500])
@pytest.mark.parametrize("N,M", [(15, 7), (16, 15), (17, 16), (31, 1), (33, 17), (48, 32), (63, 31), (64, 48), (65, 33), (80, 63), (81, 64),
                                 (127, 65), (129, 79), (161, 80), (337, 161)])
def test_level_borders(B, oracle_mod, N, M, laid_out):
    cls = [_limits_class(lam=2.2, in_p0=60.0, out_p0=260.0), _limits_class(lam=1.6, in_p0=120.0, out_p0=400.0)]
    cfg = _limits_cfg("levels", cls, N=N, M=M, B=5, steps=0, x_star=[0.3, 0.3], queue_cap=4096, dbuf_cap=2048)
    sim, orc = B.Sim(cfg, max_replications=laid_out), oracle_mod.Oracle(cfg)
    for n in (60, 1, 140, 300):
        sim.run(n, cfg.replications)
        orc.run(n)
        for r in range(cfg.replications):
            assert_replication_equal(sim, orc, r, what=f"N={N} M={M} after {orc.steps_done()} steps")
    loads = orc.slots(0)["n_dec"]
    assert loads[M:].max() == 5 and loads[:M].max() == 4 and loads[M:].min() >= 3   # both groups were filled
