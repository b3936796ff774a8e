"""GPU parity where one step gives many servers work at once: a queue that has built up behind a split without prefill
slots meets a burst of them, the constant prompts end together, and so do the decodes. Sizes lie on both sides of a
wave's worth of admissions and jobs, of what the waves that serve take, and of the candidates that the first-come
gate ranks from one fetch of their arrival steps."""
from dataclasses import replace

import pytest

from paper_2602_02987_amd import workloads as W
from parity import assert_replication_equal, assert_stats_equal
from test_gpu_parity import B, _limits_cfg, _limits_class  # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

_ROUTE = {"solo": W.ROUTE_SOLO_FIRST, "random": W.ROUTE_RANDOM_SPLIT, "weighted": W.ROUTE_WEIGHTED_SPLIT}


def _burst(B, oracle_mod, cfg, laid_out, M, wait, what):
    sim, orc = B.Sim(cfg, max_replications=laid_out), oracle_mod.Oracle(cfg)
    for m, n in ((0, wait), (M, 1), (M, 30), (max(1, M // 2), 40), (min(cfg.N, M + 70), 40)):
        for e in (sim, orc):
            e.set_split(m)
        sim.run(n, cfg.replications)
        orc.run(n)
        for r in range(cfg.replications):
            assert_replication_equal(sim, orc, r, what=f"{what} M={m} after {orc.steps_done()} steps")
    assert_stats_equal(sim.stats(), orc.stats())
    t = orc.stats()["tally"]
    assert t[:, 2].sum() > M and t[:, 6:8].sum() > 0   # every slot was given away, decodes have ended


# replications the handle is laid out for: one wave a workgroup, or several
@pytest.mark.parametrize("laid_out", [4, 5000])
@pytest.mark.parametrize("theta", [0.0, 0.3])
@pytest.mark.parametrize("K,most", [(2, 32), (3, 16), (4, 16), (7, 8), (8, 8)])
def test_first_come_candidates(B, oracle_mod, K, most, theta, laid_out):
    cls = [_limits_class(lam=3.0 * (k + 1) / (K * (K + 1) / 2), in_p0=100.0 + 50.0 * (k % 2), out_p0=4.0 + k, theta=theta) for k in range(K)]
    for M in (1, most - 1, most, most + 1):   # `most`: candidates a class that one fetch covers
        cfg = _limits_cfg("first-come", cls, N=260, M=0, B=6, steps=0, x_star=[0.1] * K, queue_cap=2048, dbuf_cap=512)
        cfg = replace(cfg, gate_mode=W.GATE_FCFS, qp_star=[0.0] * K)
        _burst(B, oracle_mod, cfg, laid_out, M, 60, f"K={K} theta={theta}")


# servers, servers a replication of which holds prefills at once, batch cap, replications laid out for
@pytest.mark.parametrize("route", list(_ROUTE))
@pytest.mark.parametrize("theta", [0.0, 0.3])
@pytest.mark.parametrize("N,M,cap,laid_out", [
    (300, 64, 4, 3000),       # one or two waves
    (1100, 65, 5, 600),       # eight waves
    (1100, 129, 5, 600),
    (1100, 256, 5, 4),        # sixteen waves: four for the admissions, four for the jobs
    (1100, 257, 5, 4),        # more than a pass admits
    (700, 600, 2, 4),         # a solo group that is full at once: jobs for the mixed servers
    (5200, 300, 3, 4),        # sixteen waves, more than 64 words
])
def test_bursts(B, oracle_mod, N, M, cap, laid_out, theta, route):
    K = 3
    cls = [_limits_class(lam=4.0 * (k + 1) / 6.0, in_p0=120.0, out_p0=3.0 + k, theta=theta) for k in range(K)]
    cfg = _limits_cfg("bursts", cls, N=N, M=0, B=cap, steps=0, x_star=[0.3, 0.2, 0.1], queue_cap=8192, dbuf_cap=4096)
    cfg = replace(cfg, route_mode=_ROUTE[route], qp_star=[0.01 * k for k in range(K)])
    if route != "solo":
        cfg = replace(cfg, p_solo=[0.8, 0.3, 0.6])
    if route == "weighted":
        cfg = replace(cfg, w_solo=[0.5, 0.3, 0.2], w_mixed=[0.1, 0.0, 0.9])
    _burst(B, oracle_mod, cfg, laid_out, M, 20 + 30 * M // N, f"{route} theta={theta} N={N}")
