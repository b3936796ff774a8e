"""GPU parity where one step gives many servers work at once: a queue that has built up behind a split without prefill
slots meets a burst of them, the constant prompts end together, so that as many requests move on to decode servers in the
step in which the slots are given away again. Sizes lie on both sides of a wave's worth of admissions and jobs, of what the
waves that serve take, and of the candidates that the first-come gate ranks from one fetch of their arrival steps."""
from dataclasses import replace

import pytest

from paper_2602_02987_amd import workloads as W
from paper_2602_02987_amd.binding import TALLY
from parity import assert_replication_equal, assert_stats_equal
from test_gpu_parity import B, _limits_cfg, _limits_class  # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

_ROUTE = {"solo": W.ROUTE_SOLO_FIRST, "random": W.ROUTE_RANDOM_SPLIT, "weighted": W.ROUTE_WEIGHTED_SPLIT}
_U_P, _U_DM, _U_DS, _S_DM, _S_DS = (TALLY.index(n) for n in ("U_P", "U_DM", "U_DS", "S_DM", "S_DS"))


def _steps(orc, n, reps):
    """Admissions and placements of each of the next n steps, in every replication."""
    def totals():
        t = [orc.tallies(r)[0].astype(int) for r in range(reps)]
        return [(x[:, _U_P].sum(), x[:, [_U_DM, _U_DS]].sum()) for x in t]
    out, before = [], totals()
    for _ in range(n):
        orc.run(1)
        after = totals()
        out.append([(a[0] - b[0], a[1] - b[1]) for a, b in zip(after, before)])
        before = after
    return out


def _burst(B, oracle_mod, cfg, laid_out, waves, M, wait, jobs, what):
    """`jobs`: requests that move on to decode servers in the step in which the first prompts end."""
    assert B.sim_launch_plan(cfg, laid_out)[0] == 64 * waves
    sim, orc = B.Sim(cfg, max_replications=laid_out), oracle_mod.Oracle(cfg)
    for m, n in ((0, wait), (M, 1), (M, 30), (max(1, M // 2), 40), (min(cfg.N, M + 70), 40)):
        for e in (sim, orc):
            e.set_split(m)
        sim.run(n, cfg.replications)
        if n == 1:     # every slot is given away in one step
            assert _steps(orc, n, cfg.replications) == [[(M, 0)] * cfg.replications]
        elif n == 30:  # ... and, two steps on, again in the step that places the requests whose prompts have ended
            assert _steps(orc, n, cfg.replications)[1] == [(M, jobs)] * cfg.replications
        else:
            orc.run(n, cfg.replications)
        for r in range(cfg.replications):
            assert_replication_equal(sim, orc, r, what=f"{what} M={m} after {orc.steps_done()} steps")
    assert_stats_equal(sim.stats(), orc.stats())
    assert orc.stats()["tally"][:, [_S_DM, _S_DS]].sum() > 0   # decodes have ended


# replications the handle is laid out for, waves a workgroup then has
@pytest.mark.parametrize("laid_out,waves", [(4, 8), (700, 2), (5000, 1)])
@pytest.mark.parametrize("theta", [0.0, 0.3])
@pytest.mark.parametrize("K,most", [(2, 32), (3, 16), (4, 16), (7, 8), (8, 8)])
def test_first_come_candidates(B, oracle_mod, K, most, theta, laid_out, waves):
    cls = [_limits_class(lam=3.0 * (k + 1) / (K * (K + 1) / 2), in_p0=100.0, out_p0=4.0 + k, theta=theta) for k in range(K)]
    for M in (1, most - 1, most, most + 1):   # `most`: candidates a class that one fetch covers
        cfg = _limits_cfg("first-come", cls, N=260, M=0, B=6, steps=0, x_star=[0.1] * K, queue_cap=2048, dbuf_cap=512)
        cfg = replace(cfg, gate_mode=W.GATE_FCFS, qp_star=[0.0] * K)
        _burst(B, oracle_mod, cfg, laid_out, waves, M, 60, M, f"K={K} theta={theta}")


# servers, of them with a prefill slot during the burst, batch cap, replications the handle is laid out for, waves a workgroup
# then has, requests that move on together. Admissions and jobs have waves of their own (64 servers each) where these are no
# more than half of the workgroup's and no job goes to the mixed group.
@pytest.mark.parametrize("route", list(_ROUTE))
@pytest.mark.parametrize("theta", [0.0, 0.3])
@pytest.mark.parametrize("N,M,cap,laid_out,waves,jobs", [
    (300, 64, 4, 4100, 1, 64),      # a pass admits and stages 64 here
    (300, 65, 4, 4100, 1, 65),
    (300, 129, 4, 700, 2, 129),     # both waves serve more than once
    (1100, 64, 5, 600, 4, 64),      # one wave for the admissions, one for the jobs
    (1100, 65, 5, 600, 4, 65),      # all four together
    (1100, 128, 5, 300, 8, 128),    # two and two
    (1100, 129, 5, 300, 8, 129),
    (2000, 256, 5, 4, 16, 256),     # four and four
    (2000, 257, 5, 4, 16, 257),     # more than a pass admits
    (5200, 300, 3, 4, 16, 300),     # sixteen waves, more than 64 words
])
def test_bursts(B, oracle_mod, N, M, cap, laid_out, waves, jobs, theta, route):
    _burst(B, oracle_mod, _bursts_cfg(N, cap, theta, route), laid_out, waves, M, 20 + 30 * M // N, jobs, f"{route} theta={theta} N={N}")


# a solo group of 100 servers with two slots each, full at once: jobs for the mixed servers, which keep a slot for a prefill
@pytest.mark.parametrize("theta", [0.0, 0.3])
@pytest.mark.parametrize("laid_out,waves", [(4, 8), (600, 4)])
def test_burst_beyond_the_solo_group(B, oracle_mod, laid_out, waves, theta):
    _burst(B, oracle_mod, _bursts_cfg(700, 2, theta, "solo"), laid_out, waves, 600, 20 + 30 * 600 // 700, 600, f"theta={theta}")


def _bursts_cfg(N, cap, theta, route):
    K = 3
    cls = [_limits_class(lam=4.0 * (k + 1) / 6.0, in_p0=120.0, out_p0=3.0 + k, theta=theta) for k in range(K)]
    cfg = _limits_cfg("bursts", cls, N=N, M=0, B=cap, steps=0, x_star=[0.3, 0.2, 0.1], queue_cap=8192, dbuf_cap=4096)
    cfg = replace(cfg, route_mode=_ROUTE[route], qp_star=[0.01 * k for k in range(K)])
    if route != "solo":
        cfg = replace(cfg, p_solo=[0.8, 0.3, 0.6])
    if route == "weighted":
        cfg = replace(cfg, w_solo=[0.5, 0.3, 0.2], w_mixed=[0.1, 0.0, 0.9])
    return cfg
