"""GPU parity where a step's last segment overlaps with the next step's events (workgroups of eight and sixteen waves): the servers
that are given work belong to the waves that serve them, and those whose event comes in the next step already are worked off by
them. Iterations are a little longer than a step, so that work placed in the middle of one joins in the step that follows; steps
serve a few servers up to more than 64 of each group; levels of which all, some or one member gets a job; impatient requests of
whom many are served in the last step they wait in."""
from dataclasses import replace

import pytest

from paper_2602_02987_amd import workloads as W
from parity import assert_replication_equal, assert_stats_equal
from test_gpu_parity import B, _limits_cfg, _limits_class  # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu

_POLICY = {"solo": (W.ROUTE_SOLO_FIRST, W.GATE_OCCUPANCY), "random": (W.ROUTE_RANDOM_SPLIT, W.GATE_PRIORITY),
           "weighted": (W.ROUTE_WEIGHTED_SPLIT, W.GATE_OCCUPANCY), "immediate": (W.ROUTE_IMMEDIATE, W.GATE_FCFS)}


def _overlap_cfg(N, M, lam, cap, prompt, theta, policy, **kw):
    K = 2
    cls = [_limits_class(lam=lam * w, in_p0=float(prompt), out_p0=2.0 + k, theta=theta) for k, w in enumerate((0.6, 0.4))]
    cfg = _limits_cfg("overlap", cls, N=N, M=M, B=cap, steps=0, x_star=[0.3, 0.2], queue_cap=8192, dbuf_cap=4096, **kw)
    route, gate = _POLICY[policy]
    # iterations of 10 to 11.5 ms, steps of 9.3 ms
    cfg = replace(cfg, dt=0.0093, c_pre=4e-6, c_dec=1e-4, route_mode=route, gate_mode=gate, p_solo=[0.7, 0.4], w_solo=[0.6, 0.4],
                  w_mixed=[0.2, 0.8])
    return replace(cfg, M=N) if policy == "immediate" else cfg


# servers, of them mixed, requests per server and second, batch cap, prompt tokens, waves a workgroup has
@pytest.mark.parametrize("policy", list(_POLICY))
@pytest.mark.parametrize("theta", [0.0, 40.0])
@pytest.mark.parametrize("N,M,lam,cap,prompt,waves", [
    (320, 100, 1.0, 4, 100, 8),      # five words, one or two servers a step
    (513, 65, 4.6, 3, 100, 8),       # the solo group begins and the system ends behind a whole word
    (1025, 600, 4.6, 2, 300, 8),     # jobs for the mixed group, prompts of two iterations
    (2050, 64, 0.5, 8, 100, 16),     # a word of mixed servers, few servers a step
    (2050, 1300, 4.6, 3, 100, 16),   # about a hundred admissions and jobs a step
    (5121, 3000, 4.6, 3, 100, 16),   # more than 64 words, more than 64 of each group a step
    (65, 30, 4.6, 3, 100, 8),        # two to four words, more waves than words
    (192, 100, 4.6, 3, 100, 8),
    (201, 64, 0.8, 4, 300, 8),
    (8705, 2100, 0.8, 3, 100, 16),   # twelve of sixteen waves look at the clocks, the last pair of words has one server
])
def test_served_servers_belong_to_those_that_serve(B, oracle_mod, N, M, lam, cap, prompt, waves, theta, policy):
    cfg = _overlap_cfg(N, M, lam, cap, prompt, theta, policy)
    if N <= 256 and policy == "solo" and not theta:   # (no overlap: four waves)
        waves = 4
    assert B.sim_launch_plan(cfg, cfg.replications)[0] == 64 * waves
    sim, orc = B.Sim(cfg), oracle_mod.Oracle(cfg)
    for n in (1, 2, 60, 61):   # (launches that end where others would have gone on)
        sim.run(n)
        orc.run(n)
        for r in range(cfg.replications):
            assert_replication_equal(sim, orc, r, what=f"{policy} theta={theta} N={N} after {orc.steps_done()} steps")
    assert_stats_equal(sim.stats(), orc.stats())


# Eight waves with more than 2560 servers: four of them draw beside the events, with more than 4096 three (with two buffers none, whatever
# the size). A handle laid out for 300 replications has them; 300 at once take the form of four waves a SIMD, two that of two.
@pytest.mark.parametrize("policy", list(_POLICY))
@pytest.mark.parametrize("theta", [0.0, 40.0])
@pytest.mark.parametrize("replications", [2, 300])
@pytest.mark.parametrize("N,M,lam,cap,prompt", [
    (2561, 900, 4.6, 3, 100),     # 41 words, about a hundred admissions and jobs a step
    (3000, 2900, 4.6, 2, 300),    # jobs for the mixed group, prompts of two iterations
    (4096, 64, 0.5, 8, 100),      # the last with four waves at the events, a word of mixed servers, few servers a step
    (4097, 1300, 4.6, 3, 100),    # a server in the last of 65 words
    (4600, 3000, 4.6, 3, 100),    # more than 64 of each group a step
])
def test_eight_waves_with_many_words(B, oracle_mod, N, M, lam, cap, prompt, replications, theta, policy):
    cfg = _overlap_cfg(N, M, lam, cap, prompt, theta, policy, replications=replications)
    assert B.sim_launch_plan(cfg, 300)[0] == 512 and B.sim_launch_plan(cfg, 300)[2] == 4
    sim, orc = B.Sim(cfg, max_replications=300), oracle_mod.Oracle(cfg)
    checked = [0, replications - 1]
    orc.select(checked)
    for n in (1, 2, 60, 61):
        sim.run(n)
        orc.run(n)
        for r in checked:
            assert_replication_equal(sim, orc, r, what=f"{policy} theta={theta} N={N} after {orc.steps_done()} steps")
    if replications == 2:
        assert_stats_equal(sim.stats(), orc.stats())


# The layout for more than 160 words (same-slot decode keeps a solo group here: with a prefill slot on every server it does not fit).
@pytest.mark.parametrize("policy", list(_POLICY))
@pytest.mark.parametrize("theta", [0.0, 40.0])
def test_sixteen_waves_with_the_most_words(B, oracle_mod, theta, policy):
    cfg = replace(_overlap_cfg(10305, 2100, 0.8, 3, 100, theta, policy), M=2100)
    assert B.sim_launch_plan(cfg, cfg.replications)[0] == 1024
    sim, orc = B.Sim(cfg), oracle_mod.Oracle(cfg)
    for n in (1, 2, 60, 61):
        sim.run(n)
        orc.run(n)
        for r in range(cfg.replications):
            assert_replication_equal(sim, orc, r, what=f"{policy} theta={theta} after {orc.steps_done()} steps")
    assert_stats_equal(sim.stats(), orc.stats())
