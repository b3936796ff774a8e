"""GPU parity where a server's next event is easiest to get wrong: events exactly on a step's boundary, several decodes
that end in one iteration, prompts of whole and of almost whole chunks, one-token outputs, iterations so long that the
first end of a decode lies beyond the furthest event a clock may hold (2^38 ns), and runs cut at every length."""
import pytest

from paper_2602_02987_amd import workloads as W
from parity import assert_replication_equal, assert_stats_equal
from test_gpu_parity import B, _limits_cfg, _limits_class  # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu


def _case(name):
    kw = dict(N=70, M=20, B=8, steps=0, x_star=[0.2, 0.2])
    const = lambda lam, p, d: _limits_class(lam=lam, in_p0=float(p), out_law=W.LAW_CONST, out_p0=float(d))  # noqa: E731
    if name == "on-the-boundary":          # every iteration lasts exactly one step
        cfg = _limits_cfg(name, [const(2.0, 512, 9), const(1.0, 300, 40)], **kw)
        cfg.c_pre = cfg.c_dec = 0.0
    elif name == "ends-together":          # full rows of equal lengths: many decodes of a row end in one iteration
        kw.update(N=10, M=5, B=128, x_star=[0.5, 0.5])
        cfg = _limits_cfg(name, [const(3.0, 16, 900), const(2.0, 16, 900)], **kw)
        cfg.c_pre = cfg.c_dec = 0.0
    elif name == "whole-chunks":           # 1, 255, 256, 257, 512, 513 prompt tokens at 256 a chunk; one output token
        p = (1, 255, 256, 257, 512, 513)
        kw.update(x_star=[0.05] * 6)
        cfg = _limits_cfg(name, [const(0.7, v, 1 + (i % 2)) for i, v in enumerate(p)], **kw)
    elif name == "far-events":             # 144 iterations of 1.9 s are as far ahead as an event may be set
        cfg = _limits_cfg(name, [const(0.008, 3, 400), const(0.008, 700, 150)], **kw)
        cfg.c0, cfg.c_pre, cfg.c_dec, cfg.dt = 1.9, 1e-5, 1e-4, 1.9
    return cfg


@pytest.mark.parametrize("name,runs", [("on-the-boundary", (1, 1, 2, 3, 97, 900)), ("ends-together", (500, 1, 950, 1, 1200)),
                                       ("whole-chunks", (1, 1, 1, 400, 900)), ("far-events", (100, 1, 60, 600, 900))])
def test_events(B, oracle_mod, name, runs):
    cfg = _case(name)
    sim, orc = B.Sim(cfg), oracle_mod.Oracle(cfg)
    for n in runs:
        sim.run(n)
        orc.run(n)
        for r in range(cfg.replications):
            assert_replication_equal(sim, orc, r, what=f"{name} after {orc.steps_done()} steps")
    assert_stats_equal(sim.stats(), orc.stats())
    assert (orc.stats()["tally"][:, 6:8].sum()) > 100   # decodes have ended
