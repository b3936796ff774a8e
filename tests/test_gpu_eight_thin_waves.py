"""Eight waves with less than two blocks of servers each in the kernel form for four waves per SIMD, which variants with
deadline rings take where two such workgroups share a compute unit: against the oracle, at the smallest and largest
numbers of servers, with ragged last blocks."""
from dataclasses import replace

import pytest

from paper_2602_02987_amd import workloads as W
from test_gpu_parity import B, run_both  # noqa: F401  (B is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("route", ["solo_first", "random", "weighted", "immediate"])
@pytest.mark.parametrize("N,reps", [(449, 257), (512, 512), (700, 300), (960, 512)])
def test_eight_thin_waves(B, oracle_mod, N, reps, route):
    cfg = W.config(3, N=N, replications=reps)
    if route == "random":
        cfg = W.with_random_split(cfg)
    elif route == "weighted":
        cfg = W.with_weighted_split(cfg)
    elif route == "immediate":
        cfg = replace(cfg, route_mode=W.ROUTE_IMMEDIATE, M=N)
    for c in cfg.classes:
        c.theta = 0.1
    assert B.sim_launch_plan(cfg)[0::2] == (512, 4)
    run_both(B, oracle_mod, cfg, 300, oracle_reps=[0, reps - 1], checkpoints=2)
