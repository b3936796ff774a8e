"""Launch shapes over sizes, class counts, patience and routers."""
import pytest

from paper_2602_02987_amd import workloads as W

SOLO, RANDOM, IMMEDIATE, WEIGHTED = (W.ROUTE_SOLO_FIRST, W.ROUTE_RANDOM_SPLIT, W.ROUTE_IMMEDIATE, W.ROUTE_WEIGHTED_SPLIT)


def _cfg(K, N, M, theta, route, chunk_cost=True):
    cls = [W.SimClass(lam=0.01, in_p0=100.0, out_p0=50.0, theta=theta) for _ in range(K)]
    return W.SimConfig(name="shape", K=K, N=N, B=64, C=256, c0=0.01, c_pre=5e-5 if chunk_cost else 0.0,
                       c_dec=2e-4 if chunk_cost else 0.0, classes=cls, M=M, x_star=[0.1] * K, qp_star=[0.0] * K,
                       route_mode=route, p_solo=[0.5] * K, w_solo=[0.5] * K, w_mixed=[0.5] * K)


# K, N, M, patience, router, replications: threads. A compute unit holds three to six waves of the small shapes here.
@pytest.mark.parametrize("K,N,M,theta,route,replications,threads", [
    (2, 4000, 1000, 0.0, SOLO, 2048, 512),        # two waves: six a compute unit in three rounds; eight: sixteen in four
    (4, 3500, 900, 0.1, SOLO, 2048, 512),
    (4, 3200, 800, 0.0, WEIGHTED, 2048, 512),
    (8, 4600, 4600, 0.0, IMMEDIATE, 2048, 512),
    (8, 3200, 800, 0.1, SOLO, 700, 128),          # six waves in one round stay
    (2, 1000, 250, 0.0, SOLO, 2048, 128),         # two waves a SIMD and more: the rounds alone
    (4, 2048, 512, 0.0, SOLO, 256, 1024),
])
def test_a_round_with_few_waves_counts_more(K, N, M, theta, route, replications, threads):
    from paper_2602_02987_amd import binding as B
    assert B.sim_launch_plan(_cfg(K, N, M, theta, route), replications)[0] == threads
