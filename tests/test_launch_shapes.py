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


# The bytes of the tables that the choice of shapes and the limit on the number of servers were measured with: one- and
# two-wave workgroups of many classes or many servers among them, where a few bytes more cost half the waves or a round.
@pytest.mark.parametrize("K,N,M,theta,route,chunk_cost,replications,shape", [
    (1, 1, 0, 0.0, SOLO, False, 1, (64, 5728, 2)),
    (8, 1, 0, 0.0, SOLO, False, 4096, (64, 5784, 4)),
    (7, 31, 31, 0.0, WEIGHTED, True, 4096, (64, 10120, 4)),  # sixteen workgroups to a compute unit up to 10240 bytes
    (8, 33, 0, 0.1, SOLO, True, 4096, (64, 10008, 4)),
    (6, 100, 50, 0.1, SOLO, True, 4096, (64, 9872, 4)),
    (8, 64, 64, 0.1, WEIGHTED, True, 2048, (64, 11000, 2)),
    (4, 257, 257, 0.1, SOLO, False, 4096, (64, 10208, 4)),
    (8, 383, 0, 0.0, SOLO, False, 4096, (64, 10040, 4)),
    (1, 769, 0, 0.0, SOLO, False, 8192, (64, 14464, 4)),
    (8, 1000, 250, 0.0, WEIGHTED, False, 4096, (64, 20208, 2)),  # eight to a compute unit up to 20480 bytes
    (2, 1024, 1024, 0.0, WEIGHTED, False, 2048, (64, 20408, 2)),
    (1, 1500, 0, 0.1, RANDOM, True, 8192, (64, 23256, 2)),
    (8, 2560, 640, 0.0, SOLO, True, 2048, (128, 38952, 2)),
    (8, 2560, 2560, 0.0, SOLO, False, 1024, (128, 40936, 2)),  # four to a compute unit up to 40960 bytes
    (8, 3001, 0, 0.0, RANDOM, False, 1024, (128, 40888, 2)),
    (8, 4000, 0, 0.0, SOLO, True, 700, (128, 54088, 2)),  # three up to 54613 bytes
    (4, 4000, 0, 0.1, SOLO, True, 700, (128, 54152, 2)),
    (8, 5120, 5120, 0.0, WEIGHTED, True, 8192, (1024, 115496, 4)),
    (3, 1025, 256, 0.0, SOLO, True, 1024, (256, 25384, 4)),
    (8, 5120, 0, 0.1, SOLO, True, 512, (256, 80744, 2)),
    (5, 5121, 1280, 0.0, SOLO, True, 512, (1024, 96824, 4)),
    (8, 10240, 5120, 0.0, IMMEDIATE, True, 256, (1024, 156392, 4)),
    (8, 10241, 5120, 0.0, IMMEDIATE, True, 256, (1024, 159240, 4)),
    (8, 12288, 0, 0.0, SOLO, False, 1, None),
])
def test_recorded_shapes(K, N, M, theta, route, chunk_cost, replications, shape):
    """Threads, bytes on chip and waves a SIMD; None: refused."""
    from paper_2602_02987_amd import binding as B
    cfg = _cfg(K, N, M, theta, route, chunk_cost)
    if shape is None:
        with pytest.raises(B.SimError) as e:
            B.sim_launch_plan(cfg, replications)
        assert e.value.code == -1
    else:
        assert tuple(B.sim_launch_plan(cfg, replications)) == shape


# Two to four blocks of servers: more waves where router, patience or same-slot decode have roles of their own for them. One block, five
# and more keep fewer waves than twice the blocks.
@pytest.mark.parametrize("N,theta,route,replications,shape", [
    (64, 0.0, IMMEDIATE, 4, (64, 2)), (65, 0.0, IMMEDIATE, 4, (512, 2)), (128, 0.0, RANDOM, 256, (512, 2)), (256, 0.1, SOLO, 16, (512, 2)),
    (100, 0.0, WEIGHTED, 300, (512, 4)), (190, 0.0, IMMEDIATE, 512, (512, 4)), (190, 0.0, RANDOM, 513, (128, 2)), (100, 0.1, SOLO, 1000, (256, 4)),
    (100, 0.0, IMMEDIATE, 1000, (128, 2)), (65, 0.0, SOLO, 4, (256, 2)), (256, 0.0, SOLO, 256, (256, 2)), (190, 0.0, SOLO, 512, (256, 2)),
    (128, 0.0, SOLO, 2000, (128, 4)), (128, 0.1, RANDOM, 4000, (64, 4)), (257, 0.0, SOLO, 4, (512, 2)), (320, 0.0, IMMEDIATE, 512, (512, 4)),
    (320, 0.0, RANDOM, 512, (256, 2)), (900, 0.0, IMMEDIATE, 1000, (256, 4)),
])
def test_few_blocks_and_many_roles(N, theta, route, replications, shape):
    from paper_2602_02987_amd import binding as B
    M = N if route == IMMEDIATE else N // 4
    assert tuple(B.sim_launch_plan(_cfg(4, N, M, theta, route), replications))[0::2] == shape
