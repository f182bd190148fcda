"""The LDS of a serving launch: the step's and a copy of the mean sequence, or
the step's alone where both exceed the limit (CPU only)."""
import pytest

import fake_hip


def lds(K, T, M):
    import paper_2209_12842_amd as R
    L, mem = R.lib(), fake_hip.memory
    p, obs, x0 = fake_hip.world(K=K, T=T, M=M, n_obs=10)
    h = fake_hip.handle(p, obs)
    V = mem(8 * T)
    fake_hip.fake.fake_reset(-1)
    R.check(L.mppi_step(h, x0, V, 0, None, None))
    R.check(L.mppi_serve_start(h, V, 100, None))
    got = [(k, n) for k, _, _, n in fake_hip.launches()]
    L.mppi_destroy(h)
    return got


@pytest.mark.parametrize("K,T,M,copy", [(300, 29, 1, True), (300, 30, 1, False), (2048, 50, 64, True), (40, 3300, 256, False)])
def test_copy_where_it_fits(K, T, M, copy):
    (step, n), (serve, m) = fake_hip.run("test_serve_lds_cpu", "lds(%d, %d, %d)" % (K, T, M))
    assert (step, serve) == ("k_rollout_fused", "k_serve")
    assert m == (n + 15) // 16 * 16 + (8 * T if copy else 0) <= 64 * 1024
