"""The gradient's rollouts run with their steps side by side only for horizons
and row counts where that is the shorter form: its grid for short horizons is
that of one lane per row (CPU only)."""
import pytest

import fake_hip


def grid(K, T, M):
    import paper_2209_12842_amd as R
    L, mem = R.lib(), fake_hip.memory
    p, obs, x0 = fake_hip.world(flags=R.MPPI_F_GRAD, K=K, T=T, M=M, B=2.0)
    h, V, out = fake_hip.handle(p, obs), mem(8 * T), mem(8 * T)
    fake_hip.fake.fake_reset(-1)
    R.check(L.mppi_grad(h, x0, V, 0, out, out, None))
    return [g for k, g, _, _ in fake_hip.launches() if k == "k_grad_rollouts"]


# rows K (1 + M): lanes in workgroups of 256, or 8 rows a workgroup up to the line
@pytest.mark.parametrize("K,T,M,want", [(1000, 1, 15, 63), (1000, 7, 15, 63), (20, 8, 15, 40), (1000, 8, 15, 1024),
                                        (1000, 24, 15, 1024), (1000, 25, 15, 2000), (4096, 50, 15, 2048),
                                        (100000, 50, 15, 6250), (100000, 5, 15, 6250)])
def test_grid_follows_the_horizon(K, T, M, want):
    assert fake_hip.run("test_grad_route_cpu", "grid(%d, %d, %d)" % (K, T, M)) == [want]
