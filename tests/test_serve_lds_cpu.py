"""The LDS of a serving launch: with a copy of the mean sequence where a million
controls read it or the nominal workgroups are packed, and both fit the limit
(CPU only)."""
import pytest

import fake_hip


def lds(K, T, M):
    import paper_2209_12842_amd as R
    L, mem = R.lib(), fake_hip.memory
    p, obs, x0 = fake_hip.world(K=K, T=T, M=M, n_obs=10)
    h = fake_hip.handle(p, obs)
    V = mem(8 * T)
    fake_hip.fake.fake_reset(-1)
    R.check(L.mppi_serve_start(h, V, 100, None))
    (got,) = [n for _, _, _, n in fake_hip.launches()]
    L.mppi_destroy(h)
    return got


# step: controls and costs of the workgroup's samples or the nominal buffers, and one group of obstacles
@pytest.mark.parametrize("K,T,M,step,copy", [
    (2048, 50, 64, 2 * 4608 + 1024, False),
    (15625, 64, 8, 4 * (2 * 32 * 64 + 2 * 256 + 32) + 1024, True),       # a million controls
    (15624, 64, 8, 4 * (2 * 32 * 64 + 2 * 256 + 32) + 1024, False),
    (3900, 50, 64, 4 * 4608 + 1024, True),                               # packed
    (34000, 30, 1, 64 * 1024, False),                                    # no room
])
def test_copy_where_it_pays_and_fits(K, T, M, step, copy):
    assert fake_hip.run("test_serve_lds_cpu", "lds(%d, %d, %d)" % (K, T, M)) == step + (8 * T if copy else 0)
