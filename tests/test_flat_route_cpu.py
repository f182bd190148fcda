"""Which step sizes take the flattened layout (CPU only)."""
import ctypes

import pytest

import fake_hip
from flat_cases import FLAT, IMPULSE, PER_SAMPLE


def kernels(kw, noalloc):
    import paper_2209_12842_amd as R
    L, mem = R.lib(), fake_hip.memory
    p, obs, x0 = fake_hip.world(**kw)
    h, V = fake_hip.handle(p, obs), mem(8 * p.T)
    fake_hip.fake.fake_reset(-1)
    if noalloc:
        R.check(L.mppi_step_noalloc(ctypes.byref(p), obs, x0, V, 0, None, None))
    else:
        R.check(L.mppi_step(h, x0, V, 0, None, None))
    return [k for k, *_ in fake_hip.launches()]


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("kw,flat", [(kw, True) for kw in FLAT] + [(kw, False) for kw in PER_SAMPLE])
def test_layout(kw, flat, noalloc):
    got = fake_hip.run("test_flat_route_cpu", "kernels(%r, %r)" % (kw, noalloc))
    assert any(k.startswith("k_cvar") for k in got) == flat


@pytest.mark.parametrize("K,T,M,n_obs", list(IMPULSE))
def test_impulses_on_the_callers_memory(K, T, M, n_obs):
    kw = dict(K=K, T=T, M=M, n_obs=n_obs, noise_kind=2, jump_prob=0.1, jump_size=0.4)
    got = fake_hip.run("test_flat_route_cpu", "kernels(%r, True)" % (kw,))
    assert any(k.startswith("k_cvar") for k in got) == IMPULSE[(K, T, M, n_obs)]
