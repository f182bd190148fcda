"""Every launch of a step stays within the LDS that parameter validation
allows, whatever layout the step takes: the flattened one holds the controls
of one sample more than the per-sample one for M > 256 (CPU only)."""
import ctypes

import pytest

import fake_hip

LIMIT = 64 * 1024
# name: sizes, and whether the flattened layout fits (16 bytes of controls a step and sample pair)
SIZES = {"M=1024 T=3500": (dict(K=100, T=3500, M=1024, n_obs=10), False),
         "M=300 T=3800": (dict(K=100, T=3800, M=300, n_obs=10), False),
         "M=300 T=3600": (dict(K=100, T=3600, M=300, n_obs=10), True),
         "M=257 T=3700 no obstacles": (dict(K=64, T=3700, M=257, n_obs=0), True)}


def launches(name, noalloc):
    import paper_2209_12842_amd as R
    L, mem = R.lib(), fake_hip.memory
    # (16: the update in a launch of its own)
    p, obs, x0 = fake_hip.world(flags=0 if noalloc else 16, **SIZES[name][0])
    h = None if noalloc else fake_hip.handle(p, obs)
    V = mem(8 * p.T)
    fake_hip.fake.fake_reset(-1)
    if noalloc:
        R.check(L.mppi_step_noalloc(ctypes.byref(p), obs, x0, V, 0, None, None))
    else:
        R.check(L.mppi_step(h, x0, V, 0, None, None))
    return fake_hip.launches()


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("name", list(SIZES))
def test_launches_stay_within_the_limit(name, noalloc):
    got = fake_hip.run("test_launch_lds_cpu", "launches(%r, %r)" % (name, noalloc))
    for kernel, grid, block, lds in got:
        assert lds <= LIMIT, (kernel, lds)
    flat = any(k.startswith("k_cvar") for k, *_ in got)
    assert flat == SIZES[name][1]
