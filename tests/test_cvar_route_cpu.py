"""Which pass the CVaR entry point takes (CPU only): the wave pass where a
wave's lanes are used and the tail is short, k_cvar otherwise."""
import ctypes

import pytest

import fake_hip

# (M, n_tail): the wave pass
CASES = {(1, 1): True, (3, 3): True, (4, 4): True, (5, 1): False, (8, 8): True, (24, 2): False, (32, 32): True, (40, 1): False,
         (47, 5): False, (48, 12): True, (48, 13): False, (54, 30): True, (55, 32): True, (55, 33): False, (64, 32): True,
         (64, 33): False, (65, 49): True, (65, 50): False, (80, 64): True, (80, 65): False, (1000, 64): True}


def launched(M, n_tail):
    import paper_2209_12842_amd as R
    fake_hip.fake.fake_reset(-1)
    R.check(R.lib().mppi_cvar(fake_hip.memory(40 * M), 10, M, 1 - (n_tail - 0.5) / M, 1.0, fake_hip.memory(40), None))
    return [k for k, *_ in fake_hip.launches()]


@pytest.mark.parametrize("M,n_tail", list(CASES))
def test_route(M, n_tail):
    got = fake_hip.run("test_cvar_route_cpu", "launched(%d, %d)" % (M, n_tail))
    assert got == ["k_cvar_wave" if CASES[(M, n_tail)] else "k_cvar"]
