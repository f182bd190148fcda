"""Where a step is one launch and how a served step's nominal workgroups are
laid out, on a device that holds 1024 workgroups at once: a step whose grid of
64-sample nominal workgroups does not fit takes two launches, and a served
one, which has no such choice, packs them (CPU only)."""
import ctypes

import pytest

import fake_hip

TWO, FLAT = ["k_rollout", "k_update"], ["k_rollout", "k_cvar_wave", "k_update"]
CASES = {  # (K, M, waves per SIMD): the step's kernels, the served grid or None where it is refused
    (3852, 64, 4): (["k_rollout_fused"], 963 + 61),
    (3855, 64, 4): (TWO, 964 + 16),                   # 964 + 61 is one too many
    (4032, 64, 4): (TWO, 1008 + 16),
    (4033, 64, 4): (TWO, None),
    (14000, 16, 4): (TWO, 875 + 55),
    (511, 512, 4): (FLAT, 511 + 1),
    (504, 300, 4): (["k_rollout_fused"], 504 + 8),   # five waves: two on one SIMD, so two workgroups a unit, not three
    (505, 300, 4): (FLAT, 505 + 2),                  # 505 + 8 is one too many
    (510, 300, 4): (FLAT, 510 + 2),
    (512, 300, 4): (FLAT, None),
    (504, 320, 4): (["k_rollout_fused"], 504 + 8),
    (512, 321, 4): (FLAT, None),                     # six waves: two workgroups a unit
    (2400, 90, 4): (["k_rollout_fused"], 1200 + 38),  # three waves
    (254, 1024, 4): (["k_rollout", "k_cvar_sorted", "k_update"], 254 + 1),
}


def launches(K, M, per_cu):
    import paper_2209_12842_amd as R
    L, mem = R.lib(), fake_hip.memory
    fake_hip.fake.fake_resident(per_cu)
    p, obs, x0 = fake_hip.world(K=K, M=M, T=20)
    h = fake_hip.handle(p, obs)
    V = mem(8 * p.T)
    fake_hip.fake.fake_reset(-1)
    R.check(L.mppi_step(h, x0, V, 0, None, None))
    ran = fake_hip.launches()
    step = [k for k, *_ in ran]
    fake_hip.fake.fake_reset(-1)
    status = L.mppi_serve_start(h, V, 100, None)
    serve = fake_hip.launches()
    assert (status == 0) == (len(serve) == 1) and (status in (0, -4))
    L.mppi_destroy(h)
    return [step, serve[0][1] if serve else None, serve[0][3] if serve else 0, ran[0][1]]


@pytest.mark.parametrize("K,M,per_cu", list(CASES))
def test_forms(K, M, per_cu):
    step, grid, lds, _ = fake_hip.run("test_nominal_forms_cpu", "launches(%d, %d, %d)" % (K, M, per_cu))
    assert step == CASES[(K, M, per_cu)][0]
    assert grid == CASES[(K, M, per_cu)][1]
    assert lds <= 64 * 1024


@pytest.mark.parametrize("K,M,grid", [(200000, 1, 782 + 782), (80001, 2, 626 + 313), (100000, 3, 1177 + 391),
                                      (100000, 4, 1563 + 391), (100000, 5, 1961 + 391), (80000, 5, 1569 + 1250),
                                      (110000, 6, 2620 + 430), (60000, 6, 1429 + 938), (120000, 7, 3334 + 1875)])
def test_few_draws_pack_their_nominal_workgroups(K, M, grid):
    step, _, _, got = fake_hip.run("test_nominal_forms_cpu", "launches(%d, %d, 4)" % (K, M))
    assert step == TWO and got == grid
