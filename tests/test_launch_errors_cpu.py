"""A launch that fails ends its call with an error and nothing is launched
after it: the update must not write a command and a mean sequence from costs
that were never computed.  Every launch of every route fails once, on a HIP
runtime that runs nothing (CPU only)."""
import ctypes

import pytest

import fake_hip

ROUTES = {  # what the call launches
    "one launch": ["k_rollout_fused"],
    "two launches": ["k_rollout", "k_update"],
    "flattened": ["k_rollout", "k_cvar_wave", "k_update"],
    "flattened, long tails": ["k_rollout", "k_cvar_sorted", "k_update"],
    "caller's memory": ["k_rollout", "k_cvar_wave", "k_update"],
    "gradient": ["k_rollout", "k_update_grad", "k_grad_rollouts", "k_grad_reduce"],
    "batch": ["k_batch_prep", "k_batch_rollout", "k_batch_cvar", "k_batch_update"],
    "batch, timed": ["k_batch_prep", "k_batch_rollout", "k_batch_cvar", "k_batch_update"],
}


def _call(route):
    import paper_2209_12842_amd as R
    L, mem = R.lib(), fake_hip.memory
    if route.startswith("batch"):
        ws = [fake_hip.world(K=8192, M=100, T=70), fake_hip.world(K=300, M=64, T=20)]
        b = fake_hip.batch([w[0] for w in ws], [w[1] for w in ws])
        x, idx = (ctypes.c_float * 8)(*ws[0][2], *ws[1][2]), (ctypes.c_uint32 * 2)(0, 0)
        if route == "batch":
            L.mppi_batch_set_graph(b, 0)
        else:
            L.mppi_batch_timing_enable(b, 1)
        return lambda: L.mppi_batch_step(b, x, idx, None, None)
    kw = {"one launch": dict(K=512), "two launches": dict(K=16384), "flattened": dict(K=3001, M=100, T=64),
          "flattened, long tails": dict(K=3001, M=300, alpha=0.5), "caller's memory": dict(K=1024, M=300, T=30),
          "gradient": dict(K=512)}[route]
    p, obs, x0 = fake_hip.world(flags=R.MPPI_F_GRAD if route == "gradient" else 0, **kw)
    V, out = mem(8 * p.T), mem(8 * p.T)
    if route == "caller's memory":
        return lambda: L.mppi_step_noalloc(ctypes.byref(p), obs, x0, V, 0, out, None)
    h = fake_hip.handle(p, obs)
    if route == "gradient":
        return lambda: L.mppi_grad(h, x0, V, 0, out, out, None)
    return lambda: L.mppi_step(h, x0, V, 0, None, None)


def outcomes(route):
    """[(status, kernels launched)] without a failure, then with each launch failing."""
    call = _call(route)
    got = []
    for fail in [-1] + list(range(len(ROUTES[route]))):
        fake_hip.fake.fake_reset(fail)
        got.append([call(), [k for k, *_ in fake_hip.launches()]])
    return got


@pytest.mark.parametrize("route", list(ROUTES))
def test_a_failed_launch_ends_the_call(route):
    names = ROUTES[route]
    got = fake_hip.run("test_launch_errors_cpu", "outcomes(%r)" % route)
    ok, failed = got[0], got[1:]
    assert ok[0] == 0 and [n.replace("k_batch_rollout_one", "k_batch_rollout") for n in ok[1]] == names
    for i, (status, ran) in enumerate(failed):
        assert status == -3, (names[i], status)        # MPPI_EDEVICE
        assert len(ran) == i + 1, (names[i], ran)      # nothing after the failure
