"""Served steps with the mean sequence in LDS, and at the sizes that leave no
room for it, bit for bit against launched steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [dict(K=300, T=29, M=1), dict(K=300, T=30, M=1),
                                dict(K=34000, T=30, M=1), dict(K=34500, T=29, M=1),  # 64 KB without the copy; with it
                                dict(K=15625, T=64, M=8), dict(K=15624, T=64, M=8),  # a million controls dict(K=64, T=1500, M=64), dict(K=40, T=3300, M=256),
                                dict(K=70, T=1, M=200), dict(K=600, T=130, M=8, lam=500.0)])
def test_sessions_follow_launched_steps(kw):
    import paper_2209_12842_amd as ra
    from paper_2209_12842_amd import workloads as W
    w = W.make_world("c2", n_obs=10, **dict(dict(lam=50.0, shift=True), **kw))
    V0 = W.random_V(kw["T"], 3)
    out = []
    for served in (False, True):
        c = ra.Controller(w["params"], w["obstacles"])
        V = c.new_V(V0)
        if served:
            c.serve_start(V)
        u = [np.array(c.serve_step(w["x0"], i) if served else c.step(w["x0"], V, i)) for i in range(8)]
        if served:
            c.serve_stop()
        torch.cuda.synchronize()
        out.append((np.stack(u), V.cpu().numpy().copy()))
        c.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
