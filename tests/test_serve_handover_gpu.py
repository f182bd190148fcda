"""Served steps hand the request and the mean sequence on without writing back
or invalidating a cache: long sessions whose every step depends on the last
one's result, from one chunk to several and from one workgroup per kind to
many, bit for bit against launched steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("K,T,M", [(1, 2, 1), (64, 7, 8), (257, 20, 16), (1000, 45, 48), (2048, 50, 64)])
def test_long_sessions_follow_launched_steps(K, T, M):
    import paper_2209_12842_amd as ra
    from paper_2209_12842_amd import workloads as W
    torch.cuda.set_device(0)
    w = W.make_world("c2", K=K, T=T, M=M, lam=50.0)     # many weighted samples; the sequence is shifted
    V0 = W.random_V(T, 3)
    n = 150
    xs = [np.asarray(w["x0"], dtype=np.float32) + np.float32(0.01 * i) * np.float32([1, -1, 0.1, 0.2]) for i in range(n)]
    launched = ra.Controller(w["params"], w["obstacles"])
    Vl = launched.new_V(V0)
    ul = [np.array(launched.step(x, Vl, i, want_u0=True), dtype=np.float32) for i, x in enumerate(xs)]
    torch.cuda.synchronize()
    served = ra.Controller(w["params"], w["obstacles"])
    Vs = served.new_V(V0)
    served.serve_start(Vs)
    us = [np.array(served.serve_step(x, i), dtype=np.float32) for i, x in enumerate(xs)]
    served.serve_stop()
    torch.cuda.synchronize()
    wrong = [i for i in range(n) if not np.array_equal(ul[i], us[i])]
    assert not wrong, wrong[:5]
    assert np.array_equal(Vl.cpu().numpy(), Vs.cpu().numpy())
    launched.close()
    served.close()
