"""What a serving session leaves in the workspace for the debug view (command,
weights, costs) is the last step's, although another workgroup may have merged
each step, bit for bit against launched steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("debug", [False, True])
@pytest.mark.parametrize("K,T,M,n", [(200, 12, 8, 40), (513, 20, 16, 60), (2048, 50, 64, 60)])
def test_debug_view_after_a_session(K, T, M, n, debug):
    import paper_2209_12842_amd as ra
    from paper_2209_12842_amd import workloads as W
    torch.cuda.set_device(0)
    w = W.make_world("c2", K=K, M=M, T=T, lam=50.0)
    V0 = W.random_V(T, 3)
    views = []
    for served in (False, True):
        c = ra.Controller(w["params"], w["obstacles"], debug=debug)
        V = c.new_V(V0)
        for stop in (1, n // 2, n):                     # sessions that end after one step, some and many
            if served:
                c.serve_start(V)
            for i in range(stop):
                x = np.asarray(w["x0"], dtype=np.float32) + np.float32(0.01 * i)
                (c.serve_step if served else lambda x, i: c.step(x, V, i))(x, i)
            if served:
                c.serve_stop()
            torch.cuda.synchronize()
            keys = ("u0", "S", "cvar", "S_tilde") + (("u", "L", "w_hat") if debug else ())
            views.append({k: v.cpu().numpy().copy() for k, v in c.debug().items() if k in keys})
        c.close()
    for a, b in zip(views[:3], views[3:]):
        for k in a:
            assert np.array_equal(a[k], b[k]), k
