"""The CVaR that rollout workgroups form, by single waves or over the whole
workgroup, on both sides of the line between them (whether the waves hold the
workgroup's samples at once; M = 512): bit for bit the CVaR entry point's of
the same stored costs, which has tests of its own."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("B", [1.0, 2.0])
@pytest.mark.parametrize("M", [1, 2, 3, 7, 8, 14, 15, 28, 29, 31, 32, 33, 51, 52, 63, 64, 65, 85, 86, 100, 128, 129, 255, 256,
                               257, 448, 511, 512, 513, 1024])
def test_rollout_cvar_equals_the_entry_point(M, B):
    import paper_2209_12842_amd as ra
    from paper_2209_12842_amd import workloads as W
    w = W.make_world("c2", K=131, M=M, T=7, B=B, lam=50.0)
    for alpha in (0.9, 0.5, 1.0 - 63.5 / M if M > 64 else 0.3):       # the last: a tail of 64
        w["params"]["alpha"] = alpha
        c = ra.Controller(w["params"], w["obstacles"], debug=True)
        V = c.new_V(W.random_V(7, 3))
        c.step(w["x0"], V, 5)
        d = c.debug()
        ref = ra.cvar(d["L"].clone(), alpha, B)
        torch.cuda.synchronize()
        assert torch.equal(d["cvar"], ref), alpha
        c.close()
