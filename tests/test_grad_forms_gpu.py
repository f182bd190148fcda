"""The gradient's two forms (steps side by side for few rows, a lane per row
for many) and its row sum (one workgroup or several per output) at the edges
of their tiles and on both sides of their lines, against the FP64 oracle.

The worlds have no jump: no obstacles, every draw in the tail, the bound C_u
always exceeded, so the gradient differs from the oracle's by rounding alone.
Costs near 1e4 at FP32 give weights to 1e-2 / lambda = 2e-5, the recomputed
rollouts and the row sums about 1e-4 of the largest component: 3e-4 together."""
import numpy as np
import pytest

import oracle
from paper_2209_12842_amd import workloads as W

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("K,M,T,noise", [(3, 2, 1, 0), (40, 8, 63, 1), (40, 8, 64, 0), (40, 8, 65, 2), (24, 6, 130, 0),
                                         (1820, 8, 7, 0),    # 16380 rows: the last by time, 64 blocks of 256
                                         (1822, 8, 7, 1),    # 16398 rows: a lane each, 65 blocks
                                         (2200, 16, 12, 0)])  # 37400 rows in several workgroups per output
def test_gradient_forms(K, M, T, noise):
    import paper_2209_12842_amd as R
    w = W.make_world("c2", K=K, M=M, T=T, n_obs=0, lam=500.0, alpha=0.001, B=2.0, C_u=-1.0e9, noise_kind=noise,
                     jump_prob=0.1, jump_size=0.45)
    V0 = W.random_V(T, 7, scale=(0.5, 0.1))
    c = R.Controller(w["params"], w["obstacles"], grad=True)
    V = c.new_V(V0)
    J, g = c.free_energy(w["x0"], V, 3)
    J2, g2 = c.free_energy(w["x0"], V, 3)
    torch.cuda.synchronize()
    assert torch.equal(J, J2) and torch.equal(g, g2)
    Jo, go = oracle.free_energy(w["params"], w["obstacles"], w["x0"], V0, 3, grad=True)
    go = np.asarray(go).reshape(T, 2)
    assert abs(float(J) - Jo) <= 1e-4 * max(1.0, abs(Jo))
    assert np.abs(g.cpu().numpy() - go).max() <= 3e-4 * np.abs(go).max()
    c.close()
