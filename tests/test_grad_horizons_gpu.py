"""The gradient around the horizons (7, 8, 24, 25 steps), row counts and sample
counts at which its form changes, against the FP64 oracle (worlds without jumps and tolerances
as in test_grad_forms_gpu)."""
import numpy as np
import pytest

import oracle
from paper_2209_12842_amd import workloads as W

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("K,M,T", [(30, 8, 7), (30, 8, 8), (910, 8, 8), (911, 8, 8), (910, 8, 24), (911, 8, 24), (911, 8, 25),
                                   (1820, 8, 25), (1821, 8, 25),
                                   # one block of 256 rows, two, 64, 65, and more than 1024
                                   (28, 8, 9), (29, 8, 9), (1820, 8, 3), (1821, 8, 3), (32768, 8, 3),
                                   # one chunk of samples, two, sixteen, seventeen
                                   (256, 4, 8), (257, 4, 8), (4096, 4, 2), (4097, 4, 2)])
def test_gradient_around_its_lines(K, M, T):
    import paper_2209_12842_amd as R
    w = W.make_world("c2", K=K, M=M, T=T, n_obs=0, lam=500.0, alpha=0.001, B=2.0, C_u=-1.0e9)
    V0 = W.random_V(T, 7, scale=(0.5, 0.1))
    c = R.Controller(w["params"], w["obstacles"], grad=True)
    J, g = c.free_energy(w["x0"], c.new_V(V0), 3)
    torch.cuda.synchronize()
    Jo, go = oracle.free_energy(w["params"], w["obstacles"], w["x0"], V0, 3, grad=True)
    go = np.asarray(go).reshape(T, 2)
    assert abs(float(J) - Jo) <= 1e-4 * max(1.0, abs(Jo))
    assert np.abs(g.cpu().numpy() - go).max() <= 3e-4 * np.abs(go).max()
    c.close()
