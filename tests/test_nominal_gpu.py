"""Nominal rollouts (64 samples per workgroup, controls drawn one run of six
steps ahead): horizons around the run length, ragged sample counts, and the
form that packs several groups into a workgroup so that a grid stays one
launch."""
import numpy as np
import pytest

import oracle
from paper_2209_12842_amd import workloads as W

torch = pytest.importorskip("torch")


def _step(split, world, **kw):
    import paper_2209_12842_amd as R
    w = W.make_world(world, **kw)
    V0 = W.random_V(int(w["params"]["T"]), 3)
    c = R.Controller(w["params"], w["obstacles"], debug=True, split_update=split)
    V = c.new_V(V0)
    u0 = c.step(w["x0"], V, 5)
    torch.cuda.synchronize()
    d = {k: v.cpu().numpy().copy() for k, v in c.debug().items()}
    d["V"], d["u0"] = V.cpu().numpy().copy(), np.asarray(u0).copy()
    c.close()
    return w, V0, d


@pytest.mark.gpu
@pytest.mark.parametrize("world,kw", [("c1", dict(K=1, T=1, M=64)), ("c1", dict(K=65, T=5, M=64)),
                                      ("c1", dict(K=64, T=6, M=16)), ("c2", dict(K=130, T=7, M=48, lam=50.0)),
                                      ("p0", dict(K=100, T=12, M=90)), ("c2", dict(K=193, T=13, M=300, eta=0.5)),
                                      # more groups of 64 than fit beside the disturbed workgroups at once
                                      ("c2", dict(K=3900, T=13, M=64))])
def test_one_launch_equals_two_and_the_oracle(world, kw):
    w, V0, a = _step(False, world, **kw)
    _, _, b = _step(True, world, **kw)
    for k in ("u", "S", "cvar", "S_tilde", "V", "u0"):
        assert np.array_equal(a[k], b[k]), k
    p = w["params"]
    if p["K"] > 512:
        return
    o = oracle.step(p, w["obstacles"], w["x0"], V0, 5)
    ok = (o["nom_margin"] >= 1e-3) & (o["nom_cond"] >= 0.25)
    assert ok.any()
    rel = np.abs(a["S"] - o["S"]) / np.maximum(np.abs(o["S"]), 1.0)
    assert rel[ok].max() <= 1e-4
