"""Rollouts laid out without gaps (256 consecutive (sample, draw) pairs per
workgroup, CVaR in a pass of its own) for draw counts that do not fill
workgroups, bit for bit against the per-sample layout that a gradient handle
keeps, and in a batch against single steps."""
import numpy as np
import pytest

from paper_2209_12842_amd import workloads as W

torch = pytest.importorskip("torch")

KEYS = ("S", "cvar", "S_tilde")


def _state(c):
    torch.cuda.synchronize()
    return {k: v.cpu().numpy().copy() for k, v in c.debug().items() if k in KEYS}


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [dict(K=3001, M=100, T=64), dict(K=3001, M=100, T=64, B=2.0),
                                dict(K=9000, M=19, T=97, noise_kind=1), dict(K=4000, M=140, T=40, alpha=0.5),
                                dict(K=3000, M=205, T=40, noise_kind=2, jump_prob=0.1, jump_size=0.4)])
def test_flat_equals_per_sample_layout(kw):
    import paper_2209_12842_amd as R
    w = W.make_world("c2", lam=50.0, **kw)
    V0 = W.random_V(int(w["params"]["T"]), 5)
    a = R.Controller(w["params"], w["obstacles"])
    Va = a.new_V(V0)
    a.step(w["x0"], Va, 9)
    b = R.Controller(w["params"], w["obstacles"], grad=True)
    b.free_energy(w["x0"], b.new_V(V0), 9)
    sa, sb = _state(a), _state(b)
    for k in KEYS:
        assert np.array_equal(sa[k], sb[k]), k
    obs = torch.as_tensor(w["obstacles"]).cuda()
    Vn = a.new_V(V0)
    try:
        R.step_noalloc(w["params"], obs, w["x0"], Vn, 9)
    except R.MppiError:  # larger than the library's scratch memory
        pass
    else:
        torch.cuda.synchronize()
        assert torch.equal(Va, Vn)
    a.close()
    b.close()


@pytest.mark.gpu
def test_flat_controllers_in_a_batch():
    import paper_2209_12842_amd as R
    ws = [W.make_world("c2", lam=5.0, shift=True, **kw) for kw in
          (dict(K=8192, M=100, T=70), dict(K=300, M=64, T=20), dict(K=777, M=37, T=31, B=2.0),
           dict(K=512, M=8, T=20, noise_kind=1), dict(K=400, M=250, T=12, alpha=0.5))]
    V0 = [W.random_V(int(w["params"]["T"]), 3 + i) for i, w in enumerate(ws)]
    b = R.Batch([w["params"] for w in ws], [w["obstacles"] for w in ws], V0=V0)
    x0 = np.stack([w["x0"] for w in ws])
    for j in range(2):
        u0 = b.step(x0, 4 + j)
    for i, w in enumerate(ws):
        c = R.Controller(w["params"], w["obstacles"])
        V = c.new_V(V0[i])
        for j in range(2):
            ui = c.step(w["x0"], V, 4 + j)
        torch.cuda.synchronize()
        assert torch.equal(V, b.V[i]), i
        assert np.array_equal(ui, u0[i]), i
        sa, d = _state(c), b.debug(i)
        for k in KEYS:
            assert np.array_equal(sa[k], d[k].cpu().numpy()), (i, k)
        c.close()
    b.close()
