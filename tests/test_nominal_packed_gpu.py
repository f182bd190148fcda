"""Packed nominal workgroups, a wave for each 64 samples: served steps whose
grid would not be resident with one workgroup for each, bit for bit against
launched steps, which take two launches at these sizes; and two-launch steps of
one or two draws against the one-launch form."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("world,kw", [("c2", dict(K=3900, T=13, M=64)), ("c2", dict(K=14001, T=6, M=16, noise_kind=1)),
                                      ("c2", dict(K=45000, T=7, M=4)), ("p0", dict(K=4030, T=5, M=60)),
                                      ("c2", dict(K=3999, T=1, M=64, n_obs=0)), ("c2", dict(K=511, T=12, M=512)),
                                      ("c2", dict(K=510, T=9, M=300)),    # five waves: two workgroups a unit
                                      ("c2", dict(K=3900, T=20, M=64, n_obs=130, debug=True))])
def test_packed_sessions_follow_launched_steps(world, kw):
    import paper_2209_12842_amd as ra
    from paper_2209_12842_amd import workloads as W
    torch.cuda.set_device(0)
    kw = dict(kw)
    debug = kw.pop("debug", False)
    w = W.make_world(world, lam=50.0, shift=True, **kw)
    V0 = W.random_V(int(w["params"]["T"]), 3)
    xs = [np.asarray(w["x0"], dtype=np.float32) + np.float32(0.01 * i) for i in range(12)]
    out = []
    for served in (False, True):
        c = ra.Controller(w["params"], w["obstacles"], debug=debug)
        V = c.new_V(V0)
        if served:
            c.serve_start(V)
        u = [np.array(c.serve_step(x, i) if served else c.step(x, V, i)) for i, x in enumerate(xs)]
        if served:
            c.serve_stop()
        torch.cuda.synchronize()
        keys = ("S", "cvar", "S_tilde") + (("u", "L", "w_hat") if debug else ())
        out.append(dict({k: v.cpu().numpy().copy() for k, v in c.debug().items() if k in keys},
                        V=V.cpu().numpy().copy(), cmd=np.stack(u)))
        c.close()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k


@pytest.mark.gpu
@pytest.mark.parametrize("world,kw", [("c2", dict(K=1, T=1, M=1)), ("c2", dict(K=65, T=5, M=2)), ("p0", dict(K=256, T=6, M=1)),
                                      ("c2", dict(K=257, T=13, M=2, n_obs=70)), ("p0", dict(K=3000, T=18, M=2, noise_kind=1)),
                                      ("c2", dict(K=1021, T=17, M=3)), ("p0", dict(K=768, T=8, M=4, n_obs=130)),
                                      ("c2", dict(K=330, T=9, M=4, n_obs=0, c_bdry=1.0, noise_kind=2, jump_prob=0.2, jump_size=0.4))])
def test_packed_two_launch_steps(world, kw):
    import paper_2209_12842_amd as ra
    from paper_2209_12842_amd import workloads as W
    w = W.make_world(world, lam=50.0, **kw)
    V0 = W.random_V(int(w["params"]["T"]), 3)
    out = []
    for split in (False, True):
        c = ra.Controller(w["params"], w["obstacles"], debug=True, split_update=split)
        V = c.new_V(V0)
        u0 = c.step(w["x0"], V, 5)
        torch.cuda.synchronize()
        out.append(dict({k: v.cpu().numpy().copy() for k, v in c.debug().items()}, V=V.cpu().numpy().copy(), cmd=u0.copy()))
        c.close()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k


@pytest.mark.gpu
@pytest.mark.parametrize("kw", [dict(K=100001, T=3, M=5), dict(K=120000, T=9, M=6, n_obs=70, noise_kind=1)])
def test_packed_steps_of_many_rounds(kw):
    """The first samples of a large step against the one-launch step of these
    samples alone (all of them warm, so a sample depends on its index only)."""
    import paper_2209_12842_amd as ra
    from paper_2209_12842_amd import workloads as W
    out = []
    for K in (kw["K"], 300):
        w = W.make_world("c2", lam=50.0, eta=0.0, **dict(kw, K=K))
        c = ra.Controller(w["params"], w["obstacles"], debug=True)
        c.step(w["x0"], c.new_V(W.random_V(kw["T"], 3)), 5)
        torch.cuda.synchronize()
        d = c.debug()
        assert torch.isfinite(d["S"]).all()
        out.append((d["S"][:300].cpu().numpy(), d["cvar"][:300].cpu().numpy(), d["u"].cpu().numpy().reshape(kw["T"], K, 2)[:, :300]))
        c.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
