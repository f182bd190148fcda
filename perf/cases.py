"""Workloads by which the framework's speed is measured, through its public
entry points: single control steps from the smallest world to the largest,
steps on caller-owned memory, a persistent serving session, batched serving
and the gradient of the free energy.

A case is a dict of plain values:
  kind    "step" (Controller.step, first command read back), "noalloc"
          (step_noalloc), "serve" (a serving session of `n` control instants),
          "batch" (Batch.step of `n` controllers of mixed sizes), "grad"
          (free_energy and its backward pass)
  world   "box" (the small 40 x 40 m world), "oval" (the 100 x 40 m track)
          or "paper" (the 0.6 m wide track with the paper's own settings)
  K, T, M, n_obs   samples, horizon, draws per sample, obstacles (for "batch"
          the upper ends of the ranges the controllers' sizes are drawn from)
  lam     temperature;  noise  0 Gaussian, 1 uniform, 2 impulse;  B  risk scaling
Each kind exists because a program calls it: a car's control loop awaits every
command, a simulation fleet steps many controllers at once, a planner that
tunes its mean sequence takes gradients.
"""
from __future__ import annotations

import copy
import math

import numpy as np
import torch

import paper_2209_12842_amd as ra
from paper_2209_12842_amd import workloads as W


def _case(name, kind, world, K, T, M, n_obs, lam, noise=0, B=1.0, n=0):
    c = dict(kind=kind, world=world, K=K, T=T, M=M, n_obs=n_obs, lam=lam, noise=noise, B=B, n=n)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest loop: few samples, latency and launches only
        _case("step_small", "step", "box", 256, 20, 16, 10, 1.0),
        # the ordinary receding-horizon loop of a car on a track
        _case("step_receding", "step", "oval", 2048, 50, 64, 50, 0.5),
        # nothing a multiple of anything; impulse disturbances and risk scaling
        _case("step_ragged_impulse", "step", "oval", 1000, 45, 48, 20, 0.5, noise=2, B=2.0),
        # the paper's own sample counts, horizon and weights
        _case("step_paper", "step", "paper", 1024, 30, 300, 10, 0.35),
        # a mid-size step whose draws do not fill whole wavefronts, uniform disturbances
        _case("step_uniform_odd", "step", "oval", 4000, 60, 100, 120, 1.0, noise=1),
        # the largest step
        _case("step_large", "step", "oval", 16384, 100, 128, 200, 1.0),
        # a program that may not allocate and reads the command on the device
        _case("noalloc_receding", "noalloc", "oval", 2048, 50, 64, 50, 0.5),
        # a serving session: 32 control instants through one resident launch
        _case("serve_receding", "serve", "oval", 2048, 50, 64, 50, 0.5, n=32),
        # a small fleet of small controllers
        _case("batch_small", "batch", "oval", 1024, 40, 64, 50, 0.5, n=8),
        # a large fleet of controllers of uneven size
        _case("batch_mixed", "batch", "oval", 8192, 100, 128, 200, 0.5, n=48),
        # the gradient at the step's own temperature: a handful of weighted samples
        _case("grad_sharp", "grad", "oval", 4096, 50, 64, 50, 0.5),
        # the gradient at a high temperature: hundreds of weighted samples
        _case("grad_smooth", "grad", "oval", 2048, 50, 64, 50, 50.0),
    ]


_LARGEST = 16384 * 100 * 128  # disturbed state steps of the largest single step


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choices(["step", "noalloc", "serve", "batch", "grad"], [8, 2, 1, 3, 3])[0]
    world = "oval" if kind == "batch" else rng.choice(["box", "oval", "oval", "paper"])
    noise = rng.choice([0, 0, 0, 1, 2])
    B = rng.choice([1.0, 1.0, 2.0, 0.5])
    n_obs = rng.randint(10, 200) if world == "oval" else rng.randint(0, 12)
    if kind == "batch":
        n = log_int(2, 48)
        return _case(None, kind, world, 256 * log_int(2, 32), rng.randint(30, 100), rng.randint(16, 128), n_obs, 0.5,
                     noise, B, n)
    if kind == "serve":  # the whole grid is resident at once: up to about the receding-horizon size
        return _case(None, kind, world, log_int(128, 2048), rng.randint(10, 60), log_int(8, 64), n_obs, 0.5, noise, B,
                     rng.randint(8, 32))
    if kind == "noalloc":  # the step's workspace has to fit the library's scratch memory
        return _case(None, kind, world, log_int(128, 4096), rng.randint(10, 100), log_int(8, 320), n_obs, 0.5, noise,
                     B)
    if kind == "grad":
        return _case(None, kind, world, log_int(256, 4096), rng.randint(10, 60), log_int(8, 128), n_obs,
                     rng.choice([0.5, 1.0, 20.0, 50.0]), noise, B)
    while True:
        c = _case(None, kind, world, log_int(128, 16384), rng.randint(10, 100), log_int(8, 512), n_obs,
                  rng.choice([0.35, 0.5, 1.0]), noise, B)
        if c["K"] * c["T"] * c["M"] <= _LARGEST:
            return c


# ---------------------------------------------------------------- inputs


def _world(case, seed, K, T, M, n_obs):
    """Parameters, obstacles, start state and mean sequence (host) of one controller, from the seed."""
    rng = np.random.default_rng(seed)
    if case["world"] == "oval":
        w = W.make_batch(1, seed=seed, k_range=(256, 256), t_range=(T, T), m_range=(M, M), obs_range=(n_obs, n_obs))[0]
        p = w["params"]
    else:
        w = W.make_world("c1" if case["world"] == "box" else "p0", T=T, n_obs=n_obs)
        p = w["params"]
        spread = 0.2 if case["world"] == "box" else 0.02
        w["obstacles"] = w["obstacles"].copy()
        w["obstacles"][:, :2] += rng.uniform(-spread, spread, (n_obs, 2)).astype(np.float32)
        w["x0"] = (w["x0"] * (1.0 + 0.1 * rng.uniform(-1.0, 1.0, 4) * (0, 0, 0, 1))).astype(np.float32)
    p.update(K=K, T=T, M=M, lam=case["lam"], gamma=case["lam"], B=case["B"], noise_kind=case["noise"], shift=True,
             seed=W.SEED_BASE + 7919 * seed)
    if case["noise"] == 2:
        p.update(jump_prob=0.02, jump_size=0.45 if case["world"] != "paper" else 0.045)
    V0 = W.random_V(T, seed, scale=(0.5, 0.1))
    return dict(params=p, obstacles=w["obstacles"], x0=w["x0"], V0=V0)


def _sizes(case):
    """(K, T, M, n_obs) of the case's controllers: one, or for a batch `n` drawn up to the case's own sizes."""
    K, T, M, n_obs = case["K"], case["T"], case["M"], case["n_obs"]
    if case["kind"] != "batch":
        return [(K, T, M, n_obs)]
    rng = np.random.default_rng([K, T, M, case["n"]])  # the sizes belong to the case, not to the seed
    return [(256 * int(rng.integers(1, K // 256 + 1)), int(rng.integers(min(20, T), T + 1)),
             int(rng.integers(8, M + 1)), int(rng.integers(min(10, n_obs), n_obs + 1))) for _ in range(case["n"])]


def _worlds(case, seed):
    sizes = _sizes(case)
    if len(sizes) == 1:
        return [_world(case, seed, *sizes[0])]
    return [_world(case, 1000 * seed + i, *s) for i, s in enumerate(sizes)]


def _session_states(case, x0, seed):
    """The measured states of a serving session: the start state with measurement scatter."""
    rng = np.random.default_rng(seed + 1)
    spread = np.asarray((0.05, 0.05, 0.01, 0.1)) * (0.1 if case["world"] == "paper" else 1.0)
    return (x0 + rng.uniform(-1.0, 1.0, (case["n"], 4)) * spread).astype(np.float32)


def prepare(case, seed):
    ws = _worlds(case, seed)
    kind = case["kind"]
    st = {"kind": kind, "step": 0, "x0": ws[0]["x0"]}
    if kind == "batch":
        st["ctl"] = ra.Batch([w["params"] for w in ws], [w["obstacles"] for w in ws], V0=[w["V0"] for w in ws])
        st["x0"] = np.stack([w["x0"] for w in ws])
        return st
    w = ws[0]
    if kind == "noalloc":
        st["params"] = w["params"]
        st["obs"] = torch.as_tensor(w["obstacles"]).cuda() if len(w["obstacles"]) else None
        st["V"] = torch.as_tensor(w["V0"]).cuda()
        st["u0"] = torch.zeros(2, device="cuda")
        return st
    st["ctl"] = ra.Controller(w["params"], w["obstacles"], grad=kind == "grad")
    st["V"] = st["ctl"].new_V(w["V0"])
    if kind == "grad":
        st["V"].requires_grad_(True)
    if kind == "serve":
        st["xs"] = _session_states(case, w["x0"], seed)
    return st


def run(state):
    kind, i = state["kind"], state["step"]
    state["step"] = i + 1
    if kind == "step":
        u0 = state["ctl"].step(state["x0"], state["V"], i)
        return {"V": state["V"], "u0": u0}
    if kind == "noalloc":
        ra.step_noalloc(state["params"], state["obs"], state["x0"], state["V"], i, u0=state["u0"])
        return {"V": state["V"], "u0": state["u0"]}
    if kind == "serve":
        ctl, xs = state["ctl"], state["xs"]
        ctl.serve_start(state["V"])
        u0 = [ctl.serve_step(x, i * len(xs) + j) for j, x in enumerate(xs)]
        ctl.serve_stop()
        return {"V": state["V"], "u0": np.stack(u0)}
    if kind == "batch":
        u0 = state["ctl"].step(state["x0"], i)
        return {"V": state["ctl"].V, "u0": u0}
    J = ra.free_energy(state["V"], state["ctl"], state["x0"], i)
    (g,) = torch.autograd.grad(J, state["V"])
    return {"J": J.detach(), "grad": g}


def work(case):
    """Per disturbed state step 80 operations (noise, dynamics, smooth costs)
    and per nominal one 60, whatever finds the obstacles; the gradient adds
    the adjoint of a few weighted rollouts, which is left out.  Bytes: the
    obstacles and mean sequences in, the sequences and commands (or the
    gradients) out."""
    sizes = _sizes(case) * (case["n"] if case["kind"] == "serve" else 1)
    flops = sum(80.0 * K * T * M + 60.0 * K * T for K, T, M, _ in sizes)
    nbytes = sum(12.0 * o + 16.0 * T + 24.0 for _, T, _, o in sizes)
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------- 64-bit values


def _philox(ctr, key, rounds=10):
    """Philox4x32 words as int64 tensors in [0, 2^32) (broadcast over the counters)."""
    mask = 0xFFFFFFFF
    c0, c1, c2, c3 = ctr
    k0, k1 = key
    for _ in range(rounds):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # wraps modulo 2^64
        c0, c1, c2, c3 = (((p1 >> 32) & mask) ^ c1 ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c3 ^ k1, p0 & mask)
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c0, c1, c2, c3


def _uniform(r):
    return ((r >> 9).double() + 0.5) * 2.0**-23


def _normal_pair(r0, r1):
    rad = torch.sqrt(-2.0 * torch.log(_uniform(r0)))
    ang = 2.0 * math.pi * _uniform(r1)
    return rad * torch.cos(ang), rad * torch.sin(ang)


class _Exact:
    """One control step in 64 bits, written from the method's equations."""

    def __init__(self, w):
        p = {k: (np.float32(v).astype(float) if isinstance(v, (float, tuple)) else v) for k, v in w["params"].items()}
        self.p, self.dev = p, torch.device("cuda" if torch.cuda.is_available() else "cpu")
        self.obs = torch.as_tensor(w["obstacles"].astype(float)).to(self.dev).reshape(-1, 3)
        self.x0 = [float(v) for v in w["x0"]]
        self.key = (int(p["seed"]) & 0xFFFFFFFF, int(p["seed"]) >> 32)
        self.K, self.T, self.M = int(p["K"]), int(p["T"]), int(p["M"])
        self.n_tail = self.M - min(self.M, max(1, math.ceil(float(p["alpha"]) * self.M - 1e-9))) + 1
        self.n_warm = min(self.K, max(0, math.ceil((1.0 - float(p["eta"])) * self.K - 1e-9)))

    def controls(self, V, k, step):
        """Sampled controls (two n x T tensors) of the samples k, and the warm mask."""
        p = self.p
        t = torch.arange(self.T, device=self.dev)[None, :]
        r = _philox((t, torch.full_like(t, 0xFFFFFFFF), k[:, None], torch.full_like(t, step)), self.key)
        z = _normal_pair(r[0], r[1])
        warm = (k < self.n_warm).double()[:, None]
        return [torch.clamp(warm * V[None, :, i] + math.sqrt(p["sigma_eps"][i]) * z[i], p["u_lo"][i], p["u_hi"][i])
                for i in range(2)]

    def running(self, x, y, v):
        p = self.p
        ox, oy, a, b, hw = (float(q) for q in p["track"])
        X, Y = x - ox, y - oy
        G = (X / a) ** 2 + (Y / b) ** 2 - 1.0
        gn = torch.sqrt((2.0 * X / (a * a)) ** 2 + (2.0 * Y / (b * b)) ** 2).clamp_min(1e-12)
        e = G / gn
        q = p["c_dev"] * e * e + p["c_v"] * (v - p["v_ref"]) ** 2
        if p["c_bdry"]:
            q = q + p["c_bdry"] * torch.clamp(torch.atan(-100.0 * (hw - e.abs())) / math.pi + 0.5, min=0.0)
        return q

    def hits(self, x, y):
        """Number of discs each point lies in."""
        n, cnt = len(self.obs), torch.zeros_like(x)
        per = max(1, (1 << 25) // max(1, x.numel()))
        for i in range(0, n, per):
            o = self.obs[i:i + per]
            shape = (-1,) + (1,) * x.dim()
            d = (x[None] - o[:, 0].reshape(shape)).square_()
            d += (y[None] - o[:, 1].reshape(shape)).square_()
            cnt += (d < o[:, 2].reshape(shape).square()).sum(0)
        return cnt

    def advance(self, s, a, d):
        p = self.p
        x, y, psi, v = s
        return (x + p["dt"] * v * torch.cos(psi), y + p["dt"] * v * torch.sin(psi),
                psi + p["dt"] * v * torch.tan(d) / p["wheelbase"], v + p["dt"] * a)

    def disturb(self, s, t, k, m, step):
        p = self.p
        sw = [float(q) for q in p["sigma_w"]]
        full = torch.zeros_like(k + m)
        r = _philox((full + t, m + full, k + full, full + step), self.key)
        kind = int(p.get("noise_kind", 0))
        if kind == 0:
            z = _normal_pair(r[0], r[1]) + _normal_pair(r[2], r[3])
            w = [math.sqrt(sw[i]) * z[i] for i in range(4)]
        elif kind == 1:
            w = [math.sqrt(3.0 * sw[i]) * (2.0 * _uniform(r[i]) - 1.0) for i in range(4)]
        else:
            j = (_uniform(r[0]) < p["jump_prob"]).double() * p["jump_size"]
            ang = 2.0 * math.pi * _uniform(r[1])
            w = [j * torch.cos(ang), j * torch.sin(ang), 0.0, 0.0]
        return tuple(q + e for q, e in zip(s, w))

    def start(self, shape):
        return tuple(torch.full(shape, q, dtype=torch.float64, device=self.dev) for q in self.x0)

    def nominal(self, V, u):
        """S of the samples whose controls are u."""
        p = self.p
        s = self.start((u[0].shape[0],))
        S = torch.zeros_like(s[0])
        for t in range(self.T):
            S = S + self.running(s[0], s[1], s[3]) + p["c_obs"] * self.hits(s[0].detach(), s[1].detach())
            for i in range(2):
                if p["gamma"]:
                    S = S + p["gamma"] * V[t, i] * u[i][:, t] / p["sigma_eps"][i]
            s = self.advance(s, u[0][:, t], u[1][:, t])
        if p["c4"] or p["c5"]:
            ox, oy, a, b, _ = (float(q) for q in p["track"])
            th = torch.atan2((s[1] - oy) / b, (s[0] - ox) / a)
            d = th - math.atan2((self.x0[1] - oy) / b, (self.x0[0] - ox) / a)
            d = d - 2.0 * math.pi * torch.ceil((d - math.pi) / (2.0 * math.pi))
            S = S + p["c4"] - p["c5"] * 0.5 * (a + b) * d
        return S

    def cvar(self, u, k, step):
        """Tail mean of the scaled risk costs of the samples k."""
        p = self.p
        m = torch.arange(self.M, device=self.dev)[None, :]
        s = self.start((u[0].shape[0], self.M))
        L = torch.zeros_like(s[0])
        for t in range(self.T):
            L = L + self.running(s[0], s[1], s[3]) + p["c_obs"] * self.hits(s[0].detach(), s[1].detach())
            if t + 1 < self.T:
                s = self.advance(s, u[0][:, t, None], u[1][:, t, None])
                s = self.disturb(s, t, k[:, None], m, step)
        if p["B"] != 1.0:
            mean = L.mean(1, keepdim=True)
            L = p["B"] * (L - mean) + mean
        return torch.topk(L, self.n_tail, dim=1).values.mean(1)

    def modified(self, V, k, step):
        """S~ of the samples k, and their controls."""
        p = self.p
        u = self.controls(V, k, step)
        cv = self.cvar(u, k, step)
        return self.nominal(V, u) + p["A"] * torch.where(cv > p["C_u"], cv, torch.zeros_like(cv)), u

    def parts(self, k, lanes):
        per = max(1, lanes // self.M)
        return [k[i:i + per] for i in range(0, len(k), per)]

    def costs(self, V, step):
        return torch.cat([self.modified(V, k, step)[0]
                          for k in self.parts(torch.arange(self.K, device=self.dev), 1 << 21)])

    def weights(self, St):
        beta = St.min()
        w = torch.exp(-(St - beta) / self.p["lam"])
        return beta, w

    def step(self, V, step):
        """(V after the shift, first command)."""
        _, w = self.weights(self.costs(V, step))
        keep = torch.nonzero(w > 1e-30)[:, 0]
        w = w[keep] / w.sum()
        Vp = torch.stack([(w[:, None] * u).sum(0) for u in self.controls(V, keep, step)], dim=1)
        return (torch.cat([Vp[1:], Vp[-1:]]) if self.p.get("shift") else Vp), Vp[0]

    def gradient(self, V, step):
        """(J, dJ/dV) with every indicator's derivative taken as zero."""
        with torch.no_grad():
            beta, w = self.weights(self.costs(V, step))
        J = beta - self.p["lam"] * torch.log(w.sum() / self.K)
        g = torch.zeros_like(V)
        wh = w / w.sum()
        for k in self.parts(torch.nonzero(wh > 1e-12)[:, 0], 1 << 17):
            v = V.clone().requires_grad_(True)
            St, _ = self.modified(v, k, step)
            g += torch.autograd.grad((wh[k] * St).sum(), v)[0]
        return J, g


def exact(case, seed):
    if case["kind"] == "serve":
        return None  # a closed loop: rounding in one step travels through all that follow
    out = []
    for w in _worlds(case, seed):
        e = _Exact(copy.deepcopy(w))
        V = torch.as_tensor(w["V0"].astype(float)).to(e.dev)
        if case["kind"] == "grad":
            J, g = e.gradient(V, 0)
            return {"J": J, "grad": g}
        with torch.no_grad():
            out.append(e.step(V, 0))
    if case["kind"] == "batch":
        return {"V": [v for v, _ in out], "u0": torch.stack([u for _, u in out])}
    return {"V": out[0][0], "u0": out[0][1]}
