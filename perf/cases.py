"""The work that a user has this library do, as cases to time: stepping one
particle system or a batch of them (exact interaction, every precision mode),
stepping with the learned surrogate, training it and applying it to rows.

A context is made once with a horizon far beyond the steps taken here, and a
pass continues it by `steps` ticks, as a program that steps in pieces and looks
at the particles in between does: it reads them in place, in the tensor that
it has bound as the context's state."""
import math

import numpy as np
import torch

from paper_2105_09688_amd import workloads as W

D2, K2 = 2, 32  # surrogate cases: state dimension, random-Fourier moments
LONG = 2.0 ** 30  # horizon in steps


# ---------------------------------------------------------------------- cases
def listed():
    return [
        # the small parity run (10 ensembles of 1000 particles): the smallest calls, bound by
        # latency, in the two precisions that it is run in
        dict(name="small_fp64", kind="run", model="gauss1", precision="fp64", N=1000, ens=10, level="8", steps=32),
        dict(name="small_fp32k", kind="run", model="gauss1", precision="fp32_kahan", N=1000, ens=10, level="8", steps=32),
        # the Ginzburg-Landau family with the mean in the implicit part (no pair term), at two step sizes on one path
        dict(name="gl_v2_two_h", kind="run", model="gl2", precision="fp32_kahan", N=1000, ens=5, level="6,7", steps=32),
        # one middle-sized system of a ragged size
        dict(name="d1_8191_fp32k", kind="run", model="gauss1", precision="fp32_kahan", N=8191, ens=1, level="10", steps=8),
        # the single-GPU case of the benchmark, in its precision and in FP64
        dict(name="d1_65536_fp32k", kind="run", model="gauss1", precision="fp32_kahan", N=65536, ens=1, level="10", steps=4),
        dict(name="d1_65536_fp64", kind="run", model="gauss1", precision="fp64", N=65536, ens=1, level="10", steps=4),
        # the batched case: 64 ensembles of 2^10 .. 2^16 particles at five step sizes, one period of them
        dict(name="batched_64x5", kind="run", model="gauss1", precision="fp32_kahan", N=65536, ens=64, level="4,5,6,7,8", steps=16),
        # the precision study in three dimensions: plain FP32 sums at full size, FP64 at a ragged size
        dict(name="d3_262144_fp32", kind="run", model="gauss3", precision="fp32", N=262144, ens=1, level="10", steps=1),
        dict(name="d3_50021_fp64", kind="run", model="gauss3", precision="fp64", N=50021, ens=1, level="10", steps=1),
        # the surrogate in two dimensions: network ticks at full size, and one exact check with the 15 ticks after it
        dict(name="surrogate_1048576", kind="surrogate", N=1048576, check=0, steps=8),
        dict(name="surrogate_check_65536", kind="surrogate", N=65536, check=16, steps=16),
        # training the surrogate's network (batches as in the surrogate study)
        dict(name="train_4096", kind="train", batch=4096, samples=262144, steps=64),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi)))) | rng.choice((0, 1))

    prec = rng.choice(("fp32_kahan", "fp32_kahan", "fp64", "fp32"))
    pick = rng.choice(("one", "one", "one", "many", "many", "batch", "free", "d2", "d3", "surrogate", "check", "train", "rows"))
    if pick == "one":
        return dict(kind="run", model="gauss1", precision=prec, N=size(512, 131072), ens=1, level="10", steps=rng.randint(2, 8),
                    ell=round(2.0 ** rng.uniform(-1.5, 1.5), 3))
    if pick == "many":
        return dict(kind="run", model="gauss1", precision=prec, N=size(50, 2000), ens=rng.randint(2, 16), level="8",
                    steps=rng.randint(8, 64))
    if pick == "batch":
        return dict(kind="run", model="gauss1", precision="fp32_kahan", N=size(2048, 16384), ens=rng.randint(4, 32), level="5,6,7",
                    steps=4 * rng.randint(1, 3))
    if pick == "free":
        return dict(kind="run", model=rng.choice(("gl2", "ou")), precision=prec, N=size(100, 100000), ens=rng.randint(1, 8), level="7",
                    steps=rng.randint(8, 32))
    if pick in ("d2", "d3"):
        return dict(kind="run", model="gauss" + pick[1], precision=prec, N=size(500, 60000), ens=1, level="10", steps=1)
    if pick == "surrogate":
        return dict(kind="surrogate", N=size(4000, 1000000), check=0, steps=rng.randint(4, 12))
    if pick == "check":
        return dict(kind="surrogate", N=size(2000, 60000), check=16, steps=16)
    if pick == "train":
        return dict(kind="train", batch=64 * size(4, 128), samples=2 ** rng.randint(14, 18), steps=rng.randint(16, 64))
    return dict(kind="rows", rows=size(1000, 500000))


def sizes(case):
    """Particles of each ensemble; ensembles of a batch (several step sizes at once) are of uneven size up to N."""
    if "," in case["level"] and case["model"] == "gauss1":
        return [min(n, case["N"]) for n in W.batched_sizes(case["ens"], 10, int(math.log2(case["N"])))]
    return [case["N"]] * case["ens"]


def workload(case, seed):
    if case["kind"] == "surrogate":
        w = W.surrogate_d2(N=case["N"])
        h = w["systems"][0][2]
    else:
        levels = [int(l) for l in case["level"].split(",")]
        h = 2.0 ** -max(levels)
        w = {"gauss1": lambda: W.small_parity(n_ens=1, h_fine=h / 16), "gauss2": lambda: W.surrogate_d2(h_fine=h / 16),
             "gauss3": W.precision_d3, "gl2": lambda: W.ginzburg_landau(version=2, h_fine=h / 16),
             "ou": lambda: W.ou(x0_std=0.5, h=h, h_fine=h / 4)}[case["model"]]()
        w = W.with_systems(w, [(N, e, 2.0 ** -l) for e, N in enumerate(sizes(case)) for l in levels])
    if "ell" in case:
        w["b"]["ell"] = case["ell"]
    w["seed"] = int(seed)
    w["T"] = LONG * max(s[2] for s in w["systems"])
    return w


def weights(d, seed):
    """Network weights of the size that training starts from and stays near (flat layout of include/ssm.h)."""
    from paper_2105_09688_amd.ssm import mlp_init
    return mlp_init(d, seed=seed)


def rows(n, d, seed):
    """Rows [y, moments] and a smooth target of the interaction's size, as sampled from a cloud."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    y = torch.randn(n, d, generator=g, device="cuda")
    U = torch.cat([y, torch.rand(n, K2, generator=g, device="cuda") * 2 - 1], dim=1)
    return U, -y * torch.exp(-0.5 * (y * y).sum(1, keepdim=True)) + 0.1 * U[:, d:2 * d]


def prepare(case, seed):
    from paper_2105_09688_amd.ssm import SSM
    if case["kind"] == "rows":
        return dict(case=case, U=rows(case["rows"], D2, seed)[0], master=torch.tensor(weights(D2, seed), device="cuda"))
    if case["kind"] == "train":
        U, T = rows(case["samples"], D2, seed)
        return dict(case=case, U=U, T=T, master=torch.tensor(weights(D2, seed), device="cuda"), seed=int(seed))
    s = SSM(workload(case, seed), precision=case.get("precision", "fp32_kahan"))
    if case["kind"] == "surrogate":
        s.surrogate_load(weights(D2, seed))
        if case["check"] == 0:  # between checks: the context resumes on a tick that is none
            s.set_state(0, s.state(0), step=1)
        s.surrogate_enable(check_every=case["check"] or 2 ** 30, tol=1e9, mode="residual")
    X = s.bind_state()
    s.sync()
    return dict(case=case, ssm=s, X=X)


def run(state):
    from paper_2105_09688_amd.ssm import mlp_forward, mlp_train
    case = state["case"]
    if case["kind"] == "rows":
        return mlp_forward(D2, state["master"], state["U"])
    if case["kind"] == "train":
        master = state["master"].clone()
        hist = mlp_train(D2, master, state["U"], state["T"], steps=case["steps"], batch=case["batch"], lr=1e-3, seed=state["seed"])
        return {"master": master, "loss": hist}
    state["ssm"].step(case["steps"])
    return state["X"]


def work(case):
    """Inputs and outputs once.  Arithmetic: the network's products; else per particle and step about 40 operations a
    normal, 60 for the implicit step and 20 per component.  Interaction sums are counted at one evaluation per
    particle: that they are made of N^2 terms is how they are defined and not what computing them needs."""
    net = 2 * (K2 + 2 * D2 + 64 + 64 + D2) * 64
    n_par = (K2 + 2 * D2) * 64 + 2 * 64 * 64 + 64 * D2 + 3 * 64 + D2
    if case["kind"] == "rows":
        return {"bytes": 4.0 * (case["rows"] * (2 * D2 + K2) + n_par), "flops": float(case["rows"] * net)}
    if case["kind"] == "train":
        n = case["steps"] * case["batch"]
        return {"bytes": 4.0 * (n * (2 * D2 + K2) + 2 * n_par), "flops": 3.0 * n * net}
    w = workload(case, 0)
    h_min, d = min(s[2] for s in w["systems"]), w["d"]
    elt = 8 if case.get("precision") == "fp64" else 4
    flops = 0.0
    for N, _, h in w["systems"]:
        stride, r = round(h / h_min), round(h / w["h_fine"])
        flops += -(-case["steps"] // stride) * N * (40 * r * d + 60 + 20 * d + (net if case["kind"] == "surrogate" else 0))
    return {"bytes": 2.0 * d * elt * sum(s[0] for s in w["systems"]), "flops": flops}


# ------------------------------------------------- the same in 64 bits, in plain torch
def _mulhilo(c, x):
    M = 0xFFFFFFFF
    a0, a1, b0, b1 = c & M, c >> 32, x & M, (x >> 32) & M
    t = a0 * b0
    u = a1 * b0 + ((t >> 32) & M)
    v = a0 * b1 + (u & M)
    return a1 * b1 + ((u >> 32) & M) + ((v >> 32) & M), (v << 32) | (t & M)


def _signed(v):
    v &= 2 ** 64 - 1
    return v - 2 ** 64 if v >= 2 ** 63 else v


def _philox(x0, x1, x2, x3, k0, k1=0):
    """Philox4x64-10 (Salmon et al., SC'11) on int64 tensors."""
    for r in range(10):
        ah, al = _mulhilo(0xD2E7470EE14C6C93, x0)
        bh, bl = _mulhilo(0xCA5A826395121157, x2)
        x0, x1, x2, x3 = bh ^ x1 ^ _signed(k0 + r * 0x9E3779B97F4A7C15), bl, ah ^ x3 ^ _signed(k1 + r * 0xBB67AE8584CAA73B), al
    return x0, x1, x2, x3


def _normals(seed, tag, i, b, e):
    """Four standard normals per (particle, block) [..., 4]."""
    z = torch.zeros_like(i + b)
    w = _philox(z + i, z + b, z + e, z + (tag << 32), seed)
    u = [(((x >> 11) & (2 ** 53 - 1)).double() + 0.5) * 2.0 ** -53 for x in w]
    out = []
    for p in (0, 2):
        rad, ang = torch.sqrt(-2.0 * torch.log(u[p])), 2.0 * math.pi * u[p + 1]
        out += [rad * torch.cos(ang), rad * torch.sin(ang)]
    return torch.stack(out, dim=-1)


def _increment(w, i, e, n, r):
    """dW [d][N] of step n: the step's r fine increments added up."""
    d = w["d"]
    q0, q1 = n * r * d, (n + 1) * r * d
    total = torch.zeros(d, i.numel(), dtype=torch.float64, device=i.device)
    for b in range(q0 // 4, -(-q1 // 4)):
        z = _normals(w["seed"], 0, i, torch.full_like(i, b), e)
        for s in range(4):
            if q0 <= 4 * b + s < q1:
                total[(4 * b + s) % d] += z[:, s]
    return math.sqrt(w["h_fine"]) * total


def _pairs(Y, ell):
    d, N = Y.shape
    K = torch.empty_like(Y)
    step = max(1, min(N, 2 ** 26 // N))
    for a in range(0, N, step):
        z = [Y[k][None, :] - Y[k][a:a + step, None] for k in range(d)]
        t = z[0] * z[0]
        for k in range(1, d):
            t.addcmul_(z[k], z[k])
        t.mul_(-0.5 / ell ** 2).exp_()
        for k in range(d):
            K[k, a:a + step] = z[k].mul_(t).sum(1) / N
    return K


def _implicit(w, h, X):
    """Y with Y = X + h v(Y, mu^X): a non-negative multiple of X + h lam mean(X) by one scalar cubic."""
    v = w["v"]
    q = X + h * v["lam"] * X.mean(1, keepdim=True)
    alpha, ha = 1.0 - h * (v["rho"] - v["kappa"] * float((X * X).sum(0).mean())), h * v["a"]
    n = torch.sqrt((q * q).sum(0))
    s = n / alpha
    for _ in range(60 if ha else 0):
        s = s - (ha * s ** 3 + alpha * s - n) / (3.0 * ha * s * s + alpha)
    return q * torch.where(n > 0, s / torch.where(n > 0, n, 1.0), 1.0 / alpha)


def _net(master, d, Y, mom):
    """Network output [d][N]: weights rounded to bfloat16, input [hi(y), lo(y), moments]."""
    m, at = torch.tensor(master, device="cuda"), 0
    hi = Y.float().bfloat16()
    x = torch.cat([hi.double().T, (Y.float() - hi.float()).bfloat16().double().T, mom.expand(Y.shape[1], -1)], dim=1)
    for out in (64, 64, 64, d):
        Wt = m[at:at + out * x.shape[1]].bfloat16().double().view(out, -1)
        at += Wt.numel()
        x = x @ Wt.T + m[at:at + out].double()
        at += out
        if at < m.numel():
            x = x * torch.sigmoid(x)
    return x.T


def _step(w, N, e, h, n, X, interaction):
    i = torch.arange(N, device="cuda")
    col = lambda v: torch.tensor(v, dtype=torch.float64, device="cuda")[:, None]  # noqa: E731
    Y = _implicit(w, h, X)
    b, s, mean = w["b"], w["sigma"], Y.mean(1, keepdim=True)
    drift = b["c0"] * Y + b["lam"] * mean
    if b["g"]:
        drift = drift + b["g"] * interaction(Y)
    dW = _increment(w, i, e, n, round(h / w["h_fine"]))
    return Y + h * drift + (col(s["s0"]) + col(s["s1"]) * Y + col(s["s2"]) * mean) * dW


def _start(w, N, e):
    i = torch.arange(N, device="cuda")
    z = _normals(w["seed"], 1, i, torch.zeros_like(i), e)[:, :w["d"]].T
    col = lambda v: torch.tensor(v, dtype=torch.float64, device="cuda")[:, None]  # noqa: E731
    return col(w["x0_mean"]) + col(w["x0_std"]) * z


def exact(case, seed):
    if case["kind"] == "rows":
        U = rows(case["rows"], D2, seed)[0].double()
        return _net(weights(D2, seed), D2, U[:, :D2].T, U[:, D2:]).T.contiguous()
    if case["kind"] == "train":
        return _train(case, seed)
    w = workload(case, seed)
    h_min, d = min(s[2] for s in w["systems"]), w["d"]
    parts = []
    for N, e, h in w["systems"]:
        X, stride = _start(w, N, e), round(h / h_min)
        if case["kind"] == "surrogate":
            X = _surrogate(case, w, N, e, h, X, weights(D2, seed))
        else:
            for t in range(0, case["steps"], stride):
                X = _step(w, N, e, h, t // stride, X, lambda Y: _pairs(Y, w["b"]["ell"]))
        parts.append(torch.cat([X, torch.zeros(d, -N % 256, dtype=torch.float64, device="cuda")], dim=1))
    return torch.cat(parts, dim=1)


def _surrogate(case, w, N, e, h, X, master):
    d, ell = w["d"], w["b"]["ell"]
    k = torch.arange(K2 // 2, device="cuda")
    omega = _normals(w["seed"], 3, k, torch.zeros_like(k), 0)[:, :d] / ell
    kept = {"r": 0.0, "t": 0}

    def interaction(Y):
        ph = omega @ Y
        s = _net(master, d, Y, torch.cat([torch.cos(ph).mean(1), torch.sin(ph).mean(1)])[None])
        s = s - s.mean(1, keepdim=True)
        if case["check"] and kept["t"] % case["check"] == 0:
            p = _pairs(Y, ell)
            kept["r"] = p - s
            return p
        return s + kept["r"]

    t0 = 0 if case["check"] else 1
    for t in range(t0, t0 + case["steps"]):
        kept["t"] = t
        X = _step(w, N, e, h, t, X, interaction)
    return X


def _train(case, seed):
    U, T = (x.double() for x in rows(case["samples"], D2, seed))
    m, at, params = torch.tensor(weights(D2, seed), device="cuda").double(), 0, []
    for out, inp in ((64, 2 * D2 + K2), (64, 64), (64, 64), (D2, 64)):
        for shape in ((out, inp), (out,)):
            n = int(np.prod(shape))
            params.append(m[at:at + n].view(shape).clone().requires_grad_(True))
            at += n
    hi = U[:, :D2].float().bfloat16()
    X = torch.cat([hi.double(), (U[:, :D2].float() - hi.float()).bfloat16().double(), U[:, D2:]], dim=1)
    opt = torch.optim.Adam(params, lr=1e-3, betas=(0.9, 0.999), eps=1e-8)
    r = torch.arange(case["batch"], device="cuda")
    z, hist = torch.zeros_like(r), []
    for t in range(case["steps"]):
        at = _philox(r, z + t, z, z + (4 << 32), int(seed))[0] & (case["samples"] - 1)
        x = X[at]
        for q in range(4):
            x = x @ params[2 * q].T + params[2 * q + 1]
            x = x * torch.sigmoid(x) if q < 3 else x
        loss = (x - T[at]).square().sum() / case["batch"]
        opt.zero_grad()
        loss.backward()
        opt.step()
        hist.append(float(loss))
    return {"master": torch.cat([p.detach().reshape(-1) for p in params]), "loss": np.array(hist)}
