"""Performance cases: the work that programs built on this library have it do.

Every case is one pass through the public entry points of
``paper_1211_2293_amd.treecode.Treecode`` on seeded synthetic bodies:

  op "forces"     build, moments, walk and forces of bodies held in device memory
  op "step"       one kick-drift-kick leapfrog step of a running simulation
  op "fmm"        build, moments, traversal and forces of the fast multipole method
  op "learned"    build, moments and the walk with the learned closure
  op "residuals"  training pairs for a set of target bodies on a built tree
  op "train"      one training step of the closure's network on a minibatch

The sizes are those of the repository's workloads and of the paper's runs
(10,000, 50,000 and 100,000 bodies, §4.1), from 4,096 to 16,777,216 bodies,
and odd ones beside them.
"""
import math

import numpy as np
import torch

from paper_1211_2293_amd.treecode import MLP_NPARAM, Treecode

DIRECT_MAX = 270_000      # bodies up to which the FP64 direct sum takes a few seconds


def listed():
    return [
        # the smallest calls: FP64 state in small leaves, where launches and latency are all there is
        {"name": "cube-4k-f64", "op": "forces", "bodies": "cube", "n": 4096, "dim": 3, "f64": True,
         "theta": 0.5, "eps": 1e-3, "leaf": 8, "order": 1},
        # time steps at two of the paper's three sizes
        {"name": "plummer-10k-step", "op": "step", "bodies": "plummer", "n": 10_000, "dim": 3, "f64": False,
         "theta": 0.5, "eps": 1e-2, "leaf": 16, "dt": 1e-3},
        {"name": "plummer-50k-step", "op": "step", "bodies": "plummer", "n": 50_000, "dim": 3, "f64": False,
         "theta": 0.5, "eps": 1e-2, "leaf": 16, "dt": 1e-3},
        # a ragged size near the paper's third, with quadrupole cells
        {"name": "plummer-100k-quad", "op": "forces", "bodies": "plummer", "n": 99_991, "dim": 3, "f64": False,
         "theta": 0.6, "eps": 1e-2, "leaf": 16, "order": 2},
        # the two-dimensional tree
        {"name": "disk-262k", "op": "forces", "bodies": "disk", "n": 262_144, "dim": 2, "f64": False,
         "theta": 0.5, "eps": 1e-2, "leaf": 16, "order": 1},
        # the benchmark's own time step
        {"name": "plummer-1m-step", "op": "step", "bodies": "plummer", "n": 1_048_576, "dim": 3, "f64": False,
         "theta": 0.5, "eps": 1e-2, "leaf": 16, "dt": 1e-3},
        # two colliding spheres
        {"name": "collision-4m", "op": "forces", "bodies": "two", "n": 4_194_304, "dim": 3, "f64": False,
         "theta": 0.5, "eps": 1e-2, "leaf": 16, "order": 1},
        # the largest run: clumps of very different density, unequal masses
        {"name": "clustered-16m-step", "op": "step", "bodies": "clustered", "n": 16_777_216, "dim": 3, "f64": False,
         "theta": 0.7, "eps": 1e-3, "leaf": 16, "dt": 5e-4},
        # the fast multipole method on its own tree of leaf size 64
        {"name": "fmm-1m", "op": "fmm", "bodies": "plummer", "n": 1_048_576, "dim": 3, "f64": False,
         "theta": 0.5, "eps": 1e-2, "leaf": 64},
        # forces with the learned closure: most learned cells kept, some falling back
        {"name": "learned-131k", "op": "learned", "bodies": "plummer", "n": 131_072, "dim": 3, "f64": False,
         "theta": 0.8, "theta_p": 0.5, "tau": 3e-2, "eps": 1e-2, "leaf": 16},
        # the closure's training data: a set of a fixed size, 256 pairs per target body
        {"name": "residuals-262k", "op": "residuals", "bodies": "plummer", "n": 262_144, "dim": 3, "f64": False,
         "theta": 0.9, "eps": 1e-2, "leaf": 16, "targets": 4096},
        # the closure's training step, run tens of thousands of times per network
        {"name": "train-4096", "op": "train", "batch": 4096, "rows": 262_144, "lr": 1e-3},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) | 1


def draw(rng):
    op = rng.choice(["step", "step", "step", "forces", "forces", "forces", "fmm", "learned", "residuals", "train"])
    if op == "train":
        return {"op": op, "batch": _log_int(rng, 512, 16_384), "rows": _log_int(rng, 65_536, 1_000_000), "lr": 1e-3}
    if op == "step":
        bodies = rng.choice(["plummer", "plummer", "two", "clustered"])
        n = _log_int(rng, 4096, 8_000_000)
        return {"op": op, "bodies": bodies, "n": n, "dim": 3, "f64": n < 500_000 and rng.random() < 0.25,
                "theta": round(rng.uniform(0.45, 0.8), 2), "eps": 1e-3 if bodies == "clustered" else 1e-2,
                "leaf": rng.choice([8, 16, 16, 32]), "dt": 5e-4}
    if op == "forces":
        bodies = rng.choice(["cube", "disk", "plummer", "two"])
        dim = 2 if bodies == "disk" else 3
        n = _log_int(rng, 4096, 4_000_000)
        return {"op": op, "bodies": bodies, "n": n, "dim": dim, "f64": n < 500_000 and rng.random() < 0.25,
                "theta": round(rng.uniform(0.45, 0.9), 2), "eps": 1e-2, "leaf": rng.choice([8, 16, 16, 32]),
                "order": 2 if dim == 3 and rng.random() < 0.25 else 1}
    if op == "fmm":
        return {"op": op, "bodies": rng.choice(["plummer", "cube"]), "n": _log_int(rng, 16_384, 1_048_575), "dim": 3,
                "f64": False, "theta": round(rng.uniform(0.45, 0.8), 2), "eps": 1e-2, "leaf": rng.choice([32, 64])}
    if op == "learned":
        return {"op": op, "bodies": "plummer", "n": _log_int(rng, 8192, 300_000), "dim": 3, "f64": False,
                "theta": round(rng.uniform(0.7, 0.9), 2), "theta_p": 0.5, "tau": rng.choice([1e-2, 3e-2, 1e9]),
                "eps": 1e-2, "leaf": 16}
    return {"op": op, "bodies": "plummer", "n": _log_int(rng, 32_768, 1_000_000), "dim": 3, "f64": False,
            "theta": round(rng.uniform(0.8, 0.9), 2), "eps": 1e-2, "leaf": 16, "targets": _log_int(rng, 256, 4096)}


# ---- inputs: FP64 draws on the GPU, rounded to the working type

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _directions(g, n):
    z = 2.0 * _rand(g, n) - 1.0
    p = 2.0 * math.pi * _rand(g, n)
    s = torch.sqrt(1.0 - z * z)
    return torch.stack([s * torch.cos(p), s * torch.sin(p), z], dim=1)


def _plummer(g, n, a, mass):
    """Positions and virial velocities of a Plummer sphere truncated at ten scale radii (G = 1)."""
    u = _rand(g, n).clamp_min(1e-12) * (1.0 + 0.01) ** -1.5
    r = 1.0 / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
    # speeds as a share q of the escape speed: density q^2 (1 - q^2)^(7/2), by its tabulated inverse
    q = torch.linspace(0.0, 1.0, 4097, device="cuda", dtype=torch.float64)
    cdf = torch.cumsum(q * q * (1.0 - q * q) ** 3.5, 0)
    cdf = cdf / cdf[-1].clone()
    at = torch.searchsorted(cdf, _rand(g, n)).clamp_max(4096)
    speed = q[at] * math.sqrt(2.0) * (1.0 + r * r) ** -0.25 * math.sqrt(mass / a)
    return _directions(g, n) * (r * a)[:, None], _directions(g, n) * speed[:, None]


def _bodies(case, seed):
    """(pos, vel, mass) of a case in its working type."""
    g, n = _gen(seed), case["n"]
    mass = torch.full((n,), 1.0 / n, device="cuda", dtype=torch.float64)
    if case["bodies"] == "cube":
        pos = _rand(g, n, 3)
        vel = torch.zeros_like(pos)
    elif case["bodies"] == "disk":
        pos = torch.randn(n, 2, generator=g, device="cuda", dtype=torch.float64)
        vel = torch.zeros_like(pos)
    elif case["bodies"] == "plummer":
        pos, vel = _plummer(g, n, 1.0, 1.0)
    elif case["bodies"] == "two":
        n1 = int(round(n / 1.3))
        p1, v1 = _plummer(g, n1, 1.0, 1.0)
        p2, v2 = _plummer(g, n - n1, 1.0, 0.3)
        p1[:, 0] -= 10.0 * 0.3 / 1.3
        p2[:, 0] += 10.0 / 1.3
        v1[:, 0] += 0.5
        v2[:, 0] -= 0.5
        pos, vel = torch.cat([p1, p2]), torch.cat([v1, v2])
        mass = mass * 1.3
    else:                                       # 32 clumps, Pareto masses
        mass = (1.0 - _rand(g, n)) ** (-1.0 / 2.35)
        mass = mass / mass.sum()
        radii = (10.0 ** (-2.0 + _rand(g, 32))).tolist()
        centres = 10.0 * _rand(g, 32, 3)
        ps, vs, o = [], [], 0
        for k in range(32):
            nk = n // 32 + (1 if k < n % 32 else 0)
            p, v = _plummer(g, nk, radii[k], float(mass[o:o + nk].sum()))
            ps.append(p + centres[k])
            vs.append(v)
            o += nk
        pos, vel = torch.cat(ps), torch.cat(vs)
    t = torch.float64 if case["f64"] else torch.float32
    return pos.to(t).contiguous(), vel.to(t).contiguous(), mass.to(t).contiguous()


def _network(seed):
    """Closure parameters (FP32, canonical order): seeded hidden layers and an output layer fitted to the
    quadrupole term of random cells, which is what a trained network mostly predicts."""
    r = np.random.default_rng(seed)
    w1 = r.uniform(-1, 1, (10, 64)) / math.sqrt(10)
    b1 = r.uniform(-0.5, 0.5, 64)
    w2 = r.uniform(-1, 1, (64, 64)) / 8.0
    b2 = r.uniform(-0.5, 0.5, 64)
    f, y = _pairs(r, 4096)
    gelu = lambda z: 0.5 * z * (1.0 + np.tanh(math.sqrt(2.0 / math.pi) * (z + 0.044715 * z ** 3)))  # noqa: E731
    h = gelu(gelu(f @ w1 + b1) @ w2 + b2)
    a = np.concatenate([h, np.ones((len(h), 1))], axis=1)
    w = np.linalg.solve(a.T @ a + 1e-3 * np.eye(65), a.T @ y)
    return np.concatenate([v.ravel() for v in (w1, b1, w2, b2, w[:64], w[64])]).astype(np.float32)


def _pairs(r, rows):
    """Features of random (body, cell) pairs and the quadrupole term in the network's units, FP64."""
    d = r.normal(size=(rows, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    u = d * r.uniform(1.2, 3.0, (rows, 1))
    q = r.normal(0.0, 0.08, (rows, 6))
    q[:, 2] = -q[:, 0] - q[:, 1]
    f = np.concatenate([u, q, r.uniform(1.0, 8.0, (rows, 1))], axis=1)
    qx = q[:, 0] * d[:, 0] + q[:, 3] * d[:, 1] + q[:, 4] * d[:, 2]
    qy = q[:, 3] * d[:, 0] + q[:, 1] * d[:, 1] + q[:, 5] * d[:, 2]
    qz = q[:, 4] * d[:, 0] + q[:, 5] * d[:, 1] + q[:, 2] * d[:, 2]
    dqd = qx * d[:, 0] + qy * d[:, 1] + qz * d[:, 2]
    return f, np.stack([qx, qy, qz], axis=1) - 2.5 * dqd[:, None] * d


def _training_set(case, seed):
    r = np.random.default_rng(seed)
    rows = case["rows"]
    f, y = _pairs(r, min(rows, 65_536))
    at = r.integers(0, len(f), rows)
    at[:len(f)] = np.arange(len(f))
    batches = 8
    order = np.concatenate([r.permutation(rows)[:case["batch"]] for _ in range(batches)]).astype(np.int32)
    params = np.concatenate([r.uniform(-1, 1, 640) / math.sqrt(10), np.zeros(64), r.uniform(-1, 1, 4096) / 8.0,
                             np.zeros(64), r.uniform(-1, 1, 192) / 8.0, np.zeros(3)]).astype(np.float32)
    return f[at].astype(np.float32), y[at].astype(np.float32), order, params


def prepare(case, seed):
    op = case["op"]
    if op == "train":
        feat, y, order, params = _training_set(case, seed)
        # the network lives in a context's workspace, beside the tree it corrects
        tc = Treecode(3)
        g = _gen(seed)
        pos = _rand(g, 4096, 3).float()
        mass = torch.full((4096,), 1.0 / 4096, device="cuda")
        tc.build(pos, mass)
        tc.mlp_load(torch.from_numpy(params).cuda())
        return {"case": case, "tc": tc, "keep": (pos, mass), "feat": torch.from_numpy(feat).cuda(),
                "y": torch.from_numpy(y).cuda(), "order": torch.from_numpy(order).cuda(), "at": 0,
                "grad": torch.empty(MLP_NPARAM, device="cuda")}
    pos, vel, mass = _bodies(case, seed)
    tc = Treecode(case["dim"], leaf_cap=case["leaf"])
    state = {"case": case, "tc": tc, "pos": pos, "vel": vel, "mass": mass}
    if op == "forces":
        tc.set_multipole(case["order"])
    elif op == "step":
        # a running simulation: the accelerations of the step before
        tc.build(pos, mass)
        tc.moments()
        tc.walk(case["theta"])
        tc.forces(1.0, case["eps"])
    elif op == "learned":
        tc.build(pos, mass)
        tc.mlp_load(torch.from_numpy(_network(seed)).cuda())
    elif op == "residuals":
        tc.build(pos, mass)
        tc.moments()
        at = torch.randperm(case["n"], generator=_gen(seed + 1), device="cuda")[:case["targets"]]
        state["targets"] = at.to(torch.int32)
    return state


def run(state):
    case, tc = state["case"], state["tc"]
    op = case["op"]
    if op == "step":
        tc.leapfrog(case["dt"], state["pos"], state["vel"])
        return state["pos"], state["vel"]
    if op == "train":
        b, k = case["batch"], state["at"]
        state["at"] = (k + 1) % 8
        tc.mlp_step(state["feat"], state["y"], state["order"][k * b:(k + 1) * b], lr=case["lr"], want_loss=False,
                    grad=state["grad"])
        return state["grad"]
    if op == "residuals":
        return tc.residuals(case["theta"], case["eps"], state["targets"], cap=256 * case["targets"])
    tc.build(state["pos"], state["mass"])
    tc.moments()
    if op == "fmm":
        tc.fmm_plan(case["theta"])
        return tc.fmm_forces(1.0, case["eps"])
    if op == "learned":
        return tc.forces_learned(case["theta"], case["theta_p"], case["tau"], 1.0, case["eps"])
    tc.walk(case["theta"])
    return tc.forces(1.0, case["eps"])


# ---- what a pass cannot do without

def _interactions(case):
    """List entries per body, about: what the group walks give on these bodies."""
    n, th = case["n"], case["theta"]
    if case["dim"] == 2:
        return min(n, 48.0 * math.log2(n) * (0.5 / th) ** 1.2)
    return min(n, 226.0 * math.log2(n) * (0.5 / th) ** 1.6)


def work(case):
    op = case["op"]
    if op == "train":
        b = case["batch"]
        net = 2 * (10 * 64 + 64 * 64 + 64 * 3)
        # rows, indices, the gradient, and the weights with both moments in and out
        return {"bytes": b * (4 + 40 + 12) + 4 * 5059 * 7, "flops": 3.0 * net * b}
    es, dim, n = (8 if case["f64"] else 4), case["dim"], case["n"]
    if op == "residuals":
        # the pairs written sum the bodies of about half of all accepted cells exactly
        return {"bytes": n * 32 + 256 * case["targets"] * 56, "flops": 10.0 * case["targets"] * n}
    if op == "step":
        nbytes = n * (es * (4 * dim + 1) + 4 * dim)
    else:
        nbytes = n * (es * (dim + 1) + 4 * (dim + 1))
    return {"bytes": nbytes, "flops": 20.0 * n * _interactions(case)}


# ---- the same in 64 bits: the direct sum over all bodies

def _direct(pos, mass, eps):
    """(acc, pot) of every body in FP64: the softened sum over all others."""
    x, m = pos.double(), mass.double()
    n, dim = x.shape
    cols = [x[:, a].contiguous() for a in range(dim)]
    acc = torch.empty_like(x)
    pot = torch.empty(n, dtype=torch.float64, device=x.device)
    rows = max(1, (1 << 26) // n)
    for i in range(0, n, rows):
        d = [c[None, :] - c[i:i + rows, None] for c in cols]
        r2 = d[0] * d[0]
        for c in d[1:]:
            r2.addcmul_(c, c)
        s = torch.rsqrt_(r2.add_(eps * eps))
        w = s * m
        pot[i:i + rows] = -(w.sum(1) - m[i:i + rows] / eps)
        w.mul_(s).mul_(s)
        for a in range(dim):
            acc[i:i + rows, a] = d[a].mul_(w).sum(1)
    return acc, pot


def exact(case, seed):
    op = case["op"]
    if op == "train":
        feat, y, order, params = _training_set(case, seed)
        at = torch.from_numpy(order[:case["batch"]].astype(np.int64))
        f, t = torch.from_numpy(feat)[at].double(), torch.from_numpy(y)[at].double()
        p = torch.from_numpy(params).double().requires_grad_(True)
        w1, b1, w2, b2, w3, b3 = torch.split(p, [640, 64, 4096, 64, 192, 3])
        gelu = lambda z: torch.nn.functional.gelu(z, approximate="tanh")  # noqa: E731
        h = gelu(gelu(f @ w1.view(10, 64) + b1) @ w2.view(64, 64) + b2) @ w3.view(64, 3) + b3
        ((h - t) ** 2).mean().backward()
        return p.grad
    if op == "residuals" or case["n"] > DIRECT_MAX:
        return None
    pos, vel, mass = _bodies(case, seed)
    acc, pot = _direct(pos, mass, case["eps"])
    if op != "step":
        return acc, pot
    dt = case["dt"]
    v = vel.double() + 0.5 * dt * acc
    x = pos.double() + dt * v
    a, _ = _direct(x, mass, case["eps"])
    return x, v + 0.5 * dt * a
