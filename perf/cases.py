"""What a user of this package has it do, as cases that can be timed and checked.

Each case is one call sequence through the package's public entry points on a two-star system (or
a batch of them) drawn from a seed:

* ``step``: ``System.step(steps)``, the leap-frog run of one system, in every precision mode and
  under both element laws;
* ``energy``: ``System.diagnostics(with_pe=True)``, the conserved quantities that a run is watched
  by, with the O(n^2) potential energy;
* ``batch``: one replay of a captured graph that advances many systems together, the round of the
  batch server;
* ``create``: ``System(...)`` from host arrays, what every request of a server and every start of
  a run pays: upload, sorted order and the initial accelerations.

``exact`` gives the same results from plain FP64 PyTorch.
"""

import math

import numpy as np
import torch

import paper_2303_12166_amd as nb

DT = 1e-4
GROWTH = 1e-4
R1, R2 = 0.30, 0.20


def listed():
    def case(name, kind, n, **kw):
        c = {"name": name, "kind": kind, "n": n, "q": 0.5, "mode": "kahan", "law": "contact",
             "steps": 1}
        c.update(kw)
        return c

    return [
        # the smallest system the model is run at (trajectory checks): launches and latency count
        case("step-2048", "step", 2048, steps=10),
        # a small request run alone; an odd size
        case("step-7001", "step", 7001, q=0.7, steps=10),
        # the mid-size and lobe-filling run
        case("step-65536", "step", 65536, steps=2),
        # the headline run
        case("step-262144", "step", 262144, q=0.3),
        # the paper's own velocity-dependent element law: a small request and a ragged mid size
        case("step-paper-3001", "step", 3001, q=0.4, law="paper", steps=10),
        case("step-paper-40009", "step", 40009, q=0.8, law="paper", steps=2),
        # the FP64 reference mode that FP32 runs are checked against
        case("step-fp64-4096", "step", 4096, mode="fp64", steps=10),
        case("step-fp64-50021", "step", 50021, q=0.3, mode="fp64"),
        # the plain FP32 mode of the precision study
        case("step-plain-131072", "step", 131072, q=0.8, mode="plain"),
        # the energy record of the precision study
        case("energy-131072", "energy", 131072, q=0.8),
        # a round of the batch server: ten steps of the small systems it serves together
        case("batch-24", "batch", 4096, n_max=32768, count=24, steps=10),
        # a request's or a run's start, from host arrays
        case("create-32768", "create", 32768),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    q = round(rng.uniform(0.1, 1.0), 3)
    kind = rng.choice(["step", "step", "step", "step", "energy", "batch", "create"])
    c = {"kind": kind, "n": 0, "q": q, "mode": "kahan", "law": "contact", "steps": 1}
    if kind == "step":
        c["mode"], c["law"] = rng.choice([("kahan", "contact"), ("kahan", "contact"),
                                          ("kahan", "paper"), ("fp64", "contact"),
                                          ("fp64", "paper"), ("plain", "contact")])
        top = {"kahan": 262144, "fp64": 131072, "plain": 131072}[c["mode"]]
        c["n"] = size(2048, top if c["law"] == "contact" else top // 2)
        c["steps"] = 10 if c["n"] <= 16384 else (2 if c["n"] <= 65536 else 1)
    elif kind == "energy":
        c["mode"] = rng.choice(["kahan", "fp64"])
        c["law"] = rng.choice(["contact", "paper"])
        c["n"] = size(2048, 131072)
    elif kind == "batch":
        c["mode"] = rng.choice(["kahan", "kahan", "fp64"])
        c["n"] = size(2048, 4096)
        c["n_max"] = size(8192, 16384 if c["mode"] == "fp64" else 32768)
        c["count"] = rng.randint(4, 32)
        c["steps"] = 10 if c["mode"] == "kahan" else 2
    else:
        c["mode"] = rng.choice(["kahan", "fp64"])
        c["n"] = size(2048, 131072)
    return c


# ------------------------------------------------------------------ inputs


def _ball(rng, count, radius, cx):
    d = rng.standard_normal((count, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    p = d * (radius * np.cbrt(rng.random(count)))[:, None]
    p -= p.mean(axis=0)
    p[:, 0] += cx
    return p


def _binary(n, q, seed, noise):
    """Two uniform balls in rigid rotation about their barycentre, total mass 1 + q, separation 1;
    ``noise``: velocity noise, so that pairs converge and separate (the paper's law)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    n2 = int(math.floor(n * q / (1.0 + q)))
    n1 = n - n2
    c1, c2 = -n2 / n, n1 / n
    pos = np.concatenate([_ball(rng, n1, R1, c1), _ball(rng, n2, R2, c2)])
    omega = math.sqrt(1.0 + q)
    vel = np.zeros_like(pos)
    vel[:, 0], vel[:, 1] = -omega * pos[:, 1], omega * pos[:, 0]
    if noise:
        vel += noise * rng.standard_normal(vel.shape)
    m = (1.0 + q) / n
    D1, D2 = (2.0 * R * (0.74 / k) ** (1.0 / 3.0) for R, k in ((R1, n1), (R2, n2)))
    return {"pos": pos.astype(np.float32), "vel": vel.astype(np.float32), "n": n, "n1": n1, "q": q,
            "m": m, "D1": D1, "D2": D2}


def _law_params(b, law):
    """Softening and repulsion of the paper's law, with a net force that is repulsive in contact."""
    if law != "paper":
        return {"law": "contact", "eps": 0.0, "gamma": 0.0, "beta": 1.0}
    gamma = 200.0 * b["m"] ** 2 / (b["D1"] ** 2 * math.pi * (0.5 * b["D1"]) ** 3)
    return {"law": "paper", "eps": 0.1 * b["D1"], "gamma": gamma, "beta": 0.5}


def _inputs(case, seed):
    return _binary(case["n"], case["q"], seed, 0.05 if case["law"] == "paper" else 0.0)


def _batch_inputs(case, seed):
    """Sizes log-uniform in [n, n_max] on multiples of 64 and mass ratios in [0.1, 1]. The first and
    the last size are the range's ends, and the sizes are the case's own, not the seed's."""
    rng = np.random.Generator(np.random.PCG64(case["n"] + case["n_max"] + case["count"]))
    u = np.concatenate([[0.0], rng.random(case["count"] - 2), [1.0]])
    sizes = [64 * max(1, int(round(case["n"] * (case["n_max"] / case["n"]) ** t / 64.0))) for t in u]
    return [_binary(n, float(q), seed * 1000 + k, 0.0)
            for k, (n, q) in enumerate(zip(sizes, rng.uniform(0.1, 1.0, case["count"])))]


def _system(b, mode, law):
    return nb.System(b["pos"], b["vel"], b["n1"], G=1.0, m=b["m"], dt=DT, D1=b["D1"], D2=b["D2"],
                     q=b["q"], a=1.0, R2_0=R2, growth_rate=GROWTH, growth_on=True, mode=mode,
                     **_law_params(b, law))


class _Batch:
    """Systems whose state arrays are slices of one tensor per quantity, and a captured graph."""

    def __init__(self, inputs, mode, steps):
        dtype = torch.float64 if mode == "fp64" else torch.float32
        total = sum(b["n"] for b in inputs)
        self.stream = torch.cuda.current_stream()
        pos = np.concatenate([b["pos"] for b in inputs])
        vel = np.concatenate([b["vel"] for b in inputs])
        cols = [np.ascontiguousarray(a[:, c]) for a in (pos, vel) for c in range(3)]
        self.arrays = [torch.from_numpy(c).to(device="cuda", dtype=dtype) for c in cols]
        self.arrays += [torch.zeros(total, dtype=dtype, device="cuda") for _ in range(3)]
        self.side = torch.zeros(total, dtype=torch.int8, device="cuda")
        self.scratch, self.handles, self.graph = [], [], None
        at = 0
        for b in inputs:
            p = nb.NbParams(n=b["n"], n1=b["n1"], G=1.0, m=b["m"], dt=DT, D1=b["D1"], D2=b["D2"],
                            q=b["q"], a=1.0, R2_0=R2, growth_rate=GROWTH, growth_on=1,
                            mode=nb.MODES[mode], law=nb.LAWS["contact"], pad=0, eps=0.0,
                            gamma=0.0, beta=1.0)
            need = nb.nb_scratch_bytes(p)
            s = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
            base = s.data_ptr() + (-s.data_ptr()) % 256
            ptrs = [t[at:].data_ptr() for t in self.arrays]
            names = ("x", "y", "z", "vx", "vy", "vz", "ax", "ay", "az")
            buffers = nb.NbBuffers(side=self.side[at:].data_ptr(), scratch=base,
                                   scratch_bytes=need, **dict(zip(names, ptrs)))
            self.scratch.append(s)
            self.handles.append(nb.nb_create(p, buffers, self.stream))
            at += b["n"]
        self.graph = nb.nb_graph_create(self.handles, steps, self.stream)

    def __del__(self):
        self.stream.synchronize()
        if self.graph is not None:
            nb.nb_graph_destroy(self.graph)
        for h in self.handles:
            nb.nb_destroy(h)


def prepare(case, seed):
    if case["kind"] == "batch":
        return case, _Batch(_batch_inputs(case, seed), case["mode"], case["steps"])
    b = _inputs(case, seed)
    if case["kind"] == "create":
        return case, b
    return case, _system(b, case["mode"], case["law"])


def run(state):
    case, s = state
    if case["kind"] == "step":
        s.step(case["steps"])
        return [s.x, s.y, s.z, s.vx, s.vy, s.vz, s.ax, s.ay, s.az, s.side]
    if case["kind"] == "energy":
        d = s.diagnostics(with_pe=True)
        return [d["com"], d["P"], d["L"], d["KE"], d["PE"], d["E"], d["step"], d["n_past_L1"]]
    if case["kind"] == "batch":
        nb.nb_graph_launch(s.graph, s.stream)
        return s.arrays + [s.side]
    made = _system(s, case["mode"], case["law"])
    return [made.x, made.y, made.z, made.vx, made.vy, made.vz, made.ax, made.ay, made.az,
            made.side]


def work(case):
    """Per unordered pair: the separation (3), its square (5), the law's scalar (about 5: root,
    powers, the contact choice; 12 under the paper's law) and both elements' sums (12; one add for
    the energy)."""
    elem = 8 if case["mode"] == "fp64" else 4
    if case["kind"] == "batch":
        sizes = [b["n"] for b in _batch_inputs(dict(case), 0)]
    else:
        sizes = [case["n"]]
    scalar = 12 if case["law"] == "paper" else 5
    pairs = sum(n * (n - 1) / 2.0 for n in sizes)
    n = sum(sizes)
    if case["kind"] == "energy":
        return {"bytes": float(n * 6 * elem), "flops": pairs * (8 + scalar + 1)}
    flops = pairs * (8 + scalar + 12) * case["steps"]
    if case["kind"] == "create":
        return {"bytes": float(n * (2 * 12 + 9 * elem)), "flops": flops}
    return {"bytes": float(n * (9 + 9) * elem), "flops": flops}


# ------------------------------------------------------------------ FP64 reference


def _chunks(n1, n, rows):
    for lo, hi in ((0, n1), (n1, n)):
        for i in range(lo, hi, rows):
            yield i, min(i + rows, hi)


def _blocks(X, n1, D, rows=None):
    """(i0, i1, j0, j1, d, r2, diameter) over row chunks of one star and columns of one star."""
    n = X.shape[1]
    rows = rows or max(1, min(4096, (1 << 28) // max(n, 1)))
    for i0, i1 in _chunks(n1, n, rows):
        for js, (j0, j1) in enumerate(((0, n1), (n1, n))):
            if j0 == j1:
                continue
            r2 = None
            for c in range(3):
                d = X[c, None, j0:j1] - X[c, i0:i1, None]
                r2 = d * d if r2 is None else r2.addcmul_(d, d)
            same = None
            if j0 <= i0 < j1:
                same = torch.arange(i0, i1, device=X.device)
            yield i0, i1, j0, j1, r2, same, 0.5 * (D[1 if i0 >= n1 else 0] + D[js])


def _accel(X, V, b, D, law):
    A = torch.zeros_like(X)
    gc = law["gamma"] * math.pi / (12.0 * b["m"] ** 2)
    for i0, i1, j0, j1, r2, same, Dij in _blocks(X, b["n1"], D):
        if same is not None:
            r2[same - i0, same - j0] = 1.0
        if law["law"] == "contact":
            w = r2.rsqrt_()
            s = torch.minimum(w * w * w, 11.0 / Dij ** 3 - (10.0 / Dij ** 2) * w)
        else:
            r = r2.sqrt_()
            s = 1.0 / ((r + law["eps"]) ** 2 * r)
            u = (Dij - r).clamp_(min=0.0)
            dot = torch.zeros_like(r)
            for c in range(3):
                dot += (V[c, None, j0:j1] - V[c, i0:i1, None]) * (X[c, None, j0:j1] -
                                                                 X[c, i0:i1, None])
            g = torch.where(dot < 0.0, gc, gc * law["beta"])
            s -= g * u * u * (r + 2.0 * Dij) / r
        if same is not None:
            s[same - i0, same - j0] = 0.0
        for c in range(3):
            d = X[c, None, j0:j1] - X[c, i0:i1, None]
            A[c, i0:i1] += (s * d).sum(dim=1)
    return A * b["m"]


def _lobe(q):
    c = q ** (1.0 / 3.0)
    return 0.49 * c * c / (0.69 * c * c + math.log(1.0 + c))


def _state(b, device):
    X = torch.from_numpy(np.ascontiguousarray(b["pos"].T.astype(np.float64))).to(device)
    V = torch.from_numpy(np.ascontiguousarray(b["vel"].T.astype(np.float64))).to(device)
    return X, V


def _leapfrog(b, law, steps, device):
    X, V = _state(b, device)
    D, grown = [b["D1"], b["D2"]], True
    A = _accel(X, V, b, D, law)
    for _ in range(steps):
        V = V + (0.5 * DT) * A
        X = X + DT * V
        A = _accel(X, V, b, D, law)
        V = V + (0.5 * DT) * A
        grown = grown and R2 * D[1] / b["D2"] <= _lobe(b["q"])
        if grown:
            D[1] *= 1.0 + GROWTH
    return [*X, *V, *A]


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    if case["kind"] == "batch":
        law = _law_params(None, "contact")
        parts = [_leapfrog(b, law, case["steps"], device) for b in _batch_inputs(case, seed)]
        return [torch.cat(p) for p in zip(*parts)] + [None]
    b = _inputs(case, seed)
    law = _law_params(b, case["law"])
    if case["kind"] == "create":
        return _leapfrog(b, law, 0, device) + [None]
    if case["kind"] == "step":
        return _leapfrog(b, law, case["steps"], device) + [None]
    X, V = _state(b, device)
    pe = 0.0
    A = b["m"] ** 2
    for i0, i1, j0, j1, r2, same, D in _blocks(X, b["n1"], [b["D1"], b["D2"]]):
        if same is not None:
            r2[same - i0, same - j0] = 1.0
        r = r2.sqrt_()
        if law["law"] == "contact":
            U = torch.where(r >= D, -A / r,
                            A * (11.0 * r * r - 20.0 * D * r + 7.0 * D * D) / (2.0 * D ** 3))
        else:
            u = (D - r).clamp_(min=0.0)
            U = -A / (r + law["eps"]) + law["gamma"] * math.pi / 48.0 * u ** 3 * (r + 3.0 * D)
        if same is not None:
            U[same - i0, same - j0] = 0.0
        pe += 0.5 * float(U.sum())
    m, n = b["m"], b["n"]
    com = X.sum(dim=1) / n
    P = m * V.sum(dim=1)
    L = m * torch.linalg.cross(X, V, dim=0).sum(dim=1)
    ke = 0.5 * m * float((V * V).sum())
    return [com.cpu().numpy(), None, L.cpu().numpy(), ke, pe, ke + pe, None, None]
