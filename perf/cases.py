"""Timed workloads of the library: the calls its users make, over the sizes they make them at.

Every case runs through the package's public entry points.  Kinds:
  wave     a running lattice Boltzmann handle (one or more driven boxes with one object each):
           `steps` more time steps and the time-averaged force; returns force, sample count and
           the populations in place
  predict  surrogate queries outside the trusted box, answered by whole lattice runs
  cavity   the calibration run that places an object in the standing wave
  infer    the surrogate network on a batch (device tensors, or host arrays as the particle
           integrator passes them)
  train    Adam steps of the network on a force data set, then its weights

listed() names the cases, draw() makes more of the same ranges, prepare() makes what a program
holds before the call, run() is one pass, work() the least bytes and operations of a pass, and
exact() the results in FP64 in plain torch and numpy.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2404_02346_amd import LBWave, cavity_calibrate
from paper_2404_02346_amd.surrogate import MLP, Surrogate

WALL_PHI = 0.99       # damping of the two x walls
THICK = 4.0           # square thickness of the object's tanh profile
OFFSET = 2.0          # integration surface: two cells outside the object
N_FIT, N_PERIODS = 5, 30
DIMS = (4, 256, 256, 256, 256, 1)
ELEM = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
EDGES = (192, 128, 96, 64)   # edges of the uneven batch


def listed():
    return [
        # one 2D force at full length: 128 x 64 cells in FP64, 20 periods from rest
        wave("cylinder_f64_1", "f64", [(128, 64)], 0.5, 5120, warm=0),
        # many object positions at once, the way a force curve F(kh) is made in 2D
        wave("cylinder_f64_32", "f64", [(128, 64)] * 32, 0.5, 5120, warm=0),
        # one 3D force on the standard box of the 3D workload (a stretch of its 15360 steps)
        wave("sphere_f32_1", "f32", [(256, 128, 128)], 0.5, 512),
        # the benchmark workload: 16 positions in one handle
        wave("sphere_f32_16", "f32", [(256, 128, 128)] * 16, 0.5, 128),
        # the same in 16-bit storage, the storage chosen for large sweeps
        wave("sphere_f16_16", "f16", [(256, 128, 128)] * 16, 0.5, 128),
        # uneven boxes in one handle: how the surrogate's training forces are made
        wave("batch_f32_16", "f32", [(e, e, e) for e in EDGES for _ in range(4)], 1 / 3, 128),
        # long channel boxes, the small-kR half of the training forces (rows longer than a block)
        wave("channel_f32_4", "f32", [(1000, 64, 64)] * 4, 1 / 3, 128),
        # a query just outside the trusted box: one whole lattice run of an odd length
        {"name": "query_lb_1", "kind": "predict", "queries": 1, "lam": 251, "radius": 8.0},
        # the calibration before every new box length
        {"name": "cavity_256", "kind": "cavity", "nx": 256, "c0": 0.5},
        # six particles' forces in one step of the particle integrator (the smallest call)
        {"name": "particles_6", "kind": "infer", "batch": 6, "host": True},
        # a dense map of the force over the whole input box
        {"name": "map_1m", "kind": "infer", "batch": 1 << 20, "host": False},
        # training on both force data sets, full batch
        {"name": "train_4800", "kind": "train", "batch": 4800, "steps": 48},
    ]


def wave(name, storage, shapes, c0, steps, warm=None):
    """A wave case: the box shapes as text (nx.ny[.nz] separated by blanks), c0, steps of a pass
    and steps already done (None: until the wave has crossed the longest box)."""
    if warm is None:
        warm = int(1.2 * max(s[0] for s in shapes) / c0)
    return {"name": name, "kind": "wave", "storage": storage, "steps": steps, "warm": warm,
            "c0": c0, "shapes": " ".join(".".join(str(v) for v in s) for s in shapes)}


def draw(rng):
    """One more case: every kind, sizes spread over the logarithm of their ranges, odd ones too."""
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["wave2", "wave3", "wave3", "wave3", "predict", "cavity", "infer", "train"])
    if kind == "wave2":
        c0 = rng.choice([0.5, 0.5, 0.25])
        n, nx = logint(1, 32), logint(64, 512)
        ny = logint(32, 128)
        shapes = [(nx, ny) if rng.random() < 0.6 else (logint(64, nx), ny) for _ in range(n)]
        c = wave("", rng.choice(["f64", "f64", "f32", "f16", "bf16"]), shapes, c0,
                 logint(512, 4096), warm=int(1.2 * nx / c0))
    elif kind == "wave3":
        c0 = rng.choice([0.5, 1 / 3])
        storage = rng.choice(["f32", "f32", "f32", "f16", "bf16", "f64"])
        room = logint(1 << 18, 32 << 20) * 4 // max(4, ELEM[storage])  # cells of the handle
        ny = rng.choice([32, 64, 64, 128, logint(28, 128)])
        nz = rng.choice([ny, ny, logint(28, 128)])
        nx = min(logint(48, 2000), max(48, room // (ny * nz)))
        n = max(1, min(16, room // (nx * ny * nz)))
        if rng.random() < 0.3:  # uneven boxes
            shapes = [(e, e, e) for e in (rng.choice(EDGES) for _ in range(n))]
            while len(shapes) > 1 and sum(s[0] ** 3 for s in shapes) > room:
                shapes.pop()
        else:
            shapes = [(nx, ny, nz)] * n
        c = wave("", storage, shapes, c0, 2 * logint(32, 256) + rng.choice([0, 0, 1]))
    elif kind == "predict":
        lam = logint(100, 250)
        c = {"kind": "predict", "queries": rng.choice([1, 1, 2]) if lam < 160 else 1, "lam": lam,
             "radius": round(rng.uniform(4, 12), 2)}
    elif kind == "cavity":
        c = {"kind": "cavity", "nx": logint(32, 2000), "c0": rng.choice([0.5, 1 / 3, 0.25])}
    elif kind == "infer":
        host = rng.random() < 0.4
        c = {"kind": "infer", "batch": logint(1, 1 << (14 if host else 20)), "host": host}
    else:
        c = {"kind": "train", "batch": logint(64, 4800), "steps": logint(16, 48)}
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------
# inputs, from the case and the seed alone
# ---------------------------------------------------------------------------

def problems(case, seed):
    """One driven box per shape with one object (a cylinder in 2D, a sphere in 3D) between the
    middle of the box and an eighth wave before its quarter, as the descriptor dicts of LBWave."""
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    c0, out = case["c0"], []
    for text in case["shapes"].split():
        s = [int(v) for v in text.split(".")]
        dim, nx = len(s), s[0]
        room = min(min(s[1:]) / 2.0 - 4.5, nx / 2.0 - 9.0)
        R = min(16.0, room) * rng.uniform(0.55, 1.0)
        ratio = rng.uniform(0.8, 1.35 if dim == 2 else 1.15 if c0 == 0.5 else 1.5)
        x0 = nx / 2.0 + rng.uniform(0.15, 0.35) * min(nx / 4.0, nx / 2.0 - R - 9.0)
        center = (x0, s[1] / 2.0, s[2] / 2.0 if dim == 3 else 0.0)
        out.append(problem(s, c0, ratio * c0, R, center, float(nx), case["warm"]))
    return out


def problem(s, c0, cp, R, center, lam, avg_start):
    dim, Rs = len(s), R + OFFSET
    if dim == 2:      # 64 equal segments of a circle
        n = 64
        th = 2.0 * np.pi * (np.arange(n) + 0.5) / n
        nrm = np.stack([np.cos(th), np.sin(th), np.zeros(n)], axis=1)
        area = np.full(n, 2.0 * np.pi * Rs / n)
    else:             # 2048 Fibonacci points of a sphere
        n = 2048
        k = np.arange(n, dtype=np.float64)
        u = 1.0 - (2.0 * k + 1.0) / n
        phi = k * np.pi * (3.0 - np.sqrt(5.0))
        q = np.sqrt(np.maximum(0.0, 1.0 - u * u))
        nrm = np.stack([u, q * np.cos(phi), q * np.sin(phi)], axis=1)
        area = np.full(n, 4.0 * np.pi * Rs * Rs / n)
    return {"dim": dim, "nx": s[0], "ny": s[1], "nz": s[2] if dim == 3 else 1, "xbc": "driven",
            "c0": c0, "rho0": 1.0, "center": center, "radius": R, "cp": cp, "d": THICK,
            "rho_a": 1.0, "omega": 2.0 * np.pi * c0 / lam, "wall_phi": WALL_PHI,
            "surf_xyz": np.asarray(center)[None, :] + Rs * nrm, "surf_normal": nrm,
            "surf_area": area, "avg_start": avg_start}


def queries(case, seed):
    """Queries with c_p/c0 in (1.5, 1.6), just above the trusted range, in boxes of case['lam']."""
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    n, R = case["queries"], case["radius"]
    kR = np.full(n, 2.0 * math.pi * R / case["lam"])
    return kR, rng.uniform(0.25, 1.3, n), rng.uniform(1.51, 1.6, n), np.full(n, R)


def network(seed):
    """Weights and biases uniform in +-1/sqrt(fan_in), layer by layer (W_l row-major, then b_l)."""
    rng = np.random.Generator(np.random.PCG64(int(seed) + 77))
    parts = []
    for k, n in zip(DIMS[:-1], DIMS[1:]):
        b = 1.0 / math.sqrt(k)
        parts += [rng.uniform(-b, b, n * k), rng.uniform(-b, b, n)]
    return np.concatenate(parts).astype(np.float32)


def samples(case, seed):
    """Normalised inputs over the whole box, and a force-like target for training."""
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    x = rng.uniform(-1.0, 1.0, (case["batch"], 4)).astype(np.float32)
    ratio = 1.15 + 0.35 * x[:, 2]
    t = (1.0 - 1.0 / ratio ** 2) * np.sin(np.pi / 2 * (x[:, 1] + 1.0)) * (1.0 - 0.1 * x[:, 0])
    return x, t.astype(np.float32)


def cavity_args(case, seed):
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    return {"rho_a": rng.uniform(0.25, 4.0), "wall_phi": rng.uniform(0.985, 0.992)}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "wave":
        h = LBWave(problems(case, seed), storage=case["storage"])
        h.autotune()
        h.set_graph(64)
        h.step(case["warm"])
        return {"kind": kind, "h": h, "case": case}
    if kind == "predict":
        net = MLP(max_batch=256, params=network(seed))
        return {"kind": kind, "s": Surrogate(net), "q": queries(case, seed)}
    if kind == "cavity":
        return {"kind": kind, "case": case, "args": cavity_args(case, seed)}
    x, t = samples(case, seed)
    if kind == "train":
        net = MLP(max_batch=case["batch"], params=network(seed))
        return {"kind": kind, "net": net, "x": x, "t": t, "steps": case["steps"]}
    net = MLP(max_batch=256, params=network(seed))
    if case["host"]:
        return {"kind": kind, "net": net, "x": x, "host": True}
    x = torch.as_tensor(x, device="cuda")
    y = torch.empty(len(x), dtype=torch.float32, device="cuda")
    return {"kind": kind, "net": net, "x": x, "y": y, "host": False}


def populations(h, i):
    """The populations of box i where they lie in the handle's workspace (Q, nz, ny, nx)."""
    v, p = h.state_view(i), h.problems[i]
    kind = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16,
            "bf16": torch.bfloat16}[h.storage]
    raw = h.ws[v.offset_bytes: v.offset_bytes + v.plane_bytes * h.Q[i]].view(kind)
    return raw.as_strided((h.Q[i], p["nz"], p["ny"], p["nx"]),
                          (v.plane_bytes // v.elem_bytes, p["ny"] * v.pitch, v.pitch, 1))


def run(state):
    kind = state["kind"]
    if kind == "wave":
        h = state["h"]
        h.step(state["case"]["steps"])
        F, n = h.force()
        return {"F": F, "n": n, "f": [populations(h, i) for i in range(h.n)]}
    if kind == "predict":
        out, outside = state["s"].predict(*state["q"])
        return {"F": out, "outside": outside}
    if kind == "cavity":
        c = state["case"]
        return cavity_calibrate(c["nx"], c["c0"], 2 * math.pi * c["c0"] / c["nx"],
                                n_periods=N_PERIODS, n_fit=N_FIT, **state["args"])
    net = state["net"]
    if kind == "train":
        net.train(state["x"], state["t"], steps=state["steps"], lr=1e-3, lr_final=3e-5)
        return {"params": net.params()}
    if state["host"]:
        return {"y": net.predict(state["x"])}
    net.forward_dev(state["x"], state["y"], len(state["x"]))
    return {"y": state["y"]}


def work(case):
    """Least traffic and operations of a pass: the populations read and written once, about
    3 Q operations per cell and step; the network's products (three times for training)."""
    kind = case["kind"]
    if kind == "wave":
        b = f = 0
        for text in case["shapes"].split():
            s = [int(v) for v in text.split(".")]
            q, cells = 2 * len(s) + 1, math.prod(s)
            b += 2 * q * ELEM[case["storage"]] * cells
            f += 3 * q * cells * case["steps"]
        return {"bytes": b, "flops": f}
    if kind == "predict":
        cells = case["lam"] * min(64, case["lam"]) ** 2 * case["queries"]
        return {"bytes": 7 * 4 * cells, "flops": 21 * cells * 90 * case["lam"]}
    if kind == "cavity":
        steps = N_PERIODS * case["nx"] / case["c0"]
        return {"bytes": 16 * case["nx"], "flops": 9 * case["nx"] * steps}
    params = sum((k + 1) * n for k, n in zip(DIMS[:-1], DIMS[1:]))
    macs = sum(k * n for k, n in zip(DIMS[:-1], DIMS[1:]))
    if kind == "train":
        return {"bytes": 20 * case["batch"] + 28 * params,
                "flops": 6 * macs * case["batch"] * case["steps"]}
    return {"bytes": 20 * case["batch"] + 2 * params, "flops": 2 * macs * case["batch"]}


# ---------------------------------------------------------------------------
# the same results in FP64
# ---------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind == "wave":
        ps, steps = problems(case, seed), case["warm"] + case["steps"]
        groups = {}                      # 3D: box by box; 2D: boxes of equal shape together
        for i, p in enumerate(ps):
            groups.setdefault(i if p["dim"] == 3 else (p["nx"], p["ny"]), []).append(i)
        cells = sum(p["nx"] * p["ny"] * p["nz"] for p in ps)
        if (2.5e-4 * len(groups) + 1e-10 * cells) * steps > 18.0:
            return None
        F, f = np.empty((len(ps), 3)), [None] * len(ps)
        for g in groups.values():
            Fg, fg = lattice([ps[i] for i in g], steps)
            for j, i in enumerate(g):
                F[i], f[i] = Fg[j], fg[:, j]
        # BF16 populations keep 8 significant bits: the force over a part of a period then has an
        # error that can be as large as itself, and no FP64 value to be held to
        return {"F": None if case["storage"] == "bf16" else F, "n": None, "f": f}
    if kind == "predict":
        return {"F": lattice_queries(case, seed), "outside": None}
    if kind == "cavity":
        return cavity(case["nx"], case["c0"], **cavity_args(case, seed))
    x, t = samples(case, seed)
    W = unpack(torch.as_tensor(network(seed), dtype=torch.float64, device="cuda"))
    x = torch.as_tensor(x, dtype=torch.float64, device="cuda")
    if kind == "train":
        return {"params": adam(W, x, torch.as_tensor(t, dtype=torch.float64, device="cuda"),
                               case["steps"])}
    y = torch.cat([forward(W, c) for c in x.split(1 << 17)])
    return {"y": y.cpu().numpy() if case["host"] else y}


def sound_speed(p):
    ax = [torch.arange(n, dtype=torch.float64, device="cuda") - c
          for n, c in zip((p["nx"], p["ny"], p["nz"]), p["center"])]
    r2 = ax[0][None, None, :] ** 2 + ax[1][None, :, None] ** 2
    if p["dim"] == 3:
        r2 = r2 + ax[2][:, None, None] ** 2
    return p["c0"] - 0.5 * (p["c0"] - p["cp"]) * (1.0 - torch.tanh((r2 - p["radius"] ** 2) / p["d"]))


def kernel3(r):
    a = np.abs(r)
    near = (1.0 + np.sqrt(np.maximum(0.0, 1.0 - 3.0 * a * a))) / 3.0
    far = (5.0 - 3.0 * a - np.sqrt(np.maximum(0.0, 1.0 - 3.0 * (1.0 - a) ** 2))) / 6.0
    return np.where(a <= 0.5, near, np.where(a <= 1.5, far, 0.0))


def stencils(p):
    """Flat cell indices and weights of every surface point's 3^dim nodes."""
    idx, wgt = 0, 1.0
    stride = (1, p["nx"], p["nx"] * p["ny"])
    for a in range(p["dim"]):
        X = p["surf_xyz"][:, a]
        node = (np.floor(X + 0.5)[:, None] + np.arange(-1, 2)[None, :])
        w = kernel3(node - X[:, None])
        shape = [len(X)] + [1] * p["dim"]
        shape[1 + a] = 3
        idx = idx + (node.astype(np.int64) * stride[a]).reshape(shape)
        wgt = wgt * w.reshape(shape)
    n = len(p["surf_xyz"])
    return (torch.as_tensor(np.ascontiguousarray(idx.reshape(n, -1)), device="cuda"),
            torch.as_tensor(np.ascontiguousarray(wgt.reshape(n, -1)), device="cuda"))


def lattice(ps, steps):
    """`steps` steps from rest of boxes of one shape, frequency and avg_start: per box the force
    averaged over t >= avg_start, and the populations (Q, box, nz, ny, nx)."""
    p, n = ps[0], len(ps)
    d, Q = p["dim"], 2 * p["dim"] + 1
    c2 = torch.stack([sound_speed(q) ** 2 for q in ps])
    rest = 1.0 - d * c2
    new = torch.zeros((Q,) + tuple(c2.shape), dtype=torch.float64, device="cuda")
    f = torch.zeros_like(new)
    rho = torch.empty_like(c2)
    nA = torch.stack([torch.as_tensor(q["surf_normal"] * q["surf_area"][:, None], device="cuda")
                      for q in ps])
    sten = [stencils(q) for q in ps]
    idx = torch.stack([s[0] + j * c2[0].numel() for j, s in enumerate(sten)])
    wgt = torch.stack([s[1] for s in sten])
    total, count = torch.zeros((n, 3), dtype=torch.float64, device="cuda"), 0

    def shift(dst, src, dim, by):       # periodic
        m = src.shape[dim]
        dst.narrow(dim, by % m, m - by % m).copy_(src.narrow(dim, 0, m - by % m))
        dst.narrow(dim, 0, by % m).copy_(src.narrow(dim, m - by % m, by % m))

    for t in range(steps):
        f[0].copy_(new[0])
        f[1][..., 1:] = new[1][..., :-1]
        f[1][..., 0] = 0.0
        f[2][..., :-1] = new[2][..., 1:]
        f[2][..., -1] = 0.0
        for i, dim in ((3, 2), (5, 1))[: d - 1]:
            shift(f[i], new[i], dim, 1)
            shift(f[i + 1], new[i + 1], dim, -1)
        torch.sum(f, dim=0, out=rho)
        if t >= p["avg_start"]:
            r = (rho.view(-1)[idx] * wgt).sum(-1)
            J = torch.zeros(r.shape + (3,), dtype=torch.float64, device="cuda")
            for a in range(d):
                J[..., a] = ((f[1 + 2 * a].view(-1)[idx] - f[2 + 2 * a].view(-1)[idx])
                             * wgt).sum(-1)
            iso = 0.5 * p["c0"] ** 2 * r * r - 0.5 * (J * J).sum(-1)
            total -= (iso[..., None] * nA + J * (J * nA).sum(-1, keepdim=True)).sum(1) / p["rho0"]
            count += 1
        torch.mul(rest, rho, out=new[0])
        new[0].mul_(2.0).sub_(f[0])
        rs = p["rho_a"] * math.sin(p["omega"] * t)
        rho.mul_(c2)
        for i in range(1, Q, 2):
            torch.sub(rho, f[i + 1], out=new[i])
            torch.sub(rho, f[i], out=new[i + 1])
        new[0][..., 1] = rs * rest[..., 1]
        for i in range(1, Q, 2):
            J = f[i][..., 1] - f[i + 1][..., 1]
            new[i][..., 1] = 0.5 * (c2[..., 1] * rs + J)
            new[i + 1][..., 1] = 0.5 * (c2[..., 1] * rs - J)
        for x in (0, -1):
            new[0][..., x] = p["wall_phi"] * f[0][..., x]
            for i in range(1, Q, 2):
                new[i][..., x] = p["wall_phi"] * f[i + 1][..., x]
                new[i + 1][..., x] = p["wall_phi"] * f[i][..., x]
    return (total / max(count, 1)).cpu().numpy(), new


def cavity(nx, c0, rho_a=1.0, wall_phi=WALL_PHI):
    """The empty box, which is a 1D lattice of three populations, and the fit of its envelope."""
    om, c2 = 2 * math.pi * c0 / nx, c0 * c0
    total, m = round(N_PERIODS * nx / c0), round(N_FIT * nx / c0)
    k = math.acos(1.0 - (1.0 - math.cos(om)) / c2)
    new, f = np.zeros((3, nx)), np.zeros((3, nx))
    P = np.zeros(nx, dtype=np.complex128)
    ends = [0, nx - 1]
    for t in range(total):
        f[0] = new[0]
        f[1, 1:] = new[1, :-1]
        f[2, :-1] = new[2, 1:]
        rho = f[0] + f[1] + f[2]
        if t >= total - m:
            P += rho * complex(math.cos(om * t), -math.sin(om * t))
        np.multiply(rho, 2.0 * (1.0 - c2), out=new[0])
        new[0] -= f[0]
        rho *= c2
        np.subtract(rho, f[2], out=new[1])
        np.subtract(rho, f[1], out=new[2])
        rs, J = rho_a * math.sin(om * t), f[1, 1] - f[2, 1]
        new[:, 1] = rs * (1.0 - c2), 0.5 * (c2 * rs + J), 0.5 * (c2 * rs - J)
        new[0, ends] = wall_phi * f[0, ends]
        new[1, ends], new[2, ends] = wall_phi * f[2, ends], wall_phi * f[1, ends]
    P *= 2.0 / m
    x = np.arange(2, nx - 2)
    M = np.stack([np.ones(len(x)), np.cos(2 * k * x), np.sin(2 * k * x)], axis=1)
    (a, b, c), *_ = np.linalg.lstsq(M, np.abs(P[2:nx - 2]) ** 2, rcond=None)
    A = math.sqrt(a + math.hypot(b, c))
    x0, gap = math.atan2(c, b) / (2 * k), math.pi / k
    mid = x0 + math.floor((0.5 * (nx - 1) - x0) / gap) * gap
    return {"A": A, "x_mid": mid, "k": k, "Pa": c0 * c0 * A,
            "fit": (float(a), float(b), float(c)), "P": P}


def lattice_queries(case, seed):
    c0, lam = 1.0 / 3.0, case["lam"]
    cal = cavity(lam, c0)
    w, out = min(64, lam), []
    for kR, kh, ratio, _ in zip(*queries(case, seed)):
        R = float(kR * lam / (2 * math.pi))
        p = problem((lam, w, w), c0, ratio * c0, R, (cal["x_mid"] + kh / cal["k"], w / 2.0, w / 2.0),
                    float(lam), 60 * lam)
        F = lattice([p], 90 * lam)[0][0]
        F0 = math.pi * R ** 3 * cal["Pa"] ** 2 * (2 * math.pi / lam) / (3 * c0 * c0)
        out.append(F[0] / F0)
    return np.array(out)


def unpack(p):
    W, off = [], 0
    for k, n in zip(DIMS[:-1], DIMS[1:]):
        W.append((p[off: off + n * k].view(n, k), p[off + n * k: off + n * k + n]))
        off += n * (k + 1)
    return W


def forward(W, x):
    for w, b in W[:-1]:
        x = torch.nn.functional.gelu(x @ w.T + b)
    return (x @ W[-1][0].T + W[-1][1])[:, 0]


def adam(W, x, t, steps, lr=1e-3, lr_final=3e-5, b1=0.9, b2=0.999, eps=1e-8):
    P = [v.clone().requires_grad_(True) for w in W for v in w]
    m, v = [torch.zeros_like(q) for q in P], [torch.zeros_like(q) for q in P]
    for s in range(steps):
        y = forward(list(zip(P[0::2], P[1::2])), x)
        g = torch.autograd.grad(((y - t) ** 2).mean(), P)
        a = float(np.float32(lr * (lr_final / lr) ** (s / max(steps - 1, 1))))
        with torch.no_grad():
            for q, gi, mi, vi in zip(P, g, m, v):
                mi.mul_(b1).add_(gi, alpha=1 - b1)
                vi.mul_(b2).addcmul_(gi, gi, value=1 - b2)
                q -= a * (mi / (1 - b1 ** (s + 1))) / ((vi / (1 - b2 ** (s + 1))).sqrt() + eps)
    return torch.cat([q.detach().reshape(-1) for q in P]).cpu().numpy()
