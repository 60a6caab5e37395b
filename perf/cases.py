"""The timed workloads of the solver: what a user's program has it do, with inputs made
from a seed, and what the same discrete schemes give in plain 64-bit torch.

Kinds of pass:
  solve    a new field on a handle that is kept: set_field, propagate to the end, density
           with n(p) left on the device (a parameter scan, or one request after another)
  series   the same in equal chunks with a snapshot of the occupation after each
  batch    members whose fields are set, solved by one Batch.run (captured and replayed),
           then each member's n(p)
  epochs   new fields on kept handles, then epochs of step_each until every member is
           complete, as the serving loop runs them

A single-precision solve's n(p) carries single precision (its state is FP32), so a program
that keeps many of them keeps them as float32; double-precision solves stay float64.
"""
import math
import random

import numpy as np
import torch

import paper_1607_03062_amd as pd

DEV = "cuda"
STAGES = {"strang": 1, "midpoint": 1, "strang4": 5, "midpoint4": 5}


def listed():
    return [
        # the repository's plain configuration, the smallest solve a scan runs: latency
        {"name": "scan_64_fp64", "kind": "solve", "nx": 64, "ny": 64, "half": 2.0, "steps": 4000,
         "precision": "fp64", "scheme": "strang", "field": "sin2", "ellipticity": 0.0},
        # one served request of ordinary size in the library's default FP32 form
        {"name": "request_512_fp32", "kind": "solve", "nx": 512, "ny": 512, "half": 4.0, "steps": 20000,
         "precision": "fp32", "scheme": "strang", "field": "sin2", "ellipticity": 0.0},
        # the FP64 configuration on the wide grid
        {"name": "solve_1024_fp64", "kind": "solve", "nx": 1024, "ny": 1024, "half": 4.0, "steps": 40000,
         "precision": "fp64", "scheme": "strang", "field": "sin2", "ellipticity": 0.0},
        # the benchmark solve, the largest: fast FP32 form
        {"name": "bench_2048_fp32fast", "kind": "solve", "nx": 2048, "ny": 2048, "half": 2.0, "steps": 80000,
         "precision": "fp32fast", "scheme": "strang", "field": "sin2", "ellipticity": 0.0},
        # a large grid of no round size, default FP32 form
        {"name": "solve_1500x2047_fp32", "kind": "solve", "nx": 1500, "ny": 2047, "half": 3.0, "steps": 12000,
         "precision": "fp32", "scheme": "strang", "field": "sin2", "ellipticity": 0.0},
        # fourth order under an elliptic pulse, FP32 (the README's first example)
        {"name": "elliptic4_1024_fp32", "kind": "solve", "nx": 1024, "ny": 1024, "half": 4.0, "steps": 4000,
         "precision": "fp32", "scheme": "strang4", "field": "sin2", "ellipticity": 0.5},
        # the paper's laser pulse, fourth order, FP64 (the README's second example)
        {"name": "pulse4_512_fp64", "kind": "solve", "nx": 512, "ny": 512, "half": 4.0, "steps": 4000,
         "precision": "fp64", "scheme": "strang4", "field": "pulse", "ellipticity": 0.0},
        # the paper's own step (midpoint exponential), FP64, a grid of no round size
        {"name": "midpoint_700x511_fp64", "kind": "solve", "nx": 700, "ny": 511, "half": 3.0, "steps": 8000,
         "precision": "fp64", "scheme": "midpoint", "field": "pulse", "ellipticity": 0.0},
        # the same step in the FP32 form
        {"name": "midpoint_1024_fp32", "kind": "solve", "nx": 1024, "ny": 1024, "half": 2.0, "steps": 10000,
         "precision": "fp32", "scheme": "midpoint", "field": "sin2", "ellipticity": 0.0},
        # time-resolved occupation: eight chunks, a snapshot after each
        {"name": "series_400x300_fp64", "kind": "series", "nx": 400, "ny": 300, "half": 2.5, "steps": 6400,
         "precision": "fp64", "scheme": "strang", "field": "sin2", "ellipticity": 0.0, "chunks": 8},
        # many solves of mixed sizes and lengths in one captured launch sequence
        {"name": "batch_16_fp32", "kind": "batch", "members": 16, "least": 128, "most": 1024, "half": 4.0,
         "steps": 12000, "mixed": False, "pick": 4},
        # the serving loop's epochs over a handful of requests, FP32 and FP64 mixed
        {"name": "epochs_6_mixed", "kind": "epochs", "members": 6, "least": 128, "most": 512, "half": 4.0,
         "steps": 9000, "mixed": True, "pick": 5, "epoch": 3000},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve"] * 5 + ["series", "batch", "epochs"])
    if kind in ("batch", "epochs"):
        c = {"kind": kind, "members": rng.randint(3, 20), "least": rng.choice([64, 96, 128]),
             "most": rng.choice([256, 512, 1024]), "half": 4.0, "steps": _logint(rng, 3000, 12000),
             "mixed": rng.random() < 0.5, "pick": rng.randrange(1 << 20)}
        if kind == "epochs":
            c["epoch"] = rng.choice([1500, 2048, 3000])
            c["members"] = min(c["members"], 8)
        return c
    scheme = rng.choice(["strang"] * 5 + ["midpoint", "midpoint", "strang4", "midpoint4"])
    precision = rng.choice(["fp64", "fp32", "fp32fast"])
    c = {"kind": kind, "nx": _logint(rng, 32, 2048), "ny": _logint(rng, 32, 2048),
         "half": rng.choice([2.0, 3.0, 4.0]), "steps": _logint(rng, 2000, 20000 if precision != "fp64" else 60000),
         "precision": precision, "scheme": scheme, "field": rng.choice(["sin2", "sin2", "pulse"]),
         "ellipticity": rng.choice([0.0, 0.0, 0.5])}
    if STAGES[scheme] == 5:
        c["steps"] = min(c["steps"], 5000)
    # at most about 2e10 FP64 (5e10 FP32) stages of a point: under the largest listed case's time
    most = 2e10 if precision == "fp64" else 5e10
    c["steps"] = max(1000, min(c["steps"], int(most / (c["nx"] * c["ny"] * STAGES[scheme]))))
    if kind == "series":
        c["chunks"] = rng.randint(3, 10)
        c["scheme"] = "strang"
        c["steps"] = max(c["steps"], 2000)
    return c


# ---- inputs ---------------------------------------------------------------------------


def _field(rng, kind, ellipticity, steps, half, stages=1):
    """A field of the seeded distributions, short enough for the step count: dt |p + A|
    stays at about 0.2 or below, as the repository's step-count rules have it."""
    if kind == "pulse":
        # the rise / flat / fall pulse in reduced units (E0 = 1, tau omega = 0.4876, 5.5 periods)
        u = rng.uniform(0.9, 1.1)
        f = {"kind": "pulse", "E0": rng.uniform(0.6, 1.0), "omega": 0.4876 * u, "phi": rng.uniform(0.0, 0.5),
             "omega_rise": 0.0609 * u, "omega_fall": 0.0609 * u, "duration": 70.9 / u}
    else:
        omega = rng.uniform(0.3, 0.6)
        E0 = rng.uniform(0.1, 0.3)
        bound = math.sqrt(2.0) * half + 3.0 * E0 / omega
        most = int(0.2 * steps * math.sqrt(stages) / bound * omega / (2.0 * math.pi))
        f = {"kind": "sin2", "E0": E0, "omega": omega, "cycles": max(2, min(rng.randint(8, 30), most))}
    if ellipticity:
        f["ellipticity"] = float(ellipticity)
    return f


def _members(case, rng):
    """Sizes, step counts and precisions of a batch's members: properties of the case."""
    pick = random.Random(case["pick"])
    sizes = [n for n in (64, 96, 128, 200, 256, 384, 512, 768, 1024) if case["least"] <= n <= case["most"]]
    out = []
    for _ in range(case["members"]):
        n, steps = pick.choice(sizes), pick.randint(case["steps"] // 4, case["steps"])
        precision = pick.choice(["fp32", "fp64"]) if case["mixed"] else "fp32"
        out.append({"grid": _grid(n, n, case["half"]), "steps": steps, "precision": precision, "scheme": "strang",
                    "field": _field(rng, "sin2", 0.0, steps, case["half"])})
    return out


def _grid(nx, ny, half):
    return {"nx": nx, "ny": ny, "px": (-half, half), "py": (-half, half)}


def _inputs(case, seed):
    rng = random.Random(seed)
    if case["kind"] in ("batch", "epochs"):
        return _members(case, rng)
    stages = STAGES[case["scheme"]]
    return [{"grid": _grid(case["nx"], case["ny"], case["half"]), "steps": case["steps"],
             "precision": case["precision"], "scheme": case["scheme"],
             "field": _field(rng, case["field"], case["ellipticity"], case["steps"], case["half"], stages)}]


def prepare(case, seed):
    jobs = _inputs(case, seed)
    solvers = [pd.Solver.for_grid(j["grid"], j["precision"], j["scheme"]) for j in jobs]
    copies = case.get("chunks", 1)
    outs = [[torch.empty(j["grid"]["nx"] * j["grid"]["ny"], dtype=torch.float64, device=DEV) for _ in range(copies)]
            for j in jobs]
    state = {"kind": case["kind"], "jobs": jobs, "solvers": solvers, "outs": outs, "case": case}
    if case["kind"] in ("batch", "epochs"):
        if case["kind"] == "batch":
            for s, j in zip(solvers, jobs):
                s.set_field(j["field"], j["steps"])
        state["batch"] = pd.Batch(solvers)
    return state


def _keep(job, n):
    return n if job["precision"] == "fp64" else n.to(torch.float32)


def run(state):
    jobs, solvers, outs = state["jobs"], state["solvers"], state["outs"]
    kind = state["kind"]
    if kind == "solve":
        s, j, n = solvers[0], jobs[0], outs[0][0]
        s.set_field(j["field"], j["steps"])
        rho = s.solve(n_out=n)
        return {"n": _keep(j, n), "rho": rho}
    if kind == "series":
        s, j = solvers[0], jobs[0]
        s.set_field(j["field"], j["steps"])
        rhos = []
        for end, prev, n in _cuts(j["steps"], outs[0]):
            s.propagate(end - prev)
            rhos.append(s.snapshot(n_out=n))
        return {"n": [_keep(j, n) for n in outs[0]], "rho": rhos}
    b = state["batch"]
    if kind == "batch":
        rho = b.run()
    else:
        for s, j in zip(solvers, jobs):
            s.set_field(j["field"], j["steps"])
        rho = np.full(len(jobs), np.nan)
        done = np.zeros(len(jobs), dtype=bool)
        while not done.all():
            r, done = b.step_each([state["case"]["epoch"]] * len(jobs))
            rho = np.where(np.isnan(r), rho, r)
    for s, n in zip(solvers, outs):
        s.density(n_out=n[0], want_rho=False)
    return {"n": [_keep(j, n[0]) for j, n in zip(jobs, outs)], "rho": [float(r) for r in rho]}


def _cuts(steps, outs):
    """(end, begin, buffer) of each of the equal chunks."""
    k = len(outs)
    ends = [steps * (i + 1) // k for i in range(k)]
    return zip(ends, [0] + ends[:-1], outs)


# ---- the work a pass cannot do without --------------------------------------------------


def work(case):
    """Bytes: the field's samples in, n(p) out, each once.  Operations: a Strang stage turns
    a three-component vector about x and about y, three multiply-adds each (12); a midpoint
    stage is the 2x2 update (16) and its coefficients (8)."""
    bytes_, flops = 0.0, 0.0
    for j in _inputs(case, 0):
        npts, stages = j["grid"]["nx"] * j["grid"]["ny"], STAGES[j["scheme"]]
        size = 8 if j["precision"] == "fp64" else 4
        bytes_ += 8.0 * j["steps"] * stages + size * npts * case.get("chunks", 1)
        flops += (24.0 if j["scheme"].startswith("midpoint") else 12.0) * npts * j["steps"] * stages
    return {"bytes": bytes_, "flops": flops}


# ---- the same schemes in 64 bits, plain torch --------------------------------------------


def _carrier(w, q, a, b):
    return (np.sin(w * b + q) - np.sin(w * a + q)) / w


def _potential(f, t, component):
    """A(t) = -int_0^t E of a field, x or y component (numpy float64)."""
    t = np.asarray(t, dtype=np.float64)
    e = f.get("ellipticity", 0.0)
    if component == "y" and not e:
        return np.zeros_like(t)
    amp = f["E0"] * (e if component == "y" else 1.0)
    w = f["omega"]
    if f["kind"] == "sin2":
        # env sin^2(W t / 2): E = amp env(t) sin(w t) (x) or cos(w t) (y)
        T = f["cycles"] * 2.0 * math.pi / w
        W = 2.0 * math.pi / T
        t = np.minimum(t, T)
        if component == "x":
            part = lambda v: 2.0 * np.sin(0.5 * v * t) ** 2 / v  # noqa: E731
        else:
            part = lambda v: np.sin(v * t) / v  # noqa: E731
        return -amp * (0.5 * part(w) - 0.25 * part(w + W) - 0.25 * part(w - W))
    # rise over [0, tr], flat, fall over [ta, D]; carrier cos(w t + q)
    q = f["phi"] - (0.5 * math.pi if component == "y" else 0.0)
    Wr, Wf, D = f["omega_rise"], f["omega_fall"], f["duration"]
    tr, ta = 0.5 * math.pi / Wr, D - 0.5 * math.pi / Wf
    t = np.minimum(t, D)

    def beat(W, c, a, b):  # int cos(2 W (s - c)) cos(w s + q) ds
        return 0.5 * (_carrier(w + 2 * W, q - 2 * W * c, a, b) + _carrier(w - 2 * W, q + 2 * W * c, a, b))

    e1 = np.minimum(t, tr)
    total = 0.5 * _carrier(w, q, 0.0, e1) - 0.5 * beat(Wr, 0.0, 0.0, e1)
    e2 = np.minimum(np.maximum(t, tr), ta)
    total = total + _carrier(w, q, tr, e2)
    e3 = np.maximum(t, ta)
    total = total + 0.5 * _carrier(w, q, ta, e3) + 0.5 * beat(Wf, ta, ta, e3)
    return -amp * total


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device=DEV)


def _shear(u, v, t, s):
    """(u, v) turned by the angle of t = tan(angle / 2), s = sin(angle), in place."""
    u.addcmul_(v, t, value=-1.0)
    v.addcmul_(u, s)
    u.addcmul_(v, t, value=-1.0)


def _project(x, y, z, px, py, ax, ay):
    Px, Py = px + ax, py + ay
    E = torch.sqrt(Px * Px + Py * Py)
    norm = torch.sqrt(x * x + y * y + z * z)
    n = 0.5 * (1.0 + (x * Px + y * Py) / (norm * E))
    return torch.where(E > 0, n, torch.zeros_like(n))


def _exact_one(job, cuts):
    """n after each of the step counts in `cuts`, and rho of each."""
    g, f, N = job["grid"], job["field"], job["steps"]
    nx, ny = g["nx"], g["ny"]
    dx, dy = (g["px"][1] - g["px"][0]) / nx, (g["py"][1] - g["py"][0]) / ny
    px, py = _dev(g["px"][0] + np.arange(nx) * dx)[None, :], _dev(g["py"][0] + np.arange(ny) * dy)[:, None]
    T = f["cycles"] * 2.0 * math.pi / f["omega"] if f["kind"] == "sin2" else f["duration"]
    dt = T / N
    S = STAGES[job["scheme"]]
    p = 1.0 / (4.0 - 4.0 ** (1.0 / 3.0))
    c = np.array([1.0]) if S == 1 else np.array([p, p, 1.0 - 4.0 * p, p, p])
    mid = (np.arange(N)[:, None] + (np.cumsum(c) - 0.5 * c)[None, :]) * dt
    Ax, Ay = _potential(f, mid, "x").reshape(-1), _potential(f, mid, "y").reshape(-1)
    cj = np.tile(c, N)
    bound = lambda k: (float(_potential(f, k * dt, "x")), float(_potential(f, k * dt, "y")))  # noqa: E731
    a_in = bound(0)
    E = torch.sqrt((px + a_in[0]) ** 2 + (py + a_in[1]) ** 2)
    good = E > 0
    one = torch.where(good, E, torch.ones_like(E))
    scale = 4.0 * dx * dy / (2.0 * math.pi) ** 2
    found = []

    def keep(n):
        n = torch.where(good, n, torch.zeros_like(n)).reshape(-1)
        found.append((n, scale * float(n.sum())))

    block = max(1, min(512, (1 << 25) // max(nx, ny)))
    if job["scheme"].startswith("strang"):
        x = torch.where(good, -(px + a_in[0]) / one, torch.zeros_like(E)).contiguous()
        y = torch.where(good, -(py + a_in[1]) / one, torch.zeros_like(E)).contiguous()
        z = torch.zeros_like(x)
        # the y rotation after sample m: the halves of m and of m + 1 merged
        hy = cj * dt
        plain = not f.get("ellipticity", 0.0)

        def y_coef(angle):
            return torch.tan(0.5 * angle), torch.sin(angle)

        def half(m):
            return y_coef(hy[m] * (py + Ay[m]))

        fixed = {}
        _shear(z, x, *half(0))
        todo = sorted(cuts)
        for m0 in range(0, N * S, block):
            m1 = min(N * S, m0 + block)
            ang = 2.0 * _dev(cj[m0:m1] * dt)[:, None] * (px + _dev(Ax[m0:m1])[:, None])
            tx, sx = torch.tan(0.5 * ang).unbind(0), torch.sin(ang).unbind(0)
            for m in range(m0, m1):
                _shear(y, z, tx[m - m0], sx[m - m0])
                if m + 1 < N * S:
                    if plain:
                        key = (m % S, (m + 1) % S)
                        if key not in fixed:
                            fixed[key] = y_coef((hy[m] + hy[m + 1]) * py)
                        t, s = fixed[key]
                    else:
                        t, s = y_coef(hy[m] * (py + Ay[m]) + hy[m + 1] * (py + Ay[m + 1]))
                else:
                    t, s = half(m)
                _shear(z, x, t, s)
                if (m + 1) % S == 0 and todo and (m + 1) // S == todo[0]:
                    k = todo.pop(0)
                    zz, xx = z, x
                    if k < N:  # the state is ahead by the next opening half: turn back
                        zz, xx = z.clone(), x.clone()
                        t, s = half(m + 1)
                        _shear(zz, xx, -t, -s)
                    keep(_project(xx, y, zz, px, py, *bound(k)))
    else:
        r2 = 1.0 / math.sqrt(2.0)
        u = torch.where(good, r2 * torch.complex(-(px + a_in[0]) / one, (py + a_in[1]) / one), torch.zeros_like(E))
        v = torch.where(good, r2 * torch.ones_like(E), torch.zeros_like(E)).to(torch.complex128)
        for m in range(N * S):
            X, Y = cj[m] * dt * (px + Ax[m]), cj[m] * dt * (py + Ay[m])
            th = torch.sqrt(X * X + Y * Y)
            co, si = torch.cos(th), torch.sinc(th / math.pi)
            w = torch.complex(si * Y, si * X)  # i si (X - i Y)
            u, v = co * u - w * v, co * v + w.conj() * u
        a = bound(N)
        Px, Py = px + a[0], py + a[1]
        Eo = torch.sqrt(Px * Px + Py * Py)
        amp = (Eo * u + torch.complex(Px.expand_as(Eo).contiguous(), -Py.expand_as(Eo)) * v).abs() ** 2
        n = amp / (2.0 * Eo * Eo) / (u.abs() ** 2 + v.abs() ** 2)
        keep(torch.where(Eo > 0, n, torch.zeros_like(n)))
    return found


def exact(case, seed):
    jobs = _inputs(case, seed)
    stages = sum(j["steps"] * STAGES[j["scheme"]] for j in jobs)
    points = max(j["grid"]["nx"] * j["grid"]["ny"] for j in jobs)
    # a stage is about six passes over the state (twenty for the midpoint step or an elliptic field)
    heavy = any(j["scheme"].startswith("midpoint") or j["field"].get("ellipticity") for j in jobs)
    if stages * (20 if heavy else 6) * (6e-6 + points * 6e-12) > 20.0:
        return None
    if case["kind"] == "series":
        cuts = [end for end, _, _ in _cuts(case["steps"], [None] * case["chunks"])]
        got = _exact_one(jobs[0], cuts)
        return {"n": [n for n, _ in got], "rho": [r for _, r in got]}
    got = [_exact_one(j, [j["steps"]])[0] for j in jobs]
    if case["kind"] == "solve":
        return {"n": got[0][0], "rho": got[0][1]}
    return {"n": [n for n, _ in got], "rho": [r for _, r in got]}
