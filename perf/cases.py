"""The work a user of this framework has it do, through its public entry points: what is timed when
the framework's speed is looked at.

Four kinds of case:
  flow      the arrested Newton flow of one field from its initial data: `steps` accepted steps of
            skyr_anf_step (dense or padded rows, exact or printed force, any model);
  batch     independent flows advanced together in one skyr_batch, as the server does it: every job is
            added, ticks of 32 sweep slots run until all have stopped, results are collected;
  observe   one call on a finished field: observables, the gradient, or the moment observables;
  block     one device's step sweep of a lattice split over devices, its shell from a buffer.

Initial data are products of unit hedgehogs or the B = 4 cube, made here with torch in 64 bits and
rounded to the field precision.  exact() repeats a case in 64 bits with plain torch: the energy is
written out and autograd gives its gradient.
"""
from __future__ import annotations

import math
import random

import torch

import skyr_inputs
from paper_2604_25876_amd import skyr

DEVICE = "cuda"
TICK = 32  # sweep slots per batch tick, the server's default
MAX_BYTES = 64 * 252 ** 3 * 128  # traffic of the largest case, the 64-bit flow on 256^3


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the first thing anyone runs: one hedgehog on 40^3, 300 steps; small launches, latency counts
        dict(name="hedgehog-40-f64", kind="flow", prec="f64", n0=40, n1=40, n2=40, h=0.2, m=1.0, model="plain",
             init="hedgehog", B=1, steps=300, padded=False),
        # the B = 4 cube relaxed in double precision on an ordinary lattice
        dict(name="cube-b4-128-f64", kind="flow", prec="f64", n0=128, n1=128, n2=128, h=0.15, m=1.0, model="plain",
             init="cube_b4", B=4, steps=100, padded=False),
        # the size the method is usually run at (151^3), single precision; rows that are not whole lines
        dict(name="cube-b4-151-f32", kind="flow", prec="f32", n0=151, n1=151, n2=151, h=0.107, m=1.0, model="plain",
             init="cube_b4", B=4, steps=100, padded=False),
        # ten Skyrmions on the largest usual lattice, both precisions: throughput
        dict(name="random-b10-256-f32", kind="flow", prec="f32", n0=256, n1=256, n2=256, h=0.1, m=1.0, model="plain",
             init="random", B=10, steps=64, padded=False),
        dict(name="random-b10-256-f64", kind="flow", prec="f64", n0=256, n1=256, n2=256, h=0.1, m=1.0, model="plain",
             init="random", B=10, steps=64, padded=False),
        # the worked examples: the printed form of the force on 151^3 in double precision
        dict(name="printed-b8-151-f64", kind="flow", prec="f64", n0=151, n1=151, n2=151, h=16.0 / 150.0, m=1.0,
             model="printed", init="random", B=8, steps=50, padded=False),
        # the extended model (four potentials and the sextic term)
        dict(name="sextic-b4-96-f32", kind="flow", prec="f32", n0=96, n1=96, n2=96, h=0.15, m=1.0, model="sextic",
             init="random", B=4, steps=50, padded=False),
        # the 64-job parameter scan: cubes of 48 .. 128 sites, single precision, padded rows
        dict(name="batch-64-f32", kind="batch", jobs=64, mix="scan", master=4, steps=48),
        # what the server holds at one time: lattices of 48 .. 192 sites, both precisions
        dict(name="served-20-mixed", kind="batch", jobs=20, mix="served", master=5, steps=48),
        # one observables call on a small field: the smallest call
        dict(name="observables-65-f32", kind="observe", what="observables", prec="f32", n0=65, n1=65, n2=65, h=0.25,
             m=1.0, model="plain", init="cube_b4", B=4),
        # inertia tensors, radius and D-term of a worked example
        dict(name="moments-151-f64", kind="observe", what="moments", prec="f64", n0=151, n1=151, n2=151,
             h=16.0 / 150.0, m=1.0, model="plain", init="random", B=8),
        # one device's 128^3 block of a 256^3 lattice on eight devices
        dict(name="block-128-of-256-f32", kind="block", prec="f32", n0=256, n1=256, n2=256, h=0.1, m=1.0,
             model="plain", init="random", B=10, o0=128, o1=0, o2=128, extent=128),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choices(["flow", "batch", "observe", "block"], [8, 3, 3, 1])[0]
    prec = rng.choice(["f32", "f64"])
    h = round(rng.uniform(0.1, 0.2), 4)
    if kind == "batch":
        mix = rng.choice(["scan", "served"])
        c = dict(kind="batch", jobs=log_int(2, 64 if mix == "scan" else 20), mix=mix, master=rng.randint(100, 9999),
                 steps=rng.randint(16, 48))
        while work(c)["bytes"] > MAX_BYTES:
            c["jobs"] -= 1
        return c
    if kind == "block":
        n = rng.randint(100, 256)
        e = rng.randint(n // 3, n // 2)
        o = [rng.randint(0, n - e) for _ in range(3)]
        return dict(kind="block", prec=prec, n0=n, n1=n, n2=n, h=h, m=1.0, model="plain", init="random", B=8,
                    o0=o[0], o1=o[1], o2=o[2], extent=e)
    n = [log_int(40, 256)] * 3
    if rng.random() < 0.35:  # a box that is not a cube
        n = [max(24, min(256, int(k * rng.uniform(0.6, 1.4)))) for k in n]
    init = rng.choice(["random", "random", "cube_b4", "hedgehog"])
    B = {"random": rng.randint(2, 12), "cube_b4": 4, "hedgehog": 1}[init]
    c = dict(kind=kind, prec=prec, n0=n[0], n1=n[1], n2=n[2], h=h, m=float(rng.randint(0, 1)), model="plain",
             init=init, B=B)
    if kind == "observe":
        c["what"] = rng.choice(["observables", "gradient", "moments"])
        return c
    c["model"] = rng.choices(["plain", "potentials", "sextic", "printed"], [5, 1, 1, 1])[0]
    c["padded"] = c["model"] != "printed" and rng.random() < 0.25
    c["steps"] = 1
    c["steps"] = min(log_int(10, 200), int(0.5 * MAX_BYTES // work(c)["bytes"]))
    return c


def work(case):
    """Each field read once and written once per step; flops of the force, energy and update."""
    word = 4 if case.get("prec") == "f32" else 8
    if case["kind"] == "batch":
        b = f = 0
        for j in _jobs(case, 0):
            inner = (j["n"] - 4) ** 3
            b += case["steps"] * inner * 16 * (4 if j["prec"] == "f32" else 8)
            f += case["steps"] * inner * 340
        return {"bytes": b, "flops": f}
    inner = (case["n0"] - 4) * (case["n1"] - 4) * (case["n2"] - 4)
    if case["kind"] == "flow":
        per = {"plain": 340, "potentials": 360, "sextic": 520, "printed": 420}[case["model"]]
        return {"bytes": case["steps"] * inner * 16 * word, "flops": case["steps"] * inner * per}
    if case["kind"] == "observe":
        arrays = 8 if case["what"] == "gradient" else 4
        return {"bytes": arrays * case["n0"] * case["n1"] * case["n2"] * word,
                "flops": inner * (700 if case["what"] == "moments" else 330)}
    own = case["extent"] ** 3
    shell = (case["extent"] + 8) ** 3 - own
    return {"bytes": (16 * own + 8 * shell) * word, "flops": own * 340}


# ------------------------------------------------------------------ initial data
def _rotation(q):
    a, b, c, d = q
    return [[a * a + b * b - c * c - d * d, 2 * (b * c + a * d), 2 * (b * d - a * c)],
            [2 * (b * c - a * d), a * a - b * b + c * c - d * d, 2 * (c * d + a * b)],
            [2 * (b * d + a * c), 2 * (c * d - a * b), a * a - b * b - c * c + d * d]]


def _constituents(init, B, rng):
    """(centre, isorotation matrix, profile length) of every constituent."""
    out = []
    for _ in range(B if init == "random" else 1):
        q = [rng.gauss(0.0, 1.0) for _ in range(4)]
        s = math.sqrt(sum(v * v for v in q))
        R = _rotation([v / s for v in q])
        if init == "random":  # uniform in the ball of radius 3
            while True:
                X = [rng.uniform(-3.0, 3.0) for _ in range(3)]
                if sum(v * v for v in X) <= 9.0:
                    break
        else:  # one soliton, not quite on the lattice's centre
            X = [rng.uniform(-0.2, 0.2) for _ in range(3)]
        out.append((X, R, 1.5 if init == "cube_b4" else 1.0))
    return out


def _field(shape, h, init, B, rng):
    """A unit 4-vector field in 64 bits, shape (4, n0, n1, n2): vacuum on the two outer layers."""
    f64 = dict(dtype=torch.float64, device=DEVICE)
    ax = [(torch.arange(n, **f64) - 0.5 * (n - 1)) * h for n in shape]
    U = None
    for X, R, lam in _constituents(init, B, rng):
        x = (ax[0] - X[0])[:, None, None].expand(shape)
        y = (ax[1] - X[1])[None, :, None].expand(shape)
        z = (ax[2] - X[2])[None, None, :].expand(shape)
        r = torch.sqrt(x * x + y * y + z * z)
        if init == "cube_b4":
            # R(z) = (z^4 + 2 sqrt3 i z^2 + 1) / (z^4 - 2 sqrt3 i z^2 + 1), z = u / w
            u2, w2 = torch.complex(x, y) ** 2, (r + z) ** 2
            p, q = u2 * u2 + w2 * w2, 2j * math.sqrt(3.0) * u2 * w2
            P, Q = p + q, p - q
            pq, p2, q2 = P * Q.conj(), P.abs() ** 2, Q.abs() ** 2
            d = [2 * pq.real / (p2 + q2), 2 * pq.imag / (p2 + q2), (q2 - p2) / (p2 + q2)]
        else:
            d = [x / r.clamp(min=1e-12), y / r.clamp(min=1e-12), z / r.clamp(min=1e-12)]
        f = math.pi * torch.exp(-r / lam)
        sf = torch.sin(f)
        V = [torch.cos(f)] + [sf * (R[i][0] * d[0] + R[i][1] * d[1] + R[i][2] * d[2]) for i in range(3)]
        U = V if U is None else _qmul(U, V)
    phi = torch.zeros((4,) + tuple(shape), **f64)
    phi[0] = 1.0
    inner = (slice(2, -2),) * 3
    for A in range(4):
        phi[(A,) + inner] = U[A][inner]
    return phi


def _qmul(a, b):
    """(a0 + i a.tau)(b0 + i b.tau) = (a0 b0 - a.b) + i (a0 b + b0 a - a x b).tau."""
    return [a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3],
            a[0] * b[1] + b[0] * a[1] - (a[2] * b[3] - a[3] * b[2]),
            a[0] * b[2] + b[0] * a[2] - (a[3] * b[1] - a[1] * b[3]),
            a[0] * b[3] + b[0] * a[3] - (a[1] * b[2] - a[2] * b[1])]


def _start(case, seed):
    """The case's initial field in its own precision."""
    shape = (case["n0"], case["n1"], case["n2"])
    phi = _field(shape, case["h"], case["init"], case["B"], random.Random(seed))
    return phi.to(_dtype(case["prec"]))


def _dtype(prec):
    return torch.float32 if prec == "f32" else torch.float64


def _couplings(case):
    """m, m_y, m_z, m_w, c6."""
    return {"plain": (case["m"], 0.0, 0.0, 0.0, 0.0), "printed": (case["m"], 0.0, 0.0, 0.0, 0.0),
            "potentials": (case["m"], 0.6, 0.5, 0.4, 0.0),
            "sextic": (case["m"], 0.6, 0.5, 0.4, 0.4)}[case["model"]]


def _dt(case):
    """A tenth of the spacing; half of that for the printed form, whose quartic term is stiffer, and
    where the sextic term is present."""
    return (0.05 if case["model"] in ("printed", "sextic") else 0.1) * case["h"]


def _rule(case):
    """The power arrest rule in single precision and for the printed form, else the energy rule."""
    return "power" if case["prec"] == "f32" or case["model"] == "printed" else "energy"


def _jobs(case, seed):
    """The jobs of a batch: lattice, precision, model and where their initial data come from.  The
    lattices are those of the workload, whatever the seed; the seed draws the fields."""
    if case["mix"] == "scan":
        raw = skyr_inputs.batch_jobs(case["master"], case["jobs"])
    else:
        raw = skyr_inputs.served_stream(case["master"], case["jobs"])
    return [dict(n=j["n"], h=j["h"], m=j["m"], dt=j["dt"], prec=j["precision"], rule=j["flow"], B=j["init"]["B"],
                 seed=seed * 1000 + k) for k, j in enumerate(raw)]


# ------------------------------------------------------------------ prepare and run
def _prec(name):
    return skyr.F32_BULK if name == "f32" else skyr.F64


def prepare(case, seed):
    if case["kind"] == "batch":
        return _prepare_batch(case, seed)
    if case["kind"] == "block":
        return _prepare_block(case, seed)
    lat = skyr.Lattice((skyr.ctypes.c_int32 * 3)(case["n0"], case["n1"], case["n2"]), 0, case["h"])
    prec = _prec(case["prec"])
    model = skyr.Model(*_couplings(case), skyr.FORM_PRINTED if case["model"] == "printed" else skyr.FORM_EXACT)
    phi = _start(case, seed)
    s = dict(case=case, lat=lat, prec=prec, model=model, work=skyr.new_workspace(lat, prec, DEVICE))
    if case["kind"] == "observe":
        s["phi"] = phi
        if case["what"] == "gradient":
            s["grad"] = torch.zeros_like(phi)
        return s
    if case["padded"]:
        s["layout"] = skyr.batch_layout(lat, prec)
        phi = skyr.to_padded(phi, s["layout"])
    s.update(start=phi, phi=phi.clone(), alt=torch.zeros_like(phi), vel=torch.zeros_like(phi),
             flow=skyr.Flow(_dt(case), 0.0, 1 << 40, 16, skyr.flow_mode(_rule(case))))
    return s


def _prepare_batch(case, seed):
    jobs = _jobs(case, seed)
    groups = {}
    for k, j in enumerate(jobs):  # the jobs of one lattice size and precision share their arrays
        groups.setdefault((j["n"], j["prec"]), []).append(k)
    stacks, at = {}, {}
    for (n, p), members in groups.items():
        lat = skyr.Lattice.cube(n, 0.1)
        lead, pitch = layout = skyr.batch_layout(lat, _prec(p))
        t = [torch.zeros((len(members), n, n, 4, pitch), dtype=_dtype(p), device=DEVICE) for _ in range(4)]
        for i, k in enumerate(members):
            f = _field((n, n, n), jobs[k]["h"], "random", jobs[k]["B"], random.Random(jobs[k]["seed"]))
            t[0][i] = skyr.to_padded(f.to(_dtype(p)), layout)
            at[k] = (n, p, i)
        stacks[n, p] = dict(start=t[0], phi=t[1], alt=t[2], vel=t[3], layout=layout)
    flows = []
    for k, j in enumerate(jobs):
        n, p, i = at[k]
        st = stacks[n, p]
        lat = skyr.Lattice.cube(n, j["h"])
        flows.append((lat, _prec(p), skyr.Model(j["m"]),
                      skyr.Flow(j["dt"], 0.0, case["steps"], 16, skyr.flow_mode(j["rule"])), st["phi"][i], st["alt"][i],
                      st["vel"][i], skyr.new_workspace(lat, _prec(p), DEVICE), st["layout"]))
    return dict(case=case, stacks=stacks, flows=flows, batch=skyr.Batch(len(jobs)))


def _prepare_block(case, seed):
    e, o = case["extent"], (case["o0"], case["o1"], case["o2"])
    whole = _start(case, seed)
    prec = _prec(case["prec"])
    lat = skyr.Lattice((skyr.ctypes.c_int32 * 3)(case["n0"], case["n1"], case["n2"]), 0, case["h"])
    blk = skyr.Block.of(lat, o, (e, e, e))
    at = [torch.arange(o[d] - 4, o[d] + e + 4, device=DEVICE).clamp(0, whole.shape[d + 1] - 1) for d in range(3)]
    padded = whole[:, at[0][:, None, None], at[1][None, :, None], at[2][None, None, :]].contiguous()
    own = torch.zeros(padded.shape[1:], dtype=torch.bool, device=DEVICE)
    own[4:-4, 4:-4, 4:-4] = True
    shell = padded[:, ~own].contiguous()
    phi = torch.zeros_like(padded)
    phi[:, own] = padded[:, own]
    return dict(case=case, blk=blk, prec=prec, model=skyr.Model(case["m"]), phi=phi, shell=shell,
                out=torch.zeros_like(phi), vel=torch.zeros_like(phi),
                work=skyr.new_block_workspace(blk, prec, DEVICE))


def run(s):
    return {"flow": _run_flow, "batch": _run_batch, "observe": _run_observe, "block": _run_block}[s["case"]["kind"]](s)


def _run_flow(s):
    """A relaxation from the initial data: a copy of the field, no velocity, a fresh state."""
    s["phi"].copy_(s["start"])
    s["vel"].zero_()
    st = skyr.anf_state()
    args = (s["lat"], s["prec"], s["model"], s["flow"], s["phi"], s["alt"], s["vel"], st, s["case"]["steps"], s["work"])
    if s["case"]["padded"]:
        skyr.anf_step_padded(*args, s["layout"])
        lead, n = s["layout"][0], s["case"]["n2"]
        phi, vel = (s[k][..., lead:lead + n].permute(2, 0, 1, 3) for k in ("phi", "vel"))
    else:
        skyr.anf_step(*args)
        phi, vel = s["phi"], s["vel"]
    return {"phi": phi, "vel": vel, "E": st.E, "max_force": st.max_force, "steps": st.steps, "arrests": st.arrests}


def _run_batch(s):
    """Every job admitted, ticks until all have stopped, every job polled and retired."""
    for st in s["stacks"].values():
        st["phi"].copy_(st["start"])
        st["vel"].zero_()
    b = s["batch"]
    slots = [b.add_padded(*f) for f in s["flows"]]
    states = []
    while not states or any(st.steps < s["case"]["steps"] and not st.nonfinite for st in states):
        b.run(TICK)
        states = [b.poll(k) for k in slots]
    for k in slots:
        b.remove(k)
    out = {}
    for (n, p), st in s["stacks"].items():
        lead = st["layout"][0]
        out["%d-%s" % (n, p)] = {k: st[k][..., lead:lead + n].permute(0, 3, 1, 2, 4) for k in ("phi", "vel")}
    out["states"] = {"E": torch.tensor([st.E for st in states], dtype=torch.float64),
                     "steps": torch.tensor([st.steps for st in states]),
                     "arrests": torch.tensor([st.arrests for st in states])}
    return out


def _run_observe(s):
    a = (s["lat"], s["prec"], s["model"], s["phi"], s["work"])
    if s["case"]["what"] == "moments":
        return skyr.moments(*a)
    if s["case"]["what"] == "observables":
        return skyr.observables(*a)
    parts = skyr.energy_gradient(*a, grad=s["grad"])
    return {"grad": s["grad"], **{k: parts[k] for k in ("E", "E2", "E4", "E0", "virial", "max_force")}}


def _run_block(s):
    sums = skyr.block_sweep(s["blk"], s["prec"], s["model"], skyr.BLOCK_STEP, s["phi"], s["shell"], s["out"],
                            vel=s["vel"], work=s["work"], dt=_dt(s["case"]))
    own = (slice(None),) + (slice(4, -4),) * 3
    return {"phi": s["out"][own], "vel": s["vel"][own], "E": sums["E"], "max_force": sums["max_force"]}


# ------------------------------------------------------------------ the same in 64 bits
def _shift(f, axis, k, axes=(0, 1, 2)):
    """f (leading dimension: components) moved by k along one axis, two sites cut off both ends of `axes`."""
    i = [slice(None)] * 4
    for d in axes:
        i[d + 1] = slice(2 + (k if d == axis else 0), f.shape[d + 1] - 2 + (k if d == axis else 0))
    return f[tuple(i)]


def _d1(f, axis, h, axes=(0, 1, 2)):
    return (8 * (_shift(f, axis, 1, axes) - _shift(f, axis, -1, axes))
            - (_shift(f, axis, 2, axes) - _shift(f, axis, -2, axes))) / (12 * h)


def _d2(f, axis, h):
    return (16 * (_shift(f, axis, 1) + _shift(f, axis, -1)) - (_shift(f, axis, 2) + _shift(f, axis, -2))
            - 30 * _shift(f, axis, 0)) / (12 * h * h)


def _det(c, a):
    m = torch.stack([c, *a], dim=-1).movedim(0, -2)  # the four vectors as columns
    if m.requires_grad:  # by minors: the derivative of linalg.det needs an inverse
        def minor(p, q, i, j):
            return m[..., i, p] * m[..., j, q] - m[..., j, p] * m[..., i, q]
        s = 0
        for i, j, k, l, sign in ((0, 1, 2, 3, 1), (0, 2, 1, 3, -1), (0, 3, 1, 2, 1), (1, 2, 0, 3, 1),
                                 (1, 3, 0, 2, -1), (2, 3, 0, 1, 1)):
            s = s + sign * minor(0, 1, i, j) * minor(2, 3, k, l)
        return s
    return torch.linalg.det(m)


def _energies(phi, h, couplings):
    """h^3 sums of the energy parts E2, E4, E0, E6 over the interior."""
    m, my, mz, mw, c6 = couplings
    c = _shift(phi, 0, 0)
    a = [_d1(phi, d, h) for d in range(3)]
    e2 = -0.5 * sum((c * _d2(phi, d, h)).sum() for d in range(3))
    G = [[(a[i] * a[j]).sum(0) if j >= i else None for j in range(3)] for i in range(3)]
    e4 = 0.5 * (G[0][0] * G[1][1] + G[0][0] * G[2][2] + G[1][1] * G[2][2]
                - G[0][1] ** 2 - G[0][2] ** 2 - G[1][2] ** 2).sum()
    u = 1 - c[0]
    e0 = (m * m * u + 0.5 * my * my * (1 - c[0] ** 2) + 0.5 * mz * mz * u ** 2 + 0.25 * mw * mw * u ** 4).sum()
    e6 = 0.5 * c6 * (_det(c, a) ** 2).sum() if c6 else torch.zeros_like(e2)
    return [e * h ** 3 for e in (e2, e4, e0, e6)]


def _gradient(phi, h, couplings, printed=False):
    """(energy parts, density gradient on the interior)."""
    if not printed:
        p = phi.clone().requires_grad_(True)
        parts = _energies(p, h, couplings)
        g, = torch.autograd.grad(sum(parts), p)
        return [float(e.detach()) for e in parts], _shift(g, 0, 0) / h ** 3
    # the printed Euler-Lagrange expression, mixed derivatives as products of first differences
    with torch.no_grad():
        parts = [float(e) for e in _energies(phi, h, couplings)]
        a = [_d1(phi, d, h) for d in range(3)]
        D = [[None] * 3 for _ in range(3)]
        for i in range(3):
            D[i][i] = _d2(phi, i, h)
            for j in range(i + 1, 3):
                other = [d for d in range(3) if d != j]
                D[i][j] = D[j][i] = _d1(_d1(phi, j, h, axes=(j,)), i, h, axes=tuple(other))
        lap = D[0][0] + D[1][1] + D[2][2]
        G = [[(a[i] * a[j]).sum(0) for j in range(3)] for i in range(3)]
        g = -(1 + G[0][0] + G[1][1] + G[2][2]) * lap
        for i in range(3):
            ci = sum((D[i][j] * a[j]).sum(0) for j in range(3)) - (lap * a[i]).sum(0)
            g -= ci * a[i]
            for j in range(3):
                g += G[i][j] * D[i][j]
        g[0] -= couplings[0] ** 2
        return parts, g


def _force(phi, h, couplings, printed=False):
    parts, g = _gradient(phi, h, couplings, printed)
    c = _shift(phi, 0, 0)
    return parts, (g * c).sum(0) * c - g


def _relax(phi, h, couplings, dt, rule, steps, printed=False):
    """`steps` accepted steps of the arrested Newton flow from rest."""
    phi = phi.double().clone()
    inner = (slice(None),) + (slice(2, -2),) * 3
    vel = torch.zeros_like(phi)
    E_prev, E, most = math.inf, math.nan, math.nan
    for _ in range(steps):
        parts, F = _force(phi, h, couplings, printed)
        E, v = sum(parts), vel[inner]
        most = float((F * F).sum(0).max().sqrt())
        if E > E_prev if rule == "energy" else float((F * v).sum()) < 0.0:
            v = torch.zeros_like(v)
        v = v + dt * F
        q = phi[inner] + dt * v
        phi[inner] = q / (q * q).sum(0).sqrt()
        vel[inner] = v
        E_prev = E
    return phi, vel, E, most


def exact(case, seed):
    if case["kind"] == "batch":
        return _exact_batch(case, seed)
    phi = _start(case, seed).double()
    h, k, printed = case["h"], _couplings(case), case["model"] == "printed"
    if case["kind"] == "flow":
        phi, vel, E, most = _relax(phi, h, k, _dt(case), _rule(case), case["steps"], printed)
        return {"phi": phi, "vel": vel, "E": E, "max_force": most, "steps": None, "arrests": None}
    if case["kind"] == "observe" and case["what"] == "moments":
        return _exact_moments(phi, h, k)
    parts, F = _force(phi, h, k, printed)
    most = float((F * F).sum(0).max().sqrt())
    if case["kind"] == "observe":
        E2, E4, E0, E6 = parts
        out = {"E": sum(parts), "E2": E2, "E4": E4, "E0": E0, "virial": E2 - E4 + 3 * E0 - 3 * E6, "max_force": most}
        if case["what"] == "gradient":
            out["grad"] = torch.zeros_like(phi)
            out["grad"][:, 2:-2, 2:-2, 2:-2] = _gradient(phi, h, k, printed)[1]
            return out
        det = _det(_shift(phi, 0, 0), [_d1(phi, d, h) for d in range(3)])
        return {**out, "E6": None, "B": -float(det.sum()) * h ** 3 / (2 * math.pi ** 2)}
    # the block's share of one step from rest: nothing is written on the frozen layers
    own = tuple(slice(case[o], case[o] + case["extent"]) for o in ("o0", "o1", "o2"))
    vel, out = torch.zeros_like(phi), torch.zeros_like(phi)
    inner = (slice(None),) + (slice(2, -2),) * 3
    vel[inner] = _dt(case) * F
    q = phi[inner] + _dt(case) * vel[inner]
    out[inner] = q / (q * q).sum(0).sqrt()
    force = torch.zeros_like(phi)
    force[inner] = F
    return {"phi": out[(slice(None),) + own], "vel": vel[(slice(None),) + own], "E": None,
            "max_force": float((force[(slice(None),) + own] ** 2).sum(0).max().sqrt())}


def _exact_batch(case, seed):
    out, E = {}, []
    for j in _jobs(case, seed):
        f = _field((j["n"],) * 3, j["h"], "random", j["B"], random.Random(j["seed"])).to(_dtype(j["prec"]))
        phi, vel, e, _ = _relax(f, j["h"], (j["m"], 0.0, 0.0, 0.0, 0.0), j["dt"], j["rule"], case["steps"])
        o = out.setdefault("%d-%s" % (j["n"], j["prec"]), {"phi": [], "vel": []})
        # as the arrays of one lattice size are laid out: job, component, x, y, z
        o["phi"].append(phi)
        o["vel"].append(vel)
        E.append(e)
    out = {g: {k: torch.stack(v) for k, v in o.items()} for g, o in out.items()}
    out["states"] = {"E": torch.tensor(E, dtype=torch.float64), "steps": None, "arrests": None}
    return out


def _exact_moments(phi, h, couplings):
    """Charge, energy and the moments of Sec. 5 in the printed normalisation."""
    dev = phi.device
    c = _shift(phi, 0, 0)
    a = [_d1(phi, d, h) for d in range(3)]
    b = -_det(c, a) / (2 * math.pi ** 2)
    r = [((torch.arange(n, dtype=torch.float64, device=dev) - 0.5 * (n - 1)) * h)[2:-2] for n in phi.shape[1:]]
    r = [r[0][:, None, None], r[1][None, :, None], r[2][None, None, :]]
    B = float(b.sum())
    X = [float((x * b).sum()) / B for x in r]
    r = torch.stack([(x - x0).expand(b.shape) for x, x0 in zip(r, X)])
    conj = [c[0], -c[1], -c[2], -c[3]]
    L = [_qmul(conj, d) for d in a]  # U^dagger d_i U
    zero = torch.zeros_like(c[0])
    T = []
    for j in range(3):  # (i/2) U^dagger [tau_j, U], with [tau_j, U] = -2 (e_j x phi).tau
        e = [zero] * 3
        e[(j + 1) % 3], e[(j + 2) % 3] = c[1 + (j + 2) % 3], -c[1 + (j + 1) % 3]
        T.append(torch.stack(_qmul(conj, [zero, *e])[1:]))
    s = torch.stack([q[0] for q in L])
    l = torch.stack([torch.stack(q[1:]) for q in L])
    T = torch.stack(T)
    dot = lambda p, q: (p[:, None] * q[None]).sum(2)  # noqa: E731  (3, 3, sites) of two sets of 3-vectors
    G, M = dot(l, l), dot(l, T)
    S = G[0, 0] + G[1, 1] + G[2, 2]
    mul = lambda p, q: (p[:, :, None] * q[None]).sum(1)  # noqa: E731  matrix product per site
    t = lambda p: p.transpose(0, 1)  # noqa: E731
    U = 2 * (1 + S) * dot(T, T) - 2 * mul(t(M), M)
    K = 2 * (G - s[:, None] * s[None]) + 2 * (S * G - mul(G, G))
    R = torch.stack([torch.stack([zero, -r[2], r[1]]), torch.stack([r[2], zero, -r[0]]),
                     torch.stack([-r[1], r[0], zero])])
    V = mul(mul(R, K), t(R))
    W = -2 * t(mul(R, (1 + S) * M - mul(G, M)))
    trK = K[0, 0] + K[1, 1] + K[2, 2]
    D = sum(r[i] * K[i, j] * r[j] for i in range(3) for j in range(3)) - (r * r).sum(0) * trK / 3
    total = lambda p: (p.sum((-1, -2, -3)) * h ** 3).cpu().numpy()  # noqa: E731
    Q2 = total(r[:, None] * r[None] * b)
    E = 2 * sum(float(e) for e in _energies(phi, h, couplings))
    tr = Q2[0, 0] + Q2[1, 1] + Q2[2, 2]
    Q = 0.5 * (3 * Q2 - tr * torch.eye(3, dtype=torch.float64).numpy())
    return {"B": B * h ** 3, "E": E, "X": torch.tensor(X, dtype=torch.float64).numpy(),
            "R": math.sqrt(tr / (B * h ** 3)), "U": total(U), "V": total(V), "W": total(W), "Q": Q,
            "D": -(2 * E / 5) * float(D.sum()) * h ** 3}
