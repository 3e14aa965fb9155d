"""The work that users of this library have it do, as timed cases.

Four kinds of call, each through the public Python entry points:

  solve   a QUBO that lives in HBM, one ``DeviceSolver.run()``: Ising
          preparation, start draw, every step, energies, best agent
  host    a QUBO in host memory, one ``solve()`` (upload, solve, download)
  batch   many events solved together, one ``DeviceBatchSolver.run()``
  build   hits in host memory to a QUBO, one ``build_qubo_gpu()``

Events are charged helices in a 2 T barrel with smeared and noise hits, the
input this repository's own workloads use; their sizes (10, 200, 1000 and
5000 particles, 20 to 1000 particles per event of a batch) and agent and step
counts are those workloads' too.  A case names its event, and the seed turns
it about the beam axis by an angle of its own (every hit, its place in the
hit order and so every index and coupling of the QUBO is another one, while
sizes stay the case's) and seeds the solver.  ``exact`` integrates in 64 bits from the
same start; for runs of more than ``EXACT_STEPS`` steps it gives only the
scalars, because each sign or wall decision that 32 bits take differently
there starts another trajectory.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2402_14718_amd as sbt

EXACT_STEPS = 60
RADII = (32.0, 72.0, 116.0, 172.0, 260.0, 360.0, 500.0, 660.0, 820.0, 1020.0)
TAN_0P1 = 0.10033467208545055
Z0_CUT = 300.0   # doublet cut (mm) of the densest events


# ------------------------------------------------------------------ cases

def _solve(name, particles, mode, agents, steps, **more):
    return dict({"name": name, "kind": "solve", "event": "plain", "particles": particles,
                 "mode": mode, "agents": agents, "steps": steps, "precision": "fp32",
                 "dt": 1.0, "every": 0, "state": False}, **more)


def listed():
    return [
        # the smallest call: a four-layer toy event, default agents and steps
        _solve("tiny_dsb", 10, "dsb", 32, 2000, event="tiny"),
        # an ordinary event at the paper's settings, ballistic and discrete;
        # the second records energies for time-to-target
        _solve("plain_bsb", 200, "bsb", 256, 5000),
        _solve("plain_dsb_trace", 200, "dsb", 256, 5000, every=50),
        # a first call from host memory with the default agents and steps
        {"name": "host_bsb", "kind": "host", "event": "plain", "particles": 450, "mode": "bsb",
         "agents": 32, "steps": 2000, "precision": "fp32", "dt": 1.0},
        # between the ordinary and the large event, an odd number of agents
        _solve("mid_dsb", 700, "dsb", 250, 2000),
        # the large event, both forms, all agents' final state wanted
        _solve("large_bsb", 1000, "bsb", 1024, 1000, state=True),
        _solve("large_dsb", 1000, "dsb", 1024, 1000, state=True),
        # the densest event, narrow couplings: a stretch of a long solve
        _solve("dense_bsb", 5000, "bsb", 512, 20, event="dense", precision="fp8_block", state=True),
        _solve("dense_dsb", 5000, "dsb", 512, 40, event="dense", precision="fp8", state=True),
        # a batch of events of every size, and one of small events
        {"name": "batch_dsb", "kind": "batch", "events": 128, "from": 20, "to": 1000,
         "mode": "dsb", "agents": 128, "steps": 3000, "precision": "bf16", "dt": 1.0, "every": 0,
         "state": False},
        {"name": "batch_bsb", "kind": "batch", "events": 96, "from": 20, "to": 400,
         "mode": "bsb", "agents": 100, "steps": 1000, "precision": "fp16", "dt": 1.0, "every": 0,
         "state": True},
        # hits to QUBO
        {"name": "build", "kind": "build", "event": "plain", "particles": 1000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "batch", "batch", "dense", "host", "build"])
    mode = rng.choice(["bsb", "dsb"])
    if kind == "build":
        return {"kind": "build", "event": "plain", "particles": _log_int(rng, 15, 1500)}
    if kind == "dense":
        p = rng.randint(2500, 5000)
        return {"kind": "solve", "event": "dense", "particles": p, "mode": mode,
                "agents": _log_int(rng, 100, 512), "steps": rng.randint(4, 20),
                "precision": rng.choice(["fp32", "fp8", "fp8_block", "bf16x2"]), "dt": 1.0,
                "every": 0, "state": True}
    steps = _log_int(rng, 20, 5000)
    dt = rng.choice([1.0, 1.0, 0.5, 0.1])
    if kind == "batch":
        lo = rng.randint(10, 300)
        return {"kind": "batch", "events": _log_int(rng, 2, 96), "from": lo,
                "to": rng.randint(lo, 1000), "mode": mode, "agents": _log_int(rng, 16, 128),
                "steps": min(steps, 3000), "precision": rng.choice(["bf16", "fp16"]), "dt": dt,
                "every": rng.choice([0, 0, 50]), "state": rng.random() < 0.3}
    p = _log_int(rng, 10, 1000)
    if kind == "host":
        return {"kind": "host", "event": "plain", "particles": p, "mode": mode,
                "agents": _log_int(rng, 16, 256), "steps": min(steps, 2000), "precision": "fp32",
                "dt": dt}
    agents = _log_int(rng, 16, 1024)
    # the largest listed solve moves 2e11 couplings and spins
    steps = max(20, min(steps, int(4e10 / (35.0 * p * agents))))
    return {"kind": "solve", "event": "plain", "particles": p, "mode": mode, "agents": agents,
            "steps": steps, "precision": rng.choice(["fp32", "fp32", "fp32", "fp32", "bf16x2", "fp8"]),
            "dt": dt, "every": rng.choice([0, 0, 50]), "state": rng.random() < 0.5}


# ----------------------------------------------------------------- inputs

def _hits(event, particles, seed, number=0):
    """Hits of one event: charged helices from the origin crossing the barrel,
    turned by the seed's angle."""
    rng = np.random.Generator(np.random.PCG64([particles, number]))
    turn = np.random.Generator(np.random.PCG64([seed, number])).uniform(0.0, 2.0 * math.pi)
    tiny, dense = event == "tiny", event == "dense"
    radii = RADII[:4] if tiny else RADII
    lo, hi = (1.0, 10.0) if tiny else (0.5, 20.0)
    eta_max, noise = (1.0, 0.0) if tiny else (2.0, 0.2) if dense else (1.5, 0.1)
    n = particles
    q = np.where(rng.random(n) < 0.5, -1, 1)
    big_r = np.exp(rng.uniform(math.log(lo), math.log(hi), n)) / (0.299792458 * 2.0) * 1000.0
    sinh_eta = np.sinh(rng.uniform(-eta_max, eta_max, n))
    phi0 = rng.uniform(0.0, 2.0 * math.pi, n)
    smear = rng.standard_normal((n, len(radii)))
    parts = []
    for layer, r in enumerate(radii):
        half = 400.0 if tiny else max(400.0, 1.1 * r * math.sinh(eta_max))
        alpha = np.arcsin(np.minimum(1.0, r / (2.0 * big_r)))
        z = 2.0 * big_r * alpha * sinh_eta
        ok = (r < 2.0 * big_r) & (np.abs(z) <= half)
        phi = (phi0 - q * alpha + smear[:, layer] * (0.020 / r))[ok]
        extra = int(round(noise * phi.size))
        phi = np.concatenate([phi, rng.uniform(0.0, 2.0 * math.pi, extra)])
        z = np.concatenate([z[ok], rng.uniform(-half, half, extra)])
        phi = np.mod(phi + turn, 2.0 * math.pi)
        order = np.argsort(phi, kind="stable")
        h = np.zeros(phi.size, dtype=sbt.HIT_DTYPE)
        h["layer"], h["x"], h["y"] = layer, (r * np.cos(phi))[order], (r * np.sin(phi))[order]
        h["z"] = z[order]
        parts.append(h)
    hits = np.concatenate(parts)
    hits["hit_id"] = np.arange(hits.size)
    return hits


def _qubo(event, particles, seed, number=0):
    hits = _hits(event, particles, seed, number)
    p = sbt.build_params_default()
    if event == "dense":
        p.z0_max = Z0_CUT
    q = sbt.build_qubo_gpu(hits, p)[0]
    # the densest event is relabelled by azimuth, as its solves are run
    return sbt.permute_qubo(q, sbt.phi_order(q, hits)) if event == "dense" else q


def _batch_qubos(case, seed):
    rng = np.random.Generator(np.random.PCG64(999))
    counts = rng.integers(case["from"], case["to"] + 1, case["events"])
    return [_qubo("plain", int(c), seed, k) for k, c in enumerate(counts)]


def _params(case, seed):
    return sbt.solve_params(agents=case["agents"], steps=case["steps"], dt=case["dt"], seed=seed,
                            energy_every=case.get("every", 0),
                            precision=case["precision"] if case["kind"] != "batch" else "fp32")


def prepare(case, seed):
    kind = case["kind"]
    if kind == "build":
        return {"case": case, "hits": _hits(case["event"], case["particles"], seed)}
    if kind == "batch":
        return {"case": case,
                "solver": sbt.DeviceBatchSolver(_batch_qubos(case, seed), case["mode"],
                                                case["precision"], _params(case, seed),
                                                want_agent_energy=True,
                                                want_trace=case["every"] > 0,
                                                want_agent_state=case["state"])}
    q = _qubo(case["event"], case["particles"], seed)
    if kind == "host":
        return {"case": case, "qubo": q, "seed": seed}
    return {"case": case,
            "solver": sbt.DeviceSolver(q, case["mode"], _params(case, seed),
                                       want_state=case["state"], want_trace=case["every"] > 0)}


# -------------------------------------------------------------------- run

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "build":
        q, _ = sbt.build_qubo_gpu(state["hits"])
        return {"a": q.a, "row_ptr": q.row_ptr, "col": q.col, "b": q.b, "trip_hits": q.trip_hits}
    if kind == "host":
        r = sbt.solve(state["qubo"], case["mode"], agents=case["agents"], steps=case["steps"],
                      dt=case["dt"], seed=state["seed"], precision=case["precision"])
        return {k: r[k] for k in ("T", "agent_energy", "energy", "best_agent", "c0", "ising_offset")}
    s = state["solver"]
    s.run()
    if kind == "batch":
        out = {"energy": s.best_energy, "best_agent": s.best_agent, "T": s.best_T,
               "offset": s.offset, "agent_energy": s.agent_energy, "agent_T": s.agent_T,
               "agent_x": s.agent_x, "trace": s.trace}
    else:
        out = {"energy": s.best_energy, "best_agent": s.best_agent, "T": s.T,
               "scalars": s.scalars, "agent_energy": s.agent_energy, "x": s.x, "y": s.y,
               "trace": s.trace}
    return {k: v for k, v in out.items() if v is not None}


# ------------------------------------------------------------------- work

def work(case):
    """Each input read once, each output written once; the state of an event
    that no chip memory holds (register files and LDS: 168 MB) read and
    written once per step.  Two operations per coupling, eight per update."""
    kind = case["kind"]
    if kind == "build":
        q = _qubo(case["event"], case["particles"], 1)
        h = _hits(case["event"], case["particles"], 1)
        return {"bytes": 40 * h.size + 40 * q.n + 12 * q.nnz, "flops": 60 * q.n + 30 * q.nnz}
    if kind == "batch":
        few = dict(case, events=min(case["events"], 16))
        qs = _batch_qubos(few, 1)
        scale = case["events"] / len(qs)
        n, nnz, events = scale * sum(q.n for q in qs), scale * sum(q.nnz for q in qs), case["events"]
    else:
        q = _qubo(case["event"], case["particles"], 1)
        n, nnz, events = q.n, q.nnz, 1
    M, K = case["agents"], case["steps"]
    size = 12 * n + 12 * nnz + n + 8 * M * events
    if case.get("state"):
        size += (5 if kind == "batch" else 8) * n * M
    if kind != "batch" and 8 * n * M > 168e6:
        size += 16 * n * M * K
    return {"bytes": size, "flops": K * M * (2 * nnz + 8 * n)}


# ------------------------------------------------------------------ exact

def _rounded(J, row, start, precision):
    """The stored couplings of a form (FP64 values): J of each entry, its row
    and its place in the row."""
    f32 = J.to(torch.float32)
    if precision == "fp32":
        return f32.double()
    if precision == "fp16":
        return J.to(torch.float16).double()
    if precision == "bf16":
        return f32.to(torch.bfloat16).double()
    if precision == "bf16x2":
        hi = f32.to(torch.bfloat16).float()
        return hi.double() + (f32 - hi).to(torch.bfloat16).double()
    # E4M3 with one scale per row, or per eight consecutive entries of a row
    group = row if precision == "fp8" else torch.unique(row * (1 << 31) + start // 8,
                                                        return_inverse=True)[1]
    top = torch.zeros(int(group.max()) + 1, dtype=torch.float32, device=J.device)
    top = top.scatter_reduce(0, group, f32.abs(), "amax")
    scale = torch.where(top > 0, top / 448.0, torch.ones_like(top))[group]
    code = (f32 / scale).clamp(-448.0, 448.0).to(torch.float8_e4m3fn)
    return (scale * code.float()).double()


def _start(n, M, event, seed, dev):
    """Philox4x32-10 start: x0, y0 in [-1/8, 1/8) for every spin and agent."""
    mask = 0xFFFFFFFF
    c0 = torch.arange(n, dtype=torch.int64, device=dev)[:, None].expand(n, M)
    c1 = torch.arange(M, dtype=torch.int64, device=dev)[None, :].expand(n, M)
    c2 = torch.full((1, 1), event, dtype=torch.int64, device=dev).expand(n, M)
    c3 = torch.zeros((1, 1), dtype=torch.int64, device=dev).expand(n, M)
    k0, k1 = seed & mask, (seed >> 32) & mask
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((p1 >> 32) & mask) ^ c1 ^ k0, p1 & mask,
                          ((p0 >> 32) & mask) ^ c3 ^ k1, p0 & mask)
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return [((v >> 8) - (1 << 23)).double() * 2.0 ** -26 for v in (c0, c1)]


def _energies(q, x, row, col, dev):
    """O(T) of every agent for T = (x >= 0)."""
    T = (x >= 0).double()
    a, b = torch.tensor(q.a, device=dev), torch.tensor(q.b, device=dev)
    e = a @ T
    upper = torch.nonzero(col > row).reshape(-1)
    for s in range(0, upper.numel(), 1 << 20):
        k = upper[s:s + (1 << 20)]
        e = e + (b[k][:, None] * T[row[k]] * T[col[k]]).sum(0)
    return e


def _trajectory(q, case, event, seed):
    """(scalars, x, y, energies) of one event; the last three None for runs
    past EXACT_STEPS."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    n, M, K = q.n, case["agents"], case["steps"]
    b = torch.tensor(q.b, device=dev)
    rp = torch.tensor(q.row_ptr, device=dev)
    col = torch.tensor(q.col, dtype=torch.int64, device=dev)
    row = torch.repeat_interleave(torch.arange(n, device=dev), rp[1:] - rp[:-1])
    J = -0.25 * b
    rowsum = torch.zeros(n, dtype=torch.float64, device=dev).index_add_(0, row, b)
    h = -(0.5 * torch.tensor(q.a, device=dev) + 0.25 * rowsum)
    mean, square = J.sum() / n ** 2, (J * J).sum() / n ** 2
    sd = math.sqrt(max(0.0, float(square - mean * mean)))
    c0 = 0.5 / (math.sqrt(n) * sd) if sd > 0 else 0.5 / math.sqrt(n)
    offset = 0.5 * float(q.a.sum()) + 0.25 * float(b[col > row].sum())
    scalars = torch.tensor([c0, offset, float(J.sum()), float((J * J).sum())], dtype=torch.float64)
    if K > EXACT_STEPS:
        return scalars, None, None, None
    Jq = _rounded(J, row, torch.arange(col.numel(), device=dev) - rp[row], case["precision"])
    A = torch.sparse_csr_tensor(rp, col, Jq, size=(n, n)) if col.numel() else None
    x, y = _start(n, M, event, seed, dev)
    for k in range(K):
        s = x if case["mode"] == "bsb" else torch.where(x >= 0, 1.0, -1.0).double()
        F = h[:, None] + (A @ s if A is not None else 0.0)
        y = y + case["dt"] * (c0 * F - (1.0 - k / K) * x)
        x = x + case["dt"] * y
        wall = x.abs() > 1.0
        x, y = x.clamp(-1.0, 1.0), torch.where(wall, 0.0, y)
    return scalars, x, y, _energies(q, x, row, col, dev)


def _build_exact(hits):
    """a and b of the QUBO (the other outputs are whole numbers), from an
    enumeration over all pairs and joins."""
    x, y, z, layer = hits["x"], hits["y"], hits["z"], hits["layer"]
    H = hits.size
    pairs = []
    for L in range(int(layer.max())):
        i, j = np.nonzero(layer == L)[0], np.nonzero(layer == L + 1)[0]
        cross = x[i][:, None] * y[j] - y[i][:, None] * x[j]
        dot = x[i][:, None] * x[j] + y[i][:, None] * y[j]
        u, v = np.nonzero((dot > 0) & (np.abs(cross) < TAN_0P1 * dot))
        pairs.append(np.stack([i[u], j[v]], 1))
    d = np.concatenate(pairs)
    d = d[np.lexsort((d[:, 1], d[:, 0]))]

    def join(left, right):
        """(i, j) for which left[i] == right[j]; right ascending."""
        lo, hi = np.searchsorted(right, left), np.searchsorted(right, left, "right")
        i = np.repeat(np.arange(left.size), hi - lo)
        return i, np.arange(i.size) - np.repeat(np.cumsum(hi - lo) - (hi - lo), hi - lo) + lo[i]

    i, j = join(d[:, 1], d[:, 0])
    t = np.stack([d[i, 0], d[i, 1], d[j, 1]], 1)
    ux, uy, wx, wy = (v[t[:, k]] - v[t[:, 0]] for k, v in ((1, x), (1, y), (2, x), (2, y)))
    vx, vy = x[t[:, 2]] - x[t[:, 1]], y[t[:, 2]] - y[t[:, 1]]
    nw = np.sqrt(wx * wx + wy * wy)
    kappa = 2.0 * (ux * vy - uy * vx) / (np.sqrt(ux * ux + uy * uy) * np.sqrt(vx * vx + vy * vy) * nw)
    r = np.sqrt(x * x + y * y)
    r1, r2, r3 = (r[t[:, k]] for k in range(3))
    z1, z2, z3 = (z[t[:, k]] for k in range(3))
    tc = (r2 - r1) * (z3 - z2) - (z2 - z1) * (r3 - r2)
    td = (r2 - r1) * (r3 - r2) + (z2 - z1) * (z3 - z2)
    ok = (np.abs(kappa) <= 8e-4) & (td > 0) & (np.abs(tc) <= TAN_0P1 * td)
    bb, cc, den = ux * ux + uy * uy, wx * wx + wy * wy, 2.0 * (ux * wy - uy * wx)
    with np.errstate(divide="ignore", invalid="ignore"):
        ox, oy = (wy * bb - uy * cc) / den, (ux * cc - wx * bb) / den
        d0 = np.abs(np.hypot(x[t[:, 0]] + ox, y[t[:, 0]] + oy) - np.hypot(ox, oy))
    d0 = np.where(den != 0, d0, np.abs(x[t[:, 0]] * wy - y[t[:, 0]] * wx) / nw)
    z0 = z1 - r1 * (z2 - z1) / (r2 - r1)
    a = 0.5 * (1.0 - np.exp(-d0)) + 0.2 * (1.0 - np.exp(-np.abs(z0) / 0.5))
    t, kappa, dth, a = t[ok], kappa[ok], np.arctan2(np.abs(tc), td)[ok], a[ok]
    i, j = join(t[:, 1] * H + t[:, 2], t[:, 0] * H + t[:, 1])
    dk = np.abs(kappa[i] - kappa[j])
    s = 1.0 - 0.5 * (dk + np.maximum(dth[i], dth[j]))
    ok = (dk <= 1e-4) & (s > 0.2)
    i, j, s = i[ok], j[ok], s[ok]
    longer = np.isin(j, i) | np.isin(i, j)   # five hits: (i, j) goes on, or came from before
    i, j, s = i[longer], j[longer], s[longer]
    alive = np.unique(np.concatenate([i, j]))
    i, j, t, a, n = np.searchsorted(alive, i), np.searchsorted(alive, j), t[alive], a[alive], alive.size
    # conflicts: pairs that share a hit and are not windows of one chain
    who, at = np.tile(np.arange(n), 3), np.concatenate([t[:, 0], t[:, 1], t[:, 2]])
    order = np.argsort(at, kind="stable")
    u, v = join(at, at[order])
    u, v = who[u], who[order][v]
    key = np.unique(u[u < v] * n + v[u < v])
    u, v = key // n, key % n
    one = lambda p, q: ((t[p, 1] == t[q, 0]) & (t[p, 2] == t[q, 1])) | (t[p, 2] == t[q, 0])  # noqa: E731
    clash = ~(one(u, v) | one(v, u))
    u, v = np.concatenate([u[clash], i]), np.concatenate([v[clash], j])
    w = np.concatenate([np.ones(int(clash.sum())), -s])
    rows, cols, w = np.concatenate([u, v]), np.concatenate([v, u]), np.concatenate([w, w])
    return a, w[np.lexsort((cols, rows))]


def exact(case, seed):
    kind = case["kind"]
    if kind == "build":
        a, b = _build_exact(_hits(case["event"], case["particles"], seed))
        return {"a": a, "row_ptr": None, "col": None, "b": b, "trip_hits": None}
    if kind == "batch":
        runs = [_trajectory(q, case, e, seed) for e, q in enumerate(_batch_qubos(case, seed))]
        out = {"energy": None, "best_agent": None, "T": None,
               "offset": torch.stack([r[0][1] for r in runs]), "agent_energy": None,
               "agent_T": None, "agent_x": None, "trace": None}
        if case["steps"] <= EXACT_STEPS:
            out["agent_energy"] = torch.cat([r[3] for r in runs])
            out["agent_x"] = torch.cat([r[1].reshape(-1) for r in runs])
        return {k: v for k, v in out.items()
                if not (k in ("agent_T", "agent_x") and not case["state"])
                and not (k == "trace" and not case["every"])}
    q = _qubo(case["event"], case["particles"], seed)
    scalars, x, y, e = _trajectory(q, case, 0, seed)
    if kind == "host":
        return {"T": None, "agent_energy": e, "energy": None, "best_agent": None,
                "c0": float(scalars[0]), "ising_offset": float(scalars[1])}
    out = {"energy": None, "best_agent": None, "T": None, "scalars": scalars, "agent_energy": e}
    if case["state"]:
        out.update(x=x, y=y)
    if case["every"] and case["steps"] >= case["every"]:
        out["trace"] = None
    return out
