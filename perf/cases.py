"""Performance cases: what users of the library have it integrate, through the public binding.

Every pass starts from an initial state on the GPU (nd_set_state), integrates it (nd_run, nd_run_batch,
nd_run_adaptive, nd_run_adaptive_dense, or the server's submit / pump / result) and reads the results back
where the caller wants them: on the GPU for the handles, in host memory for the adaptive statistics and
the server.  Handles, topologies and output buffers are made once, as a program that integrates many
initial states does.  Sizes follow the package's benchmark workloads and tests, or are generic.
"""
import math
import random

import numpy as np
import torch

from paper_2410_19075_amd import nd

KURAMOTO, INERTIA, FHN = "kuramoto", "inertia", "fhn"
MODELS = {KURAMOTO: nd.ND_KURAMOTO, INERTIA: nd.ND_KURAMOTO_INERTIA, FHN: nd.ND_FHN}
NVARS = {KURAMOTO: 1, INERTIA: 2, FHN: 2}
INERTIA_PRM = [0.0, 0.01, 0.45, 1.0, 0.05]  # omega, mu, alpha, m, eps
FHN_PRM = [0.05, 0.5, 0.1, math.pi / 2 - 0.1]  # eps, a, sigma, phi
HH_PRM = [1.0, 120.0, 36.0, 0.3, 50.0, -77.0, -54.387, 0.0, 0.0, 2.0]
DEV = "cuda"


# ------------------------------------------------------------------------------------------- cases
def ring(model, n, P, batch, steps, fp32=False, record=0, mv=False, alpha=1.46):
    return {"family": "ring", "model": model, "n": n, "P": P, "batch": batch, "steps": steps, "fp32": fp32,
            "record": record, "mv": mv, "alpha": alpha}


def lattice(family, model, n1, n2, n3, radius, steps, fp32=False, record=0, alpha=0.8):
    return {"family": family, "model": model, "n1": n1, "n2": n2, "n3": n3, "radius": radius, "steps": steps,
            "fp32": fp32, "record": record, "alpha": alpha}


def hh(n, degree, steps, fp32=False):
    return {"family": "hh", "n": n, "degree": degree, "steps": steps, "fp32": fp32}


def links(n1, n2, n3, radius, steps, fp32=False, t_end=0.0, rtol=0.0, t_out=0.0):
    """The ball given as a binary matrix; t_end > 0: the adaptive solver instead of `steps` RK4 steps."""
    return {"family": "links", "n1": n1, "n2": n2, "n3": n3, "radius": radius, "steps": steps, "fp32": fp32,
            "t_end": t_end, "rtol": rtol, "t_out": t_out}


def small_world(n, P, shortcuts, steps, fp32=False):
    return {"family": "small_world", "n": n, "P": P, "shortcuts": shortcuts, "steps": steps, "fp32": fp32}


def adaptive(model, n, P, batch, t_end, rtol, alpha=1.46):
    return {"family": "adaptive", "model": model, "n": n, "P": P, "batch": batch, "t_end": t_end, "rtol": rtol,
            "alpha": alpha}


def serve(count, log2_max, steps_min, steps_max, mix):
    return {"family": "serve", "count": count, "log2_max": log2_max, "steps_min": steps_min,
            "steps_max": steps_max, "mix": mix}


def listed():
    return [
        # one small ring with its order parameter recorded: a user exploring parameters interactively
        {"name": "ring_1024_one", **ring(KURAMOTO, 1024, 256, 1, 200, record=10)},
        # a parameter sweep of small rings in one batched call
        {"name": "rings_1024_x512", **ring(KURAMOTO, 1024, 256, 512, 2000)},
        # one FitzHugh-Nagumo ring at the benchmark's size with both observables (chimera profiles)
        {"name": "fhn_65536_one", **ring(FHN, 65536, 22937, 1, 100, record=10, mv=True)},
        # the benchmark's batch of such rings, seeds of one ensemble
        {"name": "fhn_65536_x64", **ring(FHN, 65536, 22937, 64, 10)},
        # a burst of simulations of mixed model, size, horizon and precision on the server
        {"name": "serve_rings_x24", **serve(24, 16, 300, 1000, 1)},
        # the default benchmark: the 200^3 lattice, cube of half-width 4
        {"name": "cube_200_h4", **lattice("cube", KURAMOTO, 200, 200, 200, 4, 4)},
        # a ragged lattice with inertia, FP32-bulk, R recorded
        {"name": "cube_ragged_h2_fp32", **lattice("cube", INERTIA, 101, 90, 77, 2, 20, True, 5, 0.45)},
        # the 100^3 inertia state with the ball of 33 links
        {"name": "ball_100_p2", **lattice("ball", INERTIA, 100, 100, 100, 2, 20, alpha=0.45)},
        # the same with 925 links
        {"name": "ball_100_p6", **lattice("ball", INERTIA, 100, 100, 100, 6, 10, alpha=0.45)},
        # Hodgkin-Huxley network at the benchmark's degree, a size that one prepares quickly
        {"name": "hh_200k_deg100", **hh(200000, 100, 10)},
        # the adaptive solver with dense output on a 3D state given as a compressed coupling matrix
        {"name": "adaptive_links_60", **links(60, 60, 60, 2, 0, t_end=50.0, rtol=1e-6, t_out=1.0)},
        # the adaptive solver on a sweep of small rings, one launch
        {"name": "adaptive_1024_x512", **adaptive(KURAMOTO, 1024, 256, 512, 20.0, 1e-8)},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    fp32 = rng.random() < 0.35
    alpha = round(rng.uniform(1.3, 1.55), 4)
    kind = rng.choice(["rings_small", "rings_large", "rings_large", "cube", "cube", "ball", "ball", "disk", "hh",
                       "links", "small_world", "adaptive_small", "adaptive_large", "adaptive_links", "serve"])
    if kind == "rings_small":  # rings that one workgroup holds
        n = log_int(65, 4096)
        batch = log_int(1, 512)
        steps = max(50, min(1500, int(1e9 / (n * batch))))
        return ring(rng.choice([KURAMOTO, KURAMOTO, INERTIA, FHN]), n, max(1, int(n * rng.uniform(0.05, 0.4))), batch,
                    steps, fp32, rng.choice([0, 10]), rng.random() < 0.2, alpha)
    if kind == "rings_large":  # rings over many workgroups
        n = log_int(4097, 1 << 20)
        batch = log_int(1, max(1, min(64, (1 << 22) // n)))
        steps = max(5, min(150, int(4e7 / (n * batch))))
        return ring(rng.choice([KURAMOTO, INERTIA, FHN, FHN]), n, max(1, int(n * rng.uniform(0.05, 0.4))), batch, steps,
                    fp32, rng.choice([0, 10]) if steps >= 10 else 0, rng.random() < 0.2, alpha)
    if kind == "cube":
        h = rng.choice([1, 2, 2, 3, 4, 4])
        n1, n2, n3 = (log_int(2 * h + 4, 190) for _ in range(3))
        steps = max(3, min(60, int(2e7 / (n1 * n2 * n3))))
        model = rng.choice([KURAMOTO, INERTIA])
        return lattice("cube", model, n1, n2, n3, h, steps, fp32, rng.choice([0, 3]),
                       0.8 if model == KURAMOTO else 0.45)
    if kind == "ball":
        P = rng.choice([1, 2, 2, 3, 4, 5, 6, 6, 8])
        n1, n2, n3 = (log_int(2 * P + 4, 110) for _ in range(3))
        steps = max(3, min(40, int((6e6 if P > 4 else 1.5e7) / (n1 * n2 * n3))))
        return lattice("ball", rng.choice([KURAMOTO, INERTIA, INERTIA]), n1, n2, n3, P, steps, fp32,
                       rng.choice([0, 3]), 0.45)
    if kind == "disk":
        P = rng.choice([2, 3, 6])
        n1, n2 = log_int(40, 1200), log_int(40, 1200)
        return lattice("disk", KURAMOTO, n1, n2, 1, P, max(3, min(40, int(1e7 / (n1 * n2)))), fp32, 0, 0.8)
    if kind == "hh":
        n, degree = log_int(500, 200000), rng.randint(10, 100)
        return hh(n, degree, max(5, min(50, int(2e8 / (n * degree)))), fp32)
    if kind == "links":
        P = rng.choice([1, 2, 2, 3])
        n1, n2, n3 = (log_int(2 * P + 4, 60) for _ in range(3))
        return links(n1, n2, n3, P, max(3, min(60, int(6e6 / (n1 * n2 * n3)))), fp32)
    if kind == "small_world":
        n = log_int(300, 20000)
        return small_world(n, rng.randint(2, 24), n // 20, 50, fp32)
    if kind == "adaptive_small":
        n = log_int(65, 1024)
        return adaptive(rng.choice([KURAMOTO, INERTIA, FHN]), n, max(1, int(n * rng.uniform(0.05, 0.4))),
                        log_int(1, 512), round(rng.uniform(2.0, 10.0), 2), rng.choice([1e-6, 1e-8]), alpha)
    if kind == "adaptive_large":
        n = log_int(1025, 65536)
        return adaptive(rng.choice([KURAMOTO, FHN]), n, max(1, int(n * rng.uniform(0.05, 0.4))),
                        log_int(1, max(1, min(8, 131072 // n))), round(rng.uniform(0.2, 1.0), 3), 1e-8, alpha)
    if kind == "adaptive_links":
        n1, n2, n3 = (log_int(9, 60) for _ in range(3))
        return links(n1, n2, n3, 2, 0, t_end=round(rng.uniform(5.0, 50.0), 1), rtol=rng.choice([1e-6, 1e-8]),
                     t_out=rng.choice([0.0, 1.0]))
    return serve(rng.randint(4, 24), rng.randint(12, 16), 200, 800, rng.randrange(2, 1 << 30))


# ------------------------------------------------------------------------------------------ inputs
def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + tag) % (1 << 62))
    return g


def _uniform(seed, tag, *shape):
    return torch.rand(*shape, generator=_gen(seed, tag), device=DEV, dtype=torch.float64)


def _phases(seed, tag, *shape):
    return math.pi * (2.0 * _uniform(seed, tag, *shape) - 1.0)


def _ring_state(model, seed, n, batch):
    if model == FHN:  # the circle of radius 2 at random angles
        th = 2.0 * math.pi * _uniform(seed, 1, batch, n)
        return torch.cat([2.0 * torch.cos(th), 2.0 * torch.sin(th)], 1).contiguous()
    phi = _phases(seed, 2, batch, n)
    return phi if model == KURAMOTO else torch.cat([phi, torch.zeros_like(phi)], 1).contiguous()


def _lattice_state(model, seed, n1, n2, n3):
    """Uniform phases with a planted coherent ball (a fifth of the smallest extent), psi = 0."""
    phi = _phases(seed, 3, n3, n2, n1)
    u = _uniform(seed, 4, 4).tolist()
    d2 = 0.0
    for extent, frac, shape in ((n3, u[0], (-1, 1, 1)), (n2, u[1], (1, -1, 1)), (n1, u[2], (1, 1, -1))):
        d = (torch.arange(extent, device=DEV) - int(frac * extent)).abs()
        d2 = d2 + (torch.minimum(d, extent - d).double() ** 2).view(shape)
    r = min(e for e in (n1, n2, n3) if e > 1) / 5.0
    phi[d2.expand_as(phi) <= r * r] = math.pi * (2.0 * u[3] - 1.0)
    phi = phi.reshape(-1)
    return phi if model == KURAMOTO else torch.cat([phi, torch.zeros_like(phi)])


def _hh_inputs(seed, n, degree):
    """Random directed graph (CSR by target, sources ascending), weights, currents and the state."""
    src = torch.arange(n, device=DEV).repeat_interleave(degree)
    step = torch.randint(0, n - 1, (n * degree,), generator=_gen(seed, 5), device=DEV)
    key = torch.sort(((src + 1 + step) % n) * n + src).values
    row, col = key // n, (key % n).to(torch.int32)
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    w = 0.1 * _uniform(seed, 6, n * degree)
    iapp = 8.0 + 4.0 * _uniform(seed, 7, n)
    u = _uniform(seed, 8, 4, n)
    lo = torch.tensor([-70.0, 0.03, 0.55, 0.29], device=DEV, dtype=torch.float64)
    wd = torch.tensor([10.0, 0.04, 0.10, 0.06], device=DEV, dtype=torch.float64)
    return row_ptr, row, col, w, iapp, (lo[:, None] + wd[:, None] * u).reshape(-1).contiguous()


def _rows_of(case):
    """Sorted (row, source) keys of a coupling matrix given by rows; the matrix itself does not depend on the seed."""
    if case["family"] == "small_world":
        n, P = case["n"], case["P"]
        i = torch.arange(n, device=DEV)
        off = torch.cat([torch.arange(-P, 0, device=DEV), torch.arange(1, P + 1, device=DEV)])
        ring_keys = (i[:, None] * n + (i[:, None] + off[None, :]) % n).reshape(-1)
        a = torch.randint(0, n, (2, case["shortcuts"]), generator=_gen(n, 9), device=DEV)
        a = a[:, a[0] != a[1]]
        return n, torch.unique(torch.cat([ring_keys, a[0] * n + a[1]]))
    n1, n2, n3, P = case["n1"], case["n2"], case["n3"], case["radius"]
    n = n1 * n2 * n3
    i = torch.arange(n, device=DEV)
    x, y, z = i % n1, (i // n1) % n2, i // (n1 * n2)
    keys = [i * n + (x + dx) % n1 + n1 * ((y + dy) % n2) + n1 * n2 * ((z + dz) % n3) for dx, dy, dz in _ball(P, P)]
    return n, torch.sort(torch.cat(keys)).values


def _ball(P, pz):
    r = range(-P, P + 1)
    return [(dx, dy, dz) for dz in range(-pz, pz + 1) for dy in r for dx in r if dx * dx + dy * dy + dz * dz <= P * P]


def _serve_requests(case):
    """(model, n, P, alpha, steps, fp32) of each request: the mix is part of the case."""
    r = random.Random(case["mix"])
    got = []
    for i in range(case["count"]):
        n = int(2.0 ** r.uniform(10, case["log2_max"]))
        steps = int(math.exp(r.uniform(math.log(case["steps_min"]), math.log(case["steps_max"]))))
        got.append((FHN if i % 2 else KURAMOTO, n, max(1, int(n * r.uniform(0.05, 0.4))), r.uniform(1.3, 1.55), steps,
                    i % 4 == 2))
    return got


def _params(model, alpha):
    return [0.0, 1.0, alpha] if model == KURAMOTO else INERTIA_PRM if model == INERTIA else FHN_PRM


def _dt(case):
    if case["family"] == "hh":
        return 0.01
    return 0.05 if case["family"] in ("cube", "ball", "disk", "links") else 0.01


def _prec(case):
    return nd.ND_FP32_BULK if case.get("fp32") else nd.ND_FP64


class State:
    """What the caller's program holds: handles (destroyed with it), inputs and output buffers."""

    def __init__(self, case):
        self.case, self.handles, self.server = case, [], None

    def __del__(self):
        for h in self.handles:
            nd.nd_destroy(h)
        if self.server is not None:
            nd.nd_server_destroy(self.server)


def prepare(case, seed):
    s, f = State(case), case["family"]
    if f == "serve":
        s.server = nd.nd_server_create(8 << 30, max_slots=64, chunk_steps=64)
        s.requests = []
        for q, (model, n, P, alpha, steps, fp32) in enumerate(_serve_requests(case)):
            p = nd.problem(MODELS[model], nd.ND_RING, n, _params(model, alpha), radius=P,
                           precision=nd.ND_FP32_BULK if fp32 else nd.ND_FP64)
            s.requests.append((p, _ring_state(model, 64 * seed + q, n, 1)[0].cpu().numpy(), steps))
        return s
    if f in ("ring", "adaptive"):
        model, n = case["model"], case["n"]
        p = nd.problem(MODELS[model], nd.ND_RING, n, _params(model, case["alpha"]), precision=_prec(case),
                       radius=case["P"])
        s.y0 = _ring_state(model, seed, n, case["batch"])
        s.handles = [nd.nd_create(p) for _ in range(case["batch"])]
    elif f in ("cube", "ball", "disk"):
        model, dims = case["model"], (case["n1"], case["n2"], case["n3"])
        topo = {"cube": nd.ND_CUBE3D, "ball": nd.ND_BALL3D, "disk": nd.ND_DISK2D}[f]
        p = nd.problem(MODELS[model], topo, dims[0] * dims[1] * dims[2], _params(model, case["alpha"]),
                       precision=_prec(case), radius=case["radius"], dims=dims)
        s.y0 = _lattice_state(model, seed, *dims)[None, :]
        s.handles = [nd.nd_create(p)]
    elif f == "hh":
        row_ptr, _, col, w, iapp, y0 = _hh_inputs(seed, case["n"], case["degree"])
        p = nd.problem(nd.ND_HH, nd.ND_CSR, case["n"], HH_PRM, precision=_prec(case), row_ptr=row_ptr.cpu().numpy(),
                       col=col.cpu().numpy(), weight=w.cpu().numpy(), per_elem=iapp.cpu().numpy())
        s.y0 = y0[None, :]
        s.handles = [nd.nd_create(p)]
    else:  # a coupling matrix given by rows
        n, keys = _rows_of(case)
        row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
        row_ptr[1:] = torch.cumsum(torch.bincount(keys // n, minlength=n), 0)
        model = FHN if f == "small_world" else INERTIA
        p = nd.problem(MODELS[model], nd.ND_LINKS, n, _params(model, 0.0), precision=_prec(case),
                       row_ptr=row_ptr.cpu().numpy(), col=(keys % n).to(torch.int32).cpu().numpy())
        s.y0 = (_ring_state(FHN, seed, n, 1) if model == FHN
                else _lattice_state(model, seed, case["n1"], case["n2"], case["n3"])[None, :])
        s.handles = [nd.nd_create(p)]
    s.y = torch.empty_like(s.y0)
    record = case.get("record", 0)
    s.obs = nd.observe(record, case["steps"] // 2 if case.get("mv") else -1) if record or case.get("mv") else None
    batch = len(s.handles)
    s.R = torch.empty(batch, case["steps"] // record + 1, dtype=torch.float64, device=DEV) if record else None
    s.mv = torch.empty(batch, case["n"], dtype=torch.float64, device=DEV) if case.get("mv") else None
    return s


def run(s):
    case = s.case
    if s.server is not None:
        ids = [nd.nd_server_submit(s.server, p, y0, 0.01, steps, nd.observe(10)) for p, y0, steps in s.requests]
        while nd.nd_server_pump(s.server):
            pass
        out = []
        for rid, (_, y0, steps) in zip(ids, s.requests):
            y, R = np.empty_like(y0), np.empty(steps // 10 + 1)
            nd.nd_server_result(s.server, rid, y, R)
            out.append((y, R))
        return out
    for h, y0 in zip(s.handles, s.y0):
        nd.nd_set_state(h, y0)
    batch = len(s.handles)
    if case.get("t_end"):
        te, d0 = [case["t_end"]] * batch, [1e-3] * batch
        atol = 1e-2 * case["rtol"]
        R = None
        if case.get("t_out"):
            stats, R, _ = nd.nd_run_adaptive_dense(s.handles, te, d0, case["rtol"], atol, case["t_out"])
        else:
            stats = nd.nd_run_adaptive(s.handles, te, d0, case["rtol"], atol)
        for h, y in zip(s.handles, s.y):
            nd.nd_get_state(h, y)
        return {"y": s.y, "R": R, "accepted": np.array([t.accepted for t in stats]),
                "rejected": np.array([t.rejected for t in stats])}
    dt, steps = _dt(case), case["steps"]
    if batch == 1:
        nd.nd_run(s.handles[0], dt, steps, s.obs)
    else:
        nd.nd_run_batch(s.handles, [dt] * batch, [steps] * batch, None if s.obs is None else [s.obs] * batch)
    for i, h in enumerate(s.handles):
        nd.nd_get_state(h, s.y[i])
        if s.obs is not None:
            nd.nd_get_observables(h, None if s.R is None else s.R[i], None if s.mv is None else s.mv[i])
    return {"y": s.y, "R": s.R, "mv": s.mv}


# -------------------------------------------------------------------------------------------- work
def _flops(model):
    """Per element and stage: map, O(1) neighbourhood sum, right-hand side, stage value and update."""
    return {KURAMOTO: 64, INERTIA: 72, FHN: 36}[model]


def work(case):
    f = case["family"]
    if f == "serve":
        q = _serve_requests(case)
        return {"bytes": sum(16 * NVARS[m] * n for m, n, *_ in q),
                "flops": sum(4 * steps * n * _flops(m) for m, n, _, _, steps, _ in q)}
    if f == "hh":
        n, nnz = case["n"], case["n"] * case["degree"]
        eb = 8 if case["fp32"] else 12
        return {"bytes": 2 * 32 * n + 8 * n + nnz * eb, "flops": 4 * case["steps"] * (2 * nnz + 260 * n)}
    if f in ("ring", "adaptive"):
        n, model = case["n"] * case["batch"], case["model"]
        terms = 0
    elif f == "small_world":
        n, model, terms = case["n"], FHN, 4 * case["P"]
    else:
        n, model = case["n1"] * case["n2"] * case["n3"], case.get("model", INERTIA)
        terms = 2 * len(_ball(case["radius"], case["radius"])) if f == "links" else 0
    stages = 4 * case.get("steps", 0)
    if case.get("t_end"):  # six stages a step, at least one step per unit of time
        stages = 6 * max(1, int(case["t_end"]))
    return {"bytes": 16 * NVARS[model] * n, "flops": max(stages, 1) * n * (_flops(model) + terms)}


# ------------------------------------------------------------------------- the same in 64 bits
def _ring_window(x, P):
    n = x.shape[-1]
    c = torch.cumsum(torch.cat([torch.zeros_like(x[..., :1]), x[..., n - P:], x, x[..., :P]], -1), -1)
    return c[..., 2 * P + 1:] - c[..., :n]


def _coupling(case):
    """Function of the two map components giving the neighbourhood sums, and the link count."""
    f = case["family"]
    if f in ("ring", "adaptive"):
        P = case["P"]
        return (lambda a: _ring_window(a, P) - a), 2.0 * P
    if f == "cube":
        h, dims = case["radius"], (case["n3"], case["n2"], case["n1"])

        def box(a):
            b = a.view(dims)
            for d in range(3):
                b = sum(torch.roll(b, q, d) for q in range(-h, h + 1))
            return b.reshape(a.shape) - a

        return box, (2.0 * h + 1.0) ** 3 - 1.0
    if f in ("ball", "disk"):
        P, dims = case["radius"], (case["n3"], case["n2"], case["n1"])
        pz = P if f == "ball" else 0
        offs = _ball(P, pz)
        pairs = sorted({(dy, dz) for _, dy, dz in offs})

        def ball(a):
            b = a.view(dims)
            runs = [b]
            for r in range(1, P + 1):
                runs.append(runs[-1] + torch.roll(b, r, 2) + torch.roll(b, -r, 2))
            t = torch.zeros_like(b)
            for dy, dz in pairs:
                t += torch.roll(runs[math.isqrt(P * P - dy * dy - dz * dz)], (-dz, -dy), (0, 1))
            return t.reshape(a.shape)

        return ball, float(len(offs))
    n, keys = _rows_of(case)
    row, col = keys // n, keys % n
    count = torch.bincount(row, minlength=n).double()

    def gather(a):
        return torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, row, a.reshape(-1)[col]).view(a.shape)

    return gather, count


def _rhs(case, model):
    """dy/dt for y of shape [batch, nvars, n]."""
    prm = _params(model, case.get("alpha", 0.0))
    coupling, count = _coupling(case)
    if model == FHN:
        eps, a, sigma, phi = prm

        def fhn(y):
            u, v = y[:, 0], y[:, 1]
            du, dv = coupling(u) - count * u, coupling(v) - count * v
            c, s, k = math.cos(phi), math.sin(phi), sigma / count
            return torch.stack([(u - u ** 3 / 3.0 - v + k * (c * du + s * dv)) / eps, u + a + k * (c * dv - s * du)], 1)

        return fhn
    omega, mu, alpha = prm[:3]

    def phase(y):
        C, S = coupling(torch.cos(y[:, 0])), coupling(torch.sin(y[:, 0]))
        z = y[:, 0] + alpha
        force = omega + (mu / count) * (torch.cos(z) * S - torch.sin(z) * C)
        return force[:, None] if model == KURAMOTO else torch.stack([y[:, 1], (force - prm[4] * y[:, 1]) / prm[3]], 1)

    return phase


def _hh_rhs(case, seed):
    n = case["n"]
    row_ptr, row, col, w, iapp, y0 = _hh_inputs(seed, n, case["degree"])
    col = col.long()
    C, gNa, gK, gL, ENa, EK, EL, Esyn, th, ks = HH_PRM

    def ratio(x):
        return torch.where(x.abs() < 1e-7, 1.0 + 0.5 * x, x / -torch.expm1(-x))

    def rhs(y):
        V, m, h, g = y[0]
        S = torch.sigmoid((V - th) / ks)
        G = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, row, w * S[col])
        ion = gNa * m ** 3 * h * (V - ENa) + gK * g ** 4 * (V - EK) + gL * (V - EL)
        return torch.stack([
            (iapp - ion + (Esyn - V) * G) / C,
            ratio((V + 40.0) / 10.0) * (1.0 - m) - 4.0 * torch.exp(-(V + 65.0) / 18.0) * m,
            0.07 * torch.exp(-(V + 65.0) / 20.0) * (1.0 - h) - torch.sigmoid((V + 35.0) / 10.0) * h,
            0.1 * ratio((V + 55.0) / 10.0) * (1.0 - g) - 0.125 * torch.exp(-(V + 65.0) / 80.0) * g])[None]

    return rhs, y0.view(1, 4, n)


def _order(model, y):
    u = y if model == FHN else torch.stack([torch.cos(y[:, 0]), torch.sin(y[:, 0])], 1)
    u = u / torch.linalg.vector_norm(u, dim=1, keepdim=True)
    return torch.linalg.vector_norm(u.mean(2), dim=1)


def _rk4(rhs, y, dt, steps, model=None, record=0, mv_start=-1):
    R = [_order(model, y)] if record else None
    theta = torch.zeros_like(y[:, 0])
    for i in range(steps):
        k1 = rhs(y)
        k2 = rhs(y + 0.5 * dt * k1)
        k3 = rhs(y + 0.5 * dt * k2)
        k4 = rhs(y + dt * k3)
        new = y + dt / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + k4)
        if 0 <= mv_start <= i:
            if model == FHN:
                theta += torch.atan2(y[:, 0] * new[:, 1] - y[:, 1] * new[:, 0],
                                     y[:, 0] * new[:, 0] + y[:, 1] * new[:, 1])
            else:
                theta += new[:, 0] - y[:, 0]
        y = new
        if record and (i + 1) % record == 0:
            R.append(_order(model, y))
    mv = theta / ((steps - mv_start) * dt) if mv_start >= 0 else None
    return y, None if R is None else torch.stack(R, 1), mv


DP_A = [[], [1 / 5], [3 / 40, 9 / 40], [44 / 45, -56 / 15, 32 / 9],
        [19372 / 6561, -25360 / 2187, 64448 / 6561, -212 / 729],
        [9017 / 3168, -355 / 33, 46732 / 5247, 49 / 176, -5103 / 18656],
        [35 / 384, 0.0, 500 / 1113, 125 / 192, -2187 / 6784, 11 / 84]]
DP_E = [71 / 57600, 0.0, -71 / 16695, 71 / 1920, -17253 / 339200, 22 / 525, -1 / 40]


def _dormand_prince(rhs, y, t_end, h0, rtol, atol):
    """Every network of the batch with its own step, all of them in lockstep attempts."""
    b = y.shape[0]
    t = torch.zeros(b, device=DEV, dtype=torch.float64)
    h, facmax = torch.full_like(t, h0), torch.full_like(t, 10.0)
    k1 = rhs(y)
    for _ in range(100000):
        done = t >= t_end
        if bool(done.all()):
            return y
        last = t_end - t <= h * (1.0 + 1e-12)
        hs = torch.where(last, t_end - t, h)[:, None, None]
        k = [k1]
        for s in range(1, 7):
            z = y + hs * sum(a * q for a, q in zip(DP_A[s], k))
            k.append(rhs(z))
        scale = atol + rtol * torch.maximum(y.abs(), z.abs())
        err = ((hs * sum(e * q for e, q in zip(DP_E, k)) / scale) ** 2).mean((1, 2)).sqrt()
        fac = 0.9 * err ** -0.2
        ok = (err <= 1.0) & ~done
        move = ok[:, None, None]
        y, k1 = torch.where(move, z, y), torch.where(move, k[6], k1)
        t = torch.where(ok, torch.where(last, torch.full_like(t, t_end), t + hs[:, 0, 0]), t)
        grown = hs[:, 0, 0] * torch.where(ok, torch.minimum(facmax, fac.clamp(min=0.2)), fac.clamp(0.2, 1.0))
        h = torch.where(done, h, grown)
        facmax = torch.where(ok, torch.full_like(t, 10.0), torch.ones_like(t))
    return y


def exact(case, seed):
    f = case["family"]
    if f == "serve":
        out = []
        for q, (model, n, P, alpha, steps, _) in enumerate(_serve_requests(case)):
            y0 = _ring_state(model, 64 * seed + q, n, 1).view(1, NVARS[model], n)
            y, R, _ = _rk4(_rhs({"family": "ring", "P": P, "alpha": alpha}, model), y0, 0.01, steps, model, 10)
            out.append((y.reshape(-1).cpu().numpy(), R[0].cpu().numpy()))
        return out
    if f == "hh":
        rhs, y0 = _hh_rhs(case, seed)
        return {"y": _rk4(rhs, y0, _dt(case), case["steps"])[0].reshape(1, -1), "R": None, "mv": None}
    if f in ("ring", "adaptive"):
        model, n, batch = case["model"], case["n"], case["batch"]
        y0 = _ring_state(model, seed, n, batch).view(batch, NVARS[model], n)
    elif f == "small_world":
        model, n = FHN, case["n"]
        y0 = _ring_state(model, seed, n, 1).view(1, 2, n)
    else:
        model = case.get("model", INERTIA)
        y0 = _lattice_state(model, seed, case["n1"], case["n2"], case["n3"]).view(1, NVARS[model], -1)
    rhs = _rhs(case, model)
    if case.get("t_end"):
        y = _dormand_prince(rhs, y0, case["t_end"], 1e-3, case["rtol"], 1e-2 * case["rtol"])
        return {"y": y.reshape(y.shape[0], -1), "R": None, "accepted": None, "rejected": None}
    y, R, mv = _rk4(rhs, y0, _dt(case), case["steps"], model, case.get("record", 0),
                    case["steps"] // 2 if case.get("mv") else -1)
    return {"y": y.reshape(y.shape[0], -1), "R": R, "mv": mv}
