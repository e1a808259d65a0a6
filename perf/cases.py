"""Performance cases of the near-field library: what an N-body program has it do, through its Python calls.

A program keeps a handle of cells and its particle arrays on the GPU and, step after step, rebuilds the cells,
evaluates the near-field forces, computes the far field's moments, adds its Taylor series, kicks and drifts, picks
the next step and merges its arrays into cell order.  The cases are those calls over their range of sizes: single
small boxes where launches count, batches of small boxes, early (uniform) and late (clustered) boxes, dense and
sparse cells, both softening laws, plain and compensated sums.

Inputs are made on the GPU from the seed alone: uniform particles, or a uniform background plus Plummer halos with
power-law masses, in random order (or in cell order where a program has merged its arrays).  Units: box side 1,
total mass 1, softening 1/40 of the mean spacing.
"""
import itertools
import math

import numpy as np
import torch

import paper_2110_11398_amd as nf

R = 2
KINDS = {"spline": nf.SPLINE, "plummer": nf.PLUMMER}
MODES = {"fp32": nf.SUM_FP32, "comp32": nf.SUM_COMP32}
DENSITY_RADIUS = 0.4      # density kernel radius in mean spacings
ETA = 0.25                # step-size criterion


def listed():
    return [
        # one call on a small box, nothing kept between calls: a test problem, an analysis script
        {"name": "one_shot_tiny", "op": "one_shot", "n": 32768, "K": 8, "halo": 0.0, "kind": "spline", "mode": "comp32"},
        # the force evaluation of a small clustered simulation: the handle is kept, launches count
        {"name": "step_small", "op": "step", "n": 13824, "K": 8, "halo": 0.5, "kind": "spline", "mode": "comp32"},
        # early times, nearly uniform, plain sums
        {"name": "step_uniform", "op": "step", "n": 2097152, "K": 32, "halo": 0.0, "kind": "spline", "mode": "fp32"},
        # an odd size with Plummer softening
        {"name": "step_plummer_odd", "op": "step", "n": 1000003, "K": 25, "halo": 0.5, "kind": "plummer",
         "mode": "comp32"},
        # half of the particles in halos: the clustered workload of the benchmark
        {"name": "step_clustered", "op": "step", "n": 16777216, "K": 64, "halo": 0.5, "kind": "spline",
         "mode": "comp32"},
        # late times: sparse cells (8 particles on average) around very heavy halo cores
        {"name": "step_late", "op": "step", "n": 33554432, "K": 161, "halo": 0.5, "kind": "spline", "mode": "comp32"},
        # many independent small boxes in one batch (an ensemble of simulations)
        {"name": "batch_boxes", "op": "batch", "boxes": 48, "lo": 4096, "hi": 110592, "halo": 0.3, "kind": "spline",
         "mode": "comp32"},
        # forces with the density estimate a halo finder starts from
        {"name": "density_medium", "op": "density", "n": 250007, "K": 16, "halo": 0.5, "kind": "spline",
         "mode": "comp32"},
        # cells and their multipole moments after a drift: the input of the far-field convolution
        {"name": "moments_clustered", "op": "moments", "n": 16777216, "K": 64, "halo": 0.5, "order": 8},
        # the far field of sparse late-time cells added to the near field, arrays in cell order
        {"name": "taylor_sparse", "op": "taylor", "n": 8388608, "K": 101, "halo": 0.5, "order": 8, "sorted": True},
        # the simulation loop: one leapfrog step and the size of the next
        {"name": "leapfrog", "op": "leapfrog", "n": 262144, "K": 16, "halo": 0.5, "kind": "spline", "mode": "comp32"},
        # kick, drift, move the particles to their cells and merge the arrays into cell order
        {"name": "merge", "op": "merge", "n": 6000001, "K": 46, "halo": 0.5},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) | rng.randint(0, 1)

    op = rng.choice(["one_shot", "step", "step", "step", "batch", "density", "moments", "taylor", "leapfrog", "merge"])
    halo = rng.choice([0.0, 0.3, 0.5])
    kind, mode = rng.choice(sorted(KINDS)), rng.choice(sorted(MODES))
    if op == "batch":
        lo = size(1000, 20000)
        return {"op": op, "boxes": rng.randint(2, 64), "lo": lo, "hi": lo * rng.randint(2, 8), "halo": halo,
                "kind": kind, "mode": mode}
    top = {"one_shot": 1 << 18, "step": 1 << 23, "density": 1 << 20, "leapfrog": 1 << 21, "merge": 1 << 24,
           "moments": 1 << 24, "taylor": 1 << 24}[op]
    n = size(1 << 12, top)
    per_cell = math.exp(rng.uniform(math.log(6.0), math.log(90.0)))
    case = {"op": op, "n": n, "K": max(5, int(round((n / per_cell) ** (1.0 / 3.0)))), "halo": halo}
    if op in ("moments", "taylor"):
        case["order"] = rng.choice([2, 4, 6, 8, 8, 8])
    elif op != "merge":
        case["kind"], case["mode"] = kind, mode
    if op == "taylor":
        case["sorted"] = rng.random() < 0.5
    return case


# ---------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _halo_counts(total, n_halos, seed):
    """Halo sizes from dN/dM ~ M^-1.9 on [1, 1000], scaled to add up to total."""
    u = np.random.default_rng(seed).random(n_halos)
    m = (1.0 + u * (1000.0 ** -0.9 - 1.0)) ** (-1.0 / 0.9)
    share = np.floor(m / m.sum() * total).astype(np.int64)
    share[: total - int(share.sum())] += 1
    return share


def _positions(n, K, halo, seed):
    """float32 [n, 3] in [0, 1): uniform, a fraction `halo` of the particles in Plummer halos, in random order.
    Sparse boxes (under 16 per cell) are late-time ones: scale radii of 0.05 to 0.5 cell and one halo for 8192
    particles; in the others 0.3 cell and one for 4096."""
    g = _gen(seed)
    late = n < 16 * K ** 3
    n_halos = max(1, n // (8192 if late else 4096))
    n_h = int(n * halo)
    pos = torch.rand((n, 3), generator=g, device="cuda", dtype=torch.float32)
    if n_h:
        counts = torch.from_numpy(_halo_counts(n_h, n_halos, seed)).cuda()
        a = torch.full((n_halos,), 0.3, device="cuda")
        if late:
            a = 0.05 * 10.0 ** torch.rand(n_halos, generator=g, device="cuda")
        hid = torch.repeat_interleave(torch.arange(n_halos, device="cuda"), counts)
        centre = torch.rand((n_halos, 3), generator=g, device="cuda", dtype=torch.float64)
        # radii by the Plummer inverse CDF, cut at ten scale radii
        x = torch.rand(n_h, generator=g, device="cuda", dtype=torch.float64).clamp_min(1e-12) * (1000.0 / 101.0 ** 1.5)
        r = (a.double()[hid] / K) / torch.sqrt(x ** (-2.0 / 3.0) - 1.0)
        d = torch.randn((n_h, 3), generator=g, device="cuda", dtype=torch.float64)
        p = (centre[hid] + d * (r / d.norm(dim=1))[:, None]) % 1.0
        pos[:n_h] = p.float()
        pos[pos >= 1.0] = 0.0
        pos = pos[torch.randperm(n, generator=g, device="cuda")].contiguous()
    return pos


def _spacing(n):
    return n ** (-1.0 / 3.0)


def _box_list(case):
    """[(n, K)] of the case's boxes."""
    if case["op"] != "batch":
        return [(case["n"], case["K"])]
    k = case["boxes"]
    sizes = [int(round(case["lo"] * (case["hi"] / case["lo"]) ** (i / max(1, k - 1)))) for i in range(k)]
    return [(n, max(5, int(round((n / 48.0) ** (1.0 / 3.0))))) for n in sizes]


def _box_positions(case, seed):
    return [_positions(n, K, case["halo"], 1000 * seed + i) for i, (n, K) in enumerate(_box_list(case))]


def _cell_of(pos, K):
    t = pos.double() * float(K)
    c = t.floor().clamp_max(K - 1)
    i = c.long()
    return (i[:, 0] * K + i[:, 1]) * K + i[:, 2], t - (c + 0.5)


def _components(order):
    return [(a, b, n - a - b) for n in range(order + 1) for a in range(n, -1, -1) for b in range(n - a, -1, -1)]


def _taylor_inputs(case, seed, n):
    g = _gen(seed + 77)
    comp = _components(case["order"])
    scale = torch.tensor([1e-3 * 3.0 ** -sum(c) for c in comp], dtype=torch.float64, device="cuda")
    taylor = torch.randn((case["K"] ** 3, len(comp)), generator=g, device="cuda", dtype=torch.float64) * scale
    acc = torch.randn((n, 3), generator=g, device="cuda", dtype=torch.float32) * 0.1
    return taylor, acc


def _velocities(seed, n):
    return torch.randn((n, 3), generator=_gen(seed + 55), device="cuda", dtype=torch.float32) * 1e-3


def prepare(case, seed):
    op = case["op"]
    sizes = _box_list(case)
    parts = _box_positions(case, seed)
    pos = torch.cat(parts) if len(parts) > 1 else parts[0]
    n = pos.shape[0]
    s = {"op": op, "pos": pos, "boxes": [(m, 1.0, K) for m, K in sizes], "eps": [_spacing(m) / 40.0 for m, _ in sizes],
         "gm": [1.0 / m for m, _ in sizes], "order": case.get("order"), "K": case.get("K")}
    if "kind" in case:
        s["kind"], s["mode"] = KINDS[case["kind"]], MODES[case["mode"]]
    if op != "one_shot":
        s["cells"] = nf.Cells()
    if op in ("step", "batch", "density", "leapfrog"):
        s["acc"] = torch.empty((n, 3), dtype=torch.float32, device="cuda")
    if op == "density":
        s["b"] = [DENSITY_RADIUS * _spacing(n)]
        s["rho"] = torch.empty(n, dtype=torch.float32, device="cuda")
    if op == "moments":
        s["out"] = torch.empty((case["K"] ** 3, len(_components(case["order"]))), dtype=torch.float64, device="cuda")
    if op == "taylor":
        if case["sorted"]:
            pos = pos[torch.sort(_cell_of(pos, case["K"])[0], stable=True)[1]].contiguous()
        s["taylor"], s["acc"] = _taylor_inputs(case, seed, n)
        nf.build_cells(pos, s["boxes"], R, cells=s["cells"])
    if op == "leapfrog":
        s["vel"] = _velocities(seed, n)
        s["dt"] = [1e-4]
        nf.build_cells(pos, s["boxes"], R, cells=s["cells"])
        s["cells"].forces(s["eps"], s["gm"], s["kind"], s["mode"], out=s["acc"])
    if op == "merge":
        s["vel"] = _velocities(seed, n)
        s["acc"] = _velocities(seed + 1, n) * 1e-3
        s["ids"] = torch.arange(n, dtype=torch.int64, device="cuda")
        s["dt"] = [0.5]      # a drift of a few hundredths of a cell
        nf.build_cells(pos, s["boxes"], R, cells=s["cells"])
    return s


def run(s):
    op = s["op"]
    if op == "one_shot":
        (_, L, K), = s["boxes"]
        return nf.near_field(s["pos"], L, K, s["eps"][0], s["gm"][0], s["kind"], s["mode"])
    cells = s["cells"]
    if op in ("step", "batch"):
        nf.build_cells(s["pos"], s["boxes"], R, cells=cells)
        return cells.forces(s["eps"], s["gm"], s["kind"], s["mode"], out=s["acc"])
    if op == "density":
        nf.build_cells(s["pos"], s["boxes"], R, cells=cells)
        return cells.forces_density(s["eps"], s["gm"], s["b"], s["kind"], s["mode"], out=s["acc"], rho=s["rho"])
    if op == "moments":
        nf.build_cells(s["pos"], s["boxes"], R, cells=cells)
        return cells.multipoles(s["order"], s["gm"], out=s["out"])
    if op == "taylor":
        return cells.taylor_forces(s["order"], s["taylor"], s["acc"])
    if op == "leapfrog":
        cells.kdk_step(s["dt"], s["eps"], s["gm"], s["pos"], s["vel"], s["acc"], s["kind"], s["mode"])
        s["dt"] = cells.timestep(s["vel"], None, ETA)
        return {"pos": s["pos"], "vel": s["vel"], "acc": s["acc"], "dt": s["dt"]}
    if op == "merge":
        cells.kick(s["dt"], s["acc"], s["vel"])
        cells.drift(s["dt"], s["vel"], s["pos"])
        nf.build_cells(s["pos"], s["boxes"], R, cells=cells)
        cells.reorder([s["pos"], s["vel"], s["acc"]], s["ids"])
        return {"pos": s["pos"], "vel": s["vel"], "acc": s["acc"], "ids": s["ids"]}
    raise ValueError(op)


# ---------------------------------------------------------------- work of a pass

def _pairs(pos, K):
    """Ordered pairs of the near field, self pairs included."""
    occ = torch.bincount(_cell_of(pos, K)[0], minlength=K ** 3).double().view(K, K, K)
    near = occ
    for axis in range(3):
        near = sum(torch.roll(near, d, axis) for d in range(-R, R + 1))
    return float((occ * near).sum())


def work(case):
    op, sizes = case["op"], _box_list(case)
    n, cells = sum(m for m, _ in sizes), sum(K ** 3 for _, K in sizes)
    comp = len(_components(case.get("order", 0)))
    if op == "moments":      # positions in, moments out; powers and one multiply-add a component
        return {"bytes": 12.0 * n + 8.0 * comp * cells, "flops": n * (3.0 * case["order"] + 3.0 * comp)}
    if op == "taylor":       # sorted coordinates and order in, accelerations in and out, the series in
        return {"bytes": (16.0 + 4.0 + 24.0) * n + 8.0 * comp * cells, "flops": n * 5.6 * comp}
    if op == "merge":        # three vectors in and out, identities in and out
        return {"bytes": (3 * 24.0 + 16.0) * n, "flops": 24.0 * n}
    pairs = sum(_pairs(p, K) for p, (_, K) in zip(_box_positions(case, 1), sizes))
    per = (26.0 if case["kind"] == "spline" else 20.0) + (4.0 if op == "density" else 0.0)
    moved = {"density": 28.0, "leapfrog": 72.0}.get(op, 24.0)
    return {"bytes": moved * n, "flops": per * pairs}


# ---------------------------------------------------------------- the same results in 64 bits

def _near_field_exact(pos, K, eps, gm, kind, b=None):
    """Accelerations (and densities) of one box by direct sums in float64, one cell of sinks at a time; None where
    that is too long."""
    if len(pos) > 2500000 or _pairs(pos.float(), K) > 6e10:
        return None
    cell, _ = _cell_of(pos.float(), K)
    key, order = torch.sort(cell, stable=True)
    p = pos.double()[order]
    start = torch.searchsorted(key, torch.arange(K ** 3 + 1, device="cuda")).cpu().numpy()
    acc, rho = torch.zeros_like(p), torch.zeros_like(p[:, 0])
    off = np.array(list(itertools.product(range(-R, R + 1), repeat=3)))
    for c in np.nonzero(np.diff(start))[0]:
        at = np.array([c // (K * K), c // K % K, c % K]) + off
        image = np.floor_divide(at, K)
        at = at - image * K
        nb = (at[:, 0] * K + at[:, 1]) * K + at[:, 2]
        lens = start[nb + 1] - start[nb]
        idx = np.repeat(start[nb] - (np.cumsum(lens) - lens), lens) + np.arange(lens.sum())
        src = p[torch.from_numpy(idx).cuda()]
        if image.any():
            src = src + torch.from_numpy(np.repeat(image, lens, axis=0).astype(np.float64)).cuda()
        lo, hi = int(start[c]), int(start[c + 1])
        step = max(1, (1 << 24) // len(idx))
        for s0 in range(lo, hi, step):
            s1 = min(hi, s0 + step)
            d = src[None, :, :] - p[s0:s1, None, :]
            r2 = (d * d).sum(2)
            if kind == "plummer":
                g = (r2 + eps * eps) ** -1.5
            else:
                r = r2.sqrt()
                u = r / eps
                g = torch.where(u < 1.0, (10.0 - 15.0 * u + 6.0 * u * u) / eps ** 3, 1.0 / (r2 * r))
            acc[s0:s1] = torch.matmul(g[:, None, :], d)[:, 0, :]
            if b is not None:
                rho[s0:s1] = (1.0 - r2 / (b * b)).clamp_min(0.0).sum(1)
    out, den = torch.empty_like(acc), torch.empty_like(rho)
    out[order], den[order] = gm * acc, rho
    return (out, den) if b is not None else out


def exact(case, seed):
    op, sizes = case["op"], _box_list(case)
    parts = _box_positions(case, seed)
    if op in ("one_shot", "step", "batch"):
        if sum(K ** 3 for _, K in sizes) > 50000:
            return None
        got = [_near_field_exact(p, K, _spacing(m) / 40.0, 1.0 / m, case["kind"]) for p, (m, K) in zip(parts, sizes)]
        return None if any(g is None for g in got) else torch.cat(got)
    pos, (n, K) = parts[0], sizes[0]
    eps, gm = _spacing(n) / 40.0, 1.0 / n
    if op == "density":
        return _near_field_exact(pos, K, eps, gm, case["kind"], DENSITY_RADIUS * _spacing(n)) if K <= 36 else None
    if op == "leapfrog":
        if K > 26:
            return None
        a0 = _near_field_exact(pos, K, eps, gm, case["kind"])
        if a0 is None:
            return None
        dt = 1e-4
        half = _velocities(seed, n).double() + a0 * (0.5 * dt)
        new = pos.double() + half * dt
        new = new - torch.floor(new)
        return {"pos": new, "vel": None, "acc": None, "dt": None}
    if op == "merge":
        return None          # moves and two multiply-adds: compared with the other side alone
    if op == "taylor":
        if case["sorted"]:
            pos = pos[torch.sort(_cell_of(pos, K)[0], stable=True)[1]].contiguous()
        taylor, acc = _taylor_inputs(case, seed, n)
        acc = acc.double()
    cell, u = _cell_of(pos, K)
    comp = _components(case["order"])
    power = [[torch.ones_like(u[:, 0])] for _ in range(3)]
    for d in range(3):
        for _ in range(case["order"]):
            power[d].append(power[d][-1] * u[:, d])
    if op == "moments":
        out = torch.zeros((K ** 3, len(comp)), dtype=torch.float64, device="cuda")
        col = torch.empty(K ** 3, dtype=torch.float64, device="cuda")
        for i, (a, b, k) in enumerate(comp):
            out[:, i] = col.zero_().index_add_(0, cell, power[0][a] * power[1][b] * power[2][k]) * gm
        return out
    for i, e in enumerate(comp):
        t = taylor[:, i].contiguous()[cell] * float(K)
        for d in range(3):
            if e[d]:
                term = t * float(e[d])
                for q in range(3):
                    term = term * power[q][e[q] - (q == d)]
                acc[:, d] -= term
    return acc
