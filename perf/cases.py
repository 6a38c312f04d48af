"""Workloads of the library's public entry points, for timing one build against another.

A case is a dict of plain values.  `listed()` gives the fixed ones, `draw(rng)`
one more of the same ranges, `prepare(case, seed)` what a program holds before
the call (particles, plan, flags), `run(state)` one pass, `work(case)` the bytes
and floating-point operations a pass cannot do without, and `exact(case, seed)`
the same outputs from plain FP64 torch, where that takes seconds.

Boxes are a uniform background plus Plummer spheres whose particle counts
follow dN/dM ~ M^-1.9 from 64 up, as in the `workloads` module, drawn on the
GPU.  The mesh fixes the split: r_s = 1.25 cells, r_cut = 4.5 r_s, softening
0.02 cells.  The adaptive integrator appears through the force evaluations it
consists of (whole box, active subset, reused lists, mesh force), which have
comparable outputs; its trajectories branch on rounding (a particle's step
level is a threshold on its force).
"""
import math

import numpy as np
import torch

import paper_1802_09824_amd as pp

M_MIN, SLOPE = 64.0, 1.9
SPHERE = 512                 # mean particles per sphere of the drawn boxes
FLOP_PER_PAIR = 38           # the polynomial pair kernel, per pair inside the cut
FLOP_PER_PAIR_64 = 60        # difference, root, quotients and split factor in FP64
DIRECT_MAX = 2.2e10          # pairs inside the cut that exact() sums in about 15 s


class Params:
    """L, rs, rcut, eps, G, leaf_max, key_bits of one box."""

    def __init__(self, L, mesh, leaf_max=32, key_bits=21):
        cell = L / mesh
        self.L, self.rs, self.rcut, self.eps, self.G = L, 1.25 * cell, 4.5 * 1.25 * cell, 0.02 * cell, 1.0
        self.leaf_max, self.key_bits = leaf_max, key_bits


def _box(name, kind, n, L, mesh, frac, spheres, **more):
    c = {"kind": kind, "n": n, "L": L, "mesh": mesh, "frac": frac, "spheres": spheres, "unequal": False, "leaf_max": 32,
         "chunk": 0, "waves_per_block": 0, "persistent": 1}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # the smallest box a program solves: a zoom region or a unit test of a user's code; latency only
        _box("accel-1k", "accel", 1000, 50.0, 12, 0.0, 0),
        # the 32^3 uniform box of the benchmark (early times), at the default tiles
        _box("accel-32k-uniform", "accel", 32768, 100.0, 32, 0.0, 0),
        # the allocation-free entry point inside somebody else's loop: a ragged clustered box
        _box("scratch-20k", "scratch", 20011, 80.0, 27, 0.5, 20),
        # an ordinary ragged box with unequal masses (several species), lightly clustered
        _box("accel-300k-unequal", "accel", 300007, 120.0, 67, 0.3, 176, unequal=True),
        # the benchmark's headline box
        _box("accel-2m-clustered", "accel", 2097152, 200.0, 128, 0.5, 2000),
        # the 256^3 precision box at the tiles the autotuner settles on for large boxes
        _box("accel-16m-clustered", "accel", 16777216, 400.0, 256, 0.5, 8000, chunk=8192, waves_per_block=4),
        # many independent boxes in one call (parameter studies, ensembles)
        {"name": "batch-64", "kind": "batch", "boxes": 64, "n_lo": 4096, "n_hi": 884736, "frac_hi": 0.8, "sizes": 4, "leaf_max": 32},
        # the FP64 yardstick a user checks a production force against
        _box("f64-262k", "f64", 262144, 100.0, 64, 0.5, 256, unequal=True),
        # a substep of the adaptive integrator: new lists, forces of the fifth of the particles in dense regions
        _box("active-2m", "active", 2097152, 200.0, 128, 0.5, 2000, active=0.4),
        # the same when the lists are reused on moved particles (skin 0.2 r_cut)
        _box("substep-1m-skin", "skin", 1000003, 160.0, 100, 0.5, 977, active=0.4),
        # the long-range half of every force evaluation, 128^3 mesh
        _box("pm-2m-mesh128", "pm", 2097152, 200.0, 128, 0.5, 2000),
        # the tree approximation on a larger box (both opening tests)
        _box("mono-4m", "mono", 4000000, 250.0, 160, 0.6, 1500, theta=0.3, alpha=0.005),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["accel", "accel", "accel", "scratch", "batch", "f64", "active", "skin", "pm", "mono"])
    if kind == "batch":
        lo = log_int(1000, 40000)
        return {"kind": "batch", "boxes": rng.randint(2, 40), "n_lo": lo, "n_hi": log_int(lo, 400000), "frac_hi": round(rng.uniform(0.0, 0.8), 2),
                "sizes": rng.randint(10, 9999), "leaf_max": rng.choice([32, 32, 16])}
    n = {"accel": lambda: log_int(1000, 6000000), "scratch": lambda: log_int(1000, 50000), "f64": lambda: log_int(4000, 500000),
         "active": lambda: log_int(20000, 4000000), "skin": lambda: log_int(20000, 2000000), "pm": lambda: log_int(5000, 8000000),
         "mono": lambda: log_int(100000, 4000000)}[kind]()
    frac = rng.choice([0.0, round(rng.uniform(0.05, 0.7), 2), round(rng.uniform(0.05, 0.7), 2)])
    if kind in ("active", "skin", "mono"):
        frac = max(frac, 0.2)
    side = n ** (1.0 / 3.0)
    mesh = max(12, int(round(side * rng.uniform(0.9, 1.2))))
    c = _box("", kind, n, round(rng.uniform(50.0, 300.0), 3), mesh, frac, max(1, int(n * frac / SPHERE)) if frac else 0,
             unequal=rng.random() < 0.4, leaf_max=rng.choice([32, 32, 32, 16, 64]) if kind == "accel" else 32)
    if kind == "accel" and n > 200000 and rng.random() < 0.4:
        c.update(chunk=rng.choice([1024, 4096, 8192]), waves_per_block=rng.choice([1, 2, 4]), persistent=rng.choice([1, 1, 0]))
    if kind in ("active", "skin"):
        c["active"] = round(rng.uniform(0.05, 0.9), 2)
    if kind == "mono":
        c.update(theta=rng.choice([0.3, 0.5]), alpha=rng.choice([0.0, 0.005]))
    if kind == "pm":
        c["mesh"] = max(12, min(256, int(round(side * rng.uniform(0.6, 1.2)))))
    return c


# ------------------------------------------------------------- particles --
def _m_max(mean):
    a = 1.0 - SLOPE

    def at(m):
        return (m ** (a + 1) - M_MIN ** (a + 1)) / (a + 1) / ((m ** a - M_MIN ** a) / a)

    if mean <= M_MIN * 1.001:
        return M_MIN * 1.002
    lo, hi = M_MIN * 1.001, 1e12
    for _ in range(200):
        mid = math.sqrt(lo * hi)
        lo, hi = (mid, hi) if at(mid) < mean else (lo, mid)
    return hi


def _sphere_mass(u, mean):
    """Masses of the power law at the uniform numbers u (torch or numpy)."""
    a = 1.0 - SLOPE
    lo, hi = M_MIN ** a, _m_max(mean) ** a
    return (lo + u * (hi - lo)) ** (1.0 / a)


def _particles(n, L, frac, spheres, unequal, gen):
    """Positions FP64 [3][n] in [0, L), masses FP32 [n], and which particles belong to a sphere."""
    def rand(*shape):
        return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=gen)

    pos = rand(3, n) * L
    n_cl = int(round(n * frac)) if spheres else 0
    member = torch.zeros(n, dtype=torch.bool, device="cuda")
    if n_cl:
        m = _sphere_mass(rand(spheres), n_cl / spheres)
        m = m * (n_cl / m.sum())
        scale = 0.05 * (m / (n / L ** 3)) ** (1.0 / 3.0)
        centre = rand(3, spheres) * L
        owner = torch.searchsorted(torch.cumsum(m, 0) / m.sum(), rand(n_cl)).clamp_(max=spheres - 1)
        u = (rand(n_cl) * (100.0 / 101.0) ** 1.5).clamp_(min=1e-12)
        r = scale[owner] / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
        v = torch.randn(3, n_cl, dtype=torch.float64, device="cuda", generator=gen)
        v = v / torch.sqrt((v * v).sum(0))
        x = centre[:, owner] + r * v
        at = torch.randperm(n, device="cuda", generator=gen)[:n_cl]     # input order holds no spatial order
        pos[:, at] = x - L * torch.floor(x / L)
        pos[pos >= L] = 0.0
        member[at] = True
    if unequal:
        mass = ((0.2 + 1.8 * rand(n)) / n).to(torch.float32)
    else:
        mass = torch.full((n,), 1.0 / n, dtype=torch.float32, device="cuda")
    return pos.contiguous(), mass, member


def _boxes(case):
    """(n, L, mesh, frac, spheres) of every box of a batch; the sizes are the case's, not the seed's."""
    r = np.random.RandomState(case["sizes"])
    out = []
    for _ in range(case["boxes"]):
        n = int(r.randint(case["n_lo"], case["n_hi"] + 1))
        frac = float(r.uniform(0.0, case["frac_hi"])) if case["frac_hi"] > 0 else 0.0
        out.append((n, float(r.uniform(50.0, 300.0)), max(12, int(round(n ** (1.0 / 3.0)))), frac, max(1, int(round(n * frac / SPHERE)))))
    return out


def _inputs(case, seed):
    """The pass's inputs, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(180209824 + 1000003 * int(seed))
    if case["kind"] == "batch":
        parts = [_particles(n, L, frac, sph, b % 3 == 2, gen) for b, (n, L, _, frac, sph) in enumerate(_boxes(case))]
        return {"pos": torch.cat([q[0] for q in parts], 1).contiguous(), "mass": torch.cat([q[1] for q in parts])}
    L = case["L"]
    pos, mass, member = _particles(case["n"], L, case["frac"], case["spheres"], case["unequal"], gen)
    got = {"pos": pos, "mass": mass}
    if case["kind"] in ("active", "skin"):
        u = torch.rand(case["n"], device="cuda", generator=gen)
        got["active"] = (member & (u < case["active"])).to(torch.uint8)
    if case["kind"] == "skin":
        p = _params(case)
        d = torch.randn(3, case["n"], dtype=torch.float64, device="cuda", generator=gen)
        d = d / torch.sqrt((d * d).sum(0)) * (0.08 * p.rcut) * torch.rand(case["n"], dtype=torch.float64, device="cuda", generator=gen)
        x = pos + d
        got["moved"] = (x - L * torch.floor(x / L)).contiguous()
    if case["kind"] == "f64":
        got["mass"] = mass.to(torch.float64)
    return got


def _params(case):
    return Params(case["L"], case["mesh"], case["leaf_max"])


# ------------------------------------------------------------------ runs --
def prepare(case, seed):
    s = _inputs(case, seed)
    kind = s["kind"] = case["kind"]
    n = s["pos"].shape[1]
    if kind == "batch":
        boxes = _boxes(case)
        s["plan"] = pp.BatchPlan([Params(L, mesh, case["leaf_max"]) for _, L, mesh, _, _ in boxes], [b[0] for b in boxes])
    elif kind == "scratch":
        s["params"] = _params(case)
    elif kind == "pm":
        s["plan"] = pp.PMPlan(_params(case), case["mesh"])
    else:
        s["plan"] = pp.Plan(_params(case), n)
    if kind == "accel" and case["chunk"]:
        s["plan"].set_tuning(chunk=case["chunk"], waves_per_block=case["waves_per_block"], persistent=case["persistent"])
    if kind == "mono":
        # the reference forces of the relative test: the previous step's, kept in 16 bits (a size, not a result)
        ref = s["plan"].accel(s["pos"], s["mass"]).to(torch.bfloat16).to(torch.float32) if case["alpha"] > 0 else None
        s["plan"].set_monopole(case["theta"])
        if ref is not None:
            s["plan"].set_monopole_relative(case["alpha"], ref)
    if kind == "skin":
        # the lists of an earlier substep
        s["plan"].set_skin(0.2 * _params(case).rcut)
        s["plan"].accel(s["pos"], s["mass"])
    s["out"] = torch.zeros(3, n, dtype=torch.float64 if kind == "f64" else torch.float32, device="cuda")
    return s


def run(s):
    kind = s["kind"]
    if kind == "f64":
        return s["plan"].accel_f64(s["pos"], s["mass"], s["out"])
    if kind == "scratch":
        return pp.pp_accel_scratch(s["params"], s["pos"], s["mass"], s["out"])
    if kind == "active":
        return s["plan"].accel_active(s["pos"], s["mass"], s["active"], s["out"])
    if kind == "skin":
        return s["plan"].accel_active(s["moved"], s["mass"], s["active"], s["out"])
    return s["plan"].accel(s["pos"], s["mass"], s["out"])


# ------------------------------------------------------------------ work --
def _pairs(n, L, mesh, frac, spheres):
    """Expected ordered pairs inside the cut: the background and every sphere on itself."""
    rcut = 4.5 * 1.25 * L / mesh
    pairs = float(n) * n * (4.0 / 3.0 * math.pi * rcut ** 3 / L ** 3)
    n_cl = int(round(n * frac)) if spheres else 0
    if n_cl:
        r = np.random.RandomState(1)
        m = _sphere_mass((np.arange(spheres) + 0.5) / spheres, n_cl / spheres)
        m *= n_cl / m.sum()
        a = 0.05 * (m / (n / L ** 3)) ** (1.0 / 3.0)
        u = np.maximum(r.rand(2, 4000) * (100.0 / 101.0) ** 1.5, 1e-12)
        v = r.randn(3, 2, 4000)
        x = v / np.sqrt((v * v).sum(0)) / np.sqrt(u ** (-2.0 / 3.0) - 1.0)
        d = np.sort(np.sqrt(((x[:, 0] - x[:, 1]) ** 2).sum(0)))           # separations in scale radii
        pairs += float((m * m * np.searchsorted(d, rcut / a) / d.size).sum())
    return pairs


def _case_pairs(case):
    if case["kind"] == "batch":
        return sum(_pairs(n, L, mesh, frac, sph) for n, L, mesh, frac, sph in _boxes(case))
    return _pairs(case["n"], case["L"], case["mesh"], case["frac"], case["spheres"])


def work(case):
    kind = case["kind"]
    n = sum(b[0] for b in _boxes(case)) if kind == "batch" else case["n"]
    if kind == "pm":
        # particles in and out, the mesh once through each of the transforms and the gradient; 8-point weights both ways
        cells = float(case["mesh"]) ** 3
        return {"bytes": n * (24 + 4 + 12) + 8.0 * cells * 8, "flops": n * (8 * 4 + 8 * 7) + cells * (2 * 2.5 * 3 * math.log2(case["mesh"]) + 30)}
    pairs = _case_pairs(case)
    if kind == "f64":
        return {"bytes": n * (24 + 8 + 24), "flops": pairs * FLOP_PER_PAIR_64}
    b = n * (24 + 4 + 12)
    if kind in ("active", "skin"):
        on = case["frac"] * case["active"]
        cl = pairs - float(n) * n * (4.0 / 3.0 * math.pi * (5.625 / case["mesh"]) ** 3)
        pairs = case["active"] * cl + on * (pairs - cl)          # the active particles are sphere members
        b = n * (24 + 4 + 1 + 12 * on)
    if kind == "mono":
        pairs *= 0.6                                             # about what the opening tests leave of the pairs
    return {"bytes": b, "flops": pairs * FLOP_PER_PAIR}


# ----------------------------------------------------------------- exact --
def _sum_pairs(pt, ps, ms, p):
    """FP64 accelerations of the targets pt [3][T] from the sources ps [3][S] (masses ms [S]), minimum image."""
    T, S = pt.shape[1], ps.shape[1]
    out = torch.empty(3, T, dtype=torch.float64, device=pt.device)
    step = max(1, int(2e7 // max(S, 1)))
    for a in range(0, T, step):
        d = [ps[k][None, :] - pt[k, a:a + step][:, None] for k in range(3)]
        d = [x - p.L * torch.round(x / p.L) for x in d]
        s2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
        se = torch.sqrt(s2 + p.eps ** 2)
        x = se / (2.0 * p.rs)
        f = (torch.erfc(x) + 2.0 / math.sqrt(math.pi) * x * torch.exp(-x * x)) / (se * se * se) * (p.G * ms)[None, :]
        f = torch.where((s2 < p.rcut ** 2) & (s2 > 0), f, torch.zeros_like(f))
        for k in range(3):
            out[k, a:a + step] = (f * d[k]).sum(1)
    return out


def _direct(pos, mass, p, on=None):
    """The short-range sum of one box in FP64, by cells at least r_cut wide; columns with on == 0 stay 0."""
    n = pos.shape[1]
    m = mass.to(torch.float64)
    out = torch.zeros(3, n, dtype=torch.float64, device=pos.device)
    dims = int(p.L / p.rcut * (1 - 1e-9))
    if dims < 4 or n < 5000:
        at = torch.arange(n, device=pos.device) if on is None else torch.nonzero(on).flatten()
        out[:, at] = _sum_pairs(pos[:, at], pos, m, p)
        return out
    c = (pos * (dims / p.L)).to(torch.int64).clamp_(0, dims - 1)
    cid = (c[0] * dims + c[1]) * dims + c[2]
    order = torch.argsort(cid)
    pos_s, m_s = pos[:, order].contiguous(), m[order]
    on_s = None if on is None else on[order] != 0
    beg = [0] + torch.cumsum(torch.bincount(cid, minlength=dims ** 3), 0).tolist()
    res = torch.zeros_like(pos_s)
    for cell in range(dims ** 3):
        a, b = beg[cell], beg[cell + 1]
        if a == b:
            continue
        at = torch.arange(a, b, device=pos.device) if on is None else a + torch.nonzero(on_s[a:b]).flatten()
        if at.numel() == 0:
            continue
        x, y, z = cell // (dims * dims), cell // dims % dims, cell % dims
        cells = [(((x + i) % dims) * dims + (y + j) % dims) * dims + (z + k) % dims for i in (-1, 0, 1) for j in (-1, 0, 1) for k in (-1, 0, 1)]
        ps = torch.cat([pos_s[:, beg[q]:beg[q + 1]] for q in cells], 1)
        ms = torch.cat([m_s[beg[q]:beg[q + 1]] for q in cells])
        res[:, at] = _sum_pairs(pos_s[:, at], ps, ms, p)
    out[:, order] = res
    return out


def _direct_pm(pos, mass, p, N):
    """CIC assignment, Green function with the long-range filter, 4-point gradient, CIC interpolation, in FP64."""
    L, d = p.L, p.L / N
    w = pos / d
    c = torch.floor(w)
    f = w - c
    i0 = c.to(torch.int64) % N
    corners = []
    for a in (0, 1):
        for b in (0, 1):
            for e in (0, 1):
                wt = (f[0] if a else 1 - f[0]) * (f[1] if b else 1 - f[1]) * (f[2] if e else 1 - f[2])
                corners.append(((((i0[0] + a) % N) * N + (i0[1] + b) % N) * N + (i0[2] + e) % N, wt))
    rho = torch.zeros(N ** 3, dtype=torch.float64, device=pos.device)
    for idx, wt in corners:
        rho.index_add_(0, idx, wt * mass.to(torch.float64))
    rk = torch.fft.rfftn((rho / d ** 3).reshape(N, N, N))
    k = torch.fft.fftfreq(N, 1.0 / N, dtype=torch.float64, device=pos.device)
    kz = torch.arange(N // 2 + 1, dtype=torch.float64, device=pos.device)
    kx, ky, kz = k[:, None, None], k[None, :, None], kz[None, None, :]
    S = torch.sin(math.pi * kx / N) ** 2 + torch.sin(math.pi * ky / N) ** 2 + torch.sin(math.pi * kz / N) ** 2
    S[0, 0, 0] = 1.0
    green = -math.pi * p.G * d * d / S * torch.exp(-(2 * math.pi / L) ** 2 * (kx ** 2 + ky ** 2 + kz ** 2) * p.rs ** 2)
    green[0, 0, 0] = 0.0
    phi = torch.fft.irfftn(rk * green, s=(N, N, N))
    out = torch.zeros_like(pos)
    for ax in range(3):
        g = -(8 * (torch.roll(phi, -1, ax) - torch.roll(phi, 1, ax)) - (torch.roll(phi, -2, ax) - torch.roll(phi, 2, ax))) / (12 * d)
        g = g.reshape(-1)
        for idx, wt in corners:
            out[ax] += wt * g[idx]
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "mono":
        return None                  # the opening tests define the result, not a sum
    if kind != "pm" and _case_pairs(case) > DIRECT_MAX:
        return None
    s = _inputs(case, seed)
    if kind == "pm":
        return _direct_pm(s["pos"], s["mass"], _params(case), case["mesh"])
    if kind == "batch":
        out, a = [], 0
        for n, L, mesh, _, _ in _boxes(case):
            out.append(_direct(s["pos"][:, a:a + n].contiguous(), s["mass"][a:a + n], Params(L, mesh, case["leaf_max"])))
            a += n
        return torch.cat(out, 1)
    return _direct(s["moved"] if kind == "skin" else s["pos"], s["mass"], _params(case), s.get("active"))
