"""The work that programs built on this framework have it do, as cases to be
timed: whole steps, the solve, the product and the constraint geometry on
their own, batches, gradients of rollouts, and the crosslinker kinetics with
and without the coupled filament step.

Sizes and input laws are those of the benchmark and the tests: 400 and 1,000
rods for the smallest calls, the confined suspension of 3,200 rods, 10,000
rods of mixed lengths, the 100,000-rod nematic suspension, 400,000 rods of
mixed lengths for the mixed-precision solve.  Units are um, s and pN; the
inputs are drawn on the GPU from the seed.

The constraint forces gamma of a contact network are not unique (the matrix of
the problem is only semi-definite), the velocities are: the solves return U.
"""
from __future__ import annotations

import math

import torch

import paper_2109_08206_amd as rl
from paper_2109_08206_amd.rollout import rollout

DEV = "cuda:0"
F64 = torch.float64
ETA, DT, DIAM, CUTOFF, TOL = 0.01, 1.0e-4, 0.025, 0.05, 1.0e-8
KT = 4.11e-3
UM3 = 602.214076  # molecules per um^3 at 1 uM


def listed():
    return [
        # one timestep of a small dilute suspension: the smallest whole step a
        # simulation takes, tens of short launches and a few host waits
        {"name": "step_1k", "kind": "step", "n": 1000, "phi": 0.008, "nematic": False, "mixed_len": False,
         "precision": "f64", "brownian": False},
        # one Brownian timestep of a mid-size suspension with mixed lengths
        {"name": "step_10k_lengths", "kind": "step", "n": 10_000, "phi": 0.02, "nematic": False, "mixed_len": True,
         "precision": "f64", "brownian": True},
        # one timestep of a paper-scale nematic suspension (the benchmark's rods
        # at a volume fraction where the iteration count of an unrelaxed start
        # does not yet swing severalfold with the last bit of a sum)
        {"name": "step_100k_nematic", "kind": "step", "n": 100_000, "phi": 0.03, "nematic": True, "mixed_len": False,
         "precision": "f64", "brownian": False},
        # one timestep at the largest size, through the mixed-precision solve
        {"name": "step_400k_mixed", "kind": "step", "n": 400_000, "phi": 0.02, "nematic": False, "mixed_len": True,
         "precision": "mixed", "brownian": False},
        # one solve on a list in hand, at the size of a unit test or a
        # single small cluster of an outer loop: latency only
        {"name": "solve_400", "kind": "solve", "n": 400, "phi": 0.0075, "nematic": False, "mixed_len": False},
        # the product Mc gamma + q alone on an odd-sized list (an outer
        # solver's operator)
        {"name": "product_100k", "kind": "product", "n": 100_003, "phi": 0.05, "nematic": True, "mixed_len": False},
        # neighbour search and constraint geometry alone (analysis, or a
        # program with its own solver) at paper scale
        {"name": "geometry_100k", "kind": "geometry", "n": 100_000, "phi": 0.05, "nematic": True, "mixed_len": False},
        # a parameter sweep: many systems of very different sizes in one solve
        {"name": "batch_64", "kind": "batch", "systems": 64, "n_lo": 200, "n_hi": 20_000, "phi_lo": 0.005,
         "phi_hi": 0.02},
        # forward and backward through a short differentiable rollout of a
        # small suspension
        {"name": "rollout_2k", "kind": "rollout", "n": 2000, "phi": 0.01, "steps": 4},
        # the same with the rods of the benchmark's rollout
        {"name": "rollout_50k", "kind": "rollout", "n": 50_000, "phi": 0.01, "steps": 2},
        # crosslinker kinetics of the benchmark (400,000 crosslinkers on
        # 100,000 filaments)
        {"name": "kinetics_400k", "kind": "kinetics", "n": 100_000, "m": 400_000, "phi": 0.05},
        # a coupled step of the paper's confined suspension: kinetics, then
        # contacts, links and the shell with Brownian forces and the stress
        {"name": "coupled_3200", "kind": "coupled", "n": 3200, "m": 8000},
    ]


def _log_int(rng, lo, hi):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "solve", "product", "geometry", "batch", "rollout", "kinetics",
                       "coupled"])
    nematic = rng.random() < 0.4
    phi = round(rng.uniform(0.005, 0.05 if nematic else 0.02), 4)
    mixed_len = rng.random() < 0.4
    if kind in ("step", "solve"):
        phi = min(phi, 0.03)  # iteration counts of unrelaxed starts swing beyond it
    if kind == "step":
        # beyond 50,000 rods the volume fraction stays below where the
        # largest listed step would be passed
        mixed = rng.random() < 0.25
        n = _log_int(rng, 1000, 300_000)
        if n > 50_000:
            phi = min(phi, 0.02)
        return {"kind": kind, "n": n, "phi": phi, "nematic": nematic, "mixed_len": mixed_len,
                "precision": "mixed" if mixed else "f64", "brownian": rng.random() < 0.5}
    if kind in ("solve", "product", "geometry"):
        return {"kind": kind, "n": _log_int(rng, 1000 if mixed_len else 400, 30_000 if kind == "solve" else 200_000),
                "phi": min(phi, 0.01) if mixed_len else phi if nematic else min(phi, 0.02), "nematic": nematic,
                "mixed_len": mixed_len}
    if kind == "batch":
        return {"kind": kind, "systems": rng.randint(8, 64), "n_lo": 200, "n_hi": _log_int(rng, 600, 15_000),
                "phi_lo": 0.005, "phi_hi": round(rng.uniform(0.008, 0.02), 4)}
    if kind == "rollout":
        return {"kind": kind, "n": _log_int(rng, 1000, 30_000), "phi": round(rng.uniform(0.005, 0.01), 4),
                "steps": rng.randint(1, 4)}
    if kind == "kinetics":
        n = _log_int(rng, 2000, 100_000)
        return {"kind": kind, "n": n, "m": int(n * rng.uniform(0.5, 4.0)), "phi": round(rng.uniform(0.01, 0.05), 4)}
    n = _log_int(rng, 800, 20_000)
    return {"kind": kind, "n": n, "m": int(n * rng.uniform(0.5, 2.5))}


# --- inputs -------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(shape, dtype=F64, device=DEV, generator=g)


def _randn(g, *shape):
    return torch.randn(shape, dtype=F64, device=DEV, generator=g)


def _quats(g, n, nematic):
    """Haar-uniform unit quaternions, or axes from a von Mises-Fisher law
    about z with concentration 20."""
    if not nematic:
        q = _randn(g, n, 4)
        return (q / q.norm(dim=1, keepdim=True)).contiguous()
    u = _rand(g, n)
    w = (1.0 + torch.log(u + (1.0 - u) * math.exp(-40.0)) / 20.0).clamp(-1.0, 1.0)
    return _tilt(w, _rand(g, n) * 2.0 * math.pi, _rand(g, n) * 2.0 * math.pi)


def _tilt(w, az, twist):
    beta = torch.arccos(w)
    c1, s1 = torch.cos(beta / 2), torch.sin(beta / 2)
    c2, s2 = torch.cos(twist / 2), torch.sin(twist / 2)
    ax, ay = -torch.sin(az), torch.cos(az)
    q = torch.stack([c1 * c2, s1 * (ax * c2 + ay * s2), s1 * (ay * c2 - ax * s2), c1 * s2], dim=1)
    return (q / q.norm(dim=1, keepdim=True)).contiguous()


def _box(length, n, phi):
    """Edge of the periodic cube at a volume fraction (spherocylinders)."""
    vol = math.pi * DIAM ** 2 / 4.0 * (float(length.sum()) if isinstance(length, torch.Tensor) else length * n) \
        + n * math.pi * DIAM ** 3 / 6.0
    return (vol / phi) ** (1.0 / 3.0)


def _suspension(g, n, phi, nematic, mixed_len):
    length = 0.5 + _rand(g, n) if mixed_len else 1.0
    box = _box(length, n, phi)
    x = _rand(g, n, 3) * box
    x = torch.where(x >= box, torch.zeros_like(x), x).contiguous()
    return {"n": n, "box": box, "length": length, "x0": x, "quat0": _quats(g, n, nematic), "F": _randn(g, n, 6)}


def _moved_suspension(g, case):
    """The suspension of this size, moved through its periodic box, its rods
    renumbered and loaded by the seed: lists of one length for every seed."""
    s = _suspension(_gen(case["n"]), case["n"], case["phi"], case["nematic"], case["mixed_len"])
    order = torch.randperm(case["n"], device=DEV, generator=g)
    x = torch.remainder(s["x0"] + _rand(g, 1, 3) * s["box"], s["box"])[order]
    s["x0"] = torch.where(x >= s["box"], torch.zeros_like(x), x).contiguous()
    s["quat0"] = s["quat0"][order].contiguous()
    s["F"] = _randn(g, case["n"], 6)
    if case["mixed_len"]:
        s["length"] = s["length"][order].contiguous()
    return s


def _confined(g, n):
    """Rods of length 1 in a spherical shell at the density of 3,200 rods in
    radius 3, both ends 0.02 + diam/2 inside it."""
    radius = 3.0 * (n / 3200.0) ** (1.0 / 3.0)
    box = 2.0 * radius + 3.0
    c = 0.5 * box
    m = 6 * n + 64
    x = c + radius * (2.0 * _rand(g, m, 3) - 1.0)
    a = _randn(g, m, 3)
    a = a / a.norm(dim=1, keepdim=True)
    lim = radius - 0.02 - 0.5 * DIAM
    ok = ((x + 0.5 * a - c).norm(dim=1) <= lim) & ((x - 0.5 * a - c).norm(dim=1) <= lim)
    x, a = x[ok][:n].contiguous(), a[ok][:n]
    quat = _tilt(a[:, 2].clamp(-1.0, 1.0), torch.atan2(a[:, 1], a[:, 0]), _rand(g, n) * 2.0 * math.pi)
    return {"n": n, "box": box, "length": 1.0, "x0": x, "quat0": quat, "F": _randn(g, n, 6), "radius": radius}


def _solver(box, precision="f64", tol=TOL, n=0, contacts=0.0):
    slv = rl.Solver(box=box, diam=DIAM, cutoff=CUTOFF, eta=ETA, dt=DT, tol=tol, max_iter=200_000,
                    precision=rl.FP32_MIXED if precision == "mixed" else rl.FP64)
    if n:
        # a simulation knows its size: workspace for the steps to come
        slv.reserve(n, (int(1.5 * contacts) // 4096 + 4) * 4096)
    return slv


def _constraints(s):
    """The step's constraint list, as a program that calls the solve itself holds it."""
    slv = s["slv"]
    s["dir"] = slv.directors(s["quat0"])
    pi, pj, img, _ = slv.build_pairs(s["x0"], s["dir"], s["length"])
    s["pi"], s["pj"], s["img"] = pi.contiguous(), pj.contiguous(), img.contiguous()
    s["phi"], s["e"], s["arm"], s["q"] = slv.assemble_D(s["x0"], s["dir"], s["length"], s["pi"], s["pj"], s["img"],
                                                        s["F"])


def _crosslinkers(s, g, m, koff, steps, centres):
    """Crosslinkers with the kinesin-5 parameters of the crosslinker table,
    taken from all unbound by steps of the kinetics itself."""
    s["kp"] = rl.kmc_params(eps=1625.0, Ka=90.9 / UM3, koS=koff, Ke=90.9 / UM3, koD=koff, kappa=300.0, rest=0.053,
                            lam=0.258, kT=KT, rcs=0.039, rcd=0.11, dU=1.0)
    s["state0"] = torch.zeros(m, dtype=torch.int32, device=DEV)
    s["rod0"] = torch.full((m, 2), -1, dtype=torch.int32, device=DEV)
    s["arc0"] = torch.zeros((m, 2), dtype=F64, device=DEV)
    s["xl0"] = centres
    d = s["slv"].directors(s["quat0"])
    for _ in range(steps):
        s["slv"].kmc_step(s["x0"], d, 1.0, s["kp"], s["state0"], s["rod0"], s["arc0"], s["xl0"], _rand(g, m, 4),
                          _randn(g, m, 3))
    s["u"], s["xi"] = _rand(g, m, 4), _randn(g, m, 3)
    for k in ("state", "rod", "arc", "xl"):
        s[k] = s[k + "0"].clone()


def _batch_systems(case, seed):
    """Sizes spread evenly over their logarithm in a scattered order, volume
    fractions evenly over their range."""
    g, S = _gen(seed), case["systems"]
    lo, hi = math.log(case["n_lo"]), math.log(case["n_hi"])
    out = []
    for k in range(S):
        a, b = (k * 0.6180339887498949) % 1.0, (k * 0.7548776662466927) % 1.0
        out.append(_suspension(g, int(math.exp(lo + (hi - lo) * a)),
                               case["phi_lo"] + (case["phi_hi"] - case["phi_lo"]) * b, False, False))
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        parts, ro, po = [], [0], [0]
        for s in _batch_systems(case, seed):
            s["slv"] = _solver(s["box"])
            _constraints(s)
            s["slv"].close()
            parts.append(s)
            ro.append(ro[-1] + s["n"])
            po.append(po[-1] + s["pi"].shape[0])
        cat = {k: torch.cat([p[k] for p in parts]).contiguous() for k in ("dir", "e", "arm", "q", "F")}
        cat["pi"] = torch.cat([p["pi"] + ro[k] for k, p in enumerate(parts)]).to(torch.int32).contiguous()
        cat["pj"] = torch.cat([p["pj"] + ro[k] for k, p in enumerate(parts)]).to(torch.int32).contiguous()
        return {"kind": kind, "slv": _solver(1.0), "length": 1.0, "ro": ro, "po": po, **cat}
    g = _gen(seed)
    if kind == "coupled":
        s = _confined(g, case["n"])
        s["slv"] = _solver(s["box"], n=case["n"], contacts=4.0 * case["n"] + case["m"])
        c, r = 0.5 * s["box"], s["radius"]
        pts = _randn(g, case["m"], 3)
        pts = c + r * pts / pts.norm(dim=1, keepdim=True) * _rand(g, case["m"], 1) ** (1.0 / 3.0)
        _crosslinkers(s, g, case["m"], 30.0, 8, pts.contiguous())
        s["walls"] = [(rl.WALL_SPHERE_IN, (c, c, c), (0.0, 0.0, 1.0), r)]
        s["noise"] = _randn(g, case["n"], 6)
    elif kind == "kinetics":
        s = _suspension(g, case["n"], case["phi"], True, False)
        s["slv"] = _solver(s["box"])
        _crosslinkers(s, g, case["m"], 0.11, 50, (_rand(g, case["m"], 3) * s["box"] * (1.0 - 1e-15)).contiguous())
        s["dir"] = s["slv"].directors(s["quat0"])
    elif kind == "rollout":
        s = _suspension(g, case["n"], case["phi"], False, False)
        # gradients want the forces themselves converged
        s["slv"] = _solver(s["box"], tol=1e-10, n=case["n"], contacts=_contacts(case["n"], case["phi"], False))
        s["F"] = _randn(g, case["steps"], case["n"], 6).requires_grad_()
        s["x0"].requires_grad_()
        s["quat0"].requires_grad_()
    else:
        s = _moved_suspension(g, case) if kind in ("product", "geometry") else \
            _suspension(g, case["n"], case["phi"], case["nematic"], case["mixed_len"])
        s["slv"] = _solver(s["box"], case.get("precision", "f64"), n=case["n"],
                           contacts=_contacts(case["n"], case["phi"], case["nematic"]))
        if kind in ("solve", "product"):
            _constraints(s)
        if kind == "product":
            s["gamma"] = (_randn(g, s["pi"].shape[0])).clamp(min=0.0)
        if case.get("brownian"):
            s["noise"] = _randn(g, case["n"], 6)
    s["kind"] = kind
    if kind in ("step", "coupled"):
        s["x"], s["quat"] = s["x0"].clone(), s["quat0"].clone()
    return s


# --- one pass -----------------------------------------------------------------

def _kinetics(s, dir_):
    # the pass starts from the same bound states each time
    for k in ("state", "rod", "arc", "xl"):
        s[k].copy_(s[k + "0"])
    return s["slv"].kmc_step(s["x"] if s["kind"] == "coupled" else s["x0"], dir_, 1.0, s["kp"], s["state"], s["rod"],
                             s["arc"], s["xl"], s["u"], s["xi"])


def run(s):
    kind, slv = s["kind"], s["slv"]
    if kind == "step":
        # the step advances x and quat in place, from the same configuration each time
        s["x"].copy_(s["x0"])
        s["quat"].copy_(s["quat0"])
        U, _, npairs = slv.step(s["x"], s["quat"], s["length"], F=s["F"], noise=s.get("noise"), kT=KT)
        return {"U": U, "x": s["x"], "quat": s["quat"], "pairs": npairs}
    if kind == "solve":
        _, U, _ = slv.solve_lcp(s["dir"], s["length"], s["pi"], s["pj"], s["e"], s["arm"], s["q"], F=s["F"])
        return {"U": U}
    if kind == "product":
        return {"w": slv.apply_M(s["dir"], s["length"], s["pi"], s["pj"], s["e"], s["arm"], s["q"], s["gamma"])}
    if kind == "geometry":
        d = slv.directors(s["quat0"])
        pi, pj, img, flags = slv.build_pairs(s["x0"], d, s["length"])
        phi, e, arm, q = slv.assemble_D(s["x0"], d, s["length"], pi, pj, img, s["F"])
        return {"dir": d, "pi": pi, "pj": pj, "img": img, "flags": flags, "phi": phi, "e": e, "arm": arm, "q": q}
    if kind == "batch":
        _, U, _ = slv.solve_lcp_batched(s["ro"], s["po"], s["dir"], s["length"], s["pi"], s["pj"], s["e"], s["arm"],
                                        s["q"], F=s["F"])
        return {"U": U}
    if kind == "rollout":
        xu, quat = rollout(slv, s["x0"], s["quat0"], s["length"], s["F"], checkpoint_every=2, cg_tol=1e-12)
        gx, gq, gF = torch.autograd.grad((xu * xu).sum(), (s["x0"], s["quat0"], s["F"]))
        return {"x": xu.detach(), "quat": quat.detach(), "grad_x": gx, "grad_quat": gq, "grad_F": gF}
    if kind == "kinetics":
        events = _kinetics(s, s["dir"])
        return {"events": events, "state": s["state"], "rod": s["rod"], "arc": s["arc"], "xl": s["xl"]}
    s["x"].copy_(s["x0"])
    s["quat"].copy_(s["quat0"])
    events = _kinetics(s, slv.directors(s["quat"]))
    p, q, arm, kap, rest, key = slv.kmc_links(s["kp"], s["state"], s["rod"], s["arc"], keys=True)
    U, _, npairs = slv.step(s["x"], s["quat"], 1.0, F=s["F"], links=(p, q, arm, kap, rest, None, key),
                            walls=s["walls"], noise=s["noise"], kT=KT, stress=True)
    return {"events": events, "state": s["state"], "rod": s["rod"], "arc": s["arc"], "U": U, "x": s["x"],
            "quat": s["quat"], "pairs": npairs, "wall_contacts": slv.last_wall_contacts, "stress": slv.last_stress}


# --- what a pass cannot do without ----------------------------------------------

def _contacts(n, phi, nematic):
    """Constraints of a random suspension (rods of length 1): measured per rod
    and volume fraction."""
    return (94.0 if nematic else 156.0) * phi * n


def work(case):
    kind = case["kind"]
    nematic = bool(case.get("nematic")) or kind == "kinetics"
    n = case.get("n", 0)
    if kind == "batch":
        lo, hi = case["n_lo"], case["n_hi"]
        n = case["systems"] * (hi - lo) / math.log(hi / lo)
    phi = case.get("phi", 0.5 * (case.get("phi_lo", 0.0) + case.get("phi_hi", 0.0295)))
    nc = _contacts(n, phi, nematic)
    # a product: force sums on both rods, two mobilities, two contact
    # velocities; an iteration adds the step and three dot products
    per_iter = 70.0 * nc + 60.0 * n
    solve = 150.0 * per_iter
    search = 60.0 * nc + 250.0 * nc  # distance tests that pass, geometry
    rods_step = 8.0 * n * (2 * 7 + 6 + 6)
    lists = nc * (2 * 4 + 8.0 * (3 + 2 + 1))
    if kind == "step":
        return {"bytes": rods_step, "flops": solve + search}
    if kind in ("solve", "batch"):
        return {"bytes": lists + 8.0 * n * (3 + 6 + 6), "flops": solve}
    if kind == "product":
        return {"bytes": lists + 16.0 * nc + 24.0 * n, "flops": per_iter}
    if kind == "geometry":
        return {"bytes": 8.0 * n * (3 + 4 + 3 + 6) + nc * (13 + 8.0 * 7), "flops": search}
    if kind == "rollout":
        return {"bytes": case["steps"] * (2 * rods_step + 16.0 * nc), "flops": case["steps"] * 2.0 * (solve + search)}
    m = case["m"]
    kin = {"bytes": m * (2 * (4 + 8 + 16 + 24) + 56 + 48.0) + 48.0 * n, "flops": 2000.0 * m}
    if kind == "kinetics":
        return kin
    return {"bytes": kin["bytes"] + rods_step, "flops": kin["flops"] + solve + search}


# --- the same in plain torch, 64 bits -------------------------------------------

def _directors(q):
    s, a, b, c = q.unbind(1)
    return torch.stack([2.0 * (a * c + s * b), 2.0 * (b * c - s * a), s * s - a * a - b * b + c * c], dim=1)


def _mobility(length, n):
    L = length if isinstance(length, torch.Tensor) else torch.full((n,), float(length), dtype=F64, device=DEV)
    lg = torch.log(2.0 * L / DIAM)
    perp = lg / (4.0 * math.pi * ETA * L)
    return L, 2.0 * perp, perp, 3.0 * lg / (math.pi * ETA * L ** 3)


def _apply(d, mob, F):
    """U = M F: twice the mobility along the axis, one rotational mobility."""
    _, par, perp, rot = mob
    f, t = F[:, :3], F[:, 3:]
    v = perp[:, None] * f + ((par - perp) * (d * f).sum(1))[:, None] * d
    return torch.cat([v, rot[:, None] * t], dim=1)


def _closest(r0, di, hi, dj, hj):
    """Closest points of two segments by the clamped normal equations (no
    exactly parallel pairs in these inputs)."""
    b, c, f = (di * dj).sum(1), (di * r0).sum(1), (dj * r0).sum(1)
    s = torch.minimum(torch.maximum((b * f - c) / (1.0 - b * b), -hi), hi)
    t = b * s + f
    tc = torch.minimum(torch.maximum(t, -hj), hj)
    s = torch.where(t == tc, s, torch.minimum(torch.maximum(b * tc - c, -hi), hi))
    return s, tc, r0 + s[:, None] * di - tc[:, None] * dj


def _pairs(x, d, L, box):
    """(pi, pj, shift) of the pairs whose surface gap is below the cutoff, in
    ascending (pi, pj, shift) order, by testing every pair."""
    n, reach = x.shape[0], float(L.max()) + DIAM + CUTOFF
    near = box > 2.0 * reach
    k = 0 if near else int(math.ceil(reach / box)) + 1
    rng = range(-k, k + 1)
    shifts = [None] if near else [(a, b, c) for a in rng for b in rng for c in rng]
    got, rows = [], max(1, 60_000_000 // n)
    for i0 in range(0, n, rows):
        xi = x[i0:i0 + rows]
        for sh in shifts:
            d2 = torch.zeros((xi.shape[0], n), dtype=F64, device=DEV)
            for a in range(3):
                dx = xi[:, a, None] - x[None, :, a]
                dx = dx - box * torch.round(dx / box) if near else dx - box * sh[a]
                d2 += dx * dx
            m = 0.5 * (L[i0:i0 + rows, None] + L[None, :]) + DIAM + CUTOFF
            i, j = torch.nonzero(d2 < m * m, as_tuple=True)
            i = i + i0
            keep = (i < j) if near or sh <= (0, 0, 0) else (i <= j)
            i, j = i[keep], j[keep]
            dx = x[i] - x[j]
            w = torch.round(dx / box) if near else torch.tensor(sh, dtype=F64, device=DEV).expand(i.shape[0], 3)
            _, _, r = _closest(dx - box * w, d[i], 0.5 * L[i], d[j], 0.5 * L[j])
            hit = r.norm(dim=1) - DIAM < CUTOFF
            got.append((i[hit], j[hit], w[hit]))
    pi, pj, w = (torch.cat([g[k] for g in got]) for k in range(3))
    img = ((w[:, 0] + 8) * 256 + (w[:, 1] + 8) * 16 + w[:, 2] + 8).long()
    o = torch.argsort((pi * n + pj) * 4096 + img)
    return pi[o], pj[o], w[o]


def _geometry(x, d, mob, box, pi, pj, w, F):
    """phi, e, (s_i, s_j) and q = phi/h + D^T M F of the pairs."""
    L = mob[0]
    s, t, r = _closest(x[pi] - x[pj] - box * w, d[pi], 0.5 * L[pi], d[pj], 0.5 * L[pj])
    dist = r.norm(dim=1)
    e = r / dist[:, None]
    phi = dist - DIAM
    arm = torch.stack([s, t], dim=1)
    return phi, e, arm, phi / DT + _gap_rate(d, pi, pj, e, arm, _apply(d, mob, F))


def _point(d, U, i, s):
    """Velocity of the axis point at arclength s of rod i."""
    return U[i, :3] + s[:, None] * torch.linalg.cross(U[i, 3:], d[i])


def _gap_rate(d, pi, pj, e, arm, U):
    return (e * (_point(d, U, pi, arm[:, 0]) - _point(d, U, pj, arm[:, 1]))).sum(1)


def _forces(n, d, pi, pj, e, arm, gamma):
    """D gamma."""
    f = gamma[:, None] * e
    out = torch.zeros((n, 6), dtype=F64, device=DEV)
    ti = torch.linalg.cross(arm[:, :1] * d[pi], f)
    tj = torch.linalg.cross(arm[:, 1:] * d[pj], f)
    out = out.index_add(0, pi, torch.cat([f, ti], dim=1))
    return out.index_add(0, pj, -torch.cat([f, tj], dim=1))


def _minimise(n, d, mob, pi, pj, e, arm, q, tol=2e-11):
    """gamma of the complementarity problem by projected Barzilai-Borwein steps."""
    def product(v):
        return _gap_rate(d, pi, pj, e, arm, _apply(d, mob, _forces(n, d, pi, pj, e, arm, v)))

    gam = torch.zeros_like(q)
    if not q.numel():
        return gam
    g = q.clone()
    gh = torch.where((gam <= 0) & (g > 0), torch.zeros_like(g), g)
    den = (gh * product(gh)).sum()
    alpha = torch.where(den > 0, (gh * gh).sum() / den, torch.ones_like(den))
    best = (math.inf, gam)
    for k in range(60_000):
        new = (gam - alpha * g).clamp(min=0.0)
        gn = product(new) + q
        s, y = new - gam, gn - g
        ss, sy, yy = (s * s).sum(), (s * y).sum(), (y * y).sum()
        alpha = torch.where(sy > 0, ss / sy if k % 2 == 0 else sy / yy, alpha)
        gam, g = new, gn
        if k % 8 == 7:
            res = float(torch.minimum(gam, g).abs().max())
            if res < best[0]:
                best = (res, gam)
            if res <= tol:
                break
    return best[1]


def _integrate(x, quat, U, box):
    x = x + DT * U[:, :3]
    x = x - box * torch.floor(x / box)
    return x, _turn(quat, U)


def _turn(quat, U):
    s, p, w = quat[:, :1], quat[:, 1:], U[:, 3:]
    q = quat + 0.5 * DT * torch.cat([-(p * w).sum(1, keepdim=True), s * w - torch.linalg.cross(p, w)], dim=1)
    return q / q.norm(dim=1, keepdim=True)


def _brownian(d, mob, noise):
    """sqrt(2 kT / h) M^(-1/2) xi."""
    _, par, perp, rot = mob
    f, t = noise[:, :3], noise[:, 3:]
    a, b = par.rsqrt(), perp.rsqrt()
    v = b[:, None] * f + ((a - b) * (d * f).sum(1))[:, None] * d
    return math.sqrt(2.0 * KT / DT) * torch.cat([v, rot.rsqrt()[:, None] * t], dim=1)


class _Inverse(torch.autograd.Function):
    """A symmetric positive operator's inverse, by conjugate gradients."""

    @staticmethod
    def forward(ctx, b, op):
        ctx.op = op
        return _Inverse.cg(op, b)

    @staticmethod
    def backward(ctx, z):
        return _Inverse.cg(ctx.op, z), None

    @staticmethod
    def cg(op, b):
        v, r = torch.zeros_like(b), b.clone()
        p, rr = r.clone(), (b * b).sum()
        stop = 1e-28 * float(rr)
        for k in range(4000):
            if k % 8 == 0 and float(rr) <= stop:
                break
            ap = op(p)
            a = torch.where(rr > 0, rr / (p * ap).sum(), torch.zeros_like(rr))
            v, r = v + a * p, r - a * ap
            new = (r * r).sum()
            p, rr = r + torch.where(rr > 0, new / rr, torch.zeros_like(rr)) * p, new
        return v


def _step(x, quat, length, F, box, differentiable=False):
    """U of one step and its contact count; with `differentiable`, as a
    function of x, quat and F on the active set of the solution."""
    n = x.shape[0]
    mob = _mobility(length, n)
    d = _directors(quat)
    with torch.no_grad():
        pi, pj, w = _pairs(x % box, d, mob[0], box)
        w = w - torch.floor(x[pj] / box) + torch.floor(x[pi] / box)  # x may be unwrapped
        _, e, arm, q = _geometry(x, d, mob, box, pi, pj, w, F)
        gam = _minimise(n, d, mob, pi, pj, e, arm, q)
        if differentiable:
            rate = _gap_rate(d, pi, pj, e, arm, _apply(d, mob, _forces(n, d, pi, pj, e, arm, gam))) + q
            act = torch.nonzero(gam > rate).squeeze(1)
            pi, pj, w, gam = pi[act], pj[act], w[act], gam[act]
            held = (d, e[act], arm[act])
    if differentiable:
        def op(v):
            with torch.no_grad():
                d0, e0, a0 = held
                return _gap_rate(d0, pi, pj, e0, a0, _apply(d0, mob, _forces(n, d0, pi, pj, e0, a0, v)))

        _, e, arm, q = _geometry(x, d, mob, box, pi, pj, w, F)
        rest = _gap_rate(d, pi, pj, e, arm, _apply(d, mob, _forces(n, d, pi, pj, e, arm, gam))) + q
        gam = gam - _Inverse.apply(rest, op)
    return _apply(d, mob, F + _forces(n, d, pi, pj, e, arm, gam)), int(pi.shape[0])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("kinetics", "coupled"):
        return None  # bound states follow from the kinetics' own history
    if kind == "batch":
        Us = [_step(s["x0"], s["quat0"], 1.0, s["F"], s["box"])[0] for s in _batch_systems(case, seed)]
        return {"U": torch.cat(Us)}
    g = _gen(seed)
    if kind == "rollout":
        s = _suspension(g, case["n"], case["phi"], False, False)
        F = _randn(g, case["steps"], case["n"], 6).requires_grad_()
        x0, q0 = s["x0"].requires_grad_(), s["quat0"].requires_grad_()
        x, quat = x0, q0
        for t in range(case["steps"]):
            U, _ = _step(x, quat, s["length"], F[t], s["box"], differentiable=True)
            x, quat = x + DT * U[:, :3], _turn(quat, U)
        gx, gq, gF = torch.autograd.grad((x * x).sum(), (x0, q0, F))
        # on the unit sphere
        gq = gq - (gq * q0).sum(1, keepdim=True) * q0
        return {"x": x.detach(), "quat": quat.detach(), "grad_x": gx, "grad_quat": gq.detach(), "grad_F": gF}
    s = _moved_suspension(g, case) if kind in ("product", "geometry") else \
        _suspension(g, case["n"], case["phi"], case["nematic"], case["mixed_len"])
    n, d, mob = s["n"], _directors(s["quat0"]), _mobility(s["length"], s["n"])
    if kind in ("step", "solve"):
        if n > 100_000:
            return None  # testing every pair and the solve in plain torch take too long
        F = s["F"]
        if case.get("brownian"):
            F = F + _brownian(d, mob, _randn(g, n, 6))
        U, npairs = _step(s["x0"], s["quat0"], s["length"], F, s["box"])
        if kind == "solve":
            return {"U": U}
        x, quat = _integrate(s["x0"], s["quat0"], U, s["box"])
        return {"U": U, "x": x, "quat": quat, "pairs": None}
    pi, pj, w = _pairs(s["x0"], d, mob[0], s["box"])
    phi, e, arm, q = _geometry(s["x0"], d, mob, s["box"], pi, pj, w, s["F"])
    if kind == "geometry":
        return {"dir": d, "pi": None, "pj": None, "img": None, "flags": None, "phi": phi, "e": e, "arm": arm, "q": q}
    gamma = _randn(g, pi.shape[0]).clamp(min=0.0)
    return {"w": _gap_rate(d, pi, pj, e, arm, _apply(d, mob, _forces(n, d, pi, pj, e, arm, gamma))) + q}
