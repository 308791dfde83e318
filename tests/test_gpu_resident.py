"""Solves that stay on chip, at the edges of their forms: constraint counts
around the slots of each form, rod counts around the threads, one, two and
four lanes per rod, lists longer than the records a rod holds, one workgroup
and several, contact-only and general sets, and solves longer than one
launch.  Bars as for every
solve: the answer certified by the oracle's operator (residual <= 1e-8), the
velocities within 1e-6 of the oracle's."""
import numpy as np
import pytest

import oracle
import rodsynth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _t(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _problem(n, nc, lengths):
    """n rods and nc of their near pairs (a sorted random choice)."""
    s = rodsynth.make_system(n, seed=n + nc, phi=max(1.3 * nc / (156.0 * n), 0.004),
                             length=(0.5, 1.5) if lengths else 1.0)
    d = oracle.directors(s.quat)
    L = s.length if lengths else 1.0
    pr = oracle.pairs(s.x, d, L, s.box, s.diam, s.cutoff)
    assert pr.n >= nc
    pick = np.sort(np.random.default_rng(nc).choice(pr.n, nc, replace=False))
    pr = oracle.Pairs(pr.pi[pick].copy(), pr.pj[pick].copy(), pr.img[pick].copy(), pr.flags[pick].copy())
    return s, d, L, pr, oracle.assemble(s.x, d, L, s.box, s.diam, s.eta, s.dt, pr, s.force)


# one workgroup: up to 1,023 constraints and 512 rods, 1,535 and 1,024; beyond,
# workgroups that exchange (2 and 3 of them, then up to 64 flat, then teams);
# (60, 450), (200, 1600) and (700, 4000) have lists longer than a rod holds
EDGES = [(30, 1, False), (64, 65, True), (129, 300, False), (512, 1023, True), (513, 1023, False),
         (300, 1024, False), (1024, 1535, False), (1025, 500, True), (1024, 1536, True), (60, 450, False),
         (200, 1600, False), (900, 3072, True), (700, 4000, False), (2049, 3071, False), (6000, 17000, True),
         (40_000, 33_000, False)]


@pytest.mark.parametrize("n,nc,lengths", EDGES)
def test_solve_at_the_edges(gpu_lib, n, nc, lengths):
    s, d, L, pr, cs = _problem(n, nc, lengths)
    ref = oracle.bbpgd(d, L, s.diam, s.eta, pr, cs, tol=1e-8)
    assert ref.status == oracle.OK
    Uref = oracle.velocity(d, L, s.diam, s.eta, pr, cs, ref.gamma, s.force)
    with gpu_lib.Solver(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=1e-8) as slv:
        g, U, info = slv.solve_lcp(_t(d), _t(L) if lengths else L, _t(pr.pi, torch.int32), _t(pr.pj, torch.int32),
                                   _t(cs.e), _t(cs.arm), _t(cs.q), F=_t(s.force))
    g, U = g.cpu().numpy(), U.cpu().numpy()
    assert info.status == gpu_lib.OK and info.residual <= 1e-8
    w = oracle.apply_Mc(d, L, s.diam, s.eta, pr, cs, g)
    cert = np.abs(np.minimum(g, w)).max()
    assert g.min() >= 0 and cert <= 1e-8 * 1.01
    assert info.residual == pytest.approx(cert, abs=1e-11 * np.abs(cs.q).max())
    assert np.linalg.norm(U - Uref) <= 1e-6 * np.linalg.norm(Uref)


@pytest.mark.parametrize("n,nc,lengths", [(40, 60, False), (512, 1023, False), (1000, 2047, True), (5000, 9000, False)])
def test_general_solve_at_the_edges(gpu_lib, n, nc, lengths):
    s, d, L, pr, cs = _problem(n, nc, lengths)
    rng = np.random.default_rng(n)
    kind = (rng.random(nc) < 0.2).astype(np.uint8)          # Hookean rows
    cmp = np.where(kind == 1, rng.uniform(20.0, 60.0, nc), 0.0)
    pj = pr.pj.copy()
    pj[rng.random(nc) < 0.1] = -1                           # against a fixed body
    order = rng.permutation(nc)
    gc = oracle.General(pr.pi[order].copy(), pj[order].copy(), cs.e[order].copy(), cs.arm[order].copy(),
                        cs.q[order].copy(), kind[order].copy(), cmp[order].copy())
    ref = oracle.bbpgd_gen(d, L, s.diam, s.eta, gc, tol=1e-8)
    assert ref.status == oracle.OK
    Uref = oracle.velocity_gen(d, L, s.diam, s.eta, gc, ref.gamma, s.force)
    with gpu_lib.Solver(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=1e-8) as slv:
        g, U, info = slv.solve_general(_t(d), _t(L) if lengths else L, _t(gc.pi, torch.int32),
                                       _t(gc.pj, torch.int32), _t(gc.e), _t(gc.arm), _t(gc.q),
                                       _t(gc.kind, torch.uint8), _t(gc.cmp), F=_t(s.force))
    g, U = g.cpu().numpy(), U.cpu().numpy()
    assert info.status == gpu_lib.OK and info.residual <= 1e-8
    w = oracle.apply_Mc_gen(d, L, s.diam, s.eta, gc, g)
    r = np.where(gc.kind == 1, np.abs(w), np.abs(np.minimum(g, w)))
    assert g[gc.kind == 0].min() >= 0 and r.max() <= 1e-8 * 1.01
    assert np.linalg.norm(U - Uref) <= 1e-6 * np.linalg.norm(Uref)


def test_rod_that_fits_no_workgroup(gpu_lib):
    """One rod in 5,000 constraints: more than any workgroup holds."""
    n, nc = 5001, 5000
    rng = np.random.default_rng(5)
    d, e = rng.normal(size=(n, 3)), rng.normal(size=(nc, 3))
    d, e = d / np.linalg.norm(d, axis=1)[:, None], e / np.linalg.norm(e, axis=1)[:, None]
    kind = (rng.random(nc) < 0.5).astype(np.uint8)
    gc = oracle.General(np.zeros(nc, np.int32), np.arange(1, n, dtype=np.int32), e, rng.uniform(-0.5, 0.5, (nc, 2)),
                        rng.uniform(-1.0, 0.2, nc), kind, np.where(kind == 1, 2000.0, 0.0))
    with gpu_lib.Solver(box=10.0, diam=0.08, cutoff=0.1, eta=1.0, dt=1e-3, tol=1e-8) as slv:
        g, _, info = slv.solve_general(_t(d), 1.0, _t(gc.pi, torch.int32), _t(gc.pj, torch.int32), _t(gc.e),
                                       _t(gc.arm), _t(gc.q), _t(gc.kind, torch.uint8), _t(gc.cmp))
    assert info.status == gpu_lib.OK and info.residual <= 1e-8
    g = g.cpu().numpy()
    w = oracle.apply_Mc_gen(d, 1.0, 0.08, 1.0, gc, g)
    r = np.where(kind == 1, np.abs(w), np.abs(np.minimum(g, w)))
    assert g[kind == 0].min() >= 0 and r.max() <= 1e-8 * 1.01


def test_solve_over_several_launches(gpu_lib):
    """A dense system that needs thousands of iterations (20,683 for the
    oracle): the iteration cap holds exactly on both sides of a launch's end,
    and the solution is certified."""
    s = rodsynth.make_system(300, seed=3, phi=0.05)
    d = oracle.directors(s.quat)
    pr = oracle.pairs(s.x, d, 1.0, s.box, s.diam, s.cutoff)
    cs = oracle.assemble(s.x, d, 1.0, s.box, s.diam, s.eta, s.dt, pr, s.force)
    args = (_t(d), 1.0, _t(pr.pi, torch.int32), _t(pr.pj, torch.int32), _t(cs.e), _t(cs.arm), _t(cs.q))
    for cap in (1, 2047, 2048, 2049, 4097):
        with gpu_lib.Solver(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=0.0,
                            max_iter=cap) as slv:
            _, _, info = slv.solve_lcp(*args)
        assert info.status == gpu_lib.NOT_CONVERGED and info.iterations == cap
    with gpu_lib.Solver(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=1e-8) as slv:
        g, _, info = slv.solve_lcp(*args)
    assert info.status == gpu_lib.OK
    w = oracle.apply_Mc(d, 1.0, s.diam, s.eta, pr, cs, g.cpu().numpy())
    assert np.abs(np.minimum(g.cpu().numpy(), w)).max() <= 1e-8 * 1.01


def _rates(d, L, s, pr, cs, V):
    """D^T V of per-rod velocities."""
    def at(r, arm):
        return V[r, :3] + np.cross(V[r, 3:], arm[:, None] * d[r])
    return np.einsum("ij,ij->i", cs.e, at(pr.pi, cs.arm[:, 0]) - at(pr.pj, cs.arm[:, 1]))


@pytest.mark.parametrize("n,nc,lengths", [e for e in EDGES if e[1] in (1, 1023, 1535, 3071, 4000, 17000, 33000)])
def test_adjoint_at_the_edges(gpu_lib, n, nc, lengths):
    """lambda solves Mc_AA lambda = D_A^T M U_bar by the oracle's operator: the
    recurrence stops at 1e-10, and rounding adds at most as much again."""
    s, d, L, pr, cs = _problem(n, nc, lengths)
    Ub = np.random.default_rng(n).standard_normal((n, 6))
    with gpu_lib.Solver(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=1e-10) as slv:
        args = (_t(d), _t(L) if lengths else L, _t(pr.pi, torch.int32), _t(pr.pj, torch.int32), _t(cs.e), _t(cs.arm),
                _t(cs.q))
        g, _, info = slv.solve_lcp(*args, F=_t(s.force))
        assert info.status == gpu_lib.OK
        qb, _, _, _, _, ai = slv.solve_lcp_adjoint(*args, g, _t(Ub), F=_t(s.force), cg_tol=1e-10)
    assert ai.status == gpu_lib.OK and ai.cg_residual <= 1e-10
    g, lam = g.cpu().numpy(), -qb.cpu().numpy()
    act = g > oracle.apply_Mc(d, L, s.diam, s.eta, pr, cs, g)  # Mc g + q
    b = _rates(d, L, s, pr, cs, oracle.velocity(d, L, s.diam, s.eta, pr, cs, np.zeros(nc), Ub))
    assert ai.n_active == act.sum() and not lam[~act].any()
    r = (b - (oracle.apply_Mc(d, L, s.diam, s.eta, pr, cs, lam) - cs.q))[act]
    assert np.linalg.norm(r) <= 2e-10 * np.linalg.norm(b[act])


def test_adjoint_over_several_launches(gpu_lib):
    """The iteration cap holds exactly on both sides of a launch's end (no
    residual is small enough to stop before)."""
    s = rodsynth.make_system(300, seed=3, phi=0.05)
    d = oracle.directors(s.quat)
    pr = oracle.pairs(s.x, d, 1.0, s.box, s.diam, s.cutoff)
    cs = oracle.assemble(s.x, d, 1.0, s.box, s.diam, s.eta, s.dt, pr, s.force)
    args = (_t(d), 1.0, _t(pr.pi, torch.int32), _t(pr.pj, torch.int32), _t(cs.e), _t(cs.arm), _t(cs.q))
    Ub = np.random.default_rng(0).standard_normal((300, 6))
    with gpu_lib.Solver(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=1e-10) as slv:
        g, _, info = slv.solve_lcp(*args)
        assert info.status == gpu_lib.OK
    for cap in (1, 2047, 2048, 2049):
        with gpu_lib.Solver(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=1e-10,
                            max_iter=cap) as slv:
            *_, ai = slv.solve_lcp_adjoint(*args, g, _t(Ub), cg_tol=1e-300)
        assert ai.status == gpu_lib.NOT_CONVERGED and ai.cg_iterations == cap
