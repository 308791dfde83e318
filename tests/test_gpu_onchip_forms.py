"""Every form of a solve on chip runs the solves it is asked for: with its slots
full to the last one, one too many (the next form takes over, or the two
kernels past the last), for contacts, general sets and the adjoint's conjugate
gradients, and between 2 and 256 workgroups.  Also what a handle does
without room on the device, and two handles at once.  Bars as for every solve:
the answer certified by the oracle's operator (residual <= 1e-8, 2e-10 of the
right-hand side for the conjugate gradients)."""
import threading

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SLOTS = (1024, 1536, 2048, 2560, 3072)
PRM = dict(box=10.0, diam=0.08, cutoff=0.1, eta=1.0, dt=1e-3)


def _t(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _pairs(pi, pj):
    return oracle.Pairs(pi, pj, np.full(len(pi), 0x888, np.int32), np.zeros(len(pi), np.uint8))


class Problem:
    """Two halves of `half` rods, alike in their lists, with `within` constraints
    in each and `cross` from the first to the second: two workgroups take a half
    each and need within + cross slots.  q belongs to a known solution."""

    def __init__(self, half, within, cross, general, seed=0):
        rng = np.random.default_rng(seed)
        a, b = rng.integers(0, half, within), rng.integers(0, half - 1, within)
        b += b >= a
        lo, hi = np.minimum(a, b), np.maximum(a, b)
        fixed = rng.random(within) < (0.1 if general else 0.0)
        soft = rng.random(within) < (0.2 if general else 0.0)
        hi = np.where(fixed, -1, hi)
        c0, c1 = rng.integers(0, half, cross), rng.integers(half, 2 * half, cross)
        # (the halves weigh the same where a rod's P and Q records do)
        pi = np.concatenate([lo, lo + half, c0])
        pj = np.concatenate([hi, np.where(hi < 0, -1, hi + half), c1])
        self.kind = np.concatenate([soft, soft, np.zeros(cross, bool)]).astype(np.uint8)
        order = np.argsort(pi, kind="stable")
        self.pi, self.pj = pi[order].astype(np.int32), pj[order].astype(np.int32)
        self.kind, nc = self.kind[order], len(pi)
        unit = lambda m: (lambda v: v / np.linalg.norm(v, axis=1)[:, None])(rng.standard_normal((m, 3)))
        self.n, self.nc, self.general = 2 * half, nc, general
        self.d, self.e, self.arm = unit(2 * half), unit(nc), rng.uniform(-0.5, 0.5, (nc, 2))
        self.cmp = np.where(self.kind == 1, rng.uniform(0.5, 2.0, nc), 0.0)
        self.q = np.zeros(nc)
        pushes = rng.random(nc) < 0.3
        g = np.where(self.kind == 1, rng.uniform(-1.0, 1.0, nc), np.where(pushes, rng.uniform(0.1, 1.0, nc), 0.0))
        self.q = np.where((self.kind == 1) | pushes, 0.0, rng.uniform(0.1, 1.0, nc)) - self.rate(g)

    def rate(self, g):
        """Mc g + q."""
        if self.general:
            gc = oracle.General(self.pi, self.pj, self.e, self.arm, self.q, self.kind, self.cmp)
            return oracle.apply_Mc_gen(self.d, 1.0, PRM["diam"], PRM["eta"], gc, g)
        cs = oracle.Constraints(np.zeros(self.nc), self.e, self.arm, self.q)
        return oracle.apply_Mc(self.d, 1.0, PRM["diam"], PRM["eta"], _pairs(self.pi, self.pj), cs, g)

    def solve(self, slv):
        args = (_t(self.d), 1.0, _t(self.pi, torch.int32), _t(self.pj, torch.int32), _t(self.e), _t(self.arm),
                _t(self.q))
        if self.general:
            return slv.solve_general(*args, _t(self.kind, torch.uint8), _t(self.cmp))
        return slv.solve_lcp(*args)

    def certify(self, lib, g, info, tol=1e-8):
        assert info.status == lib.OK and info.residual <= tol
        g = g.cpu().numpy()
        w = self.rate(g)
        r = np.where(self.kind == 1, np.abs(w), np.abs(np.minimum(g, w)))
        assert g[self.kind == 0].min() >= 0 and r.max() <= 1.01 * tol

    def adjoint(self, lib, slv, g):
        args = (_t(self.d), 1.0, _t(self.pi, torch.int32), _t(self.pj, torch.int32), _t(self.e), _t(self.arm),
                _t(self.q))
        Ub = np.random.default_rng(1).standard_normal((self.n, 6))
        qb, _, _, _, _, ai = slv.solve_lcp_adjoint(*args, g, _t(Ub), cg_tol=1e-10)
        assert ai.status == lib.OK and ai.cg_residual <= 1e-10
        g, lam = g.cpu().numpy(), -qb.cpu().numpy()
        act = g > self.rate(g)
        assert ai.n_active == act.sum() and not lam[~act].any()
        cs = oracle.Constraints(np.zeros(self.nc), self.e, self.arm, self.q)
        V = oracle.velocity(self.d, 1.0, PRM["diam"], PRM["eta"], _pairs(self.pi, self.pj), cs, np.zeros(self.nc), Ub)
        at = lambda r, s: V[r, :3] + np.cross(V[r, 3:], s[:, None] * self.d[r])
        b = np.einsum("ij,ij->i", self.e, at(self.pi, self.arm[:, 0]) - at(self.pj, self.arm[:, 1]))
        r = (b - (self.rate(lam) - self.q))[act]
        assert np.linalg.norm(r) <= 2e-10 * np.linalg.norm(b[act])
        return lam


@pytest.mark.parametrize("general", [False, True], ids=["contacts", "general"])
@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("form", range(5))
def test_form_full_and_one_over(gpu_lib, form, over, general):
    lanes = (4, 2, 1, 1, 1)[form]
    p = Problem(480 // lanes, SLOTS[form] - 101 + over, 100, general, seed=form)
    with gpu_lib.Solver(tol=1e-8, **PRM) as slv:
        slv.onchip_control(form=form, groups=2, lanes=lanes)
        g, _, info = p.solve(slv)
        ran = slv.onchip_read()
        last = over and form == 4
        assert ran["solves"] == (0 if last else 1) and ran["misfits"] == over and ran["timeouts"] == 0
        assert (ran["groups"], ran["lanes"]) == ((0, lanes) if last else (2, lanes))
        assert last or ran["form"] == form + over
        p.certify(gpu_lib, g, info)
        if not general:
            p.adjoint(gpu_lib, slv, g)
            ran = slv.onchip_read()
            assert ran["solves"] == (0 if last else 2) and ran["misfits"] == 2 * over


@pytest.mark.parametrize("form,groups", [(0, 3), (1, 16), (0, 64), (0, 65), (2, 128), (0, 129), (0, 255), (3, 256), (4, 256)])
def test_number_of_workgroups(gpu_lib, form, groups):
    p = Problem(300, 700, 60, False, seed=groups)
    with gpu_lib.Solver(tol=1e-8, **PRM) as slv:
        slv.onchip_control(form=form, groups=groups, lanes=2 if groups > 2 else 1)
        g, _, info = p.solve(slv)
        p.certify(gpu_lib, g, info)
        p.adjoint(gpu_lib, slv, g)
        ran = slv.onchip_read()
    assert ran["solves"] == 2 and ran["groups"] == groups and ran["form"] == form


def test_no_room_on_the_device(gpu_lib):
    """The launch is refused: the two kernels solve, each time the same."""
    p = Problem(300, 800, 60, False)
    with gpu_lib.Solver(tol=1e-8, **PRM) as slv:
        g0, U0, _ = p.solve(slv)
        assert slv.onchip_read()["solves"] == 1
        slv.onchip_control(refuse=2)
        g1, U1, info = p.solve(slv)
        p.certify(gpu_lib, g1, info)
        lam = p.adjoint(gpu_lib, slv, g1)
        assert slv.onchip_read()["refused"] == 2 and slv.onchip_read()["groups"] == 0
        g2, U2, _ = p.solve(slv)
        assert torch.equal(g1, g2) and torch.equal(U1, U2)
        slv.onchip_control()
        g3, U3, _ = p.solve(slv)
        assert torch.equal(g0, g3) and torch.equal(U0, U3)
        ref = p.adjoint(gpu_lib, slv, g1)
        assert np.linalg.norm(lam - ref) <= 1e-6 * np.linalg.norm(ref)


def test_two_handles_at_once(gpu_lib):
    """Solves of two handles, on a stream and a thread each: the workgroups of
    both cannot all be on the device together, and both come to their results."""
    probs = [Problem(600, 1500, 100, False, seed=s) for s in (1, 2)]
    want, got = [None, None], [[], []]

    def run(k, times, out):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream), gpu_lib.Solver(tol=1e-8, **PRM) as slv:
            slv.onchip_control(form=4, groups=256, lanes=2)
            for _ in range(times):
                g, _, info = probs[k].solve(slv)
                out.append((g.cpu(), info, slv.onchip_read()["timeouts"]))

    for k in (0, 1):
        first = []
        run(k, 1, first)
        want[k] = first[0][0]
    threads = [threading.Thread(target=run, args=(k, 10, got[k])) for k in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in (0, 1):
        assert len(got[k]) == 10
        for g, info, timeouts in got[k]:
            probs[k].certify(gpu_lib, g, info)
            assert timeouts > 0 or torch.equal(g, want[k])
