"""What a solve on chip must leave as it is for the caller: arrays shared
between inputs and outputs, and the bits of a result whatever the handle
solved before."""
import numpy as np
import pytest

import oracle
import rodsynth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _t(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _suspension(n, seed, phi):
    """Arguments of solve_lcp, and of the solver, for a suspension."""
    s = rodsynth.make_system(n, seed=seed, phi=phi)
    d = oracle.directors(s.quat)
    pr = oracle.pairs(s.x, d, 1.0, s.box, s.diam, s.cutoff)
    cs = oracle.assemble(s.x, d, 1.0, s.box, s.diam, s.eta, s.dt, pr, s.force)
    args = (_t(d), 1.0, _t(pr.pi, torch.int32), _t(pr.pj, torch.int32), _t(cs.e), _t(cs.arm), _t(cs.q))
    return args, dict(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=1e-8), _t(s.force)


def _hub(n, seed=5):
    """One rod in n - 1 contacts with the others."""
    nc = n - 1
    rng = np.random.default_rng(seed)
    d, e = rng.normal(size=(n, 3)), rng.normal(size=(nc, 3))
    d, e = d / np.linalg.norm(d, axis=1)[:, None], e / np.linalg.norm(e, axis=1)[:, None]
    args = (_t(d), 1.0, _t(np.zeros(nc), torch.int32), _t(np.arange(1, n), torch.int32), _t(e),
            _t(rng.uniform(-0.5, 0.5, (nc, 2))), _t(rng.uniform(-1.0, 0.2, nc)))
    return args, dict(box=10.0, diam=0.08, cutoff=0.1, eta=1.0, dt=1e-3, tol=1e-8), _t(rng.normal(size=(n, 6)))


@pytest.mark.parametrize("make", [lambda: _suspension(300, 3, 0.05), lambda: _hub(5001)],
                         ids=["several launches", "fits no workgroup"])
def test_velocities_in_the_array_of_the_forces(gpu_lib, make):
    """U may be F's array: the velocities are computed once, from the forces,
    also where a solve takes several launches or leaves the chip."""
    args, prm, F = make()
    with gpu_lib.Solver(**prm) as slv:
        g0, U0, i0 = slv.solve_lcp(*args, F=F)
        V = F.clone()
        g1, U1, i1 = slv.solve_lcp(*args, F=V, U=V)
    assert i0.status == gpu_lib.OK and i1.iterations == i0.iterations
    assert torch.equal(g1, g0) and torch.equal(U1, U0)


def test_results_do_not_depend_on_earlier_calls(gpu_lib):
    """A problem that fits no workgroup sends no other one elsewhere: solution,
    velocities and gradients have the bits of a fresh handle's."""
    args, prm, F = _suspension(2500, 11, 0.02)
    assert args[2].shape[0] >= 1536  # several workgroups
    hub, hprm, hF = _hub(5001)
    Ub = _t(np.random.default_rng(1).standard_normal((2500, 6)))

    def run(slv):
        slv.set_params(**prm)
        g, U, info = slv.solve_lcp(*args, F=F)
        *bars, ai = slv.solve_lcp_adjoint(*args, g, Ub, F=F)
        return (g, U, *bars), (info.iterations, ai.cg_iterations)

    with gpu_lib.Solver(**prm) as slv:
        want, iters = run(slv)
    with gpu_lib.Solver(**hprm) as slv:
        h0, V0, _ = slv.solve_lcp(*hub, F=hF)
        got, again = run(slv)
        slv.set_params(**hprm)
        h1, V1, _ = slv.solve_lcp(*hub, F=hF)
    assert again == iters and all(torch.equal(a, b) for a, b in zip(got, want))
    assert torch.equal(h0, h1) and torch.equal(V0, V1)


def test_no_memory_for_the_exchange(gpu_lib):
    """A problem that fitted without the exchange words still does."""
    args, prm, F = _suspension(2500, 11, 0.02)
    want = _two_kernels(gpu_lib, prm, lambda slv: slv.solve_lcp(*args, F=F))
    with gpu_lib.Solver(**prm) as slv:
        slv.onchip_control(refuse=1)
        got = slv.solve_lcp(*args, F=F)
        assert slv.onchip_read()["refused"] == 1 and slv.onchip_read()["groups"] == 0
        slv.onchip_control()
        slv.solve_lcp(*args, F=F)
        assert slv.onchip_read()["solves"] == 1
    assert got[2] == want[2] and torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def _two_kernels(gpu_lib, prm, solve):
    with gpu_lib.Solver(**prm) as slv:
        slv.onchip_control(refuse=2)
        return solve(slv)


@pytest.mark.parametrize("phi,after,general", [
    (0.04, 0, False), (0.04, 1, False), (0.04, 20, True), (0.04, "last", False), (0.04, "last", True),
    (0.05, 2056 + 5, False)])
def test_wait_that_runs_out(gpu_lib, phi, after, general):
    """Without patience from an exchange on (the last one, when some workgroups
    have left their results already, and one in a second launch among them) the
    two kernels solve from the caller's start and give the bits they give alone."""
    args, prm, F = _suspension(1500, 12, phi)
    if after == 2056 + 5:
        prm.update(tol=0.0, max_iter=3000)  # two launches
    nc = args[2].shape[0]
    start = _t(np.random.default_rng(3).uniform(-0.2, 1.0, nc))
    rng = np.random.default_rng(4)
    kind = _t(rng.random(nc) < 0.2, torch.uint8)
    pj = args[3].clone()
    pj[_t(rng.random(nc) < 0.1, torch.bool)] = -1

    def solve(slv):
        if general:
            return slv.solve_general(args[0], args[1], args[2], pj, *args[4:], kind, kind.double() * 40.0, F=F,
                                     gamma=start.clone())
        return slv.solve_lcp(*args, F=F, gamma=start.clone())

    g0, U0, i0 = _two_kernels(gpu_lib, prm, solve)
    with gpu_lib.Solver(**prm) as slv:
        slv.onchip_control(form=2, groups=64, lanes=2)
        _, _, info = solve(slv)
        assert slv.onchip_read()["solves"] == 1
        # exchanges: whether it fits, the start's two products, the iterations, the end
        last = 4 + info.iterations
        assert info.iterations == 3000 if after == 2056 + 5 else info.iterations <= 2048
        slv.onchip_control(form=2, groups=64, lanes=2, patient=last - 1 if after == "last" else after)
        g1, U1, i1 = solve(slv)
        ran = slv.onchip_read()
    assert ran["timeouts"] == 1 and ran["solves"] == 1
    assert i1.iterations == i0.iterations and torch.equal(g1, g0) and torch.equal(U1, U0)


def test_noalloc_is_solve_lcp_when_sampled(gpu_lib):
    """Kernel sampling takes the two-kernel loop: in both calls."""
    args, prm, F = _suspension(2500, 11, 0.02)
    with gpu_lib.Solver(**prm) as slv:
        slv.profile_enable(8)
        g0, U0, i0 = slv.solve_lcp(*args, F=F)
        taken = slv.profile_read()
        g1, U1 = torch.zeros_like(g0), torch.empty_like(U0)
        g1, U1, i1 = slv.solve_lcp_noalloc(*args, g1, U1, F=F)
        assert taken["rod_launches"] > 0 and slv.profile_read()["rod_launches"] == 0
    assert i0 == i1 and torch.equal(g0, g1) and torch.equal(U0, U1)


@pytest.mark.parametrize("n,phi,lengths", [(700, 0.02, False), (6000, 0.02, True), (20_000, 0.03, False)])
def test_reserved_sizes_allocate_nothing(gpu_lib, n, phi, lengths):
    """After rl_reserve the first search, steps (plain, warm-started, with the
    stress, with noise) and solve of that size take no workspace."""
    s = rodsynth.make_system(n, seed=6, phi=phi, length=(0.5, 1.5) if lengths else 1.0)
    L = _t(s.length) if lengths else 1.0
    quat, F = _t(s.quat), _t(s.force)
    prm = dict(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=1e-8, max_iter=50)
    with gpu_lib.Solver(**prm) as slv:
        dirs = slv.directors(quat)
        pi, pj, img, _ = slv.build_pairs(_t(s.x), dirs, L)
        most = pi.shape[0]
        _, e, arm, q = slv.assemble_D(_t(s.x), dirs, L, pi, pj, img, F)
    calls = {
        "search": lambda slv: slv.build_pairs(_t(s.x), dirs, L, capacity=most),
        "step": lambda slv: slv.step(_t(s.x), quat.clone(), L, F=F),
        "warm step": lambda slv: slv.step(_t(s.x), quat.clone(), L, F=F, warm_start=True),
        "step with stress": lambda slv: slv.step(_t(s.x), quat.clone(), L, F=F, stress=True),
        "step with noise": lambda slv: slv.step(_t(s.x), quat.clone(), L, F=F, kT=0.004,
                                                noise=torch.ones((n, 6), dtype=torch.float64, device="cuda")),
        "solve": lambda slv: slv.solve_lcp(dirs, L, pi, pj, e, arm, q, F=F),
    }
    for name, call in calls.items():
        with gpu_lib.Solver(**prm) as slv:
            slv.reserve(n, most)
            before = slv.onchip_read()["allocations"]
            call(slv)
            assert slv.onchip_read()["allocations"] == before, name


@pytest.mark.parametrize("n,nc,hub,longest,groups", [
    (400, 900, 36, 36, 1), (400, 900, 37, 36, 1), (1000, 1400, 400, 36, 1), (100, 900, 99, 1 << 30, 1),
    (2000, 3000, 76, 76, 12), (2000, 3000, 77, 76, 12), (10_000, 20_000, 500, 76, 64)])
def test_rod_with_many_contacts(gpu_lib, n, nc, hub, longest, groups):
    """A rod in so many contacts that its lanes would hold all others up goes to
    the two kernels; shorter lists stay on chip, whatever else the handle ran."""
    rng = np.random.default_rng(n + hub)
    pi = np.concatenate([np.zeros(hub, int), np.tile(np.arange(1, n // 2), nc)[:nc - hub]])
    pj = np.concatenate([1 + rng.permutation(n - 1)[:hub], rng.integers(n // 2, n, nc - hub)])
    order = np.argsort(pi, kind="stable")
    pi, pj = pi[order], pj[order]
    d, e = rng.normal(size=(n, 3)), rng.normal(size=(nc, 3))
    d, e = d / np.linalg.norm(d, axis=1)[:, None], e / np.linalg.norm(e, axis=1)[:, None]
    arm, q = rng.uniform(-0.5, 0.5, (nc, 2)), rng.uniform(-1.0, 0.2, nc)
    lists = np.bincount(pi, minlength=n) + np.bincount(pj, minlength=n)
    assert lists[0] == hub and (hub > longest or lists.max() <= longest)
    with gpu_lib.Solver(box=10.0, diam=0.08, cutoff=0.1, eta=1.0, dt=1e-3, tol=0.0, max_iter=20) as slv:
        args = (_t(d), 1.0, _t(pi, torch.int32), _t(pj, torch.int32), _t(e), _t(arm), _t(q))
        slv.solve_lcp(*args)
        ran = slv.onchip_read()
        assert ran["groups"] == (groups if hub <= longest else 0) and ran["misfits"] == (hub > longest)
        g, U, _ = slv.solve_lcp(*args)
        slv.onchip_control(refuse=2)
        g2, U2, _ = slv.solve_lcp(*args)
    # 20 iterations of the same method
    assert torch.linalg.norm(U - U2) <= 1e-9 * torch.linalg.norm(U2)


@pytest.mark.parametrize("nc,chip,cg_chip", [(180_000, True, True), (200_000, False, True), (260_000, False, False)])
def test_unordered_lists_leave_the_chip_where_memory_is_faster(gpu_lib, nc, chip, cg_chip):
    n, rng = 60_000, np.random.default_rng(2)
    a, b = rng.integers(0, n, nc), rng.integers(0, n - 1, nc)
    b += b >= a
    pi, pj = np.minimum(a, b), np.maximum(a, b)
    order = np.argsort(pi, kind="stable")
    pi, pj = pi[order], pj[order]
    d, e = rng.normal(size=(n, 3)), rng.normal(size=(nc, 3))
    d, e = d / np.linalg.norm(d, axis=1)[:, None], e / np.linalg.norm(e, axis=1)[:, None]
    args = (_t(d), 1.0, _t(pi, torch.int32), _t(pj, torch.int32), _t(e), _t(rng.uniform(-0.5, 0.5, (nc, 2))),
            _t(rng.uniform(-1.0, 0.2, nc)))
    Ub = _t(rng.normal(size=(n, 6)))
    with gpu_lib.Solver(box=10.0, diam=0.08, cutoff=0.1, eta=1.0, dt=1e-3, tol=0.0, max_iter=20) as slv:
        g, U, _ = slv.solve_lcp(*args)
        assert (slv.onchip_read()["groups"] > 0) == chip
        bars = slv.solve_lcp_adjoint(*args, g, Ub, cg_tol=1e-300)[:5]
        assert (slv.onchip_read()["groups"] > 0) == cg_chip
        slv.onchip_control(refuse=2)
        _, U2, _ = slv.solve_lcp(*args)
        bars2 = slv.solve_lcp_adjoint(*args, g, Ub, cg_tol=1e-300)[:5]
    # 20 iterations of the same methods
    for a, b in zip((U, *bars), (U2, *bars2)):
        assert torch.linalg.norm(a - b) <= 1e-9 * torch.linalg.norm(b)


def test_reserve_between_warm_steps(gpu_lib):
    """rl_reserve leaves the forces of the last step where the next one finds
    them: repeated with the same loads it stops at once."""
    s = rodsynth.make_system(700, seed=6, phi=0.02)
    F = _t(s.force)
    with gpu_lib.Solver(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=1e-8) as slv:
        x, quat = _t(s.x), _t(s.quat)
        _, first, n_pairs = slv.step(x.clone(), quat.clone(), 1.0, F=F, warm_start=True)
        slv.reserve(70_000, 100 * n_pairs)
        _, again, _ = slv.step(x.clone(), quat.clone(), 1.0, F=F, warm_start=True)
    assert first.iterations > 10 and again.iterations == 0
