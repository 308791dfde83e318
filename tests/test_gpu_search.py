"""The pair search and the records of a step at the edges of their forms: one
workgroup orders up to 4,096 rods in up to 4,096 cells, one workgroup scans up
to 16,384 counts.  A step is compared with its parts, which take the caller's
order: the pairs of the search, the oracle's geometry, the solve of the list.
Both solve to a residual of 1e-10, so the velocities agree to 1e-6."""
import numpy as np
import pytest

import oracle
import rodsynth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _t(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


# (rods, volume fraction, lengths): cells 4,096 and 4,913 at 260 and 320 rods
SYSTEMS = [(1, 1e-3, False), (2, 2e-3, True), (257, 0.02, True), (2048, 0.01, False), (2049, 0.01, True),
           (4096, 0.006, True), (4097, 0.006, False), (16384, 0.004, False), (16385, 0.004, True)]


def _check(gpu_lib, s, L, glen):
    d = oracle.directors(s.quat)
    pr = oracle.pairs(s.x, d, L, s.box, s.diam, s.cutoff)
    cs = oracle.assemble(s.x, d, L, s.box, s.diam, s.eta, s.dt, pr, s.force)
    with gpu_lib.Solver(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt, tol=1e-10) as slv:
        pi, pj, img, fl = slv.build_pairs(_t(s.x), _t(d), glen)
        for got, want in ((pi, pr.pi), (pj, pr.pj), (img, pr.img), (fl, pr.flags)):
            assert np.array_equal(got.cpu().numpy(), want)
        Us = []
        for _ in range(2):
            U, info, n_pairs = slv.step(_t(s.x), _t(s.quat), glen, F=_t(s.force))
            assert info.status == gpu_lib.OK and n_pairs == pr.n
            Us.append(U.cpu().numpy())
        _, U, info = slv.solve_lcp(_t(d), glen, _t(pr.pi, torch.int32), _t(pr.pj, torch.int32), _t(cs.e), _t(cs.arm),
                                   _t(cs.q), F=_t(s.force))
        assert info.status == gpu_lib.OK
    assert np.array_equal(Us[0], Us[1])
    U = U.cpu().numpy()
    assert np.linalg.norm(Us[0] - U) <= 1e-6 * np.linalg.norm(U)


@pytest.mark.parametrize("n,phi,lengths", SYSTEMS)
def test_step_and_its_parts(gpu_lib, n, phi, lengths):
    s = rodsynth.make_system(n, seed=n, phi=phi, length=(0.5, 1.5) if lengths else 1.0)
    L = s.length if lengths else 1.0
    _check(gpu_lib, s, L, _t(L) if lengths else 1.0)


@pytest.mark.parametrize("cells", [16, 17])
def test_many_cells(gpu_lib, cells):
    """300 rods in two clusters of a large box."""
    s = rodsynth.make_system(300, seed=cells, phi=0.02)
    box = cells * (1.0 + s.diam + s.cutoff) * (1.0 + 1e-12)
    x = np.mod(s.x + np.where(np.arange(300) % 2 == 0, 0.3, box - s.box / 2)[:, None], box)
    s = rodsynth.RodSystem(x=x, quat=s.quat, length=s.length, force=s.force, box=box)
    _check(gpu_lib, s, 1.0, 1.0)


@pytest.mark.parametrize("n_pairs", [113, 277, 441])
def test_first_step_of_a_handle_whatever_the_number_of_pairs(gpu_lib, n_pairs):
    """Counts whose lists, rounded up to 256 bytes each, hold different numbers
    of entries: a new handle sizes them on its first step."""
    k = np.arange(n_pairs)
    c = 1.0 + 2.5 * np.stack([k % 8, k // 8 % 8, k // 64], axis=1)
    x = np.concatenate([c, c + [0.0, 0.0, 0.02]])
    quat = np.zeros((2 * n_pairs, 4))
    quat[:, 0] = np.cos(np.pi / 4)
    quat[:n_pairs, 1] = quat[n_pairs:, 2] = np.sin(np.pi / 4)
    with gpu_lib.Solver(box=20.0, diam=rodsynth.DIAM, cutoff=rodsynth.CUTOFF, eta=rodsynth.ETA, dt=rodsynth.DT) as slv:
        _, info, got = slv.step(_t(x), _t(quat), 1.0)
    assert info.status == gpu_lib.OK and got == n_pairs
