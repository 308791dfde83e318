"""Crosslinkers that gather: the counting by cells at its edges (all in one
cell, in few, more cells than places in a workgroup's table, and not a whole
workgroup of them), crosslinker by crosslinker against the oracle, and the time
of gathered crosslinkers against scattered ones."""
import time

import numpy as np
import pytest

import oracle
import rodsynth
from test_gpu_kmc import _compare, _gpu_step, _kinesin5, _params, _solver, _t

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,spread", [(1, 0.0), (1023, 0.0), (1025, 0.05), (3000, 0.5), (5000, 1.0)])
def test_gathered_crosslinkers(gpu_lib, m, spread):
    s = rodsynth.make_system(150, seed=9, box=12.0)
    d = oracle.directors(s.quat)
    ko, kg = _params(gpu_lib, s.dt, s.diam, **_kinesin5(200.0))
    vbd = oracle.kmc_effective_volume(ko)
    rng = np.random.default_rng(m)
    # about a filament's centre, so that most can bind
    x = np.mod(s.x[0] + (rng.random((m, 3)) - 0.5) * spread * s.box, s.box)
    xl = oracle.Crosslinkers(np.zeros(m, np.int32), np.full((m, 2), -1, np.int32), np.zeros((m, 2)), x)
    events = 0
    with _solver(gpu_lib, s) as slv:
        for step in range(3):
            u, xi = rodsynth.kmc_draws(m, 7, step)
            want = xl.copy()
            wev = oracle.kmc_step(s.x, d, 1.0, s.box, ko, vbd, want, u, xi)
            got, gev, counts = _gpu_step(gpu_lib, slv, s, d, 1.0, kg, xl, u, xi)
            _compare(got, gev, want, wev)
            events += (wev != 0).sum()
            xl = want
    assert m < 1000 or spread > 0.4 or events > 0


def test_gathered_crosslinkers_cost_no_more(gpu_lib):
    """400,000 unbound crosslinkers far from all filaments: in one corner they
    took 1.9 ms longer than all over the box when each was counted by itself."""
    m, box = 400_000, 10.0
    s = rodsynth.make_system(40, seed=3, box=box)
    x = _t(np.mod(s.x, 1.0) + 6.0)
    _, kg = _params(gpu_lib, 1e-4, s.diam, **_kinesin5())
    rng = np.random.default_rng(0)
    u, xi = _t(rng.random((m, 4))), torch.zeros((m, 3), dtype=torch.float64, device="cuda")
    took = []
    with _solver(gpu_lib, s) as slv:
        d = slv.directors(_t(s.quat))
        for width in (0.1, 4.0):
            args = (torch.zeros(m, dtype=torch.int32, device="cuda"),
                    torch.full((m, 2), -1, dtype=torch.int32, device="cuda"),
                    torch.zeros((m, 2), dtype=torch.float64, device="cuda"), _t(rng.random((m, 3)) * width))
            best = np.inf
            for _ in range(8):
                torch.cuda.synchronize()
                t = time.perf_counter()
                slv.kmc_step(x, d, 1.0, kg, *args, u, xi)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t)
            took.append(best)
    assert took[0] <= 1.5 * took[1] + 200e-6
