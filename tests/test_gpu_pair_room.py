"""Workspace of the pair search: it follows the pairs there are, not the room
that the caller has for them."""
import numpy as np
import pytest

import oracle
import rodsynth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _t(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _same(got, pr):
    for a, b in zip(got, (pr.pi, pr.pj, pr.img, pr.flags)):
        assert np.array_equal(a.cpu().numpy(), b)


def test_room_for_many_more_pairs(gpu_lib):
    """9 bytes of workspace per unit of capacity were enough once (and a
    quarter more for growth): 20 million units for some 400 pairs."""
    s = rodsynth.make_system(400, seed=7, box=3.0)
    d = oracle.directors(s.quat)
    pr = oracle.pairs(s.x, d, 1.0, s.box, s.diam, s.cutoff)
    x, dirs, capacity = _t(s.x), _t(d), 20_000_000
    warm = [torch.empty(capacity, dtype=t, device="cuda") for t in (torch.int32,) * 3 + (torch.uint8,)]
    del warm  # (stays with torch)
    with gpu_lib.Solver(box=s.box, diam=s.diam, cutoff=s.cutoff, eta=s.eta, dt=s.dt) as slv:
        free = torch.cuda.mem_get_info()[0]
        got = slv.build_pairs(x, dirs, 1.0, capacity=capacity)
        used = free - torch.cuda.mem_get_info()[0]
    _same(got, pr)
    assert used <= 1.25 * 9 * capacity


@pytest.mark.parametrize("capacity", [0, 11_174, 11_175, 20_000])
def test_more_pairs_than_expected(gpu_lib, capacity):
    """150 rods that all meet: 11,175 pairs, 74 per rod, where the search
    expects 8,896 at most; fewer, then more again."""
    rng = np.random.default_rng(3)
    x = 5.0 + rng.uniform(-0.1, 0.1, (150, 3))
    d = rng.standard_normal((150, 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    pr = oracle.pairs(x, d, 1.0, 10.0, 0.025, 0.5)
    assert pr.n == 150 * 149 // 2
    with gpu_lib.Solver(box=10.0, diam=0.025, cutoff=0.5, eta=0.01, dt=1e-4) as slv:
        if capacity < pr.n:
            with pytest.raises(gpu_lib.RodLCPError) as ei:
                gpu_lib.Solver.build_pairs(slv, _t(x), _t(d), 1.0, capacity=capacity)
            assert ei.value.status == gpu_lib.ERR_CAPACITY
        for keep in (150, 40, 150):
            sub = oracle.pairs(x[:keep], d[:keep], 1.0, 10.0, 0.025, 0.5)
            _same(slv.build_pairs(_t(x[:keep]), _t(d[:keep]), 1.0, capacity=max(capacity, pr.n)), sub)
