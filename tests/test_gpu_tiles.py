"""Small levels without a march (16 x 8 x 4-cell tiles): sweeps, residual +
restriction and the folded prolongation against the oracle's steps at the
tiles' edges (exactly one tile, one pair more or fewer, two cells in a
direction), with periodic and wall sides, on level 0 (coefficients from rho)
and level 1 (stored), and with outflow sides; tolerance as for the other
single steps (1e-13: a few roundings of O(1) values).  Whole small projections
in FP64 and mixed precision equal the batched ones bit for bit."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1910_12979_amd import inputs as I
from test_gpu_outflow import _step_setup as outflow_setup
from test_gpu_projection import _get, _put, _step_setup, rel

pytestmark = pytest.mark.gpu


def steps(H, OH, levels, rng):
    for l in levels:
        (nx, ny, nz), _ = H.level_info(l)
        phi, f = rng.standard_normal((2, nz, ny, nx))
        for name, a in (("phi", phi), ("f", f)):
            _put(H, l, name, a)
            OH.set(l, name, a)
        H.level_step(l, "down", 2)
        OH.smooth(l, 2)
        OH.resid_restrict(l)
        assert rel(_get(H, l, "phi"), OH.get(l, "phi")) <= 1e-13, l
        assert rel(_get(H, l + 1, "f"), OH.get(l + 1, "f")) <= 1e-13, l
        assert np.all(_get(H, l + 1, "phi") == 0.0)
        e = rng.standard_normal(OH.get(l + 1, "phi").shape)
        _put(H, l + 1, "phi", e)
        OH.set(l + 1, "phi", e)
        H.level_step(l, "up", 1)
        OH.prolong(l)
        OH.smooth(l, 1)
        assert rel(_get(H, l, "phi"), OH.get(l, "phi")) <= 1e-13, l


@pytest.mark.parametrize("n", [(16, 8, 4), (18, 10, 6), (14, 6, 2), (2, 34, 12), (32, 16, 8), (36, 20, 12)])
@pytest.mark.parametrize("per", [(True, True, False), (False, False, False), (True, True, True)])
def test_steps(mp, n, per):
    prob = I.make_problem(n, H=0.2, rho_noise=0.1, seed=61, periodic=per, dx=1 / n[0])
    H, OH = _step_setup(mp, prob)
    steps(H, OH, range(min(2, H.nlevels - 1)), np.random.default_rng(5))


@pytest.mark.parametrize("n", [(16, 8, 4), (18, 10, 6), (36, 20, 12)])
def test_steps_outflow(mp, n):
    prob = I.make_problem(n, H=0.2, rho_noise=0.1, seed=62, periodic=(False,) * 3, outflow=(True,) * 6, dx=1 / n[0])
    H, OH = outflow_setup(mp, prob)
    steps(H, OH, range(min(2, H.nlevels - 1)), np.random.default_rng(6))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_small_solves_equal_batched(mp, precision):
    """Solo solves take the tiles, batches the march for the sweeps and the
    tiles for the operations that write norm rows."""
    probs = [I.make_problem(n, H=0.2, seed=63 + k, dx=1 / n[0], rho_noise=0.05)
             for k, n in enumerate([(32, 32, 32), (48, 48, 48), (64, 48, 32), (96, 48, 48)])]
    params = [mp.params_of(p, precision) for p in probs]
    ds = [mp.to_device(p) for p in probs]
    code, stats = mp.project_batch(params, ds)
    assert code == 0
    for p, pp, d, st in zip(probs, params, ds, stats):
        H = mp.Hierarchy(pp)
        s = mp.to_device(p)
        solo = H.mac_project(s.rho, s.beta0_cc, s.beta0_edge, s.S, s.u, s.v, s.w, s.phi)
        torch.cuda.synchronize()
        for f in ("phi", "u", "v", "w"):
            assert torch.equal(getattr(s, f), getattr(d, f)), (p.n, f)
        assert solo["hist"] == st["hist"]
        H.close()
