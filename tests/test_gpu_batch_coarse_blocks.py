"""Batches whose coarsest levels have more unknowns than one workgroup inverts
(128): they are inverted block by block, all problems in the same launches,
whatever their sizes, and give the single problem's bits."""
import pytest
import torch

from paper_1910_12979_amd import inputs as I

pytestmark = pytest.mark.gpu

# coarsest 6x7x5 = 210, 7^3 = 343, 17 x 10 x 3 = 510, 4^3 (one workgroup), 12 x 11 x 1 = 132
SHAPES = [(48, 56, 40), (56, 56, 56), (68, 40, 12), (32, 32, 32), (96, 88, 8)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batch_equals_solo(mp, precision):
    probs = [I.make_problem(n, H=0.3, rho_noise=0.05, seed=70 + k, dx=1 / n[0]) for k, n in enumerate(SHAPES)]
    pars = [mp.params_of(p, precision=precision) for p in probs]
    solo = []
    for p, par in zip(probs, pars):
        d = mp.to_device(p)
        H = mp.Hierarchy(par)
        solo.append((H.mac_project(d.rho, d.beta0_cc, d.beta0_edge, d.S, d.u, d.v, d.w, d.phi), d))
        H.close()
    pick = [0, 1, 2, 3, 4, 1, 0, 2]
    ds = [mp.to_device(probs[k]) for k in pick]
    code, stats = mp.project_batch([pars[k] for k in pick], ds)
    assert code == 0
    for k, d, st in zip(pick, ds, stats):
        assert st["hist"] == solo[k][0]["hist"], SHAPES[k]
        assert all(torch.equal(getattr(d, f), getattr(solo[k][1], f)) for f in ("phi", "u", "v", "w")), SHAPES[k]
