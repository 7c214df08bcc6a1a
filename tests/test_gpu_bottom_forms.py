"""The one-workgroup bottom of the V-cycle in each of its forms gives the bits
of the per-level launches (equal expressions in equal order, so no tolerance):
1, 2 or 4 cells of each colour per thread at their edges, one or two smoothed
levels, sizes that are no powers of two, a level that the fused sweep would
take too (another FP32 division), the wide form above 4096 cells, outflow
sides; and the nodal bottom with one or two smoothed levels, walls and
periodic sides."""
import numpy as np
import pytest
import torch

from paper_1910_12979_amd import inputs as I

pytestmark = pytest.mark.gpu


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def mac(mp, prob, precision, bottom):
    H = mp.Hierarchy(mp.params_of(prob, precision))
    H.set_bottom(bottom)
    d = mp.to_device(prob)
    if prob.beta0_r is not None:
        st = H.mac_project_radial(d.rho, d.beta0_r, prob.dr_base, prob.centre, d.S, d.u, d.v, d.w, d.phi)
    else:
        st = H.mac_project(d.rho, d.beta0_cc, d.beta0_edge, d.S, d.u, d.v, d.w, d.phi)
    out = [t.cpu().numpy() for t in (d.phi, d.u, d.v, d.w)]
    H.close()
    return st["hist"], out


@pytest.mark.parametrize("n", [(16, 16, 16),      # 8^3: 1 cell of each colour, the coarsest right below
                               (20, 16, 24),      # 10 x 8 x 12 = 960, then 5 x 4 x 6
                               (28, 12, 20),      # 14 x 6 x 10, then 7 x 3 x 5
                               (32, 16, 32),      # 16 x 8 x 16 = 2048: 2 cells, two smoothed levels
                               (48, 32, 32),      # 24 x 16 x 16 = 6144: the wide form
                               (24, 40, 32),      # 12 x 20 x 16 = 3840: 4 cells
                               (32, 32, 32),      # 16^3 = 4096: the largest
                               (128, 32, 32),     # 32 x 8 x 8, which the fused sweep covers
                               (40, 24, 56)])     # 20 x 12 x 28: wide, 10 x 6 x 14 below it
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_bottom_forms(mp, n, precision):
    prob = I.make_problem(n, H=0.2, rho_noise=0.05, seed=51, periodic=(True, False, False), dx=1 / n[0])
    h0, a = mac(mp, prob, precision, True)
    h1, b = mac(mp, prob, precision, False)
    assert h0 == h1 and same(a, b)


@pytest.mark.parametrize("n", [(16, 16, 16), (24, 24, 24), (32, 32, 32)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_bottom_forms_outflow(mp, n, precision):
    prob = I.make_star_problem(n, Hr=0.3, rho_noise=0.05, seed=52)
    h0, a = mac(mp, prob, precision, True)
    h1, b = mac(mp, prob, precision, False)
    assert h0 == h1 and same(a, b)


@pytest.mark.parametrize("n", [(16, 16, 16), (20, 12, 28), (24, 40, 32), (32, 32, 32), (48, 32, 40)])
@pytest.mark.parametrize("per", [(True, True, False), (False, False, False), (True, True, True)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_nodal_bottom_forms(mp, n, per, precision):
    prob = I.make_nodal_problem(n, H=0.3, rho_noise=0.05, seed=53, periodic=per)
    res = []
    for bottom in (True, False):
        H = mp.NodalHierarchy(mp.make_params(prob.n, prob.dx, prob.periodic, precision=precision))
        H.set_bottom(bottom)
        d = mp.nodal_to_device(prob)
        st = H.project(d.rho, d.beta0_cc, d.S, d.uc, d.vc, d.wc, d.phi)
        res.append((st["hist"], [t.cpu().numpy() for t in (d.phi, d.uc, d.vc, d.wc)]))
        H.close()
    assert res[0][0] == res[1][0] and same(res[0][1], res[1][1])
