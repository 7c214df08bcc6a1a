"""A projection whose phi output is laid over its rho (a caller done with rho
gives its memory away) gives the bits of one with a buffer of its own: the
correction reads rho of a cell's neighbours while their phi is written."""
import numpy as np
import pytest
import torch

from paper_1910_12979_amd import inputs as I

pytestmark = pytest.mark.gpu


def shifted(t, by):
    """A copy of t, `by` doubles behind a 256-byte boundary."""
    flat = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)
    out = flat[by:].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("by", [0, 1])
@pytest.mark.parametrize("how,precision", [("mac", "fp64"), ("mac", "mixed"), ("static", "fp64"), ("batch", "fp64"),
                                           ("batch", "mixed"), ("star", "fp64")])
def test_phi_over_rho(mp, how, precision, by):
    n = (64, 48, 32)
    prob = I.make_star_problem(n, Hr=0.3, rho_noise=0.05, seed=3) if how == "star" else \
        I.make_problem(n, H=0.2, rho_noise=0.05, seed=3)
    par = mp.params_of(prob, precision=precision)
    res = []
    for over in (False, True):
        d = mp.to_device(prob)
        d.rho = shifted(d.rho, by)
        if over:
            d.phi = d.rho
        if how == "static":
            mp.mac_project_static(par, d.rho, d.beta0_cc, d.beta0_edge, d.S, d.u, d.v, d.w, d.phi)
        elif how == "batch":
            other = mp.to_device(prob)
            code, _ = mp.project_batch([par, par], [d, other])
            assert code == 0
        else:
            H = mp.Hierarchy(par)
            if how == "star":
                H.mac_project_radial(d.rho, d.beta0_r, prob.dr_base, prob.centre, d.S, d.u, d.v, d.w, d.phi)
            else:
                H.mac_project(d.rho, d.beta0_cc, d.beta0_edge, d.S, d.u, d.v, d.w, d.phi)
            H.close()
        torch.cuda.synchronize()
        res.append([getattr(d, k).cpu().numpy() for k in ("phi", "u", "v", "w")])
    for a, b in zip(*res):
        assert np.array_equal(a, b)
