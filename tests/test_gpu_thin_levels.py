"""Levels that neither the march (fewer than 32 cells in x) nor the marchless
tiles (more than 2^20 cells, or more tiles than there are partial rows) take:
they run one kernel per colour, a residual + restriction per coarse cell and a
prolongation of their own.  Thin boxes have such levels, as the finest one or
below it, alone and in a batch."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1910_12979_amd import inputs as I

pytestmark = pytest.mark.gpu

THIN = (16, 256, 272)            # 2176 tiles
ABOVE = (32, 512, 544)           # a finest level that marches, over a thin one


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - b) / np.linalg.norm(b))


@pytest.mark.parametrize("per", [(True, True, False), (False, False, True)])
def test_steps(mp, per):
    """One step against the oracle's, to 1e-13: the same sums in the same order."""
    nx, ny, nz = THIN
    prob = I.make_problem(THIN, H=0.5, rho_noise=0.05, seed=61, periodic=per, dx=1 / nx)
    c = O.face_coeffs(THIN, per, prob.rho, prob.beta0_cc, prob.beta0_edge)
    rng = np.random.default_rng(62)
    phi, f = rng.standard_normal((nz, ny, nx)), rng.standard_normal((nz, ny, nx))
    d = mp.to_device(prob)
    H = mp.Hierarchy(mp.params_of(prob))
    assert H.sweep_config(0) is None
    H.set_coefficients(d.rho, d.beta0_cc, d.beta0_edge)

    def put(level, name, a):
        H.level_copy(level, name, torch.from_numpy(np.ascontiguousarray(a)).cuda(), True)

    def get(level, name):
        (mx, my, mz), _ = H.level_info(level)
        t = torch.empty((mz, my, mx), dtype=torch.float64, device="cuda")
        H.level_copy(level, name, t, False)
        torch.cuda.synchronize()
        return t.cpu().numpy()

    put(0, "phi", phi)
    put(0, "f", f)
    H.level_step(0, "smooth", 2)
    got = get(0, "phi")
    assert rel(got, O.rbgs(THIN, per, prob.dx, c, phi, f, 2)) <= 1e-13
    H.level_step(0, "resid_restrict")
    r = O.residual(THIN, per, prob.dx, c, got, f)
    assert rel(get(1, "f"), r.reshape(nz // 2, 2, ny // 2, 2, nx // 2, 2).mean((1, 3, 5))) <= 1e-13
    assert np.all(get(1, "phi") == 0.0)
    e = rng.standard_normal((nz // 2, ny // 2, nx // 2))
    put(1, "phi", e)
    H.level_step(0, "prolong")
    assert rel(get(0, "phi"), got + e.repeat(2, 0).repeat(2, 1).repeat(2, 2)) <= 1e-15
    H.close()


@pytest.mark.parametrize("n,precision", [(THIN, "fp64"), (THIN, "mixed"), (ABOVE, "fp64"), (ABOVE, "mixed")])
def test_solves_alone_and_in_a_batch(mp, n, precision):
    prob = I.make_problem(n, H=0.5, rho_noise=0.05, seed=63, dx=1 / n[0], rtol=1e-9)
    par = mp.params_of(prob, precision=precision)
    d = mp.to_device(prob)
    H = mp.Hierarchy(par)
    assert (H.sweep_config(0) is None) == (n == THIN)
    assert n == THIN or H.sweep_config(1) is None
    st = H.mac_project(d.rho, d.beta0_cc, d.beta0_edge, d.S, d.u, d.v, d.w, d.phi)
    H.close()
    assert st["status_name"] == "OK" and st["rel_resid"] <= prob.rtol
    phi = d.phi.cpu().numpy()
    c = O.face_coeffs(n, prob.periodic, prob.rho, prob.beta0_cc, prob.beta0_edge)
    f = O.rhs(n, prob.periodic, prob.dx, prob.beta0_cc, prob.beta0_edge, prob.u, prob.v, prob.w, prob.S)
    f -= f.mean()
    r = O.residual(n, prob.periodic, prob.dx, c, phi, f)
    assert np.linalg.norm(r) <= 1.05 * prob.rtol * np.linalg.norm(f)
    for got, want in zip((d.u, d.v, d.w), O.correct(n, prob.periodic, prob.dx, prob.beta0_cc, prob.beta0_edge, c, phi,
                                                    prob.u, prob.v, prob.w)):
        assert rel(got.cpu().numpy(), want) <= 1e-12
    ds = [mp.to_device(prob) for _ in range(2)]
    code, stats = mp.project_batch([par, par], ds)
    assert code == 0
    for t, s in zip(ds, stats):
        assert s["hist"] == st["hist"]
        for k in ("phi", "u", "v", "w"):
            assert torch.equal(getattr(t, k), getattr(d, k)), k
