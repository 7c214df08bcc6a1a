"""Two FP32 sweeps in one launch on large finest levels of mixed-precision
solves: bit for bit the solve whose sweeps are launched one by one (any forced
tile configuration), at sizes ragged against the 56 x 24 x 64-cell tiles, with
every kind of side the march meets, and for sweep counts that leave a single
sweep over."""
import numpy as np
import pytest
import torch

from paper_1910_12979_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,periodic,sweeps", [
    ((384, 192, 224), (True, True, False), (2, 2)),       # ragged in x and z
    ((256, 256, 256), (False, False, False), (3, 1)),     # walls everywhere; a pair and a single sweep
    ((448, 192, 192), (True, False, True), (2, 3)),       # whole tiles; periodic in z
])
def test_pairs_are_two_sweeps(mp, n, periodic, sweeps):
    prob = I.make_problem(n, seed=11, periodic=periodic)
    got = []
    for cfg in (-1, 9):
        H = mp.Hierarchy(mp.make_params(n, prob.dx, periodic, precision="mixed", pre_sweeps=sweeps[0],
                                        post_sweeps=sweeps[1]))
        mp.mg_tune_sweep(cfg)
        try:
            d = mp.to_device(prob)
            st = H.mac_project(d.rho, d.beta0_cc, d.beta0_edge, d.S, d.u, d.v, d.w, d.phi)
            torch.cuda.synchronize()
        finally:
            mp.mg_tune_sweep(-1)
        H.close()
        got.append((st["hist"], d.phi.cpu().numpy(), d.u.cpu().numpy()))
    # the norms' rows are those of the refinement's tiles: the same values in another order
    assert np.allclose(got[0][0], got[1][0], rtol=1e-12, atol=0.0)
    assert np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][2], got[1][2])
