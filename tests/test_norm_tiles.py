"""Norm rows of the finest level's sweep with the residual norm and of the
refinement of mixed precision, which a batch has to sum as the problem alone
does: the marchless tiles only on the smallest levels without ragged tiles
(above, they cost a batch more than they save), and the same history, to the
bit, alone and in a batch, which marches twice as many planes a tile where the
problem alone marches four or eight."""
import ctypes
import os

import pytest

from paper_1910_12979_amd import inputs as I

MARCHLESS = 14


@pytest.mark.parametrize("n,marchless", [
    ((32, 32, 32), True), ((48, 24, 24), True), ((40, 24, 56), False),       # ragged tiles
    ((48, 48, 24), False), ((32, 8, 256), False), ((64, 48, 32), False), ((48, 48, 48), False), ((96, 80, 48), False),
    ((64, 64, 64), False), ((16, 64, 64), True),       # nothing else takes fewer than 32 cells in x
])
def test_rule(n, marchless):
    from paper_1910_12979_amd import build, macproj
    if not os.path.exists(macproj.LIB_PATH):
        build.build()
    macproj.tune_cache_clear()
    lib = macproj.lib()
    norm, sweep = lib["_ZN2mg15norm_config_forEiiib"], lib["_ZN2mg16sweep_config_forEiiibbbb"]
    fits = lib["_ZN2mg14sweep_cfg_fitsEiii"]
    norm.argtypes = [ctypes.c_int] * 3 + [ctypes.c_bool]
    sweep.argtypes = [ctypes.c_int] * 3 + [ctypes.c_bool] * 4
    fits.argtypes = [ctypes.c_int] * 3
    fits.restype = ctypes.c_bool
    cfg = norm(*n, True)
    assert (cfg == MARCHLESS) == marchless
    assert cfg == MARCHLESS or fits(n[0], n[1], cfg)
    solo = sweep(*n, True, True, False, False)
    assert solo == MARCHLESS or cfg == solo         # else the sweep's own


@pytest.mark.gpu
@pytest.mark.parametrize("n", [(32, 32, 32), (48, 24, 24), (40, 24, 56), (48, 48, 48), (96, 80, 48), (32, 8, 256),
                               (32, 8, 10), (32, 8, 14), (40, 24, 20),       # the last planes: 2, 4 and 2, 4
                               (128, 96, 96), (96, 96, 80)])                 # 8 planes alone, 16 in a batch
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_alone_and_in_a_batch(mp, n, precision):
    import torch
    prob = I.make_problem(n, H=0.2, rho_noise=0.05, seed=17, dx=1 / n[0])
    par = mp.params_of(prob, precision=precision)
    d = mp.to_device(prob)
    H = mp.Hierarchy(par)
    st = H.mac_project(d.rho, d.beta0_cc, d.beta0_edge, d.S, d.u, d.v, d.w, d.phi)
    H.close()
    ds = [mp.to_device(prob) for _ in range(3)]
    code, stats = mp.project_batch([par] * 3, ds)
    assert code == 0 and st["cycles"] >= 3
    for t, s in zip(ds, stats):
        assert s["hist"] == st["hist"]
        assert all(torch.equal(getattr(t, k), getattr(d, k)) for k in ("phi", "u", "v", "w"))
