"""Solves that converge before the last cycle enqueued ahead, and are therefore
run again: right-hand sides whose residual falls ever faster after a good first
cycle.  Each such solve equals, bit for bit, the one that max_cycles keeps from
looking past its convergence; that it was run again at all is checked with the
host loop itself on the solve's own history."""
import numpy as np
import pytest
import torch

from paper_1910_12979_amd import inputs as I
from test_cycles_ahead import MAC, NODAL, drive, exe  # noqa: F401  (exe: fixture)

pytestmark = pytest.mark.gpu


def problem(nodal, n, S):
    p = (I.make_nodal_problem if nodal else I.make_problem)(n, H=1.0, rho_noise=0.0, seed=1, dx=1 / n[0])
    for k in ("uc", "vc", "wc") if nodal else ("u", "v", "w"):
        getattr(p, k)[...] = 0.0
    p.S[:] = S
    p.S -= (p.S * p.beta0_cc[:, None, None]).sum() / (p.beta0_cc.sum() * n[0] * n[1])
    return p


def solve(mp, p, nodal, sweeps, precision, boxes, graphs, rtol, max_cycles):
    par = mp.make_params(p.n, p.dx, p.periodic, rtol=rtol, max_cycles=max_cycles, precision=precision,
                         pre_sweeps=sweeps[0], post_sweeps=sweeps[1], inner_cycles=1)
    H = (mp.NodalHierarchy if nodal else mp.Hierarchy)(par)
    H.set_graphs(graphs)
    if nodal:
        d = mp.nodal_to_device(p)
        st = H.project(d.rho, d.beta0_cc, d.S, d.uc, d.vc, d.wc, d.phi, allow=(0, -4))
        out = (d.phi, d.uc, d.vc, d.wc)
    else:
        if boxes:
            H.set_boxes(boxes)
        d = mp.to_device(p)
        st = H.mac_project(d.rho, d.beta0_cc, d.beta0_edge, d.S, d.u, d.v, d.w, d.phi, allow=(0, -4))
        out = (d.phi, d.u, d.v, d.w)
    torch.cuda.synchronize()
    H.close()
    return st, [t.cpu().numpy() for t in out]


@pytest.mark.parametrize("nodal,n,sweeps,precision,boxes,graphs", [
    (False, 32, (1, 2), "fp64", None, False),
    (False, 32, (1, 2), "mixed", None, False),
    (False, 64, (1, 2), "fp64", (32, 32, 32), False),
    (False, 64, (1, 2), "mixed", (32, 32, 32), False),
    (True, 32, (3, 1), "fp64", None, False),
    (True, 32, (3, 1), "fp64", None, True),
    (True, 32, (3, 1), "mixed", None, False),
])
def test_run_again(mp, exe, nodal, n, sweeps, precision, boxes, graphs):  # noqa: F811
    n = (n, n, n)
    i, j = np.arange(n[0]), np.arange(n[1])[:, None]
    k = 2 * np.pi * 4 / n[0]
    S = np.cos(k * (i + 0.5)) * np.cos(k * (j + 0.5)) if nodal else (-1.0) ** i
    p = problem(nodal, n, S)
    full, _ = solve(mp, p, nodal, sweeps, precision, boxes, graphs, 1e-14, 10)
    hist = full["hist"][1:]
    first = NODAL if nodal else MAC
    over = [c for c, h in enumerate(hist, 1)
            if h > 1e-13 and drive(exe, hist + [0.1 * hist[-1]] * 10, 1.05 * h, first=first)["over"]]
    print("ratios", [b / a for a, b in zip(full["hist"], hist)], "over at", over)
    assert over
    for c in over:
        rtol = 1.05 * hist[c - 1]
        st, out = solve(mp, p, nodal, sweeps, precision, boxes, graphs, rtol, 60)
        ref, fields = solve(mp, p, nodal, sweeps, precision, boxes, False, rtol, c)
        assert st["status_name"] == ref["status_name"] == "OK" and st["cycles"] == ref["cycles"] == c
        assert st["hist"] == ref["hist"] == full["hist"][:c + 1]
        assert all(np.array_equal(a, b) for a, b in zip(out, fields))
