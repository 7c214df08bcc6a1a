"""Cycles enqueued ahead of their residual norms: the history of a solve (up to
24 cycles, three times the ring the device keeps the norms in) does not depend
on where it was cut, nor on whether the cycles are separate launches or a
replayed graph, and neither do phi and the velocities, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1910_12979_amd import inputs as I

pytestmark = pytest.mark.gpu


def mac(mp, n, precision, rtol, max_cycles, graphs, boxes=None):
    prob = I.make_problem(n, seed=4)
    H = mp.Hierarchy(mp.make_params(prob.n, prob.dx, prob.periodic, rtol=rtol, max_cycles=max_cycles,
                                    precision=precision))
    if boxes:
        H.set_boxes(boxes)
    H.set_graphs(graphs)
    d = mp.to_device(prob)
    st = H.mac_project(d.rho, d.beta0_cc, d.beta0_edge, d.S, d.u, d.v, d.w, d.phi, allow=(0, -4, -5, 1, 2))
    torch.cuda.synchronize()
    H.close()
    return st, [t.cpu().numpy() for t in (d.u, d.v, d.w, d.phi)]


def nodal(mp, n, precision, rtol, max_cycles, graphs, boxes=None):
    prob = I.make_nodal_problem(n, H=0.2, rho_noise=0.05, seed=4)
    H = mp.NodalHierarchy(mp.make_params(prob.n, prob.dx, prob.periodic, rtol=rtol, max_cycles=max_cycles,
                                         precision=precision))
    H.set_graphs(graphs)
    d = mp.nodal_to_device(prob)
    st = H.project(d.rho, d.beta0_cc, d.S, d.uc, d.vc, d.wc, d.phi, allow=(0, -4, -5, 1, 2))
    torch.cuda.synchronize()
    H.close()
    return st, [t.cpu().numpy() for t in (d.uc, d.vc, d.wc, d.phi)]


@pytest.mark.parametrize("run,n,precision,boxes", [
    (mac, 32, "fp64", None), (mac, 64, "mixed", None), (mac, 64, "fp64", (32, 32, 32)),
    (mac, 64, "mixed", (32, 32, 32)), (nodal, 32, "fp64", None), (nodal, 32, "mixed", None),
])
def test_history_where_cut(mp, run, n, precision, boxes):
    rtol = 1e-18                                  # below what FP64 reaches: every cycle runs
    full, fields = run(mp, n, precision, rtol, 24, False, boxes)
    assert full["cycles"] == 24
    hist = full["hist"]
    assert len(hist) == 25 and hist[0] == 1.0 and hist[3] < 1e-2
    if boxes is None:
        st, again = run(mp, n, precision, rtol, 24, True, boxes)
        assert st["hist"] == hist
        assert all(np.array_equal(a, b) for a, b in zip(fields, again))
    for cut in (1, 2, 3, 9, 10):
        st, _ = run(mp, n, precision, rtol, cut, False, boxes)
        assert st["cycles"] == cut and st["hist"] == hist[:cut + 1]
    # stopped by the tolerance, with cycles ahead until just before it
    for stop in (2, 3):
        st, _ = run(mp, n, precision, hist[stop] * 1.01, 24, False, boxes)
        assert st["status_name"] == "OK" and st["cycles"] == stop and st["hist"] == hist[:stop + 1]
