"""Replayed cycles (set_graphs(True); off by default): the solves of one
hierarchy, whose cycles are captured, replayed and enqueued ahead of their
norms, give the separately launched solves' bits, with eager work in between:
the same problem several times over, other buffers, an odd number of sweeps
(no capture), a forced tile, other FP32 cycles a step, the bottom switched off
and on, a solve that ends at another cycle."""
import numpy as np
import pytest
import torch

from paper_1910_12979_amd import inputs as I

pytestmark = pytest.mark.gpu


class Mac:
    def __init__(self, mp, prob, **kw):
        self.mp, self.kw, self.n, self.dx, self.per = mp, kw, prob.n, prob.dx, prob.periodic
        self.H = mp.Hierarchy(self.par())
        self.fields = "u", "v", "w", "phi"

    def par(self, **kw):
        return self.mp.make_params(self.n, self.dx, self.per, **{**self.kw, **kw})

    def device(self, prob):
        return self.mp.to_device(prob)

    def run(self, d):
        return self.H.mac_project(d.rho, d.beta0_cc, d.beta0_edge, d.S, d.u, d.v, d.w, d.phi)


class Nodal(Mac):
    def __init__(self, mp, prob, **kw):
        self.mp, self.kw, self.n, self.dx, self.per = mp, kw, prob.n, prob.dx, prob.periodic
        self.H = mp.NodalHierarchy(self.par())
        self.fields = "uc", "vc", "wc", "phi"

    def device(self, prob):
        return self.mp.nodal_to_device(prob)

    def run(self, d):
        return self.H.project(d.rho, d.beta0_cc, d.S, d.uc, d.vc, d.wc, d.phi)


class Pair:
    """A hierarchy with separate launches and one that replays."""

    def __init__(self, kind, mp, prob, **kw):
        self.eager, self.replay = kind(mp, prob, **kw), kind(mp, prob, **kw)
        self.eager.H.set_graphs(False)
        self.replay.H.set_graphs(True)

    def each(self, what):
        for k in (self.eager, self.replay):
            what(k)

    def check(self, prob, times=3):
        """Each solve of the replaying hierarchy: inputs at the same addresses (restored in between)."""
        ref = self.eager.device(prob)
        st0 = self.eager.run(ref)
        d = self.replay.device(prob)
        start = {f: getattr(d, f).clone() for f in self.replay.fields}
        for _ in range(times):
            for f, t in start.items():
                getattr(d, f).copy_(t)
            st1 = self.replay.run(d)
            torch.cuda.synchronize()
            assert st1["hist"] == st0["hist"] and st1["cycles"] == st0["cycles"]
            for f in self.replay.fields:
                assert torch.equal(getattr(d, f), getattr(ref, f)), f
        return st0

    def close(self):
        self.each(lambda k: k.H.close())


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_mac_replays(mp, precision):
    n = (64, 48, 32)
    probs = [I.make_problem(n, H=0.15, seed=41, rho_noise=0.05), I.make_problem(n, H=0.3, seed=42)]
    P = Pair(Mac, mp, probs[0], precision=precision)
    try:
        assert P.check(probs[0])["cycles"] >= 4
        P.check(probs[1])                                                   # other buffers
        P.check(probs[0])
        P.each(lambda k: k.H.set_params(k.par(post_sweeps=1)))              # odd: no capture
        P.check(probs[0])
        P.each(lambda k: k.H.set_params(k.par(post_sweeps=4)))
        P.check(probs[0])
        P.each(lambda k: k.H.set_params(k.par(rtol=1e-5)))                  # ends at another cycle
        P.check(probs[1])
        P.each(lambda k: k.H.set_params(k.par()))
        for cfg in (0, 7, -1):
            mp.mg_tune_sweep(cfg)
            P.check(probs[0])
        for on in (False, True):
            P.each(lambda k: k.H.set_bottom(on))
            P.check(probs[1])
        if precision == "mixed":
            for inner in (1, 3, 0):
                P.each(lambda k: k.H.set_params(k.par(inner_cycles=inner)))
                P.check(probs[0])
    finally:
        mp.mg_tune_sweep(-1)
        P.close()


@pytest.mark.parametrize("outflow", [False, True])
def test_mac_replays_stored_coefficients(mp, outflow):
    """A radial base state: the coefficients come from the hierarchy's arrays."""
    prob = I.make_star_problem((48, 48, 48), Hr=0.3, rho_noise=0.05, seed=43)
    res = []
    for graphs in (False, True):
        out = prob.outflow if outflow else None
        H = mp.Hierarchy(mp.make_params(prob.n, prob.dx, (False,) * 3 if outflow else (True,) * 3, outflow=out))
        H.set_graphs(graphs)
        for _ in range(3):
            d = mp.to_device(prob)
            if not outflow:
                d.S.zero_()
                for t in (d.u, d.v, d.w):
                    t.zero_()
                d.u[:, :, 1:-1].normal_(generator=torch.Generator(device="cuda").manual_seed(1))
            st = H.mac_project_radial(d.rho, d.beta0_r, prob.dr_base, prob.centre, d.S, d.u, d.v, d.w, d.phi)
            torch.cuda.synchronize()
            res.append((st["hist"], [t.cpu().numpy() for t in (d.phi, d.u, d.v, d.w)]))
        H.close()
    for hist, fields in res[1:]:
        assert hist == res[0][0]
        assert all(np.array_equal(a, b) for a, b in zip(fields, res[0][1]))


def test_nodal_replays(mp):
    n = (64, 48, 32)
    probs = [I.make_nodal_problem(n, H=0.2, rho_noise=0.05, seed=s) for s in (44, 45)]
    P = Pair(Nodal, mp, probs[0])
    try:
        assert P.check(probs[0])["cycles"] >= 4
        P.check(probs[1])
        for on in (False, True):
            P.each(lambda k: k.H.set_bottom(on))
            P.check(probs[0])
        for cfg in (3, -1):
            mp.nodal_tune_sweep(cfg)
            P.check(probs[1])
    finally:
        mp.nodal_tune_sweep(-1)
        P.close()
