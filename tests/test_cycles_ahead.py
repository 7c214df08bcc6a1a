"""Cycles enqueued ahead of their residual norms, on the CPU: the host loop of
the solves (csrc/cycles.h) driven by scripted histories (tests/cycles_ahead.cpp)
and by the oracle's histories of smooth and random right-hand sides.

* Whatever the look-ahead, a solve ends at the first cycle at or below rtol,
  at the first non-finite residual or at max_cycles, with the history up to it;
  `over` says whether cycles beyond the converged one were enqueued (the solve
  is then run again without looking ahead, which always ends without `over`).
* A smooth right-hand side keeps most of its residual in the first cycle and
  loses it fast afterwards: its first ratio must not send the solve past its
  convergence."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import oracle as O
from paper_1910_12979_amd import inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1910_12979_amd", "csrc")
OK, NOT_CONVERGED, NONFINITE = 0, -4, -5
MAC, NODAL = 0.02, 0.01                       # kFirstGainMac, kFirstGainNodal


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not installed")
    out = str(tmp_path_factory.mktemp("cycles") / "cycles_ahead")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC,
                    os.path.join(ROOT, "tests", "cycles_ahead.cpp"), "-o", out], check=True)
    return out


def drive(exe, hist, rtol, ahead=True, first=MAC, max_cycles=100):
    """hist: relative residuals after each cycle (hist[0] after the first)."""
    args = [exe, repr(float(first)), repr(float(rtol)), str(max_cycles), str(int(ahead))] + [repr(float(h)) for h in hist]
    q = subprocess.run(args, capture_output=True, text=True, check=True).stdout.split()
    rc, status, cycles, over, enqueued, looks = (int(q[i]) for i in (0, 1, 2, 4, 5, 6))
    assert rc == 0
    return dict(status=status, cycles=cycles, rel=float(q[3]), over=bool(over), enqueued=enqueued, looks=looks,
                hist=[float(x) for x in q[7:]])


def expected(hist, rtol, max_cycles):
    for c, h in enumerate(hist[:max_cycles], 1):
        if not np.isfinite(h):
            return NONFINITE, c
        if h <= rtol:
            return OK, c
    return NOT_CONVERGED, max_cycles


def ratios(*r):
    return list(np.cumprod(r))


@pytest.mark.parametrize("name,hist,rtol,max_cycles", [
    ("constant rate", ratios(*[0.05] * 30), 1e-10, 100),
    ("longer than the ring", ratios(*[0.5] * 60), 1e-9, 100),
    ("stopped by max_cycles", ratios(*[0.1] * 30), 1e-20, 13),
    ("one cycle", ratios(1e-12, 0.5), 1e-10, 100),
    ("diverging first", ratios(2.0, 0.1, *[0.3] * 40), 1e-9, 100),
    ("non-finite", ratios(0.008, 0.03, 0.04) + [float("nan")] + [1.0] * 20, 1e-10, 100),
    ("ever faster", ratios(0.01, 0.01, 1e-7, *[0.5] * 20), 1e-10, 100),
    ("faster at the last moment", ratios(0.015, 0.015, 0.015, 1e-4, *[0.5] * 20), 1e-9, 100),
])
def test_scripted_histories(exe, name, hist, rtol, max_cycles):
    status, cycles = expected(hist, rtol, max_cycles)
    got = drive(exe, hist, rtol, max_cycles=max_cycles)
    assert (got["status"], got["cycles"]) == (status, cycles)
    np.testing.assert_allclose([h for h in got["hist"]][:cycles - (status == NONFINITE)],
                               hist[:cycles - (status == NONFINITE)], rtol=1e-15)
    assert got["enqueued"] <= max_cycles
    assert got["over"] == (status == OK and got["enqueued"] > cycles)
    again = drive(exe, hist, rtol, ahead=False, max_cycles=max_cycles)
    assert not again["over"] and again["looks"] == again["enqueued"] == again["cycles"] == cycles
    assert again["status"] == status and again["hist"] == got["hist"][:cycles]


def test_over_is_reported(exe):
    """A history whose rate improves a hundredfold after two cycles overshoots."""
    hist = ratios(0.01, 0.01, 1e-4, *[0.5] * 20)
    got = drive(exe, hist, 1.01 * hist[2])
    assert got["over"] and got["cycles"] == 3 and got["status"] == OK


def test_looks_ahead_on_a_steady_rate(exe):
    """Random velocities (first ratio 0.0085) need few looks."""
    hist = ratios(0.0085, 0.033, 0.042, 0.053, 0.058, 0.062, 0.065, 0.068)
    got = drive(exe, hist, 1e-10)
    assert got["cycles"] == 8 and not got["over"] and got["looks"] <= 5


def smooth_fields(n):
    nx, ny, nz = n
    z, y, x = np.meshgrid(*[(np.arange(m) + 0.5) / m for m in (nz, ny, nx)], indexing="ij")
    return {"modes": np.cos(2 * np.pi * x) * np.cos(2 * np.pi * y) * np.cos(np.pi * z),
            "layer": np.exp(-((z - 0.4) / 0.05) ** 2), "height": np.cos(np.pi * z),
            "blob": np.exp(-((x - 0.3) ** 2 + (y - 0.6) ** 2 + (z - 0.5) ** 2) / 0.02)}


@pytest.mark.parametrize("kind,n,sweeps", [
    ("mac", (32, 32, 32), (2, 2)), ("mac", (32, 32, 32), (1, 1)), ("mac", (64, 32, 32), (2, 2)),
    ("nodal", (32, 32, 32), (2, 2)), ("nodal", (64, 32, 32), (2, 2)), ("nodal", (32, 32, 32), (1, 1)),
])
def test_smooth_right_hand_sides_are_solved_once(exe, kind, n, sweeps):
    for name, S in smooth_fields(n).items():
        make = I.make_problem if kind == "mac" else I.make_nodal_problem
        p = make(n, H=0.3, rho_noise=0.01, seed=1, dx=1 / n[0])
        for k in ("u", "v", "w") if kind == "mac" else ("uc", "vc", "wc"):
            getattr(p, k)[...] = 0.0
        p.S[:] = S
        w = p.beta0_cc[:, None, None]
        p.S -= (p.S * w).sum() / (p.beta0_cc.sum() * n[0] * n[1])
        solve = O.mac_project if kind == "mac" else O.nodal_project
        hist = solve(p, rtol=1e-11, max_cycles=40, nu1=sweeps[0], nu2=sweeps[1])["hist"]
        # one V-cycle a step, and two (the refinement steps of a mixed MAC solve)
        for step in (1, 2):
            h = list(hist[1:])[step - 1::step]
            first = (MAC if kind == "mac" else NODAL) ** step
            for rtol in 10.0 ** -np.arange(3.0, 10.6, 0.5):
                if min(h) > rtol:
                    continue
                got = drive(exe, h, rtol, first=first)
                assert got["cycles"] == expected(h, rtol, 100)[1]
                assert not got["over"], (name, step, rtol, got)
