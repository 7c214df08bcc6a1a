"""The coarsest level's direct solve at the sizes where its inversion changes
form: one workgroup with 4 or 8 matrix entries per thread and direction (up to
64 and 128 unknowns), then blocks of 16 pivots up to 512, with full and
partial last blocks.  The reference is a dense solve of the oracle's
operator on the zero-mean subspace; the tolerance is the forward error bound
of Gauss-Jordan elimination on a symmetric positive definite matrix, n eps
times its condition number (the leading constant taken as 4)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu


def dense(apply, shape):
    n = int(np.prod(shape))
    A = np.empty((n, n))
    for c in range(n):
        e = np.zeros(n)
        e[c] = 1.0
        A[:, c] = apply(e.reshape(shape)).ravel()
    return A


def check(A, f, phi):
    """A: L as a matrix (constants in its null space)."""
    n = len(A)
    M = -A + (-np.trace(A) / n) * np.ones((n, n))
    f = f.ravel() - f.mean()
    x = np.linalg.solve(M, -f)
    x -= x.mean()
    tol = 4 * n * np.finfo(float).eps * np.linalg.cond(M)
    assert np.linalg.norm(phi.ravel() - x) <= tol * np.linalg.norm(x), (n, tol)


def fields(n, seed):
    nx, ny, nz = n
    rng = np.random.default_rng(seed)
    z = (np.arange(nz) + 0.5) / nx
    b0c, b0e = np.exp(-z / 0.4), np.exp(-np.arange(nz + 1) / nx / 0.4)
    return rng, b0c, b0e, b0c[:, None, None] * (1.0 + 0.05 * rng.standard_normal((nz, ny, nx)))


def put(H, name, a):
    H.level_copy(0, name, torch.from_numpy(np.ascontiguousarray(a)).cuda(), to_hierarchy=True)


def get_phi(H, shape):
    t = torch.empty(shape, dtype=torch.float64, device="cuda")
    H.level_copy(0, "phi", t, to_hierarchy=False)
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("n", [(4, 4, 2), (4, 4, 4), (13, 5, 1), (8, 16, 1), (43, 3, 1), (32, 5, 1), (7, 23, 1), (64, 3, 1), (193, 1, 1),
                               (13, 4, 4), (7, 10, 6), (512, 1, 1)])
@pytest.mark.parametrize("per", [(True, True, False), (False, False, False)])
def test_mac_coarsest_solve(mp, n, per):
    h = 1.0 / n[0]
    rng, b0c, b0e, rho = fields(n, 3)
    H = mp.Hierarchy(mp.make_params(n, h, per))
    H.set_coefficients(*(torch.from_numpy(a).cuda() for a in (rho, b0c, b0e)))
    assert H.nlevels == 1
    f = rng.standard_normal(rho.shape)
    put(H, "f", f)
    H.level_step(0, "coarse")
    phi = get_phi(H, rho.shape)
    H.close()
    coeffs = O.face_coeffs(n, per, rho, b0c, b0e)
    check(dense(lambda e: O.apply(n, per, h, coeffs, e), rho.shape), f, phi)


@pytest.mark.parametrize("n", [(3, 3, 3), (5, 4, 3), (5, 5, 3), (7, 7, 1), (7, 7, 2), (7, 5, 5), (7, 7, 7)])
@pytest.mark.parametrize("per", [(True, True, False), (False, False, False)])
def test_nodal_coarsest_solve(mp, n, per):
    h = 1.0 / n[0]
    rng, b0c, _, rho = fields(n, 4)
    H = mp.NodalHierarchy(mp.make_params(n, h, per))
    assert H.nlevels == 1
    H.set_coefficients(torch.from_numpy(rho).cuda(), torch.from_numpy(b0c).cuda())
    sig = O.nodal_sigma(rho, b0c)
    shape = O.node_dims(n, per)[::-1]
    f = rng.standard_normal(shape)
    put(H, "f", f)
    H.level_step(0, "coarse")
    phi = get_phi(H, shape)
    H.close()
    check(dense(lambda e: O.nodal_apply(n, per, h, sig, e), shape), f, phi)
