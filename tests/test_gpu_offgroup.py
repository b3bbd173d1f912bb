"""Links that are in SU(3) only to single precision: an ensemble stored as
complex64 and read back (GPU).

The library reads rows 0 and 1 of a link and completes row 2 = conj(row0 x
row1).  On such links the order of completing and multiplying matters at the
deviation from SU(3) (1e-8 here), so the results are held to their definition
with the links so completed: F and theta of a solve are those of the links it
returns, a gradient's links are rotated and then completed, F_U[g] and the
plaquette are products of three rows.

Bars: FP64 rounding, as for links in SU(3) (1e-14 on F and the plaquette, 1e-12
relative on theta far from the solution and on gradients).  At theta = 1e-15 the
entries of Delta are about 3e-8, rounding errors in them 1e-15, so theta is held
to 1e-6.
"""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

ALPHA = 0.08


def gpu(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def cpu(t):
    return t.detach().cpu().numpy()


def fp32_links(L, seed):
    return inputs.make_config(L, 0.5, seed)[0].astype(np.complex64).astype(np.complex128)


def completed(U):
    """Rows 0,1 of U and row 2 from them."""
    return np.concatenate([U[..., :2, :],
                           np.cross(U[..., 0, :], U[..., 1, :]).conj()[..., None, :]], axis=-2)


def dag(a):
    return a.conj().swapaxes(-1, -2)


def ahead(a, mu):
    """a(x + mu) of a site field (t, z, y, x, ...)."""
    return np.roll(a, -1, axis=3 - mu)


def gell_mann():
    lam = np.zeros((8, 3, 3), complex)
    for (i, j), a in (((0, 1), 0), ((0, 2), 3), ((1, 2), 5)):
        lam[a, i, j] = lam[a, j, i] = 1
        lam[a + 1, i, j], lam[a + 1, j, i] = -1j, 1j
    lam[2] = np.diag([1, -1, 0])
    lam[7] = np.diag([1, 1, -2]) / np.sqrt(3)
    return lam


def expm(X):
    E = one = np.broadcast_to(np.eye(3, dtype=complex), X.shape)
    for k in range(16, 0, -1):
        E = one + X @ E / (64 * k)
    for _ in range(6):
        E = E @ E
    return E


# the update whose threads form the links of their own site, above the smallest
# volume that keeps the input links; rows that are no multiple of a wavefront;
# the update that shares links through LDS; stored links
SHAPES = [(16, 16, 16, 12), (27, 9, 16, 18), (64, 32, 16, 16), (12, 12, 12, 12)]


@pytest.mark.parametrize("L", SHAPES)
def test_sweeps_report_the_returned_links(lgf_gpu, L):
    Ug = gpu(fp32_links(L, 60 + sum(L)))
    r = lgf_gpu.iterate(Ug, ALPHA, 5)
    assert r.F == pytest.approx(lgf_gpu.functional(Ug), abs=1e-14)
    assert r.theta == pytest.approx(lgf_gpu.theta(Ug), rel=1e-12)
    out = cpu(Ug)
    assert r.F == pytest.approx(oracle.F(out), abs=1e-14)
    assert r.theta == pytest.approx(oracle.theta(out), rel=1e-12)


@pytest.mark.parametrize("L", SHAPES)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solve_reports_the_returned_links(lgf_gpu, L, precision):
    Ug = gpu(fp32_links(L, 70 + sum(L)))
    r = lgf_gpu.fix(Ug, ALPHA, 1e-15, precision=precision)
    assert r.status == 0
    assert r.F == pytest.approx(lgf_gpu.functional(Ug), abs=1e-14)
    assert r.theta == pytest.approx(lgf_gpu.theta(Ug), rel=1e-6)
    assert lgf_gpu.theta(Ug) < 1e-15


def test_omega_gradient_of_the_rotated_links(lgf_gpu):
    L = (4, 6, 4, 8)
    V = int(np.prod(L))
    U = fp32_links(L, 81)
    om = inputs.random_omega(L, 0.3, 82)
    lam = gell_mann()
    g = expm(0.5j * np.tensordot(om, lam, (-1, 0)))
    Uc = completed(U)
    W = completed(np.stack([g @ Uc[mu] @ dag(ahead(g, mu)) for mu in range(4)]))
    F = np.trace(W, axis1=-2, axis2=-1).real.sum() / (12 * V)
    X = sum(np.roll(W[mu], 1, axis=3 - mu) - W[mu] for mu in range(4))
    D = X - dag(X)
    y = np.einsum("aij,...ji->...a", lam, D).imag / (48 * V)
    # the transpose of sum_k A^k / (k+1)!, A the bracket with i om.T
    f = np.einsum("aij,bjk,cki->abc", lam, lam, lam)
    f = (f - f.swapaxes(0, 1)).imag / 4
    term, grad = y, y.copy()
    for k in range(1, 40):
        term = -np.einsum("abc,...c,...b->...a", f, om, term) / (k + 1)
        grad += term
    Fg, dF = lgf_gpu._ctx(gpu(U)).functional_omega_grad(gpu(U), gpu(om))
    assert Fg == pytest.approx(F, abs=1e-14)
    assert np.max(np.abs(cpu(dF) - grad)) < 1e-12 * np.max(np.abs(grad))


def test_products_of_three_rows(lgf_gpu):
    L = (4, 6, 4, 8)
    V = int(np.prod(L))
    U = fp32_links(L, 83)
    om = inputs.random_omega(L, 0.3, 84)
    Uc = completed(U)
    g = expm(0.5j * np.tensordot(om, gell_mann(), (-1, 0)))
    F = sum(np.trace(g @ Uc[mu] @ dag(ahead(g, mu)), axis1=-2, axis2=-1).real.sum()
            for mu in range(4)) / (12 * V)
    P = sum(np.trace(Uc[mu] @ ahead(Uc[nu], mu) @ dag(Uc[nu] @ ahead(Uc[mu], nu)),
                     axis1=-2, axis2=-1).real.sum()
            for mu in range(4) for nu in range(mu + 1, 4)) / (18 * V)
    Ug = gpu(U)
    assert lgf_gpu._ctx(Ug).functional_omega(Ug, gpu(om)) == pytest.approx(F, abs=1e-14)
    assert lgf_gpu.functional(Ug, gpu(g)) == pytest.approx(F, abs=1e-14)
    assert lgf_gpu.plaquette(Ug) == pytest.approx(P, abs=1e-14)
