"""Measurements and gradients that read the caller's links directly (GPU).

Blocks that end inside the lattice, wavefronts that straddle rows, both site
orders, and exponents from tiny (a single term of the exponential map's
derivative) to order one (several terms, and squarings of the exponential).
Bars: those of the per-step tests (1e-13 absolute on O(1) quantities) and of
the gradient tests (1e-12 of the largest entry).
"""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu


def gpu(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def cpu(t):
    return t.detach().cpu().numpy()


SHAPES = [(2, 3, 4, 6), (9, 3, 4, 2), (8, 8, 2, 4), (27, 4, 3, 6), (4, 16, 6, 64)]


@pytest.mark.parametrize("L", SHAPES)
def test_plaquette_functional_and_divergence(lgf_gpu, L):
    U, _ = inputs.make_config(L, 0.5, 50 + sum(L))
    Ug = gpu(U)
    g = inputs.haar_su3(int(np.prod(L)), np.random.default_rng(1)).reshape(
        inputs.site_shape(L) + (3, 3))
    assert lgf_gpu.plaquette(Ug) == pytest.approx(oracle.plaquette(U), abs=1e-14)
    assert lgf_gpu.functional(Ug) == pytest.approx(oracle.F(U), abs=1e-14)
    assert lgf_gpu.functional(Ug, gpu(g)) == pytest.approx(oracle.functional(U, g), abs=1e-14)
    assert lgf_gpu.theta(Ug) == pytest.approx(oracle.theta(U), rel=1e-13)
    assert np.max(np.abs(cpu(lgf_gpu.divergence(Ug)) - oracle.delta(U))) < 1e-13


@pytest.mark.parametrize("L", SHAPES[:3])
@pytest.mark.parametrize("sigma", [0.0, 1e-9, 0.5])
def test_omega_gradient(lgf_gpu, L, sigma):
    U, _ = inputs.make_config(L, 0.5, 60 + sum(L))
    om = inputs.random_omega(L, sigma, 61)
    F, grad = lgf_gpu.functional_omega_grad(gpu(U), gpu(om))
    Fr, ref = oracle.functional_omega_grad(U, om)
    assert F == pytest.approx(Fr, abs=1e-13)
    assert lgf_gpu.functional_omega(gpu(U), gpu(om)) == pytest.approx(Fr, abs=1e-13)
    assert np.max(np.abs(cpu(grad) - ref)) < 1e-12 * np.max(np.abs(ref))


@pytest.mark.parametrize("sigma", [1e-9, 0.5])
def test_theta_gradient_at_eps(lgf_gpu, sigma):
    """theta(exp(i eps.T) U) against the links rotated on the host, and its
    gradient: the derivative at eps along the left-invariant directions of
    exp(i eps.T), which the eps = 0 gradient of the rotated links gives through
    the oracle, mapped by the derivative of the exponential (central
    differences of scipy's expm)."""
    from scipy.linalg import expm

    L = (2, 3, 4, 6)
    U, _ = inputs.make_config(L, 0.5, 70)
    eps = sigma * np.random.default_rng(71).standard_normal((4,) + inputs.site_shape(L) + (8,))
    T = inputs.GELL_MANN / 2
    E = np.array([expm(1j * np.tensordot(w, T, 1)) for w in eps.reshape(-1, 8)]).reshape(U.shape)
    th, grad = lgf_gpu.theta_grad(gpu(U), gpu(eps))
    thr, left = oracle.theta_grad(E @ U)
    assert th == pytest.approx(thr, rel=1e-12)
    g, lf = cpu(grad).reshape(-1, 8), left.reshape(-1, 8)
    rng, h = np.random.default_rng(72), 1e-5
    for i in rng.integers(0, g.shape[0], 16):
        w = eps.reshape(-1, 8)[i]
        for a in range(8):
            d = np.zeros(8)
            d[a] = h
            dE = (expm(1j * np.tensordot(w + d, T, 1)) - expm(1j * np.tensordot(w - d, T, 1))) / (2 * h)
            X = dE @ E.reshape(-1, 3, 3)[i].conj().T  # i sum_b J_ab T^b
            J = np.array([2 * np.trace(X @ T[b]).imag for b in range(8)])
            # h^2/6 of the third derivative, at most |T|^3 < 1: 2e-11, and 1e-16/h of rounding
            assert abs(J @ lf[i] - g[i, a]) < 1e-9 * np.max(np.abs(lf))


def test_unaligned_parameters(lgf_gpu):
    """Parameters that begin 8 bytes into a buffer (a contiguous view) give the same gradients."""
    import torch

    L = (4, 4, 6, 4)
    U = gpu(inputs.make_config(L, 0.5, 80)[0])
    om = gpu(inputs.random_omega(L, 0.5, 81))
    flat = torch.empty(om.numel() + 1, dtype=torch.float64, device="cuda")
    view = flat[1:].view(om.shape)
    view.copy_(om)
    a, b = lgf_gpu.functional_omega_grad(U, om), lgf_gpu.functional_omega_grad(U, view)
    assert a[0] == b[0] and torch.equal(a[1], b[1])


@pytest.mark.parametrize("L", [(8, 8, 8, 8), (27, 9, 4, 6)])
def test_outputs_over_the_inputs(lgf_gpu, L):
    """Delta, dF/domega and dtheta/deps written over the links, or over omega or
    eps, are those written elsewhere (C ABI; the binding allocates them)."""
    import ctypes

    import torch

    lib = lgf_gpu.load()
    U = gpu(inputs.make_config(L, 0.5, 91)[0])
    om = gpu(inputs.random_omega(L, 0.3, 92))
    eps = gpu(np.random.default_rng(93).normal(0, 0.3, (4,) + inputs.site_shape(L) + (8,)))
    ctx = lgf_gpu._ctx(U)
    val = ctypes.c_double()
    p = lambda t, off=0: ctypes.c_void_p(t.data_ptr() + off)
    V = int(np.prod(L))

    def written(call, ref, start, off=0):
        """What call(buffer) leaves at `off` bytes of a copy of `start`."""
        buf = start.clone()
        assert call(buf, p(buf, off)) == 0
        got = torch.view_as_real(buf) if buf.is_complex() else buf
        flat = got.reshape(-1)[off // 8:off // 8 + ref.numel()]
        return torch.equal(flat, ref.reshape(-1))

    D = torch.view_as_real(ctx.divergence(U))
    _, dF = ctx.functional_omega_grad(U, om)
    _, t0 = ctx.theta_grad(U)
    _, t1 = ctx.theta_grad(U, eps)
    for off in (0, 16 * V):
        assert written(lambda b, o: lib.lgf_divergence(ctx._h, p(b), o), D, U, off)
        assert written(lambda b, o: lib.lgf_functional_omega_grad(
            ctx._h, p(b), p(om), ctypes.byref(val), o), dF, U, off)
        assert written(lambda b, o: lib.lgf_theta_grad(
            ctx._h, p(b), None, ctypes.byref(val), o), t0, U, off)
        assert written(lambda b, o: lib.lgf_theta_grad(
            ctx._h, p(b), p(eps), ctypes.byref(val), o), t1, U, off)
    assert written(lambda b, o: lib.lgf_functional_omega_grad(
        ctx._h, p(U), p(b), ctypes.byref(val), o), dF, om)
    assert written(lambda b, o: lib.lgf_theta_grad(
        ctx._h, p(U), p(b), ctypes.byref(val), o), t1, eps)
