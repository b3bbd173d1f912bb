"""Small lattices (GPU): the whole transform of a field in one block (up to 2048
sites), the stopping test taken along by the next sweep's first kernel (up to
640 pairs of partials), the update with a lane per link (up to 20480 sites).

Each against the oracle sweep by sweep (1e-13 a sweep, as in the lockstep
tests), at the largest and just above the smallest sizes of each rule, with
blocks smaller than a wavefront and blocks that end in a part of one.  The
stopping test's history must agree with the oracle's: every sweep's F and
theta come from it, whichever kernel took it.
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


SHAPES = [(2, 2, 2, 2), (4, 4, 4, 4), (9, 3, 2, 6), (8, 8, 8, 4), (2, 2, 2, 64), (64, 2, 2, 2),
          (32, 4, 4, 4), (27, 9, 2, 4), (8, 8, 8, 8), (6, 9, 8, 16), (16, 16, 16, 4),
          (4, 4, 16, 64), (16, 16, 8, 9), (12, 18, 9, 12)]


@pytest.mark.parametrize("L", SHAPES)
@pytest.mark.parametrize("kw", [{}, {"exact_exp": True}])
def test_sweeps_and_history(lgf_gpu, L, kw):
    U, _ = inputs.make_config(L, 0.5, 300 + sum(L))
    n = 9
    ref = oracle.fix(U, ALPHA, 0.0, n, **kw)
    Ug = gpu(U)
    lgf_gpu.iterate(Ug, ALPHA, n, **kw)
    assert np.max(np.abs(cpu(Ug) - ref["U"])) < n * 1e-13
    F, T = lgf_gpu._ctx(Ug).history()
    assert len(F) == n + 1
    assert np.max(np.abs(F - ref["F_hist"][:n + 1])) < 1e-13
    assert np.max(np.abs(T / ref["theta_hist"][:n + 1] - 1)) < 1e-9


@pytest.mark.parametrize("L", [(4, 4, 4, 4), (9, 3, 2, 6), (8, 8, 8, 8), (4, 4, 16, 64)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nc", [3, 2])
def test_solve_stops_where_theta_crosses(lgf_gpu, L, precision, nc):
    """The last theta is below the tolerance and the one before is not."""
    make = inputs.make_config if nc == 3 else inputs.make_config_su2
    Ug = gpu(make(L, 0.5, 400 + sum(L))[0])
    r = lgf_gpu.fix(Ug, ALPHA, 1e-13, precision=precision, max_iter=500)
    ctx = lgf_gpu._ctx(Ug, precision)
    F, T = ctx.history()
    assert r.status == 0 and len(T) == r.iterations + 1
    assert T[-1] == r.theta < 1e-13 and np.all(T[:-1] >= 1e-13)
    assert ctx.theta(Ug) == pytest.approx(r.theta, rel=1e-6)
    assert ctx.functional(Ug) == pytest.approx(r.F, abs=1e-14)


@pytest.mark.parametrize("L", [(4, 4, 4, 4), (8, 8, 8, 8), (4, 4, 16, 64)])
def test_max_iter_ends_inside_a_batch(lgf_gpu, L):
    U, _ = inputs.make_config(L, 0.5, 500)
    for k in (1, 2, 3, 5, 7):
        Ug = gpu(U)
        r = lgf_gpu.fix(Ug, ALPHA, 1e-15, max_iter=k)
        assert r.status == lgf_gpu.LGF_NOT_CONVERGED and r.iterations == k
        assert np.max(np.abs(cpu(Ug) - oracle.iterate(U, ALPHA, k))) < k * 1e-13


# register-column planes of fewer than 64 threads (4 x 12; SU(2) 2 x 27 and, with
# most lanes of the sum missing, 2 x 6), of one wavefront and of two, and the
# one-block transform
@pytest.mark.parametrize("L,nc", [((12, 18, 9, 12), 3), ((27, 16, 12, 8), 2), ((6, 16, 16, 16), 2),
                                  ((16, 16, 8, 9), 3), ((32, 8, 8, 8), 3), ((8, 8, 8, 4), 3)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_history_does_not_depend_on_the_batches(lgf_gpu, L, nc, precision):
    """A sweep's F and theta are the same bits whether its stopping test had a
    kernel of its own (the last sweep of a call) or rode along."""
    make = inputs.make_config if nc == 3 else inputs.make_config_su2
    U, _ = make(L, 0.5, 600 + sum(L))
    hist = []
    for n in (6, 1, 2, 3, 4, 5):
        Ug = gpu(U)
        lgf_gpu.iterate(Ug, ALPHA, n, precision=precision)
        hist.append(lgf_gpu._ctx(Ug, precision).history())
    for F, T in hist[1:]:
        assert np.array_equal(F, hist[0][0][:len(F)])
        assert np.array_equal(T, hist[0][1][:len(T)])


# the one-block transform, with 49 KB of LDS at the second shape
@pytest.mark.parametrize("L", [(8, 8, 8, 4), (2, 4, 16, 16), (9, 3, 2, 6)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nc", [3, 2])
def test_runs_are_bitwise_equal(lgf_gpu, L, precision, nc):
    make = inputs.make_config if nc == 3 else inputs.make_config_su2
    U, _ = make(L, 0.5, 650 + sum(L))
    a, b = gpu(U), gpu(U)
    ra = lgf_gpu.iterate(a, ALPHA, 9, precision=precision)
    rb = lgf_gpu.iterate(b, ALPHA, 9, precision=precision)
    assert np.array_equal(cpu(a), cpu(b))
    assert ra.F == rb.F and ra.theta == rb.theta
