"""Links that are in SU(3) only to single precision: an ensemble stored as
complex64 and read back (GPU).

The library reads rows 0 and 1 of a link and completes row 2 = conj(row0 x
row1).  On such links the order of completing and multiplying matters at the
deviation from SU(3) (1e-8 here): F and theta of a solve must be those of the
links it returns all the same.

Bars: FP64 rounding, as for links in SU(3) (1e-14 on F, 1e-12 relative on theta
far from the solution).  At theta = 1e-15 the entries of Delta are about 3e-8,
rounding errors in them 1e-15, so theta is held to 1e-6.
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
