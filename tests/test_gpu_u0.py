"""FP64 sweeps that keep the input links and the accumulated transformation
(12-real SU(3) links from 49152 sites on) against the FP64 oracle (GPU).

Bars: three sweeps of rounding at the 1e-13 per-sweep bar of the lockstep
tests; F and theta against the oracle's values of the returned links, which
round once more than the links the kernel formed.
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


# G accumulated in the inverse (x,y) pass (16 and 32 wide register columns;
# rows of 27, no multiple of a wavefront), after it where the pass cannot take
# it ((x,t)/(y,z) split; whole (x,y) planes in LDS); the smallest volume of
# the rule and one just below it
SHAPES = [(16, 16, 16, 12), (32, 32, 8, 6), (27, 9, 16, 18), (16, 8, 8, 48), (64, 12, 8, 8),
          (16, 16, 16, 9)]


@pytest.mark.parametrize("L", SHAPES)
@pytest.mark.parametrize("kw", [{}, {"exact_exp": True}, {"accelerate": False}])
def test_three_sweeps(lgf_gpu, L, kw):
    U, _ = inputs.make_config(L, 0.5, 700 + sum(L))
    Ug = gpu(U)
    r = lgf_gpu.iterate(Ug, ALPHA, 3, **kw)
    out = cpu(Ug)
    ref = oracle.fix(U, ALPHA, 0.0, 3, **kw)["U"]
    assert r.iterations == 3
    assert np.max(np.abs(out - ref)) < 3e-13
    assert r.F == pytest.approx(oracle.F(out), abs=1e-14)
    assert r.theta == pytest.approx(oracle.theta(out), rel=1e-12)
    mu, md = oracle.unitarity(out)
    assert mu < 1e-13 and md < 1e-13


@pytest.mark.parametrize("L", [(16, 16, 16, 12), (16, 8, 8, 48)])
def test_fp32_field(lgf_gpu, L):
    """The FP32 Fourier field perturbs one sweep by less than 1e-5, on the gauge orbit."""
    U, _ = inputs.make_config(L, 0.5, 800 + sum(L))
    Ug = gpu(U)
    lgf_gpu.iterate(Ug, ALPHA, 1, field_bits=32)
    out = cpu(Ug)
    assert np.max(np.abs(out - oracle.iterate(U, ALPHA, 1))) < 1e-5
    assert abs(oracle.plaquette(out) - oracle.plaquette(U)) < 1e-13
    mu, md = oracle.unitarity(out)
    assert mu < 1e-13 and md < 1e-13


@pytest.mark.parametrize("L", [(4, 4, 4, 4), (16, 16, 16, 12)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_no_sweep_leaves_the_links(lgf_gpu, L, precision):
    """No update (max_iter 0, or 0 sweeps): the transformation is the identity
    although no sweep has written it.  Row 2 is rebuilt to one rounding."""
    U, _ = inputs.make_config(L, 0.5, 900 + sum(L))
    for call in (lambda V: lgf_gpu.fix(V, ALPHA, 1e-15, precision=precision, max_iter=0),
                 lambda V: lgf_gpu.iterate(V, ALPHA, 0, precision=precision)):
        Ug = gpu(U)
        lgf_gpu.iterate(Ug, ALPHA, 2, precision=precision)  # leaves another G behind
        Ug = gpu(U)
        r = call(Ug)
        assert r.iterations == 0
        assert np.max(np.abs(cpu(Ug) - U)) < 1e-14


def test_resume_to_rounding(lgf_gpu):
    """2 + 3 sweeps equal 5 to the rounding of the links between them."""
    U, _ = inputs.make_config((16, 16, 16, 12), 0.5, 901)
    a, b = gpu(U), gpu(U)
    lgf_gpu.iterate(a, ALPHA, 5)
    lgf_gpu.iterate(b, ALPHA, 2)
    lgf_gpu.iterate(b, ALPHA, 3)
    assert np.max(np.abs(cpu(a) - cpu(b))) < 5e-13


# from 524288 sites the links are shared through LDS (blocks of 64 xy-sites x 4
# t): rows of one block, rows that straddle blocks, rows longer than a block;
# one row below the rule's volume
@pytest.mark.parametrize("L", [(64, 32, 16, 16), (48, 32, 8, 48), (128, 16, 16, 16),
                               (64, 32, 16, 12)])
def test_three_sweeps_shared_links(lgf_gpu, L):
    test_three_sweeps(lgf_gpu, L, {})


def test_exact_step_needs_no_memory_of_its_own(lgf_gpu):
    """G takes the exponential inside the pass that accumulates it; the buffer
    for it comes with a format whose sweeps store their links."""
    import torch

    L = (32, 32, 16, 16)
    U, _ = inputs.make_config(L, 0.5, 902)
    ctx = lgf_gpu.Context(L, "fp64")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx.set_exponential(True)
    assert torch.cuda.mem_get_info()[0] == free
    a, b = gpu(U), gpu(U)
    ctx.iterate(a, ALPHA, 2)
    ctx.set_link_format(18)
    ctx.iterate(b, ALPHA, 2)
    ctx.close()
    assert np.max(np.abs(cpu(a) - cpu(b))) < 3e-13


# one shape per path whose blocks exchange data through LDS: the update of each
# thread's own links after blocks that end in part of a wave, the FP64 and FP32
# updates that share links, (x,y) planes of the four fields in LDS
@pytest.mark.parametrize("L", [(27, 9, 16, 18), (48, 32, 8, 48), (64, 12, 8, 8)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_runs_are_bitwise_equal(lgf_gpu, L, precision):
    U, _ = inputs.make_config(L, 0.5, 950 + sum(L))
    a, b = gpu(U), gpu(U)
    ra = lgf_gpu.iterate(a, ALPHA, 4, precision=precision)
    rb = lgf_gpu.iterate(b, ALPHA, 4, precision=precision)
    assert np.array_equal(cpu(a), cpu(b))
    assert ra.F == rb.F and ra.theta == rb.theta


@pytest.mark.parametrize("kw", [{"exact_exp": True}, {"accelerate": False}])
def test_shared_links_step_options(lgf_gpu, kw):
    test_three_sweeps(lgf_gpu, (48, 32, 8, 48), kw)


def test_shared_links_fp32_field(lgf_gpu):
    test_fp32_field(lgf_gpu, (64, 32, 16, 16))
