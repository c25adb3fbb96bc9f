"""Whole-state transforms at every length along each axis, forward and inverse:
lines that share a wave, blocks of rows, tiles that a
line of 40 points fills in part.

One transform against NumPy's in double, one kinetic term against the FP64
oracle's: 1e-12 of the largest value in double and 2e-6 in single precision,
the tolerances of the other one-step tests."""
import numpy as np
import pytest

import swf_workloads as W
from oracle.swf import SWFSolve

pytestmark = pytest.mark.gpu

LENGTHS = [16, 32, 40, 48, 64, 80, 96, 128, 160, 192, 256, 320, 384, 512, 768, 1024]
TOL = {"fp64": 1e-12, "mixed": 2e-6}


@pytest.fixture(scope="module")
def S():
    from paper_2512_16889_amd import swf
    return swf


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("n", LENGTHS)
def test_every_length_along_each_axis(S, n, axis):
    shape = [40, 16, 16]
    shape[axis] = n
    grid = W.Grid(3, shape, [m / 4.0 for m in shape])
    field = [[W.Term(0, 0.3, W.gauss(1.0), [W.sech2(3.0), W.const(), W.const()])]]
    prob = W.Problem("transforms", [grid], field, [W.Solve(W.U_OUT, 1, [0.3, -0.2, 0.4])], W.Window(-1.0, 1.0, 0.05))
    sv = SWFSolve(prob, 0)
    psi = W.random_state([4] + shape, seed=3)
    fwd = np.fft.fftn(psi, axes=(1, 2, 3))
    kin = sv.kinetic(psi)
    for prec, tol in TOL.items():
        with S.Context(prob, precision=prec) as ctx:
            for op, ref in ((0, fwd), (1, kin)):
                err = np.abs(ctx.apply_op(op, 0, psi) - ref).max() / np.abs(ref).max()
                assert err < tol, (shape, prec, op, err)


@pytest.mark.parametrize("n", LENGTHS)
def test_kinetic_term_in_two_dimensions(S, n):
    """y is the last axis here: its pass multiplies by H0 between the transforms."""
    shape = [40, n]
    grid = W.Grid(2, shape + [1], [m / 4.0 for m in shape] + [1.0])
    field = [[W.Term(0, 0.3, W.gauss(1.0), [W.sech2(3.0), W.const(), W.const()])]]
    prob = W.Problem("transforms", [grid], field, [W.Solve(W.U_OUT, 1, [0.3, -0.2, 0.4])], W.Window(-1.0, 1.0, 0.05))
    psi = W.random_state([4] + shape, seed=4)
    ref = SWFSolve(prob, 0).kinetic(psi)
    for prec, tol in TOL.items():
        with S.Context(prob, precision=prec) as ctx:
            err = np.abs(ctx.apply_op(1, 0, psi) - ref).max() / np.abs(ref).max()
            assert err < tol, (shape, prec, err)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_batches_beyond_the_cache(S, prec):
    """Whole-state passes over more than 128 MB stream past the caches: the
    interaction-picture steps of four 1024^2 solves (268 MB, 134 MB in single
    precision) are those of one, bit for bit (the same operations)."""
    shape = [1024, 1024]
    grid = W.Grid(2, shape + [1], [m / 4.0 for m in shape] + [1.0], absorb_cells=8, absorb_strength=0.2)
    field = [[W.Term(0, 0.3, W.gauss(1.0), [W.sech2(3.0), W.const(), W.const()])]]
    psi = W.random_state([4] + shape, seed=6)
    out = []
    for count in (1, 4):
        solves = [W.Solve(W.U_OUT, 1, [0.3, -0.2, 0.4]) for _ in range(count)]
        prob = W.Problem("stream", [grid], field, solves, W.Window(-1.0, 1.0, 0.05, "iprk4"))
        with S.Context(prob, precision=prec) as ctx:
            for i in range(count):
                ctx.set_psi(i, psi, 0)
            ctx.step(2)
            out += [ctx.get_psi(i) for i in (0, count - 1)]
    assert np.abs(out[0]).max() > 0
    for other in out[1:]:
        assert np.array_equal(out[0], other)
