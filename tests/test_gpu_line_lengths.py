"""The 1D whole-loop kernel at every line length (the smallest use part of a
wave, 48 to 320 one wave, 256 and 384 two, 512 to 1024 four), with step counts
on both sides of the block whose time factors are formed together, fields of one term, of
as many as a thread keeps in registers and of more, and the absorber, against
the FP64 oracle.  Rounding grows by about 1e-15 a step: 1e-12 of the largest
value in double, 1e-5 in single precision (the tolerances of the kernel's other
tests)."""
import numpy as np
import pytest

import swf_workloads as W
from oracle.swf import SWFSolve

from swf_cases import field_mix

pytestmark = pytest.mark.gpu

LENGTHS = [16, 32, 40, 48, 64, 80, 96, 128, 160, 192, 256, 320, 384, 512, 768, 1024]


@pytest.fixture(scope="module")
def S():
    from paper_2512_16889_amd import swf
    return swf


def fields(nterm):
    extra = [W.Term(j % 4, 0.05 * (j + 1), W.gauss(1.0 + 0.2 * j), [W.sech2(3.0 + j), W.const(), W.const()]) for j in range(3)]
    return (field_mix(1) + extra)[:nterm]


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("mixed", 1e-5)])
@pytest.mark.parametrize("n", LENGTHS)
def test_every_length(S, n, prec, tol):
    grid = W.Grid(1, [n, 1, 1], [n / 4.0, 1.0, 1.0], absorb_cells=4, absorb_strength=0.2)
    for nterm, steps in ((1, 1), (4, 16), (5, 17), (8, 35)):
        if n == 1024 and prec == "fp64" and nterm > 4:
            continue   # the further profiles do not fit the LDS: the pass path takes these
        solves = [W.Solve(W.U_OUT, 1, [0.3, -0.2, 0.4]), W.Solve(W.V_OUT, -1, [-0.1, 0.25, 0.3])]
        prob = W.Problem("line", [grid], [fields(nterm)], solves, W.Window(-1.0, 1.0, 0.05))
        states = [W.random_state((4, n), seed=9 + i, scale=0.1) for i in range(2)]
        with S.Context(prob, precision=prec, profile=True) as ctx:
            for i, psi in enumerate(states):
                ctx.set_psi(i, psi, 2)
            ctx.step(steps)
            ctx.sync()
            assert ctx.kernel_stats(5)[0] == 1, (n, nterm)
            for i, psi in enumerate(states):
                ref = SWFSolve(prob, i).run(psi, start=2, count=steps)
                err = np.abs(ctx.get_psi(i) - ref).max() / np.abs(ref).max()
                assert err < tol, (n, nterm, steps, i, err)
