"""The 1D whole-loop kernel at the LDS limit: 1024 points in double with five
field terms, whose fifth profile takes 8 of the 9 KB that are left (162 816 of
163 840 bytes), and the pass path from six terms on, against the FP64 oracle.
Rounding as in the other line tests: 1e-12 of the largest value."""
import numpy as np
import pytest

import swf_workloads as W
from oracle.swf import SWFSolve

from swf_cases import field_mix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nterm,kernels", [(5, 1), (6, 0), (8, 0)])
def test_terms_that_fit(nterm, kernels):
    from paper_2512_16889_amd import swf as S
    n, steps = 1024, 17
    grid = W.Grid(1, [n, 1, 1], [n / 4.0, 1.0, 1.0], absorb_cells=4, absorb_strength=0.2)
    extra = [W.Term(j % 4, 0.05 * (j + 1), W.gauss(1.0 + 0.2 * j), [W.sech2(3.0 + j), W.const(), W.const()]) for j in range(3)]
    solves = [W.Solve(W.U_OUT, 1, [0.3, -0.2, 0.4]), W.Solve(W.V_OUT, -1, [-0.1, 0.25, 0.3])]
    prob = W.Problem("line", [grid], [(field_mix(1) + extra)[:nterm]], solves, W.Window(-1.0, 1.0, 0.05))
    states = [W.random_state((4, n), seed=19 + i, scale=0.1) for i in range(2)]
    with S.Context(prob, precision="fp64", profile=True) as ctx:
        for i, psi in enumerate(states):
            ctx.set_psi(i, psi, 2)
        ctx.step(steps)
        ctx.sync()
        assert ctx.kernel_stats(5)[0] == kernels
        for i, psi in enumerate(states):
            ref = SWFSolve(prob, i).run(psi, start=2, count=steps)
            err = np.abs(ctx.get_psi(i) - ref).max() / np.abs(ref).max()
            assert err < 1e-12, (nterm, i, err)
