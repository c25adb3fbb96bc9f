"""The stage row pass at every x length: lines that share a wave (16 to 320
points of 2 to 16 threads a component), fill one (256, 384) or four (512 to
1024); a single line (most of a workgroup idle), a partial last workgroup, and
fields that use each coupling alone and all of them (the pass skips the
components no term has).

One step from a random state against the FP64 oracle: 1e-12 of the largest
value in double (rounding of 1024-point transforms is a few 1e-15), 2e-6 in
single precision, the tolerances of the other one-step tests."""
import numpy as np
import pytest

import swf_workloads as W
from oracle.swf import SWFSolve

from swf_cases import field_mix

pytestmark = pytest.mark.gpu

LENGTHS = [16, 32, 40, 48, 64, 80, 96, 128, 160, 192, 256, 320, 384, 512, 768, 1024]
TOL = {"fp64": 1e-12, "mixed": 2e-6}


@pytest.fixture(scope="module")
def S():
    from paper_2512_16889_amd import swf
    return swf


def check(S, prob, prec, steps=1):
    k0 = prob.window.steps // 2
    shape = tuple(prob.grids[0].n[:prob.grids[0].dim])
    states = [W.random_state((4,) + shape, seed=5 + i, scale=0.1) for i in range(len(prob.solves))]
    with S.Context(prob, precision=prec, persistent=False) as ctx:
        for i, psi in enumerate(states):
            ctx.set_psi(i, psi, k0)
        ctx.step(steps)
        for i, psi in enumerate(states):
            ref = SWFSolve(prob, i).run(psi, start=k0, count=steps)
            err = np.abs(ctx.get_psi(i) - ref).max() / np.abs(ref).max()
            assert err < TOL[prec], (shape, i, err)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", LENGTHS)
def test_every_length_one_line_and_a_partial_workgroup(S, n, prec):
    L = n / 4.0
    for grid in (W.Grid(1, [n, 1, 1], [L, 1.0, 1.0]), W.Grid(2, [n, 40, 1], [L, 10.0, 1.0])):
        solves = [W.Solve(W.U_OUT, 1, [0.3, -0.2, 0.4]), W.Solve(W.V_OUT, -1, [-0.1, 0.25, 0.3])]
        check(S, W.Problem("row", [grid], [field_mix(grid.dim)], solves, W.Window(-1.0, 1.0, 0.05)), prec)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("mus", [(), (0,), (1,), (2,), (3,), (0, 2), (3, 1)])
def test_every_coupling(S, mus, prec):
    # solves with different fields share the launch
    g = W.Grid(3, [48, 16, 40], [12.0, 5.0, 10.0])
    fx = [W.gauss(3.0), W.sech2(2.0), W.gauss(2.5)]
    fields = [[W.Term(m, 0.5 + 0.1 * m, W.gauss(1.0, c=0.1 * m), fx) for m in mus], field_mix(3)]
    solves = [W.Solve(W.U_OUT, 1, [0.3, -0.2, 0.4], 0, 0), W.Solve(W.V_OUT, 1, [0.1, 0.2, 0.4], 0, 1)]
    check(S, W.Problem("mu", [g], fields, solves, W.Window(-1.0, 1.0, 0.05)), prec, steps=2)
