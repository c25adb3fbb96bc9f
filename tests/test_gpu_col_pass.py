"""The stepping column passes at every length and tile width, along y and along
z: tiles that share a wave, partial tiles (a row of 40 points against tiles of
8 to 64 columns), one workgroup and many.

One step from a random state against the FP64 oracle, 1e-12 of the largest
value in double and 2e-6 in single precision, the tolerances of the other
one-step tests."""
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


@pytest.mark.parametrize("axis", [1, 2])
@pytest.mark.parametrize("n", LENGTHS)
def test_every_length_and_tile_width(S, n, axis):
    shape = [40, n] if axis == 1 else [40, 16, n]
    dim = len(shape)
    grid = W.Grid(dim, shape + [1] * (3 - dim), [m / 4.0 for m in shape] + [1.0] * (3 - dim))
    solves = [W.Solve(W.U_OUT, 1, [0.3, -0.2, 0.4]), W.Solve(W.V_OUT, -1, [-0.1, 0.25, 0.3])]
    prob = W.Problem("col", [grid], [field_mix(dim)], solves, W.Window(-1.0, 1.0, 0.05))
    k0 = prob.window.steps // 2
    states = [W.random_state([4] + shape, seed=5 + i, scale=0.1) for i in range(2)]
    refs = [SWFSolve(prob, i).step(k0, psi) for i, psi in enumerate(states)]
    for prec in ("fp64", "mixed"):
        for variant in (None, 0, 1, 2):
            with S.Context(prob, precision=prec, variant=variant) as ctx:
                for i, psi in enumerate(states):
                    ctx.set_psi(i, psi, k0)
                ctx.step(1)
                for i in range(2):
                    err = np.abs(ctx.get_psi(i) - refs[i]).max() / np.abs(refs[i]).max()
                    assert err < TOL[prec], (shape, prec, variant, i, err)
