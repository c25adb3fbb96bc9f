"""Breit-Wheeler stage sums of every group shape (one or two U solves with one
or two V solves that share a photon), each of which a wave sums in its own
number of exchanges, on a lattice with a remainder and on one that takes
several sites per thread (each one's states loaded an iteration ahead).

The first stage-complete integrals against the FP64 oracle at 1e-12 of the
largest (up to 5e5 products added in double), and single precision at 2e-6."""
import numpy as np
import pytest

import swf_workloads as W
from oracle import bw as obw

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_2512_16889_amd import swf
    return swf


@pytest.mark.parametrize("shape", [[320], [768, 768]])
@pytest.mark.parametrize("nu,nv", [(1, 1), (1, 2), (2, 1), (2, 2)])
def test_group_shapes(S, nu, nv, shape):
    dim = len(shape)
    grid = W.Grid(dim, shape + [1] * (3 - dim), [n / 2.0 for n in shape] + [1.0] * (3 - dim))
    field = [W.Term(1, 0.7, W.gauss(2.0), [W.gauss(5.0), W.const(), W.const()])]
    k, eps = [0.0, 0.0, 1.3], [-1.0, 0.2, 0.0]
    spins = [1, -1]
    solves = [W.Solve(W.U_OUT, spins[i], [0.2, 0.0, 0.7]) for i in range(nu)]
    solves += [W.Solve(W.V_OUT, spins[i], [-0.1, 0.0, 0.6]) for i in range(nv)]
    verts = [W.Vertex(u, nu + v, k, eps) for u in range(nu) for v in range(nv)]
    prob = W.Problem("shapes", [grid], [field], solves, W.Window(-0.05, 0.05, 0.05), verts)
    refs = [obw.Vertex(prob, v).run()[2] for v in range(len(verts))]
    for prec, tol in (("fp64", 1e-12), ("mixed", 2e-6)):
        with S.Context(prob, precision=prec) as ctx:
            ctx.step()
            for v, ref in enumerate(refs):
                got = ctx.get_bw_state(v)
                assert np.abs(got - ref).max() <= tol * np.abs(ref).max(), (prec, v, got, ref)
