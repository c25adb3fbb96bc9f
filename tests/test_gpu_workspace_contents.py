"""A context clears psi_s alone of its state arrays, at init and at reset: the
stage inputs, accumulators, slopes and transform buffers are written before they
are read.  With a workspace full of NaN, and after a run whose every array holds
NaN, a job gives bit for bit what it gives in a cleared workspace."""
import numpy as np
import pytest
import torch

import swf_workloads as W

import swf_cases as cases

pytestmark = pytest.mark.gpu

STEPS = 4


@pytest.fixture(scope="module")
def S():
    from paper_2512_16889_amd import swf
    return swf


def problem(dim, scheme, vertices):
    n = {1: [48], 2: [40, 32], 3: [16, 40, 32]}[dim]
    L = [0.5 * k for k in n]
    grid = W.Grid(dim, n + [1] * (3 - dim), L + [1.0] * (3 - dim), absorb_cells=4, absorb_strength=0.2)
    p, q = [0.2, 0.0, 0.7], [-0.2, 0.0, 0.6]
    if not vertices:
        q = [-0.2, 0.0, -0.7]
    solves = [W.Solve(W.U_OUT, 1, p), W.Solve(W.U_OUT, -1, p), W.Solve(W.V_OUT, 1, q)]
    verts = []
    if vertices:
        k, eps = [0.0, 0.0, 1.3], [-1.0, 0.2, 0.0]
        packet = W.gaussian_packet([0.1, 0.0, 1.3], eps, 0, 0.05, 3, 0.04)
        verts = [W.Vertex(0, 2, k, eps), W.Vertex(1, 2, k, eps)]
        if vertices == "packet":
            verts.append(W.Vertex(0, 2, k, eps, modes=packet))
    return W.Problem("fill", [grid], [cases.field_mix(dim)], solves, W.Window(-0.1, 0.1, 0.05, scheme), verts)


def results(ctx, prob, partial):
    out = [ctx.get_psi(i) for i in range(3)] + [np.array(ctx.diagnostics(i)) for i in range(3)]
    out.append(np.array([ctx.marginal(i) for i in range(3)]))
    if prob.vertices:
        out += [np.array([ctx.bw(v), *ctx.get_bw_state(v)]) for v in range(len(prob.vertices))]
        if partial:
            out.append(np.array([ctx.bw_partial(v) for v in range(len(prob.vertices))]))
    else:
        out.append(ctx.pair_matrix([0, 1], [2]))
    return out


def run(S, monkeypatch, prob, fill, **kw):
    """Results of the job in a workspace of bytes `fill`, of the same job after a run in NaN and a reset, and of the
    three operator hooks on a context of their own."""
    real = torch.empty

    def filled(*a, **k):
        t = real(*a, **k)
        t.fill_(fill)
        torch.cuda.synchronize()
        return t
    with monkeypatch.context() as m:
        m.setattr(S.torch, "empty", filled)
        first, hooks = S.Context(prob, **kw), S.Context(prob, **kw)
    with first as ctx:
        ctx.step()
        out = results(ctx, prob, kw.get("bw_partial"))
        if fill:
            nan = np.full((4, *[n for n in prob.grids[0].n[:prob.grids[0].dim]]), np.nan, dtype=complex)
            for i in range(3):
                ctx.set_psi(i, nan, 0)
            ctx.step()
            ctx.sync()
            ctx.reset()
            ctx.step()
            again = results(ctx, prob, kw.get("bw_partial"))
            assert all(np.array_equal(a, b) for a, b in zip(out, again))
    with hooks as ctx:
        psi = W.random_state((4, *prob.grids[0].n[:prob.grids[0].dim]), seed=3)
        out += [ctx.apply_op(op, 0, psi, 0.1) for op in (0, 1, 2)]
    return out


CASES = [(d, s, v, {}) for d in (1, 2, 3) for s in ("rk4", "dp5", "iprk4") for v in ("", "packet")] + \
        [(1, "rk4", "", {"persistent": False}), (2, "rk4", "plane", {"bw_partial": True}), (3, "rk4", "plane", {"bw_partial": True}),
         (3, "rk4", "", {"batched": False}), (2, "dp5", "", {"use_graph": True}), (2, "rk4", "", {"tune": True}),
         (3, "dp5", "", {"tune": True})]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("dim,scheme,vertices,kw", CASES)
def test_nan_in_the_workspace(S, monkeypatch, dim, scheme, vertices, kw, prec):
    prob = problem(dim, scheme, vertices)
    clean = run(S, monkeypatch, prob, 0, precision=prec, **kw)
    poisoned = run(S, monkeypatch, prob, 0xFF, precision=prec, **kw)
    assert all(np.all(np.isfinite(a)) for a in clean)
    for i, (a, b) in enumerate(zip(clean, poisoned)):
        assert np.array_equal(a, b), i
