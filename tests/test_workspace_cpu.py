"""What a Breit-Wheeler vertex adds to the workspace: its tables and the partials
of its stage sums, whose number follows the lattice."""
import ctypes as C

import pytest

import swf_workloads as W


@pytest.fixture(scope="module")
def S():
    from paper_2512_16889_amd import swf
    return swf


def size(S, n, m, nverts, scheme):
    """m U and m V solves, the first nverts of their pairs as vertices."""
    dim = len(n)
    grid = W.Grid(dim, list(n) + [1] * (3 - dim), [k / 2.0 for k in n] + [1.0] * (3 - dim))
    field = [W.Term(1, 0.7, W.gauss(2.0), [W.gauss(5.0), W.const(), W.const()])]
    k, eps = [0.0, 0.0, 1.3], [-1.0, 0.2, 0.0]
    solves = [W.Solve(W.U_OUT, 1, [0.02 * i, 0.0, 0.7]) for i in range(m)]
    solves += [W.Solve(W.V_OUT, 1, [-0.02 * i, 0.0, 0.6]) for i in range(m)]
    verts = [W.Vertex(i // m, m + i % m, k, eps) for i in range(nverts)]
    return S.workspace_size(W.Problem("bytes", [grid], [field], solves, W.Window(-0.1, 0.1, 0.05, scheme), verts))


@pytest.mark.parametrize("scheme,stages", [("rk4", 4), ("dp5", 6), ("iprk4", 4)])
@pytest.mark.parametrize("n,m,most", [((512,), 16, 2), ((16,), 16, 1), ((128, 128), 8, 64), ((128, 128, 128), 4, 256)])
def test_bytes_per_vertex(S, n, m, most, scheme, stages):
    """`most` workgroups (one site per thread, 256 at most where four groups or more share a launch) leave three
    numbers per stage; the tables are exp(i k.x) of the vertex and at most four products of it per group (of one
    vertex at least), the descriptors under 1 KB."""
    tables = 5 * 16 * (sum(n) + 3 - len(n))
    per = (size(S, n, m, m * m, scheme) - size(S, n, m, 0, scheme)) / (m * m)
    assert 48 * stages * most <= per <= 48 * stages * most + tables + 1024
