"""GPU tests of invalid input whose error is read only with the results: the
code of every entry point, the output left as it was, and a correct run in the
same workspace afterwards."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_util import dev, edges_graph, lib, say

pytestmark = pytest.mark.gpu


def _bad_edge_lists(n, s, d):
    """(name, n, src, dst, code) of edge lists with one or several faults."""
    T = lib()
    a, b = s.copy(), d.copy()
    yield "repeated", n, np.append(a, b[5]).astype(np.int32), np.append(b, a[5]).astype(np.int32), T.E_DUP
    yield "loop", n, np.append(a, 7).astype(np.int32), np.append(b, 7).astype(np.int32), T.E_SELFLOOP
    yield "range", n, np.append(a, n).astype(np.int32), np.append(b, 0).astype(np.int32), T.E_RANGE
    yield "negative", n, np.append(a, -3).astype(np.int32), np.append(b, 0).astype(np.int32), T.E_RANGE
    yield "loop and repeated", n, np.append(a, [4, a[0]]).astype(np.int32), np.append(b, [4, b[0]]).astype(
        np.int32), T.E_SELFLOOP
    yield "all", n, np.append(a, [4, a[0], n + 9]).astype(np.int32), np.append(b, [4, b[0], 1]).astype(
        np.int32), T.E_RANGE
    yield "every pair the same", n, np.zeros(5000, np.int32), np.ones(5000, np.int32), T.E_DUP
    yield "no vertices", 0, a, b, T.E_RANGE


@pytest.mark.parametrize("scale", [9, 16])
def test_edge_lists(scale):
    """Below and above the size from which rows are compacted."""
    torch = pytest.importorskip("torch")
    T = lib()
    n, s, d = graphgen.rmat(scale, 8, 3)
    ref = oracle.truss(n, s, d)[0]
    good = edges_graph(n, s, d)
    for name, bn, bs, bd, code in _bad_edge_lists(n, s, d):
        say(f"case: {name}, {bs.size} pairs")
        g = T.Graph.from_edges(bn, dev(bs), dev(bd))
        out = torch.full((bs.size,), -7, dtype=torch.int32, device="cuda:0")
        ws = torch.empty(T.truss_workspace_size(g) + T.truss_workspace_size(good), dtype=torch.uint8, device="cuda:0")
        for call in (lambda: T.truss_decompose(g, out=out, ws=ws), lambda: T.truss_support(g, out=out, ws=ws),
                     lambda: T.truss_upper_bound(g, out=out, ws=ws), lambda: T.truss_topdown(g, 2, out=out),
                     lambda: T.truss_cohen(g)):
            with pytest.raises(T.TrussError) as ex:
                call()
            assert ex.value.code == code
            assert bool((out == -7).all())
        got, _ = T.truss_decompose(good, ws=ws)
        np.testing.assert_array_equal(got.cpu().numpy(), ref)


@pytest.mark.parametrize("scale", [9, 16])
def test_csr(scale):
    torch = pytest.importorskip("torch")
    T = lib()
    n, s, d = graphgen.rmat(scale, 8, 4)
    rp, col = graphgen.to_csr(n, s, d)
    row = int(np.argmax(np.diff(rp)))
    at = int(rp[row])
    lone = int(np.argmax(np.diff(rp) > 0))
    cases = []
    c = col.copy(); c[at + 1] = c[at]; cases.append(("repeated", c, T.E_DUP))
    c = col.copy(); c[at], c[at + 1] = c[at + 1], c[at]; cases.append(("unsorted", c, T.E_UNSORTED))
    c = col.copy(); c[at] = row; cases.append(("loop", c, T.E_SELFLOOP))
    c = col.copy(); c[at] = n; cases.append(("range", c, T.E_RANGE))
    c = col.copy(); c[at] = -1; cases.append(("negative", c, T.E_RANGE))
    # another neighbour in place of the last one of a row: sorted, but not symmetric
    c = col.copy()
    e = int(rp[lone + 1]) - 1
    free = [x for x in range(int(c[e]) + 1, n) if x != lone]
    c[e] = free[0]
    cases.append(("asymmetric", c, T.E_ASYM))
    for name, c, code in cases:
        say(f"case: CSR {name}, {c.size} entries")
        g = T.Graph.from_csr(n, dev(rp), dev(c))
        out = torch.full((c.size // 2,), -7, dtype=torch.int32, device="cuda:0")
        for call in (lambda: T.truss_decompose(g, out=out), lambda: T.truss_support(g, out=out),
                     lambda: T.truss_upper_bound(g, out=out), lambda: T.truss_core_numbers(g)):
            with pytest.raises(T.TrussError) as ex:
                call()
            assert ex.value.code == code, name
            assert bool((out == -7).all())
