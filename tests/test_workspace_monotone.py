"""CPU tests of the workspace queries: a graph with no more vertices and edges
never needs more, so a workspace sized for the largest graph serves them all."""
import ctypes
import random

import pytest

QUERIES = ["truss_workspace_size", "truss_topdown_workspace_size", "truss_core_workspace_size",
           "truss_cohesion_workspace_size", "truss_cohen_workspace_size"]


def _size(T, query, n, m, fmt):
    g = T._Graph()
    g.n, g.m, g.fmt = n, m, fmt
    g.src = g.dst = g.row_ptr = g.col = 4096  # never dereferenced by the size query
    b = ctypes.c_size_t(0)
    fn = getattr(T.load_library(), query)
    opts = (None,) if query in ("truss_workspace_size", "truss_topdown_workspace_size") else ()
    assert fn(ctypes.byref(g), *opts, ctypes.byref(b)) == 0
    return b.value


@pytest.mark.parametrize("fmt", [0, 1], ids=["edges", "csr"])
@pytest.mark.parametrize("query", QUERIES)
def test_grows_with_the_graph(query, fmt):
    import paper_1205_6693_amd as T
    rng = random.Random(query + str(fmt))
    for _ in range(1500):
        n = int(2 ** rng.uniform(0, 24))
        m = int(n * 2 ** rng.uniform(-6, 6))
        size = _size(T, query, n, m, fmt)
        for dn, dm in ((1, 0), (0, 1), (n // 10, 0), (0, m // 1000), (0, m // 10), (n, m)):
            more = _size(T, query, n + dn, m + dm, fmt)
            assert more >= size, (n, m, dn, dm)
