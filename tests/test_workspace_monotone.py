"""CPU tests of the workspace queries: a graph with no more vertices and edges
never needs more, so a workspace sized for the largest graph serves them all."""
import ctypes
import random

import numpy as np
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


def _batch_size(T, sizes):
    b = ctypes.c_size_t(0)
    vo, eo = (np.concatenate([[0], np.cumsum(x)]).astype(np.int64) for x in zip(*sizes))
    assert T.load_library().truss_batch_workspace_size(len(sizes), vo.ctypes.data, eo.ctypes.data, None,
                                                       ctypes.byref(b)) == 0
    return b.value


@pytest.mark.parametrize("top", [(300, 2000), (8192, 1 << 18), (20000, 1 << 20)])
def test_batch_grows_with_its_graphs(top):
    """Up to, at and beyond the sizes of the compact kernel; all below those of the device-wide path."""
    import paper_1205_6693_amd as T
    rng = random.Random(top[0])
    for _ in range(300):
        sizes = [(rng.randint(1, top[0]), rng.randint(0, top[1])) for _ in range(rng.choice([1, 2, 40, 1500]))]
        size = _batch_size(T, sizes)
        i = rng.randrange(len(sizes))
        n, m = sizes[i]
        for more in ((n + 1, m), (n, m + 1), (max(n, 8193), m), (n, max(m, (1 << 18) + 1)), (n + n // 9, m + m // 9)):
            assert _batch_size(T, sizes[:i] + [more] + sizes[i + 1:]) >= size, (sizes[i], more)
        assert _batch_size(T, sizes + [(5, 5)]) >= size
