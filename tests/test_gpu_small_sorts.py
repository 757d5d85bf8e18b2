"""GPU tests of the builds around the sizes that are sorted in one workgroup: edge
counts beside the workgroup's item steps and its limit, in shuffled order.  Expected
truss numbers are closed forms."""
import numpy as np
import pytest

from gpu_util import canonical_sorted, csr_graph, edges_graph, gpu_support, gpu_truss, say

pytestmark = pytest.mark.gpu


def cliques_and_path(m, k, n_extra, seed):
    """m edges: as many K_k as fit into two thirds, the rest a path; ids and order shuffled."""
    rng = np.random.default_rng(seed)
    i, j = np.triu_indices(k, 1)
    copies = (2 * m // 3) // i.size
    base = (np.arange(copies) * k)[:, None]
    s, d = (base + i).ravel(), (base + j).ravel()
    rest = m - s.size
    v = copies * k + np.arange(rest)
    s, d = np.concatenate([s, v]), np.concatenate([d, v + 1])
    want = np.concatenate([np.full(copies * i.size, k), np.full(rest, 2)])
    n = copies * k + rest + 1 + n_extra
    ids = rng.permutation(n)
    order = rng.permutation(m)
    return n, ids[s][order].astype(np.int32), ids[d][order].astype(np.int32), want[order]


@pytest.mark.parametrize("m", [2, 63, 64, 65, 1023, 1024, 1025, 2049, 7169, 8191, 8192, 8193, 16385])
@pytest.mark.parametrize("k,n_extra", [(3, 0), (9, 40000)])
def test_shuffled_edges(m, k, n_extra):
    n, s, d, want = cliques_and_path(m, k, n_extra, m + k)
    say(f"case: {m} edges, K_{k}, {n} vertices")
    got, _ = gpu_truss(edges_graph(n, s, d))
    assert (got == want).all()
    sup, _ = gpu_support(edges_graph(n, s, d))
    assert (sup == want - 2).all()
    a, b, order = canonical_sorted(s, d)
    got, _ = gpu_truss(csr_graph(n, a, b))
    assert (got == want[order]).all()
