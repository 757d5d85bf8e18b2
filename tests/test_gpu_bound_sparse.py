"""GPU tests of the upper bound psi on sparse graphs, in the workspace that the
size query states, against the oracle, bit-exact."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_util import csr_graph, edges_graph, lib, say

pytestmark = pytest.mark.gpu


def _distinct(n, u, v):
    lo, hi = np.minimum(u, v).astype(np.int64), np.maximum(u, v).astype(np.int64)
    key = np.unique((lo * n + hi)[lo < hi])
    return (key // n).astype(np.int32), (key % n).astype(np.int32)


def _graph(kind, n):
    v = np.arange(1, n, dtype=np.int64)
    if kind == "path":
        return _distinct(n, v - 1, v)
    if kind == "tree":
        return _distinct(n, (v - 1) // 2, v)
    if kind == "star":
        return _distinct(n, np.zeros(n - 1, np.int64), v)
    if kind == "one triangle":
        return _distinct(n, np.array([0, 0, n - 2]), np.array([n - 2, n - 1, n - 1]))
    if kind == "strip":  # triangles side by side: mean degree 4, every edge in one or two
        return _distinct(n, np.concatenate([v - 1, v[1:] - 2]), np.concatenate([v, v[1:]]))
    # a mean degree of 2, 4 or 8 at random, with a hub that has a long row
    rng = np.random.default_rng(n)
    u, w = (rng.integers(0, n, int(kind) * n // 2) for _ in range(2))
    hub = rng.choice(n, 500, replace=False)
    return _distinct(n, np.concatenate([u, np.full(500, 7)]), np.concatenate([w, hub]))


@pytest.mark.parametrize("n", [1500, 100003])
@pytest.mark.parametrize("kind", ["path", "tree", "star", "one triangle", "strip", "2", "4", "8"])
def test_upper_bound(kind, n):
    T = lib()
    s, d = _graph(kind, n)
    say(f"case: psi, {kind}, {n} vertices, {s.size} edges")
    ss, dd = graphgen.shuffle(s, d, 5)
    for g, a, b in ((edges_graph(n, ss, dd), ss, dd), (csr_graph(n, s, d), s, d)):
        got = T.truss_upper_bound(g, ws=T.workspace(g)).cpu().numpy()
        np.testing.assert_array_equal(got, oracle.upper_bound(n, a, b))
        got, kmin, kmax, _ = T.truss_topdown(g, 2)
        phi, top = oracle.truss(n, a, b)
        assert kmax == top
        np.testing.assert_array_equal(got.cpu().numpy(), np.where(phi >= kmin, phi, 0))
