"""GPU tests of the core-number kernel's level steps: cascades inside one
workgroup, cascades that overflow its list, vertices handed to the grid, and
graphs of almost only isolated vertices.  Expected core numbers are closed
forms, so every comparison is exact."""
import numpy as np
import pytest

from gpu_util import edges_graph, lib, say

pytestmark = pytest.mark.gpu


def _cores(n, s, d):
    got, cmax = lib().truss_core_numbers(edges_graph(n, s, d))
    return got.cpu().numpy(), cmax


@pytest.mark.parametrize("n", [2, 3, 1025, 20001])
def test_path_cascade(n):
    """A path: level 1 eats it from both ends, one vertex at a time."""
    say(f"case: path of {n}")
    got, cmax = _cores(n, np.arange(n - 1, dtype=np.int32), np.arange(1, n, dtype=np.int32))
    assert (got == 1).all() and cmax == 1


@pytest.mark.parametrize("a", [70, 1500, 6000])
def test_bipartite_less_one_edge(a):
    """K_{a,a} less one edge: level a - 1 takes two vertices, whose removal takes all others at
    once: at a = 6000 more than a workgroup's list holds."""
    torch = pytest.importorskip("torch")
    T = lib()
    say(f"case: K_{a},{a} less one edge")
    i = torch.arange(1, a * a, device="cuda:0", dtype=torch.int64)
    g = T.Graph.from_edges(2 * a, i // a, i % a + a)
    got, cmax = T.truss_core_numbers(g)
    assert bool((got == a - 1).all()) and cmax == a - 1


@pytest.mark.parametrize("n,k", [(50, 7), (300000, 7), (3000000, 40)])
def test_mostly_isolated(n, k):
    """K_k among isolated vertices: no room for live lists beside the graph."""
    say(f"case: K_{k} and {n - k} isolated vertices")
    ids = np.random.default_rng(n).permutation(n)[:k].astype(np.int32)
    i, j = np.triu_indices(k, 1)
    got, cmax = _cores(n, ids[i], ids[j])
    want = np.zeros(n, np.int32)
    want[ids] = k - 1
    np.testing.assert_array_equal(got, want)
    assert cmax == k - 1


def test_binary_tree_and_star():
    say("case: binary tree, star")
    n = 100001
    v = np.arange(1, n, dtype=np.int32)
    got, cmax = _cores(n, (v - 1) // 2, v)
    assert (got == 1).all() and cmax == 1
    got, cmax = _cores(n, np.zeros(n - 1, np.int32), v)
    assert (got == 1).all() and cmax == 1
