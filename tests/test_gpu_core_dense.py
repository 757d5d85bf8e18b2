"""GPU tests of core numbers where one level takes a dense part of the graph at
once: rows that add up to just under and over what a workgroup walks itself
(65536 entries), lists cut part of the way, and hubs with long rows of leaves.
Expected core numbers are closed forms."""
import numpy as np
import pytest

from gpu_util import dev, lib, say

pytestmark = pytest.mark.gpu


def _cores(n, s, d):
    T = lib()
    got, cmax = T.truss_core_numbers(T.Graph.from_edges(n, dev(s.astype(np.int32)), dev(d.astype(np.int32))))
    return got.cpu().numpy(), cmax


@pytest.mark.parametrize("k", [255, 256, 257, 1024, 1025, 2049, 3000])
def test_complete(k):
    say(f"case: K_{k}")
    got, cmax = _cores(k, *np.triu_indices(k, 1))
    assert (got == k - 1).all() and cmax == k - 1


@pytest.mark.parametrize("k,leaves", [(64, 1000), (65, 1009), (1100, 60), (20, 30000)])
def test_hubs_with_leaves(k, leaves):
    """K_k, each of its vertices joined to leaves of its own."""
    say(f"case: K_{k} with {leaves} leaves a vertex")
    i, j = np.triu_indices(k, 1)
    n = k + k * leaves
    s = np.concatenate([i, np.repeat(np.arange(k), leaves)])
    d = np.concatenate([j, np.arange(k, n)])
    ids = np.random.default_rng(k).permutation(n)
    got, cmax = _cores(n, ids[s], ids[d])
    want = np.ones(n, np.int32)
    want[ids[:k]] = k - 1
    np.testing.assert_array_equal(got, want)
    assert cmax == k - 1


@pytest.mark.parametrize("n,r", [(3000, 40), (300001, 9), (1000003, 3)])
def test_ring(n, r):
    """Every vertex joined to the r next ones: one level takes all of them."""
    say(f"case: ring of {n}, {r} neighbours on each side")
    i = np.arange(n)
    got, cmax = _cores(n, np.tile(i, r), np.concatenate([(i + q) % n for q in range(1, r + 1)]))
    assert (got == 2 * r).all() and cmax == 2 * r
