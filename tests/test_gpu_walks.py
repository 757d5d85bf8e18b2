"""GPU tests of the peeling rounds' split into parts: frontiers whose walks are
all of one entry, fill a part exactly, or run over many parts and record
chunks.  Expected truss numbers are closed forms, so every comparison is exact."""
import numpy as np
import pytest

from gpu_util import edges_graph, gpu_truss, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaves", [1, 255, 256, 257, 1023, 1025, 65535, 65537, 300001, 5000000])
def test_star_one_entry_walks(leaves):
    """A star: one round whose walks are one entry each, as many records as entries."""
    say(f"case: star with {leaves} leaves")
    s = np.zeros(leaves, np.int32)
    d = np.arange(1, leaves + 1, dtype=np.int32)
    for mode in (1, 2):
        got, st = gpu_truss(edges_graph(leaves + 1, s, d), peel_mode=mode)
        assert (got == 2).all() and st["peel_work"] == leaves and st["subrounds"] == 1


@pytest.mark.parametrize("pages", [1, 2, 127, 128, 129, 513, 4097, 200001])
@pytest.mark.parametrize("shape", [1, 2])
def test_book(pages, shape):
    """Triangles sharing one edge: 2-entry walks beside one of all pages; every edge has truss number 3."""
    say(f"case: book with {pages} pages, shape {shape}")
    v = np.arange(2, pages + 2, dtype=np.int32)
    s = np.concatenate([[0], np.zeros(pages), np.ones(pages)]).astype(np.int32)
    d = np.concatenate([[1], v, v]).astype(np.int32)
    got, st = gpu_truss(edges_graph(pages + 2, s, d), peel_shape=shape)
    assert (got == 3).all() and st["triangles"] == pages and st["kmax"] == 3


@pytest.mark.parametrize("k,copies", [(3, 100000), (17, 5000), (90, 300)])
def test_disjoint_cliques_one_round(k, copies):
    """copies of K_k: one round with equal walks of k - 1 entries, over many parts."""
    say(f"case: {copies} x K_{k}")
    i, j = np.triu_indices(k, 1)
    base = (np.arange(copies, dtype=np.int64) * k)[:, None]
    s, d = (base + i).ravel().astype(np.int32), (base + j).ravel().astype(np.int32)
    for probe in (1, 2):
        got, st = gpu_truss(edges_graph(k * copies, s, d), peel_probe=probe)
        assert (got == k).all() and st["peel_work"] == s.size * (k - 1)
