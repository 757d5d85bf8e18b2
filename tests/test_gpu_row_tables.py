"""GPU tests of the row hash tables: rows that fill their table to its half, with
neighbours that hash to one bucket, so that lookups run over many buckets and
around the table's end.  Expected truss numbers are closed forms."""
import numpy as np
import pytest

from gpu_util import csr_graph, canonical_sorted, edges_graph, gpu_truss, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [2, 3, 4, 5, 9, 17, 33, 65, 129])
@pytest.mark.parametrize("peel_shape", [1, 2])
def test_cliques_of_colliding_ids(k, peel_shape):
    """Disjoint K_k whose members are neighbours in the order of the hash: all
    degrees are equal, so the ids keep their order, and the members' home buckets agree."""
    copies = 50
    n = k * copies
    hashed = np.argsort((np.arange(n, dtype=np.uint64) * 2654435769) & 0xFFFFFFFF, kind="stable")
    hashed = np.roll(hashed, k // 2)  # one clique holds both ends of the hash range
    i, j = np.triu_indices(k, 1)
    member = hashed.reshape(copies, k)
    s, d = member[:, i].ravel(), member[:, j].ravel()
    s, d, _ = canonical_sorted(s, d)
    say(f"case: {copies} x K_{k}, shape {peel_shape}")
    for g in (edges_graph(n, s, d), csr_graph(n, s, d)):
        for cut in (s.size, s.size - 1):
            if cut < s.size:
                if k < 4:
                    continue
                g = edges_graph(n, s[:cut], d[:cut])
            got, st = gpu_truss(g, peel_shape=peel_shape)
            want = np.full(cut, k)
            if cut < s.size:  # K_k without one edge: truss number k - 1
                u = int(s[-1])
                c = int(np.nonzero((member == u).any(1))[0][0])
                inside = np.isin(s[:cut], member[c])
                want[inside] = k - 1
            assert (got == want).all()
            assert st["triangles"] == copies * (k * (k - 1) * (k - 2) // 6) - (k - 2 if cut < s.size else 0)
