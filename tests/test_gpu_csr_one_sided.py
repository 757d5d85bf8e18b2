"""GPU tests of CSR inputs that lack upper entries: asymmetric, whatever else the
missing entries would be taken for."""
import numpy as np
import pytest

from gpu_util import dev, lib, say

pytestmark = pytest.mark.gpu


def _csr(n, pairs):
    """CSR of the directed pairs (u, v): v is listed in row u."""
    pairs = sorted(pairs)
    rp = np.zeros(n + 1, np.int64)
    for u, _ in pairs:
        rp[u + 1] += 1
    return np.cumsum(rp), np.array([v for _, v in pairs], np.int32)


# (name, n, directed pairs): an even number of entries, sorted rows, no repeats
CASES = [
    ("lower halves alone", 4, [(1, 0), (2, 0), (2, 1), (3, 0), (3, 1), (3, 2)]),
    ("two upper entries missing", 5, [(0, 1), (1, 0), (2, 0), (2, 1), (3, 2), (4, 2), (4, 3), (3, 4)]),
    ("one upper entry missing", 4, [(0, 1), (1, 0), (2, 0), (2, 1), (1, 2), (3, 2)]),
    ("upper halves alone", 4, [(0, 1), (0, 2), (0, 3), (1, 2), (1, 3), (2, 3)]),
]


@pytest.mark.parametrize("name,n,pairs", CASES, ids=[c[0] for c in CASES])
def test_asymmetric(name, n, pairs):
    torch = pytest.importorskip("torch")
    T = lib()
    rp, col = _csr(n, pairs)
    g = T.Graph.from_csr(n, dev(rp), dev(col))
    for call in (T.truss_decompose, T.truss_support, T.truss_upper_bound, lambda g: T.truss_topdown(g, 2),
                 T.truss_core_numbers, T.truss_cohesion, T.truss_cohen):
        say(f"case: {name}")
        with pytest.raises(T.TrussError) as ex:
            call(g)
        assert ex.value.code == T.E_ASYM, name
