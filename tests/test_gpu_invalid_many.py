"""GPU tests of invalid input most of which is bad: ids beyond n, padding,
one pair over and over, a CSR of one half of its entries.  The later phases do
nothing for it (they would take time quadratic in the number of bad pairs), the
code comes back and the output is left as it was."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_util import dev, edges_graph, lib, say

pytestmark = pytest.mark.gpu

# 2 M pairs, and more than 2^23, from where the walks of a vertex with that many
# out-neighbours would no longer fit 32 bits
SIZES = [2000003, 9000001]


def _edge_lists(m):
    """(name, n, src, dst, code)"""
    T = lib()
    rng = np.random.default_rng(m)
    n = 300000
    u, v = (rng.integers(0, n, m).astype(np.int32) for _ in range(2))
    yield "n half as large", n // 2, u, v, T.E_RANGE
    yield "padding alone", n, np.full(m, -1, np.int32), np.full(m, -1, np.int32), T.E_RANGE
    a, b = u.copy(), v.copy()
    bad = rng.choice(m, 50000, replace=False)
    a[bad], b[bad] = -1, n
    yield "some padding", n, a, b, T.E_RANGE
    yield "one pair", n, np.full(m, 9, np.int32), np.full(m, 5, np.int32), T.E_DUP
    yield "one loop", n, np.full(m, 9, np.int32), np.full(m, 9, np.int32), T.E_SELFLOOP


def _check(g, code, good, ref):
    torch = pytest.importorskip("torch")
    T = lib()
    out = torch.full((g.m,), -7, dtype=torch.int32, device="cuda:0")
    ws = torch.empty(max(T.truss_workspace_size(g), T.truss_workspace_size(good)), dtype=torch.uint8,
                     device="cuda:0")
    for call in (lambda: T.truss_decompose(g, out=out, ws=ws),
                 lambda: T.truss_decompose(g, T.make_options(scheduler=T.SCHED_PLAIN), out=out, ws=ws),
                 lambda: T.truss_support(g, out=out, ws=ws), lambda: T.truss_upper_bound(g, out=out, ws=ws),
                 lambda: T.truss_topdown(g, 2, out=out), lambda: T.truss_cohen(g), lambda: T.truss_core_numbers(g)):
        with pytest.raises(T.TrussError) as ex:
            call()
        assert ex.value.code == code
        assert bool((out == -7).all())
    got, _ = T.truss_decompose(good, ws=ws)
    np.testing.assert_array_equal(got.cpu().numpy(), ref)


@pytest.mark.parametrize("m", SIZES)
def test_edge_lists(m):
    T = lib()
    n, s, d = graphgen.rmat(9, 8, 3)
    good, ref = edges_graph(n, s, d), oracle.truss(n, s, d)[0]
    for name, n, u, v, code in _edge_lists(m):
        say(f"case: {name}, {m} pairs")
        _check(T.Graph.from_edges(n, dev(u), dev(v)), code, good, ref)


@pytest.mark.parametrize("m", SIZES)
@pytest.mark.parametrize("which", ["lower", "upper", "either"])
def test_one_sided_csr(m, which):
    """Every pair listed once, in the row of its larger, smaller or either end."""
    T = lib()
    n, s, d = graphgen.rmat(9, 8, 3)
    good, ref = edges_graph(n, s, d), oracle.truss(n, s, d)[0]
    n = 100000
    rng = np.random.default_rng(m)
    u, v = (rng.integers(0, n, m + m // 8) for _ in range(2))
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique((lo * n + hi)[lo < hi])[:2 * (m // 2)]
    lo, hi = key // n, key % n
    flip = {"lower": np.ones(key.size, bool), "upper": np.zeros(key.size, bool),
            "either": rng.random(key.size) < 0.7}[which]
    row, col = np.where(flip, hi, lo), np.where(flip, lo, hi)
    order = np.argsort(row * n + col, kind="stable")
    rp = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]).astype(np.int64)
    say(f"case: CSR with {which} entries, {key.size} of them")
    _check(T.Graph.from_csr(n, dev(rp), dev(col[order].astype(np.int32))), T.E_ASYM, good, ref)
