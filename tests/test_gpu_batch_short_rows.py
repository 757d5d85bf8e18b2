"""GPU tests of the batch's compact kernel on sparse graphs: rows that a thread, a
quarter wavefront and a wavefront take, at the edges between them, hubs among
short rows, repeated pairs in each kind of row, and batches of tiny graphs."""
import itertools

import numpy as np
import pytest

import graphgen
import oracle
from gpu_util import dev, lib, say

pytestmark = pytest.mark.gpu

SHAPES = list(itertools.product((256, 512, 1024), (1, 2, 4)))


def _ring(n, r):
    """Every vertex joined to the r next ones on a circle: rows of 2r entries."""
    i = np.arange(n)
    a, b = np.tile(i, r), np.concatenate([(i + j) % n for j in range(1, r + 1)])
    return n, np.minimum(a, b).astype(np.int32), np.maximum(a, b).astype(np.int32)


def _star_of_cliques(k, times):
    """Cliques of k vertices whose first vertex is joined to a hub."""
    i, j = np.triu_indices(k, 1)
    at = 1 + k * np.arange(times)
    s = np.concatenate([(at[:, None] + i).ravel(), np.zeros(times, int)])
    d = np.concatenate([(at[:, None] + j).ravel(), at])
    return 1 + k * times, s.astype(np.int32), d.astype(np.int32)


def _run(gs, **opt):
    T = lib()
    vo, eo, s, d = graphgen.pack(gs)
    out, st = T.truss_batch(vo, eo, dev(s), dev(d), T.make_options(**opt) if opt else None)
    return out.cpu().numpy(), st


def _check(gs, **opt):
    gs = [(n, *graphgen.shuffle(s, d, i)) for i, (n, s, d) in enumerate(gs)]
    got, st = _run(gs, **opt)
    ref = [oracle.truss(n, s, d) for n, s, d in gs]
    np.testing.assert_array_equal(got, np.concatenate([r[0] for r in ref]))
    assert st["kmax"] == max(r[1] for r in ref)
    assert st["triangles"] == sum(oracle.support_fwd(n, s, d)[1] for n, s, d in gs)


@pytest.mark.parametrize("block,ilp", SHAPES)
def test_rows_around_the_limits(block, ilp):
    """Rows of 2 to 34 entries (limits 4 and 16), ends of the id ranges off the group and wavefront sizes."""
    say(f"case: short rows, shape {block} x {ilp}")
    gs = [_ring(n, r) for n, r in ((67, 1), (70, 2), (1025, 2), (130, 3), (515, 7), (1031, 8), (203, 9), (8191, 8),
                                   (140, 17))]
    gs += [_star_of_cliques(k, t) for k, t in ((3, 900), (4, 333), (5, 101), (6, 60), (15, 40), (16, 40), (17, 33),
                                               (18, 20))]
    gs += [graphgen.er(4001, 0.001, 7), graphgen.er(8192, 0.0012, 8), graphgen.er(300, 0.03, 9),
           graphgen.rmat(12, 3, 10)]
    _check(gs, batch_block=block, batch_ilp=ilp)


def test_tiny_graphs_alone_and_beside_others():
    """Up to 64 vertices and 256 edges in the whole batch, and one graph beyond that."""
    say("case: tiny graphs")
    tiny = [graphgen.er(n, min(0.9, 5.0 / n), n) for n in range(4, 65)]
    tiny = [g for g in tiny if 0 < g[1].size <= 256]
    _check(tiny)
    _check(tiny + [_ring(65, 2)])
    _check([_ring(64, 4)])
    _check([_ring(65, 3)])


@pytest.mark.parametrize("r", [1, 2, 3, 8, 9])
def test_repeated_pair(r):
    """The same pair once more, in rows of each kind."""
    T = lib()
    say(f"case: repeated pair, rows of {2 * r}")
    n, s, d = _ring(500, r)
    for k in (0, s.size // 2, s.size - 1):
        with pytest.raises(T.TrussError) as ex:
            _run([(n, np.append(s, d[k]).astype(np.int32), np.append(d, s[k]).astype(np.int32))])
        assert ex.value.code == T.E_DUP
