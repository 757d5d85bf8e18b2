"""GPU tests of batches whose graphs are of both kinds, within the compact
kernel's limits (2^13 vertices, 2^18 edges) and beyond them, which come from one
queue of one kernel."""
import itertools

import numpy as np
import pytest

import graphgen
import oracle
from gpu_util import dev, lib, say

pytestmark = pytest.mark.gpu


def _graphs():
    i, j = np.triu_indices(40, 1)
    v = np.arange(1, 9001, dtype=np.int32)
    gs = [graphgen.er(9000, 0.002, 1),                           # more vertices
          (9001, np.zeros(9000, np.int32), v),                   # a star of them
          graphgen.er(700, 0.02, 2), graphgen.rmat(12, 8, 3),
          (20000, i.astype(np.int32) * 400, j.astype(np.int32) * 400),  # few edges on many ids
          (40, i.astype(np.int32), j.astype(np.int32)),
          (8192, np.array([8190], np.int32), np.array([8191], np.int32)),
          (30000, np.zeros(0, np.int32), np.zeros(0, np.int32)),
          graphgen.rmat(14, 20, 4),                              # more edges
          graphgen.er(8192, 0.003, 5)]
    gs += [graphgen.er(60 + 7 * k, 0.2, k) for k in range(20)]
    return [(n, *(graphgen.shuffle(s, d, k) if s.size else (s, d))) for k, (n, s, d) in enumerate(gs)]


@pytest.mark.parametrize("block,ilp", list(itertools.product((256, 512, 1024), (1, 2, 4))))
def test_both_kinds(block, ilp):
    T = lib()
    say(f"case: mixed batch, shape {block} x {ilp}")
    gs = _graphs()
    vo, eo, s, d = graphgen.pack(gs)
    ref = [oracle.truss(n, a, b) if a.size else (a, 0) for n, a, b in gs]
    got, st = T.truss_batch(vo, eo, dev(s), dev(d), T.make_options(batch_block=block, batch_ilp=ilp))
    np.testing.assert_array_equal(got.cpu().numpy(), np.concatenate([r[0] for r in ref]))
    assert st["kmax"] == max(r[1] for r in ref)
    assert st["triangles"] == sum(oracle.support_fwd(n, a, b)[1] for n, a, b in gs if a.size)


@pytest.mark.parametrize("bad", [[2], [0], [4, 3], [3, 8]])
def test_first_bad_graph_decides(bad):
    """A loop in the first graph of `bad`, an id out of range in the second."""
    T = lib()
    say(f"case: mixed batch, bad graphs {bad}")
    gs = [(n, a.copy(), b.copy()) for n, a, b in _graphs()]
    gs[bad[0]][1][1] = gs[bad[0]][2][1]
    if len(bad) > 1:
        gs[bad[1]][1][1] = gs[bad[1]][0]
    vo, eo, s, d = graphgen.pack(gs)
    with pytest.raises(T.TrussError) as ex:
        T.truss_batch(vo, eo, dev(s), dev(d))
    assert ex.value.code == (T.E_SELFLOOP if len(bad) == 1 or bad[0] < bad[1] else T.E_RANGE)
