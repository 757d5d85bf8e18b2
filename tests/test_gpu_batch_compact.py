"""GPU tests of the batch's compact kernel at the edges of its range: the
largest vertex id, hubs, rows around a bitmap word and a table bucket, the
largest edge count, and repeated pairs that overflow a degree counter."""
import itertools

import numpy as np
import pytest

import graphgen
import oracle
from gpu_util import dev, lib, say

pytestmark = pytest.mark.gpu


def _run(gs, **opt):
    T = lib()
    vo, eo, s, d = graphgen.pack(gs)
    out, st = T.truss_batch(vo, eo, dev(s), dev(d), T.make_options(**opt) if opt else None)
    return out.cpu().numpy(), st


def _clique_on(ids):
    i, j = np.triu_indices(len(ids), 1)
    return np.asarray(ids, np.int32)[i], np.asarray(ids, np.int32)[j]


def _hub(n, extra, seed):
    """Vertex 0 joined to all others, plus random pairs among them."""
    rng = np.random.default_rng(seed)
    e = {(0, v) for v in range(1, n)}
    while len(e) < n - 1 + extra:
        a, b = sorted(rng.integers(1, n, 2).tolist())
        if a != b:
            e.add((a, b))
    a = np.array(sorted(e), np.int32)
    return n, a[:, 0].copy(), a[:, 1].copy()


@pytest.mark.parametrize("block,ilp", list(itertools.product((256, 512, 1024), (1, 2, 4))))
def test_edges_of_the_range(block, ilp):
    say(f"case: compact batch, shape {block} x {ilp}")
    gs = [_hub(8192, 9000, 1), _hub(8191, 500, 2), (8193, *_clique_on(range(8170, 8193))),
          (8192, *_clique_on([0, 31, 32, 33, 63, 64, 4095, 4096, 8159, 8160, 8190, 8191])),
          (2, np.array([1], np.int32), np.array([0], np.int32)),
          (8192, np.zeros(0, np.int32), np.zeros(0, np.int32))]
    gs += [(k, *_clique_on(range(k))) for k in (3, 4, 5, 33, 64, 65, 66, 129)]
    gs = [(n, *(graphgen.shuffle(s, d, i) if s.size else (s, d))) for i, (n, s, d) in enumerate(gs)]
    ref = np.concatenate([oracle.truss(n, s, d)[0] if s.size else s for n, s, d in gs])
    got, st = _run(gs, batch_block=block, batch_ilp=ilp)
    np.testing.assert_array_equal(got, ref)
    assert st["triangles"] == sum(oracle.support_fwd(n, s, d)[1] for n, s, d in gs if s.size)


@pytest.mark.parametrize("m", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1])
def test_largest_edge_count(m):
    """G(8192, m) around the compact kernel's limit (one more edge takes the general kernel)."""
    say(f"case: {m} edges on 8192 vertices")
    n, s, d = graphgen.er(8192, 0.0085, 5)
    assert s.size > m
    keep = np.random.default_rng(m).permutation(s.size)[:m]
    s, d = graphgen.shuffle(s[keep], d[keep], 7)
    got, _ = _run([(n, s, d), (3, *_clique_on(range(3)))])
    np.testing.assert_array_equal(got, np.concatenate([oracle.truss(n, s, d)[0], [3, 3, 3]]))


def test_many_repeats_are_refused():
    """One pair 70,000 times (more than a 16-bit degree counter holds), one pair twice, and a
    self-loop beside a repeated pair: the codes of the single-graph path."""
    T = lib()
    say("case: repeated pairs")
    ok = (3, *_clique_on(range(3)))
    many = (40, np.zeros(70000, np.int32), np.ones(70000, np.int32))
    twice = (5, np.array([0, 3, 1], np.int32), np.array([1, 4, 0], np.int32))
    loop = (5, np.array([0, 3, 1, 2], np.int32), np.array([1, 4, 0, 2], np.int32))
    for bad, code in ((many, T.E_DUP), (twice, T.E_DUP), (loop, T.E_SELFLOOP)):
        with pytest.raises(T.TrussError) as ex:
            _run([ok, bad])
        assert ex.value.code == code
