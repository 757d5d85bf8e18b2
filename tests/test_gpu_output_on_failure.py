"""GPU tests of a peeling that is stopped at its cap on sub-rounds: the code
comes back and the output is left as it was, whether the output kernel follows
the peeling at once (few edges) or on the host's word."""
import pytest

import graphgen
from gpu_util import csr_graph, edges_graph, lib, say

pytestmark = pytest.mark.gpu

# below and above the size from which rows are compacted, 2^15 edges
GRAPHS = {"er2000": lambda: graphgen.er_small(1), "rmat13": lambda: graphgen.rmat(13, 16, 3)}


@pytest.mark.parametrize("cap", [1, 3])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_capped(name, cap):
    torch = pytest.importorskip("torch")
    T = lib()
    n, s, d = GRAPHS[name]()
    for g in (edges_graph(n, s, d), csr_graph(n, s, d)):
        say(f"case: {name}, {g.m} edges, at most {cap} sub-rounds")
        out = torch.full((g.m,), -7, dtype=torch.int32, device="cuda:0")
        ws = T.workspace(g).fill_(85)
        with pytest.raises(T.TrussError) as ex:
            T.truss_decompose(g, T.make_options(max_subrounds=cap), out=out, ws=ws)
        assert ex.value.code == T.E_INTERNAL
        assert bool((out == -7).all())
