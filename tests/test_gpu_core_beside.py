"""GPU tests of core numbers beside other work on the device: calls on several
streams at once, a decomposition that holds every compute unit, and long
products queued on another stream.  Whether the persistent kernel or the
stepped launches run, the core numbers are the oracle's."""
import threading

import numpy as np
import pytest

import graphgen
import oracle
from gpu_util import csr_graph, edges_graph, lib, say

pytestmark = pytest.mark.gpu


def _rmat(scale, factor, seed):
    n, s, d = graphgen.rmat(scale, factor, seed)
    return n, s, d, oracle.core_numbers(n, s, d)[0]


def _repeat(g, want, times, errors):
    import torch
    T = lib()
    try:
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(times):
                got, cmax = T.truss_core_numbers(g)
                np.testing.assert_array_equal(got.cpu().numpy(), want)
                assert cmax == int(want.max())
    except BaseException as e:  # noqa: B036 (reported by the main thread)
        errors.append(e)


def _run(threads, errors):
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    if errors:
        raise errors[0]


@pytest.mark.parametrize("callers", [2, 4])
def test_at_once(callers):
    say(f"case: core numbers on {callers} streams")
    errors, threads = [], []
    for i in range(callers):
        n, s, d, want = _rmat(12 + i, 8, i)
        g = edges_graph(n, s, d) if i % 2 else csr_graph(n, s, d)
        threads.append(threading.Thread(target=_repeat, args=(g, want, 12, errors)))
    _run(threads, errors)


def test_beside_a_decomposition():
    """The peeling kernel of another thread holds every compute unit for milliseconds at a time."""
    import torch
    T = lib()
    n, s, d, want = _rmat(14, 8, 3)
    bn, bs, bd = graphgen.rmat(17, 16, 5)
    big, phi = edges_graph(bn, bs, bd), oracle.truss(bn, bs, bd)[0]
    errors = []

    def decompose():
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(10):
                    got, _ = T.truss_decompose(big)
                    np.testing.assert_array_equal(got.cpu().numpy(), phi)
        except BaseException as e:  # noqa: B036
            errors.append(e)

    say("case: core numbers beside a decomposition")
    _run([threading.Thread(target=decompose),
          threading.Thread(target=_repeat, args=(csr_graph(n, s, d), want, 40, errors))], errors)


def test_beside_products():
    """Products queued on another stream leave no compute unit free for a whole workgroup."""
    import torch
    n, s, d, want = _rmat(14, 8, 4)
    g = csr_graph(n, s, d)
    x = torch.randn(8192, 8192, device="cuda:0").to(torch.bfloat16)
    y = torch.empty_like(x)
    other = torch.cuda.Stream()
    say("case: core numbers beside products")
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        for _ in range(60):
            torch.mm(x, x, out=y)
    errors = []
    _repeat(g, want, 10, errors)
    torch.cuda.synchronize()
    if errors:
        raise errors[0]
