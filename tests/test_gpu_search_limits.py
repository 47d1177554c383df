"""Product searches around their limits: the levels that one narrow launch may
expand, and the pairs that the visited set holds before it grows.  Pairs and
verdict equal to the oracle's, levels to the closed form.
"""
import numpy as np
import pytest

import oracle
from paper_2508_20735_amd import binding as B
from paper_2508_20735_amd import workloads as W

pytestmark = pytest.mark.gpu


def chain(n, k):
    delta = np.minimum(np.arange(n) + 1, n - 1).astype(np.uint32)
    return W.DFA(np.repeat(delta[:, None], k, axis=1), np.ones(n, np.uint8), 0)


@pytest.mark.parametrize("n", [255, 256, 257, 4095, 4096, 4097, 8193])
def test_thin_searches(n):
    d = chain(n, 2)
    verdict, pairs, st = B.included(d, d)
    assert (verdict, pairs, st["rounds"]) == (True, n, n)
    last = W.DFA(d.delta, d.accepting.copy(), 0)
    last.accepting[-1] = 0
    assert B.included(d, last)[0] is False and B.included(last, d)[0] is True


@pytest.mark.parametrize("na,nb", [(361, 363), (362, 362), (363, 363), (500, 530)])
@pytest.mark.parametrize("k", [2, 8])
def test_the_set_grows(na, nb, k):
    """About half of 2^18 pairs, all of them reached."""
    a, b = W.random_dfa(na, k, 0.5, na), W.random_dfa(nb, k, 0.5, nb + 1)
    b.accepting[:] = 1
    verdict, pairs, _ = B.included(a, b)
    want = oracle.product_bfs(a.delta, a.accepting, a.start, b.delta, b.accepting, b.start,
                              "inclusion")
    assert (verdict, pairs) == (want[0], want[1])
