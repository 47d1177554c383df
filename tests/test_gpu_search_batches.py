"""The searches that queue several levels per host wait: reachability pruning
and product exploration where they change between narrow and wide levels,
run past one batch of levels, or outgrow the visited set.  Whole numbers:
element-by-element equality with the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_2508_20735_amd import binding as B
from paper_2508_20735_amd import workloads as W

pytestmark = pytest.mark.gpu


def two_bulbs(n, k, chain, seed):
    """A random part, a chain it leads into, and a second random part at the
    chain's end: a wide search that thins out and widens again."""
    a, b = W.random_dfa(n, k, 0.3, seed), W.random_dfa(n, k, 0.4, seed + 1)
    delta = np.concatenate([a.delta, np.zeros((chain, k), np.uint32), b.delta + n + chain])
    delta[n:n + chain] = (np.arange(chain) + n + 1).astype(np.uint32)[:, None]
    delta[0, 0] = n
    acc = np.concatenate([a.accepting, np.zeros(chain, np.uint8), b.accepting])
    return W.DFA(delta, acc, 0)


@pytest.mark.parametrize("d", [
    two_bulbs(20000, 2, 60, 1), two_bulbs(9001, 5, 40, 2), two_bulbs(700, 3, 30, 3),
    W.random_dfa(300_001, 2, 0.5, 4), W.random_dfa(2049, 2, 0.5, 5), W.random_dfa(4096, 1, 0.5, 6),
    W.random_dfa(1025, 4, 0.5, 7), W.extended_bitsplitter(12),
], ids=["bulbs2", "bulbs5", "bulbs3", "deep", "edge2", "unary", "edge4", "bits"])
def test_pruned_search(d):
    res = B.minimise(d.delta, d.accepting, start=d.start, prune=True)
    block, nb, nr = oracle.minimise_reachable(d.delta, d.accepting, d.start)
    np.testing.assert_array_equal(res.block, block)
    assert res.stats["num_blocks"] == nb and res.stats["reachable"] == nr


def accepting_everywhere(d):
    return W.DFA(d.delta, np.ones(d.n, np.uint8), d.start)


@pytest.mark.parametrize("a,b", [
    # nearly every pair is reached: the visited set grows again and again
    (W.random_dfa(300, 3, 0.5, 11), W.random_dfa(301, 3, 0.5, 12)),
    (W.random_dfa(64, 5, 0.5, 13), W.random_dfa(63, 5, 0.5, 14)),
    (W.random_dfa(1000, 4, 0.5, 15), W.random_dfa(700, 4, 0.5, 16)),
    (W.random_dfa(150, 7, 0.5, 17), W.random_dfa(200, 7, 0.5, 18)),
    (W.random_dfa(9, 1, 0.5, 19), W.random_dfa(8, 1, 0.5, 20)),
    (two_bulbs(5000, 4, 50, 21), two_bulbs(5000, 4, 50, 21)),
    (two_bulbs(3000, 2, 300, 22), two_bulbs(3000, 2, 300, 22)),
], ids=["grow3", "grow5", "grow4", "grow7", "tiny", "bulbs4", "bulbs2"])
def test_product_search(a, b):
    all_b = accepting_everywhere(b)
    verdict, pairs, st = B.included(a, all_b)
    want = oracle.product_bfs(a.delta, a.accepting, a.start, all_b.delta, all_b.accepting,
                              all_b.start, "inclusion")
    assert verdict and (verdict, pairs) == (want[0], want[1])
    # refuted at the first accepting state of a that is reached
    none_b = W.DFA(b.delta, np.zeros(b.n, np.uint8), b.start)
    verdict, pairs, st = B.included(a, none_b)
    assert verdict == oracle.product_bfs(a.delta, a.accepting, a.start, none_b.delta,
                                         none_b.accepting, none_b.start, "inclusion")[0]


def test_product_bad_target():
    a, b = W.random_dfa(500, 3, 0.5, 31), W.random_dfa(400, 3, 0.5, 32)
    bad = b.delta.copy()
    bad[7, 2] = b.n
    for pair in ((a, W.DFA(bad, b.accepting, 0)), (W.DFA(bad, b.accepting, 0), a)):
        with pytest.raises(B.DfaError) as e:
            B.included(*pair)
        assert e.value.status == B.DFA_EINVAL
    assert B.included(a, accepting_everywhere(b))[0]
