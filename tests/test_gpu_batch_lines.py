"""Batches on both sides of the lines between their rounds, with no DFA left to
a workgroup of its own: parts of 896 states on average (staged ids or tiles),
and more than 8,192 tiles that are mostly padding (the general path).  Against
the oracle, equal.
"""
import numpy as np
import pytest

import oracle
from paper_2508_20735_amd import binding as B
from paper_2508_20735_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def segments_only():
    before = B.get_tuning()
    B.set_tuning(batch_lds_states=0)
    yield
    B.set_tuning(**before)


def check_minimise(dfas):
    blocks, nb, rounds, _ = B.minimise_batch(dfas)
    known = {}
    for d, block, count, r in zip(dfas, blocks, nb, rounds):
        if id(d) not in known:
            known[id(d)] = oracle.moore(d.delta, d.accepting)
        ref, n, _, changing = known[id(d)]
        np.testing.assert_array_equal(block, ref)
        assert (count, r) == (n, changing + 1), d.n


def check_pairs(pairs):
    got, _ = B.equivalent_batch(pairs)
    known = {}
    for d, e in pairs:
        if (id(d), id(e)) not in known:
            known[id(d), id(e)] = oracle.equiv_hk(d.delta, d.accepting, d.start, e.delta,
                                                  e.accepting, e.start)
    assert list(got) == [known[id(d), id(e)] for d, e in pairs]


def other(d, i):
    return W.mutate_one(d, i)[0] if i % 2 and d.n > 1 else W.permuted_copy(d, i)[0]


@pytest.mark.parametrize("k", [1, 3, 8, 9])
@pytest.mark.parametrize("n", [895, 896, 897, 1024])
def test_mean_of_a_part(n, k):
    """Small parts beside large ones, n states on average."""
    sizes = [1, 2, 255, 256, 257, 500, 700]
    sizes.append((len(sizes) + 1) * n - sum(sizes))
    dfas = [W.random_dfa(s, k, 0.3, s + k) for s in sizes]
    check_minimise(dfas)
    check_pairs([(d, other(d, i)) for i, d in enumerate(dfas)])


@pytest.mark.parametrize("count", [8192, 8193])
@pytest.mark.parametrize("n", [16, 31, 32, 33])
def test_padding(n, count):
    made = [W.random_dfa(n, 2 + i % 3, 0.3, i) for i in range(40)]
    check_minimise([made[i % 40] for i in range(count)])
    pairs = [(d, other(d, i)) for i, d in enumerate(made)]
    check_pairs([pairs[i % 40] for i in range(count // 2 + 1)])


@pytest.mark.parametrize("n", [458_752, 458_753])
@pytest.mark.parametrize("k", [2, 3])
def test_largest_unions(n, k):
    """Unions of 7 * 2^17 states and two more."""
    d = W.random_dfa(n, k, 0.3, n + k)
    small = W.random_dfa(3000, k, 0.3, 5)
    check_pairs([(d, W.permuted_copy(d, 3)[0]), (small, W.mutate_one(small, 4)[0]),
                 (d, W.mutate_one(d, 5)[0])])


@pytest.mark.parametrize("last", [209_716, 209_717])
def test_few_large_dfas_with_eight_letters(last):
    """2^20 states in five DFAs, and one more."""
    check_minimise([W.random_dfa(209_715, 8, 0.3, i) for i in range(4)] +
                   [W.random_dfa(last, 8, 0.3, 9)])
