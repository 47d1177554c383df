"""The first table round grouped by buckets of the key hash, against the
oracle: one bucket and several, ragged last tiles, every width that takes it,
states with twins, and keys shared by so many states that a bucket overflows
and the table does the round.  Whole numbers, equal.
"""
import numpy as np
import pytest

import oracle
from paper_2508_20735_amd import binding as B
from paper_2508_20735_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def small_slices():
    before = B.get_tuning()
    B.set_tuning(slice_min_states=1024)
    yield
    B.set_tuning(**before)


def check(d):
    res = B.minimise(d.delta, d.accepting, tc="off")
    ref, nb, rounds, changing = oracle.moore(d.delta, d.accepting)
    np.testing.assert_array_equal(res.block, ref)
    assert (res.stats["num_blocks"], res.stats["rounds"], res.stats["changing_rounds"]) == \
        (nb, rounds, changing)


@pytest.mark.parametrize("n", [1024, 2047, 2049, 8192, 8193, 16_385, 100_001, 131_073, 200_001])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 8])
def test_sizes_and_widths(n, k):
    check(W.random_dfa(n, k, 0.3, n + k))


@pytest.mark.parametrize("copies", [2, 3, 9])
def test_blocks_of_several(copies):
    d = W.random_dfa(12_000, 4, 0.2, copies)
    delta = np.concatenate([d.delta + i * d.n for i in range(copies)]).astype(np.uint32)
    check(W.DFA(delta, np.tile(d.accepting, copies), 0))


@pytest.mark.parametrize("n", [1500, 3000, 20_000])
@pytest.mark.parametrize("k", [3, 4, 8])
def test_most_keys_are_known_before(n, k):
    """Almost every label is a state's own: that round does not take slices."""
    d = W.random_dfa(n, k, 0.5, n)
    twin = np.random.default_rng(7).integers(0, n, n // 20)
    d.delta[:len(twin)] = d.delta[twin]
    d.accepting[:len(twin)] = d.accepting[twin]
    check(d)


@pytest.mark.parametrize("share", [0.2, 0.6, 0.999])
def test_a_bucket_overflows(share):
    """A share of the states have the same successors: one key for them."""
    d = W.random_dfa(60_000, 4, 0.3, 5)
    same = np.random.default_rng(6).random(d.n) < share
    d.delta[same] = d.delta[0]
    d.accepting[same] = d.accepting[0]
    check(d)
    check(W.chain_with_tail(20_000, 30_000, 7, k=4) if share < 0.3 else
          W.chain_with_tail(30, 30_000, 8, k=2))


@pytest.mark.parametrize("mutate", [False, True])
@pytest.mark.parametrize("k", [2, 4, 8])
def test_unions(k, mutate):
    d = W.random_dfa(30_011, k, 0.2, 40 + k)
    e = W.mutate_one(d, 3)[0] if mutate else W.permuted_copy(d, 3)[0]
    assert B.equivalent(d, e)[0] == oracle.equiv_hk(d.delta, d.accepting, d.start, e.delta,
                                                    e.accepting, e.start)
