"""Batched rounds that hold the ids of a part in LDS, against the oracle: parts
at the edges of a workgroup's share (1,024 to 8,192 states) and of the ids that
fit, every number of letters, one key for almost all states, pairs with the
whole union in LDS and without, and the batches beside them that take the other
rounds.  Whole numbers, equal.
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
    for d, block, count, r in zip(dfas, blocks, nb, rounds):
        ref, n, _, changing = oracle.moore(d.delta, d.accepting)
        np.testing.assert_array_equal(block, ref)
        assert (count, r) == (n, changing + 1), d.n


def check_pairs(pairs):
    got, _ = B.equivalent_batch(pairs)
    want = [oracle.equiv_hk(d.delta, d.accepting, d.start, e.delta, e.accepting, e.start)
            for d, e in pairs]
    assert list(got) == want


def with_copies(d, times):
    delta = np.concatenate([d.delta + i * d.n for i in range(times)]).astype(np.uint32)
    return W.DFA(delta, np.tile(d.accepting, times), 0)


@pytest.mark.parametrize("k", range(1, 9))
def test_sizes_and_letters(k):
    sizes = [1, 2, 63, 255, 256, 257, 1023, 1024, 1025, 2047, 2049, 4096, 5001]
    check_minimise([W.random_dfa(n, k, 0.3, n + k) for n in sizes])
    check_minimise([with_copies(W.random_dfa(n, k, 0.1, n), 3) for n in sizes])


def test_largest_windows():
    """65,536 states are staged; one more, or a ninth letter, are not."""
    full = [W.random_dfa(n, k, 0.2, n + k) for n, k in
            [(65_535, 2), (65_536, 3), (65_536, 4), (8_191, 5), (8_192, 8), (8_193, 2)]]
    check_minimise(full)
    check_minimise([with_copies(W.random_dfa(21_845, 4, 0.2, 9), 3)] + full[:1])
    check_minimise(full[:1] + [W.random_dfa(65_537, 2, 0.2, 4)])
    check_minimise(full[3:] + [W.random_dfa(3_000, 9, 0.4, 5)])


def test_many_rows_to_a_workgroup():
    """Enough states for eight rows of them to a workgroup."""
    rng = np.random.default_rng(11)
    check_minimise([W.random_dfa(int(n), int(k), 0.2, i) for i, (n, k) in enumerate(
        zip(rng.integers(30_000, 65_537, 90), rng.integers(2, 5, 90)))])


@pytest.mark.parametrize("p", [0.0, 0.0005, 0.01, 1.0])
def test_keys_shared_by_most_states(p):
    check_minimise([W.random_dfa(n, k, p, n) for n, k in
                    [(1_000, 2), (30_000, 2), (65_536, 2), (40_000, 4), (20_000, 8)]])


def test_chains():
    check_minimise([W.chain_with_tail(60, 5_000, 3, k=4), W.chain_with_tail(20, 60_000, 4, k=2),
                    W.bitsplitter(10), W.random_dfa(700, 2, 0.5, 1)])


@pytest.mark.parametrize("mutate", [False, True])
@pytest.mark.parametrize("n", [500, 8_193, 32_768, 32_769, 65_536])
def test_pairs(n, mutate):
    """Unions of up to 65,536 states lie in LDS whole, larger ones by operand."""
    pairs = []
    for k in (2, 3, 4, 8):
        d = W.random_dfa(n, k, 0.2, n + k)
        pairs.append((d, W.mutate_one(d, 3)[0] if mutate else W.permuted_copy(d, 3)[0]))
    d = with_copies(W.random_dfa(n // 2, 4, 0.3, n), 2)
    pairs.append((d, W.random_dfa(n // 2, 4, 0.3, n)))
    check_pairs(pairs)
