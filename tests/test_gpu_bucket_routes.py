"""Which way the first table round goes, by buckets or by the table, and the
same answer either way: a key shared by more states than a bucket has room
for, found by the pass itself (the sample of its inputs lets them through) or
by the sample.  Whole numbers, equal to the oracle's.
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


def grouped_by_buckets(d, check=True):
    """States that buckets grouped; the answer is checked."""
    try:
        B.profile_only("k_group_part")
        B.profile_enable(True)
        timed = B.minimise(d.delta, d.accepting, tc="off")
        states = B.profile_read().get("k_group_part", {"states": 0})["states"]
    finally:
        B.profile_enable(False)
        B.profile_only(None)
    plain = B.minimise(d.delta, d.accepting, tc="off")
    if check:
        ref, nb, rounds, changing = oracle.moore(d.delta, d.accepting)
        for res in (timed, plain):
            np.testing.assert_array_equal(res.block, ref)
            assert (res.stats["num_blocks"], res.stats["rounds"],
                    res.stats["changing_rounds"]) == (nb, rounds, changing)
    return states


def with_a_frequent_key(n, k, share, seed):
    """A share of the states have the same successors: one key for them."""
    d = W.random_dfa(n, k, 0.3, seed)
    same = np.random.default_rng(seed + 1).random(n) < share
    d.delta[same] = d.delta[0]
    d.accepting[same] = d.accepting[0]
    return d


@pytest.mark.parametrize("k", [3, 4, 8])
@pytest.mark.parametrize("n", [2049, 8193, 100_001])
def test_spread_keys_go_by_buckets(n, k):
    assert grouped_by_buckets(W.random_dfa(n, k, 0.3, n + k)) == n


@pytest.mark.parametrize("k", [4, 8])
@pytest.mark.parametrize("n,share", [
    (16_000, 0.8),    # 2 buckets, which no sample stops: 14,400 states for 10,512 places
    (16_384, 0.999),  # all states in one bucket
    (9000, 0.9),      # 8,550 for 6,137
    (65_000, 0.05),   # 8 buckets, 1.4 times the mean in one
    (65_000, 0.08),   # 1.6 times
    (130_000, 0.045), # 16 buckets, 1.7 times
])
def test_a_bucket_overflows_in_the_pass(n, share, k):
    assert grouped_by_buckets(with_a_frequent_key(n, k, share, 5)) == 0


@pytest.mark.parametrize("share", [0.3, 0.6, 0.999])
def test_the_sample_stops_the_pass(share):
    assert grouped_by_buckets(with_a_frequent_key(60_000, 4, share, 5)) == 0


@pytest.mark.parametrize("n,share", [(16_000, 0.1), (65_000, 0.01), (130_000, 0.01)])
def test_a_frequent_key_fits(n, share):
    assert grouped_by_buckets(with_a_frequent_key(n, 4, share, 5)) == n


def test_a_fill_outgrows_its_16_bits():
    """The states that the sample looks at have spread keys, all others one:
    half a million states for one bucket, whose count (16 bits, four to a
    word) carries into its neighbours'."""
    n, sample = 500_000, 16_384
    d = W.random_dfa(n, 4, 0.3, 9)
    at = np.arange(sample, dtype=np.int64) * n // sample
    rows = at[np.random.default_rng(10).integers(0, sample, (sample, 4))]
    accepting = d.accepting[at].copy()
    d.delta[:] = d.delta[1]
    d.accepting[:] = 0
    d.delta[at] = rows
    d.accepting[at] = accepting
    assert grouped_by_buckets(d) == 0


@pytest.mark.parametrize("n,k,seed", [(4_200_000, 4, 3), (4_200_000, 4, 6), (4_200_000, 4, 29),
                                      (4_300_007, 3, 5), (4_300_007, 3, 39)])
def test_the_sample_lets_spread_keys_through(n, k, seed):
    """1,024 buckets have 16 states of the sample each: some bucket of these
    inputs has more than twice that by chance."""
    d = W.random_dfa(n, k, 0.3, seed)
    assert grouped_by_buckets(d, check=False) == n
    buckets = B.minimise(d.delta, d.accepting, tc="off")
    B.set_tuning(slice_min_states=0)
    table = B.minimise(d.delta, d.accepting, tc="off")
    np.testing.assert_array_equal(buckets.block, table.block)
    assert [buckets.stats[s] for s in ("num_blocks", "rounds", "changing_rounds")] == \
        [table.stats[s] for s in ("num_blocks", "rounds", "changing_rounds")]
