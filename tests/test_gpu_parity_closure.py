"""Closure rounds whose keys stay in LDS, against the oracle and against the
two passes over signature rows (which grouping without LDS keeps): partitions,
rounds and block counts, for one column more or less than a batch of letters
and than the LDS limit, ragged tiles, chains, bit-splitters and random DFAs,
and unions.  Whole numbers, equal.
"""
import numpy as np
import pytest

import oracle
from paper_2508_20735_amd import binding as B
from paper_2508_20735_amd import workloads as W

pytestmark = pytest.mark.gpu


def figures(res):
    return {key: res.stats[key] for key in
            ("num_blocks", "rounds", "changing_rounds", "k_eff", "tc_used")}


def check(d, tc="on", **kw):
    res = B.minimise(d.delta, d.accepting, tc=tc, **kw)
    two = B.minimise(d.delta, d.accepting, tc=tc, lds_stage=0, **kw)
    ref, nb = oracle.hopcroft(d.delta, d.accepting)
    np.testing.assert_array_equal(res.block, ref)
    assert res.stats["num_blocks"] == nb
    assert figures(res) == figures(two)
    return res.stats


@pytest.mark.parametrize("n", [9, 255, 256, 257, 1023, 2049, 8192, 30_001])
@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_random(n, k):
    check(W.random_dfa(n, k, 0.3, n + k))


@pytest.mark.parametrize("bits", [8, 10, 12])
def test_bitsplitter(bits):
    check(W.bitsplitter(bits))


@pytest.mark.parametrize("chain,tail", [(300, 700), (4_000, 4_000), (65_537, 65_535)])
@pytest.mark.parametrize("tc", ["auto", "on"])
def test_chains(chain, tail, tc):
    check(W.chain_with_tail(chain, tail, 3, k=4), tc)


def test_blocks_of_several_members():
    """Twins of a chain: every block keeps two members that gather alike."""
    d = W.chain_with_tail(6_000, 2_000, 5, k=2)
    delta = np.concatenate([d.delta, d.delta + d.n]).astype(np.uint32)
    stats = check(W.DFA(delta, np.tile(d.accepting, 2), 0))
    assert stats["tc_used"]


@pytest.mark.parametrize("mutate", [False, True])
def test_unions(mutate):
    d = W.chain_with_tail(5_000, 3_000, 7, k=3)
    e = W.mutate_one(d, 3)[0] if mutate else W.permuted_copy(d, 3)[0]
    assert B.equivalent(d, e, tc="on")[0] == oracle.equiv_hk(
        d.delta, d.accepting, d.start, e.delta, e.accepting, e.start)
