"""What the host decides from the rounds' reports while they run, against the
same call with kernel timing on, where it reads the round state back after
each chunk: the same rounds, the same switch to the closure, the same totals.
"""
import numpy as np
import pytest

import oracle
from paper_2508_20735_amd import binding as B
from paper_2508_20735_amd import workloads as W

pytestmark = pytest.mark.gpu


def counted(stats):
    """(The refined states, and so the bytes, depend on which member of a block
    came first: they differ from call to call.)"""
    return {k: v for k, v in stats.items()
            if not k.endswith("_ms") and k != "algorithmic_bytes"}


def both_ways(call):
    seen = call()
    try:
        B.profile_only("k_round_end")
        B.profile_enable(True)
        read = call()
    finally:
        B.profile_enable(False)
        B.profile_only(None)
    return seen, read


DFAS = {
    "stalls": W.chain_with_tail(3000, 3000, 1), "stalls4": W.chain_with_tail(20_000, 100, 2, k=4),
    "random": W.random_dfa(30_000, 3, 0.2, 3), "bits": W.bitsplitter(13), "fib": W.fibonacci(11),
    "one block": W.DFA(np.zeros((5000, 2), np.uint32), np.ones(5000, np.uint8), 0),
}


@pytest.mark.parametrize("tc", ["off", "on", "auto"])
@pytest.mark.parametrize("loop", ["chunk", "graph"])
@pytest.mark.parametrize("name", list(DFAS))
def test_signature_rounds(name, loop, tc):
    d = DFAS[name]
    seen, read = both_ways(lambda: B.minimise(d.delta, d.accepting, tc=tc, loop=loop, lds_stage=1))
    np.testing.assert_array_equal(seen.block, read.block)
    assert counted(seen.stats) == counted(read.stats)
    np.testing.assert_array_equal(seen.block, oracle.hopcroft(d.delta, d.accepting)[0])


@pytest.mark.parametrize("tc", ["off", "auto"])
@pytest.mark.parametrize("name", ["stalls", "bits", "fib", "one block"])
def test_leader_rounds(name, tc):
    d = DFAS[name]
    seen, read = both_ways(
        lambda: B.minimise(d.delta, d.accepting, tc=tc, algorithm="leader"))
    np.testing.assert_array_equal(seen.block, read.block)
    assert counted(seen.stats) == counted(read.stats)


@pytest.mark.parametrize("max_rounds", [1, 5, 6, 7, 13, 30])
def test_a_round_limit(max_rounds):
    d = DFAS["fib"]
    for kw in ({}, {"algorithm": "leader"}):
        with pytest.raises(B.DfaError) as e:
            B.minimise(d.delta, d.accepting, tc="off", max_rounds=max_rounds, **kw)
        assert e.value.status == B.DFA_ELIMIT


@pytest.mark.parametrize("mutate", [False, True])
def test_unions(mutate):
    d = W.random_dfa(20_000, 2, 0.3, 9)
    e = W.mutate_one(d, 4)[0] if mutate else W.permuted_copy(d, 4)[0]
    seen, read = both_ways(lambda: B.equivalent(d, e, lds_stage=1))
    assert seen[0] == read[0]
    assert counted(seen[1]) == counted(read[1])
