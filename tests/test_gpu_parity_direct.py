"""The one-workgroup path of small sizes and the one-launch-per-round path of
ordinary ones against the oracle and the general path (reached with
loop="host"): tile edges, every letter count they take, unaligned rows, unions
whose operands meet inside a tile, refinements that need more rounds than they
run.  Whole numbers, equal.
"""
import numpy as np
import pytest

import oracle
from paper_2508_20735_amd import binding as B
from paper_2508_20735_amd import workloads as W

pytestmark = pytest.mark.gpu

WHOLE = 6144     # the largest refinement of one workgroup (2,048 x k = 16 fit its LDS too)
LIMIT = 1 << 19  # the largest minimisation with a launch per round


def doubled(d):
    """Every state twice: no block of one state."""
    return W.DFA(np.concatenate([d.delta, d.delta + d.n]),
                 np.concatenate([d.accepting, d.accepting]), d.start)


def quotient_of(d, block, start):
    leaders = np.flatnonzero(block == np.arange(d.n, dtype=np.uint32))
    dense = np.full(d.n, -1, dtype=np.int64)
    dense[leaders] = np.arange(len(leaders))
    return (len(leaders), dense[block[d.delta[leaders]]].astype(np.uint32),
            (d.accepting[leaders] != 0).astype(np.uint8), int(dense[block[start]]))


def check(d, tc="auto"):
    res = B.minimise(d.delta, d.accepting, tc=tc, start=d.start, quotient=True)
    ref = oracle.hopcroft(d.delta, d.accepting)[0]
    np.testing.assert_array_equal(res.block, ref)
    want = quotient_of(d, ref, d.start)
    assert res.quotient[0] == want[0] and res.quotient[3] == want[3]
    np.testing.assert_array_equal(res.quotient[1], want[1])
    np.testing.assert_array_equal(res.quotient[2], want[2])
    other = B.minimise(d.delta, d.accepting, tc=tc, loop="host")
    np.testing.assert_array_equal(other.block, ref)
    if not res.stats["tc_used"] and not other.stats["tc_used"]:
        for key in ("rounds", "changing_rounds", "num_blocks", "k_eff", "transitions_refined"):
            assert res.stats[key] == other.stats[key], key
    return res


@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 1023, 1024, 1025, 2049, WHOLE - 1,
                               WHOLE, WHOLE + 1, 6399, 6400, 6401, 40_000])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 16])
def test_sizes_and_letters(n, k):
    check(W.random_dfa(n, k, 0.3, n * 17 + k))


@pytest.mark.parametrize("n,k", [(500, 4), (3000, 7), (9000, 2), (20_000, 12)])
def test_blocks_of_two(n, k):
    check(doubled(W.random_dfa(n, k, 0.2, n + k)))


@pytest.mark.parametrize("n", [LIMIT - 1, LIMIT, LIMIT + 1])
def test_largest(n):
    check(W.random_dfa(n, 4, 0.1, n))


def test_identity_letters_and_single_classes():
    d = W.random_dfa(700, 3, 0.4, 5)
    ident = np.arange(d.n, dtype=np.uint32)[:, None]
    check(W.DFA(np.concatenate([ident, d.delta, ident], axis=1), d.accepting, 3))
    check(W.DFA(np.tile(ident, (1, 2)), d.accepting, 0))
    for value in (0, 1):
        res = check(W.DFA(d.delta, np.full(d.n, value, np.uint8), 0))
        assert res.stats["num_blocks"] == 1 and res.stats["rounds"] == 1


@pytest.mark.parametrize("n", [12, 14, 15, 16, 17, 40, 300, 5000])
@pytest.mark.parametrize("tc", ["auto", "off"])
def test_more_rounds_than_the_path_runs(n, tc):
    """A chain splits one state a round: the general path goes on."""
    check(W.fig1_chain(n), tc=tc)
    check(W.chain_with_tail(n, n // 2, n, k=4), tc=tc)


@pytest.mark.parametrize("n,k", [(1, 1), (100, 2), (129, 4), (5000, 4), (30_000, 8), (60_000, 3)])
@pytest.mark.parametrize("change", [False, True])
def test_equivalence(n, k, change):
    d = W.random_dfa(n, k, 0.3, n + 3 * k)
    e = W.mutate_one(d, 7)[0] if change else W.permuted_copy(d, 7)[0]
    got, st = B.equivalent(d, e)
    assert got == oracle.equiv_hk(d.delta, d.accepting, d.start, e.delta, e.accepting, e.start)
    other, st2 = B.equivalent(d, e, loop="host")
    assert got == other
    for key in ("rounds", "changing_rounds", "num_blocks", "k_eff"):
        assert st[key] == st2[key], key


def test_unaligned_rows_on_the_device():
    for n in (3001, 7001):
        check_unaligned(W.random_dfa(n, 4, 0.3, 9))


def check_unaligned(d):
    import torch
    flat = torch.zeros(d.n * 4 + 8, dtype=torch.int32, device="cuda:0")
    ref = oracle.hopcroft(d.delta, d.accepting)[0]
    acc = torch.from_numpy(d.accepting).cuda()
    for shift in range(4):
        rows = flat[shift:shift + d.n * 4].view(d.n, 4)
        rows.copy_(torch.from_numpy(d.delta.view(np.int32)))
        res = B.minimise_device(rows, acc, quotient=True)
        np.testing.assert_array_equal(res.block.cpu().numpy().view(np.uint32), ref)
        assert B.equivalent_device(rows, acc, 0, rows, acc, 0)[0]


@pytest.mark.parametrize("n", [2000, 9000])
def test_bad_targets(n):
    d = W.random_dfa(n, 4, 0.3, 10)
    for q, a in ((0, 0), (n - 1, 3)):
        bad = d.delta.copy()
        bad[q, a] = d.n
        with pytest.raises(B.DfaError) as e:
            B.minimise(bad, d.accepting)
        assert e.value.status == B.DFA_EINVAL
        for pair in ((W.DFA(bad, d.accepting), d), (d, W.DFA(bad, d.accepting))):
            with pytest.raises(B.DfaError) as e:
                B.equivalent(*pair)
            assert e.value.status == B.DFA_EINVAL
    check(d)
