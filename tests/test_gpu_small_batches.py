"""Batches of so many small DFAs that workgroups of few threads take them, and
larger ones in the same call: every size around the line, the largest and the
smallest jobs, rows in LDS and not, a bad target.  Against the oracle, equal.
"""
import numpy as np
import pytest

import oracle
from paper_2508_20735_amd import binding as B
from paper_2508_20735_amd import workloads as W

pytestmark = pytest.mark.gpu

MANY = 1100  # more than four jobs for each of 256 CUs


def dfas(sizes, ks, seed):
    """MANY DFAs of these sizes and letters, 24 different ones of each."""
    kinds = [(n, k) for n in sizes for k in ks]
    made = {}
    out = []
    for i in range(MANY):
        n, k = kinds[i % len(kinds)]
        s = (i // len(kinds)) % 24
        if (n, k, s) not in made:
            made[n, k, s] = W.random_dfa(n, k, 0.3, seed + 131 * s + n + k)
        out.append(made[n, k, s])
    return out


def answers(ds):
    ref = {}
    for d in ds:
        if id(d) not in ref:
            ref[id(d)] = oracle.moore(d.delta, d.accepting)
    return ref


def check(ds):
    ref = answers(ds)
    blocks, nb, rounds, _ = B.minimise_batch(ds)
    for i, d in enumerate(ds):
        block, num, ran, changing = ref[id(d)]
        np.testing.assert_array_equal(blocks[i], block, err_msg=str((i, d.n, d.k)))
        assert (nb[i], rounds[i]) == (num, ran), (i, d.n, d.k)


@pytest.mark.parametrize("ks", [(1, 2, 3), (5, 8), (9, 16), (16, 17)], ids=str)
@pytest.mark.parametrize("sizes", [(1, 2, 63), (64, 65, 257), (1000, 1023, 1024), (1025, 40),
                                   (4096, 5, 700)], ids=str)
def test_minimise(sizes, ks):
    check(dfas(sizes, ks, 1))


@pytest.mark.parametrize("ks", [(1, 2, 4), (7, 16)], ids=str)
@pytest.mark.parametrize("sizes", [(1, 31, 32), (511, 512, 513), (2048, 30)], ids=str)
def test_equivalent(sizes, ks):
    a = dfas(sizes, ks, 2)
    b = [W.mutate_one(d, i)[0] if i % 2 and d.n > 1 else W.permuted_copy(d, i)[0]
         for i, d in enumerate(a)]
    got = B.equivalent_batch(list(zip(a, b)))[0]
    want = [oracle.equiv_hk(x.delta, x.accepting, x.start, y.delta, y.accepting, y.start)
            for x, y in zip(a, b)]
    assert list(map(bool, got)) == want


@pytest.mark.parametrize("bad", [0, 1, MANY - 1])
def test_a_target_out_of_range(bad):
    ds = dfas((4000, 40, 41), (3,), 3)
    delta = ds[bad].delta.copy()
    delta[-1, -1] = ds[bad].n
    ds[bad] = W.DFA(delta, ds[bad].accepting, 0)
    with pytest.raises(B.DfaError):
        B.minimise_batch(ds)
    check(dfas((30,), (3,), 4))
