"""The workloads on which the speed of this package is measured.

Every case is one call through the package's public entry points, on inputs
of the families and size ranges that the benchmark, the tests and the serving
workload use: random complete DFAs of 1,000 to 2^22 states and 2 to 16
letters, chains, the paper's families, batches of small DFAs.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  the inputs a program holds before the call
  run(state)           the call; returns its whole outputs
  work(case)           bytes the call cannot do without
  exact(case, seed)    the same outputs from plain torch, without the library
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2508_20735_amd import binding as B
from paper_2508_20735_amd import workloads as W

LETTERS = (2, 4, 8, 16)


def listed() -> list[dict]:
    return [
        # the smallest request of the serving mix: latency and launches only
        {"name": "min_1k_k4", "kind": "minimise", "n": 1009, "k": 4, "p": 0.3, "dup": 0.2,
         "quotient": True},
        # a program that holds its DFA in host memory and wants the minimal
        # DFA back there (copies both ways included)
        {"name": "min_host_100k_k4", "kind": "minimise_host", "n": 100_003, "k": 4, "p": 0.2,
         "dup": 0.2, "quotient": True},
        # an ordinary request of the serving mix with its widest alphabet
        {"name": "min_300k_k16", "kind": "minimise", "n": 300_007, "k": 16, "p": 0.4, "dup": 0.1,
         "quotient": False},
        # the benchmark's random DFA: minimal DFA, resident in device memory
        {"name": "min_4m_k4", "kind": "minimise", "n": 1 << 22, "k": 4, "p": 0.1, "dup": 0.0,
         "quotient": True},
        # the benchmark's equivalence against a renamed copy (equal languages:
        # every round runs), at its size
        {"name": "eq_perm_4m_k4", "kind": "equivalent", "n": 1 << 22, "k": 4, "p": 0.1,
         "dup": 0.05, "mutate": False},
        # equivalence against a copy with one redirected transition: few
        # blocks change per round, many rounds
        {"name": "eq_mut_500k_k8", "kind": "equivalent", "n": 500_009, "k": 8, "p": 0.25,
         "dup": 0.1, "mutate": True},
        # the chain-structured workload: splitting stalls and the closure is
        # switched on
        {"name": "chain_2m_k4", "kind": "chain", "chain": 1 << 20, "tail": 1 << 20, "k": 4},
        # many small DFAs in one call: minimisation, then equivalence pairs
        {"name": "batch_min_1024", "kind": "batch_minimise", "count": 1024, "mix": 4,
         "nmin": 64, "nmax": 65_536},
        {"name": "batch_eq_512", "kind": "batch_equivalent", "count": 512, "mix": 5,
         "nmin": 64, "nmax": 65_536},
        # inclusion in a DFA that accepts more: the whole reachable product is
        # explored
        {"name": "incl_2m_k4", "kind": "included", "n": 2_097_169, "k": 4, "p": 0.1,
         "holds": True},
        # the usual minimal DFA: unreachable states pruned first
        {"name": "prune_1m_k2", "kind": "prune", "n": 1_048_583, "k": 2, "p": 0.3, "dup": 0.1,
         "quotient": False},
        # the paper's leader rounds (Table 2's naivePR) on a bit-splitter
        {"name": "leader_b18", "kind": "leader", "bits": 18},
    ]


def _log_size(rng, lo: int, hi: int) -> int:
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng) -> dict:
    kind = rng.choice(["minimise", "minimise", "minimise_host", "equivalent", "equivalent", "chain",
                       "batch_minimise", "batch_equivalent", "included", "prune", "leader"])
    p = round(rng.uniform(0.05, 0.5), 3)
    dup = round(rng.uniform(0.05, 0.3), 3)
    k = rng.choice(LETTERS)
    if kind == "minimise":
        return {"kind": kind, "n": _log_size(rng, 1000, (1 << 24) // max(k, 4)), "k": k, "p": p,
                "dup": dup, "quotient": k >= 4 and rng.random() < 0.7}
    if kind == "minimise_host":
        return {"kind": kind, "n": _log_size(rng, 1000, 400_000), "k": k, "p": p, "dup": dup,
                "quotient": k >= 4 and rng.random() < 0.7}
    if kind == "equivalent":
        return {"kind": kind, "n": _log_size(rng, 1000, (1 << 23) // max(k, 4)), "k": k, "p": p,
                "dup": dup, "mutate": rng.random() < 0.5}
    if kind == "chain":
        n = _log_size(rng, 1000, 1 << 19)
        return {"kind": kind, "chain": n, "tail": n + rng.randrange(2), "k": 4}
    if kind in ("batch_minimise", "batch_equivalent"):
        return {"kind": kind, "count": _log_size(rng, 96, 512), "mix": rng.randrange(1 << 20),
                "nmin": 64, "nmax": _log_size(rng, 1000, 65_536)}
    if kind == "included":
        k = min(k, 8)
        return {"kind": kind, "n": _log_size(rng, 1000, (1 << 22) // k), "k": k, "p": p,
                "holds": rng.random() < 0.7}
    if kind == "prune":
        k = min(k, 4)
        return {"kind": kind, "n": _log_size(rng, 1000, (1 << 21) // k), "k": k, "p": p,
                "dup": dup, "quotient": False}
    return {"kind": kind, "bits": rng.randint(10, 18)}


# ---------------------------------------------------------------- inputs

def _renamed(d: W.DFA, mask: int) -> W.DFA:
    """The same automaton with state s named s ^ mask (2^m states): other
    inputs for other seeds, the locality of the family's own numbering kept."""
    s = np.arange(d.n, dtype=np.uint32) ^ np.uint32(mask)
    return W.DFA((d.delta ^ np.uint32(mask))[s], d.accepting[s], int(d.start) ^ mask)


def _random(case: dict, seed: int, exact_share: bool = True) -> W.DFA:
    """A random complete DFA of which the share `dup` of the states are copies
    of other states (same acceptance, transitions to the target or to a copy
    of it), in a random order of the names; exactly that share of them, or
    a number near it that the seed decides."""
    n, dup = case["n"], case.get("dup", 0.0)
    if not dup:
        return W.random_dfa(n, case["k"], case["p"], seed)
    rng = np.random.Generator(np.random.PCG64([seed, 77]))
    copies = int(n * dup * (1.0 if exact_share else rng.uniform(0.5, 1.5)))
    m = n - copies
    base = W.random_dfa(m, case["k"], case["p"], seed)
    of = np.concatenate([np.arange(m), rng.integers(0, m, copies)])  # the state copied
    twin = np.arange(m, dtype=np.uint32)  # the state itself, or one of its copies
    twin[of[m:]] = np.arange(m, n, dtype=np.uint32)
    delta = base.delta[of]
    delta = np.where(rng.integers(0, 2, delta.shape, dtype=np.uint8) == 1, twin[delta], delta)
    return W.permuted_copy(W.DFA(delta, base.accepting[of], 0), seed + 3)[0]


def _other(d: W.DFA, mutate: bool, seed: int) -> W.DFA:
    return W.mutate_one(d, seed)[0] if mutate else W.permuted_copy(d, seed)[0]


def _mix(case: dict) -> list[tuple[int, int, float]]:
    """Sizes, letters and acceptance rates of a batch (the same for every seed)."""
    rng = np.random.Generator(np.random.PCG64(case["mix"]))
    c = case["count"]
    ns = np.rint(np.exp(rng.uniform(math.log(case["nmin"]), math.log(case["nmax"]), size=c)))
    ks = rng.integers(2, 9, size=c)
    ps = rng.uniform(0.05, 0.5, size=c)
    return [(int(n), int(k), float(p)) for n, k, p in zip(ns, ks, ps)]


def _dfas(case: dict, seed: int) -> list[W.DFA]:
    """The automata of a case, on the host, from the seed alone."""
    kind = case["kind"]
    if kind in ("minimise", "minimise_host", "prune"):
        return [_random(case, seed)]
    if kind == "equivalent":
        d = _random(case, seed, exact_share=False)
        return [d, _other(d, case["mutate"], seed + 1)]
    if kind == "chain":
        return [W.chain_with_tail(case["chain"], case["tail"], seed, k=case["k"])]
    if kind == "batch_minimise":
        return [W.random_dfa(n, k, p, seed * 65_537 + i) for i, (n, k, p) in enumerate(_mix(case))]
    if kind == "batch_equivalent":
        a = [W.random_dfa(n, k, p, seed * 65_537 + i) for i, (n, k, p) in enumerate(_mix(case))]
        return a + [_other(d, i % 2 == 1, seed * 65_537 + i + 1) for i, d in enumerate(a)]
    if kind == "included":
        # the second accepts whatever the first does, and in up to 16 more
        # states; the other way round the inclusion fails at the first of them
        d = W.random_dfa(case["n"], case["k"], case["p"], seed)
        more = W.permuted_copy(d, seed + 1)[0]
        rng = np.random.Generator(np.random.PCG64(seed + 2))
        more.accepting[rng.integers(0, more.n, 16)] = 1
        return [d, more] if case["holds"] else [more, d]
    rng = np.random.Generator(np.random.PCG64(seed))
    return [_renamed(W.bitsplitter(case["bits"]), int(rng.integers(0, 1 << case["bits"])))]


def _gpu(d: W.DFA):
    dev = torch.device("cuda:0")
    return (torch.from_numpy(d.delta.view(np.int32)).to(dev), torch.from_numpy(d.accepting).to(dev),
            d.start)


def prepare(case: dict, seed: int) -> dict:
    kind = case["kind"]
    dfas = _dfas(case, seed)
    if kind == "minimise_host":
        return {"case": case, "dfas": dfas}
    if kind == "batch_minimise":
        batch = B.PackedBatch.from_dfas(dfas)
        out = torch.empty(batch.states, dtype=torch.int32, device="cuda:0")
        return {"case": case, "batch": batch, "out": out}
    if kind == "batch_equivalent":
        half = len(dfas) // 2
        return {"case": case, "a": B.PackedBatch.from_dfas(dfas[:half]),
                "b": B.PackedBatch.from_dfas(dfas[half:])}
    return {"case": case, "dfas": [_gpu(d) for d in dfas]}


# ---------------------------------------------------------------- the call

def _minimised(res) -> dict:
    out = {"block": res.block, "num_blocks": res.stats["num_blocks"]}
    if res.quotient is not None:
        out["quotient"] = list(res.quotient)
    return out


def run(state: dict):
    case = state["case"]
    kind = case["kind"]
    if kind == "minimise_host":
        d = state["dfas"][0]
        return _minimised(B.minimise(d.delta, d.accepting, quotient=case["quotient"]))
    if kind == "batch_minimise":
        nb, rounds, _ = B.minimise_batch_device(state["batch"], None, state["out"])
        return {"block": state["out"], "num_blocks": nb, "rounds": rounds}
    if kind == "batch_equivalent":
        return {"verdicts": B.equivalent_batch_device(state["a"], state["b"])[0]}
    delta, acc, start = state["dfas"][0]
    if kind == "minimise":
        return _minimised(B.minimise_device(delta, acc, start=start, quotient=case["quotient"]))
    if kind == "prune":
        return _minimised(B.minimise_device(delta, acc, start=start, quotient=case["quotient"],
                                            prune=True))
    if kind == "chain":
        return _minimised(B.minimise_device(delta, acc, start=start, quotient=True))
    if kind == "leader":
        return _minimised(B.minimise_device(delta, acc, start=start, quotient=True,
                                            algorithm="leader", tc="off"))
    delta2, acc2, start2 = state["dfas"][1]
    if kind == "equivalent":
        verdict, stats = B.equivalent_device(delta, acc, start, delta2, acc2, start2)
        return {"verdict": verdict, "num_blocks": stats["num_blocks"]}
    verdict, pairs, _ = B.included_device(delta, acc, start, delta2, acc2, start2)
    return {"verdict": verdict, "pairs": pairs}


def work(case: dict) -> dict:
    """Inputs read once, outputs written once (a quotient is counted as large
    as the input)."""
    kind = case["kind"]
    if kind in ("batch_minimise", "batch_equivalent"):
        mix = _mix(case)
        one = sum(n * (4 * k + 1) for n, k, _ in mix)
        outputs = sum(4 * n for n, _, _ in mix) if kind == "batch_minimise" else 4 * len(mix)
        return {"bytes": (1 if kind == "batch_minimise" else 2) * one + outputs, "flops": 0}
    if kind == "leader":
        n, k = 1 << case["bits"], case["bits"] - 1
    elif kind == "chain":
        n, k = case["chain"] + case["tail"], case["k"]
    else:
        n, k = case["n"], case["k"]
    one = n * (4 * k + 1)
    if kind == "included" and not case["holds"]:
        return {"bytes": 1 << 12, "flops": 0}  # a few levels, then the refuting pair
    if kind in ("equivalent", "included"):
        return {"bytes": 2 * one, "flops": 0}
    quotient = one if case.get("quotient", True) else 0
    return {"bytes": one + 4 * n + quotient, "flops": 0}


# ---------------------------------------------------------------- plain torch

def _moore(delta, acc, stop=None):
    """Signature rounds with torch.unique: (labels, blocks, rounds).  stop =
    two states: ends once they are separated."""
    labels = acc.long()
    blocks = int(labels.unique().numel())
    rounds = 0
    while True:
        new = labels
        for a in range(delta.shape[1]):
            new = (new << 32) | labels[delta[:, a]]
            new = torch.unique(new, return_inverse=True)[1]
        rounds += 1
        count = int(new.max()) + 1
        if count == blocks:
            return labels, blocks, rounds
        labels, blocks = new, count
        if stop is not None and int(labels[stop[0]]) != int(labels[stop[1]]):
            return labels, blocks, rounds


def _canonical(labels):
    n = labels.numel()
    first = torch.full((int(labels.max()) + 1,), n, dtype=torch.int64, device=labels.device)
    first.scatter_reduce_(0, labels, torch.arange(n, device=labels.device), "amin")
    return first[labels]


def _plain(d: W.DFA):
    return (torch.from_numpy(d.delta.astype(np.int64)).cuda(),
            torch.from_numpy(d.accepting).cuda())


def _minimise_plain(delta, acc, start: int, quotient: bool):
    labels, blocks, _ = _moore(delta, acc)
    block = _canonical(labels)
    out = {"block": block, "num_blocks": blocks}
    if quotient:
        leaders = torch.nonzero(block == torch.arange(block.numel(), device=block.device))[:, 0]
        dense = torch.empty_like(block)
        dense[leaders] = torch.arange(blocks, device=block.device)
        qd = dense[block[delta[leaders]]]
        out["quotient"] = [blocks, qd, acc[leaders], int(dense[block[start]])]
    return out


def _reachable(delta, start: int):
    seen = torch.zeros(delta.shape[0], dtype=torch.bool, device=delta.device)
    front = torch.tensor([start], device=delta.device)
    seen[front] = True
    while front.numel():
        nxt = delta[front].reshape(-1).unique()
        front = nxt[~seen[nxt]]
        seen[front] = True
    return torch.nonzero(seen)[:, 0]


def _narrow(out: dict) -> dict:
    """64-bit results in the types of the library's outputs."""
    out["block"] = out["block"].to(torch.int32)
    if "quotient" in out:
        q = out["quotient"]
        q[1], q[2] = q[1].to(torch.int32), q[2].to(torch.uint8)
    return out


def exact(case: dict, seed: int):
    kind = case["kind"]
    if kind == "chain":
        return None  # as many rounds as the chain has states
    dfas = _dfas(case, seed)
    if kind == "batch_minimise":
        blocks, nb, rounds = [], [], []
        for d in dfas:
            labels, b, r = _moore(*_plain(d))
            blocks.append(_canonical(labels).to(torch.int32))
            nb.append(b)
            rounds.append(r)
        return {"block": torch.cat(blocks), "num_blocks": np.array(nb, dtype=np.uint32),
                "rounds": np.array(rounds, dtype=np.uint32)}
    if kind in ("batch_equivalent", "equivalent"):
        half = len(dfas) // 2
        same, blocks = [], 0
        for x, y in zip(dfas[:half], dfas[half:]):
            (dx, ax), (dy, ay) = _plain(x), _plain(y)
            stop = (x.start, x.n + y.start)
            labels, blocks, _ = _moore(torch.cat([dx, dy + x.n]), torch.cat([ax, ay]), stop)
            same.append(bool(labels[stop[0]] == labels[stop[1]]))
        if kind == "equivalent":
            return {"verdict": same[0], "num_blocks": blocks}
        return {"verdicts": np.array(same)}
    if kind == "included":
        (dx, ax), (dy, ay) = _plain(dfas[0]), _plain(dfas[1])
        front = torch.tensor([(dfas[0].start << 32) | dfas[1].start], device=dx.device)
        seen = front
        while front.numel():
            p, q = front >> 32, front & 0xFFFFFFFF
            if bool(((ax[p] != 0) & (ay[q] == 0)).any()):
                return {"verdict": False, "pairs": int(seen.numel())}
            nxt = ((dx[p] << 32) | dy[q]).reshape(-1).unique()
            at = torch.searchsorted(seen, nxt).clamp_(max=seen.numel() - 1)
            front = nxt[seen[at] != nxt]
            seen = torch.cat([seen, front]).sort()[0]
        return {"verdict": True, "pairs": int(seen.numel())}
    d = dfas[0]
    delta, acc = _plain(d)
    if kind == "prune":
        kept = _reachable(delta, d.start)
        number = torch.full((d.n,), -1, dtype=torch.int64, device=delta.device)
        number[kept] = torch.arange(kept.numel(), device=delta.device)
        out = _minimise_plain(number[delta[kept]], acc[kept], int(number[d.start]),
                              case["quotient"])
        block = torch.full((d.n,), -1, dtype=torch.int64, device=delta.device)
        block[kept] = kept[out["block"]]
        out["block"] = block
        return _narrow(out)
    out = _narrow(_minimise_plain(delta, acc, d.start, case.get("quotient", True)))
    if kind == "minimise_host":  # unsigned host arrays
        out["block"] = out["block"].cpu().numpy().view(np.uint32)
        if "quotient" in out:
            q = out["quotient"]
            q[1], q[2] = q[1].cpu().numpy().view(np.uint32), q[2].cpu().numpy()
    return out
