"""A plan run on another network of its shape: a program that keeps the order
and changes the weights. 64-bit counts are exact for the network they are of,
whatever entries and bound the plan was made with."""
import itertools
import math

import pytest

import instances as I
from paper_1805_00475_amd import tn

pytestmark = pytest.mark.gpu


def _weighted_path(n, weights):
    cons = [((v,), list(weights[v - 1])) for v in range(1, n + 1)]
    cons += [((v, v + 1), [1, 1, 1, 0]) for v in range(1, n)]
    return I.CSP(n, [2] * n, cons)


def _brute(n, weights):
    total = 0
    for x in itertools.product((0, 1), repeat=n):
        if all(not (x[v] and x[v + 1]) for v in range(n - 1)):
            total += math.prod(weights[v][x[v]] for v in range(n))
    return total


@pytest.mark.parametrize("top", [100, 200, 300, 4095])
def test_larger_entries(top):
    n = 5
    plan = tn.Network(_weighted_path(n, [(1, 2)] * n)).order("greedy", 0)
    w = [(top - v, top) for v in range(n)]
    print("[gpu case] plan reuse, entries up to", top, flush=True)
    net = tn.Network(_weighted_path(n, w))
    assert tn.moduli(plan) == []
    assert tn.count_plan(net, plan) == _brute(n, w)
    assert tn.count_plan(net, plan, flags=tn.FLAG_GENERIC_ONLY) == _brute(n, w)


def test_larger_counts_of_a_wide_plan():
    # 3-CNF as a weighted network; the same with two tables times 1000 counts
    # 10^6 times as much, beyond the bound the plan was made with
    rng = I.Rng(2)
    f = I.exactly_one_3(40, 48, rng)
    cons = [(tuple(abs(v) for v in c), [0] + [1] * 7) for _, c in f.clauses]
    big = [(s, [1000 * x for x in t] if k in (5, 30) else t) for k, (s, t) in enumerate(cons)]
    a, b = (tn.Network(I.CSP(40, [2] * 40, c)) for c in (cons, big))
    plan = a.order("best", 2, rounds=1)
    assert plan.stats["macs"] >= 2 ** 25 and tn.moduli(plan) == []
    print("[gpu case] plan reuse, wide plan", flush=True)
    want = tn.count(I.Formula(40, [(I.OR, list(s)) for s, _ in cons]))
    assert 2 ** 48 < 10 ** 6 * want < 2 ** 63
    assert tn.count_plan(a, plan) == want
    assert tn.count_plan(b, plan) == 10 ** 6 * want
    assert tn.count_plan(b, plan, arith="u64") == 10 ** 6 * want
