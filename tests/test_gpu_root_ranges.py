"""GPU test of the template rewrite under new root ranges: ranges that travel in the launch's arguments (together at
most 256 weights) and longer ones that go through a copy of the root's chances both give, bitwise, the solve of
set_root_chance with p(a) = r1 r2 / W, and a later set_payoffs reads the chances they left."""
import dataclasses

import numpy as np
import pytest

import gamegen as gg
import paper_2609_11923_amd as cfr

pytestmark = pytest.mark.gpu


def dealt(n1, n2, pairs):
    """A chance root of `pairs` joint deals; under each, player 1 (one set per hand) picks one of two payoffs."""
    rng = np.random.default_rng(n1)
    h1, h2 = np.arange(pairs) % n1, np.arange(pairs) * 7 % n2
    kind, kids, probs, key, pay = [0], [[]], [None], [-1], [0.0]
    for a in range(pairs):
        n = len(kind)
        kids[0].append(n)
        kind += [1, 3, 3]
        kids += [[n + 1, n + 2], [], []]
        probs += [None, None, None]
        key += [int(h1[a]), -1, -1]
        pay += [0.0, *rng.uniform(-1, 1, 2)]
    probs[0] = [1.0 / pairs] * pairs
    game = gg.from_arrays(kind, kids, probs, key, pay)
    return dataclasses.replace(game, meta=dict(hands1=list(range(n1)), hands2=list(range(n2)), pair_h1=h1, pair_h2=h2))


@pytest.mark.parametrize("precision", [cfr.CFR_PRECISION_FP32, cfr.CFR_PRECISION_FP64])
@pytest.mark.parametrize("n1,n2,pairs", [(1, 1, 1), (3, 2, 6), (128, 128, 400), (1, 255, 255), (129, 128, 400),
                                         (1, 256, 300), (300, 2, 1000)])
def test_ranges_equal_the_root_chance_they_give(n1, n2, pairs, precision):
    print(f"[root ranges] {n1}+{n2} hands, {pairs} deals, precision {precision}", flush=True)
    game = dealt(n1, n2, pairs)
    rng = np.random.default_rng(5)
    r1, r2 = rng.uniform(0.1, 1, n1), rng.uniform(0.1, 1, n2)
    w = r1[game.meta["pair_h1"]] * r2[game.meta["pair_h2"]]
    total = 0.0
    for x in w:   # the sum in child order
        total += float(x)
    a, b = [cfr.Solver(game, precision=precision, lifecycle=True) for _ in range(2)]
    a.set_root_ranges(r1, r2)
    b.set_root_chance(w / total)
    payoff = np.array(game.payoff) * 0.75
    for step in range(2):
        a.iterate(9)
        b.iterate(9)
        assert all(np.array_equal(x, y) for x, y in zip(a.state(), b.state())), step
        assert a.exploitability() == b.exploitability()
        a.set_payoffs(payoff)
        b.set_payoffs(payoff)
