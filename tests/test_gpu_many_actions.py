"""GPU tests of the affine update's slot pass with five to sixteen actions per set and FP32 state: a group's child
offsets and strategy go through LDS 256 slots at a time, up to the group's last slot."""
import time

import numpy as np
import pytest
import torch

import gamegen as gg
import paper_2609_11923_amd as cfr

pytestmark = pytest.mark.gpu


def singles(sets, actions, seed):
    """A deal that player 1 alone sees, `sets` ways; he takes one of `actions` actions, player 2 answers unseen."""
    rng = np.random.default_rng(seed)
    p = rng.uniform(0.1, 1.0, sets)
    T, kids, probs, key, pay, pub = [0], [[]], [list(p / p.sum())], [-1], [0.0], [0]

    def add(parent, t, k, s):
        T.append(t), kids.append([]), probs.append(None), key.append(k), pay.append(rng.uniform(-1, 1)), pub.append(s)
        kids[parent].append(len(T) - 1)
        return len(T) - 1

    for i in range(sets):
        one = add(0, gg.GG_P1, i, 1)
        for a in range(actions):
            two = add(one, gg.GG_P2, 10**6 + a, 2 + a)
            for b in range(2):
                add(two, gg.GG_TERMINAL, -1, 2 + actions + 2 * a + b)
    return gg.from_arrays(T, kids, probs, key, pay, pub=pub, name=f"singles{sets}x{actions}")


def tree(actions, depth):
    """Every move is seen by both, who take turns: each decision node is a set of its own."""
    rng = np.random.default_rng(3)
    T, kids, probs, key, pay, level = [gg.GG_P1], [[]], [None], [0], [0.0], [0]
    for d in range(1, depth + 1):
        below = []
        for x in level:
            for _ in range(actions):
                below.append(len(T))
                kids[x].append(len(T)), kids.append([]), probs.append(None)
                T.append(gg.GG_TERMINAL if d == depth else (gg.GG_P2 if d % 2 else gg.GG_P1))
                key.append(len(T) - 1), pay.append(rng.uniform(-1, 1))
        level = below
    return gg.from_arrays(T, kids, probs, key, pay, name=f"tree{actions}^{depth}")


# slots of a group on both sides of a round (256) and of four (1,024), and the most there are (4,096)
@pytest.mark.parametrize("sets,actions", [(1, 5), (51, 5), (52, 5), (204, 5), (205, 5), (16, 16), (17, 16), (64, 16),
                                          (65, 16), (256, 16), (257, 16), (100, 11)])
@pytest.mark.parametrize("rule,order", [(cfr.CFR_RULE_CFR_PLUS, cfr.CFR_ORDER_SIMULTANEOUS),
                                        (cfr.CFR_RULE_DCFR, cfr.CFR_ORDER_ALTERNATING)])
def test_slot_counts(sets, actions, rule, order):
    game = singles(sets, actions, sets)
    a, b = [cfr.Solver(game, rule=rule, order=order, affine=f) for f in (True, False)]
    assert (a.counts["child_addressing"], b.counts["child_addressing"]) == (2, 1)
    for s in (a, b):
        s.iterate(20)
    assert all(np.array_equal(x, y) for x, y in zip((*a.state(), a.strategy()), (*b.state(), b.strategy())))


# bars half way between the sixteen-round slot pass (1.22 and 1.10 times the child lists) and this one (1.03 and 0.94)
@pytest.mark.parametrize("actions,depth,bar", [(6, 3, 1.13), (5, 6, 1.02)])
def test_small_groups_cost_no_more_than_child_lists(actions, depth, bar):
    """The affine update reads less than the child-list update and must not take longer on groups of few slots."""
    game = tree(actions, depth)
    solvers = [cfr.Solver(game, affine=f) for f in (True, False)]
    best = [1e9, 1e9]
    for _ in range(12):
        for k, s in enumerate(solvers):
            torch.cuda.synchronize()
            t = time.perf_counter()
            s.iterate(100)
            torch.cuda.synchronize()
            best[k] = min(best[k], (time.perf_counter() - t) * 1e4)
    print(f"[many actions] {actions}^{depth}: affine {best[0]:.2f} us, child lists {best[1]:.2f} us", flush=True)
    assert best[0] <= bar * best[1]
