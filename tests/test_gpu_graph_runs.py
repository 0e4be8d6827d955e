"""GPU test of the graph of several iterations that a handle with one iteration per graph captures once it has
replayed 32 of them: the iterates are bitwise those of direct launches on either side of the switch, with
strategies and evaluations read between the calls, and after games were retired and brought back."""
import numpy as np
import pytest

import gamegen as gg
import paper_2609_11923_amd as cfr

pytestmark = pytest.mark.gpu

ORDERS = {"sim": cfr.CFR_ORDER_SIMULTANEOUS, "alt": cfr.CFR_ORDER_ALTERNATING}


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a.state(), b.state())) and a.iterations == b.iterations


@pytest.mark.parametrize("order", list(ORDERS))
@pytest.mark.parametrize("games", [1, 3])
def test_runs_of_iterations_equal_direct_launches(games, order):
    trees = [gg.random_game(seed, 4, 3, 6) for seed in (7, 9, 11)][:games]
    print(f"[graph runs] {games} games {order}", flush=True)
    a, b = [cfr.Solver(trees if games > 1 else trees[0], rule=cfr.CFR_RULE_DCFR, order=ORDERS[order], use_graph=g)
            for g in (True, False)]
    # 32 replays end with the second call; the third takes no run, the others one or more and a remainder
    for n in (30, 3, 4, 5, 1, 17, 6):
        a.iterate(n)
        b.iterate(n)
        assert same(a, b), n
        assert np.array_equal(a.strategy(), b.strategy())
    if games > 1:
        for active in ([1, 0, 1], [1, 1, 1]):
            a.set_active(active)
            b.set_active(active)
            for n in (40, 12):
                a.iterate(n)
                b.iterate(n)
                assert same(a, b), (active, n)


@pytest.mark.parametrize("per_graph", [1, 5])
def test_a_failed_capture_of_several_iterations_stays_inside(per_graph):
    """HIP keeps a failed call's error until it is read: a capture that fails, where single iterations (or direct
    launches) go on, must not make the calls after it fail."""
    game = gg.random_game(7, 4, 3, 6)
    a = cfr.Solver(game, iters_per_graph=per_graph, test_fail_capture=2)
    b = cfr.Solver(game, use_graph=False)
    for n in (40, 12, 6, 40):
        a.iterate(n)
        b.iterate(n)
        assert np.array_equal(a.strategy(), b.strategy())
        assert same(a, b), n
    assert a.exploitability() == b.exploitability()
