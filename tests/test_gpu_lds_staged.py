"""GPU test of the LDS schedule's instantiations: games of at most two actions and wider ones, with the structure
arrays beside the state in LDS (small games) and without (the state fits a workgroup's 160 KiB, both do not).  Each
gives bitwise the state of the level launches and counts its iterations."""
import numpy as np
import pytest

import gamegen as gg
import paper_2609_11923_amd as cfr

pytestmark = pytest.mark.gpu

# nodes and bytes in FP32: state alone, state and structure
GAMES = {
    "two actions, 811 nodes, staged": lambda: gg.random_game(4, 3, 3, 6, p_terminal=0.15, max_actions=2),
    "two actions, 156 KB with the structure, staged": lambda: gg.random_game(8, 4, 4, 10, p_terminal=0.12, max_actions=2),
    "two actions, 172 KB with the structure": lambda: gg.random_game(8, 4, 4, 12, p_terminal=0.12, max_actions=2),
    "two actions, 153 KB of state alone": lambda: gg.random_game(29, 4, 4, 12, p_terminal=0.12, max_actions=2),
    "three actions, staged": lambda: gg.random_game(7, 4, 3, 6),
    "one action": lambda: gg.random_game(2, 3, 3, 6, p_terminal=0.15, max_actions=2),
}


@pytest.mark.parametrize("rule,order", [(cfr.CFR_RULE_CFR_PLUS, cfr.CFR_ORDER_SIMULTANEOUS),
                                        (cfr.CFR_RULE_DCFR, cfr.CFR_ORDER_ALTERNATING)])
@pytest.mark.parametrize("name", list(GAMES))
def test_every_instantiation_equals_level_launches(name, rule, order):
    print(f"[lds] {name} rule {rule}", flush=True)
    game = GAMES[name]()
    a, b = [cfr.Solver(game, rule=rule, order=order, persistent=p)
            for p in (cfr.CFR_SCHEDULE_LDS, cfr.CFR_SCHEDULE_LEVEL)]
    for n in (1, 12):
        a.iterate(n)
        b.iterate(n)
    assert a.iterations == b.iterations == 13
    assert all(np.array_equal(x, y) for x, y in zip(a.state(), b.state()))
    assert np.array_equal(a.strategy(), b.strategy())
