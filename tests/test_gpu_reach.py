"""GPU tests of the reach pass (one lookup or walk per slot along the player's own sequence): sequences
shorter and longer than the walk that stays in registers (8 slots), in the level launches, which split the
pass there, and in the LDS-resident and persistent schedules, which walk every sequence whole."""
import numpy as np
import pytest

import gamegen as gg
import oracle
import paper_2609_11923_amd as cfr

pytestmark = pytest.mark.gpu


def chain(moves, seed=0):
    """A deal only player 1 sees, then both in turn stop (with a payoff) or go on, `moves` times each."""
    rng = np.random.default_rng(seed)
    ty, kids, probs, key, pay = [gg.GG_CHANCE], [[]], [[0.4, 0.6]], [-1], [0.0]

    def add(t, k):
        ty.append(t), kids.append([]), probs.append(None), key.append(k), pay.append(rng.uniform(-1, 1))
        return len(ty) - 1

    for deal in range(2):
        at = add(gg.GG_P1, 1000 * (deal + 1))
        kids[0].append(at)
        for step in range(1, 2 * moves):
            stop, nxt = add(gg.GG_TERMINAL, -1), add(
                gg.GG_P2 if step % 2 else gg.GG_P1, step if step % 2 else 1000 * (deal + 1) + step)
            kids[at] = [stop, nxt]
            at = nxt
        kids[at] = [add(gg.GG_TERMINAL, -1), add(gg.GG_TERMINAL, -1)]
    return gg.from_arrays(ty, kids, probs, key, pay, name=f"chain{moves}")


def state(s):
    return (*s.state(), s.strategy(), s.strategy(average=True))


@pytest.mark.parametrize("layout", [cfr.CFR_LAYOUT_PUBLIC, cfr.CFR_LAYOUT_BFS])
@pytest.mark.parametrize("precision", [cfr.CFR_PRECISION_FP32, cfr.CFR_PRECISION_FP64])
@pytest.mark.parametrize("moves", [1, 8, 9, 10, 17, 20])
def test_walks_of_every_length(moves, precision, layout):
    game = chain(moves)
    s = cfr.Solver(game, precision=precision, layout=layout)
    # a launch walks at most 8 slots, so sequences of 9 and 18 slots need a second and a third
    assert s.counts["kernels_per_iteration"] == s.counts["blocks"] + 1 + (moves - 1) // 9
    s.iterate(25)
    want = state(s)
    t = cfr.Solver(game, precision=precision, layout=layout, persistent=cfr.CFR_SCHEDULE_LDS)
    t.iterate(25)
    assert all(np.array_equal(a, b) for a, b in zip(want, state(t)))
    batch = cfr.Solver([game, gg.kuhn(), chain(3, 1)], precision=precision, layout=layout)
    batch.set_schedule(cfr.CFR_SCHEDULE_PERSISTENT, 1024)
    batch.iterate(25)
    R, S = batch.game_state(0)
    assert np.array_equal(R, want[0]) and np.array_equal(S, want[1])
    if precision == cfr.CFR_PRECISION_FP64:
        o = oracle.Oracle(game)
        o.iterate(25)
        Ro, So, _, sao = o.state()
        assert np.abs(want[0] - Ro).max() <= 1e-5 * np.abs(Ro).max()
        assert np.abs(want[1] - So).max() <= 1e-5 * np.abs(So).max()
        assert np.abs(want[3] - sao).max() <= 1e-5


def test_retired_games_keep_their_reach_tiles():
    """Two batches of small games whose slots share tiles: the active games iterate as in a batch of their own."""
    games = [chain(m, m) for m in (2, 12, 5, 20, 9)]
    s = cfr.Solver(games)
    s.iterate(5)
    s.set_active([1, 0, 1, 1, 0])
    s.iterate(7)
    for k in (0, 2, 3):
        alone = cfr.Solver(games[k])
        alone.iterate(12)
        assert all(np.array_equal(a, b) for a, b in zip(alone.state(), s.game_state(k)))
