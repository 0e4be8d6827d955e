"""GPU tests of games in which a player moves many times in a row, on the schedules that run whole iterations in one
launch: the reach pass goes in parts of at most eight own moves there, with a barrier between them (of one
workgroup or of several), and its cost grows with the number of moves, not with its square."""
import time

import numpy as np
import pytest
import torch

import gamegen as gg
import paper_2609_11923_amd as cfr
from test_gpu_reach import chain, state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [cfr.CFR_PRECISION_FP32, cfr.CFR_PRECISION_FP64])
@pytest.mark.parametrize("order", [cfr.CFR_ORDER_SIMULTANEOUS, cfr.CFR_ORDER_ALTERNATING])
@pytest.mark.parametrize("moves", [8, 9, 18, 19, 70])
def test_parts_of_long_sequences(moves, order, precision):
    game = chain(moves)
    s = cfr.Solver(game, precision=precision, order=order)
    s.iterate(12)
    want = state(s)
    lds = cfr.Solver(game, precision=precision, order=order, persistent=cfr.CFR_SCHEDULE_LDS)
    lds.iterate(12)
    assert all(np.array_equal(a, b) for a, b in zip(want, state(lds)))
    batch = cfr.Solver([chain(3, 1), game, chain(moves + 5, 2)], precision=precision, order=order)
    for wg_nodes in (16384, 64, 16):       # one workgroup a game, then up to dozens
        batch.reset()
        batch.set_schedule(cfr.CFR_SCHEDULE_PERSISTENT, wg_nodes)
        batch.iterate(12)
        R, S = batch.game_state(1)
        assert np.array_equal(R, want[0]) and np.array_equal(S, want[1]), wg_nodes


@pytest.mark.parametrize("schedule", [cfr.CFR_SCHEDULE_PERSISTENT, cfr.CFR_SCHEDULE_LDS])
def test_cost_grows_with_the_number_of_moves(schedule):
    def us(moves):
        s = cfr.Solver([chain(moves, k) for k in range(2)] if schedule == cfr.CFR_SCHEDULE_PERSISTENT else chain(moves))
        s.set_schedule(schedule)
        s.iterate(20)
        times = []
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            s.iterate(20)
            torch.cuda.synchronize()
            times.append((time.perf_counter() - t) / 20 * 1e6)
        return min(times)

    # ten times the moves: ten times the levels, where whole walks took a hundred times the lookups
    short, long = us(10), us(100)
    print(f"[long sequences] schedule {schedule}: 10 moves {short:.1f} us, 100 moves {long:.1f} us", flush=True)
    assert long <= 15 * short


def ragged(actions, goes_on, depth, cap, seed):
    """Every move is seen by both, who take turns; of a node's moves the first and a share of the others go on."""
    rng = np.random.default_rng(seed)
    T, kids, probs, key, pay, level = [gg.GG_P1], [[]], [None], [0], [0.0], [0]
    for d in range(1, depth + 1):
        below = []
        for x in level:
            for a in range(actions):
                leaf = d == depth or (a > 0 and rng.random() > goes_on) or len(below) >= cap
                T.append(gg.GG_TERMINAL if leaf else (gg.GG_P2 if d % 2 else gg.GG_P1))
                kids[x].append(len(T) - 1), kids.append([]), probs.append(None)
                key.append(-1 if leaf else len(T) - 1), pay.append(rng.uniform(-1, 1))
                if not leaf:
                    below.append(len(T) - 1)
        level = below
    return gg.from_arrays(T, kids, probs, key, pay, name=f"ragged{actions}")


# LDS: a walk per slot up to 256 slots of the game, a walk per set beyond; the last moves are left out of the pass
@pytest.mark.parametrize("precision", [cfr.CFR_PRECISION_FP32, cfr.CFR_PRECISION_FP64])
@pytest.mark.parametrize("actions,goes_on,depth,cap", [(2, 0.5, 7, 9), (3, 0.4, 12, 30), (4, 0.3, 8, 60), (5, 0.2, 4, 4),
                                                       (16, 0.1, 3, 7), (16, 0.1, 6, 40), (20, 0.1, 5, 30), (64, 0.1, 3, 9)])
def test_games_with_many_ends(actions, goes_on, depth, cap, precision):
    game = ragged(actions, goes_on, depth, cap, actions)
    print(f"[many ends] {actions} actions: {len(game.type)} nodes", flush=True)
    s = cfr.Solver(game, precision=precision)
    s.iterate(9)
    want = state(s)
    if actions <= 16:
        lds = cfr.Solver(game, precision=precision, persistent=cfr.CFR_SCHEDULE_LDS)
        lds.iterate(9)
        assert all(np.array_equal(a, b) for a, b in zip(want, state(lds)))
    batch = cfr.Solver([chain(3, 1), game, ragged(actions, goes_on, 3, 5, 9)], precision=precision)
    for wg_nodes in (16384, 100):
        batch.reset()
        batch.set_schedule(cfr.CFR_SCHEDULE_PERSISTENT, wg_nodes)
        batch.iterate(9)
        R, S = batch.game_state(1)
        assert np.array_equal(R, want[0]) and np.array_equal(S, want[1]), wg_nodes
