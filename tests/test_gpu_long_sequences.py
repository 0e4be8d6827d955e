"""GPU tests of games in which a player moves many times in a row, on the schedules that run whole iterations in one
launch: the reach pass goes in parts of at most eight own moves there, with a barrier between them (of one
workgroup or of several), and its cost grows with the number of moves, not with its square."""
import time

import numpy as np
import pytest
import torch

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
