"""GPU tests of the evaluation sweep (all three values in one pass per level) and of the strategies' way out:
slots and chance nodes with terminal, internal and mixed children, chance nodes of one to many children
(8 lanes up to 64, a block above), action counts around the instantiations' bounds, groups of one and of
several staging chunks, in every child addressing."""
import numpy as np
import pytest
import torch

import gamegen as gg
import oracle
import paper_2609_11923_amd as cfr

pytestmark = pytest.mark.gpu


def deal(fan, seed=0, actions=3):
    """A chance root over `fan` outcomes that player 1 sees and player 2 does not; a third of them end the game."""
    rng = np.random.default_rng(seed)
    ty, kids, key, pay = [gg.GG_CHANCE], [[]], [-1], [0.0]

    def add(t, k=-1):
        ty.append(t), kids.append([]), key.append(k), pay.append(rng.uniform(-1, 1))
        return len(ty) - 1

    for c in range(fan):
        if c % 3 == 2:
            kids[0].append(add(gg.GG_TERMINAL))
            continue
        one = add(gg.GG_P1, 1000 + c)
        kids[0].append(one)
        two = add(gg.GG_P2, 1)
        kids[one] = [add(gg.GG_TERMINAL), two]
        kids[two] = [add(gg.GG_TERMINAL) for _ in range(actions)]
    p = rng.dirichlet(np.ones(fan))
    p[-1] = 1.0 - p[:-1].sum()
    return gg.from_arrays(ty, kids, [list(p)] + [None] * (len(ty) - 1), key, pay, name=f"deal{fan}")


GAMES = {**{f"deal{n}": (lambda n=n: deal(n)) for n in (1, 3, 4, 7, 8, 9, 64, 65, 256, 257, 1500)},
         "all_chance": lambda: gg.degenerate("all_chance"), "root_terminal": lambda: gg.degenerate("root_terminal"),
         "random7": lambda: gg.random_game(7, 4, 3, 6), "leduc3": lambda: gg.leduc(3, 2),
         "actions5": lambda: gg.random_game(3, 4, 4, 5, max_actions=5, max_chance=3),
         "actions8": lambda: gg.random_game(21, 5, 4, 5, max_actions=8, max_chance=3),
         "actions16": lambda: deal(7, actions=16), "actions17": lambda: deal(300, actions=17),
         "actions64": lambda: deal(20, actions=64)}


def averages(s):
    """The average strategy from the strategy sums, canonical order."""
    lay = s.layout()
    off = lay["slot_off"]
    S = s.state()[1]
    n = np.diff(off)
    tot = np.add.reduceat(S, off[:-1]) if len(n) else np.zeros(0)
    tot, n = np.repeat(tot, n), np.repeat(n, n)
    return np.where(tot > 0, S / np.where(tot > 0, tot, 1.0), 1.0 / n)


@pytest.mark.parametrize("how", ["affine", "listed", "bfs"])
@pytest.mark.parametrize("precision", [cfr.CFR_PRECISION_FP32, cfr.CFR_PRECISION_FP64])
@pytest.mark.parametrize("name", list(GAMES))
def test_values_and_strategies(name, precision, how):
    game = GAMES[name]()
    s = cfr.Solver(game, precision=precision, affine=how == "affine", keep_layout=True,
                   layout=cfr.CFR_LAYOUT_BFS if how == "bfs" else cfr.CFR_LAYOUT_PUBLIC)
    o = oracle.Oracle(game)
    o.iterate(12)
    s.iterate(12)
    # the oracle's profile, so that the sweep is all that is compared; FP64 sums of at most a few
    # thousand terms of magnitude <= 1 (chips <= 13 in Leduc) agree to 1e-12 of that
    _, So, _, _ = o.state()
    s.set_state(strategy_sum=So, t=12)
    want = o.exploitability()
    assert np.allclose(s.exploitability(), want, rtol=0, atol=2e-11)
    if s.A == 0:
        return
    avg = averages(s).astype(np.float32)
    # the sums of a set may be added in another order: one unit in the last place of the quotient
    assert np.allclose(s.strategy(average=True), avg, rtol=2e-7, atol=0)
    cur = s.strategy()
    for average, ref in ((True, s.strategy(average=True)), (False, cur)):
        # into a whole tensor, and into part of a larger one that begins off any 16-byte line
        out = torch.full((s.A + 3,), -1.0, device="cuda")
        s.strategy_into(out[1:], average=average)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.array_equal(got[1:-2], ref) and (got[[0, -2, -1]] == -1.0).all()
