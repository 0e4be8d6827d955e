"""GPU tests of the affine update's packed records: groups whose members' nodes and sequences need more than 32 bits
together keep wide records (several sets in a group, set-major and node-order lists), others the packed ones."""
import numpy as np
import pytest

import gamegen as gg
import paper_2609_11923_amd as cfr

pytestmark = pytest.mark.gpu


def spread(log_n, log_members, seed=0):
    """A deal of 2^log_n outcomes player 1 sees; he stops or goes on, and player 2, who sees the outcome modulo
    2^(log_n - log_members), chooses among three ends: his sets' members are far apart, and so are the
    sequences that lead to them."""
    n = 1 << log_n
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    one, two, stop, end = 1 + i, 1 + n + i, 1 + 2 * n + i, 1 + 3 * n
    N = 1 + 6 * n
    ty = np.full(N, gg.GG_TERMINAL, np.int8)
    ty[0], ty[one], ty[two] = gg.GG_CHANCE, gg.GG_P1, gg.GG_P2
    key = np.full(N, -1, np.int64)
    key[one], key[two] = n + i, i % (n >> log_members)
    kids = np.concatenate([one, np.stack([stop, two], 1).ravel(), (end + 3 * i[:, None] + np.arange(3)).ravel()])
    nc = np.zeros(N, np.int32)
    nc[0], nc[one], nc[two] = n, 2, 3
    prob = np.zeros(len(kids))
    prob[:n] = 1.0 / n
    pub = np.zeros(N, np.int64)
    pub[one], pub[two], pub[stop] = 1, 2, 3
    pub[end:] = 4 + np.arange(3 * n) % 3
    payoff = np.where(ty == gg.GG_TERMINAL, rng.uniform(-1, 1, N), 0.0)
    return gg.Game(type=ty, child_begin=np.concatenate([[0], np.cumsum(nc)[:-1]]).astype(np.int64), n_children=nc,
                   children=kids.astype(np.int64), prob=prob, key=key, payoff=payoff, pub=pub, name="spread")


@pytest.mark.parametrize("order", [cfr.CFR_ORDER_SIMULTANEOUS, cfr.CFR_ORDER_ALTERNATING])
@pytest.mark.parametrize("precision", [cfr.CFR_PRECISION_FP32, cfr.CFR_PRECISION_FP64])
@pytest.mark.parametrize("log_n,log_members", [(17, 1), (17, 3), (16, 5), (10, 3), (12, 11)])
def test_affine_records_equal_the_child_lists(log_n, log_members, precision, order):
    """2^17 outcomes span 17 bits of nodes and 18 of sequences (wide; with 8 members per set in node order), 2^16 with
    32 members 16 + 17 bits, 2^10 fit the packed word, and sets of 2,048 members need several chunks."""
    game = spread(log_n, log_members)
    kw = dict(precision=precision, order=order)
    a, b = cfr.Solver(game, **kw), cfr.Solver(game, affine=False, **kw)
    assert a.counts["child_addressing"] == 2 and b.counts["child_addressing"] == 1
    p = cfr.Solver(game, **kw)
    p.set_schedule(cfr.CFR_SCHEDULE_PERSISTENT, 65536)
    for s in (a, b, p):
        s.iterate(3)
    for x, y, z in zip(a.state(), b.state(), p.state()):
        assert np.array_equal(x, y) and np.array_equal(x, z)
    assert np.array_equal(a.strategy(), b.strategy())
    # the deal's sum is the same block's in both, the rest set by set
    assert a.exploitability() == b.exploitability()
