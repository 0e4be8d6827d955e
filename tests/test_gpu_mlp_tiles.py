"""GPU tests of the network's row tiles: 32 rows per block up to 8,192 rows and 128 beyond, ragged tiles, and the
training step's pieces on both sides of that line (the weight sum inside the blocks or before them, 16-row
bias partials, row splits of the weight gradients)."""
import numpy as np
import pytest
import torch

import gamegen as gg
import paper_2609_11923_amd as cfr
from oracle import mlp as om

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [(i, h) for i in (64, 128, 256) for h in (64, 128, 256)]


def net(n_in, hidden, layers, max_rows, seed=0):
    m = cfr.Mlp(in_dim=n_in, hidden=hidden, n_hidden=layers, max_rows=max_rows)
    sizes = om.layer_sizes(n_in, hidden, layers, om.OUT)
    theta = gg.mlp_init(sizes, seed)
    m.set_params(theta)
    return m, sizes, theta.astype(np.float64)


def rows_of(n, n_in, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn(n, n_in, generator=g, device=DEV).to(torch.bfloat16)
    nact = torch.randint(1, 5, (n,), generator=g, device=DEV)
    T = torch.rand(n, 4, generator=g, device=DEV) * (torch.arange(4, device=DEV)[None] < nact[:, None])
    T = (T / T.sum(1, keepdim=True)).contiguous()
    return x, T, 0.1 + torch.rand(n, generator=g, device=DEV), nact.to(torch.uint8)


@pytest.mark.parametrize("n_in,hidden", SHAPES)
def test_logits_do_not_depend_on_the_tile(n_in, hidden):
    """A row's logits are bitwise the same in a call of any size: the large tile against slices that take the small."""
    m, _, _ = net(n_in, hidden, 3, 64)
    n = 8192 + 128 + 37
    x = rows_of(n, n_in, 1)[0]
    whole = torch.full((n + 1, 4), float("nan"), device=DEV)
    m.forward(x, n, whole)
    for lo, hi in ((0, 1), (5, 36), (100, 133), (8, 8200), (n - 65, n), (n - 1, n)):
        part = torch.full((hi - lo + 1, 4), float("nan"), device=DEV)
        m.forward(x[lo:hi], hi - lo, part)
        assert torch.equal(part[:-1], whole[lo:hi])
        assert part[-1].isnan().all()      # nothing is written past the last row
    assert whole[-1].isnan().all() and whole[:-1].isfinite().all()


@pytest.mark.parametrize("n_in,hidden,layers", [(128, 256, 3), (64, 64, 1), (256, 128, 4), (64, 128, 2)])
@pytest.mark.parametrize("rows", [1, 15, 17, 32, 33, 257, 8192, 8193, 8300])
def test_gradients_on_both_sides_of_the_tile_size(n_in, hidden, layers, rows):
    m, sizes, theta = net(n_in, hidden, layers, 8300, seed=3)
    x, T, w, nact = rows_of(rows + 50, n_in, 2)
    idx = torch.randperm(rows + 50, device=DEV)[:rows].to(torch.int32)
    loss = m.backward(x, T, w, nact, rows, idx=idx, n_data=rows + 50)
    g = m.get(cfr.CFR_MLP_GRADS)
    i = idx.long().cpu().numpy()
    a = [t.float().cpu().numpy().astype(np.float64)[i] for t in (x, T, w, nact)]
    L, ref = om.loss_and_grad(theta, sizes, a[0], a[1], a[2], a[3].astype(int), quant=True)
    # the bar of BF16 kernels against FP64, 1e-3 in the norm: FP32 accumulation order, rare bfloat16 rounding
    # flips and, in deep nets, units whose pre-activation changes sign with one.  A logit's gradient is
    # a difference of FP32 terms of order one, so a gradient that vanishes (a single row with a single
    # legal action) comes out as a few of their units in the last place: 1e-6 absolute
    assert loss == pytest.approx(L, rel=1e-5, abs=1e-6)
    assert np.linalg.norm(g - ref) <= 1e-3 * max(np.linalg.norm(ref), 1e-3)
    # the same minibatch gathered beforehand, from rows that begin off a 16-byte line, gives the same bits
    store = torch.zeros(rows * n_in + 1, dtype=torch.bfloat16, device=DEV)
    store[1:] = x[idx.long()].flatten()
    perm = torch.arange(rows, device=DEV, dtype=torch.int32)
    j = idx.long()
    again = m.backward(store[1:], T[j].contiguous(), w[j].contiguous(), nact[j].contiguous(), rows, idx=perm, n_data=rows)
    assert again == loss and np.array_equal(m.get(cfr.CFR_MLP_GRADS), g)


@pytest.mark.parametrize("rows", [100, 4096, 8300])
def test_train_step_equals_backward_and_adam(rows):
    a, _, _ = net(128, 256, 3, 8300, seed=5)
    b, _, _ = net(128, 256, 3, 8300, seed=5)
    x, T, w, nact = rows_of(rows, 128, 4)
    for _ in range(3):
        la = a.train_step(x, T, w, nact, rows, 1e-3, want_loss=True)
        lb = b.backward(x, T, w, nact, rows)
        b.adam(1e-3)
        assert la == lb
    for which in (cfr.CFR_MLP_PARAMS, cfr.CFR_MLP_GRADS, cfr.CFR_MLP_ADAM_M, cfr.CFR_MLP_ADAM_V):
        assert np.array_equal(a.get(which), b.get(which))
    # and both have refreshed the weights that inference reads
    za, zb = torch.empty(rows, 4, device=DEV), torch.empty(rows, 4, device=DEV)
    a.forward(x, rows, za)
    b.set_params(a.get())
    b.forward(x, rows, zb)
    assert torch.equal(za, zb)
