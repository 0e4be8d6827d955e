"""GPU test of a network's first call: cfr_mlp_create returns once the network is ready on every stream."""
import numpy as np
import pytest
import torch

import gamegen as gg
import paper_2609_11923_amd as cfr
from oracle import mlp as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 8192, 8320])
def test_a_new_network_is_ready_on_any_stream(rows):
    old = cfr.Mlp()     # leaves memory that is not zero for the next network
    old.set_params(gg.mlp_init(om.layer_sizes(128, 256, 3, om.OUT), 1))
    x = torch.randn(rows, 128, device="cuda").to(torch.bfloat16)
    z = torch.full((rows, 4), float("nan"), device="cuda")
    side = torch.cuda.Stream()
    old.forward(x, rows, z)
    torch.cuda.synchronize()
    old.close()
    torch.cuda._sleep(1_000_000)     # the null stream is busy when the network is set up
    new = cfr.Mlp()
    new.forward(x, rows, z, stream=side)
    side.synchronize()
    assert np.array_equal(z.cpu().numpy(), np.zeros((rows, 4), np.float32))     # parameters are zero until they are set
