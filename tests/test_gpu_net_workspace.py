"""The network on a stream of its own.  Its workspace is cleared on the null
stream when it is made; the first call on another stream must not overtake that
(the padding of its buffers is read as zeros, and its first activations would be
cleared).  Parameters and gradients are read and set in order with its calls."""
import numpy as np
import pytest
import torch

import paper_1504_02264_amd as les

pytestmark = pytest.mark.gpu


def test_first_call_waits_for_the_cleared_workspace():
    x = torch.randn((1, 16, 32, 32, 3), device="cuda")
    a = torch.randn((8192, 8192), device="cuda")
    side = torch.cuda.Stream()
    net, again = les.Net(seed=3), les.Net(seed=3)
    try:
        want = again.forward(x).cpu()
        torch.cuda.synchronize()
        for _ in range(8):
            b = a @ a            # some 50 ms on the null stream
        with torch.cuda.stream(side):
            got = net.forward(x)
            done = torch.cuda.default_stream().query()
        assert done              # the clearing, queued behind the products, has ended
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), want) and b.shape == a.shape
    finally:
        net.close()
        again.close()


def test_parameters_and_gradients_in_order_with_a_side_stream():
    x = torch.randn((2, 16, 32, 32, 3), device="cuda")
    t = torch.randn((2, 16, 32, 32), device="cuda")
    a = torch.randn((8192, 8192), device="cuda")
    side = torch.cuda.Stream()
    net, ref = les.Net(seed=3), les.Net(seed=3)
    try:
        want = ref.gradients(x, t)
        torch.cuda.synchronize()
        ref.train_step(x, t)
        start = net.get_params()
        net.forward(x)               # (the workspace is there)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(8):
                b = a @ a            # some 50 ms ahead of each call
            got = net.gradients(x, t)
            assert np.array_equal(got, want)
            b = a @ a
            net.train_step(x, t, want_loss=False)
            stepped = net.get_params()
            torch.cuda.synchronize()
            assert np.array_equal(stepped, ref.get_params())
            for _ in range(8):
                b = a @ a
            y = net.forward(x)       # with the trained weights, set only afterwards to the first ones
            net.set_params(start)
            z = net.forward(x)
            torch.cuda.synchronize()
        net.set_params(stepped)
        assert torch.equal(y, net.forward(x)) and not torch.equal(y, z)
        assert b.shape == a.shape
    finally:
        net.close()
        ref.close()
