"""The network's workspace is cleared on the null stream when it is made; the
first call on another stream must not overtake that (the padding of its buffers
is read as zeros, and its first activations would be cleared)."""
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
