"""Parameters and gradients of one network read by two host threads at once."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_concurrent_downloads():
    import torch
    import paper_2606_12850_amd as P
    from paper_2606_12850_amd.surrogate import MLP
    net = MLP([64, 512, 9000], 8, seed=1)
    x, g = torch.randn((8, 64), device="cuda"), torch.randn((8, 9000), device="cuda")
    net.forward(x)
    P.semx_mlp_backward(net.net, g, 8)
    want = net.params(), np.empty(net.nparam, np.float32)
    P.semx_mlp_get_grads(net.net, want[1])
    assert not np.array_equal(*want)
    wrong = [0, 0]

    def read(k, call):
        out = np.empty(net.nparam, np.float32)
        for _ in range(30):
            out.fill(np.nan)
            call(net.net, out)
            wrong[k] += not np.array_equal(out, want[k])

    threads = [threading.Thread(target=read, args=a) for a in ((0, P.semx_mlp_get_params), (1, P.semx_mlp_get_grads))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    net.close()
    assert wrong == [0, 0]
