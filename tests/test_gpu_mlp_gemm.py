"""The network's matrix products at the edges of their tiles, against the same
network in FP64 on operands rounded to BF16.

Shapes: widths that are no multiple of 8 (element-wise operand loads), of 64 or
128 (partial tiles), products of 512 wide tiles and more, split sums, a batch
of one.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# FP32 sums against FP64 differ by about 1e-7, which moves a value across a BF16 rounding boundary (a step of 2^-8)
# with probability 1e-7 / 2^-9 = 5e-5: 2^-8 sqrt(5e-5) = 3e-5 of a layer's norm, twice per layer and direction
TOL = 3e-4

SHAPES = [((27, 33, 7), 1), ((64, 200, 4433), 17), ((8, 8, 16), 3), ((64, 72, 136), 65), ((27, 256, 256, 1102), 130),
          ((512, 129, 48), 64), ((40, 512, 24576), 100), ((64, 512, 512, 8320), 1100), ((64, 512, 8320), 1000),
          ((16, 1000, 64), 260)]


def _bf(x):
    return x.to(torch.float32).to(torch.bfloat16).to(torch.float64)


@pytest.mark.parametrize("widths,batch", SHAPES)
def test_products(widths, batch):
    from paper_2606_12850_amd import semx_mlp_backward, semx_mlp_get_grads
    from paper_2606_12850_amd.surrogate import MLP
    net = MLP(list(widths), batch, seed=3)
    theta = net.params()
    rng = np.random.default_rng(batch)
    at = 0
    layers = []
    for a, b in zip(widths[:-1], widths[1:]):
        theta[at + a * b:at + a * b + b] = rng.uniform(-0.2, 0.2, b)
        layers.append((torch.from_numpy(theta[at:at + a * b].reshape(b, a)).double(),
                       torch.from_numpy(theta[at + a * b:at + a * b + b]).double()))
        at += a * b + b
    net.set_params(theta)
    x = torch.from_numpy(rng.standard_normal((batch, widths[0]), dtype=np.float32))
    g = torch.from_numpy(rng.standard_normal((batch, widths[-1]), dtype=np.float32))
    y = net.forward(x.cuda()).cpu().double()
    xd, gd = x.cuda(), g.cuda()
    net.forward(xd)
    semx_mlp_backward(net.net, gd, batch)
    grads = np.empty(net.nparam, np.float32)
    semx_mlp_get_grads(net.net, grads)
    net.close()
    h, hs, zs = _bf(x), [], []
    for k, (w, b) in enumerate(layers):
        hs.append(h)
        z = h @ _bf(w).T + b
        zs.append(z)
        h = _bf(torch.nn.functional.silu(z))
    assert torch.linalg.norm(y - zs[-1]) <= TOL * torch.linalg.norm(zs[-1])
    d, want = g.double(), [None] * len(layers)
    for k in range(len(layers) - 1, -1, -1):
        want[k] = torch.cat([(_bf(d).T @ hs[k]).reshape(-1), d.sum(0)])
        if k:
            s = torch.sigmoid(zs[k - 1])
            d = (_bf(d) @ _bf(layers[k][0])) * s * (1.0 + zs[k - 1] * (1.0 - s))
    at = 0
    for k, w in enumerate(want):
        got = torch.from_numpy(grads[at:at + w.numel()]).double()
        at += w.numel()
        assert torch.linalg.norm(got - w) <= TOL * torch.linalg.norm(w), k
