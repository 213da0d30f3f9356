"""Products with one operand in aligned rows and one not (widths that are multiples
of 4 but not of 8, and mixtures), against the network in FP64; the
allocation-free forward agrees to the bit.
"""
import numpy as np
import pytest
import torch

from tests.test_gpu_mlp_gemm import test_products as check_products

pytestmark = pytest.mark.gpu

SHAPES = [((12, 20, 24, 8), 5), ((36, 516, 204, 1030), 67), ((28, 512, 4433), 130), ((64, 68, 4444), 65),
          ((27, 128, 132, 1100), 33)]


@pytest.mark.parametrize("widths,batch", SHAPES)
def test_mixed_alignment(widths, batch):
    check_products(widths, batch)


@pytest.mark.parametrize("widths,batch", SHAPES)
def test_forward_noalloc_equal(widths, batch):
    from paper_2606_12850_amd import semx_mlp_forward_noalloc
    from paper_2606_12850_amd.surrogate import MLP
    net = MLP(list(widths), batch, seed=5)
    x = torch.from_numpy(np.random.default_rng(1).standard_normal((batch, widths[0]), dtype=np.float32)).cuda()
    y = net.forward(x)
    z = torch.empty_like(y)
    semx_mlp_forward_noalloc(net.net, x, batch, z)
    torch.cuda.synchronize()
    assert torch.equal(y, z)
    net.close()
