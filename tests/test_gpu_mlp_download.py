"""Parameter downloads: whole and partial pinned pieces, destinations at any
offset, pinned destinations."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# 4 MB pieces: just under one, one and a few values, several and an odd rest
@pytest.mark.parametrize("widths", [(511, 2047), (513, 2048), (64, 512, 5021)])
@pytest.mark.parametrize("offset", [0, 1, 1023])
def test_params_round_trip(widths, offset):
    import torch
    import paper_2606_12850_amd as P
    from paper_2606_12850_amd.surrogate import MLP
    net = MLP(list(widths), 4)
    theta = np.random.default_rng(0).standard_normal(net.nparam).astype(np.float32)
    net.set_params(theta)
    for buf in (np.full(net.nparam + offset + 7, np.nan, np.float32),
                torch.full((net.nparam + offset + 7,), float("nan"), dtype=torch.float32, pin_memory=True).numpy()):
        P.semx_mlp_get_params(net.net, buf[offset:offset + net.nparam])
        assert np.array_equal(buf[offset:offset + net.nparam], theta)
        assert np.isnan(buf[:offset]).all() and np.isnan(buf[offset + net.nparam:]).all()
    net.close()
