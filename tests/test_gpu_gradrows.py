"""Gradients of many boxes of the smallest networks: which kernels they take."""
import pytest

from paper_2511_15624_amd import ibp, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, ibp.IBP_F_LOWER_ONLY])
def test_short_outage_rows_are_not_split(flags):
    """With few outages and lines the split forms lose from fewer tiles on: 6000 boxes at
    14 buses take the plain kernels as 12000 do, so their gradients are the same bits."""
    import torch
    net = synth.make_network(14, 20, 5, 11, 1)
    n = ibp.Network(net, device=0)
    lo, hi = (torch.from_numpy(x).cuda() for x in synth.sub_boxes(net, 12000, seed=2))
    g = torch.linspace(0.5, 1.5, 12000, dtype=torch.float64, device="cuda")
    a = ibp.ibp_bound_backward(n, lo, hi, g, g, flags=flags)
    b = ibp.ibp_bound_backward(n, lo[:6000], hi[:6000], g[:6000], g[:6000], flags=flags)
    for x, y in zip(a, b):
        assert torch.equal(x[:6000], y)
    n.close()
