"""Gradients of few boxes: the outage sweep and the transposed PTDF product split
over the waves of a block, against the kernels of one-box calls, at outage counts around
their steps and parts (4 and 32 outages, 32 lines) and ragged box counts.

Both round float32 sums of at most a few hundred terms in another order, so the
tolerance is the 2e-5 relative L2 per box of the other gradient comparisons."""
import pytest

from paper_2511_15624_amd import ibp, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_bus,n_line,nb", [(14, 20, 4), (24, 35, 5), (150, 225, 33), (350, 545, 7), (660, 1031, 34)])
def test_split_gradients(n_bus, n_line, nb):
    import torch
    net = synth.make_network(n_bus, n_line, max(2, n_bus // 5), n_bus // 2, 29)
    n = ibp.Network(net, device=0)
    blo, bhi = synth.sub_boxes(net, nb, seed=nb)
    lo, hi = torch.from_numpy(blo).cuda(), torch.from_numpy(bhi).cuda()
    a = torch.linspace(0.5, 1.5, nb, dtype=torch.float64, device="cuda")
    print(f"[gradients] {n_bus} buses, {n.n_line} lines, {n.n_ctg} outages, {nb} boxes", flush=True)
    for g_lo, g_hi, flags in ((a, a.flip(0), 0), (a, None, ibp.IBP_F_LOWER_ONLY), (-a, a, 0)):
        x = torch.cat(ibp.ibp_bound_backward(n, lo, hi, g_lo, g_hi, flags=flags), 1)
        y = torch.cat([torch.cat(ibp.ibp_bound_backward(n, lo[i:i + 1], hi[i:i + 1], g_lo[i:i + 1],
                                                        None if g_hi is None else g_hi[i:i + 1], flags=flags), 1)
                       for i in range(nb)])
        assert float(((x - y).norm(dim=1) / y.norm(dim=1)).max()) <= 2e-5
    n.close()
