"""The screened sweeps of few boxes: the screen split over outage ranges and the
marked lines walked in segments (many waves share one tile), against the dense
sweeps, at box counts ragged against the 4-box tiles and networks whose line and
outage counts leave partial chunks.

Forward: the same elements in another summation order, 1e-6 relative (four
float32 additions per partial, as in the dense sweep's sums of eight); gradient:
2e-5 relative L2 per box, as for the unsplit sweep."""
import numpy as np
import pytest

from paper_2511_15624_amd import ibp, synth
from tests.test_gpu_forward import gpu_bounds, one_sided_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_bus,n_line,nb", [(300, 470, 4), (300, 470, 7), (700, 1089, 33), (1100, 1663, 66)])
def test_screened_sweeps_of_few_boxes(monkeypatch, n_bus, n_line, nb):
    import torch
    net = synth.make_network(n_bus, n_line, n_bus // 5, n_bus // 2, 17)
    n = ibp.Network(net, device=0)
    monkeypatch.setenv("IBP_TILE", "k3s=0,k5s=0")
    d = ibp.Network(net, device=0)
    monkeypatch.delenv("IBP_TILE")
    blo, bhi = synth.sub_boxes(net, nb, seed=nb)
    mid = (0.5 * (blo + bhi)).astype(np.float32)
    print(f"[segments] {n_bus} buses, {n.n_line} lines, {n.n_ctg} outages, {nb} boxes", flush=True)
    for lo, hi, flags, side in ((blo, bhi, ibp.IBP_F_UPPER_ONLY, 1), (mid, mid, ibp.IBP_F_LOWER_ONLY, 0),
                                (blo, bhi, 0, 0), (blo, bhi, 0, 1)):
        scr = 0 if flags == ibp.IBP_F_UPPER_ONLY else ibp.IBP_F_SCREEN_UPPER
        assert one_sided_close(gpu_bounds(n, lo, hi, flags=flags | scr)[side], gpu_bounds(d, lo, hi, flags=flags)[side])
    lo, hi = torch.from_numpy(blo).cuda(), torch.from_numpy(bhi).cuda()
    g = torch.linspace(0.5, 1.5, nb, dtype=torch.float64, device="cuda")
    x = torch.cat(ibp.ibp_bound_backward(n, lo, hi, None, g, flags=ibp.IBP_F_UPPER_ONLY), 1)
    y = torch.cat(ibp.ibp_bound_backward(d, lo, hi, None, g, flags=ibp.IBP_F_UPPER_ONLY), 1)
    assert float(((x - y).norm(dim=1) / y.norm(dim=1)).max()) <= 2e-5
    n.close()
    d.close()


def test_screened_relaxation_matches_the_dense_slopes(monkeypatch):
    """The upper relaxation over the screened lines takes the dense sweep's
    slopes; its per-outage float32 sums of eight are inside the ten roundings
    both paths' error bounds allow, so the bounds agree to 1e-6 of their size."""
    import torch
    net = synth.make_network(1100, 1663, 220, 550, 17)
    n = ibp.Network(net, device=0)
    monkeypatch.setenv("IBP_TILE", "k5s=0")
    d = ibp.Network(net, device=0)
    monkeypatch.delenv("IBP_TILE")
    blo, bhi = synth.sub_boxes(net, 230, seed=5)
    lo, hi = torch.from_numpy(blo).cuda(), torch.from_numpy(bhi).cuda()
    for flags in (0, ibp.IBP_F_UPPER_ONLY):
        a = ibp.ibp_crown_bound_boxes(n, lo, hi, crown=True, flags=flags)[2]
        b = ibp.ibp_crown_bound_boxes(d, lo, hi, crown=True, flags=flags)[2]
        assert float(((a - b).abs() / b.abs()).max()) <= 1e-6
    n.close()
    d.close()
