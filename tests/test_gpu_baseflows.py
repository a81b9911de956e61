"""Base flows over thin tiles (few line x box tiles: a block's waves share staged
operands), against the vector kernel, at bus counts around its 32-bus stages, box
counts ragged against its 16-box tiles and line counts that leave partial tiles.
Both sum float64 products in another order; where that flips the rounding of a
line's flow to float32 the sweep's terms move by 2^-24 of it, a small part of a
bound: 1e-8 of the largest."""
import numpy as np
import pytest

from paper_2511_15624_amd import ibp, synth
from tests.test_gpu_forward import gpu_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_bus,n_line,nb", [(14, 20, 4), (95, 140, 16), (97, 145, 17), (129, 194, 15), (500, 733, 37),
                                             (640, 961, 48)])
def test_thin_base_flows(monkeypatch, n_bus, n_line, nb):
    net = synth.make_network(n_bus, n_line, max(2, n_bus // 5), n_bus // 2, 23)
    n = ibp.Network(net, device=0)
    monkeypatch.setenv("IBP_TILE", "k2b=0")
    d = ibp.Network(net, device=0)
    monkeypatch.delenv("IBP_TILE")
    lo, hi = synth.sub_boxes(net, nb, seed=nb)
    print(f"[base flows] {n_bus} buses, {n.n_line} lines, {nb} boxes", flush=True)
    scr = ibp.IBP_F_SCREEN_UPPER  # (keeps small networks on the box-tiled kernels)
    for x, y in zip(gpu_bounds(n, lo, hi, flags=scr), gpu_bounds(d, lo, hi, flags=scr)):
        assert np.abs(x - y).max() <= 1e-8 * np.abs(y).max()
    n.close()
    d.close()
