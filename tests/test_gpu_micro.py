"""One-block calls of small networks over a wide block: PTDF rows staged in one and
several steps, line counts around a wave and around the staging quads, odd outage
counts, one and several outage items per thread, against the box-tiled kernels on
the same box four times.

The sums over buses have different orders there (a flip of a line's float32 rounding
moves its terms by 2^-24) and the outage sums other groupings of float32 terms:
1e-6 relative, as between the other forward kernels."""
import numpy as np
import pytest

from paper_2511_15624_amd import ibp, synth
from tests.test_gpu_forward import gpu_bounds, one_sided_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_bus,n_line,n_ctg", [(40, 63, None), (60, 129, 7), (129, 190, None), (170, 257, 131),
                                                (256, 400, 40), (250, 1020, 61)])
def test_wide_block(monkeypatch, n_bus, n_line, n_ctg):
    net = synth.make_network(n_bus, n_line, n_bus // 5, n_bus // 2, 31, n_ctg=n_ctg)
    monkeypatch.setenv("IBP_TILE", "mb=0")
    n = ibp.Network(net, device=0)
    monkeypatch.delenv("IBP_TILE")
    print(f"[wide block] {n_bus} buses, {n.n_line} lines, {n.n_ctg} outages", flush=True)
    for nb, seed in ((1, 3), (2, 4)):
        lo, hi = synth.sub_boxes(net, nb, seed=seed)
        one = gpu_bounds(n, lo, hi)
        four = gpu_bounds(n, np.tile(lo, (4, 1)), np.tile(hi, (4, 1)))
        for side in (0, 1):
            assert one_sided_close(one[side], four[side][:nb])
    n.close()


@pytest.mark.parametrize("n_bus,n_line,n_ctg,nb", [(14, 20, None, 4), (25, 38, None, 2047), (45, 70, 1, 5),
                                                   (60, 129, 7, 256), (133, 200, None, 64), (200, 301, None, 255),
                                                   (256, 400, 161, 17)])
def test_several_boxes_one_block_each(monkeypatch, n_bus, n_line, n_ctg, nb):
    """Against the box-tiled kernels: the same float32 elements and sums (buses in the same
    order, outages paired in the same rows), float64 sums in another order: 1e-13."""
    net = synth.make_network(n_bus, n_line, max(2, n_bus // 5), n_bus // 2, 41, n_ctg=n_ctg)
    n = ibp.Network(net, device=0)
    monkeypatch.setenv("IBP_TILE", "mb=0")
    d = ibp.Network(net, device=0)
    monkeypatch.delenv("IBP_TILE")
    lo, hi = synth.sub_boxes(net, nb, seed=nb)
    print(f"[blocks] {n_bus} buses, {n.n_line} lines, {n.n_ctg} outages, {nb} boxes", flush=True)
    for x, y in zip(gpu_bounds(n, lo, hi, terms=True), gpu_bounds(d, lo, hi, terms=True)):
        assert np.abs(x - y).max() <= 1e-13 * max(1.0, np.abs(y).max())
    n.close()
    d.close()
