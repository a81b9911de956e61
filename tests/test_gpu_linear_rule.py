"""Which calls of many boxes take the linear outage sweep: both bounds from fewer
boxes on than the lower bound alone, whose dense sweep costs less, and neither
below the sizes where the dense sweep is faster.  And the device memory of handles
that cannot take it."""
import pytest

from paper_2511_15624_amd import ibp, synth
from tests.test_gpu_linear_outages import runs_linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_bus,n_line,nb,both,lower", [
    (1500, 2300, 1024, False, False), (1500, 2300, 1536, True, False),
    (2600, 4000, 256, False, False), (2600, 4000, 384, True, False), (2600, 4000, 512, True, True)])
def test_linear_sweep_by_size(n_bus, n_line, nb, both, lower):
    import torch
    net = synth.make_network(n_bus, n_line, n_bus // 5, n_bus // 2, 7)
    n = ibp.Network(net, device=0)
    lo, hi = (torch.from_numpy(x).cuda() for x in synth.sub_boxes(net, nb, seed=9))
    print(f"[rule] {n.n_line} lines, {n.n_ctg} outages, {nb} boxes", flush=True)
    assert runs_linear(n, lambda: ibp.ibp_bound_boxes(n, lo, hi))[1] is both
    assert runs_linear(n, lambda: ibp.ibp_bound_boxes(n, lo, hi, flags=ibp.IBP_F_LOWER_ONLY))[1] is lower
    n.close()


def test_no_digit_planes_where_the_sweep_is_off(monkeypatch):
    net = synth.make_network(1300, 2000, 260, 650, 7)
    held = {}
    for tile in ("", "k3l=0", "k3s=0"):
        monkeypatch.setenv("IBP_TILE", tile)
        n = ibp.Network(net, device=0)
        held[tile] = n.info.device_bytes
        elements = n.n_ctg * n.n_line
        n.close()
    assert elements > 2500000
    assert held["k3l=0"] == held["k3s=0"] <= held[""] - 10 * elements
