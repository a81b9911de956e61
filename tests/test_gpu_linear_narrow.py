"""The linear outage sweep on narrow boxes, whose totals it moves by an estimate of what
the dense sweep's float32 radii lose: within the error budget whatever the width, and the
same bounds whatever the unit of the flows."""
import numpy as np
import pytest

import oracle
from paper_2511_15624_amd import ibp, synth
from tests.error_budget import budget
from tests.test_gpu_linear_outages import runs_linear

pytestmark = pytest.mark.gpu


def _narrow(net, nb, half):
    """Boxes of this half-width (per unit of a device's range) about seeded points."""
    lo, hi = synth.sub_boxes(net, nb, seed=11)
    mid = 0.5 * (lo.astype(np.float64) + hi)
    w = half * (hi.astype(np.float64) - lo)
    return (mid - w).astype(np.float32), (mid + w).astype(np.float32)


@pytest.mark.parametrize("half", [0.0, 1e-6, 1e-4, 4e-3])
def test_narrow_boxes_within_the_budget_in_any_unit(monkeypatch, half):
    import torch
    net = synth.make_network(333, 500, 66, 170, 7)
    fac = oracle.factors(net)
    lo, hi = _narrow(net, 128, half)
    # the same network in a unit 1024 times smaller: every flow and bound is exactly
    # 1024 times as large
    big = dict(net)
    for key in ("fmax_base", "fmax_ctg", "gen_pmin", "gen_pmax", "load_dmin", "load_dmax"):
        big[key] = 1024.0 * np.asarray(net[key])
    out = []
    for m, scale in ((net, 1.0), (big, 1024.0)):
        monkeypatch.setenv("IBP_TILE", "k3l=1")
        n = ibp.Network(m, device=0)
        monkeypatch.delenv("IBP_TILE")
        print(f"[narrow] half-width {half}, unit 1/{scale:.0f}", flush=True)
        tlo, thi = (torch.from_numpy(np.float32(scale) * x).cuda() for x in (lo, hi))
        (f_lo, f_hi), linear = runs_linear(n, lambda: ibp.ibp_bound_boxes(n, tlo, thi))
        assert linear
        out.append((f_lo.cpu().numpy() / scale, f_hi.cpu().numpy() / scale))
        phi_err = n.info.phi_abs_err
        n.close()
    for b in (0, 64, 127):
        bu = budget(net, fac, lo[b], hi[b], phi_err)
        assert 0.0 <= bu["r"]["f_lo"] - out[0][0][b] <= bu["lo"], (b, bu["r"]["f_lo"] - out[0][0][b], bu["lo"])
        assert 0.0 <= out[0][1][b] - bu["r"]["f_hi"] <= bu["hi"], (b, out[0][1][b] - bu["r"]["f_hi"], bu["hi"])
    for x, y in zip(*out):
        assert np.max(np.abs(x - y) / np.abs(x)) <= 1e-14
