"""The linear outage sweep, asserted to have run, where its parts other than the
products do the work: every penalty active (heavy quads), none, every line's limit on
the base flow of one box (pairs near a kink); more lines and outages than one segment
and one chunk of the pairs' kernel, at a box count ragged against its groups.

Against the oracle within the box's error budget, and against the dense sweep within
that budget: element roundings go with the limits, not with the totals, so the
budget is what the padding allows either of them."""
import numpy as np
import pytest

import oracle
from paper_2511_15624_amd import ibp, synth
from tests.error_budget import budget
from tests.test_gpu_forward import gpu_bounds
from tests.test_gpu_linear_outages import runs_linear

pytestmark = pytest.mark.gpu


def _compare(monkeypatch, net, fac, lo, hi, sample, flags):
    handles = []
    for tile in ("k3l=1", "k3l=0"):
        monkeypatch.setenv("IBP_TILE", tile)
        handles.append(ibp.Network(net, device=0))
        monkeypatch.delenv("IBP_TILE")
    n, d = handles
    sides = [s for s in (0, 1) if not (flags & ibp.IBP_F_LOWER_ONLY and s == 1)]
    g, linear = runs_linear(n, lambda: gpu_bounds(n, lo, hi, flags=flags))
    w, dense = runs_linear(d, lambda: gpu_bounds(d, lo, hi, flags=flags))
    assert linear and not dense
    for b in sample:
        bu = budget(net, fac, lo[b], hi[b], n.info.phi_abs_err)
        for s, key, sign in ((0, "lo", 1.0), (1, "hi", -1.0)):
            if s in sides:
                gap = sign * (bu["r"]["f_" + key] - g[s][b])
                assert 0.0 <= gap <= bu[key], (b, key, gap, bu[key])
                assert abs(g[s][b] - w[s][b]) <= bu[key], (b, key, g[s][b], w[s][b], bu[key])
    n.close()
    d.close()


@pytest.mark.parametrize("limit", [1e-6, 1e30, "kink"])
@pytest.mark.parametrize("nb", [64, 127])
def test_extreme_limits(monkeypatch, limit, nb):
    net = dict(synth.make_network(150, 225, 30, 75, 6))
    lo, hi = synth.sub_boxes(net, nb, seed=3)
    fac = oracle.factors(net)
    if limit == "kink":
        r = oracle.ibp(net, lo[9], hi[9], fac, keep_intermediates=True)
        net["fmax_ctg"] = np.maximum(np.abs(r["c_f"]) + r["r_f"], 1e-3)
    else:
        net["fmax_ctg"] = np.full(len(net["fmax_ctg"]), limit)
    fac = oracle.factors(net)
    print(f"[linear] limits {limit}, {nb} boxes", flush=True)
    for flags in (0, ibp.IBP_F_LOWER_ONLY):
        _compare(monkeypatch, net, fac, lo, hi, sorted({9, *range(0, nb, 8), nb - 1}), flags)


@pytest.mark.parametrize("kink", [False, True])
def test_more_than_a_segment_of_lines_and_outages(monkeypatch, kink):
    net = dict(synth.make_network(1500, 2300, 300, 750, 7))
    lo, hi = synth.sub_boxes(net, 129, seed=4)
    fac = oracle.factors(net)
    assert fac["L"] > 2048 and fac["K"] > 2048
    if kink:
        r = oracle.ibp(net, lo[128], hi[128], fac, keep_intermediates=True)
        net["fmax_ctg"] = np.maximum(np.abs(r["c_f"]) - r["r_f"], 1e-3)
    print(f"[linear] {fac['L']} lines, {fac['K']} outages, kink {kink}", flush=True)
    _compare(monkeypatch, net, fac, lo, hi, range(0, 129, 16), 0)
