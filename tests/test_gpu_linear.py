"""The linear outage sweep of many boxes (integer matrix products of the outage
factors with the base flows' activity signs, plus the exceptions) against the
dense sweep (IBP_TILE=k3s=0) and the oracle, at sizes ragged against its groups
of 64 boxes, 32 lines, 32 and 64 outages.

Both paths bound the same real sums with the same padding: each must enclose the
oracle, within the box's error budget (the largest gap that the padding allows),
so the two differ by at most that budget.  Over all boxes, beyond the sampled
ones, 1e-5 of the terms' magnitude (a lost line or outage shows far above it)."""
import numpy as np
import pytest

import oracle
from paper_2511_15624_amd import ibp, synth
from tests.error_budget import budget
from tests.test_gpu_forward import gpu_bounds

pytestmark = pytest.mark.gpu

def _pair(net, monkeypatch):
    """(linear sweep wherever it fits, dense sweep) handles of one network."""
    monkeypatch.setenv("IBP_TILE", "k3l=1")
    n = ibp.Network(net, device=0)
    monkeypatch.setenv("IBP_TILE", "k3s=0")
    d = ibp.Network(net, device=0)
    monkeypatch.delenv("IBP_TILE")
    return n, d


def _agree(net, n, d, lo, hi, fac, sample, flags=0, skip=()):
    """Bounds of the linear sweep, checked against the dense sweep's and the oracle's."""
    g = gpu_bounds(n, lo, hi, terms=True, flags=flags)
    w = gpu_bounds(d, lo, hi, terms=True, flags=flags)
    sides = [s for s in (0, 1) if not flags & (ibp.IBP_F_UPPER_ONLY if s == 0 else ibp.IBP_F_LOWER_ONLY)]
    keep = np.array([b not in skip for b in range(lo.shape[0])])
    t = np.abs(w[2])
    for s in sides:
        scale = t[:, s] + net["zeta_inj"] * t[:, 3 - s] + net["zeta_f"] * (t[:, 5 - s] + t[:, 7 - s])
        assert np.all((np.abs(g[s] - w[s]) <= 1e-5 * scale)[keep]), float(np.max((np.abs(g[s] - w[s]) / scale)[keep]))
    for b in sample:
        bu = budget(net, fac, lo[b], hi[b], n.info.phi_abs_err)
        for s, key, sign in ((0, "lo", 1.0), (1, "hi", -1.0)):
            if s in sides:
                gap = sign * (bu["r"]["f_" + key] - g[s][b])
                assert 0.0 <= gap <= bu[key], (b, key, gap, bu[key])
                assert abs(g[s][b] - w[s][b]) <= bu[key], (b, key, g[s][b], w[s][b], bu[key])
    return g


@pytest.mark.parametrize("n_bus,n_line,seed,nb", [(40, 61, 5, 64), (150, 225, 6, 129), (333, 500, 7, 300),
                                                  (700, 1089, 8, 67)])
def test_linear_sweep_matches_the_dense_sweep(monkeypatch, n_bus, n_line, seed, nb):
    net = synth.make_network(n_bus, n_line, max(3, n_bus // 5), max(5, n_bus // 2), seed)
    fac = oracle.factors(net)
    n, d = _pair(net, monkeypatch)
    blo, bhi = synth.sub_boxes(net, nb, seed=seed)
    mid = (0.5 * (blo + bhi)).astype(np.float32)
    print(f"[linear] {n_bus} buses, {n.n_line} lines, {n.n_ctg} outages, {nb} boxes", flush=True)
    for lo, hi in ((blo, bhi), (mid, mid)):
        for flags in (0, ibp.IBP_F_LOWER_ONLY):
            _agree(net, n, d, lo, hi, fac, (0, nb // 2, nb - 1), flags)
    n.close()
    d.close()


@pytest.mark.parametrize("limit", [1e-6, 1e30, "kink"])
def test_linear_sweep_with_extreme_limits(monkeypatch, limit):
    """Every penalty active, none active, and every line's limit on the base
    flow of one box (all of that box's pairs are near a kink)."""
    net = dict(synth.make_network(150, 225, 30, 75, 6))
    blo, bhi = synth.sub_boxes(net, 70, seed=3)
    fac = oracle.factors(net)
    if limit == "kink":
        r = oracle.ibp(net, blo[9], bhi[9], fac, keep_intermediates=True)
        net["fmax_ctg"] = np.maximum(np.abs(r["c_f"]) + r["r_f"], 1e-3)
    else:
        net["fmax_ctg"] = np.full(len(net["fmax_ctg"]), limit)
    fac = oracle.factors(net)
    n, d = _pair(net, monkeypatch)
    print(f"[linear] limits {limit}", flush=True)
    _agree(net, n, d, blo, bhi, fac, (0, 9, 69))
    n.close()
    d.close()


def test_linear_sweep_keeps_an_invalid_box_to_itself(monkeypatch):
    net = synth.make_network(150, 225, 30, 75, 6)
    blo, bhi = synth.sub_boxes(net, 100, seed=4)
    blo[17, 3] = np.nan
    bhi[80, 5] = np.inf
    n, d = _pair(net, monkeypatch)
    f_lo, f_hi, _ = _agree(net, n, d, blo, bhi, oracle.factors(net), (16, 81), skip=(17, 80))
    assert np.all(np.isnan(f_lo[[17, 80]])) and np.all(np.isnan(f_hi[[17, 80]]))
    assert np.all(np.isfinite(np.delete(f_lo, [17, 80])))
    n.close()
    d.close()
