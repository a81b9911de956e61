"""The chord sweep with the lanes over outages, against the sweep with the lanes over
lines (two boxes per lane), at box counts ragged against its two-box tiles, outage
counts that leave partial waves and line counts that leave partial quads of lines and
groups of 256.

Elements, slopes and float32 sums are the same and the slope totals are integers, so the
bounds differ by float64 roundings at most: 1e-12 relative."""
import pytest

from paper_2511_15624_amd import ibp, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_bus,n_line,n_ctg,nb", [(150, 229, None, 1031), (300, 470, None, 587), (700, 1091, 513, 231),
                                                   (1100, 1663, None, 87), (40, 61, 3, 4096)])
@pytest.mark.parametrize("wide", [False, True])
def test_chord_sweep_by_outages(monkeypatch, n_bus, n_line, n_ctg, nb, wide):
    import torch
    net = synth.make_network(n_bus, n_line, n_bus // 5, n_bus // 2, 37, n_ctg=n_ctg)
    n = ibp.Network(net, device=0)
    monkeypatch.setenv("IBP_TILE", "ckb=2")
    d = ibp.Network(net, device=0)
    monkeypatch.delenv("IBP_TILE")
    lo, hi = synth.sub_boxes(net, nb, seed=nb)
    if wide:  # every line near its limit in many outages
        lo, hi = lo.min(0, keepdims=True).repeat(nb, 0), hi.max(0, keepdims=True).repeat(nb, 0)
        hi[:, 0] = lo[:, 0]
    lo, hi = torch.from_numpy(lo).cuda(), torch.from_numpy(hi).cuda()
    print(f"[chord] {n_bus} buses, {n.n_line} lines, {n.n_ctg} outages, {nb} boxes", flush=True)
    a = ibp.ibp_crown_lower_boxes(n, lo, hi, crown=True)
    b = ibp.ibp_crown_lower_boxes(d, lo, hi, crown=True)
    for x, y in zip(a, b):
        if x is not None:
            assert float(((x - y).abs() / y.abs().clamp_min(1e-300)).max()) <= 1e-12
    n.close()
    d.close()
