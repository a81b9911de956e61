"""The linear outage sweep where a chosen set of outages is studied (``ctg_line``
given).

Loops of which one line alone is an outage: no other outage moves that line, and its own
outage has no element of it, so it is summed over one outage fewer than a bridge is.
Only such lines are overloaded, so one element too many or too few is far above the
box's error budget on either side.

More lines than the int32 sums of two digits hold: the dense sweep serves."""
import numpy as np
import pytest

import oracle
from paper_2511_15624_amd import ibp, synth
from tests.error_budget import budget

pytestmark = pytest.mark.gpu


def runs_linear(n, call):
    """Runs a call without the screen's flag; whether it took the linear sweep (whose
    line kernels are timed apart from its products)."""
    n.set_kernel_timing(True)
    out = call()
    times = n.kernel_times()
    n.set_kernel_timing(False)
    return out, "forward_line_screen" in times


def _pendant_loops(loop, count):
    """A 40-bus network of 60 lines with `count` loops of `loop` lines hung on one bus
    each, a load at each of the loops' own buses; the outages are the mesh's
    and the first line of every loop, whose limits are half its flow and, for the
    loops, in a quad of lines of their own."""
    net = dict(synth.make_network(40, 60, 8, 20, 5))
    mesh = np.flatnonzero(~synth.find_bridges(40, net["line_from"], net["line_to"]))
    fr, to, b = list(net["line_from"]), list(net["line_to"]), list(net["line_b"])
    first = []
    for i in range(count):
        n0 = net["n_bus"]
        new = list(range(n0, n0 + loop - 1))
        ring = [3 + 5 * i] + new
        first.append(len(fr))
        for j in range(loop):
            fr.append(ring[j])
            to.append(ring[(j + 1) % loop])
            b.append(20.0 + j)
        for j in range(4 - loop):  # the quad's other lines: more circuits of a mesh line
            fr.append(int(net["line_from"][mesh[i]]))
            to.append(int(net["line_to"][mesh[i]]))
            b.append(10.0)
        net["n_bus"] = n0 + loop - 1
        net["load_bus"] = np.concatenate([net["load_bus"], np.array(new, np.int32)])
        for key, v in (("load_value", 90.0), ("load_dmin", 0.5), ("load_dmax", 0.6 + 0.1 * i)):
            net[key] = np.concatenate([net[key], np.full(len(new), v)])
    net["line_from"], net["line_to"] = np.array(fr, np.int32), np.array(to, np.int32)
    net["line_b"] = np.array(b)
    net["ctg_line"] = np.sort(np.concatenate([mesh, first])).astype(np.int32)
    net["fmax_base"] = np.full(len(fr), 1e3)
    net["fmax_ctg"] = np.full(len(fr), 1e3)
    lo, hi = synth.full_box(net)
    c = np.abs(oracle.ibp(net, lo, hi, keep_intermediates=True)["c_f"])
    for key in ("fmax_base", "fmax_ctg"):
        net[key][first] = 0.5 * c[first]
    return net


@pytest.mark.parametrize("loop,count", [(3, 1), (3, 4), (2, 3)])
def test_a_line_counts_in_no_outage_of_its_own(monkeypatch, loop, count):
    import torch
    net = _pendant_loops(loop, count)
    fac = oracle.factors(net)
    monkeypatch.setenv("IBP_TILE", "k3l=1")
    n = ibp.Network(net, device=0)
    monkeypatch.delenv("IBP_TILE")
    print(f"[own outage] loops of {loop}, {count} of them, {n.n_line} lines, {n.n_ctg} outages", flush=True)
    lo, hi = synth.sub_boxes(net, 64, seed=7)
    tlo, thi = torch.from_numpy(lo).cuda(), torch.from_numpy(hi).cuda()
    (f_lo, f_hi), linear = runs_linear(n, lambda: ibp.ibp_bound_boxes(n, tlo, thi))
    assert linear
    _within_budget(net, fac, n, lo, hi, f_lo.cpu().numpy(), f_hi.cpu().numpy(), (0, 31, 63))
    n.close()


def _within_budget(net, fac, n, lo, hi, f_lo, f_hi, sample):
    for b in sample:
        bu = budget(net, fac, lo[b], hi[b], n.info.phi_abs_err)
        assert 0.0 <= bu["r"]["f_lo"] - f_lo[b] <= bu["lo"], (b, bu["r"]["f_lo"] - f_lo[b], bu["lo"])
        assert 0.0 <= f_hi[b] - bu["r"]["f_hi"] <= bu["hi"], (b, f_hi[b] - bu["r"]["f_hi"], bu["hi"])


def test_more_lines_than_the_digit_sums_hold(monkeypatch):
    """A chain of 520 stages of 130 equal circuits, all overloaded, and two weak lines
    across it, the outages: each moves its flow onto 67600 lines by about 1/130 = 32264 /
    2^22 apiece, whose two middle digits add up to 67600 * 32264 > 2^31."""
    import torch
    stages, m = 520, 130
    fr = np.concatenate([np.repeat(np.arange(stages), m), [0, 0]]).astype(np.int32)
    to = np.concatenate([np.repeat(np.arange(1, stages + 1), m), [stages, stages]]).astype(np.int32)
    L = fr.size
    net = dict(n_bus=stages + 1, slack_bus=0, line_from=fr, line_to=to,
               line_b=np.concatenate([np.full(L - 2, 20.0), [2e-3, 1e-3]]),
               gen_bus=np.array([0, 0], np.int32), gen_cost=np.array([20.0, 30.0]), gen_pmin=np.array([0.2, 0.0]),
               gen_pmax=np.array([2.0, 1.0]), load_bus=np.full(3, stages, np.int32),
               load_value=np.array([80.0, 90.0, 70.0]), load_dmin=np.array([0.4, 0.5, 0.6]),
               load_dmax=np.array([0.5, 0.6, 0.7]), zeta_inj=1e3, zeta_f=5e2,
               ctg_line=np.array([L - 2, L - 1], np.int32))
    net["fmax_base"] = np.full(L, 0.5 * 1.65 / m)
    net["fmax_ctg"] = net["fmax_base"]
    fac = oracle.factors(net)
    monkeypatch.setenv("IBP_TILE", "k3l=1")
    n = ibp.Network(net, device=0)
    monkeypatch.delenv("IBP_TILE")
    print(f"[digit sums] {n.n_line} lines, {n.n_ctg} outages", flush=True)
    lo, hi = synth.sub_boxes(net, 64, seed=3)
    tlo, thi = torch.from_numpy(lo).cuda(), torch.from_numpy(hi).cuda()
    (f_lo, f_hi), linear = runs_linear(n, lambda: ibp.ibp_bound_boxes(n, tlo, thi))
    _within_budget(net, fac, n, lo, hi, f_lo.cpu().numpy(), f_hi.cpu().numpy(), (0, 40))
    assert not linear
    n.close()
