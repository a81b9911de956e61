"""Networks that study no outage (n_ctg = 0): the gradient has no outage part, whatever the
workspace held before."""
import numpy as np
import pytest

import oracle
from paper_2511_15624_amd import ibp, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [1, 5, 130])
def test_gradient_without_outages(nb):
    import torch
    net = dict(synth.make_network(40, 64, 8, 20, 3))
    net["ctg_line"] = np.zeros(0, np.int32)
    net["fmax_base"] = 0.1 * net["fmax_base"]  # overloaded lines, so that the penalties take part
    fac = oracle.factors(net)
    n = ibp.Network(net, device=0)
    lo, hi = synth.sub_boxes(net, nb, seed=4)
    tlo, thi = torch.from_numpy(lo).cuda(), torch.from_numpy(hi).cuda()
    g = torch.ones(nb, dtype=torch.float64, device="cuda")
    out = []
    for fill in (0, 255):  # 255: NaN wherever a partial is read that nothing wrote
        ws = ibp.Workspace(n)
        ws.buf = torch.full((n.workspace_bytes(nb, ibp.IBP_F_BACKWARD),), fill, dtype=torch.uint8, device="cuda")
        out.append(torch.cat(ibp.ibp_bound_backward(n, tlo, thi, 0.5 * g, g, ws=ws), 1).cpu().numpy())
    assert np.array_equal(*out)
    for b in (0, nb - 1):
        want = np.concatenate(oracle.grad(net, lo[b], hi[b], 0.5, 1.0, fac)[:2])
        assert np.linalg.norm(out[0][b] - want) <= 1e-4 * np.linalg.norm(want)  # the other gradient tests' bound
    n.close()
