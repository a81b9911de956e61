"""Screened calls of more than 4 x 65535 boxes (their tiles of four boxes exceed a
launch grid's 65535 rows), against the same call in two parts.

The parts take the same kernels over the same tiles, so the bounds agree to float64
rounding and the gradients (float32 sums per box, in one order) bit for bit."""
import pytest

from paper_2511_15624_amd import ibp, synth

pytestmark = pytest.mark.gpu

BOXES = 4 * 65535 + 8


@pytest.mark.parametrize("call", ["upper", "points", "gradient", "relaxation"])
def test_more_tiles_than_grid_rows(call):
    import torch
    net = synth.make_network(60, 96, 12, 30, 3)
    n = ibp.Network(net, device=0)
    lo, hi = synth.sub_boxes(net, 4096, seed=5)
    lo, hi = torch.from_numpy(lo).cuda().repeat(65, 1)[:BOXES], torch.from_numpy(hi).cuda().repeat(65, 1)[:BOXES]
    # every copy of the 4096 boxes is another part of the way to their lower ends
    f = torch.linspace(0.0, 0.9, BOXES, device="cuda")[:, None]
    hi = torch.maximum(lo, hi - f * (hi - lo)).contiguous()
    print(f"[many boxes] {call}, {BOXES} boxes, {n.n_line} lines, {n.n_ctg} outages", flush=True)
    g = torch.ones(BOXES, dtype=torch.float64, device="cuda")

    def run(a, b):
        x, y = lo[a:b], hi[a:b]
        if call == "upper":
            return ibp.ibp_bound_boxes(n, x, y, flags=ibp.IBP_F_UPPER_ONLY)[1:]
        if call == "points":
            return ibp.ibp_bound_boxes(n, x, x, flags=ibp.IBP_F_LOWER_ONLY | ibp.IBP_F_SCREEN_UPPER)[:1]
        if call == "gradient":
            return ibp.ibp_bound_backward(n, x, y, None, g[a:b], flags=ibp.IBP_F_UPPER_ONLY)
        return ibp.ibp_crown_bound_boxes(n, x, y)

    half = BOXES // 2 & ~63
    for whole, p, q in zip(run(0, BOXES), run(0, half), run(half, BOXES)):
        parts = torch.cat([p, q])
        if call == "gradient":
            assert torch.equal(whole, parts)
        else:
            assert float(((whole - parts).abs() / parts.abs().clamp_min(1.0)).max()) <= 1e-13
    n.close()
