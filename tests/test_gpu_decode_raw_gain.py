"""The latency kernel for raw weights and its gain: none at all, one that is aligned to a float only, and between values (NaN) that are not its own; gains on slices that
are not full and on several passes."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gain", ["none", 0, 1, 2, 3])
@pytest.mark.parametrize("C,dtype,T,d,b", [(2, "f16", 1, 4096, 128), (3, "bf16", 8, 640, 64), (2, "f32", 4, 1028, 128), (2, "f32", 8, 384, 256), (1, "bf16", 23, 1608, 128)])
def test_gain(C, dtype, T, d, b, gain):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"raw_gain_{gain}_{dtype}_C{C}_T{T}_d{d}_b{b}", 113, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    assert tr.call_route(tr.DTYPE_CODES[dtype], C, T, d, b, raw_weights=True)["kernel"] == tr.ROUTE_LATENCY
    rt, hb = w.routers(), w.hidden()
    if gain == "none":
        rt.gamma[:] = 1.0
    g, W1, b1, w2 = routers_to_device(rt)
    if gain == "none":
        g = None
    else:
        room = torch.full((C * d + 8,), float("nan"), device="cuda")
        room[gain + 1:gain + 1 + C * d] = g.flatten()
        g = room[gain + 1:gain + 1 + C * d].view(C, d)
    ex, z, m = tr.select_exit(to_device(hb, dtype), g, w.eps, W1, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers)
    torch.cuda.synchronize()
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    # fp32 weights, products and sums: independent roundings of d products and sums, relative to a logit of about unit size (slopes of SiLU up to 1.1)
    assert np.abs(z.cpu().numpy() - z_o).max() <= 4 * d ** 0.5 * 2.0 ** -24 * max(1.0, np.abs(z_o).max())
    report(compare_select(w.name, dtype, z.cpu().numpy(), ex.cpu().numpy(), m.cpu().numpy(), z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
