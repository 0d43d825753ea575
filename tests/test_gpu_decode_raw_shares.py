"""The latency kernel for raw weights, its last workgroup's shares of the slices: the largest there are (32 slices: shares of 4, 8, 16 and 32) and on both sides of each
batch of loads, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [16384, 8320, 8192, 4224, 4096, 2176])           # 32, 17, 16, 9, 8 and 5 slices
@pytest.mark.parametrize("T,b", [(1, 128), (2, 64), (2, 256), (4, 128), (3, 256), (8, 128)])
def test_shares(T, b, d):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"raw_shares_T{T}_d{d}_b{b}", 109, "f16", d, 8, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    assert tr.call_route(tr.F16, w.C, T, d, b, raw_weights=True)["kernel"] == tr.ROUTE_LATENCY
    assert tr.workspace_bytes(tr.F16, w.C, T, d, b, raw_weights=True) >= w.C * -(-d // 512) * T * (128 * -(-b // 128) + 4) * 4
    rt, hb = w.routers(), w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    ex, z, m = tr.select_exit(to_device(hb, "f16"), g, w.eps, W1, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers)
    torch.cuda.synchronize()
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    # fp32 weights, products and sums: independent roundings of d products and sums, relative to a logit of about unit size (slopes of SiLU up to 1.1)
    assert np.abs(z.cpu().numpy() - z_o).max() <= 4 * d ** 0.5 * 2.0 ** -24 * max(1.0, np.abs(z_o).max())
    report(compare_select(w.name, "f16", z.cpu().numpy(), ex.cpu().numpy(), m.cpu().numpy(), z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
