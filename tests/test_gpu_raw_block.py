"""The latency kernel on raw weights in a block of exactly the bytes its call asks for: served, right, and nothing written behind the block."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,dtype,T,d,b", [(2, "f16", 1, 128, 64), (3, "bf16", 8, 640, 128), (8, "f16", 4, 4096, 128), (2, "f32", 8, 1028, 64), (5, "bf16", 7, 1408, 256),
                                           (4, "f16", 32, 1000, 128)])
def test_exact_block(C, dtype, T, d, b):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"raw_block_{dtype}_C{C}_T{T}_d{d}_b{b}", 107, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    code = tr.DTYPE_CODES[dtype]
    need = tr.workspace_bytes(code, C, T, d, b, raw_weights=True)
    assert tr.call_route(code, C, T, d, b, raw_weights=True, block_bytes=need)["kernel"] == tr.ROUTE_LATENCY
    rt, hb = w.routers(), w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    whole = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    block = whole[:need]
    tr.workspace_init(block)
    ex, z, m = tr.select_exit_ws(to_device(hb, dtype), g, w.eps, W1, None, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, block, d=d)
    torch.cuda.synchronize()
    tr.workspace_forget(block)
    assert bool((whole[need:] == 0xA5).all())
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    assert np.isfinite(z.cpu().numpy()).all()
    report(compare_select(w.name, dtype, z.cpu().numpy(), ex.cpu().numpy(), m.cpu().numpy(), z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
