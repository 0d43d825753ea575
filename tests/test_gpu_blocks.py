"""GPU: one caller-owned block, sized for the largest of a program's calls, through calls of other row counts: every one is served and right."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,C,d,rows", [("bf16", 8, 768, (4096, 1000, 64, 1, 4096)), ("bf16", 8, 768, (1, 64, 1000, 4096, 1)),
                                            ("bf16", 1, 2048, (8000, 3000, 500, 8000)), ("f32", 6, 1024, (9000, 600, 20)), ("f16", 8, 4096, (4096, 96, 17))])
def test_row_counts_through_a_block_for_the_largest(dtype, C, d, rows):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"block_{dtype}_C{C}_d{d}", 131, dtype, d, 4 * C, 4, max(rows), None)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, C) if C > 1 else 0.05
    hb = w.hidden()
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    g, W1, b1, w2 = routers_to_device(rt)
    pk = tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    h = to_device(hb, dtype)
    ws = torch.empty(tr.workspace_bytes(tr.DTYPE_CODES[dtype], C, max(rows), d), dtype=torch.uint8, device="cuda")
    tr.workspace_init(ws)
    for T in rows:
        print(f"[gpu-case] {w.name} T={T} in {ws.numel()} bytes", flush=True)
        ex, z, m = tr.select_exit_ws(h[:, :T], None, w.eps, None, pk, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, ws, d=d)
        torch.cuda.synchronize()
        report(compare_select(f"{w.name}_T{T}", dtype, z.cpu().numpy(), ex.cpu().numpy(), m.cpu().numpy(), z_o[:, :T], ex_o[:T], m_o[:T], rt.theta,
                              w.layer_ids, 0, w.n_layers))
    tr.workspace_forget(ws)
