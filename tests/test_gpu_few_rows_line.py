"""The few-rows kernel on both sides of the line between eight and sixteen waves (rows of 16 KiB, fp32 of 12 KiB, or more than 80 KiB of rows per workgroup), with idle waves at the end
of a row, against the fp64 oracle; twice each: a wait that is missing shows as results that differ."""
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,dtype,T,d,b", [
    (3, "f16", 10, 4096, 128), (3, "f16", 11, 4096, 128), (2, "bf16", 12, 3080, 64), (2, "bf16", 13, 3080, 64), (8, "f16", 16, 2600, 128), (4, "bf16", 16, 2560, 256),
    (1, "f32", 1, 4096, 128), (2, "f32", 1, 3072, 64), (2, "f32", 1, 2944, 64), (2, "f32", 6, 2944, 128), (2, "f32", 7, 2944, 128), (2, "bf16", 1, 8192, 128), (2, "bf16", 1, 8064, 128),
    (8, "bf16", 50, 2688, 128), (8, "bf16", 50, 2560, 128), (5, "f32", 16, 1288, 128), (5, "f32", 16, 1280, 128)])
def test_line(C, dtype, T, d, b):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"few_line_{dtype}_C{C}_T{T}_d{d}_b{b}", 127, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    assert tr.call_route(tr.DTYPE_CODES[dtype], C, T, d, b)["kernel"] == tr.ROUTE_FEW_ROWS
    rt, hb = w.routers(), w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    dev, pk = to_device(hb, dtype), tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    call = lambda: tr.select_exit_packed(dev, pk, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, d=d)
    ex, z, m = call()
    again = call()
    torch.cuda.synchronize()
    assert torch.equal(ex, again[0]) and torch.equal(z, again[1]) and torch.equal(m, again[2])
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    report(compare_select(w.name, dtype, z.cpu().numpy(), ex.cpu().numpy(), m.cpu().numpy(), z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
