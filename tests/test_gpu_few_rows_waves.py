"""The few-rows kernel on eight and on sixteen waves against the fp64 oracle: rows of exactly one turn of eight waves and just above,
exactly one turn of sixteen and just above, waves without any share of a row, a workgroup on every CU and more than that."""
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,dtype,T,d,b", [
    (2, "bf16", 5, 2048, 128), (2, "bf16", 5, 2056, 128), (3, "f16", 1, 4096, 64), (2, "f16", 16, 4104, 128), (1, "bf16", 7, 8192, 256),
    (2, "f32", 16, 1024, 128), (2, "f32", 3, 1152, 128), (2, "f32", 9, 2048, 256), (2, "f32", 17, 2056, 128), (4, "f32", 32, 1032, 128),
    (8, "bf16", 64, 2560, 128), (8, "f16", 64, 2304, 128), (20, "bf16", 20, 2056, 128)])
def test_waves(C, dtype, T, d, b):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"few_waves_{dtype}_C{C}_T{T}_d{d}_b{b}", 89, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    assert tr.call_route(tr.DTYPE_CODES[dtype], C, T, d, b)["kernel"] == 12
    rt = w.routers()
    hb = w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    ex, z, m = tr.select_exit_packed(to_device(hb, dtype), tr.router_pack(tr.DTYPE_CODES[dtype], g, W1), w.eps, b1, w2, rt.b2, rt.theta,
                                     w.layer_ids, 0, w.n_layers, d=d)
    torch.cuda.synchronize()
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    report(compare_select(w.name, dtype, z.cpu().numpy(), ex.cpu().numpy(), m.cpu().numpy(), z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
