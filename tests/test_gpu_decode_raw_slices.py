"""The latency kernel for raw weights (up to 8 rows per checkpoint) against the fp64 oracle at the edges of its slices of k: one slice that is not full, two unequal
ones, a last one of a few values, as many as a long row makes; groups of columns at every width; passes of more tokens than a pass holds."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,dtype,T,d,b", [
    (2, "f16", 1, 256, 128), (3, "bf16", 2, 512, 64), (2, "f32", 4, 520, 128), (5, "bf16", 3, 640, 256), (2, "f16", 8, 1160, 128), (3, "f32", 7, 1028, 64),
    (1, "bf16", 5, 8192, 128), (8, "f16", 4, 4096, 256), (31, "bf16", 1, 768, 128), (2, "bf16", 6, 1544, 64)])
def test_slices(C, dtype, T, d, b):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"raw_slices_{dtype}_C{C}_T{T}_d{d}_b{b}", 101, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    assert tr.call_route(tr.DTYPE_CODES[dtype], C, T, d, b, raw_weights=True)["kernel"] == 0
    rt, hb = w.routers(), w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    dev = to_device(hb, dtype)
    call = lambda: tr.select_exit(dev, g, w.eps, W1, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers)
    ex, z, m = call()
    again = call()
    torch.cuda.synchronize()
    assert torch.equal(ex, again[0]) and torch.equal(z, again[1]) and torch.equal(m, again[2])
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    # fp32 weights, products and sums: independent roundings of d products and sums, relative to a logit of about unit size (slopes of SiLU up to 1.1)
    assert np.abs(z.cpu().numpy() - z_o).max() <= 4 * d ** 0.5 * 2.0 ** -24 * max(1.0, np.abs(z_o).max())
    report(compare_select(w.name, dtype, z.cpu().numpy(), ex.cpu().numpy(), m.cpu().numpy(), z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))


@pytest.mark.parametrize("T", [9, 23])
def test_several_passes_when_forced(T):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"raw_passes_T{T}", 103, "bf16", 1408, 8, 4, T, None)
    rt, hb = w.routers(), w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    try:
        tr.set_variant(tr.VARIANT_DECODE)
        ex, z, m = tr.select_exit(to_device(hb, "bf16"), g, w.eps, W1, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers)
        torch.cuda.synchronize()
    finally:
        tr.set_variant(tr.VARIANT_AUTO)
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    report(compare_select(w.name, "bf16", z.cpu().numpy(), ex.cpu().numpy(), m.cpu().numpy(), z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
