"""GPU parity of the raw-weight latency kernel at the edges of its token counts (1, 2, 4 and 8 tokens per pass, several passes),
its slices (one, fewer than a finishing thread's batch, more than 32, every size of the last batch) and its widths, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,dtype,T,d,b", [
    (8, "f16", 1, 4096, 128), (8, "bf16", 2, 2048, 64), (5, "f32", 3, 4096, 128), (8, "f16", 4, 8192, 256), (32, "bf16", 5, 1024, 128),
    (3, "f32", 8, 16384, 64), (2, "bf16", 1, 16384, 256), (1, "f16", 9, 72, 128), (4, "f32", 32, 1004, 128), (7, "bf16", 17, 4104, 64),
    (2, "f32", 4, 12, 128), (6, "f16", 7, 128, 256),
    (16, "bf16", 5, 2344, 128), (4, "f16", 25, 4296, 64), (2, "f32", 6, 5320, 128), (3, "bf16", 8, 648, 128), (2, "f16", 5, 1024, 256)])
def test_raw_weights_few_rows(C, dtype, T, d, b):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"raw_{dtype}_C{C}_T{T}_d{d}_b{b}", 107, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, C) if C > 1 else 0.05
    hb = w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    dev = to_device(hb, dtype)
    tr.set_variant(tr.VARIANT_DECODE if T <= 32 else tr.VARIANT_AUTO)
    try:
        out = [tr.select_exit(dev, g, w.eps, W1, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers) for _ in range(3)]
        torch.cuda.synchronize()
    finally:
        tr.set_variant(tr.VARIANT_AUTO)
    for o in out[1:]:
        assert all(torch.equal(x, y) for x, y in zip(out[0], o)), "two calls differ"
    ex, z, m = (o.cpu().numpy() for o in out[0])
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    # fp32 weights, products and sums of up to 16384 terms of order 1/sqrt(d): 1e-5 covers their rounding, exact otherwise
    assert np.abs(z - z_o).max() < 1e-5
    report(compare_select(w.name, dtype, z, ex, m, z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers, tol=1e-5))
