"""GPU parity of the fp32 band and wide-tile kernels against the fp64 oracle where their one-step read-ahead begins and ends: rows of the fewest stages,
odd and even numbers of them, rows that end within a stage, several tiles in a row, blocks without a consumer wave's rows."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu
BAND_F32, WIDE_F32 = 11, 3

# two waves per block (shares of up to four blocks) and one (up to six); rows that are no whole k-tiles always take the band
BAND = [(10, 3001, 512), (32, 600, 544), (32, 290, 40), (16, 1600, 136), (8, 2400, 520), (8, 6100, 512), (16, 2700, 1064), (1, 20000, 640)]
WIDE = [(1, 257, 128), (3, 1000, 128), (2, 700, 256), (1, 70000, 128), (5, 4000, 384)]


@pytest.mark.parametrize("kernel,C,T,d", [(BAND_F32, *s) for s in BAND] + [(WIDE_F32, *s) for s in WIDE])
def test_read_ahead(kernel, C, T, d):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    form = 4 if kernel == WIDE_F32 else 0
    assert tr.prefill_plan(tr.F32, C, T, d, form=form)[0]["kernel"] == kernel
    w = synth.Workload(f"steps_C{C}_T{T}_d{d}", 113, "f32", d, 4 * C, 4, T, None)
    print(f"[gpu-case] {w.name}", flush=True)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, C) if C > 1 else 0.05
    hb = w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    pk = tr.router_pack(tr.F32, g, W1)
    tr.set_prefill_form(form)
    try:
        out = [tr.select_exit_packed(to_device(hb, "f32"), pk, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, d=d) for _ in range(2)]
        torch.cuda.synchronize()
    finally:
        tr.set_prefill_form(0)
    assert all(torch.equal(x, y) for x, y in zip(*out)), "two calls differ"
    ex, z, m = (o.cpu().numpy() for o in out[0])
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    report(compare_select(w.name, "f32", z, ex, m, z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
