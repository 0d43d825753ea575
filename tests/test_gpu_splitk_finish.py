"""GPU parity of the split-k pair's second launch at the edges of its row groups (8 or 16 rows per workgroup), against the fp64
oracle: row counts one below, at and one above a group's and a block's end, both group sizes, both widths of workgroup, and with the
slices of a tile on one XCD or (few tiles of 4 MiB and more of weights) dealt out over them."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,dtype,T,d,b,rows,slices", [
    (1, "bf16", 7, 512, 128, 32, 2), (2, "f16", 9, 512, 128, 32, 4), (1, "f32", 33, 512, 128, 64, 8), (3, "bf16", 41, 1408, 256, 64, 8),
    (1, "f16", 1025, 512, 64, 128, 4), (1, "bf16", 3079, 512, 128, 64, 2), (1, "f32", 4095, 256, 128, 32, 2), (2, "bf16", 1801, 512, 256, 32, 2),
    (1, "bf16", 455, 16384, 256, 32, 8), (1, "f32", 70, 8192, 128, 64, 4), (2, "f32", 33, 16384, 256, 32, 8)])
def test_row_groups_of_the_second_launch(C, dtype, T, d, b, rows, slices):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"finish_{dtype}_C{C}_T{T}_d{d}_b{b}", 101, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, C) if C > 1 else 0.05
    hb = w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    pk = tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    tr.set_prefill_form(tr.splitk_form(rows, slices))
    try:
        out = [tr.select_exit_packed(to_device(hb, dtype), pk, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, d=d) for _ in range(2)]
        torch.cuda.synchronize()
    finally:
        tr.set_prefill_form(0)
    assert all(torch.equal(x, y) for x, y in zip(*out)), "two calls differ"
    ex, z, m = (o.cpu().numpy() for o in out[0])
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    report(compare_select(w.name, dtype, z, ex, m, z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
