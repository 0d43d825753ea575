"""GPU parity of the split-k pair's first launch against the fp64 oracle at the edges of its ring of k-tiles: fewer k-tiles than it fills at
the start, a few more, as many as it holds and several times round it, every tile height and storage type, both halves of the last k-tile's
exchange, more workgroups than CUs (a shorter ring), rows that end within a k-tile; and the direct exit of a single checkpoint."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


def check(C, dtype, T, d, b, form, min_layer=0):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"ring_{dtype}_C{C}_T{T}_d{d}_b{b}_min{min_layer}", 103, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name} {form}", flush=True)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, C) if C > 1 else 0.05
    hb = w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    pk = tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    tr.set_prefill_form(form(tr) if form else 0)
    try:
        out = [tr.select_exit_packed(to_device(hb, dtype), pk, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, min_layer, w.n_layers, d=d) for _ in range(2)]
        torch.cuda.synchronize()
    finally:
        tr.set_prefill_form(0)
    assert all(torch.equal(x, y) for x, y in zip(*out)), "two calls differ"
    ex, z, m = (o.cpu().numpy() for o in out[0])
    ex_o, z_o, m_o = oracle_select(w, rt, hb, min_layer=min_layer)
    report(compare_select(w.name, dtype, z, ex, m, z_o, ex_o, m_o, rt.theta, w.layer_ids, min_layer, w.n_layers))


# k-tiles of a slice: d * bytes / 256 / slices
@pytest.mark.parametrize("C,dtype,T,d,b,rows,slices", [
    (2, "bf16", 45, 256, 128, 32, 2), (2, "f16", 70, 256, 128, 64, 2), (1, "bf16", 130, 256, 64, 128, 2),           # one
    (3, "f16", 65, 1408, 128, 64, 2), (2, "bf16", 33, 1664, 256, 32, 2), (1, "f32", 129, 1408, 128, 128, 4),        # 5 and 6, 6 and 7, 5 and 6
    (1, "bf16", 97, 4096, 128, 64, 4), (2, "f32", 64, 1024, 128, 32, 2),                                            # eight
    (1, "bf16", 40, 16384, 128, 32, 2), (1, "f16", 65, 8192, 128, 64, 2), (1, "bf16", 129, 8192, 128, 128, 2),      # 64, 32, 32
    (1, "f32", 65, 8192, 128, 64, 2), (1, "f32", 128, 4096, 256, 128, 2), (8, "bf16", 700, 2048, 128, 32, 8)])
def test_ring(C, dtype, T, d, b, rows, slices):
    check(C, dtype, T, d, b, lambda tr: tr.splitk_form(rows, slices))


@pytest.mark.parametrize("dtype,T,d,min_layer", [("bf16", 1500, 1608, 0), ("f16", 2100, 4096, 3), ("f16", 2100, 4096, 4), ("f32", 700, 2048, 0)])
def test_single_checkpoint(dtype, T, d, min_layer):
    check(1, dtype, T, d, 128, None, min_layer)
