"""The one-tile kernel against the fp64 oracle where its k loop can go wrong: tiles of 64 rows (two k-tiles per stage) on one, two, three and five k-tiles, on
rows that end inside a k-tile, with a last tile of a few rows; tiles of 128 rows in bursts (up to three quarters of the CUs) and without, odd and even counts of
stages, on both sides of that line.  Twice each: a wait that is missing shows as results that differ."""
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu

TILE = 4


@pytest.mark.parametrize("C,dtype,T,d,b,rows", [
    (22, "bf16", 380, 128, 128, 64), (22, "f16", 380, 256, 64, 64), (22, "bf16", 380, 384, 128, 64), (22, "bf16", 333, 640, 128, 64),
    (17, "f16", 449, 1000, 128, 64), (2, "f16", 5000, 72, 128, 64), (9, "bf16", 1025, 2304, 128, 64), (1, "bf16", 16384, 1152, 128, 64),
    (3, "bf16", 5470, 128, 128, 128), (3, "f16", 8192, 256, 64, 128), (3, "bf16", 8193, 384, 128, 128), (10, "bf16", 2250, 648, 128, 128),
    (8, "bf16", 3072, 512, 128, 128), (8, "bf16", 3073, 512, 128, 128), (8, "f16", 3000, 1000, 128, 128), (8, "f16", 3100, 1000, 128, 128)])
def test_one_tile(C, dtype, T, d, b, rows):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"one_tile_{dtype}_C{C}_T{T}_d{d}_b{b}", 97, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    route = tr.call_route(tr.DTYPE_CODES[dtype], C, T, d, b)
    assert (route["kernel"], route["rows_per_tile"]) == (TILE, rows)
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
