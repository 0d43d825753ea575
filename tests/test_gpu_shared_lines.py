"""GPU: rows that are no whole k-tiles, laid out on whole 128-byte lines and not (row stride, checkpoint stride or base off a line): the same plan
and the same products, so the same bits, and right against the fp64 oracle.  One size for every kernel that such rows reach."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,C,T,d,kernel", [
    ("bf16", 9, 3700, 1032, 8), ("f16", 8, 765, 600, 8), ("f16", 8, 765, 392, 5), ("f32", 8, 700, 520, 11), ("f32", 16, 1600, 132, 11), ("bf16", 10, 3001, 200, 4),
    ("f16", 8, 1900, 1000, 4), ("bf16", 1, 2000, 2600, 1), ("f32", 2, 300, 1300, 1), ("bf16", 7, 4650, 264, 7)])
def test_rows_on_and_off_whole_lines(dtype, C, T, d, kernel):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    code = tr.DTYPE_CODES[dtype]
    assert tr.prefill_plan(code, C, T, d)[0]["kernel"] == kernel
    w = synth.Workload(f"lines_{dtype}_C{C}_T{T}_d{d}", 127, dtype, d, 4 * C, 4, T, None)
    print(f"[gpu-case] {w.name}", flush=True)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, C) if C > 1 else 0.05
    hb = w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    pk = tr.router_pack(code, g, W1)
    src = to_device(hb, dtype)
    line, chunk = (32, 4) if dtype == "f32" else (64, 8)         # elements in 128 and in 16 bytes
    width = -(-d // line) * line
    outs = []
    for base, stride, gap in ((0, width, 0), (chunk, width, 0), (0, width + chunk, 0), (0, width, chunk)):
        ckpt = T * stride + gap
        room = torch.full((base + C * ckpt,), float("nan"), dtype=src.dtype, device="cuda")
        h = room[base:].as_strided((C, T, d), (ckpt, stride, 1))
        h.copy_(src)
        out = tr.select_exit_packed(h, pk, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, d=d)
        torch.cuda.synchronize()
        outs.append([o.cpu().numpy() for o in out])
    for other in outs[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(outs[0], other))
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    report(compare_select(w.name, dtype, outs[0][1], outs[0][0], outs[0][2], z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
