"""GPU parity of the few-rows kernel (packed weights, automatic choice, few rows per call) against the fp64 oracle, at the
edges of its tiles: one row, a second tile of one row, as many row tiles as there are counters, hidden sizes with a partial
last 32-k group and a partial last turn, every width and storage type, and rows that were re-aligned first."""
import numpy as np
import pytest

import oracle
from paper_2603_21365_amd import synth
from parity import TOL, compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tr():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2603_21365_amd import tide_route
    tide_route.load_library()
    return tide_route


@pytest.mark.parametrize("C,dtype,T,d,b", [
    (1, "f16", 1, 4096, 128), (8, "bf16", 17, 4096, 128), (3, "f32", 16, 768, 128), (8, "f32", 5, 4096, 128),
    (5, "bf16", 33, 1608, 128), (2, "f16", 15, 72, 64), (7, "bf16", 40, 2056, 64), (3, "f32", 20, 100, 128),
    (4, "bf16", 9, 4096, 256), (15, "f16", 7, 1024, 256), (31, "f16", 3, 256, 128), (1, "bf16", 1024, 256, 64),
    (1, "f16", 1009, 384, 64), (3, "bf16", 8, 16384, 128), (2, "bf16", 50, 1001, 128), (2, "f16", 30, 200, 256),
    (2, "f32", 8, 8192, 128), (2, "f32", 9, 8192, 256), (1, "bf16", 24, 16384, 128), (2, "f16", 12, 12288, 64)])
def test_few_rows(tr, C, dtype, T, d, b):
    import torch
    w = synth.Workload(f"few_{dtype}_C{C}_T{T}_d{d}_b{b}", 71, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, C) if C > 1 else 0.05
    hb = w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    pk = tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    dev = to_device(hb, dtype)
    min_layer = 4 * (C // 3)
    first = None
    for rep in range(3):            # the counters and the partial logits return to zero: identical bits every time
        out = tr.select_exit_packed(dev, pk, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, min_layer, w.n_layers, d=d)
        torch.cuda.synchronize()
        got = [o.cpu().numpy() for o in out]
        first = got if first is None else first
        assert all(np.array_equal(a, b_) for a, b_ in zip(first, got)), f"call {rep} differs from the first"
    ex_o, z_o, m_o = oracle_select(w, rt, hb, min_layer=min_layer)
    report(compare_select(w.name, dtype, first[1], first[0], first[2], z_o, ex_o, m_o, rt.theta, w.layer_ids, min_layer, w.n_layers))


@pytest.mark.parametrize("T,d", [(1, 2048), (23, 1544)])
def test_every_output_without_exit_selection(tr, T, d):
    import torch
    w = synth.Workload(f"few_eval_T{T}", 73, "bf16", d, 4, 4, T, None)
    h, rt = w.hidden(), w.routers()
    z_o, p_o, f_o = oracle.router_eval(h[0], "bf16", rt.gamma[0], w.eps, rt.W1[0], None, rt.w2[0], 0.1, 0.5)
    g, W1, _, w2 = routers_to_device(rt)
    prob, fire, logit = tr.router_eval_packed(to_device(h[0], "bf16"), tr.router_pack(tr.BF16, g[:1], W1[:1]), w.eps, None, w2[0], 0.1,
                                              0.5, d=d)
    torch.cuda.synchronize()
    assert np.abs(logit.cpu().numpy() - z_o).max() <= TOL["bf16"] and np.abs(prob.cpu().numpy() - p_o).max() <= TOL["bf16"]
    away = np.abs(z_o) > TOL["bf16"]
    assert np.array_equal(fire.cpu().numpy()[away], f_o[away])


@pytest.mark.parametrize("C,T,d,b", [(1, 8, 128, 128), (8, 1, 128, 64), (8, 32, 1000, 128), (4, 32, 4104, 64), (2, 9, 1608, 128)])
def test_fp32_rows_keep_all_their_bits_where_the_latency_kernel_does(tr, C, T, d, b):
    """fp32 rows, up to 32 per checkpoint, d = 128 or no multiple of 128, packed weights that the packed form holds exactly (16 bits
    of fraction at most): what is left is fp32 summation.  A pre-activation is a sum of about unit size, in error by the rounding
    of its d products and sums, at most 2 sqrt(d) * 2^-24 of it (the roundings are independent), and the logit, a sum of b terms
    of |w2| = 1 / sqrt(b) with slopes of SiLU up to 1.1, by at most the same relative to its own unit size.  Rows cut to two
    bf16 terms (2^-17 of a value) show 3e-6 and more of the norm."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(1000 * T + d)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    h, W1, w2, b1 = r(C, T, d), torch.round(r(C, d, b) / d ** 0.5 * 2 ** 14) / 2 ** 14, r(C, b) / b ** 0.5, 0.1 * r(C, b)
    print(f"[gpu-case] fp32 bits C={C} T={T} d={d} b={b}", flush=True)
    ids = [4 * c + 3 for c in range(C)]
    z = tr.select_exit_packed(h, tr.router_pack(tr.F32, None, W1), 1e-6, b1, w2, [0.0] * C, [0.5] * C, ids, 0, 4 * C, d=d)[1].cpu().double()
    hd, Wd, bd, wd = (x.cpu().double() for x in (h, W1, b1, w2))
    x = hd / torch.sqrt((hd * hd).mean(-1, keepdim=True) + 1e-6)
    pre = torch.stack([x[c] @ Wd[c] for c in range(C)]) + bd[:, None]
    z_o = (pre * torch.sigmoid(pre) * wd[:, None]).sum(-1)
    err = ((z - z_o).norm() / z_o.norm()).item()
    assert err < min(2 * d ** 0.5 * 2.0 ** -24, 1.5e-6), err


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_non_finite_rows_stay_by_themselves(tr, dtype):
    """A row with an infinity or a NaN has a NaN logit and fires nothing; the rows beside it in its tile, and the zeros that
    stand in beyond the end of a row (d = 1544), are not touched by it."""
    import torch
    w = synth.Workload("few_nonfinite", 79, dtype, 1544, 12, 4, 21, None)
    rt = w.routers()
    g, W1, b1, w2 = routers_to_device(rt)
    pk = tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    h = to_device(w.hidden(), dtype)
    args = (w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers)
    ex0, z0, m0 = tr.select_exit_packed(h, pk, *args, d=w.d)
    bad = h.clone()
    bad[:, 3, 1543] = float("inf")
    bad[:, 20, 0] = float("nan")
    ex1, z1, m1 = tr.select_exit_packed(bad, pk, *args, d=w.d)
    torch.cuda.synchronize()
    rows = np.array([3, 20])
    assert torch.isnan(z1[:, rows]).all() and (m1[rows] == 0).all() and (ex1[rows] == w.n_layers).all()
    keep = np.setdiff1d(np.arange(w.T), rows)
    assert torch.equal(z0[:, keep], z1[:, keep]) and torch.equal(ex0[keep], ex1[keep]) and torch.equal(m0[keep], m1[keep])


def test_a_block_stays_usable_and_a_small_one_suffices(tr):
    """On a caller's block the call leaves zeros behind its state words, so a call with more state may follow without another
    tide_workspace_init; a block that holds only what the other paths need (state words: d = 768) is still accepted."""
    import torch
    few = synth.Workload("few_ws", 83, "bf16", 768, 16, 4, 48, None)
    many = synth.Workload("few_ws_many", 83, "bf16", 768, 16, 4, 5000, None)
    rt = few.routers()
    g, W1, b1, w2 = routers_to_device(rt)
    pk = tr.router_pack(tr.BF16, g, W1)
    hf, hm = to_device(few.hidden(), "bf16"), to_device(many.hidden(), "bf16")
    args = (b1, w2, rt.b2, rt.theta, few.layer_ids, 0, few.n_layers)

    def both(h, ws):
        want = tr.select_exit_packed(h, pk, few.eps, *args, d=768)
        got = tr.select_exit_ws(h, None, few.eps, None, pk, *args, ws, d=768)
        torch.cuda.synchronize()
        return want, got
    big = torch.empty(tr.workspace_bytes(tr.BF16, 4, 5000, 768) + 65536, dtype=torch.uint8, device="cuda")
    small = torch.empty(256 + 512, dtype=torch.uint8, device="cuda")
    for ws in (big, small):
        tr.workspace_init(ws)
    for h in (hf, hm, hf, hm):
        assert all(torch.equal(a, b) for a, b in zip(*both(h, big)))
    assert tr.workspace_bytes(tr.BF16, 4, 48, 768) > small.numel()
    want, got = both(hf, small)     # the streaming kernel: the same weights, sums in another order
    assert (want[1] - got[1]).abs().max().item() < 1e-4
    for ws in (big, small):
        tr.workspace_forget(ws)
