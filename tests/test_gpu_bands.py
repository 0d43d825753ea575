"""GPU parity of the band kernels' newer branches against the fp64 oracle: fp32 rows in bands (pairs of waves per block up to
four blocks per workgroup, a wave per block beyond), checkpoints that do not divide the workgroups, and hidden sizes that are
no multiple of 128 on every kernel the automatic settings give them."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tr():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2603_21365_amd import tide_route
    tide_route.load_library()
    return tide_route


def check(tr, C, dtype, T, d, b, *, packed, pad=0):
    import torch
    w = synth.Workload(f"bands_{dtype}_C{C}_T{T}_d{d}_b{b}", 89, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, C) if C > 1 else 0.05
    hb = w.hidden(row_stride=d + pad)
    g, W1, b1, w2 = routers_to_device(rt)
    dev = to_device(hb, dtype)
    args = (b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers)
    out = []
    for rep in range(2):
        if packed:
            pk = tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
            out.append(tr.select_exit_packed(dev, pk, w.eps, *args, d=d))
        else:
            out.append(tr.select_exit(dev, g, w.eps, W1, *args))
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(*out)), "two calls differ"
    ex, z, m = (o.cpu().numpy() for o in out[0])
    ex_o, z_o, m_o = oracle_select(w, rt, hb, d=d)
    report(compare_select(w.name, dtype, z, ex, m, z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))


@pytest.mark.parametrize("C,T,d,b,what", [
    (3, 6001, 512, 128, "2 and 3 blocks per workgroup, the last one block of one row"),
    (7, 4500, 768, 64, "3 and 4 blocks; 4 workgroups without a checkpoint"),
    (1, 32768, 512, 128, "exactly 4 blocks: the most that pairs of waves take"),
    (1, 32800, 512, 128, "one block more: 4 and 5 blocks, a wave each"),
    (10, 4700, 512, 128, "5 and 6 blocks: the largest of its range"),
    (32, 540, 640, 128, "32 checkpoints, 8 workgroups each, 2 and 3 blocks")])
def test_fp32_bands(tr, C, T, d, b, what):
    assert [L["kernel"] for L in tr.prefill_plan(tr.F32, C, T, d, b)] == [11], what
    check(tr, C, "f32", T, d, b, packed=C % 2 == 1)


@pytest.mark.parametrize("C,dtype,T,d", [
    (3, "bf16", 16000, 256), (7, "f16", 5000, 384), (12, "bf16", 4000, 256), (10, "bf16", 3300, 512)])
def test_checkpoints_that_do_not_divide_the_workgroups(tr, C, dtype, T, d):
    assert [L["kernel"] for L in tr.prefill_plan(tr.DTYPE_CODES[dtype], C, T, d)] == [8]
    check(tr, C, dtype, T, d, 128, packed=True)


@pytest.mark.parametrize("C,dtype,T,d,b", [
    (9, "bf16", 600, 128, 128), (10, "f16", 161, 384, 64), (16, "bf16", 385, 640, 128), (8, "f16", 1024, 896, 128), (1, "bf16", 8192, 1920, 64)])
def test_few_rows_of_k_tiles_no_multiple_of_four(tr, C, dtype, T, d, b):
    """At most a quarter as many 128-row tiles as CUs, k-tiles that do not go four to a stage: the band, most or all of its
    workgroups with at most one block."""
    assert [L["kernel"] for L in tr.prefill_plan(tr.DTYPE_CODES[dtype], C, T, d, b)] == [8]
    check(tr, C, dtype, T, d, b, packed=True)
    check(tr, C, dtype, T, d, b, packed=False)


@pytest.mark.parametrize("C,dtype,T,d,b,pad,what", [
    (1, "bf16", 1100, 2000, 128, 0, "split-k, 16-bit rows"),
    (4, "f32", 260, 1100, 128, 4, "split-k, fp32 rows: the last two k-tiles are partial and empty; padded strides"),
    (2, "f16", 40, 8200, 64, 0, "few rows, one 16-byte chunk into a k-tile"),
    (32, "bf16", 12, 1000, 128, 0, "too many checkpoints for the few-rows kernel: the latency kernel"),
    (32, "f16", 33, 456, 128, 8, "pieces of the streaming kernel, the last k-tile partial"),
    (32, "f16", 33, 264, 128, 8, "bands of few rows, the last two k-tiles one chunk and none"),
    (8, "bf16", 1500, 200, 128, 0, "64-row tiles"),
    (8, "f16", 3001, 1032, 128, 8, "one 128-row tile per CU"),
    (8, "bf16", 5003, 136, 128, 0, "bands, two k-tiles"),
    (12, "bf16", 4000, 808, 64, 0, "bands of one checkpoint each"),
    (12, "bf16", 2700, 1600, 128, 0, "more than half a round of 256-row tiles, four blocks per CU at most: bands"),
    (10, "bf16", 3100, 1608, 128, 8, "the same, a 128-row tile per CU at most: the one-tile kernel"),
    (31, "f16", 1040, 1032, 64, 0, "the same, short last tiles: bands"),
    (7, "bf16", 4650, 1000, 128, 0, "the same, two 64-row tiles per CU at most: the register-ring kernel"),
    (3, "f32", 700, 132, 128, 0, "fp32 bands of one block, one chunk in the last k-tile"),
    (10, "f32", 9000, 140, 128, 4, "fp32 bands in several tiles"),
    (2, "f32", 9000, 1000, 64, 0, "fp32 bands in pairs of waves")])
def test_hidden_sizes_that_are_no_multiple_of_128(tr, C, dtype, T, d, b, pad, what):
    print(f"[gpu-case] {what}", flush=True)
    check(tr, C, dtype, T, d, b, packed=True, pad=pad)
    check(tr, C, dtype, T, d, b, packed=False, pad=pad)


def test_rows_beside_a_ragged_end_do_not_reach_each_other(tr):
    """d = 1000 in a buffer whose columns beyond d hold NaN: nothing beyond a row's end is used, on every kernel that
    fetches zeros there."""
    import torch
    for dtype, C, T in (("bf16", 2, 24), ("bf16", 1, 900), ("f16", 8, 3001), ("bf16", 8, 5003), ("f32", 4, 260), ("f32", 3, 1500)):
        w = synth.Workload(f"bands_nan_{dtype}_T{T}", 97, dtype, 1000, 4 * C, 4, T, None)
        print(f"[gpu-case] {w.name}", flush=True)
        rt = w.routers()
        g, W1, b1, w2 = routers_to_device(rt)
        pk = tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
        h = to_device(w.hidden(), dtype)
        wide = torch.full((C, T, 1016), float("nan"), dtype=h.dtype, device="cuda")
        wide[:, :, :1000] = h
        args = (w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers)
        a, b = tr.select_exit_packed(h, pk, *args, d=1000), tr.select_exit_packed(wide, pk, *args, d=1000)
        torch.cuda.synchronize()
        assert torch.isfinite(a[1]).all() and all(torch.equal(x, y) for x, y in zip(a, b))
