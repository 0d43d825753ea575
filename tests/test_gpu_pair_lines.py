"""GPU parity against the fp64 oracle on both sides of the lines between the few-rows kernel, the split-k pair and the forms behind it: rows of up to
4 KiB, up to 8 KiB and longer at every width, hidden sizes that are no multiple of 128, the pair's wider range at width 256, weights packed by the call; and the
fixed scratch array, whose calls take a pair that fits it."""
import ctypes

import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu


def inputs(dtype, C, T, d, b):
    w = synth.Workload(f"lines_{dtype}_C{C}_T{T}_d{d}_b{b}", 109, dtype, d, 4 * C, 4, T, None, b=b)
    print(f"[gpu-case] {w.name}", flush=True)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, C) if C > 1 else 0.05
    hb = w.hidden()
    return w, rt, hb, to_device(hb, dtype), routers_to_device(rt)


LATENCY, PAIR, STREAM128, STREAM64, FEW = 0, 1, 5, 6, 12          # tide_call_route's kernels
# (dtype, C, T, d, b): the kernel on 256 CUs
KERNELS = {}
# few rows | what lies behind it: one 16-row tile below and above the line
for dtype, C, d, b, last in (("f16", 8, 2048, 128, 96), ("f32", 4, 1024, 128, 192), ("bf16", 1, 2560, 128, 512), ("bf16", 1, 4096, 128, 448), ("f32", 8, 2048, 128, 48),
                             ("bf16", 2, 4096, 256, 112), ("f16", 8, 5120, 128, 16), ("bf16", 1, 8192, 128, 16), ("bf16", 8, 2904, 128, 64), ("f32", 6, 1448, 128, 80),
                             ("bf16", 1, 5120, 128, 96), ("bf16", 3, 6144, 128, 32), ("f32", 2, 3072, 128, 64), ("bf16", 8, 6144, 64, 32)):
    KERNELS[dtype, C, last, d, b], KERNELS[dtype, C, last + 1, d, b] = FEW, PAIR
KERNELS["bf16", 8, 96, 1024, 128], KERNELS["bf16", 8, 97, 1024, 128] = FEW, STREAM128
KERNELS.update({("f32", 3, 16, 2560, 64): FEW, ("f32", 3, 17, 2560, 64): FEW, ("bf16", 8, 32, 2904, 128): FEW, ("bf16", 8, 33, 2904, 128): FEW, ("f32", 6, 32, 1448, 128): FEW,
                ("f32", 6, 33, 1448, 128): FEW, ("bf16", 1, 33, 8192, 128): PAIR, ("f16", 20, 40, 1000, 128): PAIR, ("bf16", 8, 97, 1448, 128): PAIR})
# pair | streaming forms
KERNELS.update({("bf16", 1, 3000, 2048, 128): PAIR, ("f16", 1, 5000, 4096, 128): PAIR, ("f32", 6, 700, 768, 128): PAIR, ("f32", 6, 600, 768, 256): PAIR, ("f32", 5, 1000, 1024, 256): PAIR})
# ... width 256 with fp32 rows beyond a 64-row tile per CU, long rows: the packed call only
PACKED_ONLY = {("f32", 5, 3400, 512, 256): STREAM64, ("f32", 7, 1676, 2560, 256): STREAM64, ("f16", 6, 1500, 8192, 256): PAIR, ("bf16", 7, 722, 8192, 128): PAIR}
CASES = [(*case, False, kernel) for case, kernel in {**KERNELS, **PACKED_ONLY}.items()]
CASES += [(*case, True, LATENCY if case[2] <= 32 and case[3] % 128 else kernel) for case, kernel in KERNELS.items()]


@pytest.mark.parametrize("dtype,C,T,d,b,raw,kernel", CASES)
def test_either_side_of_a_line(dtype, C, T, d, b, raw, kernel):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w, rt, hb, h, (g, W1, b1, w2) = inputs(dtype, C, T, d, b)
    tail = (b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers)
    pk = None if raw else tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert tr.call_route(tr.DTYPE_CODES[dtype], C, T, d, b, raw_weights=raw)["kernel"] == kernel
    call = lambda: tr.select_exit(h, g, w.eps, W1, *tail) if raw else tr.select_exit_packed(h, pk, w.eps, *tail, d=d)
    out = [call() for _ in range(2)]
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(*out)), "two calls differ"
    ex, z, m = (o.cpu().numpy() for o in out[0])
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    report(compare_select(w.name, dtype, z, ex, m, z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))


# what the call takes without a limit and within the array (kernel, rows per tile, slices): fewer slices, lower tiles, no pair; and one that fits
@pytest.mark.parametrize("dtype,C,T,d,b,free,fits", [
    ("f32", 1, 4151, 8192, 256, (PAIR, 64, 8), (PAIR, 64, 4)), ("f32", 1, 5127, 8192, 256, (PAIR, 128, 8), (PAIR, 64, 4)), ("f32", 10, 1650, 2048, 256, (PAIR, 64, 2), (STREAM64, 64, 1)),
    ("f16", 10, 796, 8192, 256, (PAIR, 128, 4), (STREAM64, 64, 1)), ("f16", 8, 669, 8192, 256, (PAIR, 128, 2), (PAIR, 128, 2))])
def test_the_fixed_scratch_array(dtype, C, T, d, b, free, fits):
    """Calls whose cheapest pair keeps more partial results than the array holds take one that fits, or a form without any."""
    import torch
    from paper_2603_21365_amd import tide_route as tr
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        room = tr.noalloc_scratch_bytes()
        assert (tr.workspace_bytes(tr.DTYPE_CODES[dtype], C, T, d, b) > room) == (free != fits)
        for block, want in ((1 << 40, free), (room, fits)):
            route = tr.call_route(tr.DTYPE_CODES[dtype], C, T, d, b, block_bytes=block)
            assert (route["kernel"], route["rows_per_tile"], route["k_slices"]) == want
    lib = tr.load_library()
    w, rt, hb, h, (g, W1, b1, w2) = inputs(dtype, C, T, d, b)
    pk = tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    ex = torch.full((T,), -7, dtype=torch.int32, device="cuda")
    z = torch.full((C, T), float("nan"), dtype=torch.float32, device="cuda")
    m = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    vp, arr = ctypes.c_void_p, lambda a, t: np.ascontiguousarray(np.broadcast_to(np.asarray(a, t), (C,)))
    b2, th, ids = arr(rt.b2, np.float32), arr(rt.theta, np.float32), arr(w.layer_ids, np.int32)
    for _ in range(2):
        rc = lib.tide_select_exit_packed_noalloc(vp(h.data_ptr()), tr.DTYPE_CODES[dtype], C, T, d, b, h.stride(0), h.stride(1), vp(pk.data_ptr()),
                                                 ctypes.c_float(w.eps), vp(b1.data_ptr()), vp(w2.data_ptr()), vp(b2.ctypes.data), vp(th.ctypes.data),
                                                 vp(ids.ctypes.data), 0, w.n_layers, vp(ex.data_ptr()), vp(z.data_ptr()), vp(m.data_ptr()),
                                                 vp(torch.cuda.current_stream().cuda_stream))
        assert rc == 0, tr.last_error()
    torch.cuda.synchronize()
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    report(compare_select(w.name, dtype, z.cpu().numpy(), ex.cpu().numpy(), m.cpu().numpy(), z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))


@pytest.mark.parametrize("dtype,C,T,d,b", [("f16", 8, 96, 4096, 128), ("bf16", 1, 3000, 2048, 128), ("f32", 6, 600, 768, 256), ("bf16", 8, 96, 2904, 128),
                                           ("f32", 8, 64, 5120, 128)])
def test_captured_without_an_eager_call(dtype, C, T, d, b):
    """A graph of a call that the pair would take, captured while the library's workspace holds no partial results of that size: it takes a route that needs no more."""
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w0, rt0, _, h0, (g0, W0, b10, w20) = inputs("bf16", 2, 3100, 256, 128)
    w, rt, hb, h, (g, W1, b1, w2) = inputs(dtype, C, T, d, b)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        route, room = tr.call_route(tr.DTYPE_CODES[dtype], C, T, d, b), max(tr.call_route(tr.BF16, 2, t, 256)["scratch_bytes"] for t in (8, 16, *range(32, 3104, 32)))
        assert route["kernel"] == PAIR and route["scratch_bytes"] > room
    pk0, pk = tr.router_pack(tr.BF16, g0, W0), tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    out = (torch.empty(T, dtype=torch.int32, device="cuda"), torch.empty((C, T), dtype=torch.float32, device="cuda"), torch.empty(T, dtype=torch.int32, device="cuda"))
    call = lambda **kw: tr.select_exit_packed(h, pk, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, d=d, **kw)
    torch.cuda.synchronize()
    tr.release()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):                   # arrival words for T tokens, room for few partial results
        tr.select_exit_packed(h0, pk0, w0.eps, b10, w20, rt0.b2, rt0.theta, w0.layer_ids, 0, w0.n_layers, d=256)
        tr.select_exit_packed(h0[:, :40], pk0, w0.eps, b10, w20, rt0.b2, rt0.theta, w0.layer_ids, 0, w0.n_layers, d=256)
    torch.cuda.synchronize()
    allocations = tr.workspace_allocations()
    with torch.cuda.graph(graph, stream=stream):
        call(out=out)
    assert tr.workspace_allocations() == allocations
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    for rep in range(3):
        for o in out:
            o.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        report(compare_select(f"{w.name}_{rep}", dtype, out[1].cpu().numpy(), out[0].cpu().numpy(), out[2].cpu().numpy(), z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
    del graph
