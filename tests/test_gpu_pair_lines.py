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


# few rows | pair: one 16-row tile below and above the line
FEW = [("bf16", 8, T, 1024, 128) for T in (96, 97)] + [("f16", 8, T, 2048, 128) for T in (96, 97)] + [("f32", 4, T, 1024, 128) for T in (192, 193)]
FEW += [("bf16", 1, T, 2560, 128) for T in (512, 513)] + [("bf16", 1, T, 4096, 128) for T in (448, 449)] + [("f32", 8, T, 2048, 128) for T in (48, 49)]
FEW += [("bf16", 2, T, 4096, 256) for T in (112, 113)] + [("f16", 8, T, 5120, 128) for T in (16, 17)] + [("f32", 3, T, 2560, 64) for T in (16, 17)]
FEW += [("bf16", 1, T, 8192, 128) for T in (16, 17, 33)] + [("bf16", 8, T, 2904, 128) for T in (32, 33, 64, 65)] + [("f32", 6, T, 1448, 128) for T in (32, 33, 80, 81)]
FEW += [("f16", 20, 40, 1000, 128), ("bf16", 8, 97, 1448, 128)] + [("bf16", 1, T, 5120, 128) for T in (96, 97)]
FEW += [("bf16", 3, T, 6144, 128) for T in (32, 33)] + [("f32", 2, T, 3072, 128) for T in (64, 65)] + [("bf16", 8, T, 6144, 64) for T in (32, 33)]
# pair | streaming forms, width 256 with fp32 rows beyond a 64-row tile per CU
PAIR = [("bf16", 1, 3000, 2048, 128), ("f16", 1, 5000, 4096, 128), ("f32", 6, 700, 768, 128), ("f32", 6, 600, 768, 256), ("f32", 5, 1000, 1024, 256),
        ("f32", 5, 3400, 512, 256), ("f32", 7, 1676, 2560, 256), ("f16", 6, 1500, 8192, 256), ("bf16", 7, 722, 8192, 128)]


@pytest.mark.parametrize("raw", [False, True])
@pytest.mark.parametrize("dtype,C,T,d,b", FEW + PAIR)
def test_either_side_of_a_line(dtype, C, T, d, b, raw):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    if raw and (dtype, C, T, d, b) in PAIR[5:]:
        pytest.skip("the packed call covers this size")
    w, rt, hb, h, (g, W1, b1, w2) = inputs(dtype, C, T, d, b)
    tail = (b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers)
    pk = None if raw else tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    call = lambda: tr.select_exit(h, g, w.eps, W1, *tail) if raw else tr.select_exit_packed(h, pk, w.eps, *tail, d=d)
    out = [call() for _ in range(2)]
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(*out)), "two calls differ"
    ex, z, m = (o.cpu().numpy() for o in out[0])
    ex_o, z_o, m_o = oracle_select(w, rt, hb)
    report(compare_select(w.name, dtype, z, ex, m, z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))


@pytest.mark.parametrize("dtype,C,T,d,b", [("f32", 10, 1763, 512, 256), ("f32", 4, 1056, 8192, 256), ("f16", 8, 669, 8192, 256), ("f16", 8, 64, 4096, 128)])
def test_the_fixed_scratch_array(dtype, C, T, d, b):
    """Calls whose cheapest pair keeps more partial results than the array holds take a smaller one."""
    import torch
    from paper_2603_21365_amd import tide_route as tr
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
