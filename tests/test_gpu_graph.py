"""GPU: the entry points under HIP graph capture.  Once the workspace exists (one eager call of the
same size), a call enqueues kernels only -- no allocation, no memset, no host synchronisation --
so a serving loop can capture it and replay it.  Every replay is checked against the eager result
on the same inputs, with eager work and synchronisations between the replays."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import routers_to_device, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tr():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2603_21365_amd import tide_route
    tide_route.load_library()
    yield tide_route
    tide_route.set_variant(tide_route.VARIANT_AUTO)


@pytest.mark.parametrize("case", ["decode_T8_raw", "decode_T8_packed", "prefill_T600_packed_then_project",
                                  "prefill_width256_two_launches_then_project"])
def test_captured_calls_replay_like_eager_calls(tr, case):
    import torch
    decode = case.startswith("decode")
    two_launches = "two_launches" in case                      # width 256 beyond one round of 256-row tiles: the square
    T = 8 if decode else 4100 if two_launches else 600         # form, then 128-row tiles; the arrival words carry the state
    dtype = "f16" if decode else "bf16"
    if two_launches:
        w = synth.Workload(f"graph_{case}", 53, dtype, 320, 40, 2, T, None, b=256)
        if torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert [L["kernel"] for L in tr.prefill_plan(tr.BF16, w.C, T, w.d, 256)] == [10, 4]
    else:
        w = synth.Workload(f"graph_{case}", 53, dtype, 1024, 16, 4, T, None)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, w.C)
    g, W1, b1, w2 = routers_to_device(rt)
    batches = [to_device(synth.make_hidden(w.cfg + i, w.C, T, w.d, dtype), dtype) for i in range(4)]
    final = to_device(synth.make_hidden(w.cfg + 9, 1, T, w.d, dtype)[0], dtype)
    hidden = torch.empty_like(batches[0])                      # the buffer the graph reads
    out = (torch.empty(T, dtype=torch.int32, device="cuda"), torch.empty((w.C, T), dtype=torch.float32, device="cuda"),
           torch.empty(T, dtype=torch.int32, device="cuda"))
    proj = torch.empty((T, w.d), dtype=hidden.dtype, device="cuda")
    raw = case.endswith("raw")
    packed = None if raw else tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)

    def step():
        if raw:                                                # the latency kernel
            tr.select_exit(hidden, g, w.eps, W1, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, out=out)
        elif decode:                                           # the split-k pair: two kernels, partial results in the workspace
            tr.select_exit_packed(hidden, packed, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, d=w.d, out=out)
        else:
            tr.select_exit_packed(hidden, packed, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, d=w.d, out=out)
            tr.exit_project(hidden, final, out[0], w.layer_ids, None, 1e-6, out=proj)

    def eager(batch):
        hidden.copy_(batch)
        step()
        torch.cuda.synchronize()
        return [o.clone() for o in out] + [proj.clone()]

    want = [eager(b) for b in batches]                         # also creates the workspace
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        hidden.copy_(batches[0])
        step()                                                 # warm-up on the capture stream
        stream.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            step()
    torch.cuda.synchronize()
    for rep in range(3):
        for i, b in enumerate(batches):
            hidden.copy_(b)                                    # eager work between the replays
            for o in out:
                o.fill_(-7)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            got = list(out) + [proj]
            n = 3 if decode else 4
            for k in range(n):
                assert torch.equal(got[k], want[i][k]), f"{case}: replay {rep} of batch {i}, output {k} differs from the eager call"
    print(f"[gpu-case] {case}: 12 replays equal to the eager results", flush=True)


@pytest.mark.parametrize("T,d", [(40, 1608), (600, 1608)])     # few rows; rows beyond a multiple of 128, split over k
def test_capture_after_an_eager_call_that_left_no_partial_results(tr, T, d):
    """The workspace of a larger streaming call is enough to capture a smaller one, although the smaller one keeps partial
    results when it may allocate them."""
    import torch
    from parity import compare_select, oracle_select, report
    w = synth.Workload(f"graph_small_T{T}_d{d}", 57, "bf16", d, 4, 4, T, None)      # one checkpoint
    rt = w.routers()
    hb = w.hidden()
    g, W1, b1, w2 = routers_to_device(rt)
    packed = tr.router_pack(tr.BF16, g, W1)
    hidden = to_device(hb, "bf16")
    large = hidden.repeat(1, 16384 // T + 1, 1).contiguous()
    out = (torch.empty(T, dtype=torch.int32, device="cuda"), torch.empty((w.C, T), dtype=torch.float32, device="cuda"),
           torch.empty(T, dtype=torch.int32, device="cuda"))

    def call(h, **kw):
        return tr.select_exit_packed(h, packed, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, d=d, **kw)

    torch.cuda.synchronize()
    tr.release()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        call(large)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        call(hidden, out=out)
    for rep in range(3):
        for o in out:
            o.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = [o.cpu().numpy() for o in out]
        ex_o, z_o, m_o = oracle_select(w, rt, hb, min_layer=0)
        report(compare_select(f"{w.name} replay {rep}", "bf16", got[1], got[0], got[2], z_o, ex_o, m_o, rt.theta, w.layer_ids, 0, w.n_layers))
    with torch.cuda.stream(stream):
        call(hidden)                    # eager again: may allocate (after the last replay)
    torch.cuda.synchronize()
    del graph


@pytest.mark.parametrize("dtype,C,d,b,raw,T_graph,T_later", [
    ("bf16", 4, 768, 128, False, 48, (96, 300, 5, 1000)),      # few rows where larger calls stream: no partial results there
    ("bf16", 4, 1608, 128, False, 300, (48, 600, 2000)),       # a ragged hidden size, split over k
    ("f16", 8, 4096, 128, False, 8, (16, 48, 64, 500)),        # few rows, then the split-k pair
    ("f32", 3, 1000, 64, False, 20, (32, 33, 150)),
    ("bf16", 2, 1024, 256, False, 30, (70, 800)),
    ("f16", 4, 2048, 128, True, 4, (8, 40, 300))])
def test_a_captured_call_survives_later_calls_that_are_no_larger_than_the_first(tr, dtype, C, d, b, raw, T_graph, T_later):
    """One eager call of the largest T sizes the workspace for every smaller one of the shape: neither the captured call nor the
    eager ones behind it allocate, so the addresses in the graph stay the workspace's."""
    import torch
    w = synth.Workload(f"graph_later_{dtype}_d{d}", 59, dtype, d, 4 * C, 4, 4000, None, b=b)
    rt = w.routers()
    rt.b2[:] = np.linspace(-0.2, 0.2, C)
    g, W1, b1, w2 = routers_to_device(rt)
    packed = None if raw else tr.router_pack(tr.DTYPE_CODES[dtype], g, W1)
    hidden = to_device(w.hidden(), dtype)

    def call(T, **kw):
        h = hidden[:, :T]
        if raw:
            return tr.select_exit(h, g, w.eps, W1, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, **kw)
        return tr.select_exit_packed(h, packed, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, d=d, **kw)

    out = (torch.empty(T_graph, dtype=torch.int32, device="cuda"), torch.empty((C, T_graph), dtype=torch.float32, device="cuda"),
           torch.empty(T_graph, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    tr.release()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        call(w.T)
    torch.cuda.synchronize()
    allocations = tr.workspace_allocations()
    with torch.cuda.stream(stream):
        want = [o.clone() for o in call(T_graph)]
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        call(T_graph, out=out)
    for T in T_later:
        with torch.cuda.stream(stream):
            call(T)
        torch.cuda.synchronize()
        assert tr.workspace_allocations() == allocations, f"T = {T} outgrew the workspace of T = {w.T}"
        for o in out:
            o.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b_) for a, b_ in zip(out, want)), f"replay after T = {T}"
    del graph

def test_few_rows_are_captured_on_what_a_few_rows_call_left(tr):
    """d = 4096 with the partial results of a d = 768 call of the few-rows kernel in the workspace: enough for that kernel, too
    little for the split-k form of the same call."""
    import torch
    def call_of(d, T):
        w = synth.Workload(f"graph_few_d{d}", 61, "f16", d, 16, 4, T, None)
        rt = w.routers()
        g, W1, b1, w2 = routers_to_device(rt)
        packed, h = tr.router_pack(tr.F16, g, W1), to_device(w.hidden(), "f16")
        out = (torch.empty(T, dtype=torch.int32, device="cuda"), torch.empty((w.C, T), dtype=torch.float32, device="cuda"),
               torch.empty(T, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        return lambda: tr.select_exit_packed(h, packed, w.eps, b1, w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, d=d, out=out)
    small, large = call_of(768, 48), call_of(4096, 8)
    tr.release()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        small()
    torch.cuda.synchronize()
    allocations = tr.workspace_allocations()
    with torch.cuda.graph(graph, stream=stream):
        out = large()
    assert tr.workspace_allocations() == allocations
    got = []
    for rep in range(3):
        for o in out:
            o.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got.append([o.clone() for o in out])
    del graph
    with torch.cuda.stream(stream):
        large()
    torch.cuda.synchronize()
    for g_ in got:
        assert all(torch.equal(a, b) for a, b in zip(g_, out))
