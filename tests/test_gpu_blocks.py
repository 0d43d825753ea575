"""GPU: one caller-owned block, sized for the largest of a program's calls, through calls of other row counts: every one is served and right."""
import numpy as np
import pytest

from paper_2603_21365_amd import synth
from parity import compare_select, oracle_select, report, routers_to_device, to_device

pytestmark = pytest.mark.gpu



class Program:
    """A program's calls of one shape but the row count, on one block, each compared with the oracle."""

    def __init__(self, dtype, C, d, most):
        from paper_2603_21365_amd import tide_route as tr
        self.tr, self.dtype, self.d, self.code = tr, dtype, d, tr.DTYPE_CODES[dtype]
        self.w = synth.Workload(f"block_{dtype}_C{C}_d{d}", 131, dtype, d, 4 * C, 4, most, None)
        self.rt = self.w.routers()
        self.rt.b2[:] = np.linspace(-0.2, 0.2, C) if C > 1 else 0.05
        hb = self.w.hidden()
        self.want = oracle_select(self.w, self.rt, hb)
        g, W1, self.b1, self.w2 = routers_to_device(self.rt)
        self.pk = tr.router_pack(self.code, g, W1)
        self.h = to_device(hb, dtype)

    def block(self, nbytes):
        import torch
        self.ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        self.tr.workspace_init(self.ws)

    def call(self, T, **kw):
        print(f"[gpu-case] {self.w.name} T={T} in {self.ws.numel()} bytes", flush=True)
        rt, w = self.rt, self.w
        return self.tr.select_exit_ws(self.h[:, :T], None, w.eps, None, self.pk, self.b1, self.w2, rt.b2, rt.theta, w.layer_ids, 0, w.n_layers, self.ws,
                                      d=self.d, **kw)

    def check(self, T, out):
        import torch
        torch.cuda.synchronize()
        ex, z, m = (o.cpu().numpy() for o in out)
        ex_o, z_o, m_o = self.want
        report(compare_select(f"{self.w.name}_T{T}", self.dtype, z, ex, m, z_o[:, :T], ex_o[:T], m_o[:T], self.rt.theta, self.w.layer_ids, 0, self.w.n_layers))


@pytest.mark.parametrize("dtype,C,d,rows", [("bf16", 8, 768, (4096, 1000, 64, 1, 4096)), ("bf16", 8, 768, (1, 64, 1000, 4096, 1)),
                                            ("bf16", 1, 2048, (8000, 3000, 500, 8000)), ("f32", 6, 1024, (9000, 600, 20)), ("f16", 8, 4096, (4096, 96, 17))])
def test_row_counts_through_a_block_for_the_largest(dtype, C, d, rows):
    p = Program(dtype, C, d, max(rows))
    p.block(p.tr.workspace_bytes(p.code, C, max(rows), d))
    for T in rows:
        p.check(T, p.call(T))
    p.tr.workspace_forget(p.ws)


@pytest.mark.parametrize("spare", [0, 1 << 20])
@pytest.mark.parametrize("dtype,C,d,rows", [("bf16", 1, 2048, (3000, 8000, 500, 3000, 8000)), ("bf16", 8, 768, (1, 40, 4096, 700, 4096)), ("f16", 8, 1024, (16, 700, 4096, 1))])
def test_growing_row_counts_need_no_second_init(dtype, C, d, rows, spare):
    """In a block for the hungriest of the calls, alone and with room for its partial results behind all calls' state."""
    p = Program(dtype, C, d, max(rows))
    p.block(max(p.tr.workspace_bytes(p.code, C, T, d) for T in rows) + spare)
    for T in rows:
        p.check(T, p.call(T))
    p.tr.workspace_forget(p.ws)


@pytest.mark.parametrize("spare", [0, 1 << 20])
def test_a_captured_call_survives_smaller_ones_on_its_block(spare):
    import torch
    p = Program("bf16", 1, 2048, 8000)
    need = p.tr.workspace_bytes(p.code, 1, 3000, 2048)
    assert p.tr.call_route(p.code, 1, 3000, 2048, block_bytes=need)["kernel"] == 1        # the split-k pair: partial results over most of the block
    p.block(need + spare)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    out = (torch.empty(8000, dtype=torch.int32, device="cuda"), torch.empty((1, 8000), dtype=torch.float32, device="cuda"), torch.empty(8000, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        p.call(8000, out=out)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        p.call(8000, out=out)
    for _ in range(3):
        with torch.cuda.stream(stream):
            small = p.call(3000)
        p.check(3000, small)
        for o in out:
            o.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        p.check(8000, out)
    p.tr.workspace_forget(p.ws)
    del graph
