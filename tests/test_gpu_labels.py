"""GPU: the cosine labels where the kernel's shape changes -- every number of 16-byte chunks per thread and its edges (rows of whole and of
partial chunk rounds, a wave and a workgroup per row), one, two and four units per token, fewer checkpoints than units -- against the fp64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2603_21365_amd import synth
from parity import to_device

pytestmark = pytest.mark.gpu

SHAPES = [("bf16", d, 5, 37) for d in (8, 512, 1024, 1032, 1536, 1544, 2048, 2560, 2568, 3072, 3080, 4096, 4104, 5120, 5128, 6144, 6152, 8192, 8200, 16384)]
SHAPES += [("f16", 2552, 9, 70), ("f32", 512, 4, 33), ("f32", 1276, 6, 41), ("f32", 2560, 5, 90), ("f32", 4096, 5, 18), ("f32", 4100, 7, 21), ("f32", 8192, 10, 19)]
# the lines between one, two and four units per token, and checkpoints that do not divide among them
SHAPES += [("bf16", 768, 7, T) for T in (999, 1001, 1501, 2599, 2602)] + [("f16", 2560, 6, T) for T in (1000, 1003)]
SHAPES += [("bf16", 3072, 5, T) for T in (700, 701, 1500, 1503, 1899, 1901)] + [("f16", 1024, C, T) for C in (1, 2, 3) for T in (50, 1500, 1505)] + [("f32", 8192, C, 11) for C in (1, 2, 3)]

SHAPES += [("bf16", 768, 8, T) for T in (1800, 1801, 3200, 3201)] + [("f16", 1536, 4, T) for T in (3200, 3203)] + [("bf16", 2048, 5, T) for T in (2500, 2501)]
SHAPES += [("bf16", 2560, C, T) for C in (4, 9) for T in (2000, 2001, 2401, 3201)] + [("f16", 3072, 4, T) for T in (2001, 4801)] + [("bf16", 4096, 3, 1901), ("f32", 4104, 3, 501)]


@pytest.mark.parametrize("dtype,d,C,T", SHAPES)
def test_labels_where_the_kernel_changes_shape(dtype, d, C, T):
    import torch
    from paper_2603_21365_amd import tide_route as tr
    w = synth.Workload(f"labels_{dtype}_C{C}_T{T}_d{d}", 107, dtype, d, 4 * C, 4, T, None)
    print(f"[gpu-case] {w.name}", flush=True)
    hb, fin = w.hidden(), synth.make_hidden(108, 1, T, d, dtype)[0]
    tau = 0.5
    sim_o, lab_o = oracle.cosine_labels(hb, dtype, fin, tau)
    sim, lab = tr.cosine_labels(to_device(hb, dtype), to_device(fin, dtype), tau)
    torch.cuda.synchronize()
    # three fp32 sums of d products in a fixed order (d / 64 per lane, then six levels), relative to the rows' norms: the square root of the
    # longest chain in units of 2^-24, with a factor of four
    bound = 4 * np.sqrt(d / 64 + 8) * 2.0 ** -24 + 2e-7
    assert np.abs(sim.cpu().numpy() - sim_o).max() <= bound
    clear = np.abs(sim_o - tau) > bound
    np.testing.assert_array_equal(lab.cpu().numpy()[clear], lab_o[clear])


def test_more_tokens_than_a_launch_has_threads_for_four_units():
    """17 million rows of just over 4 KiB: four waves per token would be 2^32 threads.  One buffer serves as both rows (the last layer's one token
    ahead) and, without a stride between them, as all checkpoints'; the rows are one row and its negative by turns of seven, so the similarity is 1 or -1."""
    import torch
    from paper_2603_21365_amd import tide_route as tr
    C, T, d = 4, (1 << 24) + 5, 2056
    if torch.cuda.get_device_properties(0).total_memory < 100 << 30:
        pytest.skip("69 GB of rows")
    print(f"[gpu-case] labels C={C} T={T} d={d}", flush=True)
    sign = (torch.arange(T + 1, device="cuda") % 7 < 3).to(torch.bfloat16) * 2 - 1
    row = torch.randn(d, generator=torch.Generator(device="cuda").manual_seed(5), device="cuda").to(torch.bfloat16)
    buf = torch.empty((T + 1, d), dtype=torch.bfloat16, device="cuda")
    torch.mul(sign[:, None], row[None, :], out=buf)
    hidden = buf.as_strided((C, T, d), (0, d, 1))
    sim, label = tr.cosine_labels(hidden, buf[1:], 0.5)
    torch.cuda.synchronize()
    want = sign[:-1].float() * sign[1:].float()
    assert (sim - want).abs().max().item() < 1e-5 and torch.equal(label.bool(), (want > 0).expand(C, T))
    del buf, hidden
    torch.cuda.empty_cache()
