"""CPU: which kernel a call takes and in how much scratch memory (tide_call_route): a caller's block that holds what a call cannot do without is
never too small, whatever the route without a limit would use."""
import random

import pytest

from paper_2603_21365_amd import tide_route as tr

SPLITK, FUSED = 1, 9
SIZES = (200, 512, 768, 1000, 1024, 1608, 2048, 2560, 4096, 5120, 8192)


def state_bytes(T):
    return 256 + -(-8 * T // 256) * 256


def refused(*shape, **kw):
    try:
        tr.call_route(*shape, **kw)
    except tr.TideError as e:
        assert e.status == -4
        return True
    return False


@pytest.mark.parametrize("dtype,C,d,T,smaller", [(tr.BF16, 8, 768, 4096, (1, 8, 16, 64, 300, 1000)), (tr.BF16, 8, 1024, 4096, (1, 16, 64, 1000)),
                                                 (tr.F16, 1, 2048, 8000, (1, 40, 500, 3000)), (tr.F32, 6, 1024, 9000, (20, 600))])
def test_a_block_for_the_largest_call_serves_the_smaller_ones(dtype, C, d, T, smaller):
    block = tr.workspace_bytes(dtype, C, T, d)
    for t in smaller:
        assert tr.call_route(dtype, C, t, d, block_bytes=block)["scratch_bytes"] <= block
    # and one that holds their state words only: without partial results
    for t in smaller:
        assert tr.call_route(dtype, C, t, d, block_bytes=state_bytes(t))["kernel"] not in (SPLITK, FUSED)


def test_any_block_that_holds_what_the_call_cannot_do_without():
    rng = random.Random(3)
    for _ in range(4000):
        dtype, C, d, b, raw = rng.choice((tr.F32, tr.F16, tr.BF16)), rng.randint(1, 32), rng.choice(SIZES), rng.choice((64, 128, 256)), rng.random() < 0.3
        T = int(round(2 ** rng.uniform(0, 13)))
        shape = (dtype, C, T, d, b)
        full, free = tr.workspace_bytes(*shape, raw_weights=raw), tr.call_route(*shape, raw_weights=raw, block_bytes=1 << 40)
        assert free["scratch_bytes"] == full
        fits = tr.call_route(*shape, raw_weights=raw, block_bytes=full)
        assert all(fits[k] == free[k] for k in ("kernel", "rows_per_tile", "k_slices", "scratch_bytes"))
        least = state_bytes(T) + (C * tr.packed_router_bytes(dtype, d, b) if raw else 0)
        if d * (4 if dtype == tr.F32 else 2) % 16 or (b == 256 and d % 128):
            least += -(-C * T * -(-d // 128) * 128 * (4 if dtype == tr.F32 else 2) // 256) * 256
        elif free["kernel"] == tr.ROUTE_LATENCY or (d % 128 or d < 256) and T <= 32 or raw and T <= 8:
            continue                                # the latency kernel needs its partial results (the few-rows kernel may stand in for it)
        for block in (least, least + 256, (least + full) // 512 * 256, full - 256):
            if least <= block < full:
                assert tr.call_route(*shape, raw_weights=raw, block_bytes=block)["scratch_bytes"] <= block, (shape, raw, block, full)
        assert refused(*shape, raw_weights=raw, block_bytes=least - 256)


def test_a_small_block_gives_the_few_rows_kernel_what_it_uses():
    """C = 8, T = 48, d = 4096: a float per row and 16 columns, where the split-k pair behind it would keep megabytes."""
    shape = (tr.BF16, 8, 48, 4096)
    least = state_bytes(48) + 48 * 8 * 8 * 4
    assert tr.workspace_bytes(*shape) > 64 * least
    assert tr.call_route(*shape)["kernel"] == tr.ROUTE_FEW_ROWS
    assert tr.call_route(*shape, block_bytes=least) == {"kernel": tr.ROUTE_FEW_ROWS, "rows_per_tile": 16, "k_slices": 1, "scratch_bytes": least, "zeros_kept": least}
    assert tr.call_route(*shape, block_bytes=least - 256)["kernel"] not in (SPLITK, FUSED, tr.ROUTE_FEW_ROWS)


@pytest.mark.parametrize("dtype,C,T,d,b", [(tr.BF16, 1, 3000, 2048, 128), (tr.BF16, 8, 48, 4096, 128), (tr.F32, 6, 600, 1024, 256), (tr.F16, 8, 700, 1024, 64),
                                           (tr.BF16, 8, 4096, 768, 128), (tr.BF16, 28, 8, 2560, 128)])
def test_a_call_leaves_the_state_of_larger_ones_alone(dtype, C, T, d, b):
    """In a block with room for both: partial results lie at its end, and the few-rows kernel leaves zeros where it wrote."""
    block = (16 << 20) + 512
    route = tr.call_route(dtype, C, T, d, b, block_bytes=block)
    assert route["zeros_kept"] > state_bytes(16384)
    assert route["zeros_kept"] == (block - (route["scratch_bytes"] - state_bytes(T)) if route["kernel"] in (SPLITK, FUSED) else block)


def test_a_forced_form_is_refused_below_its_need():
    shape = (tr.BF16, 8, 700, 1024)
    tr.set_prefill_form(tr.splitk_form(32, 8))
    try:
        full = tr.workspace_bytes(*shape)
        assert tr.call_route(*shape, block_bytes=full)["kernel"] == SPLITK
        assert refused(*shape, block_bytes=full - 256)
    finally:
        tr.set_prefill_form(0)


# up to 16 rows of more checkpoints than the few-rows kernel takes: (dtype, T, d) -> kernel and slices at C = 28
@pytest.mark.parametrize("dtype,T,d,kernel,slices", [(tr.BF16, 8, 512, 5, 1), (tr.BF16, 16, 512, 5, 1), (tr.BF16, 8, 768, FUSED, 2), (tr.BF16, 16, 1024, FUSED, 4),
                                                     (tr.F16, 1, 2560, FUSED, 4), (tr.BF16, 16, 2560, FUSED, 4), (tr.BF16, 8, 4096, FUSED, 8), (tr.F32, 8, 1024, FUSED, 4)])
def test_few_rows_of_many_checkpoints(dtype, T, d, kernel, slices):
    for C in (28, 32):
        route = tr.call_route(dtype, C, T, d)
        assert (route["kernel"], route["k_slices"]) == (kernel, slices)


# the most rows of C checkpoints that the few-rows kernel takes before the split-k pair does
@pytest.mark.parametrize("dtype,C,d,b,most", [(tr.BF16, 1, 5120, 128, 96), (tr.F16, 2, 5376, 128, 48), (tr.BF16, 3, 6144, 128, 32), (tr.BF16, 8, 6144, 64, 32), (tr.BF16, 4, 5120, 64, 48), (tr.F32, 4, 2560, 64, 48),
                                              (tr.F32, 1, 2560, 128, 96), (tr.F32, 2, 3072, 128, 64), (tr.F32, 3, 2688, 128, 32), (tr.F32, 8, 3072, 64, 32), (tr.BF16, 1, 8192, 128, 16),
                                              (tr.F32, 2, 4096, 128, 16)])
def test_the_line_between_few_rows_and_the_pair(dtype, C, d, b, most):
    assert tr.call_route(dtype, C, most, d, b)["kernel"] == tr.ROUTE_FEW_ROWS
    assert tr.call_route(dtype, C, most + 1, d, b)["kernel"] == SPLITK


def test_raw_weights_on_few_rows_fit_the_fixed_array():
    """The latency kernel on raw weights keeps partial results of d / 512 slices: its largest call fits where d / 128 would not."""
    shape = (tr.BF16, 32, 8, 16384, 256)
    need = state_bytes(8) + 32 * 32 * 8 * (256 + 4) * 4
    assert tr.workspace_bytes(*shape, raw_weights=True) == need
    route = tr.call_route(*shape, raw_weights=True, block_bytes=tr.noalloc_scratch_bytes())
    assert route["kernel"] == tr.ROUTE_LATENCY and route["scratch_bytes"] == need
    assert tr.call_route(*shape, raw_weights=True, block_bytes=need)["kernel"] == tr.ROUTE_LATENCY
    assert refused(*shape, raw_weights=True, block_bytes=need - 256)
