"""CPU-side checks of the boundary: the shared library loads, exports every symbol the
header declares, and rejects bad arguments before anything is enqueued (no GPU needed:
none of these calls reaches a kernel launch)."""
import ctypes
import os
import re

import numpy as np
import pytest

from conftest import ROOT, read_golden
from paper_2603_21365_amd import stats
from paper_2603_21365_amd import tide_route as tr

HEADER = os.path.join(ROOT, "include", "tide_route.h")


def declared_symbols():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(tide_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = tr.load_library()
    names = declared_symbols()
    assert set(names) == set(tr.EXPORTS), (names, tr.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None
    assert tr.version() >= 100
    assert tr.last_error() == "" or isinstance(tr.last_error(), str)


def test_packed_size_query():
    assert tr.packed_router_bytes(tr.BF16, 4096) == 4096 * 128 * 2
    assert tr.packed_router_bytes(tr.F32, 768) == 768 * 128 * 4
    # any hidden size up to 16384: packed with zero rows up to the next multiple of 128 (the generic fallback)
    assert tr.packed_router_bytes(tr.F16, 100) == 128 * 128 * 2
    assert tr.packed_router_bytes(tr.F32, 333) == 384 * 128 * 4 and tr.packed_router_bytes(tr.BF16, 1001, 256) == 1024 * 256 * 2
    assert tr.packed_router_bytes(tr.F16, 0) == 0 and tr.packed_router_bytes(tr.F16, 16385) == 0
    assert tr.packed_router_bytes(7, 4096) == 0
    # width 64 is stored padded to 128 columns, width 256 as two 128-column halves (Table 2's widths)
    assert tr.packed_router_bytes(tr.BF16, 2048, 64) == 2048 * 128 * 2
    assert tr.packed_router_bytes(tr.BF16, 8192, 256) == 8192 * 256 * 2
    assert tr.packed_router_bytes(tr.BF16, 4096, 96) == 0 and tr.packed_router_bytes(tr.BF16, 4096, 512) == 0


FAKE = 0x10000  # never dereferenced: every call below fails its checks first


def _eval(lib, hidden=FAKE, dtype=2, T=4, d=256, rs=256, W1=FAKE, w2=FAKE, eps=1e-6, b=128):
    return lib.tide_router_eval(hidden, dtype, T, d, b, rs, None, eps, W1, None, w2, 0.0, 0.5, None, None, None, None)


def test_router_eval_rejects_bad_arguments():
    lib = tr.load_library()
    assert _eval(lib, dtype=5) == -1 and "dtype" in tr.last_error()
    assert _eval(lib, T=-1) == -1
    assert _eval(lib, d=0) == -1
    assert _eval(lib, d=32768, rs=32768) == -2 and "16384" in tr.last_error()
    assert _eval(lib, b=96) == -2 and "bottleneck" in tr.last_error()
    assert _eval(lib, b=0) == -2 and _eval(lib, b=512) == -2
    assert _eval(lib, rs=128) == -1
    assert _eval(lib, hidden=None) == -1
    assert _eval(lib, W1=None) == -1
    assert _eval(lib, w2=None) == -1
    assert _eval(lib, eps=-1.0) == -1
    assert _eval(lib, eps=float("nan")) == -1
    assert _eval(lib, hidden=FAKE + 2) == -3
    assert _eval(lib, hidden=FAKE + 1, d=100, rs=100) == -3 and "element" in tr.last_error()   # rows that cannot be chunk-aligned: elements must be
    assert _eval(lib, rs=260) == -3            # 260 bf16 = 520 bytes: not a multiple of 16
    assert _eval(lib, T=0, hidden=None, W1=None, w2=None) == 0   # empty input: successful no-op


def test_select_exit_rejects_bad_arguments():
    lib = tr.load_library()
    def call(C=2, T=4, d=256, ids=(3, 7), b2=(0, 0), th=(.5, .5), exit_ptr=FAKE, cs=1024, hidden=FAKE, b=128):
        b2a, tha = np.asarray(b2, np.float32), np.asarray(th, np.float32)
        ida = np.asarray(ids, np.int32) if ids is not None else None
        p = lambda a: a.ctypes.data_as(ctypes.c_void_p) if a is not None else None
        return lib.tide_select_exit(hidden, 2, C, T, d, b, cs, d, None, 1e-6, FAKE, None, FAKE, p(b2a), p(tha),
                                    p(ida), 0, 32, exit_ptr, None, None, None)

    assert call(ids=(7, 3)) == -1 and "ascending" in tr.last_error()
    assert call(ids=(3, 3)) == -1
    assert call(ids=None) == -1
    assert call(C=0, ids=(), b2=(), th=()) == -1
    assert call(C=33, ids=tuple(range(33)), b2=(0,) * 33, th=(.5,) * 33) == -2
    assert call(exit_ptr=None) == -1
    assert call(b=100) == -2
    assert call(cs=1028) == -3
    assert call(T=0, hidden=None) == 0


def test_exit_project_rejects_bad_arguments():
    lib = tr.load_library()
    ids = np.asarray([3, 7], np.int32)
    idp = ids.ctypes.data_as(ctypes.c_void_p)

    def call(T=4, d=256, out=FAKE, out_rs=256, ex=FAKE, fin=None, fin_rs=0, ids_p=idp):
        return lib.tide_exit_project(FAKE, 2, 2, T, d, 1024, 256, fin, fin_rs, ex, ids_p, None, 1e-6, out, out_rs, None)

    assert call(out=None) == -1
    assert call(ex=None) == -1
    assert call(ids_p=None) == -1
    assert call(out_rs=128) == -1
    assert call(fin=FAKE, fin_rs=100) == -1
    assert call(out=FAKE + 4) == -3
    assert call(d=100, out_rs=100) == -2
    bad = np.asarray([7, 3], np.int32)
    assert call(ids_p=bad.ctypes.data_as(ctypes.c_void_p)) == -1
    assert call(T=0) == 0


def test_cosine_labels_rejects_bad_arguments():
    lib = tr.load_library()
    call = lambda T=4, d=256, fin=FAKE, frs=256, dtype=2: lib.tide_cosine_labels(FAKE, dtype, 2, T, d, 1024, 256, fin, frs, 0.98,
                                                                                  None, None, None)
    assert call(fin=None) == -1 and call(frs=128) == -1 and call(dtype=9) == -1
    assert call(fin=FAKE + 8) == -3 and call(d=100, frs=100) == -2 and call(T=0) == 0


def test_batch_compact_rejects_bad_arguments():
    lib = tr.load_library()
    call = lambda ex=FAKE, T=4, e=FAKE, c=FAKE, n=FAKE: lib.tide_batch_compact(ex, T, 7, e, c, n, None)
    assert call(n=None) == -1 and call(ex=None) == -1 and call(e=None) == -1 and call(c=None) == -1 and call(T=-2) == -1


def test_batch_exit_rejects_bad_arguments():
    lib = tr.load_library()
    ids = np.asarray([3, 7], np.int32).ctypes.data_as(ctypes.c_void_p)
    call = lambda fm=FAKE, T=4, C=2, idp=ids, outp=FAKE: lib.tide_batch_exit(fm, T, C, idp, 0, 8, outp, None, None, None)
    assert call(fm=None) == -1 and call(outp=None) == -1 and call(idp=None) == -1
    assert call(C=0) == -1 and call(C=33) == -1 and call(T=-1) == -1
    bad = np.asarray([7, 3], np.int32)
    assert call(idp=bad.ctypes.data_as(ctypes.c_void_p)) == -1
    assert call(T=0, fm=None, outp=None) == 0


def test_set_variant_validates():
    prev = tr.set_variant(tr.VARIANT_AUTO)
    assert prev in (0, 1, 2)
    with pytest.raises(tr.TideError):
        tr.set_variant(9)
    tr.set_variant(prev)


def test_set_prefill_form_validates():
    prev = tr.set_prefill_form(0)
    assert prev & 0xff in (0, 1, 2, 3, 4, 5, 6, 7, 8, 9)
    with pytest.raises(tr.TideError):
        tr.set_prefill_form(10)
    # forms 5 and 8 may carry a forced split-k shape (rows << 8 | slices << 16); no other form may, and only the shapes that exist
    # (the single-launch form 8 has 32-row tiles)
    word = tr.splitk_form(64, 4)
    assert word == 5 | 64 << 8 | 4 << 16
    assert tr.set_prefill_form(word) == 0
    assert tr.set_prefill_form(0) == word
    assert tr.set_prefill_form(8 | 32 << 8 | 4 << 16) == 0
    assert tr.set_prefill_form(0) == 8 | 32 << 8 | 4 << 16
    for bad in (2 | 64 << 8, 5 | 48 << 8, 5 | 16 << 16, 5 | 1 << 24, 8 | 64 << 8, 9 | 2 << 16, -1):
        with pytest.raises(tr.TideError):
            tr.set_prefill_form(bad)
    assert tr.set_prefill_form(prev) == 0


def test_mfma_probe_validates_its_arguments():
    lib = tr.load_library()
    out = (ctypes.c_double * 4)()
    for waves, iters, launches, outp in ((3, 16, 1, out), (4, 0, 1, out), (4, 16, 0, out), (8, 1 << 21, 1, out), (4, 16, 1001, out), (4, 16, 1, None)):
        assert lib.tide_mfma_probe(waves, iters, launches, 0, outp) == -1, (waves, iters, launches)
        assert "tide_mfma_probe" in tr.last_error()


def test_exit_statistics_reproduce_fig3(golden_dir):
    g = read_golden(os.path.join(golden_dir, "fig3_exit_example.txt"))
    ex = [int(x) for x in g["exit_layers"]]
    used, full, saved = stats.layer_ops(ex, int(g["n_layers"][0]))
    assert (used, full) == (int(g["layer_ops"][0]), int(g["layer_ops_full"][0]))
    assert round(100 * saved) == int(g["reduction_percent_rounded"][0])
    hist = stats.exit_histogram(ex, [int(x) for x in g["router_layers"]], int(g["n_layers"][0]))
    assert hist == {"L8": 1, "L16": 1, "none": 1}
    assert stats.exit_rate(ex, 32) == pytest.approx(2 / 3)


def test_workspace_size_query():
    """Host arithmetic of tide_workspace_bytes: state words (a counter block + 8 bytes per token), the packed
    weights of a raw-weight prefill call, the partial results of the split-k pair / the latency kernel."""
    # one 128-row tile per CU (the 8B-shaped prefill): state only
    assert tr.workspace_bytes(tr.BF16, 8, 4096, 4096) == 256 + 4096 * 8
    # the same call on raw weights packs 8 routers inside the call
    assert tr.workspace_bytes(tr.BF16, 8, 4096, 4096, raw_weights=True) == 256 + 4096 * 8 + 8 * tr.packed_router_bytes(tr.BF16, 4096)
    # a decode step on packed weights: split-k pair, 32-row tiles x 8 slices -> 16.5 KiB per workgroup
    assert tr.workspace_bytes(tr.F16, 8, 8, 4096) == 256 + 256 + 8 * 8 * (32 * 128 + 4 * 32) * 4
    # ... on raw weights: the latency kernel, d/512 slices of 128 + 4 floats per row
    assert tr.workspace_bytes(tr.F16, 8, 1, 4096, raw_weights=True) == 256 + 256 + 8 * 8 * 1 * 132 * 4
    # (five blocks of 128: two slices, of three and of two)
    assert tr.workspace_bytes(tr.F16, 8, 1, 640, raw_weights=True) == 256 + 256 + 8 * 2 * 1 * 132 * 4
    # multiples of 256, monotone in T for a fixed path, zero for unsupported shapes
    for T in (1, 33, 500, 4096, 16384):
        assert tr.workspace_bytes(tr.BF16, 9, T, 4096) % 256 == 0
    assert tr.workspace_bytes(tr.BF16, 8, 4096, 20000) == 0 and "unsupported" in tr.last_error()
    # the generic fallback's aligned copy of the rows: C x T x (d rounded up to 128) elements
    assert tr.workspace_bytes(tr.F16, 2, 4096, 100) >= 2 * 4096 * 128 * 2
    assert tr.workspace_bytes(tr.BF16, 2, 4096, 200, 256) >= 2 * 4096 * 256 * 2 and tr.workspace_bytes(tr.BF16, 2, 4096, 200, 128) < 4096 * 256
    assert tr.workspace_bytes(tr.BF16, 0, 4096, 4096) == 0 and tr.workspace_bytes(9, 8, 64, 4096) == 0
    assert tr.noalloc_scratch_bytes() == 32 << 20


def test_ws_entry_points_reject_bad_arguments():
    lib = tr.load_library()
    b2a, tha, ida = np.zeros(2, np.float32), np.full(2, .5, np.float32), np.asarray([3, 7], np.int32)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)

    def sel(W1=None, packed=FAKE, gamma=None, ws=0x20000, ws_bytes=1 << 20, exit_ptr=FAKE, T=4):
        return lib.tide_select_exit_ws(FAKE, 2, 2, T, 256, 128, 1024, 256, gamma, 1e-6, W1, packed, None, FAKE, p(b2a), p(tha),
                                       p(ida), 0, 32, exit_ptr, None, None, ws, ws_bytes, None)

    def ev(W1=None, packed=FAKE, gamma=None, ws=0x20000, ws_bytes=1 << 20, T=4, rs=256):
        return lib.tide_router_eval_ws(FAKE, 2, T, 256, 128, rs, gamma, 1e-6, W1, packed, None, FAKE, 0.0, 0.5, None, None, None,
                                       ws, ws_bytes, None)

    for call in (sel, ev):
        assert call(W1=FAKE, packed=FAKE) == -1 and "exactly one" in tr.last_error()
        assert call(W1=None, packed=None) == -1
        assert call(gamma=FAKE) == -1 and "gamma" in tr.last_error()
        assert call(ws=None) == -1 and call(ws_bytes=0) == -1
        assert call(ws=0x20010) == -3 and "256" in tr.last_error()
    assert sel(exit_ptr=None) == -1
    assert ev(rs=128) == -1
    # parameter arrays are read with 16-byte loads
    assert lib.tide_router_eval(FAKE, 2, 4, 256, 128, 256, None, 1e-6, FAKE + 4, None, FAKE, 0.0, 0.5, None, None, None, None) == -3
    assert lib.tide_router_eval(FAKE, 2, 4, 256, 128, 256, None, 1e-6, FAKE, None, FAKE + 8, 0.0, 0.5, None, None, None, None) == -3
    assert lib.tide_router_eval(FAKE, 2, 4, 256, 128, 256, FAKE + 2, 1e-6, FAKE, None, FAKE, 0.0, 0.5, None, None, None, None) == -3
    assert lib.tide_router_eval(FAKE, 2, 4, 256, 128, 256, None, 1e-6, FAKE, FAKE + 12, FAKE, 0.0, 0.5, None, None, None, None) == -3
    # workspace registration
    assert lib.tide_workspace_init(None, 4096, None) == -1
    assert lib.tide_workspace_init(0x20000, 100, None) == -1
    assert lib.tide_workspace_init(0x20010, 4096, None) == -3
    assert lib.tide_workspace_forget(0x30000) == -1
