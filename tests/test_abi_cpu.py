"""CPU checks of the C-ABI library: it loads, exports every function the
headers declare, and its host-only logic (validation, chunk planning) works
without a GPU.  No kernel is launched here."""
import ctypes
import glob
import os
import re
import subprocess

import numpy as np
import pytest
from hypothesis import given, settings, strategies as st

import paper_2202_06009_amd as zo
from synth import configs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    names = set()
    for h in glob.glob(os.path.join(ROOT, "include", "*.h")):
        text = re.sub(r"/\*.*?\*/", "", open(h).read(), flags=re.S)
        for m in re.finditer(r"^\s*[A-Za-z_][\w\s\*]*?\b(zo_\w+)\s*\(", text, flags=re.M):
            names.add(m.group(1))
    return names


def test_library_exports_every_declared_function():
    declared = header_functions()
    assert {"zo_adam_init", "zo_local_step", "zo_compress_pack_ef", "zo_unpack_average",
            "zo_sync_update", "zo_variance_update"} <= declared
    out = subprocess.run(["nm", "-D", "--defined-only", zo.LIB_PATH], capture_output=True,
                         text=True, check=True).stdout
    exported = {l.split()[-1] for l in out.splitlines() if " T " in l}
    missing = declared - exported
    assert not missing, missing
    assert declared == set(zo.EXPORTS)
    lib = zo.lib()
    for name in declared:
        assert hasattr(lib, name)


def _cfg(**over):
    d = dict(beta1=0.9, beta2=0.999, eps=1e-8, world=4, chunk=2048,
             seg_off=[0, 4096, 8192], tv=[0, 1], tu=[1, 3])
    d.update(over)
    return d


@pytest.mark.parametrize("over,code", [
    ({}, zo.ZO_OK),
    ({"beta1": 1.0}, zo.ZO_EINVAL),
    ({"beta1": -0.1}, zo.ZO_EINVAL),
    ({"beta2": float("nan")}, zo.ZO_EINVAL),
    ({"eps": -1e-8}, zo.ZO_EINVAL),
    ({"eps": float("inf")}, zo.ZO_EINVAL),
    ({"world": 0}, zo.ZO_EINVAL),
    ({"chunk": 0}, zo.ZO_EINVAL),
    ({"chunk": 1}, zo.ZO_OK),
    ({"chunk": 6}, zo.ZO_OK),
    ({"chunk": 16383}, zo.ZO_OK),
    ({"chunk": 16385}, zo.ZO_EINVAL),
    ({"chunk": 16388}, zo.ZO_EINVAL),
    ({"chunk": 16384}, zo.ZO_OK),
    ({"chunk": 4}, zo.ZO_OK),
    ({"seg_off": [0, 4098, 8192]}, zo.ZO_EALIGN),
    ({"seg_off": [4, 8192]}, zo.ZO_EINVAL),
    ({"seg_off": [0, 8192, 4096]}, zo.ZO_EINVAL),
    ({"seg_off": [0, 0, 0]}, zo.ZO_OK),
    ({"tv": [1, 1]}, zo.ZO_EINVAL),
    ({"tu": [3, 1]}, zo.ZO_EINVAL),
    ({"tu": [-1]}, zo.ZO_EINVAL),
    ({"srv_chunk_begin": 1, "srv_chunk_end": 3}, zo.ZO_OK),
    ({"srv_chunk_begin": 3, "srv_chunk_end": 5}, zo.ZO_EINVAL),
    ({"srv_chunk_begin": 2, "srv_chunk_end": 1}, zo.ZO_EINVAL),
    ({"algorithm": "frozen-variance", "tu": []}, zo.ZO_OK),
    ({"algorithm": "frozen-variance"}, zo.ZO_EINVAL),            # T_u must be empty
    ({"algorithm": "frozen-variance", "tu": [], "defer_sync_writes": True}, zo.ZO_EINVAL),
])
def test_config_validation(over, code):
    assert zo.zo_config_check(**_cfg(**over)) == code


@pytest.mark.parametrize("name", ["tiny", "bert-base", "resnet50", "gpt2-1.5b"])
def test_chunk_plan_matches_oracle_layout(name):
    """Two independent chunkings of the same segment table agree."""
    import oracle as orc
    wl = configs.get(name)
    start, ln, word, nw = zo.zo_plan_chunks(wl.seg_off, wl.chunk)
    lay = orc.Layout.from_segments(wl.seg_off, wl.chunk)
    np.testing.assert_array_equal(start, lay.cstart)
    np.testing.assert_array_equal(ln, lay.clen)
    np.testing.assert_array_equal(word, lay.cword)
    assert nw == lay.nwords


@settings(max_examples=200, deadline=None)
@given(lens=st.lists(st.integers(0, 3000).map(lambda v: 4 * v), min_size=1, max_size=12),
       chunk=st.integers(1, 16384))
def test_chunk_plan_properties(lens, chunk):
    """Random segment tables (empty segments, ragged tails, any chunk
    length from 1 to 16384): the library's plan equals the oracle's, its
    chunks tile every segment in order without crossing a boundary, and each
    chunk's packed words start where the previous chunk's 64-element words end."""
    import oracle as orc
    seg_off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64).tolist()
    start, ln, word, nw = zo.zo_plan_chunks(seg_off, chunk)
    lay = orc.Layout.from_segments(seg_off, chunk)
    np.testing.assert_array_equal(start, lay.cstart)
    np.testing.assert_array_equal(ln, lay.clen)
    np.testing.assert_array_equal(word, lay.cword)
    assert nw == lay.nwords
    expect = [(a + k, min(chunk, b - a - k)) for a, b in zip(seg_off[:-1], seg_off[1:])
              for k in range(0, b - a, chunk)]
    assert list(zip(start, ln)) == expect
    w = 0
    for s0, l0, w0 in zip(start, ln, word):
        assert w0 == w
        w += (l0 + 63) // 64
    assert nw == w


def test_chunk_plan_counts_match_workload_shapes():
    expect = {"tiny": (512, 0), "bert-base": (26823, 125), "bert-large": (41116, 245),
              "resnet50": (25021, 86), "gpt2-1.5b": (95442, 483)}
    for name, (nch, partial) in expect.items():
        wl = configs.get(name)
        _, ln, _, _ = zo.zo_plan_chunks(wl.seg_off, wl.chunk)
        assert len(ln) == nch
        assert sum(1 for l in ln if l != wl.chunk) == partial


def test_unbuilt_library_raises(monkeypatch, tmp_path):
    monkeypatch.setattr(zo, "_lib", None)
    monkeypatch.setattr(zo, "LIB_PATH", str(tmp_path / "missing.so"))
    with pytest.raises(ImportError):
        zo.lib()


def test_state_calls_reject_null_handle():
    lib = zo.lib()
    assert lib.zo_materialize(None) == zo.ZO_EINVAL
    assert lib.zo_state_location(None, None, None, None) == zo.ZO_EINVAL


def test_config_carries_deferred_writes_flag():
    cfg, keep = zo.make_config(**_cfg(), defer_sync_writes=True)
    assert cfg.defer_sync_writes == 1
    assert zo.zo_config_check(**_cfg(), defer_sync_writes=True) == zo.ZO_OK



def test_diag_stream_validates_before_touching_the_device():
    lib = zo.lib()
    assert lib.zo_diag_stream(None, 1, None, 1, 16, None) == zo.ZO_EINVAL
    arr = (ctypes.c_void_p * 7)()
    assert lib.zo_diag_stream(arr, 7, arr, 1, 16, None) == zo.ZO_EINVAL   # too many reads
    assert lib.zo_diag_stream(arr, 1, arr, 6, 16, None) == zo.ZO_EINVAL   # too many writes
    assert lib.zo_diag_stream(arr, 1, arr, 1, 6, None) == zo.ZO_EINVAL    # n not a multiple of 4
    assert lib.zo_diag_stream(arr, 1, arr, 1, 16, None) == zo.ZO_EINVAL   # null buffers
    # two writers of one array (the pointers are never dereferenced: the
    # call fails validation before anything is launched)
    src = (ctypes.c_void_p * 1)(0x10000)
    dst = (ctypes.c_void_p * 2)(0x20000, 0x20000)
    assert lib.zo_diag_stream(src, 1, dst, 2, 16, None) == zo.ZO_EINVAL


def test_unknown_algorithm_is_rejected():
    cfg, keep = zo.make_config(**_cfg())
    cfg.algorithm = 7
    assert zo.lib().zo_config_check(ctypes.byref(cfg)) == zo.ZO_EINVAL


def test_fullprec_step_rejects_null_handle():
    assert zo.lib().zo_fullprec_step(None, 0, 1e-4, None) == zo.ZO_EINVAL


def test_server_pattern_diagnostic_rejects_null_handle():
    assert zo.lib().zo_diag_server_pattern(None, None) == zo.ZO_EINVAL


class _Slots(ctypes.Structure):
    _fields_ = [("wide", ctypes.c_bool), ("bpc", ctypes.c_int), ("lanes_log2", ctypes.c_int),
                ("magic", ctypes.c_uint32)]


@pytest.mark.parametrize("chunk", [1, 4, 512, 513, 1024, 1025, 2049, 3073, 6145, 10241, 14337,
                                   15361, 16384])
def test_chunk_grid(chunk):
    """The grid of the chunk-mapped kernels: the multiply-high that finds a
    workgroup's chunk is exact up to the largest grid, and a grid beyond what a
    launch holds is refused (a table of short segments with long chunks)."""
    f = getattr(zo.lib(), "_ZN2zo11chunk_slotsEilRNS_5SlotsE")
    f.restype = ctypes.c_int64
    f.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.POINTER(_Slots)]
    most = 2 ** 24 - 1
    g = _Slots()
    assert f(chunk, 0, g) == 0
    assert f(chunk, 1, g) == (-(-chunk // 1024) if g.wide else 1)
    assert g.wide == (chunk > 512)
    per = g.bpc if g.wide else 256 >> g.lanes_log2
    full = most // per if g.wide else most * per
    assert 0 < f(chunk, full, g) <= most
    for nch in (full + 1, 2 ** 28, 2 ** 31 - 1) if g.wide else (full + 1,):
        assert f(chunk, nch, g) == -1, nch
    if g.wide:
        c = np.unique(np.concatenate([np.arange(200), full - np.arange(200),
                                      np.random.default_rng(0).integers(0, full, 10000)]))
        for b in (c * g.bpc, c * g.bpc + g.bpc - 1):
            got = (b.astype(np.uint64) * np.uint64(g.magic)) >> np.uint64(32) if g.magic else b
            assert np.array_equal(got.astype(np.int64), c)
