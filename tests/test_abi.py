"""The C boundary: libplc.so loads without a GPU, exports every symbol that
include/plc.h declares, and rejects bad arguments on the host before anything
is enqueued.  No compute call is made here."""
import ctypes as C
import os
import re

import pytest

from paper_2604_15356_amd import plc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "plc.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(plc_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = _declared()
    assert set(names) == set(plc.EXPORTS)
    lib = plc.lib()
    for name in names:
        assert getattr(lib, name) is not None


def test_host_only_calls():
    assert plc.plc_version() >= 100
    assert plc.strerror(plc.PLC_OK) == "ok"
    for code in (1, 2, 3, 4, 99):
        assert plc.strerror(code)
    assert plc.plc_units_per_stream(1000, 0) == 1
    assert plc.plc_units_per_stream(1000, 32) == 32
    assert plc.plc_units_per_stream(1024, 512) == 2
    dm = plc.make_dims(1, 32, 8, 4096, 8, 128, 0.02)
    ws = plc.plc_workspace_bytes(dm)
    tiles = 32 * 8 * (2 * 4096 * 128 // 2048)
    assert ws >= 4096 * 8 * 4 + 2 * 4 * tiles and ws % 256 == 0


def test_one_kernel_or_two_calls():
    one = plc.plc_decode_one_kernel
    assert one(256, 1 << 20, 0, 8) and one(5120, 1 << 17, 0, 4) and not one(256, 1 << 20, 4096, 8)
    assert not one(256, 1 << 20, 0, 9) and not one(256, 1001, 0, 4)
    assert one(512, 1 << 16, 0, 8, cond=True, per_depth=True) and not one(513, 1 << 16, 0, 8, cond=True, per_depth=True)
    assert one(2048, 1 << 16, 0, 8, cond=True) and not one(2049, 1 << 16, 0, 8, cond=True)
    # in pieces: long ones, and more rounds of them than one, are for two calls
    points = lambda streams, n: plc.plc_restart_points(streams, n, 0)
    assert one(8, 1 << 16, 0, 4, per_stream=points(8, 1 << 16))
    assert one(1024, 1 << 13, 0, 4, cond=True, per_stream=points(1024, 1 << 13))
    assert not one(256, 1 << 20, 0, 8, per_stream=points(256, 1 << 20))
    assert not one(300, 1 << 16, 0, 5, per_stream=points(300, 1 << 16))
    assert not one(8, 1 << 16, 0, 4, cond=True, per_depth=True, per_stream=points(8, 1 << 16))
    assert not one(1025, 1 << 16, 0, 4, per_stream=8) and not one(8, 1 << 16, 0, 4, per_stream=1)


@pytest.mark.parametrize("field,value", [("k", 0), ("k", 33), ("d", 12), ("d", 0), ("n", 0), ("S", 0),
                                         ("delta", 0.0), ("delta", -1.0), ("delta", float("nan")),
                                         ("qmax", 0), ("qmax", 128)])
def test_invalid_dims_are_rejected(field, value):
    dm = plc.make_dims(1, 2, 2, 16, 4, 64, 0.02)
    setattr(dm, field, value)
    assert plc.plc_workspace_bytes(dm) == 0
    p = C.c_void_p(4096)
    rc = plc.lib().plc_predict_residual(C.byref(dm), p, p, p, p, p, p, p, 0, p, p, None, p, 1 << 20, p, None)
    assert rc == plc.PLC_ERR_INVALID
    rc = plc.lib().plc_reconstruct(C.byref(dm), p, p, p, p, p, 0, p, p, p, p, 1 << 20, p, None)
    assert rc == plc.PLC_ERR_INVALID


def test_bad_strides_pointers_and_sizes_are_rejected():
    L = plc.lib()
    p = C.c_void_p(4096)
    dm = plc.make_dims(1, 2, 2, 16, 4, 64, 0.02)
    dm.cand_stride[3] = 4 * 64 + 4          # rows not 16-byte aligned
    assert L.plc_predict_residual(C.byref(dm), p, p, p, p, p, p, p, 0, p, p, None, p, 1 << 20, p, None) == 1
    dm = plc.make_dims(1, 2, 2, 16, 4, 64, 0.02)
    odd = C.c_void_p(4098)
    assert L.plc_predict_residual(C.byref(dm), odd, p, p, p, p, p, p, 0, p, p, None, p, 1 << 20, p, None) == 1
    assert L.plc_predict_residual(C.byref(dm), p, p, p, p, p, p, p, 0, p, p, None, p, 16, p, None) == 1   # ws too small
    assert L.plc_predict_residual(C.byref(dm), None, p, p, p, p, p, p, 0, p, p, None, p, 1 << 20, p, None) == 1
    # byte-stream calls
    assert L.plc_histogram(p, 0, 10, p, None) == 1
    assert L.plc_histogram(p, 1, 0, p, None) == 1
    assert L.plc_histogram(None, 1, 10, p, None) == 1
    assert L.plc_build_freq(p, 0, p, p, p, None) == 1
    assert L.plc_rans_encode(p, 1, 100, 48, p, p, p, p, 100, p, p, None) == 1      # chunk not a multiple of 32
    assert L.plc_rans_encode(p, 1, 100, -32, p, p, p, p, 100, p, p, None) == 1
    assert L.plc_rans_decode(p, p, p, 10, p, p, 1, 0, 0, p, p, None) == 1
    assert L.plc_rans_decode(p, p, p, 10, p, p, 1, 1 << 31, 0, p, p, None) == 1
    # the single decode call: its own checks, and those of the two calls it stands for
    dm = plc.make_dims(1, 2, 2, 16, 4, 64, 0.02)
    dec = L.plc_rans_decode_reconstruct
    assert dec(C.byref(dm), p, p, p, 10, p, p, 0, odd, p, p, p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    assert dec(C.byref(dm), p, p, p, 10, p, p, 0, p, p, p, p, 0, p, p, p, odd, p, 1 << 20, p, None) == 1
    assert dec(C.byref(dm), p, p, p, 10, p, p, 0, p, p, p, p, 0, p, p, p, p, p, 16, p, None) == 1       # ws too small
    assert dec(C.byref(dm), p, p, p, 10, p, p, 0, p, p, p, C.c_void_p(4097), 8, p, p, p, p, p, 1 << 20, p, None) == 1
    assert dec(C.byref(dm), p, p, p, 10, p, p, 48, p, p, p, p, 0, p, p, p, p, p, 1 << 20, p, None) == 1  # chunk not a multiple of 32
    assert dec(C.byref(dm), None, p, p, 10, p, p, 0, p, p, p, p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    bad = plc.make_dims(1, 2, 2, 16, 0, 64, 0.02)
    assert dec(C.byref(bad), p, p, p, 10, p, p, 0, p, p, p, p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    decc = L.plc_rans_decode_reconstruct_cond
    assert decc(C.byref(dm), p, p, p, 10, p, p, 0, p, p, p, None, p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    assert decc(C.byref(dm), p, p, p, 10, p, p, 0, p, p, p, C.c_void_p(4098), p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    assert decc(C.byref(dm), p, p, p, 10, p, p, 0, p, p, p, p, p, 0, p, p, p, odd, p, 1 << 20, p, None) == 1
    assert decc(C.byref(dm), p, None, p, 10, p, p, 0, p, p, p, p, p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    deca = L.plc_rans_decode_reconstruct_adapt
    r03 = C.c_float(0.3)
    assert deca(C.byref(dm), p, p, p, 10, p, p, 0, 4, p, p, p, p, None, r03, p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    assert deca(C.byref(dm), p, p, p, 10, p, p, 0, 4, p, p, p, p, p, C.c_float(0.0), p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    assert deca(C.byref(dm), p, p, p, 10, p, p, 0, 5, p, p, p, p, p, r03, p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    assert deca(C.byref(dm), p, p, p, 10, p, p, 0, 4, p, p, p, None, p, r03, p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    assert deca(C.byref(dm), p, p, p, 10, p, p, 0, 4, odd, p, p, p, p, r03, p, 0, p, p, p, p, p, 1 << 20, p, None) == 1
    # token-conditional calls
    dm = plc.make_dims(1, 2, 2, 16, 4, 64, 0.02)
    odd4 = C.c_void_p(4098)
    assert L.plc_predict_residual_cond(C.byref(dm), p, p, p, None, p, p, p, p, 0, p, p, None, p, 1 << 20, p, None) == 1
    assert L.plc_predict_residual_cond(C.byref(dm), p, p, p, odd4, p, p, p, p, 0, p, p, None, p, 1 << 20, p, None) == 1
    assert L.plc_reconstruct_cond(C.byref(dm), p, p, p, None, p, p, 0, p, p, p, p, 1 << 20, p, None) == 1
    assert L.plc_reconstruct_cond(C.byref(dm), p, p, p, p, p, p, 0, p, p, p, p, 16, p, None) == 1       # ws too small
    assert L.plc_select_candidate(C.byref(dm), p, p, C.c_float(-1.0), p, None) == 1
    assert L.plc_select_candidate(C.byref(dm), p, p, C.c_float(float("nan")), p, None) == 1
    assert L.plc_select_candidate(C.byref(dm), p, None, C.c_float(1.0), p, None) == 1
    assert L.plc_index_encode(p, p, 1, 16, 0, p, p, p, 16, p, p, None) == 1        # k out of range
    assert L.plc_index_encode(p, p, 1, 16, 33, p, p, p, 16, p, p, None) == 1
    assert L.plc_index_encode(p, p, 0, 16, 4, p, p, p, 16, p, p, None) == 1
    assert L.plc_index_encode(p, None, 1, 16, 4, p, p, p, 16, p, p, None) == 1
    assert L.plc_index_decode(p, p, None, 10, p, p, 1, 16, 4, p, p, None) == 1
    assert L.plc_index_decode(p, p, p, 10, p, p, 1, 0, 4, p, p, None) == 1
    # surprisal-adaptive calls
    thr = (C.c_uint16 * 5)(0, 0, 1000, 500, 250)
    up = (C.c_uint16 * 5)(0, 0, 100, 500, 250)                # thresholds must not increase
    assert L.plc_surprisal_bits(p, p, 1, 16, 4, up, 4, p, p, None) == 1
    assert L.plc_surprisal_bits(p, p, 1, 16, 4, thr, 5, p, p, None) == 1        # bmax beyond PLC_MAX_BITS
    assert L.plc_surprisal_bits(p, None, 1, 16, 4, thr, 4, p, p, None) == 1
    f0, fneg = C.c_float(0.0), C.c_float(-1.0)
    assert L.plc_predict_residual_adapt(C.byref(dm), p, p, p, p, p, f0, p, p, p, p, 0, p, p, None, p, 1 << 20, p, None) == 1
    assert L.plc_predict_residual_adapt(C.byref(dm), p, p, p, p, None, C.c_float(0.3), p, p, p, p, 0, p, p, None, p, 1 << 20, p, None) == 1
    assert L.plc_reconstruct_adapt(C.byref(dm), p, p, p, p, p, fneg, p, p, 0, p, p, p, p, 1 << 20, p, None) == 1
    assert L.plc_histogram_bucketed(p, 2, 1024, 48, 1, p, 4, p, p, None) == 1   # positions must hold a multiple of 32
    assert L.plc_histogram_bucketed(p, 2, 1000, 64, 1, p, 4, p, p, None) == 1   # and divide the stream
    assert L.plc_histogram_bucketed(p, 2, 1024, 64, 1, p, 5, p, p, None) == 1
    assert L.plc_build_freq_bucketed(p, 2, 0, p, p, None) == 1
    assert L.plc_rans_encode_bucketed(p, 1, 1024, 0, 64, 1, None, 4, p, p, p, p, 100, p, p, None) == 1
    assert L.plc_rans_encode_bucketed(p, 1, 1024, 0, 16, 1, p, 4, p, p, p, p, 100, p, p, None) == 1
    assert L.plc_rans_decode_bucketed(p, p, p, 10, p, p, 1, 1024, 48, 64, 1, p, 4, p, p, None) == 1
    # linear-embedding predictor: whole tiles only, 16-byte aligned operands
    assert L.plc_expected_embedding(p, p, 100, 64, 128, p, None) == 1            # rows not a multiple of 128
    assert L.plc_expected_embedding(p, p, 128, 50, 128, p, None) == 1            # vocabulary not a multiple of 32
    assert L.plc_expected_embedding(p, p, 128, 64, 96, p, None) == 1             # embedding dim not a multiple of 128
    assert L.plc_expected_embedding(C.c_void_p(4104), p, 128, 64, 128, p, None) == 1
    lin = plc.make_dims(1, 2, 2, 128, 1, 32, 0.02)
    lin.n = 100                                                                   # positions not a multiple of 128
    assert L.plc_predict_residual_linear(C.byref(lin), p, 128, p, p, p, p, p, p, p, 0, p, p, p, 1 << 20, p, None) == 1
    lin = plc.make_dims(1, 2, 1, 128, 1, 32, 0.02)                                # 2*H*d = 64: not a whole tile
    assert L.plc_reconstruct_linear(C.byref(lin), p, 128, p, p, p, p, p, 0, p, p, p, p, 1 << 20, p, None) == 1
    lin = plc.make_dims(1, 2, 2, 128, 1, 32, 0.02)
    assert L.plc_reconstruct_linear(C.byref(lin), p, 100, p, p, p, p, p, 0, p, p, p, p, 1 << 20, p, None) == 1
    # null pointers anywhere, a missing status word or a workspace that is too small: refused on the host,
    # before the contraction is enqueued
    pl, rl = L.plc_predict_residual_linear, L.plc_reconstruct_linear
    assert L.plc_expected_embedding(None, p, 128, 64, 128, p, None) == 1
    assert L.plc_expected_embedding(p, None, 128, 64, 128, p, None) == 1
    assert L.plc_expected_embedding(p, p, 128, 64, 128, None, None) == 1
    big = 1 << 24
    for hole in range(1, 15):
        if hole in (2, 10, 14):                 # m, esc_cap, ws_bytes: not pointers
            continue
        args = [C.byref(lin), p, 128, p, p, p, p, p, p, p, 0, p, p, p, big, p]
        args[hole] = None
        want = 0 if hole == 9 else 1             # an empty escape list needs no storage
        if want:
            assert pl(*args, None) == 1, hole
    assert pl(C.byref(lin), p, 128, p, p, p, p, p, p, p, 0, p, p, p, big, None, None) == 1      # no status word
    assert pl(C.byref(lin), p, 128, p, p, p, p, p, p, p, 0, p, p, p, 16, p, None) == 1          # workspace too small
    assert pl(C.byref(lin), p, 128, p, p, p, p, p, p, None, 8, p, p, p, big, p, None) == 1      # list without storage
    for hole in (1, 3, 4, 5, 6, 9, 10, 11, 12):
        args = [C.byref(lin), p, 128, p, p, p, p, p, 0, p, p, p, p, big, p]
        args[hole] = None
        assert rl(*args, None) == 1, hole
    assert rl(C.byref(lin), p, 128, p, p, p, p, p, 0, p, p, p, p, big, None, None) == 1
    assert rl(C.byref(lin), p, 128, p, p, p, p, p, 0, p, p, p, p, 16, p, None) == 1
    assert rl(C.byref(lin), p, 128, p, p, p, p, None, 8, p, p, p, p, big, p, None) == 1
    # thresholds of the adaptive quantiser (host call)
    out = (C.c_uint16 * 5)()
    assert L.plc_surprisal_thresholds(3.0, 3.9, 4, out) == 0 and list(out)[:2] == [0, 0]
    assert L.plc_surprisal_thresholds(0.0, 3.9, 4, out) == 1
    assert L.plc_surprisal_thresholds(3.0, float("nan"), 4, out) == 1
    assert L.plc_surprisal_thresholds(3.0, 3.9, 5, out) == 1                     # beyond PLC_MAX_BITS
    assert L.plc_surprisal_thresholds(3.0, 3.9, 4, None) == 1


def test_noalloc_entry_point_refuses_shapes_beyond_its_static_buffer():
    """Host-side refusals of plc_predict_residual_noalloc come before any GPU call."""
    L = plc.lib()
    p = C.c_void_p(4096)
    long_ctx = plc.make_dims(1, 32, 8, 32768, 4, 128, 0.02)
    assert plc.plc_workspace_bytes(long_ctx) > plc.STATIC_SCRATCH_BYTES
    assert L.plc_predict_residual_noalloc(C.byref(long_ctx), p, p, p, p, p, p, p, 0, p, p, None, p, None) == plc.PLC_ERR_SCRATCH
    bad = plc.make_dims(1, 2, 2, 16, 0, 64, 0.02)
    assert L.plc_predict_residual_noalloc(C.byref(bad), p, p, p, p, p, p, p, 0, p, p, None, p, None) == plc.PLC_ERR_INVALID
    assert plc.strerror(plc.PLC_ERR_SCRATCH) != plc.strerror(99)
    llama = plc.make_dims(1, 32, 8, 4096, 8, 128, 0.02)
    assert plc.plc_workspace_bytes(llama) <= plc.STATIC_SCRATCH_BYTES


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    monkeypatch.setattr(plc, "_lib", None)
    monkeypatch.setattr(plc, "LIB_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(RuntimeError, match="no fallback"):
        plc.lib()
