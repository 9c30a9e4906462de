"""libkata on the CPU: the library loads, exports every symbol include/kata.h
declares, and rejects bad arguments on the host before any GPU call."""
import ctypes
import os
import re

import pytest

import paper_2607_17419_amd as kata

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    with open(os.path.join(ROOT, "include", "kata.h")) as f:
        text = f.read()
    return sorted(set(re.findall(r"\b(kata_[a-z_0-9]+)\s*\(", text)))


def test_header_matches_binding():
    assert _declared_symbols() == sorted(kata.EXPORTED)


def test_library_exports_every_symbol():
    L = kata.lib()
    for name in _declared_symbols():
        assert hasattr(L, name), name


def test_status_strings_and_version():
    L = kata.lib()
    assert L.kata_status_string(0) == b"KATA_OK"
    assert L.kata_status_string(1) == b"KATA_ERR_INVALID_ARG"
    assert L.kata_status_string(2) == b"KATA_ERR_UNSUPPORTED"
    assert L.kata_status_string(3) == b"KATA_ERR_HIP"
    assert L.kata_status_string(42) == b"KATA_UNKNOWN_STATUS"
    assert L.kata_abi_version() == 106


FAKE = ctypes.c_void_p(0x10000)  # aligned, never dereferenced: validation fails first
NUL = ctypes.c_void_p(0)


@pytest.mark.parametrize("args,expect", [
    ((NUL, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 0), 1),          # null q
    ((FAKE, FAKE, FAKE, FAKE, 0, 1, 8, 16, 16, 32, 0), 1),         # B < 1
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 0, 16, 16, 32, 0), 1),         # T < 1
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 0, 0), 1),          # C < 1
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 7), 1),         # bad dtype
    ((FAKE, FAKE, FAKE, ctypes.c_void_p(0x10004), 1, 1, 8, 16, 16, 32, 0), 1),  # misaligned
    ((FAKE, FAKE, FAKE, FAKE, 1 << 20, 1 << 20, 1 << 20, 16, 16, 32, 0), 1),  # overflow
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 65, 16, 32, 1), 2),         # d > 64
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 300, 32, 0), 2),        # dv > 256 on fp32 path
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 200, 0), 2),        # C > 128 on fp32 path
])
def test_fwd_rejects_before_gpu(args, expect):
    L = kata.lib()
    st = L.kata_fwd_chunked(*args, NUL)
    assert st == expect


def test_ws_variant_rejects():
    L = kata.lib()
    # workspace too small for a valid bf16 MFMA shape
    need = L.kata_fwd_workspace_bytes(1, 1, 128, 64, 64, 64, 1, 0)
    assert need > 0
    st = L.kata_fwd_chunked_ws(FAKE, FAKE, FAKE, FAKE, 1, 1, 128, 64, 64, 64, 1, 0,
                               ctypes.c_void_p(0x100000), need - 1, NUL)
    assert st == 1
    # misaligned workspace
    st = L.kata_fwd_chunked_ws(FAKE, FAKE, FAKE, FAKE, 1, 1, 128, 64, 64, 64, 1, 0,
                               ctypes.c_void_p(0x100010), need, NUL)
    assert st == 1
    # negative span
    st = L.kata_fwd_chunked_ws(FAKE, FAKE, FAKE, FAKE, 1, 1, 128, 64, 64, 64, 1, -1,
                               ctypes.c_void_p(0x100000), need, NUL)
    assert st == 1


def test_workspace_and_span_host_logic():
    L = kata.lib()
    # fp32 path: one fp32 record (S n x dv, then z n) per chunk and head
    n = 16 * 17 // 2
    assert L.kata_fwd_workspace_bytes(1, 2, 256, 16, 16, 32, 0, 0) == 2 * 8 * (n * 16 + n) * 4
    assert L.kata_fwd_default_span(1, 2, 256, 16, 16, 32, 0) == 1
    # MFMA path: default span folds about 1024 tokens (512 at d = 32)
    assert L.kata_fwd_default_span(1, 16, 131072, 64, 64, 64, 1) == 16
    assert L.kata_fwd_default_span(4, 8, 16384, 32, 64, 128, 1) == 4
    # MFMA path: one bf16 record (2112 slots x 64 dv + 64 x 64 Z) per span and
    # head, scanned in place (the output kernel reads V itself)
    rec = 2112 * 64 + 64 * 64
    NS = 131072 // 1024
    expect = 16 * NS * rec * 2
    assert L.kata_fwd_workspace_bytes(1, 16, 131072, 64, 64, 64, 1, 0) == expect
    # invalid -> 0
    assert L.kata_fwd_workspace_bytes(1, 1, 0, 64, 64, 64, 1, 0) == 0
    assert L.kata_fwd_default_span(1, 1, 8, 65, 64, 64, 1) == 0


@pytest.mark.parametrize("args,expect", [
    ((NUL, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 16, 16, 0), 1),
    ((FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 0, 16, 16, 0), 1),
    ((FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 80, 16, 0), 2),
    ((FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 16, 512, 1), 2),
])
def test_decode_rejects_before_gpu(args, expect):
    assert kata.lib().kata_decode_step(*args, NUL) == expect


@pytest.mark.parametrize("args,expect", [
    ((FAKE, NUL, FAKE, FAKE, 1, 1, 8, 16, 16, 0), 1),
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 0, 16, 16, 0), 1),
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 100, 16, 0), 2),
])
def test_prefill_rejects_before_gpu(args, expect):
    assert kata.lib().kata_prefill_state(*args, NUL) == expect


@pytest.mark.parametrize("args,expect", [
    ((NUL, FAKE, FAKE, FAKE, 1, 1, 8, 64, 64, 1), 1),           # null q
    ((FAKE, FAKE, FAKE, FAKE, 1, 0, 8, 64, 64, 1), 1),          # H < 1
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 64, 64, 5), 1),          # bad dtype
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 64, 64, 0), 2),          # fp32: no quadratic path
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 64, 1), 2),          # d = 16
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 64, 32, 1), 2),          # dv = 32
    ((FAKE, FAKE, FAKE, FAKE, 256, 256, 8, 64, 64, 1), 2),      # B*H above the grid limit
])
def test_quadratic_rejects_before_gpu(args, expect):
    assert kata.lib().kata_fwd_quadratic(*args, NUL) == expect


def test_quadratic_workspace_host_logic():
    L = kata.lib()
    # one permuted bf16 V^T per head: dv rows of T rounded up to 128 keys
    assert L.kata_fwd_quadratic_workspace_bytes(2, 3, 1000, 64, 64, 1) == 6 * 64 * 1024 * 2
    assert L.kata_fwd_quadratic_workspace_bytes(1, 1, 1, 32, 64, 1) == 64 * 128 * 2
    assert L.kata_fwd_quadratic_workspace_bytes(1, 1, 8, 64, 64, 0) == 0
    need = L.kata_fwd_quadratic_workspace_bytes(1, 1, 128, 64, 64, 1)
    st = L.kata_fwd_quadratic_ws(FAKE, FAKE, FAKE, FAKE, 1, 1, 128, 64, 64, 1,
                                 ctypes.c_void_p(0x100000), need - 1, NUL)
    assert st == 1
    st = L.kata_fwd_quadratic_ws(FAKE, FAKE, FAKE, FAKE, 1, 1, 128, 64, 64, 1,
                                 ctypes.c_void_p(0x100040), need, NUL)
    assert st == 1


@pytest.mark.parametrize("g,expect", [(0, 1), (3, 1), (65, 1), (-1, 1)])
def test_mg_rejects_bad_block_count(g, expect):
    L = kata.lib()
    st = L.kata_mg_fwd_chunked(FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 64, 64, 64, g, 1, NUL)
    assert st == expect
    assert L.kata_mg_fwd_workspace_bytes(1, 1, 8, 64, 64, 64, g, 1, 0) == 0
    assert L.kata_mg_decode_step(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 64, 64, g, 1, NUL) == 1


def test_mg_workspace_host_logic():
    L = kata.lib()
    # M2 on the MFMA path: one bf16 record per span and head, S^T over
    # 2 x 544 slots (the rotated layout of each 32-dim block) x 64 dv, then
    # two 32 x 32 Z blocks
    rec = 2 * 544 * 64 + 2 * 32 * 32
    NS = 131072 // 1024
    expect = 16 * NS * rec * 2
    assert L.kata_mg_fwd_workspace_bytes(1, 16, 131072, 64, 64, 64, 2, 1, 0) == expect
    # g = 1 is M1
    assert (L.kata_mg_fwd_workspace_bytes(1, 16, 131072, 64, 64, 64, 1, 1, 0)
            == L.kata_fwd_workspace_bytes(1, 16, 131072, 64, 64, 64, 1, 0))
    # fp32 path with g blocks: n = g m(m+1)/2 per chunk record
    n = 2 * (8 * 9 // 2)
    assert L.kata_mg_fwd_workspace_bytes(1, 2, 256, 16, 16, 32, 2, 0, 0) == 2 * 8 * (n * 16 + n) * 4
    # M4 at d = 64 runs on the fp32 path (no MFMA shape for it)
    n4 = 4 * (16 * 17 // 2)
    assert L.kata_mg_fwd_workspace_bytes(1, 1, 128, 64, 64, 64, 4, 1, 0) == 2 * (n4 * 64 + n4) * 4
    # quadratic M2 exists, M4 does not
    assert L.kata_mg_fwd_quadratic_workspace_bytes(1, 1, 100, 64, 64, 2, 1) == 64 * 128 * 2
    assert L.kata_mg_fwd_quadratic_workspace_bytes(1, 1, 100, 64, 64, 4, 1) == 0


# ---- linear features ----------------------------------------------------------

F_ = ctypes.c_float


@pytest.mark.parametrize("args,expect", [
    ((NUL, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 1, F_(0.0), 1, 0), 1),     # null q
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 0, 16, 16, 32, 1, F_(0.0), 1, 0), 1),    # T < 1
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 5, F_(0.0), 1, 0), 1),    # unknown feature
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, -1, F_(0.0), 1, 0), 1),   # unknown feature
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 1, F_(-1e-3), 1, 0), 1),  # eps < 0
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 1, F_(float("nan")), 1, 0), 1),  # eps NaN
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 1, F_(0.0), 2, 0), 1),    # normalize not 0/1
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 1, F_(0.0), 1, 3), 1),    # bad dtype
    ((FAKE, FAKE, FAKE, ctypes.c_void_p(0x10008), 1, 1, 8, 16, 16, 32, 1, F_(0.0), 1, 0), 1),
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 65, 16, 32, 1, F_(0.0), 1, 0), 2),    # d > 64
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 300, 32, 1, F_(0.0), 1, 0), 2),   # dv > 256
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 200, 1, F_(0.0), 1, 0), 2),   # C > 128, fp32
    ((FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 64, 64, 2048, 0, F_(0.0), 0, 1), 2),  # C > 1024, bf16
])
def test_lin_rejects_before_gpu(args, expect):
    assert kata.lib().kata_lin_fwd_chunked(*args, NUL) == expect


def test_lin_workspace_and_span_host_logic():
    L = kata.lib()
    assert [L.kata_lin_dim(64, f) for f in range(5)] == [64, 64, 64, 65, 64]
    assert L.kata_lin_dim(0, 1) == 0 and L.kata_lin_dim(8, 7) == 0
    # MFMA path (bf16, d = dv = 64, n_psi = d): one fp32 record (S 64 x 64, z 64)
    # per span and head; the default span folds 1024 tokens at T = 131072
    # (128 spans x 16 heads = 2048 workgroups) and shrinks for short sequences
    assert L.kata_lin_default_span(1, 16, 131072, 64, 64, 128, 0, 1) == 8
    assert L.kata_lin_fwd_workspace_bytes(1, 16, 131072, 64, 64, 128, 0, 1, 0) == \
        16 * 128 * (64 * 64 + 64) * 4
    assert L.kata_lin_default_span(1, 16, 2048, 64, 64, 128, 0, 1) == 1
    assert L.kata_lin_default_span(1, 16, 16384, 64, 64, 64, 2, 1) == 4
    # the Lorentz lift (n_psi = d + 1) on the MFMA path: the d x d record, the
    # extra row sum ||k|| v (64), sum ||k|| and three zeros per span
    assert L.kata_lin_default_span(1, 16, 131072, 64, 64, 128, 3, 1) == 8
    assert L.kata_lin_fwd_workspace_bytes(1, 16, 131072, 64, 64, 128, 3, 1, 0) == \
        16 * 128 * (64 * 64 + 64 + 64 + 4) * 4
    # ... and on the fp32 path (C not a multiple of 64): one record per chunk
    assert L.kata_lin_default_span(1, 16, 131072, 64, 64, 96, 3, 1) == 1
    assert L.kata_lin_default_span(1, 16, 131072, 32, 32, 256, 3, 1) == 0  # C > 128 there
    assert L.kata_lin_fwd_workspace_bytes(1, 2, 1000, 64, 64, 100, 3, 1, 0) == \
        2 * 10 * (65 * 64 + 65) * 4
    # fp32 inputs take the fp32 path, whatever the shape
    assert L.kata_lin_default_span(1, 16, 4096, 64, 64, 64, 0, 0) == 1
    assert L.kata_lin_fwd_workspace_bytes(1, 16, 4096, 64, 64, 64, 0, 0, 0) == \
        16 * 64 * (64 * 64 + 64) * 4
    # workspace too small / misaligned / negative span
    need = L.kata_lin_fwd_workspace_bytes(1, 1, 256, 64, 64, 64, 1, 1, 0)
    base = (FAKE, FAKE, FAKE, FAKE, 1, 1, 256, 64, 64, 64, 1, F_(0.01), 1, 1)
    assert L.kata_lin_fwd_chunked_ws(*base, 0, ctypes.c_void_p(0x100000), need - 1, NUL) == 1
    assert L.kata_lin_fwd_chunked_ws(*base, 0, ctypes.c_void_p(0x100080), need, NUL) == 1
    assert L.kata_lin_fwd_chunked_ws(*base, -1, ctypes.c_void_p(0x100000), need, NUL) == 1
    assert L.kata_lin_fwd_chunked_timed(*base, 0, ctypes.c_void_p(0x100000), need, NUL, NUL) == 1


# ---- backward ------------------------------------------------------------------

@pytest.mark.parametrize("args,expect", [
    ((NUL, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 1, 0), 1),  # null q
    ((FAKE, FAKE, FAKE, FAKE, NUL, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 1, 0), 1),  # null dout
    ((FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, NUL, 1, 1, 8, 16, 16, 32, 1, 0), 1),  # null dv
    ((FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 0, 16, 16, 32, 1, 0), 1),  # T < 1
    ((FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 3, 0), 1),  # g !| d
    ((FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 1, 4), 1),  # dtype
    ((FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 65, 1, 0), 2),  # C > 64
    ((FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 80, 16, 32, 1, 0), 2),  # d > 64
    ((FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 16, 300, 32, 1, 0), 2),  # dv > 256
    ((ctypes.c_void_p(0x100002), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 1, 1, 8, 64, 64, 64,
      1, 1), 1),  # bf16 q not 16-byte aligned
    ((FAKE, FAKE, FAKE, FAKE, FAKE, ctypes.c_void_p(0x100008), FAKE, FAKE, 1, 1, 8, 64, 64, 64,
      1, 1), 1),  # dq not 16-byte aligned
])
def test_bwd_rejects_before_gpu(args, expect):
    assert kata.lib().kata_bwd_chunked(*args, NUL) == expect


def test_bwd_fused_scan_host_logic():
    L = kata.lib()
    # bf16 inputs at d = dv = C = 64, g = 1 fuse the state launches with the
    # scans from 16 heads on; every other supported shape keeps both launches
    assert L.kata_bwd_fused_scan(2, 8, 333, 64, 64, 64, 1, 1) == 1
    assert L.kata_bwd_fused_scan(1, 15, 4096, 64, 64, 64, 1, 1) == 0
    assert L.kata_bwd_fused_scan(8, 16, 4096, 64, 64, 64, 1, 0) == 0   # fp32 inputs
    assert L.kata_bwd_fused_scan(8, 16, 4096, 64, 64, 32, 1, 1) == 0   # C = 32
    assert L.kata_bwd_fused_scan(8, 16, 4096, 64, 64, 64, 2, 1) == 0   # g = 2
    assert L.kata_bwd_fused_scan(8, 16, 4096, 64, 64, 65, 1, 1) == -1  # unsupported
    assert L.kata_bwd_fused_scan(8, 16, 4096, 64, 64, 64, 1, 7) == -1  # bad dtype
    assert kata.bwd_fused_scan(8, 16, 4096, 64, 64, 64, 1, kata.KATA_BF16) == 1


def test_forms_host_logic():
    f, b = kata.fwd_form, kata.bwd_form
    F32, BF = kata.KATA_F32, kata.KATA_BF16
    # bf16 forward: quadratic up to a length, where the span is left to the library
    assert f(8, 16, 4096, 64, 64, 64, 1, BF) == kata.FWD_QUADRATIC
    assert f(8, 16, 4096, 64, 64, 64, 1, BF, span_chunks=16) == kata.FWD_STATES
    assert f(1, 2, 6144, 64, 64, 64, 1, BF) == kata.FWD_QUADRATIC
    assert f(1, 2, 6145, 64, 64, 64, 1, BF) == kata.FWD_STATES
    assert f(8, 16, 6144, 64, 64, 64, 1, BF) == kata.FWD_QUADRATIC
    assert f(129, 1, 6144, 64, 64, 64, 1, BF) == kata.FWD_STATES
    assert f(1, 16, 5632, 64, 64, 64, 2, BF) == kata.FWD_QUADRATIC
    assert f(1, 17, 5632, 64, 64, 64, 2, BF) == kata.FWD_STATES
    assert f(1, 1, 8, 65, 64, 64, 1, BF) == f(1, 1, 8, 64, 64, 64, 3, BF) == -1
    assert f(1, 1, 8, 64, 64, 64, 1, BF, span_chunks=-1) == f(1, 1, 8, 64, 64, 64, 1, 5) == -1
    # fp32 forward: widths, heads and chunk size on both sides, whatever the span
    assert f(1, 8, 1000, 64, 64, 64, 1, F32, span_chunks=3) == kata.FWD_QUADRATIC
    assert f(1, 8, 62400, 64, 64, 64, 1, F32) == kata.FWD_QUADRATIC
    assert f(1, 8, 62401, 64, 64, 64, 1, F32) == kata.FWD_STATES
    assert f(1, 8, 16384, 64, 1, 64, 1, F32) == kata.FWD_STATES
    assert f(1, 8, 1024, 4, 4, 64, 1, F32) == kata.FWD_QUADRATIC
    assert f(8, 8, 4096, 4, 4, 64, 1, F32) == kata.FWD_STATES
    assert f(8, 8, 4096, 4, 4, 1, 1, F32) == kata.FWD_QUADRATIC  # one state per token
    assert f(1, 2, 300, 16, 16, 32, 2, F32) == kata.FWD_STATES   # feature blocks
    # 65535 heads of 4200 tokens would be 2^32 threads and more
    assert f(65535, 1, 4200, 64, 64, 64, 1, F32) == kata.FWD_STATES
    # backward
    assert b(8, 16, 4096, 64, 64, 64, 1, BF) == kata.BWD_QUADRATIC
    assert b(1, 16, 8193, 64, 64, 64, 1, BF) == kata.BWD_FUSED_STATES
    assert b(1, 7, 4097, 64, 64, 64, 1, BF) == kata.BWD_STATES
    assert b(1, 2, 300, 64, 64, 32, 2, BF) == kata.BWD_STATES
    assert b(1, 8, 8192, 64, 64, 64, 1, F32) == kata.BWD_QUADRATIC
    assert b(1, 8, 8193, 64, 64, 64, 1, F32) == kata.BWD_STATES
    assert b(1, 8, 1024, 8, 64, 64, 1, F32) == kata.BWD_QUADRATIC
    assert b(1, 8, 4096, 8, 64, 64, 1, F32) == kata.BWD_STATES
    assert b(1, 8, 100, 64, 65, 32, 1, F32) == kata.BWD_STATES   # wide values
    assert b(1, 8, 100, 64, 64, 65, 1, F32) == -1


def test_bwd_workspace_host_logic():
    L = kata.lib()
    # forward and backward records (n dv + n fp32 per chunk) plus (a_t, b_t)
    n = 64 * 65 // 2
    NC = 4096 // 64
    expect = 128 * (2 * NC * (n * 64 + n) + 4096 * 65) * 4
    assert L.kata_bwd_workspace_bytes(8, 16, 4096, 64, 64, 64, 1, 1) == expect
    n2 = 2 * (32 * 33 // 2)
    assert L.kata_bwd_workspace_bytes(1, 1, 100, 64, 64, 50, 2, 0) == \
        (2 * 2 * (n2 * 64 + n2) + 100 * 65) * 4
    assert L.kata_bwd_workspace_bytes(1, 1, 100, 64, 64, 65, 1, 0) == 0
    need = L.kata_bwd_workspace_bytes(1, 1, 128, 16, 16, 32, 1, 0)
    base = (FAKE,) * 8 + (1, 1, 128, 16, 16, 32, 1, 0)
    assert L.kata_bwd_chunked_ws(*base, ctypes.c_void_p(0x100000), need - 1, NUL) == 1
    assert L.kata_bwd_chunked_ws(*base, ctypes.c_void_p(0x100010), need, NUL) == 1
    assert L.kata_bwd_chunked_timed(*base, ctypes.c_void_p(0x100000), need, NUL, NUL) == 1


# Shapes whose workspace (terabytes) no device holds: the allocating entry
# points validate them, fail the stream-ordered allocation and return
# KATA_ERR_HIP before any launch, on a machine with or without a GPU.
HUGE_BH, HUGE_T = 16384, 983040


def huge_alloc_calls(L, ptr):
    F = ptr
    B, H, T = 1, HUGE_BH, HUGE_T
    return [
        ("kata_fwd_chunked", lambda: L.kata_fwd_chunked(F, F, F, F, B, H, T, 64, 64, 64, 1, NUL)),
        ("kata_mg_fwd_chunked",
         lambda: L.kata_mg_fwd_chunked(F, F, F, F, B, H, T, 64, 64, 64, 2, 1, NUL)),
        ("kata_fwd_quadratic",
         lambda: L.kata_fwd_quadratic(F, F, F, F, B, H, T, 64, 64, 1, NUL)),
        ("kata_bwd_chunked",
         lambda: L.kata_bwd_chunked(F, F, F, F, F, F, F, F, B, H, T, 64, 64, 64, 1, 1, NUL)),
    ]


def test_allocation_failure_is_hip_error():
    L = kata.lib()
    assert L.kata_fwd_workspace_bytes(1, HUGE_BH, HUGE_T, 64, 64, 64, 1, 0) > (1 << 40)
    for name, call in huge_alloc_calls(L, FAKE):
        assert call() == 3, name
        # nothing is left behind: a plain validation error reports as such
        assert L.kata_fwd_chunked(NUL, FAKE, FAKE, FAKE, 1, 1, 8, 16, 16, 32, 0, NUL) == 1


def test_train_forward_and_extended_backward_validate_before_gpu():
    L = kata.lib()
    # forward with denominators: den is required
    st = L.kata_fwd_chunked_train_ws(FAKE, FAKE, FAKE, FAKE, NUL, 1, 1, 256, 64, 64, 64, 1, 0,
                                     FAKE, 1 << 30, NUL)
    assert st == 1
    # misaligned den
    st = L.kata_fwd_chunked_train_ws(FAKE, FAKE, FAKE, FAKE, ctypes.c_void_p(0x10004), 1, 1, 256,
                                     64, 64, 64, 1, 0, FAKE, 1 << 30, NUL)
    assert st == 1
    # fp32 inputs take the fp32 path, which writes no denominators
    need = L.kata_fwd_workspace_bytes(1, 2, 256, 16, 16, 32, 0, 0)
    st = L.kata_fwd_chunked_train_ws(FAKE, FAKE, FAKE, FAKE, FAKE, 1, 2, 256, 16, 16, 32, 0, 0,
                                     FAKE, need, NUL)
    assert st == 2
    # backward: misaligned den, and an event array with a null entry
    ws = L.kata_bwd_workspace_bytes(1, 1, 128, 64, 64, 64, 1, 1)
    st = L.kata_bwd_chunked_ex(FAKE, FAKE, FAKE, FAKE, FAKE, ctypes.c_void_p(0x10004), FAKE, FAKE,
                               FAKE, 1, 1, 128, 64, 64, 64, 1, 1, FAKE, ws, NUL, NUL)
    assert st == 1
    events = (ctypes.c_void_p * 7)(*([0x10000] * 6 + [0]))
    st = L.kata_bwd_chunked_ex(FAKE, FAKE, FAKE, FAKE, FAKE, NUL, FAKE, FAKE, FAKE, 1, 1, 128, 64,
                               64, 64, 1, 1, FAKE, ws, events, NUL)
    assert st == 1
