"""C-ABI contract checks that need no GPU.

The library loads without a device, exports every function include/resonator.h
declares, and rejects bad arguments with the documented status before it makes
any HIP call (so these error paths run on the CPU).
"""
import ctypes
import os
import re

import pytest

from paper_2607_05583_amd import _lib as L

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    src = open(os.path.join(ROOT, "include", "resonator.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(resonator_\w+)\s*\(", src)))


def test_header_symbols_exported():
    lib = L.lib()
    names = header_functions()
    assert set(names) == set(L.SYMBOLS)
    for n in names:
        assert hasattr(lib, n), n


def test_version_and_workspace_sizes():
    lib = L.lib()
    assert lib.resonator_version() >= 100
    ws = lib.resonator_workspace_bytes
    assert ws(L.RES_OP_FWD, L.RES_BF16, 4, 32768, 256, 8) > 0
    assert ws(L.RES_OP_BWD, L.RES_F32, 2, 100, 7, 3) > 0
    assert ws(L.RES_OP_STATE_INIT, L.RES_BF16, 2, 0, 7, 3) == 0      # empty prompt needs none
    assert ws(L.RES_OP_FWD, L.RES_F32, 1, 100, 7, 17) == 0           # M > M_MAX
    assert ws(9, L.RES_F32, 1, 100, 7, 3) == 0                        # bad op
    assert ws(L.RES_OP_FWD, 7, 1, 100, 7, 3) == 0                     # bad dtype
    # workspace grows with the problem
    assert ws(L.RES_OP_FWD, L.RES_F32, 2, 4096, 64, 8) > ws(L.RES_OP_FWD, L.RES_F32, 1, 4096, 64, 8)


def test_forward_workspaces_keep_the_counters_apart():
    """A forward with more than 8 modes leaves the first 256 bytes (status), the
    1 MiB of chain counters and the 2 MiB of tagged states (256 work-groups of
    8 KiB) to the calls with at most 8 modes that share its workspace."""
    ws = L.lib().resonator_workspace_bytes
    for M in (9, 16):
        assert ws(L.RES_OP_FWD, L.RES_F32, 1, 16, 4, M) > 256 + (1 << 20) + (2 << 20)
    assert ws(L.RES_OP_FWD, L.RES_BF16, 70000, 16, 64, 8) > 256 + (1 << 20) + (2 << 20)  # beyond 65536 chains


FAKE = ctypes.c_void_p(0x7F0000000000)      # never dereferenced: validation fails first
FAKE2 = ctypes.c_void_p(0x7F0100000000)


def _fwd(**kw):
    a = dict(x=FAKE, xdt=L.RES_F32, y=FAKE2, ydt=L.RES_F32, B=1, Ln=16, D=4, M=2,
             g=FAKE, w=FAKE, amp=FAKE, ph=FAKE, h0=None, hout=None, ws=None, wsb=0, st=None)
    a.update(kw)
    return L.lib().resonator_mix_fwd(a["x"], a["xdt"], a["y"], a["ydt"], a["B"], a["Ln"], a["D"],
                                     a["M"], a["g"], a["w"], a["amp"], a["ph"], a["h0"], a["hout"],
                                     a["ws"], a["wsb"], a["st"])


def _err():
    return L.lib().resonator_last_error().decode()


def test_fwd_validation_codes():
    assert _fwd(B=0) == L.RES_ERR_INVALID_ARG and "B and D" in _err()
    assert _fwd(Ln=0) == L.RES_ERR_INVALID_ARG
    assert _fwd(M=0) == L.RES_ERR_INVALID_ARG
    assert _fwd(M=17) == L.RES_ERR_UNSUPPORTED
    assert _fwd(xdt=L.RES_F32, ydt=L.RES_BF16) == L.RES_ERR_UNSUPPORTED
    assert _fwd(xdt=5) == L.RES_ERR_INVALID_ARG
    assert _fwd(x=None) == L.RES_ERR_INVALID_ARG
    assert _fwd(g=None) == L.RES_ERR_INVALID_ARG
    assert _fwd(g=ctypes.c_void_p(0x7F0000000002)) == L.RES_ERR_MISALIGNED
    assert _fwd(x=ctypes.c_void_p(0x7F0000000002)) == L.RES_ERR_MISALIGNED
    assert _fwd(y=FAKE) == L.RES_ERR_INVALID_ARG and "overlap" in _err()
    assert _fwd() == L.RES_ERR_WORKSPACE and "workspace" in _err()
    need = L.lib().resonator_workspace_bytes(L.RES_OP_FWD, L.RES_F32, 1, 16, 4, 2)
    assert _fwd(ws=ctypes.c_void_p(0x7F0200000010), wsb=need) == L.RES_ERR_MISALIGNED


def test_workspace_init_and_sizes_validation_codes():
    lib = L.lib()
    init = lambda dt=L.RES_F32, B=1, Ln=16, D=4, M=2, ws=None, wsb=0: lib.resonator_fwd_workspace_init(
        dt, B, Ln, D, M, ws, wsb, None)
    need = lambda *a: lib.resonator_workspace_bytes(*a)
    n = need(L.RES_OP_FWD, L.RES_F32, 1, 16, 4, 2)
    assert init(B=0) == L.RES_ERR_INVALID_ARG
    assert init(Ln=0) == L.RES_ERR_INVALID_ARG
    assert init(M=17) == L.RES_ERR_UNSUPPORTED
    assert init(dt=5) == L.RES_ERR_INVALID_ARG
    assert init() == L.RES_ERR_WORKSPACE
    assert init(ws=FAKE, wsb=n - 1) == L.RES_ERR_WORKSPACE
    assert init(ws=ctypes.c_void_p(0x7F0200000010), wsb=n) == L.RES_ERR_MISALIGNED
    # prompt state: one record (complex float64 per channel of the block and mode of
    # whole groups of 8) per tile, and per work-group where there are more tiles
    assert need(L.RES_OP_STATE_INIT, L.RES_BF16, 2, 300, 65, 3) == 2 * 2 * 2 * 64 * 8 * 16
    assert need(L.RES_OP_STATE_INIT, L.RES_F32, 4, 1 << 20, 64, 16) == 256 * 32 * 16 * 16


def test_bwd_state_decode_validation_codes():
    lib = L.lib()
    rc = lib.resonator_mix_bwd(FAKE, FAKE2, L.RES_F32, FAKE, 1, 16, 4, 2, FAKE, FAKE, FAKE, FAKE,
                               None, FAKE, FAKE, FAKE, FAKE, None, None, 0, None)
    assert rc == L.RES_ERR_INVALID_ARG and "overlap" in _err()
    rc = lib.resonator_mix_bwd(FAKE, FAKE2, L.RES_F32, ctypes.c_void_p(0x7F0300000000), 1, 16, 4, 2,
                               FAKE, FAKE, FAKE, FAKE, None, None, FAKE, FAKE, FAKE, None, None, 0, None)
    assert rc == L.RES_ERR_INVALID_ARG
    rc = lib.resonator_mix_bwd(FAKE, FAKE2, L.RES_F32, ctypes.c_void_p(0x7F0300000000), 1, 16, 4, 2,
                               FAKE, FAKE, FAKE, FAKE, None, FAKE, FAKE, FAKE, FAKE, None, None, 0, None)
    assert rc == L.RES_ERR_WORKSPACE
    rc = lib.resonator_state_init(None, L.RES_BF16, 1, 5, 4, 2, FAKE, FAKE, FAKE, FAKE, FAKE2, None, 0, None)
    assert rc == L.RES_ERR_INVALID_ARG and "x_prompt" in _err()
    rc = lib.resonator_state_init(FAKE, L.RES_BF16, 1, -1, 4, 2, FAKE, FAKE, FAKE, FAKE, FAKE2, None, 0, None)
    assert rc == L.RES_ERR_INVALID_ARG
    rc = lib.resonator_decode_step(FAKE, L.RES_BF16, FAKE, L.RES_BF16, 2, 4, 2, FAKE, FAKE, FAKE, FAKE,
                                   FAKE2, None)
    assert rc == L.RES_ERR_INVALID_ARG and "overlap" in _err()
    rc = lib.resonator_decode_step(FAKE, L.RES_BF16, FAKE2, L.RES_BF16, 2, 4, 2, FAKE, FAKE, FAKE, FAKE,
                                   ctypes.c_void_p(0x7F0300000004), None)
    assert rc == L.RES_ERR_MISALIGNED
    rc = lib.resonator_decode_step(FAKE, L.RES_F32, FAKE2, L.RES_BF16, 2, 4, 2, FAKE, FAKE, FAKE, FAKE,
                                   ctypes.c_void_p(0x7F0300000000), None)
    assert rc == L.RES_ERR_UNSUPPORTED


def test_product_path_has_no_fallback(monkeypatch, tmp_path):
    """A missing library raises; nothing silently computes elsewhere."""
    monkeypatch.setattr(L, "_lib", None)
    monkeypatch.setattr(L, "LIB_PATH", str(tmp_path / "missing.so"))
    with pytest.raises(RuntimeError, match="not built"):
        L.lib()


F3 = ctypes.c_void_p(0x7F0200000000)
F4 = ctypes.c_void_p(0x7F0300000000)
ODD = ctypes.c_void_p(0x7F0400000002)   # not 4-byte aligned


def test_decode_steps_and_projection_validation_codes():
    lib = L.lib()
    ds = lib.resonator_decode_steps
    assert ds(None, L.RES_BF16, FAKE2, L.RES_BF16, 2, 3, 4, 2, FAKE, FAKE, FAKE, FAKE, F3, None) == \
        L.RES_ERR_INVALID_ARG
    assert ds(FAKE, L.RES_F32, FAKE2, L.RES_BF16, 2, 3, 4, 2, FAKE, FAKE, FAKE, FAKE, F3, None) == \
        L.RES_ERR_UNSUPPORTED
    assert ds(FAKE, L.RES_BF16, FAKE, L.RES_BF16, 2, 3, 4, 2, FAKE, FAKE, FAKE, FAKE, F3, None) == \
        L.RES_ERR_INVALID_ARG and "overlap" in _err()
    gl = lib.resonator_grouped_linear
    assert gl(FAKE, FAKE2, L.RES_F32, F3, 5, 8, 8, 3, None) == L.RES_ERR_INVALID_ARG and "multiples" in _err()
    assert gl(FAKE, FAKE2, L.RES_F32, F3, 0, 8, 8, 2, None) == L.RES_ERR_INVALID_ARG
    assert gl(FAKE, FAKE2, 7, F3, 5, 8, 8, 2, None) == L.RES_ERR_INVALID_ARG
    assert gl(FAKE, FAKE2, L.RES_F32, FAKE, 5, 8, 8, 2, None) == L.RES_ERR_INVALID_ARG and "overlap" in _err()
    assert gl(ODD, FAKE2, L.RES_F32, F3, 5, 8, 8, 2, None) == L.RES_ERR_MISALIGNED
    gl2 = lib.resonator_grouped_linear2
    F4_ = ctypes.c_void_p(0x7F0300000000)
    assert gl2(FAKE, FAKE2, FAKE2, L.RES_F32, F3, F4_, 5, 8, 8, 3, None) == L.RES_ERR_INVALID_ARG and \
        "multiples" in _err()
    assert gl2(FAKE, None, FAKE2, L.RES_F32, F3, F4_, 5, 8, 8, 2, None) == L.RES_ERR_INVALID_ARG
    assert gl2(FAKE, FAKE2, FAKE2, L.RES_F32, F3, F3, 5, 8, 8, 2, None) == L.RES_ERR_INVALID_ARG and \
        "overlap" in _err()
    assert gl2(FAKE, FAKE2, FAKE2, L.RES_F32, FAKE, F4_, 5, 8, 8, 2, None) == L.RES_ERR_INVALID_ARG and \
        "overlap" in _err()
    assert gl2(ODD, FAKE2, FAKE2, L.RES_F32, F3, F4_, 5, 8, 8, 2, None) == L.RES_ERR_MISALIGNED
    assert lib.resonator_grouped_linear_bwd_data(None, FAKE2, L.RES_F32, F3, 5, 8, 8, 2, 0, None) == \
        L.RES_ERR_INVALID_ARG
    wgs = lib.resonator_grouped_linear_bwd_weight_sum
    I3 = ctypes.c_int * 3
    P3_ = ctypes.c_void_p * 3
    F5 = ctypes.c_void_p(0x7F0500000000)
    assert lib.resonator_grouped_linear_bwd_weight_sum_workspace_bytes(3, 2, 131072, 256, 256, 8, L.RES_BF16) == \
        256 * 64 * 1024
    assert lib.resonator_grouped_linear_bwd_weight_sum_workspace_bytes(1, 1, 1000, 256, 256, 8, L.RES_F32) == 0
    assert wgs(1, FAKE, P3_(FAKE2, FAKE2, FAKE2), I3(2, 0, 0), L.RES_BF16, F3, F5, 5, 64, 64, 2, 0, None, 0, None) == \
        L.RES_ERR_INVALID_ARG and "out[0]" in _err()
    assert wgs(1, FAKE, P3_(FAKE2, FAKE2, FAKE2), I3(1, 0, 0), L.RES_BF16, F3, F5, 5, 64, 64, 2, 0, None, 0, None) == \
        L.RES_ERR_INVALID_ARG and "dW0" in _err()
    assert wgs(2, FAKE, P3_(FAKE2, FAKE2, FAKE2), I3(0, 1, 0), L.RES_BF16, F3, None, 5, 64, 64, 2, 0, None, 0,
               None) == L.RES_ERR_INVALID_ARG and "dW1" in _err()
    assert wgs(2, FAKE, P3_(FAKE2, FAKE2, FAKE2), I3(0, 1, 0), L.RES_BF16, F3, F3, 5, 64, 64, 2, 0, None, 0,
               None) == L.RES_ERR_INVALID_ARG and "overlap" in _err()
    assert wgs(1, FAKE, P3_(FAKE2, FAKE2, FAKE2), I3(0, 0, 0), L.RES_BF16, F3, None, 5, 64, 64, 2, 0, None, 0,
               None) == L.RES_ERR_INVALID_ARG and "workspace" in _err()
    dg_ = lib.resonator_diagnostics
    assert dg_(FAKE, FAKE, FAKE, FAKE, 0, 4, 16, F3, None, None, None) == L.RES_ERR_INVALID_ARG
    assert dg_(FAKE, None, FAKE, FAKE, 8, 4, 16, None, None, F3, None) == L.RES_ERR_INVALID_ARG and \
        "spectrum" in _err()
    assert dg_(FAKE, FAKE, FAKE, FAKE, 8, 4, 0, None, F3, None, None) == L.RES_ERR_INVALID_ARG and "T must" in _err()
    assert dg_(FAKE, FAKE, FAKE, FAKE, 8, 4, 16, FAKE, None, None, None) == L.RES_ERR_INVALID_ARG and \
        "overlap" in _err()
    dgs = lib.resonator_grouped_linear_bwd_data_sum
    P3 = ctypes.c_void_p * 3
    assert dgs(4, P3(FAKE, FAKE, FAKE), P3(FAKE2, FAKE2, FAKE2), L.RES_F32, F3, 5, 8, 8, 2, 0, None) == \
        L.RES_ERR_INVALID_ARG and "n must be" in _err()
    assert dgs(2, P3(FAKE, None, FAKE), P3(FAKE2, FAKE2, FAKE2), L.RES_F32, F3, 5, 8, 8, 2, 0, None) == \
        L.RES_ERR_INVALID_ARG and "dy[1]" in _err()
    assert dgs(2, P3(FAKE, F3, FAKE), P3(FAKE2, FAKE2, FAKE2), L.RES_F32, F3, 5, 8, 8, 2, 0, None) == \
        L.RES_ERR_INVALID_ARG and "overlap" in _err()
    assert dgs(1, P3(ODD, FAKE, FAKE), P3(FAKE2, FAKE2, FAKE2), L.RES_F32, F3, 5, 8, 8, 2, 0, None) == \
        L.RES_ERR_MISALIGNED
    assert lib.resonator_grouped_linear_bwd_weight(FAKE, FAKE2, L.RES_BF16, FAKE, 5, 8, 8, 2, 0, None) == \
        L.RES_ERR_INVALID_ARG and "overlap" in _err()
    bd = lib.resonator_block_diag_weight
    assert bd(FAKE, L.RES_F32, 8, 8, 0, FAKE2, None) == L.RES_ERR_INVALID_ARG
    assert bd(FAKE, L.RES_F32, 8, 8, 2, FAKE, None) == L.RES_ERR_INVALID_ARG and "overlap" in _err()
    assert lib.resonator_grouped_linear_bwd_weight_split_workspace_bytes(0, 8, 8) == 0
    assert lib.resonator_grouped_linear_bwd_weight_split_workspace_bytes(131072, 256, 256) == 64 * 256 * 256 * 4
    ws_ = lib.resonator_grouped_linear_bwd_weight_split
    assert ws_(FAKE, FAKE2, L.RES_F32, F3, 1000, 8, 8, 2, 0, None, 0, None) == L.RES_ERR_WORKSPACE
    assert ws_(FAKE, FAKE2, L.RES_F32, FAKE, 1000, 8, 8, 2, 0, F4, 1 << 20, None) == L.RES_ERR_INVALID_ARG
    be = lib.resonator_block_diag_extract
    assert be(FAKE, 8, 6, 4, FAKE2, 0, None) == L.RES_ERR_INVALID_ARG
    assert be(FAKE, 8, 8, 2, FAKE, 0, None) == L.RES_ERR_INVALID_ARG and "overlap" in _err()
    assert be(ODD, 8, 8, 2, FAKE2, 1, None) == L.RES_ERR_MISALIGNED


def test_reference_params_and_epilogue_validation_codes():
    lib = L.lib()
    assert lib.resonator_quadratic_reference_workspace_bytes(0, 4) == 0
    qr = lib.resonator_quadratic_reference
    assert qr(None, FAKE2, 1, 16, 4, 2, FAKE, FAKE, FAKE, FAKE, F3, 1 << 20, None) == L.RES_ERR_INVALID_ARG
    assert qr(FAKE, FAKE2, 1, 16, 4, 2, FAKE, FAKE, FAKE, FAKE, F3, 8, None) == L.RES_ERR_WORKSPACE
    # the FFT reference rejects sizes before it makes any plan (no HIP call)
    assert lib.resonator_fft_reference_workspace_bytes(0, 16, 4) == 0
    assert lib.resonator_fft_reference_workspace_bytes(1, (1 << 26) + 1, 4) == 0
    fr = lib.resonator_fft_reference
    assert fr(None, FAKE2, 1, 16, 4, 2, FAKE, FAKE, FAKE, FAKE, F3, 1 << 20, None) == L.RES_ERR_INVALID_ARG
    assert fr(FAKE, FAKE2, 70000, 16, 4, 2, FAKE, FAKE, FAKE, FAKE, F3, 1 << 20, None) == L.RES_ERR_UNSUPPORTED
    pm = lib.resonator_params_map
    assert pm(FAKE, FAKE2, 0, 1e-4, F3, F4, None) == L.RES_ERR_INVALID_ARG
    assert pm(FAKE, FAKE2, 8, float("nan"), F3, F4, None) == L.RES_ERR_INVALID_ARG
    assert pm(FAKE, FAKE2, 8, 1e-4, F3, F3, None) == L.RES_ERR_INVALID_ARG and "overlap" in _err()
    assert pm(FAKE, FAKE2, 8, 1e-4, ODD, F4, None) == L.RES_ERR_MISALIGNED
    pi = lib.resonator_params_init
    assert pi(0, 2, 2.0, 2048.0, 4.0, 2048.0, 1e-4, FAKE, FAKE2, None) == L.RES_ERR_INVALID_ARG
    assert pi(4, 2, 100.0, 2.0, 4.0, 2048.0, 1e-4, FAKE, FAKE2, None) == L.RES_ERR_INVALID_ARG
    assert pi(4, 2, 2.0, 2048.0, 1.0, 2048.0, 1e-4, FAKE, FAKE2, None) == L.RES_ERR_INVALID_ARG
    # ln 2 / 1e5 is below alpha_min = 1e-4: the longest half-life cannot be reached
    assert pi(4, 2, 2.0, 1e5, 4.0, 2048.0, 1e-4, FAKE, FAKE2, None) == L.RES_ERR_INVALID_ARG and "half-life" in _err()
    ef = lib.resonator_epilogue_fwd
    assert ef(FAKE, FAKE2, F3, L.RES_BF16, F4, 1, 16, 0, 8, 2, FAKE, 0.5, FAKE, FAKE, None) == L.RES_ERR_INVALID_ARG
    assert ef(FAKE, FAKE2, None, L.RES_BF16, F4, 1, 16, 2, 8, 2, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_INVALID_ARG
    assert ef(FAKE, FAKE2, F3, L.RES_BF16, FAKE, 1, 16, 2, 8, 2, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_INVALID_ARG and "overlap" in _err()
    assert ef(FAKE, FAKE2, F3, L.RES_BF16, F4, 1, 16, 2, 8, 1000, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_UNSUPPORTED
    epf = lib.resonator_epilogue_proj_fwd
    W5 = ctypes.c_void_p(0x7F0400000000)
    # y, gate, v, dt, Wo, out, z, B, L, H, dh, K, d_out, Ct, lambda_c, w, s, stream
    assert epf(FAKE, FAKE2, F3, L.RES_BF16, W5, F4, None, 1, 16, 16, 32, 4, 512, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_UNSUPPORTED  # more than eight heads
    assert epf(FAKE, FAKE2, F3, L.RES_BF16, W5, F4, None, 1, 16, 8, 16, 4, 256, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_UNSUPPORTED  # a bf16 head of 16 channels
    assert epf(FAKE, FAKE2, F3, L.RES_F32, W5, F4, None, 1, 16, 8, 16, 4, 512, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_UNSUPPORTED  # 64 outputs per head
    assert epf(FAKE, FAKE2, F3, L.RES_BF16, W5, F4, None, 1, 16, 8, 32, 4, 100, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_INVALID_ARG  # d_out not a multiple of H
    assert epf(FAKE, FAKE2, F3, L.RES_BF16, W5, FAKE, None, 1, 16, 8, 32, 4, 256, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_INVALID_ARG and "overlap" in _err()
    assert epf(ODD, FAKE2, F3, L.RES_BF16, W5, F4, None, 1, 16, 8, 32, 4, 256, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_MISALIGNED
    assert epf(FAKE, FAKE2, None, L.RES_BF16, W5, F4, None, 1, 16, 8, 32, 4, 256, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_INVALID_ARG
    assert epf(FAKE, FAKE2, F3, L.RES_BF16, W5, F4, FAKE2, 1, 16, 8, 32, 4, 256, FAKE, 0.5, FAKE, FAKE, None) == \
        L.RES_ERR_INVALID_ARG and "z must not overlap" in _err()
