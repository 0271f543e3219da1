"""The C-ABI library loads and exports every symbol include/lbscan.h declares;
host-side validation paths that need no GPU."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2506_15976_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2506_15976_amd import build
        build.build(force=True, verbose=False)
    return binding.load()


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "lbscan.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(lbscan_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    from paper_2506_15976_amd import binding
    names = _declared_functions()
    assert set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_struct_layout_matches_header():
    from paper_2506_15976_amd.binding import LbscanArgs
    # 8 int32 + 9 pointers + (workspace pointer, size_t) + (saved_state pointer, size_t)
    # + h0, hT + 4 int32 (scan order)
    assert ctypes.sizeof(LbscanArgs) == 8 * 4 + 10 * 8 + 8 + 16 + 16 + 16
    assert LbscanArgs.scan_order.offset == 32 + 15 * 8
    assert LbscanArgs.x.offset == 32
    from paper_2506_15976_amd.binding import LbscanConvArgs
    # 7 int32 (padded to 32 bytes) + 4 pointers
    assert ctypes.sizeof(LbscanConvArgs) == 32 + 4 * 8
    assert LbscanConvArgs.x.offset == 32
    assert LbscanArgs.workspace_bytes.offset == 32 + 10 * 8
    assert LbscanArgs.saved_state.offset == 32 + 11 * 8


def test_default_window_rule(lib):
    # Sec. 4, first paragraph: L > 256 -> 16; 128 < L <= 256 -> 8; L <= 128 -> 4
    f = lib.lbscan_default_window
    assert [f(64), f(128), f(129), f(197), f(256), f(257), f(4096)] == [4, 4, 8, 8, 8, 16, 16]


def test_validation_without_gpu(lib):
    from paper_2506_15976_amd.binding import LbscanArgs, EINVAL, EUNSUPPORTED, EWORKSPACE, OK
    a = LbscanArgs()
    a.batch, a.dim, a.dstate, a.seqlen, a.window = 1, 4, 16, 8, 0
    assert lib.lbscan_fwd(ctypes.byref(a), None) == EINVAL          # window < 1
    a.window = 4
    assert lib.lbscan_fwd(ctypes.byref(a), None) == EINVAL          # null x
    a.dtype = 7
    assert lib.lbscan_fwd(ctypes.byref(a), None) == EUNSUPPORTED
    a.dtype = 0
    a.dstate = 17
    assert lib.lbscan_fwd(ctypes.byref(a), None) == EUNSUPPORTED
    a.dstate = 16
    a.seqlen = 0
    assert lib.lbscan_fwd(ctypes.byref(a), None) == OK              # empty: nothing to do
    assert lib.lbscan_fwd(None, None) == EINVAL
    a.seqlen = 64
    a.window = 3
    a.x = a.delta = a.y = a.A = a.Bm = a.Cm = 256                   # never dereferenced on the host
    # every window length has a backward pass: with no workspace given the call stops
    # at the workspace check, not at the window
    fake = ctypes.c_void_p(256)
    for window in (3, 17, 100):
        a.window = window
        assert lib.lbscan_bwd(ctypes.byref(a), *([fake] * 9), None) == EWORKSPACE
    # a state size of zero with steps to take has no kernel (and must not reach one)
    a.dstate, a.window = 0, 4
    assert lib.lbscan_fwd(ctypes.byref(a), None) == EUNSUPPORTED
    assert lib.lbscan_bwd(ctypes.byref(a), *([fake] * 9), None) == EUNSUPPORTED
    assert lib.lbscan_bidir_fwd(ctypes.byref(a), ctypes.byref(a), None) == EUNSUPPORTED
    a.dstate = 16
    a.x = 257
    a.window = 4
    assert lib.lbscan_fwd(ctypes.byref(a), None) == EINVAL          # misaligned pointer
    assert lib.lbscan_strerror(EINVAL) == b"invalid argument"
    assert lib.lbscan_version().startswith(b"0.")


def test_workspace_sizes(lib):
    from paper_2506_15976_amd.binding import LbscanArgs, WS_BIDIR, WS_FWD
    a = LbscanArgs()
    a.batch, a.dim, a.dstate, a.seqlen, a.window = 2, 8, 16, 10, 4
    assert lib.lbscan_workspace_bytes(ctypes.byref(a), WS_FWD) == 0
    assert lib.lbscan_workspace_bytes(ctypes.byref(a), WS_BIDIR) == 0
    a.dtype = 1
    assert lib.lbscan_workspace_bytes(ctypes.byref(a), WS_BIDIR) == 2 * 8 * 10 * 4


def test_workspace_sizes_follow_the_launch_plan(lib):
    """Host logic only: scratch sizes for uncut rows, rows cut into segments, window
    lengths without a fused kernel, and the saved-state buffer."""
    from paper_2506_15976_amd.binding import LbscanArgs, WS_BWD, WS_FWD, WS_SAVED
    B, D, N, L = 2, 128, 16, 200
    a = LbscanArgs()
    a.batch, a.dim, a.dstate, a.seqlen, a.window = B, D, N, L, 4
    ws = lambda which: lib.lbscan_workspace_bytes(ctypes.byref(a), which)
    rows, tiles16, nbx = B * D, (L + 15) // 16, (D + 63) // 64
    part = 2 * nbx * B * N * L          # fp32 dBm, dCm per block of 64 channels
    try:
        assert lib.lbscan_set_option(b"segments", 1) == 0
        assert ws(WS_FWD) == 0
        assert ws(WS_SAVED) == tiles16 * rows * N * 4
        assert ws(WS_BWD) == (tiles16 * rows * (N + 1) + part) * 4              # checkpoints + dt sums + partials
        a.dtype = 1                                                            # bf16: the same (fp32 scratch)
        assert ws(WS_BWD) == (tiles16 * rows * (N + 1) + part) * 4
        a.window = 8                                                           # run-time window masks, tiles aligned
        assert ws(WS_BWD) == (tiles16 * rows * (N + 1) + part) * 4
        a.window = 3                                                           # no fused forward kernel
        assert ws(WS_FWD) == rows * L * 4                                      # fp32 first-pass result
        assert ws(WS_SAVED) == 0
        # windows straddle tile starts: checkpoints of the local adjoint as well
        assert ws(WS_BWD) == (tiles16 * rows * (2 * N + 1) + part) * 4
        a.window = 17
        assert ws(WS_BWD) == (tiles16 * rows * (2 * N + 1) + part) * 4
        a.window = 1000                                                        # one window: as window = L
        assert ws(WS_BWD) == (tiles16 * rows * (2 * N + 1) + part) * 4
        a.dtype, a.window = 0, 4
        assert lib.lbscan_set_option(b"segments", 3) == 0                      # 7 tiles of 32 -> 3 + 3 + 1
        assert ws(WS_FWD) == 3 * rows * (N + 1) * 4
        assert ws(WS_SAVED) == 0
        assert ws(WS_BWD) == (tiles16 * rows * (N + 1) + 3 * rows * (2 * N + 1) + part) * 4
        a.window = 3                          # segments of whole windows: 3 tiles of 32 hold 32 windows
        assert ws(WS_BWD) == (tiles16 * rows * (2 * N + 1) + 3 * rows * (2 * N + 1) + part) * 4
        a.window = 5                          # 5 tiles of 32 per segment: 7 tiles -> 2 segments
        assert ws(WS_BWD) == (tiles16 * rows * (2 * N + 1) + 2 * rows * (2 * N + 1) + part) * 4
    finally:
        assert lib.lbscan_set_option(b"segments", 0) == 0
    assert lib.lbscan_set_option(b"segments", -1) != 0
    assert lib.lbscan_set_option(b"waves_log2", 4) != 0
    assert lib.lbscan_set_option(b"waves_log2", 2) == 0 and lib.lbscan_set_option(b"waves_log2", -1) == 0
    assert lib.lbscan_set_option(b"mapping", 3) != 0 and lib.lbscan_set_option(b"mapping", -1) != 0
    assert lib.lbscan_set_option(b"mapping", 2) == 0 and lib.lbscan_set_option(b"mapping", 0) == 0
    assert lib.lbscan_set_option(b"no_such_option", 0) != 0
    assert lib.lbscan_set_option(None, 0) != 0


def test_header_is_plain_c(tmp_path):
    """include/lbscan.h compiles as C99 on its own (no C++ or framework types)."""
    import subprocess
    src = tmp_path / "use_header.c"
    src.write_text('#include "lbscan.h"\n'
                   'int main(void) { lbscan_args a; lbscan_conv_args c; (void)a; (void)c;\n'
                   '  return sizeof(a) == 0 || sizeof(c) == 0; }\n')
    subprocess.run(["gcc", "-std=c99", "-Wall", "-Werror", "-pedantic", "-fsyntax-only",
                    "-I", os.path.join(ROOT, "include"), str(src)], check=True)
