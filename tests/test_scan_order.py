"""Column-by-column scan order of a 2-D token grid (the vertical scans of the
multi-direction models, paper Sec. 4.5 / Appendix D): the index permutation the tests
use, pinned against a plain reshape/transpose, and the host-side validation."""
import ctypes

import numpy as np
import pytest


@pytest.mark.parametrize("H,W,prefix,suffix", [(14, 14, 0, 1), (14, 14, 1, 0), (3, 5, 0, 0), (5, 3, 2, 3),
                                               (64, 64, 0, 0), (1, 7, 0, 0), (7, 1, 1, 1)])
def test_column_order_is_the_transposed_grid(H, W, prefix, suffix):
    """Scanning the grid column by column visits the stored tokens in the order in
    which the transposed grid stores them."""
    from paper_2506_15976_amd.inputs import column_order
    L = prefix + H * W + suffix
    perm = column_order(L, H, W, prefix)
    stored = np.arange(L)
    want = np.concatenate([stored[:prefix],
                           stored[prefix:prefix + H * W].reshape(H, W).T.reshape(-1),
                           stored[prefix + H * W:]])
    assert np.array_equal(perm, want)
    assert np.array_equal(np.sort(perm), stored)            # a permutation
    # first steps: down the first column
    if H > 1 and W > 1:
        assert perm[prefix] == prefix and perm[prefix + 1] == prefix + W


def test_oracle_on_reordered_sequence_is_the_row_scan_of_the_transposed_grid(oracle):
    """order = columns on an H x W grid equals order = stored on the transposed grid:
    the oracle (which only knows sequence order) applied to the reordered inputs gives,
    put back, what it gives on the transposed grid read row by row."""
    from paper_2506_15976_amd.inputs import column_order, make_inputs
    H, W = 5, 4
    s = make_inputs(1, 3, 4, H * W, seed=11)
    perm = column_order(H * W, H, W)
    keys3 = ("x", "delta", "Bm", "Cm", "z")
    re = {k: (np.ascontiguousarray(v[..., perm]) if k in keys3 else v) for k, v in s.items()
          if k in keys3 + ("A", "Dskip", "delta_bias")}
    out_cols = oracle.fwd(**re, window=4)                    # in scanned order
    def transposed(v):          # the grid of every (.., L) tensor, transposed, stored row by row
        return np.ascontiguousarray(v.reshape(v.shape[:-1] + (H, W)).swapaxes(-1, -2).reshape(v.shape))
    tr = {k: (transposed(s[k]) if k in keys3 else s[k]) for k in re}
    out_tr = oracle.fwd(**tr, window=4)
    assert np.array_equal(out_cols, out_tr)


def test_scan_order_validation(tmp_path):
    from paper_2506_15976_amd import binding
    lib = binding.load()
    a = binding.LbscanArgs()
    a.batch, a.dim, a.dstate, a.seqlen, a.window = 1, 4, 16, 197, 4
    a.x = a.delta = a.y = a.A = a.Bm = a.Cm = 256
    a.scan_order = 7
    assert lib.lbscan_fwd(ctypes.byref(a), None) == binding.EINVAL
    a.scan_order = binding.ORDER_COLUMNS
    a.grid_h, a.grid_w, a.grid_prefix = 14, 14, 2                   # 2 + 196 > 197
    assert lib.lbscan_fwd(ctypes.byref(a), None) == binding.EINVAL
    a.grid_h = 0
    assert lib.lbscan_fwd(ctypes.byref(a), None) == binding.EINVAL
    a.grid_h, a.grid_prefix, a.window = 14, 1, 3                    # two-pass forward path: stored order only
    assert lib.lbscan_fwd(ctypes.byref(a), None) == binding.EUNSUPPORTED
    assert lib.lbscan_bidir_fwd(ctypes.byref(a), ctypes.byref(a), None) == binding.EUNSUPPORTED


@pytest.mark.parametrize("dtype, B, D, L, grid, fwd, bwd", [
    # calls that gather faster than they copy, and their neighbours that do not
    ("fp32", 128, 384, 50, (7, 7), False, False), ("bf16", 128, 384, 50, (7, 7), False, False),
    ("fp32", 1042, 384, 50, (7, 7), False, False),
    ("fp32", 88, 384, 65, (8, 8), False, False), ("bf16", 88, 384, 65, (8, 8), False, True),
    ("fp32", 103, 384, 101, (10, 10), False, True), ("bf16", 516, 384, 101, (10, 10), False, True),
    ("fp32", 72, 384, 145, (12, 12), False, True), ("fp32", 90, 384, 145, (12, 12), True, True),
    ("bf16", 359, 384, 145, (12, 12), False, True),
    ("fp32", 29, 384, 197, (14, 14), True, True), ("bf16", 106, 384, 197, (14, 14), False, True),
    ("bf16", 132, 384, 197, (14, 14), True, True), ("fp32", 128, 768, 197, (14, 14), True, True),
    ("bf16", 30, 384, 257, (16, 16), False, True), ("bf16", 35, 384, 257, (16, 16), True, True),
    ("bf16", 32, 384, 325, (18, 18), True, True), ("bf16", 1, 768, 4096, (64, 64), True, True),
    ("fp32", 119, 384, 197, (2, 98), False, False), ("bf16", 119, 384, 197, (98, 2), False, True),
    ("fp32", 40, 384, 197, (65, 3), False, True), ("fp32", 119, 384, 197, (65, 3), True, True),
    ("fp32", 8, 384, 1025, (4, 256), False, True), ("bf16", 30, 384, 1025, (4, 256), True, True),
    ("bf16", 8, 384, 1025, (8, 128), False, True), ("bf16", 11, 384, 1025, (8, 128), True, True),
    ("fp32", 6, 384, 1025, (8, 128), True, True), ("bf16", 6, 384, 1025, (32, 32), True, True),
    ("fp32", 1, 64, 50, (7, 7), False, True),               # too small to fill the chip
    ("fp32", 16, 384, 4097, (64, 64), False, False),        # longer than a block's LDS holds
])
def test_copies_only_where_they_are_faster(dtype, B, D, L, grid, fwd, bwd):
    """Which calls in column order take scratch for reordered copies (both sides of each
    line as measured, beside the rule in lbscan_dispatch.hip)."""
    from paper_2506_15976_amd import binding
    a = binding.LbscanArgs(B, D, 16, L, 4, binding.LBSCAN_FP32 if dtype == "fp32" else binding.LBSCAN_BF16)
    a.scan_order, (a.grid_h, a.grid_w) = binding.ORDER_COLUMNS, grid
    assert (binding.lbscan_workspace_bytes(a, binding.WS_FWD_ORDER) > 0) == fwd
    assert (binding.lbscan_workspace_bytes(a, binding.WS_BWD_ORDER) > 0) == bwd
