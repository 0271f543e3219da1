"""Which forward calls take scratch for rows cut into segments, on both sides of the lines that
cut_pays and gather_cut_pays in lbscan_dispatch.hip draw (within them whole_is_faster leaves some rows
whole, which the launch decides: test_gpu_fwd_wave.py).  Host logic only."""
import pytest

from paper_2506_15976_amd import binding


@pytest.mark.parametrize("B, D, L, fp32, bf16", [
    (24, 384, 160, False, False),                           # 288 row blocks of 32
    (28, 384, 197, True, True), (29, 384, 197, False, False), (348, 32, 256, False, False),
    (29, 384, 300, True, True), (30, 384, 300, False, False),
    (29, 384, 400, True, True), (30, 384, 400, False, True), (32, 384, 700, False, True), (33, 384, 700, False, False),
    (31, 384, 1601, True, True), (32, 384, 1601, False, True), (64, 176, 1601, False, True),
    (34, 384, 1601, False, True), (35, 384, 1601, False, False),
    (64, 128, 513, True, True),                             # 256 row blocks: always
])
def test_rows_are_cut_where_that_is_faster(B, D, L, fp32, bf16):
    for dtype, cut in ((binding.LBSCAN_FP32, fp32), (binding.LBSCAN_BF16, bf16)):
        a = binding.LbscanArgs(B, D, 16, L, 4, dtype)
        assert (binding.lbscan_workspace_bytes(a, binding.WS_FWD) > 0) == cut
        a.reverse = 1                                       # one size for both directions
        assert (binding.lbscan_workspace_bytes(a, binding.WS_FWD) > 0) == cut


@pytest.mark.parametrize("B, D, grid, fp32, bf16", [
    (24, 384, (12, 12), False, False),                      # 288 row blocks, 145 tokens
    (24, 384, (16, 16), True, True), (32, 384, (16, 16), False, False),
    (12, 384, (32, 32), True, True), (16, 384, (32, 32), False, True), (18, 384, (32, 32), False, True),
    (30, 384, (4, 256), True, True),                        # few rows of the grid
    (8, 384, (64, 64), True, True), (12, 384, (64, 64), False, False), (10, 384, (64, 64), False, True),
])
def test_gathered_rows_are_cut_where_that_is_faster(B, D, grid, fp32, bf16):
    for dtype, cut in ((binding.LBSCAN_FP32, fp32), (binding.LBSCAN_BF16, bf16)):
        a = binding.LbscanArgs(B, D, 16, grid[0] * grid[1] + 1, 4, dtype)
        a.scan_order, (a.grid_h, a.grid_w) = binding.ORDER_COLUMNS, grid
        assert (binding.lbscan_workspace_bytes(a, binding.WS_FWD) > 0) == cut
