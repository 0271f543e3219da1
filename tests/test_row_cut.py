"""Which forward calls cut their rows into segments (and so take scratch), on both sides of the
lines that the rule in lbscan_dispatch.hip draws.  Host logic only."""
import pytest

from paper_2506_15976_amd import binding


@pytest.mark.parametrize("B, D, L, fp32, bf16", [
    (24, 384, 160, False, False),                           # 288 row blocks of 32
    (27, 384, 197, True, True), (28, 384, 197, False, False), (336, 32, 256, False, False),
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
