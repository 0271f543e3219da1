"""Backward kernel at the edges of its tiles: waves with few rows or none, every number of
states per lane, rows around the 16 tokens of a tile; fp64 oracle as the reference."""
import pytest

pytestmark = pytest.mark.gpu

GRADS = ("dx", "ddelta", "dz", "dBm", "dCm", "dA", "dDskip", "ddelta_bias")


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", [
    (1, 1, 16, 1), (2, 17, 13, 16), (1, 65, 16, 31), (2, 80, 5, 47), (1, 49, 4, 4), (1, 100, 1, 18), (3, 33, 8, 17),
    (1, 128, 16, 3), (2, 16, 2, 64),
])
def test_gradients_at_the_edges_of_a_tile(oracle, shape, dtype):
    import torch
    import paper_2506_15976_amd as lb
    from gpu_util import assert_close, flip_time, fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import make_inputs
    B, D, N, L = shape
    s = make_inputs(B, D, N, L, seed=9100 + D + L, dtype=dtype, random_A=True, with_dout=True)
    dev = to_device(s, dtype)
    for window, reverse in ((2, False), (4, True), (8, True), (16, False), (5, False), (24, True)):
        got = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=window, reverse=reverse)
        torch.cuda.synchronize()
        src = flip_time(s) if reverse else s
        ref = oracle.bwd(**fwd_inputs(src), dout=src["dout"], window=window)
        for k in GRADS:
            r = ref[k][..., ::-1] if reverse and ref[k].ndim == 3 else ref[k]
            # parameter gradients of a single row are sums of a few terms: the elementwise
            # bounds of the other parity tests hold for them as they do for long rows
            assert_close(to_numpy(got[k]), r, dtype, f"{k} window {window} reverse {reverse}")
