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


@pytest.mark.parametrize("tokens, segments", [(97, 2), (1100, 18), (1100, 35), (9000, 282)])
def test_carry_chains_of_any_length(oracle, tokens, segments):
    """Chains folded in the pass, of more segments than a wave takes (16) with a second and a
    third wave partly filled, and of more than a block takes (256): forward states and the
    right-to-left recurrence."""
    import numpy as np
    import torch
    import paper_2506_15976_amd as lb
    from gpu_util import assert_close, fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(1, 35, 5, tokens, seed=9500 + tokens, with_dout=True)
    dev = to_device(s, "fp32")
    rng = np.random.default_rng(tokens)
    h0, dhT = (rng.standard_normal((1, 35, 5)).astype(np.float32) for _ in range(2))
    lb.lbscan_set_option("segments", segments)
    try:
        # (a count that the rounding to whole tiles leaves as it is)
        assert lb.lbscan_workspace_bytes(lb.make_args(**fwd_inputs(dev), window=4), 0) == segments * 35 * (5 + 1) * 4
        out, hT = lb.lbscan_fwd(**fwd_inputs(dev), window=4, h0=torch.from_numpy(h0).cuda(), return_state=True)
        got = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=4, h0=torch.from_numpy(h0).cuda(),
                            dhT=torch.from_numpy(dhT).cuda())
        torch.cuda.synchronize()
    finally:
        lb.lbscan_set_option("segments", 0)
    ref, ref_state = oracle.fwd(**fwd_inputs(s), window=4, h0=h0, return_state=True)
    assert_close(to_numpy(out), ref, "fp32", "out")
    assert_close(to_numpy(hT), ref_state, "fp32", "state")
    grads = oracle.bwd(**fwd_inputs(s), dout=s["dout"], window=4, h0=h0, dhT=dhT)
    for k in GRADS + ("dh0",):
        assert_close(to_numpy(got[k]), grads[k], "fp32", k)
