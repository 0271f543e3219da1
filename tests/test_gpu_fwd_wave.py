"""Forward kernel at the edges of its tiles (8 rows a wave, 32 a block, 32 tokens), and rows of
one chunk, which a rule shares out between it and the chunk-per-lane kernel; fp64 oracle as the
reference."""
import pytest

pytestmark = pytest.mark.gpu


def _check(lb, oracle, s, dtype, window, reverse, h0=None):
    import numpy as np
    import torch
    from gpu_util import assert_close, flip_time, fwd_inputs, to_device, to_numpy
    dev = to_device(s, dtype)
    state = None if h0 is None else torch.from_numpy(h0).to("cuda:0")
    got, hT = lb.lbscan_fwd(**fwd_inputs(dev), window=window, reverse=reverse, h0=state, return_state=True)
    torch.cuda.synchronize()
    src = flip_time(s) if reverse else s
    ref, ref_state = oracle.fwd(**fwd_inputs(src), window=window, h0=h0, return_state=True)
    what = f"window {window} reverse {reverse}"
    assert_close(to_numpy(got), np.ascontiguousarray(ref[..., ::-1]) if reverse else ref, dtype, what)
    assert_close(to_numpy(hT), ref_state, "fp32", what + " state")


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", [
    (1, 1, 16, 1), (2, 9, 9, 31), (1, 33, 8, 32), (3, 40, 16, 33), (1, 24, 1, 65), (2, 65, 5, 3), (1, 31, 16, 100),
    (2, 21, 16, 197), (1, 8, 7, 256), (1, 17, 16, 257), (2, 3, 16, 509), (1, 9, 16, 512), (1, 9, 16, 513),
])
def test_outputs_at_the_edges_of_a_tile(oracle, shape, dtype):
    import numpy as np
    import paper_2506_15976_amd as lb
    from paper_2506_15976_amd.inputs import make_inputs
    B, D, N, L = shape
    s = make_inputs(B, D, N, L, seed=9300 + D + L, dtype=dtype, random_A=True)
    h0 = np.random.default_rng(D).standard_normal((B, D, N)).astype(np.float32)
    for window, reverse in ((1, True), (2, False), (4, True), (8, False), (16, True), (5, False), (24, True)):
        _check(lb, oracle, s, dtype, window, reverse, h0)
    lb.lbscan_set_option("segments", 3)
    try:
        _check(lb, oracle, s, dtype, 4, False, h0)
        _check(lb, oracle, s, dtype, 8, True, h0)
    finally:
        lb.lbscan_set_option("segments", 0)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("tokens", [39, 40, 41, 69, 72, 104, 105])
def test_a_short_last_tile(oracle, tokens, dtype):
    """Rows whose last tile holds seven to nine tokens (up to eight are staged one a lane, beyond
    that a quad a lane), whole, cut and in the summary of a cut backward pass."""
    import numpy as np
    import torch
    import paper_2506_15976_amd as lb
    from gpu_util import assert_close, fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import make_inputs
    for D, N in ((13, 16), (40, 7)):
        s = make_inputs(2, D, N, tokens, seed=9700 + D + tokens, dtype=dtype, random_A=True, with_dout=True)
        h0 = np.random.default_rng(D).standard_normal((2, D, N)).astype(np.float32)
        dev = to_device(s, dtype)
        for segments in (1, 2):
            lb.lbscan_set_option("segments", segments)
            try:
                for window, reverse in ((4, False), (8, True), (16, False), (16, True), (6, True)):
                    _check(lb, oracle, s, dtype, window, reverse, h0)
                for window in (4, 6):
                    got = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=window)
                    torch.cuda.synchronize()
                    ref = oracle.bwd(**fwd_inputs(s), dout=s["dout"], window=window)
                    for k in ("dx", "ddelta", "dz", "dBm", "dCm", "dA"):
                        assert_close(to_numpy(got[k]), ref[k], dtype, f"{k} window {window} segments {segments}")
            finally:
                lb.lbscan_set_option("segments", 0)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("tokens", [1, 3, 9, 31, 32, 35, 41, 62, 64, 66, 95, 96, 129, 197, 230])
def test_every_way_of_loading_rows_gives_the_same_bits(monkeypatch, tokens, dtype):
    """A grid of one column is the stored order, and its rows are gathered token by token: the same
    values as whole quads (even rows), unaligned ones (odd rows of a 2-byte type) and the
    last tiles of either, and the same arithmetic behind them.  Rows whole, cut, and (few tiles, few
    rows) in one block; forward call, and the gradients that no atomics are in."""
    import torch
    import paper_2506_15976_amd as lb
    from gpu_util import fwd_inputs, to_device
    from paper_2506_15976_amd import binding
    from paper_2506_15976_amd.inputs import make_inputs
    monkeypatch.setattr(binding, "_optional_block", lambda n, device: None)
    for D, N, gate in ((13, 16, True), (40, 7, False)):
        s = make_inputs(2, D, N, tokens, seed=9800 + D + tokens, dtype=dtype, random_A=True, with_dout=True)
        if not gate:
            s["z"] = None
        dev = to_device(s, dtype)
        for segments in (0, 1, 2):
            lb.lbscan_set_option("segments", segments)
            try:
                for window in (1, 4, 8, 16):
                    for reverse in (False, True):
                        def both(**grid):
                            out = lb.lbscan_fwd(**fwd_inputs(dev), window=window, reverse=reverse, **grid)
                            g = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=window, reverse=reverse, **grid)
                            torch.cuda.synchronize()
                            return {"out": out, **g}
                        stored, gathered = both(), both(grid=(tokens, 1))
                        for k in ("out", "dx", "ddelta", "dz", "dBm", "dCm"):
                            if gathered[k] is not None:
                                assert torch.equal(stored[k], gathered[k]), (k, N, segments, window, reverse)
            finally:
                lb.lbscan_set_option("segments", 0)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 5, 16, 1024), (2, 3, 7, 820), (1, 200, 16, 1000), (1, 1537, 5, 822)])
def test_rows_of_one_chunk(oracle, shape, dtype):
    """Rows of 820 to 1024 tokens, which the library hands to one family or the other: its own
    choice (the wave tiles for the third), and each family asked for."""
    import numpy as np
    import paper_2506_15976_amd as lb
    from paper_2506_15976_amd.inputs import make_inputs
    B, D, N, L = shape
    s = make_inputs(B, D, N, L, seed=9400 + D + L, dtype=dtype, random_A=True)
    h0 = np.random.default_rng(D).standard_normal((B, D, N)).astype(np.float32)
    for mapping in (0, 1, 2):
        lb.lbscan_set_option("mapping", mapping)
        try:
            for window, reverse in ((4, False), (16, True)):
                _check(lb, oracle, s, dtype, window, reverse, h0)
        finally:
            lb.lbscan_set_option("mapping", 0)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("tokens, segments", [(1024, 3), (1024, 32)])
def test_a_forced_cut_is_made(oracle, tokens, segments, dtype):
    """Option "segments" at sizes that the library itself hands to the chunk-per-lane kernel, which
    takes rows whole: the summaries are written to the scratch, and the result is right."""
    import ctypes
    import torch
    import paper_2506_15976_amd as lb
    from gpu_util import assert_close, fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(1, 64, 16, tokens, seed=9450 + tokens, dtype=dtype)
    dev = to_device(s, dtype)
    y = torch.empty_like(dev["x"])
    a = lb.make_args(**fwd_inputs(dev), window=4, y=y)
    lb.lbscan_set_option("segments", segments)
    try:
        need = lb.lbscan_workspace_bytes(a, 0)
        assert need == segments * 64 * (16 + 1) * 4
        ws = torch.full((need // 4,), float("nan"), device="cuda:0")
        a.workspace, a.workspace_bytes = ws.data_ptr(), need
        rc = lb.load().lbscan_fwd(ctypes.byref(a), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        lb.lbscan_set_option("segments", 0)
    assert rc == 0
    written = torch.isfinite(ws).sum().item()
    assert written >= (segments - 1) * 64 * (16 + 1)        # nobody reads the last segment's
    assert_close(to_numpy(y), oracle.fwd(**fwd_inputs(s), window=4), dtype)


@pytest.mark.parametrize("blocks, tokens, states, dtype, cut", [
    # on both sides of the lines beside whole_is_faster, within those that scratch is sized by
    (324, 197, 16, "fp32", False), (336, 256, 16, "bf16", False), (207, 300, 16, "fp32", True), (208, 300, 16, "bf16", False),
    (240, 300, 8, "bf16", True), (312, 300, 8, "fp32", False), (287, 448, 16, "fp32", True), (288, 448, 16, "fp32", False),
    (311, 448, 16, "bf16", True), (312, 448, 16, "bf16", False), (317, 449, 16, "fp32", True), (318, 449, 16, "fp32", False),
    (341, 700, 16, "bf16", True), (342, 700, 16, "bf16", False), (365, 1100, 16, "bf16", True), (366, 1100, 16, "bf16", False),
    (366, 1100, 8, "bf16", True), (252, 700, 16, "fp32", True),
])
def test_rows_stay_whole_where_that_is_faster(blocks, tokens, states, dtype, cut):
    """A call that takes scratch for a cut writes it only where it cuts its rows."""
    import ctypes
    import torch
    import paper_2506_15976_amd as lb
    from paper_2506_15976_amd import binding
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.ones(blocks, 32, tokens, dtype=t, device="cuda:0")
    b = torch.ones(blocks, states, tokens, dtype=t, device="cuda:0")
    A = -torch.ones(32, states, device="cuda:0")
    y = torch.empty_like(x)
    lb.lbscan_set_option("mapping", 1)
    try:
        a = binding.make_args(x, x, A, b, b, window=4, y=y)
        need = binding.lbscan_workspace_bytes(a, binding.WS_FWD)
        ws = torch.full((need // 4,), float("nan"), device="cuda:0")
        a.workspace, a.workspace_bytes = ws.data_ptr(), need
        assert need > 0 and lb.load().lbscan_fwd(ctypes.byref(a), torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
    finally:
        lb.lbscan_set_option("mapping", 0)
    assert bool(torch.isnan(ws).all()) != cut
    assert bool(torch.isfinite(y.float()).all())
