"""GPU parity of lbscan_fwd / lbscan_bidir_fwd against the fp64 CPU oracle,
element by element on the same seeded inputs, through the C ABI."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2506_15976_amd as pkg
    pkg.load()
    return pkg


def _run_fwd(lb, oracle, s, *, window, dtype="fp32", reverse=False, softplus=True):
    import torch
    from gpu_util import assert_close, flip_time, fwd_inputs, to_device, to_numpy
    dev = to_device(s, dtype)
    got = lb.lbscan_fwd(**fwd_inputs(dev), window=window, delta_softplus=softplus, reverse=reverse)
    torch.cuda.synchronize()
    got = to_numpy(got)
    src = flip_time(s) if reverse else s
    ref = oracle.fwd(**fwd_inputs(src), window=window, delta_softplus=softplus)
    if reverse:
        ref = ref[..., ::-1]
    return assert_close(got, ref, dtype)


@pytest.mark.parametrize("window", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("reverse", [False, True])
def test_tiny_workload_all_windows(lb, oracle, window, reverse):
    from paper_2506_15976_amd.inputs import make_workload
    s = make_workload("tiny")
    _run_fwd(lb, oracle, s, window=window, reverse=reverse)


@pytest.mark.parametrize("shape", [
    # (B, D, N, L): ragged tails, several tiles, partial blocks, small state sizes
    (2, 70, 16, 37), (1, 130, 16, 197), (3, 5, 16, 5), (2, 64, 16, 1), (1, 300, 16, 16),
    (2, 33, 16, 17), (1, 64, 8, 50), (2, 20, 3, 29), (1, 7, 1, 63), (1, 257, 16, 33),
])
@pytest.mark.parametrize("window", [1, 4, 8])
def test_ragged_shapes(lb, oracle, shape, window):
    from paper_2506_15976_amd.inputs import make_inputs
    B, D, N, L = shape
    s = make_inputs(B, D, N, L, seed=1234 + B * 7 + D + L, random_A=True)
    _run_fwd(lb, oracle, s, window=window)
    _run_fwd(lb, oracle, s, window=window, reverse=True)


@pytest.mark.parametrize("N", [1, 7, 8, 9, 16])
@pytest.mark.parametrize("segments", [0, 1, 3])
def test_every_spread_of_the_states(lb, oracle, N, segments):
    """A lane holds one state of a row up to N = 8 and two beyond, with lanes that hold fewer or
    none: rows whose segments are the waves of a block (the library's choice for the long
    ones here), whole rows and rows cut by the launch."""
    from paper_2506_15976_amd.inputs import make_inputs
    lb.lbscan_set_option("segments", segments)
    try:
        for (B, D, L, M) in [(2, 70, 37, 4), (1, 130, 100, 8), (1, 64, 33, 2), (2, 64, 197, 16)]:
            s = make_inputs(B, D, N, L, seed=4000 + D + L, random_A=True)
            _run_fwd(lb, oracle, s, window=M)
            _run_fwd(lb, oracle, s, window=M, reverse=True)
        s = make_inputs(1, 96, N, 64, seed=4100, dtype="bf16")
        _run_fwd(lb, oracle, s, window=4, dtype="bf16")
    finally:
        lb.lbscan_set_option("segments", 0)


@pytest.mark.parametrize("segments", [2, 3, 7])
def test_rows_cut_into_segments(lb, oracle, segments):
    """Long rows with few channels are cut into segments scanned in parallel
    (summary pass, carry chain, full pass); force several cuts."""
    from paper_2506_15976_amd.inputs import make_inputs
    lb.lbscan_set_option("segments", segments)
    try:
        for (B, D, N, L, M) in [(1, 70, 16, 333, 4), (2, 64, 8, 128, 8), (1, 130, 16, 97, 16), (1, 64, 16, 700, 1)]:
            s = make_inputs(B, D, N, L, seed=6000 + D + L, random_A=True)
            _run_fwd(lb, oracle, s, window=M)
            _run_fwd(lb, oracle, s, window=M, reverse=True)
        s = make_inputs(1, 96, 16, 256, seed=6100, dtype="bf16")
        _run_fwd(lb, oracle, s, window=8, dtype="bf16")
        sf = make_inputs(1, 70, 16, 333, seed=6200, random_A=True)
        sb = make_inputs(1, 70, 16, 333, seed=6201, random_A=True)
        _run_bidir(lb, oracle, sf, sb)
        sf = make_inputs(1, 64, 16, 200, seed=6300, dtype="bf16")
        sb = make_inputs(1, 64, 16, 200, seed=6301, dtype="bf16")
        _run_bidir(lb, oracle, sf, sb, dtype="bf16")
    finally:
        lb.lbscan_set_option("segments", 0)


def test_long_rows_pick_segments_by_themselves(lb, oracle):
    from gpu_util import fwd_inputs, to_device
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(1, 64, 16, 5000, seed=6400)
    dev = to_device(s, "fp32")
    a = lb.make_args(**fwd_inputs(dev), window=4)
    assert lb.lbscan_workspace_bytes(a, 0) > 0          # segmented: needs scratch
    _run_fwd(lb, oracle, s, window=4)
    _run_fwd(lb, oracle, s, window=16, reverse=True)


def test_missing_workspace_is_an_error(lb):
    import ctypes
    import torch
    from gpu_util import fwd_inputs, to_device
    from paper_2506_15976_amd.inputs import make_inputs
    dev = to_device(make_inputs(1, 64, 16, 5000, seed=6500), "fp32")
    y = torch.empty_like(dev["x"])
    a = lb.make_args(**fwd_inputs(dev), window=4, y=y)
    rc = lb.load().lbscan_fwd(ctypes.byref(a), None)
    assert rc == -3


def test_optional_arguments_absent(lb, oracle):
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 96, 16, 61, seed=77, with_z=False)
    s["Dskip"] = None
    s["delta_bias"] = None
    _run_fwd(lb, oracle, s, window=4)
    s2 = make_inputs(2, 96, 16, 61, seed=78)
    s2["delta"] = np.abs(s2["delta"]) * 0.2 + 0.01
    s2["delta_bias"] = None
    _run_fwd(lb, oracle, s2, window=4, softplus=False)


def test_call_on_a_side_stream(lb, oracle):
    """The binding's scratch and outputs are tied to the stream the kernels run on
    (default priority), not only to the current one."""
    import torch
    from gpu_util import assert_close, fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(1, 64, 16, 3000, seed=55, with_dout=True)      # long rows: scratch in use
    dev = to_device(s, "fp32")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    out = lb.lbscan_fwd(**fwd_inputs(dev), window=4, stream=side)
    g = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=4, stream=side)
    junk = [torch.full((1 << 20,), float("nan"), device="cuda:0") for _ in range(8)]   # current stream
    side.synchronize()
    torch.cuda.synchronize()
    assert_close(to_numpy(out), oracle.fwd(**fwd_inputs(s), window=4), "fp32")
    ref = oracle.bwd(**fwd_inputs(s), dout=s["dout"], window=4)
    for k in ("dx", "dBm", "dA"):
        assert_close(to_numpy(g[k]), ref[k], "fp32", k)
    del junk


def test_window_covering_short_row(lb, oracle):
    """M >= L with L <= 16 is one window over the whole row."""
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 64, 16, 11, seed=5)
    _run_fwd(lb, oracle, s, window=11)
    _run_fwd(lb, oracle, s, window=1000)


def test_any_window_bf16_rows_of_even_length_with_odd_windows(lb, oracle):
    """2-byte storage, even row length, odd window length: the second pass walks
    segments of odd length, whose mirrored quads would start at odd elements; they
    must take the element-wise path (default segmentation and forced cuts)."""
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(1, 70, 16, 1000, seed=77, dtype="bf16")
    for window in (5, 3, 13):
        _run_fwd(lb, oracle, s, window=window, dtype="bf16")
        _run_fwd(lb, oracle, s, window=window, dtype="bf16", reverse=True)
    lb.lbscan_set_option("segments", 7)
    try:
        _run_fwd(lb, oracle, s, window=5, dtype="bf16")
        _run_fwd(lb, oracle, s, window=5, dtype="bf16", reverse=True)
    finally:
        lb.lbscan_set_option("segments", 0)


@pytest.mark.parametrize("shape,window", [
    ((2, 70, 16, 37), 3), ((1, 130, 16, 197), 5), ((3, 5, 16, 50), 7), ((2, 64, 16, 64), 12),
    ((1, 64, 8, 100), 33), ((2, 20, 3, 29), 6), ((1, 7, 1, 63), 63), ((2, 64, 16, 200), 1000),
    ((1, 66, 16, 131), 32), ((1, 64, 16, 64), 64),
])
@pytest.mark.parametrize("reverse", [False, True])
def test_any_window_length(lb, oracle, shape, window, reverse):
    """Window lengths without a fused kernel (the paper's figures use 3) run as two
    passes: plain forward scan, then the local backward part."""
    from paper_2506_15976_amd.inputs import make_inputs
    B, D, N, L = shape
    s = make_inputs(B, D, N, L, seed=700 + L + window, random_A=True)
    _run_fwd(lb, oracle, s, window=window, reverse=reverse)


@pytest.mark.parametrize("nseg", [1, 3, 11])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_any_window_length_long_rows_in_segments(lb, oracle, nseg, dtype):
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(1, 70, 16, 1001, seed=720 + nseg, dtype=dtype)
    lb.lbscan_set_option("segments", nseg)
    try:
        for window in (3, 24):
            _run_fwd(lb, oracle, s, window=window, dtype=dtype)
            _run_fwd(lb, oracle, s, window=window, dtype=dtype, reverse=True)
    finally:
        lb.lbscan_set_option("segments", 0)


def test_any_window_length_default_segmentation_of_long_rows(lb, oracle):
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(1, 64, 16, 5000, seed=730)
    _run_fwd(lb, oracle, s, window=6)


def test_any_window_length_with_states(lb, oracle):
    import torch
    from gpu_util import assert_close, fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 64, 16, 90, seed=740)
    h0 = np.random.default_rng(741).standard_normal((2, 64, 16)).astype(np.float32)
    dev = to_device(s, "fp32")
    out, hT = lb.lbscan_fwd(**fwd_inputs(dev), window=9, h0=torch.from_numpy(h0).cuda(), return_state=True)
    torch.cuda.synchronize()
    ref, ref_hT = oracle.fwd(**fwd_inputs(s), window=9, h0=h0, return_state=True)
    assert_close(to_numpy(out), ref, "fp32", "out")
    assert_close(to_numpy(hT), ref_hT, "fp32", "hT")


def test_zero_timestep_is_skip_times_gate(lb):
    """delta = 0 without softplus: out = Dskip * x * SiLU(z)."""
    import torch
    from gpu_util import fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 128, 16, 45, seed=8)
    s["delta"] = np.zeros_like(s["delta"])
    s["delta_bias"] = None
    s["Dskip"] = np.random.default_rng(9).standard_normal(128).astype(np.float32)
    dev = to_device(s, "fp32")
    got = to_numpy(lb.lbscan_fwd(**fwd_inputs(dev), window=4, delta_softplus=False))
    z = s["z"].astype(np.float64)
    ref = s["Dskip"][None, :, None] * s["x"] * (z / (1 + np.exp(-z)))
    np.testing.assert_allclose(got, ref, rtol=2e-6, atol=1e-7)


def test_bf16_storage_small(lb, oracle):
    from paper_2506_15976_amd.inputs import make_inputs
    for L in (64, 197, 33):
        s = make_inputs(2, 96, 16, L, seed=300 + L, dtype="bf16")
        _run_fwd(lb, oracle, s, window=8, dtype="bf16")
        _run_fwd(lb, oracle, s, window=4, dtype="bf16", reverse=True)


@pytest.mark.parametrize("L", [197, 193, 225, 65, 37])
def test_bf16_rows_of_odd_length(lb, oracle, L):
    """bf16 rows of odd length start at odd elements every other row: tiles inside the
    row go through the unaligned quad path (not allowed to reach past the tensor: the
    last batch entry's end tile keeps element accesses), ragged tiles through element
    loads.  Several batch entries, partial row blocks, both directions, rows cut."""
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(3, 70, 16, L, seed=3300 + L, dtype="bf16", random_A=True)
    for window in (4, 8, 1):
        _run_fwd(lb, oracle, s, window=window, dtype="bf16")
        _run_fwd(lb, oracle, s, window=window, dtype="bf16", reverse=True)
    lb.lbscan_set_option("segments", 3)
    try:
        _run_fwd(lb, oracle, s, window=4, dtype="bf16")
        _run_fwd(lb, oracle, s, window=4, dtype="bf16", reverse=True)
    finally:
        lb.lbscan_set_option("segments", 0)


@pytest.mark.parametrize("name", ["vim_tiny", "vim_small", "hires_4096", "wsi_bag"])
def test_full_size_workloads(lb, oracle, name):
    from paper_2506_15976_amd.inputs import WORKLOADS, make_workload
    w = WORKLOADS[name]
    s = make_workload(name)
    err = _run_fwd(lb, oracle, s, window=w["window"], dtype=w["dtype"])
    print(f"{name}: err={err:.3e}")


def _run_bidir(lb, oracle, sf, sb, dtype="fp32"):
    import torch
    from gpu_util import assert_close, fwd_inputs, to_device, to_numpy
    df, db = to_device(sf, dtype), to_device(sb, dtype)
    got = lb.lbscan_bidir_fwd(fwd_inputs(df), fwd_inputs(db))
    torch.cuda.synchronize()
    ref = oracle.bidir_fwd(fwd_inputs(sf), fwd_inputs(sb))
    assert_close(to_numpy(got), ref, dtype, "bidir")


def test_bidir_small_and_ragged(lb, oracle):
    from paper_2506_15976_amd.inputs import make_inputs
    for (B, D, N, L) in [(2, 70, 16, 37), (1, 64, 16, 256), (1, 130, 8, 19)]:
        sf = make_inputs(B, D, N, L, seed=500 + L, random_A=True)
        sb = make_inputs(B, D, N, L, seed=1500 + L, random_A=True)
        _run_bidir(lb, oracle, sf, sb)
    sf = make_inputs(2, 64, 16, 100, seed=600, dtype="bf16")
    sb = make_inputs(2, 64, 16, 100, seed=1600, dtype="bf16")
    _run_bidir(lb, oracle, sf, sb, dtype="bf16")


def test_bidir_vim_tiny(lb, oracle):
    from paper_2506_15976_amd.inputs import make_workload
    _run_bidir(lb, oracle, make_workload("vim_tiny"), make_workload("vim_tiny", direction_b=True))


def test_extreme_time_steps_and_decay_rates(lb, oracle):
    """Time steps from the linear branch of softplus (argument above 20) down to
    underflow, decay rates up to abar = 0, and rows cut into segments: nothing
    overflows and the result stays within the parity bar."""
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 64, 16, 300, seed=9100, with_dout=True)
    r = np.random.default_rng(9101)
    s["delta"] = r.choice(np.array([-90.0, -12.0, -1.0, 0.5, 3.0, 25.0], dtype=np.float32),
                          size=s["delta"].shape).astype(np.float32)
    s["delta_bias"] = np.zeros_like(s["delta_bias"])
    s["A"] = -r.choice(np.array([1e-3, 0.5, 4.0, 40.0, 1e3], dtype=np.float32), size=s["A"].shape).astype(np.float32)
    for nseg in (0, 3):
        lb.lbscan_set_option("segments", nseg)
        try:
            _run_fwd(lb, oracle, s, window=4)
            _run_fwd(lb, oracle, s, window=4, reverse=True)
            _run_fwd(lb, oracle, s, window=7)
        finally:
            lb.lbscan_set_option("segments", 0)
