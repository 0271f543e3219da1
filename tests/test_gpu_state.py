"""GPU parity of the state-in / state-out path (lbscan_args.h0 / hT, lbscan_bwd_state)
against the fp64 CPU oracle, through the C ABI: uncut rows, rows cut into segments,
reversed direction, bf16 storage, the saved-state shortcut, and a sequence processed
in chunks on the GPU."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GRADS = ("dx", "ddelta", "dz", "dBm", "dCm", "dA", "dDskip", "ddelta_bias", "dh0")


@pytest.fixture(scope="module")
def lb():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2506_15976_amd as pkg
    pkg.load()
    return pkg


@pytest.fixture()
def segments(lb):
    """Sets the number of segments for one test and restores the default after it."""
    def set_(k):
        lb.lbscan_set_option("segments", k)
    yield set_
    lb.lbscan_set_option("segments", 0)


def _states(B, D, N, seed):
    r = np.random.default_rng(seed)
    return (r.standard_normal((B, D, N)).astype(np.float32),
            r.standard_normal((B, D, N)).astype(np.float32))


def _check_fwd(lb, oracle, s, h0, *, window, dtype="fp32", reverse=False):
    import torch
    from gpu_util import assert_close, flip_time, fwd_inputs, to_device, to_numpy
    dev = to_device(s, dtype)
    h0d = None if h0 is None else torch.from_numpy(h0).cuda()
    out, hT = lb.lbscan_fwd(**fwd_inputs(dev), window=window, reverse=reverse, h0=h0d, return_state=True)
    torch.cuda.synchronize()
    src = flip_time(s) if reverse else s
    ref, ref_hT = oracle.fwd(**fwd_inputs(src), window=window, h0=h0, return_state=True)
    if reverse:
        ref = ref[..., ::-1]
    assert_close(to_numpy(out), ref, dtype, "out")
    assert_close(to_numpy(hT), ref_hT, "fp32", "hT")


def _check_bwd(lb, oracle, s, h0, dhT, *, window, dtype="fp32", reverse=False, saved=False):
    import torch
    from gpu_util import assert_close, flip_time, fwd_inputs, to_device, to_numpy
    dev = to_device(s, dtype)
    h0d = None if h0 is None else torch.from_numpy(h0).cuda()
    dhTd = None if dhT is None else torch.from_numpy(dhT).cuda()
    st = None
    if saved:
        st = lb.lbscan_saved_state(dev["x"], dev["A"], window=window)
        assert st is not None
        lb.lbscan_fwd(**fwd_inputs(dev), window=window, reverse=reverse, h0=h0d, saved_state=st)
    got = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=window, reverse=reverse,
                        h0=h0d, dhT=dhTd, saved_state=st)
    torch.cuda.synchronize()
    src = flip_time(s) if reverse else s
    ref = oracle.bwd(**fwd_inputs(src), dout=src["dout"], window=window, h0=h0, dhT=dhT)
    for k in GRADS:
        r = ref[k]
        if r is None:
            assert got[k] is None
            continue
        if reverse and r.ndim == 3 and k != "dh0":
            r = r[..., ::-1]
        assert_close(to_numpy(got[k]), r, "fp32" if k == "dh0" else dtype, k)


@pytest.mark.parametrize("shape,window", [((2, 70, 16, 37), 4), ((1, 130, 16, 197), 4), ((3, 5, 16, 5), 8),
                                          ((2, 64, 8, 64), 16), ((1, 7, 3, 100), 1)])
@pytest.mark.parametrize("reverse", [False, True])
def test_forward_with_entering_state(lb, oracle, shape, window, reverse):
    from paper_2506_15976_amd.inputs import make_inputs
    B, D, N, L = shape
    s = make_inputs(B, D, N, L, seed=5100 + L, random_A=True)
    h0, _ = _states(B, D, N, 5101 + L)
    _check_fwd(lb, oracle, s, h0, window=window, reverse=reverse)


def test_forward_state_out_without_state_in(lb, oracle):
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 66, 16, 75, seed=5110)
    _check_fwd(lb, oracle, s, None, window=4)


@pytest.mark.parametrize("nseg", [2, 5])
@pytest.mark.parametrize("reverse", [False, True])
def test_forward_with_state_rows_cut_into_segments(lb, oracle, segments, nseg, reverse):
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(1, 70, 16, 400, seed=5120 + nseg, random_A=True)
    h0, _ = _states(1, 70, 16, 5121)
    segments(nseg)
    _check_fwd(lb, oracle, s, h0, window=8, reverse=reverse)


def test_forward_with_state_bf16(lb, oracle):
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 64, 16, 96, seed=5130, dtype="bf16")
    h0, _ = _states(2, 64, 16, 5131)
    _check_fwd(lb, oracle, s, h0, window=8, dtype="bf16")


@pytest.mark.parametrize("shape,window", [((2, 70, 16, 37), 4), ((1, 130, 16, 197), 4), ((3, 5, 16, 5), 8),
                                          ((1, 64, 8, 50), 1)])
@pytest.mark.parametrize("reverse", [False, True])
def test_backward_with_states(lb, oracle, shape, window, reverse):
    from paper_2506_15976_amd.inputs import make_inputs
    B, D, N, L = shape
    s = make_inputs(B, D, N, L, seed=5200 + L, with_dout=True, random_A=True)
    h0, dhT = _states(B, D, N, 5201 + L)
    _check_bwd(lb, oracle, s, h0, dhT, window=window, reverse=reverse)


def test_backward_with_only_the_arriving_gradient(lb, oracle):
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 40, 16, 45, seed=5210, with_dout=True)
    _, dhT = _states(2, 40, 16, 5211)
    _check_bwd(lb, oracle, s, None, dhT, window=4)


@pytest.mark.parametrize("nseg", [17, 18, 33, 256, 257, 258, 300])
def test_chains_of_many_segments(lb, oracle, segments, nseg):
    """The chain kernel at the edges of a wave's share (16 segments) and of a block's (256): rows of
    two batch entries in two blocks of rows, with and without an entering state, both chains."""
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 35, 3, 32 * nseg - 5, seed=5140 + nseg, with_dout=True, random_A=True)
    h0, dhT = _states(2, 35, 3, 5141 + nseg)
    segments(nseg)
    _check_fwd(lb, oracle, s, h0, window=4)
    _check_fwd(lb, oracle, s, None, window=4, reverse=True)
    _check_bwd(lb, oracle, s, h0, dhT, window=4)
    _check_bwd(lb, oracle, s, None, dhT, window=4, reverse=True)


@pytest.mark.parametrize("nseg", [2, 5])
def test_backward_with_states_rows_cut_into_segments(lb, oracle, segments, nseg):
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(1, 70, 16, 400, seed=5220 + nseg, with_dout=True, random_A=True)
    h0, dhT = _states(1, 70, 16, 5221)
    segments(nseg)
    _check_bwd(lb, oracle, s, h0, dhT, window=8)


def test_backward_with_states_from_saved_checkpoints(lb, oracle, segments):
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 70, 16, 90, seed=5230, with_dout=True)
    h0, dhT = _states(2, 70, 16, 5231)
    segments(1)
    _check_bwd(lb, oracle, s, h0, dhT, window=4, saved=True)


def test_backward_with_states_bf16(lb, oracle):
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 64, 16, 96, seed=5240, dtype="bf16", with_dout=True)
    h0, dhT = _states(2, 64, 16, 5241)
    _check_bwd(lb, oracle, s, h0, dhT, window=8, dtype="bf16")


def test_chunked_sequence_on_the_gpu_equals_the_whole(lb, oracle):
    """Three chunk calls with the state handed over reproduce the oracle's single
    call over the whole row (chunk lengths are multiples of the window)."""
    import torch
    from gpu_util import assert_close, fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 96, 16, 200, seed=5300)
    ref, ref_hT = oracle.fwd(**fwd_inputs(s), window=4, return_state=True)
    dev = to_device(s, "fp32")
    cuts = [0, 64, 148, 200]
    outs, h = [], None
    for lo, hi in zip(cuts[:-1], cuts[1:]):
        part = {k: (v[..., lo:hi].contiguous() if v is not None and v.dim() == 3 else v)
                for k, v in fwd_inputs(dev).items()}
        o, h = lb.lbscan_fwd(**part, window=4, h0=h, return_state=True)
        outs.append(o)
    torch.cuda.synchronize()
    assert_close(to_numpy(torch.cat(outs, dim=-1)), ref, "fp32", "out")
    assert_close(to_numpy(h), ref_hT, "fp32", "hT")


def test_empty_row_passes_the_state_through(lb):
    import torch
    x = torch.empty((2, 8, 0), device="cuda")
    Bm = torch.empty((2, 4, 0), device="cuda")
    A = -torch.ones((8, 4), device="cuda")
    h0 = torch.randn((2, 8, 4), device="cuda")
    out, hT = lb.lbscan_fwd(x, x, A, Bm, Bm, window=4, h0=h0, return_state=True)
    torch.cuda.synchronize()
    assert out.shape == (2, 8, 0)
    assert torch.equal(hT, h0)


def test_comparison_method_rejects_states(lb):
    import torch
    from gpu_util import fwd_inputs, to_device
    from paper_2506_15976_amd.inputs import make_inputs
    dev = fwd_inputs(to_device(make_inputs(1, 8, 4, 16, seed=5400), "fp32"))
    h0 = torch.zeros((1, 8, 4), device="cuda")
    y = torch.empty_like(dev["x"])
    a = lb.make_args(**dev, window=1, y=y, h0=h0)
    import ctypes
    rc = lb.load().lbscan_bidir_fwd(ctypes.byref(a), ctypes.byref(a), None)
    assert rc == lb.binding.EINVAL
