"""GPU parity of the column-by-column scan order (vertical scan of a 2-D token grid,
paper Sec. 4.5 / Appendix D) against the oracle applied to the reordered sequence."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS3 = ("x", "delta", "Bm", "Cm", "z", "dout")
GRADS3 = ("dx", "ddelta", "dz", "dBm", "dCm")


@pytest.fixture(scope="module")
def lb():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2506_15976_amd as pkg
    pkg.load()
    return pkg


def _reordered(s, perm):
    return {k: (np.ascontiguousarray(v[..., perm]) if (k in KEYS3 and v is not None) else v) for k, v in s.items()}


def _check(lb, oracle, s, grid, *, window, dtype="fp32", reverse=False, bwd=True):
    import torch
    from gpu_util import assert_close, flip_time, fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import column_order
    L = s["x"].shape[-1]
    perm = column_order(L, *grid)
    inv = np.argsort(perm)
    dev = to_device(s, dtype)
    got = lb.lbscan_fwd(**fwd_inputs(dev), window=window, reverse=reverse, grid=grid)
    torch.cuda.synchronize()
    # the oracle sees the sequence in scanned order (reversed on top when asked)
    seq = _reordered(s, perm)
    src = flip_time(seq) if reverse else seq
    ref = oracle.fwd(**fwd_inputs(src), window=window)
    ref = (ref[..., ::-1] if reverse else ref)[..., inv]
    assert_close(to_numpy(got), ref, dtype)
    if not bwd:
        return
    g = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=window, reverse=reverse, grid=grid)
    torch.cuda.synchronize()
    gr = oracle.bwd(**fwd_inputs(src), dout=src["dout"], window=window)
    for k, r in gr.items():
        if r is None:
            continue
        if k in GRADS3:
            r = (r[..., ::-1] if reverse else r)[..., inv]
        assert_close(to_numpy(g[k]), r, dtype, k)


@pytest.mark.parametrize("reverse", [False, True])
@pytest.mark.parametrize("window", [4, 8, 1])
def test_vim_grid_with_class_token(lb, oracle, window, reverse):
    """14 x 14 patches + a class token (L = 197), the class token after or before the grid."""
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 70, 16, 197, seed=3100 + window, with_dout=True, random_A=True)
    _check(lb, oracle, s, (14, 14, 0), window=window, reverse=reverse)
    _check(lb, oracle, s, (14, 14, 1), window=window, reverse=reverse)


def test_high_resolution_grid_bf16_and_fp32(lb, oracle):
    """64 x 64 patches (L = 4096): rows cut into segments, bf16 and fp32 storage."""
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(1, 130, 16, 4096, seed=3200, with_dout=True)
    _check(lb, oracle, s, (64, 64), window=8)
    s = make_inputs(1, 64, 16, 4096, seed=3201, with_dout=True, dtype="bf16")
    _check(lb, oracle, s, (64, 64), window=8, dtype="bf16", reverse=True)


def test_rectangular_grids_ragged_shapes_and_long_windows(lb, oracle):
    from paper_2506_15976_amd.inputs import make_inputs
    for (B, D, N, L, grid, M) in [(1, 64, 16, 60, (5, 12), 4), (2, 33, 8, 77, (7, 10, 3), 2),
                                  (1, 64, 16, 40, (40, 1), 4), (1, 64, 16, 40, (1, 40), 16)]:
        s = make_inputs(B, D, N, L, seed=3300 + L, with_dout=True, random_A=True)
        _check(lb, oracle, s, grid, window=M)
    # a window length that only the backward kernel covers in this order: forward refuses
    s = make_inputs(1, 64, 16, 60, seed=3350, with_dout=True)
    from gpu_util import fwd_inputs, to_device
    dev = to_device(s, "fp32")
    with pytest.raises(lb.LbscanError) as ei:
        lb.lbscan_fwd(**fwd_inputs(dev), window=3, grid=(5, 12))
    assert ei.value.code == -2


def test_full_size_vim_small_column_order(lb, oracle):
    from paper_2506_15976_amd.inputs import WORKLOADS, make_workload
    w = WORKLOADS["vim_small"]
    s = make_workload("vim_small")
    _check(lb, oracle, s, (14, 14, 0), window=w["window"], bwd=False)


# fwd: the storage types in which the forward call of these sizes copies too (the backward
# call does at all of them but the last of the first group)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("B, D, N, L, grid, window, gate, fwd", [
    (3, 5, 16, 6, (2, 3), 4, True, ()),             # 15 rows: an odd number, and more rows than one block's waves
    (2, 33, 8, 77, (7, 10, 3), 2, False, ()),       # tokens before and after the grid, no gate
    (1, 70, 16, 257, (16, 16, 1), 8, True, ()),     # one token past a wave's 256
    (1, 3, 16, 1025, (32, 32), 16, True, ()),       # columns of a width that the LDS banks divide
    (2, 1, 4, 4096, (64, 64), 4, True, ()),         # the longest row that is copied, odd rows
    (1, 2, 16, 4097, (64, 64), 4, True, ()),        # one token longer: gathered
    (9, 61, 16, 4096, (64, 64), 4, True, ("fp32", "bf16")),
    (130, 83, 4, 197, (14, 14, 1), 8, True, ("fp32",)),           # bf16 rows of this length: only larger calls
    (67, 83, 4, 401, (20, 20, 1), 8, True, ("fp32", "bf16")),     # 5561 rows, ten (copy back: four) to a block: one left
    (8, 257, 8, 1025, (32, 32), 16, False, ("fp32", "bf16")),
])
def test_reordered_copies_match_the_gather(lb, monkeypatch, B, D, N, L, grid, window, gate, fwd, dtype):
    """With scratch for copies and without: the same operation, on the same kernels where
    the rows are not handed to another family; fp32 sums in another order differ by a few
    2^-24 of the sum, bf16 results by one rounding (2^-8)."""
    import torch
    from gpu_util import fwd_inputs, to_device
    from paper_2506_15976_amd import binding
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(B, D, N, L, seed=3400 + L, with_dout=True, random_A=True, dtype=dtype)
    if not gate:
        s["z"] = None
    dev = to_device(s, dtype)
    rel = 2e-5 if dtype == "fp32" else 2 ** -7

    def both():
        out = lb.lbscan_fwd(**fwd_inputs(dev), window=window, grid=grid, reverse=bool(L & 1))
        g = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=window, grid=grid, reverse=bool(L & 1))
        torch.cuda.synchronize()
        return {"out": out, **g}

    a = binding.make_args(**fwd_inputs(dev), window=window, grid=grid)
    assert (binding.lbscan_workspace_bytes(a, binding.WS_BWD_ORDER) > 0) == (L <= 4096)
    assert (binding.lbscan_workspace_bytes(a, binding.WS_FWD_ORDER) > 0) == (dtype in fwd)
    copied = both()
    size = binding.lbscan_workspace_bytes
    monkeypatch.setattr(binding, "lbscan_workspace_bytes",
                        lambda a, which: 0 if which in (binding.WS_FWD_ORDER, binding.WS_BWD_ORDER) else size(a, which))
    gathered = both()
    for k, v in gathered.items():
        if v is None:
            assert copied[k] is None
            continue
        r = v.float()
        bound = rel * torch.maximum(r.abs(), r.square().mean().sqrt())
        assert bool(((copied[k].float() - r).abs() <= bound).all()), k


# ---- column order with everything else a call can take, gathers and copies ----------

@pytest.fixture
def route(monkeypatch):
    """route(False): calls get no scratch for reordered copies, as on a full device."""
    from paper_2506_15976_amd import binding
    have = binding._optional_block
    return lambda copies: monkeypatch.setattr(binding, "_optional_block", have if copies else lambda n, device: None)


def _states(B, D, N, seed):
    r = np.random.default_rng(seed)
    return (r.standard_normal((B, D, N)).astype(np.float32), r.standard_normal((B, D, N)).astype(np.float32))


def _scanned(s, grid, reverse):
    """Inputs as the oracle takes them, and the way back to stored order."""
    from gpu_util import flip_time
    from paper_2506_15976_amd.inputs import column_order
    perm = column_order(s["x"].shape[-1], *grid)
    seq = _reordered(s, perm)
    inv = np.argsort(perm)
    return (flip_time(seq) if reverse else seq), lambda v: (v[..., ::-1] if reverse else v)[..., inv]


PAIRS = [(True, True), (False, False), (True, False), (False, True)]


@pytest.mark.parametrize("shape, grid, dtype, pairs", [
    # the forward call gathers, the backward call copies (when it may); with checkpoints
    ((3, 70, 16, 50), (7, 7), "fp32", [(True, True), (True, False)]),
    ((3, 70, 16, 50), (7, 7, 1), "bf16", [(True, True), (True, False)]),
    # both copy, rows not cut: with checkpoints
    ((130, 83, 16, 197), (14, 14, 1), "fp32", PAIRS),
    # both copy, rows cut into segments: no checkpoints
    ((9, 61, 16, 4096), (64, 64), "bf16", [(True, True), (False, True)]),
])
@pytest.mark.parametrize("reverse", [False, True])
def test_states_and_checkpoints(lb, oracle, route, shape, grid, dtype, pairs, reverse):
    """The state entering and leaving the call, its gradients, and checkpoints that one
    route leaves and the other one reads, on a stream of the caller's."""
    import torch
    from gpu_util import assert_close, fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import make_inputs
    B, D, N, L = shape
    s = make_inputs(B, D, N, L, seed=3500 + L, with_dout=True, random_A=True, dtype=dtype)
    h0, dhT = _states(B, D, N, 3501 + L)
    src, back = _scanned(s, grid, reverse)
    ref, ref_hT = oracle.fwd(**fwd_inputs(src), window=4, h0=h0, return_state=True)
    gr = oracle.bwd(**fwd_inputs(src), dout=src["dout"], window=4, h0=h0, dhT=dhT)
    dev = to_device(s, dtype)
    h0d, dhTd = torch.from_numpy(h0).cuda(), torch.from_numpy(dhT).cuda()
    stream = torch.cuda.Stream()
    for fwd_copies, bwd_copies in pairs:
        saved = lb.lbscan_saved_state(dev["x"], dev["A"], window=4)
        assert (saved is not None) == (L < 4096)
        torch.cuda.synchronize()
        route(fwd_copies)
        out, hT = lb.lbscan_fwd(**fwd_inputs(dev), window=4, reverse=reverse, grid=grid, h0=h0d, saved_state=saved,
                                return_state=True, stream=stream)
        route(bwd_copies)
        g = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=4, reverse=reverse, grid=grid, h0=h0d,
                          dhT=dhTd, saved_state=saved, stream=stream)
        torch.cuda.synchronize()
        assert_close(to_numpy(out), back(ref), dtype, "out")
        assert_close(to_numpy(hT), ref_hT, "fp32", "hT")
        for k, r in gr.items():
            assert_close(to_numpy(g[k]), back(r) if k in GRADS3 else r, "fp32" if k == "dh0" else dtype, k)


@pytest.mark.parametrize("copies", [True, False])
@pytest.mark.parametrize("window", [3, 12, 1000])
def test_backward_windows_without_a_compiled_kernel(lb, oracle, route, window, copies):
    import torch
    from gpu_util import assert_close, fwd_inputs, to_device, to_numpy
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(2, 70, 16, 101, seed=3600 + window, with_dout=True, random_A=True)
    src, back = _scanned(s, (10, 10), False)
    gr = oracle.bwd(**fwd_inputs(src), dout=src["dout"], window=window)
    dev = to_device(s, "fp32")
    route(copies)
    g = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=window, grid=(10, 10))
    torch.cuda.synchronize()
    for k, r in gr.items():
        if r is not None:
            assert_close(to_numpy(g[k]), back(r) if k in GRADS3 else r, "fp32", k)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_copies_replay_from_a_graph(lb, dtype):
    """Forward call with checkpoints and backward call from them, both on copies, recorded
    once; every replay against the eager results, with eager work in between."""
    import torch
    from gpu_util import fwd_inputs, to_device
    from paper_2506_15976_amd import binding
    from paper_2506_15976_amd.inputs import make_inputs
    s = make_inputs(67, 83, 4, 401, seed=3700, with_dout=True, dtype=dtype)
    dev = to_device(s, dtype)
    a = binding.make_args(**fwd_inputs(dev), window=8, grid=(20, 20, 1))
    assert all(binding.lbscan_workspace_bytes(a, w) for w in (binding.WS_FWD_ORDER, binding.WS_BWD_ORDER))

    def step():
        out = lb.lbscan_fwd(**fwd_inputs(dev), window=8, grid=(20, 20, 1))
        return {"out": out, **lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=8, grid=(20, 20, 1))}
    eager = {k: v.clone() for k, v in step().items()}
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        recorded = step()
    summed = ("dA", "dDskip", "ddelta_bias")        # fp32 atomics: their last bits vary
    for k in range(3):
        for v in recorded.values():
            v.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for name, v in recorded.items():
            if name in summed:
                assert float((v - eager[name]).norm() / eager[name].norm()) <= 1e-5, (name, k)
            else:
                assert torch.equal(v, eager[name]), (name, k)
        again = step()
        torch.cuda.synchronize()
        assert torch.equal(again["out"], eager["out"])


@pytest.mark.parametrize("dtype, B, grid", [
    ("fp32", 20, (14, 14, 0)), ("fp32", 20, (13, 16, 1)), ("fp32", 20, (16, 16, 0)), ("fp32", 20, (9, 25, 3)),
    # bf16 rows copy in the forward call from 208 tokens on, smaller calls from 320
    ("bf16", 12, (18, 18, 0)), ("bf16", 32, (13, 16, 1)), ("bf16", 32, (16, 16, 0)), ("bf16", 32, (9, 25, 3)),
])
def test_copies_with_room_behind_their_rows(lb, oracle, dtype, B, grid):
    """The copies' rows start at multiples of 32 tokens: ragged rows (of odd length among them) and
    whole ones, both directions, at sizes that copy in both passes."""
    from paper_2506_15976_amd import binding
    from paper_2506_15976_amd.inputs import make_inputs
    h, w, prefix = grid
    L = prefix + h * w + (1 if h in (14, 18) else 0)
    D, N = 560, 16
    a = binding.LbscanArgs(B, D, N, L, 4, 0 if dtype == "fp32" else 1)
    a.scan_order, a.grid_h, a.grid_w, a.grid_prefix = binding.ORDER_COLUMNS, h, w, prefix
    assert all(binding.lbscan_workspace_bytes(a, which) > 0 for which in (binding.WS_FWD_ORDER, binding.WS_BWD_ORDER))
    s = make_inputs(B, D, N, L, seed=9700 + L, dtype=dtype, with_dout=True)
    for reverse in (False, True):
        _check(lb, oracle, s, grid, window=4, dtype=dtype, reverse=reverse)


@pytest.mark.parametrize("dim", [220, 400, 480, 560])
@pytest.mark.parametrize("batch, segments", [(1, 3), (3, 2)])
def test_gathered_rows_in_segments(lb, oracle, route, batch, segments, dim):
    """Row blocks that are padded to whole rounds of the XCDs, or not (7 to 54 of them), without
    copies: the forward call, and the summary pass of the backward one."""
    from paper_2506_15976_amd.inputs import make_inputs
    route(False)
    s = make_inputs(batch, dim, 5, 91, seed=9800 + dim, with_dout=True, random_A=True)
    lb.lbscan_set_option("segments", segments)
    try:
        _check(lb, oracle, s, (9, 10, 1), window=4, reverse=bool(batch & 2))
    finally:
        lb.lbscan_set_option("segments", 0)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("after", [0, 1, 2])
@pytest.mark.parametrize("reverse", [False, True])
def test_what_lies_behind_a_copied_row_is_not_scanned(lb, route, after, reverse, dtype):
    """One to three tokens in the copies' last tile, and copies of the last scanned one behind them,
    which are loaded with it.  That token is not finite: it reaches what it reaches in the gathered
    rows, whose last tile holds zeros there."""
    import torch
    from gpu_util import fwd_inputs, to_device
    from paper_2506_15976_amd import binding
    from paper_2506_15976_amd.inputs import column_order, make_inputs
    B, D, N, L, grid = 32, 560, 4, 257 + after, (16, 16, 1)
    a = binding.LbscanArgs(B, D, N, L, 8, 0 if dtype == "fp32" else 1)
    a.scan_order, a.grid_h, a.grid_w, a.grid_prefix = binding.ORDER_COLUMNS, *grid
    assert all(binding.lbscan_workspace_bytes(a, which) > 0 for which in (binding.WS_FWD_ORDER, binding.WS_BWD_ORDER))
    s = make_inputs(B, D, N, L, seed=9900 + after, dtype=dtype, with_dout=True)
    last = column_order(L, *grid)[-1]
    s["Bm"][0, 1, last] = np.inf
    s["Cm"][1, 2, last] = -np.inf
    s["x"][2, 3, last] = np.nan
    s["delta"][3, 4, last] = np.inf
    dev = to_device(s, dtype)
    rel = 2e-5 if dtype == "fp32" else 2 ** -7          # as the finite values of copies and gathers differ

    def both():
        out = lb.lbscan_fwd(**fwd_inputs(dev), window=8, reverse=reverse, grid=grid)
        g = lb.lbscan_bwd(**fwd_inputs(dev), dout=dev["dout"], window=8, reverse=reverse, grid=grid)
        torch.cuda.synchronize()
        return {"out": out, **g}
    copied = both()
    route(False)
    for k, v in both().items():
        c, v = copied[k].float(), v.float()
        fine = torch.isfinite(v)
        assert torch.equal(torch.isfinite(c), fine), k
        assert torch.equal(torch.isnan(c), torch.isnan(v)), k
        size = v[fine]
        bound = rel * torch.maximum(size.abs(), size.square().mean().sqrt()) if size.numel() else size
        assert bool(((c[fine] - size).abs() <= bound).all()), k
