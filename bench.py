#!/usr/bin/env python3
"""Benchmark of the locally bi-directional selective scan on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME]

A step is one lbscan_fwd call over one batch of synthetic input: the
Vim-small-shaped workload by default (the shape the target is quoted on).
Inputs are resident in HBM before the timed region; launches rotate over several
independent input sets so that the 256 MB Infinity Cache cannot serve them.  One
JSON line is printed: tokens/s of the locally bi-directional scan, the HBM
roofline of its kernel, the fp32 issue bound at the algorithmic operation count,
the speed-up over the two-pass global bi-directional scan on the same inputs,
the fp64 CPU oracle timed on the host cores as a reported baseline, and under
"workloads" the same figures (forward, two-pass comparison, backward) for every
named workload.
"""
import argparse
import ctypes
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0          # MI355X HBM3E, published
# fp32 VALU slots of four clocks a wave instruction: 256 CUs x 64 lanes x 2.4 GHz.  That is what
# compares, selects, shifts and DPP take (measured 4.2 clocks; v_exp_f32 8.2, two slots) and
# about what a plain add, mul or fma takes of a wave alone (4.9); plain ones of several waves overlap down to
# 2.3 clocks.  So the slots compare kernels of one kind with each other, and a kernel of
# plain instructions only could pass this peak.
VALU_PEAK_LANE_OPS = 256 * 64 * 2.4e9
FWD_KEYS = ("x", "delta", "A", "Bm", "Cm", "Dskip", "z", "delta_bias")

# Two figures come from the rocprofv3 summaries committed under profiles/ (counters
# cannot be read from inside this program); both are None when the summary is absent.
#  * L2-to-fabric bytes of one lbscan_fwd call: FETCH_SIZE and WRITE_SIZE (KiB per
#    dispatch) summed over the launches of one call, each scaled by what the same
#    counter reads for a plain elementwise kernel that reads and writes 1 GiB
#    (--copy-calibration: FETCH_SIZE x 2.0, WRITE_SIZE x 1.0);
#  * issue slots per state update of the forward kernels as built (SQ_INSTS_VALU +
#    SQ_INSTS_VALU_TRANS_F32): the secondary figure of alu_bound.
_PROFILE_LINES = {
    "traffic": ("lbscan_kernels_{}.md", r"lbscan_fwd call traffic: (\d+) bytes"),
    "slots": ("lbscan_counters_{}.md", r"lbscan_fwd call issue slots per state update: ([0-9.]+)"),
}


# The launches of one lbscan_fwd call (the library's own choice at these shapes).
FWD_KERNELS = {
    "vim_tiny": "wave_fwd_kernel", "vim_small": "wave_fwd_kernel",
    "hires_4096": "chunk_fwd_kernel",
    "wsi_bag": "wave_fwd_kernel summary pass + carry_chain_kernel + wave_fwd_kernel full pass",
}


def profile_figure(kind, workload):
    import re
    fname, pattern = _PROFILE_LINES[kind]
    if kind == "slots" and workload == "vim_tiny":
        workload = "vim_small"          # the same kernel instance; counters were taken on vim_small
    try:
        text = open(os.path.join(ROOT, "profiles", fname.format(workload))).read()
    except OSError:
        return None
    m = re.search(pattern, text)
    if not m:
        return None
    return int(m.group(1)) if kind == "traffic" else float(m.group(1))


def algorithmic_slots(window):
    """fp32 issue slots one state update needs in the leanest sequential form of the
    method (Eq. 1, 3, 7, 8): dt*A (1), exp (2: half rate), u = (dt x) B (1), f = fma (1),
    y += C h (1), and per window of M steps M-2 fmas for the local backward state and M-1
    for h = f + abar S: 6 + (2M-3)/M for M >= 2, 6 for M = 1 (7.25 at M = 4)."""
    m = max(int(window), 1)
    return 6.0 + (max(2 * m - 3, 0) / m if m >= 2 else 0.0)


def alu_bound(su_per_s, window, workload=None):
    slots = algorithmic_slots(window)
    peak = VALU_PEAK_LANE_OPS / slots
    measured = profile_figure("slots", workload) if workload else None
    return {"bound": "alu", "unit": "state updates/s", "achieved": su_per_s, "peak": peak,
            "frac": su_per_s / peak, "slots_per_state_update": slots,
            "peak_lane_ops_per_s": VALU_PEAK_LANE_OPS,
            "slots_per_state_update_measured": measured,
            "frac_at_measured_slots": None if measured is None else su_per_s * measured / VALU_PEAK_LANE_OPS,
            "note": "fp32 VALU slots of four clocks (256 CUs x 64 lanes x 2.4 GHz) at the "
                    "algorithmic slots per state update; plain instructions of several waves can "
                    "overlap, so both fractions compare kernels and are no end"}


def algorithmic_bytes(w, which="fwd"):
    """Bytes one call must move: x, delta, z read + y written over (B,D,L), Bm and
    Cm read over (B,N,L), plus the small per-channel parameters."""
    e = 4 if w["dtype"] == "fp32" else 2
    bdl = w["batch"] * w["dim"] * w["seqlen"]
    bnl = w["batch"] * w["dstate"] * w["seqlen"]
    par = w["dim"] * (w["dstate"] + 2) * 4
    if which == "fwd":
        return 4 * bdl * e + 2 * bnl * e + par
    if which == "bwd":     # x, delta, z, dout read; dx, ddelta, dz written; Bm, Cm read; dBm, dCm written
        return 7 * bdl * e + 4 * bnl * e + 2 * par
    if which == "bidir":   # pass 1: x, delta read, partial written; pass 2: x, delta, z, partial read, y written
        return (3 + 5) * bdl * e + 4 * bnl * e + 2 * par
    raise ValueError(which)


def upload(s, dtype):
    import numpy as np
    import torch
    from paper_2506_15976_amd.inputs import fp32_to_bf16_bits
    out = {}
    for k in FWD_KEYS + ("dout",):
        v = s.get(k)
        if v is None:
            out[k] = None
        elif dtype == "bf16" and v.ndim == 3:
            out[k] = torch.from_numpy(fp32_to_bf16_bits(v).view(np.int16)).view(torch.bfloat16).to("cuda:0")
        else:
            out[k] = torch.from_numpy(v).to("cuda:0")
    return out


def device_inputs(w, seed):
    """One input set drawn on the GPU with the recipe of paper_2506_15976_amd.inputs
    (x, Bm, Cm, z, dout ~ N(0,1); delta = 0.5 N(0,1); delta_bias = log(expm1(U[1e-3,
    0.1])); A[d,n] = -(n+1); Dskip = 1), rounded to the storage type.  Used for the
    rotation sets, which only have to be distinct memory with the same statistics."""
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    B, D, N, L = w["batch"], w["dim"], w["dstate"], w["seqlen"]
    dt = torch.float32 if w["dtype"] == "fp32" else torch.bfloat16
    rn = lambda *shape: torch.randn(*shape, device="cuda:0", generator=g)
    s = dict(x=rn(B, D, L).to(dt), delta=(0.5 * rn(B, D, L)).to(dt),
             A=-torch.arange(1, N + 1, device="cuda:0", dtype=torch.float32).repeat(D, 1).contiguous(),
             Bm=rn(B, N, L).to(dt), Cm=rn(B, N, L).to(dt), Dskip=torch.ones(D, device="cuda:0"),
             z=rn(B, D, L).to(dt),
             delta_bias=torch.log(torch.expm1(torch.rand(D, device="cuda:0", generator=g) * 0.099 + 1e-3)),
             dout=rn(B, D, L).to(dt))
    return s


def time_calls(calls, steps, warmup, per_launch=False):
    """Run `calls[i % len]()` warmup + steps times on the current stream.  Returns the
    average milliseconds per step from HIP events around the whole timed region and,
    with per_launch, also mean / median / min of per-launch durations from an event
    pair around every launch (without the gaps between dependent launches)."""
    import torch
    for i in range(warmup):
        calls[i % len(calls)]()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for i in range(steps):
        calls[i % len(calls)]()
    e1.record()
    torch.cuda.synchronize()
    region = e0.elapsed_time(e1) / steps
    if not per_launch:
        return region
    n = min(steps, 200)
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(n)]
    for i in range(n):
        ev[i][0].record()
        calls[i % len(calls)]()
        ev[i][1].record()
    torch.cuda.synchronize()
    per = sorted(a.elapsed_time(b) for a, b in ev)
    return region, {"mean": sum(per) / n, "median": per[n // 2], "min": per[0]}


def measure_workload(lb, lib, name, w, sets, steps, warmup, with_bwd, per_launch=False, grid=None):
    """Times lbscan_fwd, lbscan_bidir_fwd, lbscan_bwd (alone, and after a forward call
    that saved its checkpoints) on the rotating input sets.  Returns a dict of results
    (times in ms)."""
    import torch
    from paper_2506_15976_amd import binding
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    nsets = len(sets)
    ys = [torch.empty_like(s["x"]) for s in sets]
    mk = lambda s, **kw: lb.make_args(**{k: s[k] for k in FWD_KEYS}, grid=grid, **kw)
    fwd_args = [mk(s, window=w["window"], y=y) for s, y in zip(sets, ys)]
    need = max(lb.lbscan_workspace_bytes(fwd_args[0], w) for w in (binding.WS_FWD, binding.WS_FWD_ORDER))
    ws_fwd = torch.empty(max(need // 4, 1), dtype=torch.float32, device="cuda:0")
    for ar in fwd_args:
        ar.workspace, ar.workspace_bytes = ws_fwd.data_ptr(), need
    fwd_calls = [(lambda ar=ar: lib.lbscan_fwd(ctypes.byref(ar), stream)) for ar in fwd_args]
    rc = fwd_calls[0]()
    assert rc == 0, f"lbscan_fwd failed: {rc}"
    out = {}
    if per_launch:
        out["fwd_ms"], out["fwd_launch"] = time_calls(fwd_calls, steps, warmup, per_launch=True)
        out["fwd_cache_hot_ms"] = time_calls(fwd_calls[:1], steps, warmup)
        # the GPU runs slower for about 20 ms after an idle spell: a few steps after a few warmup
        # steps lie inside them, 200 calls after 300 do not
        out["fwd_settled_ms"] = time_calls(fwd_calls, 200, 300)
    else:
        out["fwd_ms"] = time_calls(fwd_calls, steps, warmup)
    # the same call with the wave-tile kernels forced (rows cut into segments), where
    # the library itself picks the chunk-per-lane kernel
    out["fwd_wave_tiles_ms"] = None
    if w["seqlen"] >= 1024 and w["batch"] * w["dim"] >= 1536 and grid is None:
        lb.lbscan_set_option("mapping", 1)
        try:
            out["fwd_wave_tiles_ms"] = time_calls(fwd_calls, max(steps // 2, 1), max(warmup // 2, 1))
        finally:
            lb.lbscan_set_option("mapping", 0)

    # two-pass global bi-directional scan on the same inputs (direction b = the
    # (B,D,L)/(B,N,L) tensors of the next rotation slot: both passes read distinct memory);
    # stored order only
    if grid is not None:
        out["bidir_ms"] = None
    bi_f = [] if grid is not None else [mk(s, window=1, y=y) for s, y in zip(sets, ys)]
    if bi_f:
        bi_b = [mk(sets[(i + 1) % nsets], window=1) for i in range(nsets)]
        need = lb.lbscan_workspace_bytes(bi_f[0], binding.WS_BIDIR)
        ws = torch.empty(max(need // 4, 1), dtype=torch.float32, device="cuda:0")
        for ar in bi_f:
            ar.workspace, ar.workspace_bytes = ws.data_ptr(), need
        bi_calls = [(lambda f=f, b=b: lib.lbscan_bidir_fwd(ctypes.byref(f), ctypes.byref(b), stream))
                    for f, b in zip(bi_f, bi_b)]
        rc = bi_calls[0]()
        assert rc == 0, f"lbscan_bidir_fwd failed: {rc}"
        out["bidir_ms"] = time_calls(bi_calls, max(steps // 2, 1), max(warmup // 2, 1))

    out["bwd_ms"] = out["fwd_plus_bwd_ms"] = None
    if with_bwd:
        g_args = []
        for s_, ar in list(zip(sets, fwd_args))[:2]:     # two sets are enough to defeat the cache here
            outs = [torch.empty_like(s_["x"]) for _ in range(3)] + [torch.empty_like(s_["Bm"]) for _ in range(2)] + \
                   [torch.empty_like(s_["A"]), torch.empty_like(s_["Dskip"]), torch.empty_like(s_["delta_bias"])]
            g_args.append((ar, s_["dout"], outs))
        bneed = max(lb.lbscan_workspace_bytes(fwd_args[0], w) for w in (binding.WS_BWD, binding.WS_BWD_ORDER))
        ws_bwd = torch.empty(max(bneed // 4, 1), dtype=torch.float32, device="cuda:0")

        def bwd_call(ar, dout, outs):
            ar.workspace, ar.workspace_bytes = ws_bwd.data_ptr(), bneed
            rc_ = lib.lbscan_bwd(ctypes.byref(ar), dout.data_ptr(), *[o.data_ptr() for o in outs], stream)
            ar.workspace, ar.workspace_bytes = ws_fwd.data_ptr(), ws_fwd.numel() * 4
            return rc_
        assert bwd_call(*g_args[0]) == 0, "lbscan_bwd failed"
        out["bwd_ms"] = time_calls([(lambda g=g: bwd_call(*g)) for g in g_args],
                                   max(steps // 4, 1), max(warmup // 4, 1))
        # training step: the forward call saves its checkpoints for the backward call
        sneed = lb.lbscan_workspace_bytes(fwd_args[0], binding.WS_SAVED)
        saved = torch.empty(max(sneed // 4, 1), dtype=torch.float32, device="cuda:0")

        def train_call(ar, dout, outs):
            if sneed:
                ar.saved_state, ar.saved_state_bytes = saved.data_ptr(), sneed
            r1 = lib.lbscan_fwd(ctypes.byref(ar), stream)
            r2 = bwd_call(ar, dout, outs)
            ar.saved_state, ar.saved_state_bytes = None, 0
            return r1 or r2
        assert train_call(*g_args[0]) == 0, "training step failed"
        out["fwd_plus_bwd_ms"] = time_calls([(lambda g=g: train_call(*g)) for g in g_args],
                                            max(steps // 4, 1), max(warmup // 4, 1))
        # the plain Mamba scan (window 1) trained the same way: what the local backward
        # scan adds to a training step (paper Appendix B compares the two kernels)
        keepw = [ar.window for ar, _, _ in g_args]
        for ar, _, _ in g_args:
            ar.window = 1
        assert train_call(*g_args[0]) == 0
        out["fwd_plus_bwd_window1_ms"] = time_calls([(lambda g=g: train_call(*g)) for g in g_args],
                                                    max(steps // 4, 1), max(warmup // 4, 1))
        for (ar, _, _), m in zip(g_args, keepw):
            ar.window = m
    return out


def summarize(name, w, r):
    """Per-workload record of the "workloads" map."""
    fb, bb = algorithmic_bytes(w, "fwd"), algorithmic_bytes(w, "bwd")
    tokens = w["batch"] * w["seqlen"]
    su = tokens * w["dim"] * w["dstate"]
    rec = {
        "shape": {k: w[k] for k in ("batch", "dim", "dstate", "seqlen", "window")},
        "storage": w["dtype"], "arithmetic": "f32",
        "fwd_ms": r["fwd_ms"], "fwd_tokens_per_s": tokens / (r["fwd_ms"] * 1e-3),
        "fwd_algorithmic_bytes": fb, "fwd_gbps": fb / (r["fwd_ms"] * 1e-3) / 1e9,
        "fwd_hbm_frac": fb / (r["fwd_ms"] * 1e-3) / 1e9 / HBM_PEAK_GBPS,
        "fwd_alu_frac": su / (r["fwd_ms"] * 1e-3) / (VALU_PEAK_LANE_OPS / algorithmic_slots(w["window"])),
        "fwd_traffic_bytes": profile_figure("traffic", name),
        "two_pass_bidir_ms": r["bidir_ms"],
        "speedup_vs_two_pass_bidir": None if r["bidir_ms"] is None else r["bidir_ms"] / r["fwd_ms"],
    }
    if r.get("fwd_wave_tiles_ms") is not None:
        rec["fwd_wave_tiles_ms"] = r["fwd_wave_tiles_ms"]
    if r.get("bwd_ms") is not None:
        rec.update({
            "bwd_ms": r["bwd_ms"], "bwd_algorithmic_bytes": bb,
            "bwd_gbps": bb / (r["bwd_ms"] * 1e-3) / 1e9,
            "bwd_hbm_frac": bb / (r["bwd_ms"] * 1e-3) / 1e9 / HBM_PEAK_GBPS,
            "fwd_plus_bwd_ms": r["fwd_plus_bwd_ms"],
            "fwd_plus_bwd_window1_ms": r.get("fwd_plus_bwd_window1_ms"),
        })
    return rec


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=400)
    ap.add_argument("--warmup", type=int, default=40)
    ap.add_argument("--workload", default="vim_small", help="the workload of the headline figures")
    ap.add_argument("--shape", default="", help="B,D,N,L,M[,dtype]: time a custom shape instead of a named workload")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-bwd", action="store_true", help="skip the backward-pass timings")
    ap.add_argument("--no-others", action="store_true", help="only the headline workload (profiling runs)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain 1 GiB elementwise copy kernel, for scaling rocprofv3 FETCH_SIZE / WRITE_SIZE")
    ap.add_argument("--segments", type=int, default=0, help="force the number of row segments (tuning)")
    ap.add_argument("--sets", type=int, default=0, help="independent input sets to rotate over (0: enough for 640 MB)")
    a = ap.parse_args()
    if a.gpus != 1:
        print("bench.py: this build runs on one GPU only (the scan needs no cross-GPU exchange in "
              "forward: rows shard over batch or channels); run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    import paper_2506_15976_amd as lb
    from paper_2506_15976_amd.inputs import BASE_SEED, WORKLOADS, make_inputs, make_workload

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    if a.copy_calibration:
        src = torch.ones(1 << 28, dtype=torch.float32, device="cuda:0")      # 1 GiB
        dst = torch.empty_like(src)
        for _ in range(3):
            torch.add(src, 1.0, out=dst)     # one elementwise kernel: reads 1 GiB, writes 1 GiB
        torch.cuda.synchronize()
        del src, dst
    lib = lb.load()
    lb.lbscan_set_option("segments", a.segments)
    if a.shape:
        f = a.shape.split(",")
        w = dict(batch=int(f[0]), dim=int(f[1]), dstate=int(f[2]), seqlen=int(f[3]), window=int(f[4]),
                 dtype=f[5] if len(f) > 5 else "fp32", grad=False, idx=99)
        a.workload = "custom"
    else:
        w = WORKLOADS[a.workload]

    def nsets_for(wl):
        n = a.sets or max(2, int(np.ceil(640e6 / algorithmic_bytes(wl, "fwd"))))
        return min(n, 12)

    # ---- headline workload: set 0 is the named workload drawn on the host (it also feeds
    # the CPU baseline), the other rotation sets are drawn on the GPU
    host0 = (make_workload(a.workload) if not a.shape else
             make_inputs(w["batch"], w["dim"], w["dstate"], w["seqlen"], seed=BASE_SEED + 99, dtype=w["dtype"]))
    if host0.get("dout") is None:
        host0["dout"] = np.random.default_rng(BASE_SEED + 7).standard_normal(host0["x"].shape, dtype=np.float32)
        if w["dtype"] == "bf16":
            from paper_2506_15976_amd.inputs import round_to_bf16
            host0["dout"] = round_to_bf16(host0["dout"])
    nsets = nsets_for(w)
    sets = [upload(host0, w["dtype"])] + [device_inputs(w, BASE_SEED + 100 * (i + 1) + w["idx"])
                                          for i in range(1, nsets)]
    head = measure_workload(lb, lib, a.workload, w, sets, a.steps, a.warmup, not a.no_bwd, per_launch=True)
    del sets
    torch.cuda.empty_cache()

    # ---- the other named workloads
    workloads = {a.workload: summarize(a.workload, w, head)}
    if not a.no_others and not a.shape:
        for name, wl in WORKLOADS.items():
            if name in (a.workload, "tiny"):
                continue
            ss = [device_inputs(wl, BASE_SEED + 100 * (i + 1) + wl["idx"]) for i in range(nsets_for(wl))]
            r = measure_workload(lb, lib, name, wl, ss, max(a.steps // 2, 1), max(a.warmup // 2, 1), not a.no_bwd)
            workloads[name] = summarize(name, wl, r)
            del ss
            torch.cuda.empty_cache()

        # the vertical scan of the Vim-small token grid (14 x 14 patches, class token last):
        # the same kernels on copies in scanned order (paper Sec. 4.5 / Appendix D)
        wl = WORKLOADS["vim_small"]
        ss = [device_inputs(wl, BASE_SEED + 900 + i) for i in range(nsets_for(wl))]
        r = measure_workload(lb, lib, "vim_small_columns", wl, ss, max(a.steps // 2, 1), max(a.warmup // 2, 1),
                             not a.no_bwd, grid=(14, 14, 0))
        workloads["vim_small_columns"] = dict(summarize("vim_small_columns", wl, r),
                                              scan_order="columns of the 14 x 14 grid, class token last")
        del ss
        torch.cuda.empty_cache()

    # the block's pre-scan step (depthwise causal conv + SiLU, width 4) on x tensors of the
    # headline shape: an HBM-bound kernel of the same library, timed as extra information
    xs = [torch.randn(w["batch"], w["dim"], w["seqlen"], device="cuda:0").to(
        torch.float32 if w["dtype"] == "fp32" else torch.bfloat16) for _ in range(3)]
    ysc = [torch.empty_like(x) for x in xs]
    wconv = torch.randn(w["dim"], 4, device="cuda:0") * 0.5
    bconv = torch.randn(w["dim"], device="cuda:0")
    conv_calls = [(lambda x_=x_, y_=y_: lb.lbscan_conv1d_fwd(x_, wconv, bconv, out=y_)) for x_, y_ in zip(xs, ysc)]
    ms_conv = time_calls(conv_calls, max(a.steps // 4, 1), max(a.warmup // 4, 1))
    conv_bytes = 2 * w["batch"] * w["dim"] * w["seqlen"] * (2 if w["dtype"] == "bf16" else 4)
    del xs, ysc

    ms_fwd = head["fwd_ms"]
    fwd_bytes = algorithmic_bytes(w, "fwd")
    tokens = w["batch"] * w["seqlen"]
    # average launch duration over the timed region (includes the ~5 us gap between
    # dependent launches; an event pair per launch reads slightly more, a kernel trace less)
    gbps = fwd_bytes / (ms_fwd * 1e-3) / 1e9

    cpu = None
    if not a.no_cpu_baseline:
        import oracle
        host = {k: host0.get(k) for k in FWD_KEYS}
        # bounded sample: whole batch entries of the same workload, sized for ~2e8 state updates
        su_per_b = w["dim"] * w["dstate"] * w["seqlen"]
        nb = max(1, min(w["batch"], int(2e8 // su_per_b)))
        sub = {k: (v[:nb] if isinstance(v, np.ndarray) and v.ndim == 3 else v) for k, v in host.items()}
        oracle.fwd(**{k: (v[:1] if isinstance(v, np.ndarray) and v.ndim == 3 else v) for k, v in host.items()},
                   window=w["window"])
        t0 = time.perf_counter()
        oracle.fwd(**sub, window=w["window"])
        once = time.perf_counter() - t0
        reps = max(3, int(np.ceil(1.5 / max(once, 1e-4))))       # about 1.5 s of wall time on all cores
        t0 = time.perf_counter()
        for _ in range(reps):
            oracle.fwd(**sub, window=w["window"])
        per_call = (time.perf_counter() - t0) / reps
        # the same loop on one core, on a smaller slice
        threads = oracle.num_threads()
        nb1 = max(1, nb // 8)
        sub1 = {k: (v[:nb1] if isinstance(v, np.ndarray) and v.ndim == 3 else v) for k, v in host.items()}
        oracle.set_num_threads(1)
        t0 = time.perf_counter()
        oracle.fwd(**sub1, window=w["window"])
        one_core = time.perf_counter() - t0
        oracle.set_num_threads(threads)
        cpu = {"value": nb * w["seqlen"] / per_call, "unit": "tokens/s", "cores": threads,
               "kind": "oracle",
               "sample": f"fp64 oracle forward on {nb} of {w['batch']} batch entries of {a.workload}, "
                         f"mean of {reps} calls, {per_call:.4f} s per call",
               "one_core_value": nb1 * w["seqlen"] / one_core,
               "one_core_sample": f"{nb1} batch entries, one call, {one_core:.3f} s"}

    fl = head["fwd_launch"]
    line = {
        "metric": "lbscan_fwd_tokens_per_s", "value": tokens / (ms_fwd * 1e-3), "unit": "tokens/s",
        "n_gpus": 1, "steps": a.steps, "warmup": a.warmup, "ms_per_step": ms_fwd,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        # the type the path computes in (storage is the workload's: config and "workloads")
        "dtype": workloads[a.workload]["arithmetic"] if a.workload in workloads else "f32",
        "storage_dtype": w["dtype"], "data": "synthetic",
        "config": {"workload": f"{a.workload}: B={w['batch']} D={w['dim']} N={w['dstate']} L={w['seqlen']} "
                               f"M={w['window']} {w['dtype']} storage, fp32 arithmetic, forward",
                   "input_sets_rotated": nsets},
        "roofline": {"bound": "hbm", "achieved": gbps, "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                     "frac": gbps / HBM_PEAK_GBPS, "traffic": profile_figure("traffic", a.workload),
                     "kernel": FWD_KERNELS.get(a.workload, "wave_fwd_kernel"),
                     "algorithmic_bytes_per_launch": fwd_bytes,
                     "launch_ms": ms_fwd, "launch_ms_event_pairs": fl["mean"],
                     "launch_ms_median": fl["median"], "launch_ms_min": fl["min"]},
        "alu_bound": alu_bound(tokens * w["dim"] * w["dstate"] / (ms_fwd * 1e-3), w["window"], a.workload),
        "cpu_baseline": cpu,
        "speedup_vs_two_pass_bidir": head["bidir_ms"] / ms_fwd,
        "two_pass_bidir_ms": head["bidir_ms"],
        "cache_hot_ms_per_step": head["fwd_cache_hot_ms"],
        "settled_ms_per_step": head["fwd_settled_ms"],
        "settled_note": "the same calls timed after 300 others: the first 150 or so after an idle spell take "
                        "up to 1.3 times as long (value and ms_per_step are of the steps asked for)",
        "bwd_ms": head["bwd_ms"],
        "fwd_plus_bwd_ms": head["fwd_plus_bwd_ms"],
        "fwd_plus_bwd_window1_ms": head.get("fwd_plus_bwd_window1_ms"),
        "bwd_algorithmic_gbps": None if head["bwd_ms"] is None
        else algorithmic_bytes(w, "bwd") / (head["bwd_ms"] * 1e-3) / 1e9,
        "prescan_conv_fwd_ms": ms_conv,
        "prescan_conv_fwd_gbps": conv_bytes / (ms_conv * 1e-3) / 1e9,
        "workloads": workloads,
    }
    print(json.dumps(line))


if __name__ == "__main__":
    main()
