"""Workloads of the library as its users run them, for timing one tree against another.

A case names what is called ("op"), the sizes, the storage type and the options:

    op "fwd"          inference: one forward scan
    op "train"        one training step of the scan through autograd: forward, then the
                      gradients of every input
    op "columns"      inference over a token grid scanned column by column
    op "columns_train"  the same with its gradients (the two library calls, as a
                      multi-direction block's own autograd function makes them)
    op "stream"       one piece of a long sequence: the state enters and leaves the call
    op "conv_train"   one training step of the pre-scan convolution

The sizes are those of the package's named workloads (inputs.WORKLOADS); value
distributions are theirs too: x, Bm, Cm, z, dout ~ N(0,1), delta = 0.5 N(0,1),
softplus of delta + bias with time steps of 1e-3 .. 0.1, A[d,n] = -(n+1), Dskip = 1.
"""
import math

import torch

import paper_2506_15976_amd as lb
from paper_2506_15976_amd.autograd import causal_conv1d_silu, lb_selective_scan
from paper_2506_15976_amd.inputs import WORKLOADS


def _workload(name, op, *, label=None, dtype=None, window=None, reverse=False, batch=None,
              seqlen=None, grid=None):
    w = WORKLOADS[name]
    c = dict(name=label or "%s_%s" % (name, op), op=op, batch=batch or w["batch"], dim=w["dim"],
             dstate=w["dstate"], seqlen=seqlen or w["seqlen"], window=window or w["window"],
             dtype=dtype or w["dtype"], reverse=reverse)
    if grid:
        c.update(grid_h=grid[0], grid_w=grid[1], grid_prefix=grid[2])
    return c


def listed():
    return [
        # the smallest call: one short sequence of one sample, where latency counts
        _workload("tiny", "fwd"),
        # ImageNet inference, small model, stored in bf16; every second layer of the network
        # scans the reversed sequence; window 8 is the paper's rule for 197 tokens.  Rows
        # of an odd length in a 2-byte type: every other row starts at an odd element
        _workload("vim_tiny", "fwd", label="vim_tiny_fwd_bf16", dtype="bf16", window=8, reverse=True),
        # ImageNet inference and training in fp32 (14 x 14 patches and a class token)
        _workload("vim_small", "fwd"),
        _workload("vim_small", "train"),
        # dense prediction on 1024 x 1024 images, stored in bf16
        _workload("hires_4096", "fwd"),
        _workload("hires_4096", "train"),
        # a whole-slide bag: one very long sequence, few channels
        _workload("wsi_bag", "fwd"),
        _workload("wsi_bag", "train"),
        # the vertical scans of multi-direction models, class token last
        _workload("vim_small", "columns", grid=(14, 14, 0)),
        _workload("vim_small", "columns_train", grid=(14, 14, 0)),
        # a bag too long for one call is taken in pieces, each starting from the last one's state
        _workload("wsi_bag", "stream", label="wsi_bag_stream_8192", seqlen=8192),
        # the step before the scan
        _workload("vim_small", "conv_train"),
    ]


# State updates (batch x dim x dstate x seqlen) a drawn case may have: the largest listed one's.
_MOST = 8 * 768 * 16 * 4096


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["fwd", "fwd", "fwd", "train", "train", "train", "columns", "columns_train", "stream",
                     "conv_train"])
    c = dict(op=op, dstate=16, window=rng.choice([4, 4, 8, 8, 16, 1, 2]), dtype=rng.choice(["fp32", "bf16"]),
             reverse=rng.random() < 0.4)
    if rng.random() < 0.125:
        c["dstate"] = 8
    if op in ("columns", "columns_train"):
        h, w = rng.randint(7, 32), rng.randint(7, 32)
        prefix = rng.randint(0, 1)
        c.update(batch=_log_uniform(rng, 4, 128), dim=8 * _log_uniform(rng, 12, 96), grid_h=h, grid_w=w,
                 grid_prefix=prefix, seqlen=prefix + h * w + rng.randint(0, 1))
        most = 128 * 768 * 16 * 197                       # the listed ones' size
    else:
        most = _MOST
        family = "pieces" if op == "stream" else rng.choice(["images", "images", "dense", "bags"])
        if family == "images":      # batches of short rows
            c.update(batch=_log_uniform(rng, 1, 128), dim=8 * _log_uniform(rng, 8, 96), seqlen=_log_uniform(rng, 50, 1025))
        elif family == "dense":     # few images, thousands of tokens each
            c.update(batch=_log_uniform(rng, 1, 8), dim=8 * _log_uniform(rng, 24, 96), seqlen=_log_uniform(rng, 1024, 4608))
        elif family == "bags":      # whole-slide bags
            c.update(batch=1, dim=rng.choice([128, 192, 256, 384, 512]), seqlen=_log_uniform(rng, 4096, 65536))
        else:                       # pieces of a bag: whole windows, or they would not add up
            c.update(batch=1, dim=rng.choice([128, 192, 256, 384, 512]), seqlen=16 * _log_uniform(rng, 64, 1024))
    while c["batch"] * c["dim"] * 16 * c["seqlen"] > most:
        if c["batch"] > 1:
            c["batch"] = (c["batch"] + 1) // 2
        else:
            c["dim"] = max(8, c["dim"] // 16 * 8)
    return c


def _tensors(case, seed):
    """The inputs of one call on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    B, D, N, L = case["batch"], case["dim"], case["dstate"], case["seqlen"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(*shape):
        return torch.randn(*shape, device="cuda", generator=g)

    if case["op"] == "conv_train":
        return dict(x=normal(B, D, L).to(dt), weight=normal(D, 4) / 2, bias=normal(D) / 4,
                    dout=normal(B, D, L).to(dt))
    step = torch.empty(D, device="cuda").uniform_(1e-3, 0.1, generator=g)
    s = dict(x=normal(B, D, L).to(dt), delta=(0.5 * normal(B, D, L)).to(dt),
             A=-torch.arange(1, N + 1, device="cuda", dtype=torch.float32).repeat(D, 1),
             Bm=normal(B, N, L).to(dt), Cm=normal(B, N, L).to(dt), Dskip=torch.ones(D, device="cuda"),
             z=normal(B, D, L).to(dt), delta_bias=torch.log(torch.expm1(step)))
    if case["op"].endswith("train"):
        s["dout"] = normal(B, D, L).to(dt)
    if case["op"] == "stream":
        s["h0"] = normal(B, D, N)
    return s


def prepare(case, seed):
    t = _tensors(case, seed)
    if case["op"] in ("train", "conv_train"):
        for k, v in t.items():
            if k != "dout":
                v.requires_grad_(True)
    return dict(case=case, tensors=t)


def run(state):
    case, t = state["case"], state["tensors"]
    op = case["op"]
    options = dict(window=case["window"], reverse=case["reverse"])
    if op == "fwd":
        return lb.lbscan_fwd(**t, **options)
    if op == "stream":
        return lb.lbscan_fwd(**t, **options, return_state=True)
    if op == "train":
        inputs = {k: v for k, v in t.items() if k != "dout"}
        out = lb_selective_scan(**inputs, **options)
        return out, torch.autograd.grad(out, list(inputs.values()), t["dout"])
    if op == "conv_train":
        inputs = {k: v for k, v in t.items() if k != "dout"}
        out = causal_conv1d_silu(**inputs, reverse=case["reverse"])
        return out, torch.autograd.grad(out, list(inputs.values()), t["dout"])
    options["grid"] = (case["grid_h"], case["grid_w"], case["grid_prefix"])
    if op == "columns":
        return lb.lbscan_fwd(**t, **options)
    inputs = {k: v for k, v in t.items() if k != "dout"}
    # (the size of the checkpoint buffer does not depend on the scan order)
    saved = lb.lbscan_saved_state(t["x"], t["A"], window=case["window"])
    out = lb.lbscan_fwd(**inputs, **options, saved_state=saved)
    return out, lb.lbscan_bwd(**inputs, **options, dout=t["dout"], saved_state=saved)


def work(case):
    B, D, N, L = case["batch"], case["dim"], case["dstate"], case["seqlen"]
    e = 2 if case["dtype"] == "bf16" else 4
    row, mat, par = B * D * L * e, B * N * L * e, D * (N + 2) * 4
    if case["op"] == "conv_train":
        # x, dout in; y, dx out; four taps, their gradients, SiLU and its derivative
        return dict(bytes=4 * row + 2 * D * 5 * 4, flops=B * D * L * 44)
    updates = B * D * N * L
    # per state update: dt A, exp, u, f, the local backward state and its sum, y
    flops, size = 12 * updates, 4 * row + 2 * mat + par
    if case["op"] == "stream":
        size += 2 * B * D * N * 4
    if case["op"].endswith("train"):
        # dout in; dx, ddelta, dz, dBm, dCm out
        flops, size = flops + 30 * updates, size + 4 * row + 2 * mat + par
    return dict(bytes=size, flops=flops)


def tolerance(case):
    if case["dtype"] == "bf16":
        return {"rel": 6e-3, "max": 0.03}
    return {"rel": 4e-6, "max": 2e-4}


def _scan64(a, u):
    """f_t = a_t f_{t-1} + u_t from f_{-1} = 0 along the last axis, by doubling; also the products of a."""
    s, L = 1, a.shape[-1]
    while s < L:
        u = torch.cat([u[..., :s], u[..., s:] + a[..., s:] * u[..., :-s]], -1)
        a = torch.cat([a[..., :s], a[..., s:] * a[..., :-s]], -1)
        s *= 2
    return u, a


def _lbscan64(window, x, delta, A, Bm, Cm, Dskip, z, delta_bias, h0=None):
    """The definition (include/lbscan.h) in the scanned order, 64 bits: the output and the leaving state."""
    L = x.shape[-1]
    dt = torch.nn.functional.softplus(delta + delta_bias[:, None])
    a = torch.exp(dt[:, :, None] * A[:, :, None])                        # (B, D, N, L)
    u = dt[:, :, None] * Bm[:, None] * x[:, :, None]
    f, prod = _scan64(a, u)
    if h0 is not None:
        f = f + prod * h0[..., None]
    pad = -L % window
    aw, uw = (torch.nn.functional.pad(v, (0, pad)).unflatten(-1, (-1, window)) for v in (a, u))
    g = [torch.zeros_like(uw[..., 0])]
    for t in range(window - 2, -1, -1):
        g.append(aw[..., t] * (g[-1] + uw[..., t + 1]))
    g = torch.stack(g[::-1], -1).flatten(-2)[..., :L]
    y = (Cm[:, None] * (f + g)).sum(2) + Dskip[:, None] * x
    return y * torch.nn.functional.silu(z), f[..., -1]


def exact(case, seed):
    t = {k: v.double() for k, v in _tensors(case, seed).items()}
    op, L = case["op"], case["seqlen"]
    if op == "conv_train":
        flip = (lambda v: v.flip(-1)) if case["reverse"] else (lambda v: v)
        x, weight, bias = (t[k].requires_grad_(True) for k in ("x", "weight", "bias"))
        pre = torch.nn.functional.pad(flip(x), (3, 0))
        pre = sum(weight[:, k, None] * pre[..., k:k + L] for k in range(4)) + bias[:, None]
        out = flip(torch.nn.functional.silu(pre))
        return out.detach(), torch.autograd.grad(out, [x, weight, bias], t["dout"])
    order = torch.arange(L, device="cuda")
    if op.startswith("columns"):
        h, w, first = case["grid_h"], case["grid_w"], case["grid_prefix"]
        order[first:first + h * w] = order[first:first + h * w].reshape(h, w).t().flatten()
    if case["reverse"]:
        order = order.flip(0)
    back = order.argsort()
    along = [k for k in ("x", "delta", "Bm", "Cm", "z", "dout") if k in t]
    for k in along:
        t[k] = t[k][..., order]
    # slices of the batch and the channels, small enough for the doubling's steps
    B, D, N = case["batch"], case["dim"], case["dstate"]
    most = 32 << 20
    nb = max(1, min(B, most // (D * N * L)))
    nd = max(1, min(D, most // (nb * N * L)))
    dout = t.pop("dout", None)
    out = torch.empty_like(t["x"])
    state = torch.empty(B, D, N, device="cuda", dtype=torch.float64)
    grads = {k: torch.zeros_like(v) for k, v in t.items()}
    for b in range(0, B, nb):
        for d in range(0, D, nd):
            bs, ds = slice(b, b + nb), slice(d, d + nd)
            where = {k: (bs, ds) if k in ("x", "delta", "z", "h0") else (bs,) if k in ("Bm", "Cm") else (ds,) for k in t}
            part = {k: v[where[k]].clone().requires_grad_(dout is not None) for k, v in t.items()}
            y, left = _lbscan64(case["window"], **part)
            out[bs, ds], state[bs, ds] = y.detach(), left.detach()
            if dout is not None:
                for k, v in zip(part, torch.autograd.grad(y, list(part.values()), dout[bs, ds])):
                    grads[k][where[k]] += v
            del y, left
    out = out[..., back]
    for k in along:
        if k in grads:
            grads[k] = grads[k][..., back]
    if op in ("fwd", "columns"):
        return out
    if op == "stream":
        return out, state
    if op == "train":
        return out, tuple(grads.values())
    return out, {"d" + k: grads[k] for k in ("x", "delta", "z", "Bm", "Cm", "A", "Dskip", "delta_bias")}
