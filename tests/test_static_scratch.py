"""lbscan_fwd_static holds what a call's scratch is, up to 8 MiB: a finer cut of the rows
must not push sizes over that which a coarser cut keeps inside.  Host logic only."""
import random

import pytest

from paper_2506_15976_amd import binding


def _need(B, D, N, L, window, dtype):
    a = binding.LbscanArgs(B, D, N, L, window, dtype)
    return binding.lbscan_workspace_bytes(a, binding.WS_FWD)


def _coarse(B, D, N, L):
    """Bytes of the fp32 first pass in bf16 and of the summaries of rows cut for 768 blocks of
    64 rows (uncut from 256 such row blocks on), segments of 64 tokens at least."""
    blocks, tiles = (D + 63) // 64 * B, (L + 31) // 32
    segments = 1
    if blocks < 256:
        per = max(2, -(-tiles // -(-768 // blocks)))
        segments = -(-tiles // per)
    return B * D * L * 4 + (segments * B * D * (N + 1) * 4 if segments > 1 else 0)


@pytest.mark.parametrize("shape, window", [((128, 32, 16, 400), 3), ((128, 32, 16, 400), 14), ((48, 5, 16, 8192), 3)])
def test_sizes_next_to_a_first_pass_that_nearly_fills_the_array(shape, window):
    assert _need(*shape, window, 1) <= binding.STATIC_SCRATCH_BYTES


def test_what_a_coarse_cut_keeps_inside_stays_inside():
    rng = random.Random(5)
    near = 0
    for _ in range(20000):
        N = rng.choice([1, 4, 8, 13, 16])
        D = int(2 ** rng.uniform(0, 11))
        L = int(2 ** rng.uniform(5, 16))
        B = max(1, int(binding.STATIC_SCRATCH_BYTES * rng.uniform(0.5, 1.0) / (4 * D * L)))
        if _coarse(B, D, N, L) > binding.STATIC_SCRATCH_BYTES:
            continue
        near += 1
        need = _need(B, D, N, L, 3, 1)
        assert need <= binding.STATIC_SCRATCH_BYTES, (B, D, N, L, need)
    assert near > 1000


def test_compiled_windows_and_fp32_always_fit():
    rng = random.Random(6)
    for _ in range(20000):
        B, D, L = (int(2 ** rng.uniform(0, top)) for top in (9, 11, 18))
        for window, dtype in ((4, 0), (4, 1), (3, 0)):
            need = _need(B, D, 16, L, window, dtype)
            assert need <= binding.STATIC_SCRATCH_BYTES, (B, D, L, window, dtype, need)
