"""The optional scratch of column-order calls near the memory limit, with the device's
memory figures stood in for: an allocation that cannot succeed is tried once, not on
every call."""
import pytest
import torch

from paper_2506_15976_amd import binding

MB = 1 << 20


def _args():
    """Column order, fp32, sizes that copy in both passes: 225 MB and more of scratch."""
    a = binding.LbscanArgs(128, 768, 16, 197, 4, binding.LBSCAN_FP32)
    a.scan_order, a.grid_h, a.grid_w = binding.ORDER_COLUMNS, 14, 14
    return a


@pytest.fixture
def device(monkeypatch):
    """free / reserved / active MB and the process's fraction of 1000 MB; the sizes asked for."""
    class Device:
        free, reserved, active, fraction, looks = 1000, 0, 0, 1.0, 0
    d = Device()
    d.asked = []

    def look(dev=None):
        d.looks += 1
        return d.free * MB, 1000 * MB

    def empty(n, dtype, device):
        d.asked.append(4 * n)
        if 4 * n > (min(d.free, 1000 * d.fraction - d.reserved) + d.reserved - d.active) * MB:
            raise torch.cuda.OutOfMemoryError("stood in for")
        return torch.zeros(8)
    monkeypatch.setattr(torch.cuda, "mem_get_info", look)
    monkeypatch.setattr(torch.cuda, "get_per_process_memory_fraction", lambda dev=None: d.fraction)
    monkeypatch.setattr(torch.cuda, "memory_stats_as_nested_dict", lambda dev=None: {
        "reserved_bytes": {"all": {"current": d.reserved * MB}}, "active_bytes": {"all": {"current": d.active * MB}}})
    monkeypatch.setattr(torch, "empty", empty)
    binding._short_of_memory.clear()
    yield d
    binding._short_of_memory.clear()


@pytest.mark.parametrize("which, larger", [(binding.WS_FWD, binding.WS_FWD_ORDER), (binding.WS_BWD, binding.WS_BWD_ORDER)])
@pytest.mark.parametrize("free, reserved, active, fraction", [
    (10, 900, 780, 1.0),         # the device is full, and so is the allocator's cache
    (900, 200, 80, 0.21),        # the process may not grow
])
def test_a_block_that_cannot_be_had_is_asked_for_once(device, which, larger, free, reserved, active, fraction):
    device.free, device.reserved, device.active, device.fraction = free, reserved, active, fraction
    a, like = _args(), torch.zeros(1)
    need, more = (binding.lbscan_workspace_bytes(a, w) for w in (which, larger))
    assert more > 200 * MB and need < 130 * MB
    base = [need] if need else []
    binding._workspace_for(a, which, like)
    assert device.asked == [more] + base
    for _ in range(3):
        binding._workspace_for(a, which, like)
    assert device.asked == [more] + base * 4
    # room again: in the allocator's cache, then on the device
    device.active, device.fraction = 0, 1.0
    binding._workspace_for(a, which, like)
    assert device.asked[-1] == more
    looks = device.looks
    binding._workspace_for(a, which, like)
    assert device.asked[-1] == more and device.looks == looks


def test_no_look_while_there_is_room(device):
    a = _args()
    for _ in range(2):
        binding._workspace_for(a, binding.WS_BWD, torch.zeros(1))
    assert device.asked == [binding.lbscan_workspace_bytes(a, binding.WS_BWD_ORDER)] * 2 and device.looks == 0
