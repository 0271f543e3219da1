"""What make_args does with arguments that the library refuses: LbscanError, whatever is
wrong.  Host logic only: the tensors are stand-ins that claim to be on a device."""
import pytest
import torch

from paper_2506_15976_amd import binding


class DeviceTensor:
    """Shape, type and address of a contiguous device tensor; nothing reads it."""
    is_cuda = True

    def __init__(self, *shape):
        self.shape, self.dtype = torch.Size(shape), torch.float32

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 256


class Stream:
    cuda_stream = 0


def _inputs(B=1, D=4, N=16, L=8):
    row, mat = DeviceTensor(B, D, L), DeviceTensor(B, N, L)
    return dict(x=row, delta=row, A=DeviceTensor(D, N), Bm=mat, Cm=mat)


@pytest.mark.parametrize("name", ["delta", "Bm", "Cm"])
def test_a_required_tensor_left_out(name):
    s = dict(_inputs(), **{name: None})
    assert not getattr(binding.make_args(**s, window=4), name)       # sizes can be asked for without it
    with pytest.raises(binding.LbscanError) as e:
        binding.lbscan_fwd(**s, window=4, out=s["x"], stream=Stream())
    assert e.value.code == binding.EINVAL


@pytest.mark.parametrize("sizes", [dict(B=1 << 31, D=0), dict(D=0, L=1 << 31), dict(D=0, N=1 << 31)])
def test_sizes_beyond_32_bits(sizes):
    """Empty tensors with an edge that the struct cannot hold."""
    with pytest.raises(binding.LbscanError) as e:
        s = _inputs(**sizes)
        binding.lbscan_fwd(**s, window=4, out=s["x"], stream=Stream())
    assert e.value.code == binding.EINVAL
