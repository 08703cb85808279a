"""The binding's argument checks (csrc/torch_calls.cpp): what a call refuses it refuses before it asks the device for
anything, so fake device tensors on the CPU reach them."""
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

import paper_1801_02108_amd as sb


def fake(*shape, dtype=torch.float32):
    with FakeTensorMode():
        return torch.empty(shape, dtype=dtype, device="cuda")


def packed(kh, kw, cin, cout, dtype=torch.float32):
    return sb.PackedWeights(torch.empty(16, dtype=torch.uint8), (kh, kw, cin, cout), dtype)


def convolutions(tile, out, stride):
    """The four calls whose output extent is formed from the stride, on tiles of tile x tile pixels and 3x3 weights."""
    t, d, cnt = fake(2, tile, tile, 16), fake(2, out, out, 16), fake(1, dtype=torch.int32)
    return [
        lambda: sb.conv_on_tiles(t, cnt, packed(3, 3, 16, 16), stride=stride),
        lambda: sb.conv_on_tiles_f8(fake(2, tile, tile, 16, dtype=torch.uint8), cnt, packed(3, 3, 16, 16, torch.uint8), stride=stride),
        lambda: sb.conv_on_tiles_backward_data(d, cnt, packed(3, 3, 16, 16), tile, tile, stride=stride),
        lambda: sb.conv_on_tiles_backward_weights(t, d, cnt, 3, stride=stride),
    ]


@pytest.mark.parametrize("which", range(4))
def test_a_stride_of_zero_is_an_error(which):
    with pytest.raises(ZeroDivisionError):
        convolutions(6, 4, 0)[which]()


@pytest.mark.parametrize("which", (2, 3))
def test_extents_of_tiles_smaller_than_the_kernel_round_down(which):
    """floor((2 - 3) / 2) + 1 = 0: gradients of one pixel do not belong to such tiles."""
    with pytest.raises(AssertionError):
        convolutions(2, 1, 2)[which]()
