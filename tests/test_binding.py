"""The binding's argument checks (csrc/torch_calls.cpp): what a call refuses it refuses before it asks the device for
anything, so fake device tensors on the CPU reach them."""
import ctypes
import weakref

import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from torch.utils._python_dispatch import TorchDispatchMode

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


class _Reached(Exception):
    pass


class _AtFirstAllocation(TorchDispatchMode):
    """Calls `look` and ends the call under test where it allocates its first result."""

    def __init__(self, look):
        super().__init__()
        self.look = look

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        if func is not torch.ops.aten.empty.memory_format:
            return func(*args, **(kwargs or {}))
        self.look()
        raise _Reached


def test_weights_that_only_an_iterator_holds_live_until_the_call_is_over():
    g, _, _, _ = sb.geometry(16, 16, 3, 1, 4)
    tiles, idx, cnt = fake(2, 6, 6, 16), fake(2, 3, dtype=torch.int32), fake(1, dtype=torch.int32)
    made = [packed(*shape) for shape in ((1, 1, 16, 8), (3, 3, 8, 8), (1, 1, 8, 16))]
    refs, alive = [weakref.ref(w) for w in made], []

    def weights():
        while made:
            yield made.pop(0)
            yield None                                # this call takes a missing bias

    with pytest.raises(_Reached), _AtFirstAllocation(lambda: alive.extend(r() is not None for r in refs)):
        sb.bottleneck_forward_keep_on_tiles(tiles, idx, cnt, g, 16, 16, weights())
    assert alive == [True] * 3


@pytest.mark.parametrize("n", (5, 7))
def test_a_wrong_number_of_weights_is_an_error(n):
    g, _, _, _ = sb.geometry(16, 16, 3, 1, 4)
    tiles, idx, cnt = fake(2, 6, 6, 16), fake(2, 3, dtype=torch.int32), fake(1, dtype=torch.int32)
    with pytest.raises(ValueError):
        sb.bottleneck_forward_keep_on_tiles(tiles, idx, cnt, g, 16, 16, [None] * n)


def test_a_geometry_is_a_geom_and_nothing_of_its_size():
    g, _, _, _ = sb.geometry(16, 16, 3, 1, 4)
    mask, idx, cnt = fake(1, 16, 16), fake(16, 3, dtype=torch.int32), fake(1, dtype=torch.int32)

    def reduce(geom):
        sb.reduce_mask(mask, geom, 1, 0.0, None, cnt, None)

    for wrong in (bytes(g), bytearray(g), (ctypes.c_int * 8)(*g.astuple()), g.astuple(), 7):
        with pytest.raises(TypeError, match="Geom"):
            reduce(wrong)
    with pytest.raises(sb.SbnetError) as e:
        reduce(None)
    assert e.value.code == sb.EINVAL
    for right in (g, type("Derived", (sb.Geom,), {})(*g.astuple()), ctypes.pointer(g), ctypes.byref(g)):
        with pytest.raises(_Reached), _AtFirstAllocation(lambda: None):
            reduce(right)
