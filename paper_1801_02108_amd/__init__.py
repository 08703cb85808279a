"""Thin Python binding of libsbnet_hip.so (see include/sbnet.h for the contract of every call).

Argument marshalling only: torch tensors supply device memory and the current stream; every
step of the path runs in the library's HIP kernels.  The marshalling itself is native
(csrc/torch_calls.cpp); ctypes serves the host-only calls and the packing of weights.  There is
no CPU or PyTorch fallback: if a shared library is missing, the first call into it raises.
"""
import ctypes
import importlib
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libsbnet_hip.so")

F32, BF16, F16, U8 = 0, 1, 2, 3
POOL_MAX, POOL_AVG = 0, 1
OK, EINVAL, ECAP, EUNSUPPORTED, EHIP = 0, 1, 2, 3, 4

_DTYPES = {torch.float32: F32, torch.bfloat16: BF16, torch.float16: F16, torch.uint8: U8}


class SbnetError(RuntimeError):
    def __init__(self, code, text):
        super().__init__("sbnet status %d: %s" % (code, text))
        self.code = code


class Tuning(ctypes.Structure):
    """sbnet_tuning: the compute-tile choices the kernels make from the device-side count of active blocks."""
    _fields_ = [(n, ctypes.c_int) for n in (
        "unit_small_item_cost_eighths", "conv3_small_item_cost_eighths", "wgrad_split_factor_3x3", "wgrad_split_factor_1x1")]

    def asdict(self):
        return {n: getattr(self, n) for n, _ in self._fields_}


class Geom(ctypes.Structure):
    """sbnet_geom: block extent, stride, origin and count along h and w."""
    _fields_ = [(n, ctypes.c_int) for n in (
        "bsize_h", "bsize_w", "bstride_h", "bstride_w", "boffset_h", "boffset_w", "bcount_h", "bcount_w")]

    def astuple(self):
        return tuple(getattr(self, n) for n, _ in self._fields_)


_lib = None
_vp, _ci, _sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t
_gp = ctypes.POINTER(Geom)

_SIGNATURES = {
    "sbnet_last_error": (ctypes.c_char_p, []),
    "sbnet_set_tuning": (_ci, [ctypes.POINTER(Tuning)]),
    "sbnet_get_tuning": (_ci, [ctypes.POINTER(Tuning)]),
    "sbnet_geometry": (_ci, [_ci] * 8 + [_gp, _gp, ctypes.POINTER(_ci), ctypes.POINTER(_ci)]),
    "sbnet_coarse_geometry": (_ci, [_gp, _ci, _gp]),
    "sbnet_workspace_bytes": (_sz, [_ci, _gp]),
    "sbnet_reduce_mask": (_ci, [_vp, _ci, _ci, _ci, _ci, _gp, _ci, ctypes.c_float, _vp, _vp, _ci, _vp, _sz, _vp]),
    "sbnet_reduce_mask_static": (_ci, [_vp, _ci, _ci, _ci, _ci, _gp, _ci, ctypes.c_float, _vp, _vp, _ci, _vp]),
    "sbnet_read_count": (_ci, [_vp, _ci, ctypes.POINTER(_ci), _vp]),
    "sbnet_sparse_gather": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _vp, _vp]),
    "sbnet_sparse_scatter": (_ci, [_vp, _ci, _vp, _vp, _ci, _gp, _vp, _ci, _ci, _ci, _ci, _ci, _vp]),
    "sbnet_sparse_gather_chw": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _vp, _vp]),
    "sbnet_sparse_scatter_chw": (_ci, [_vp, _ci, _vp, _vp, _ci, _gp, _vp, _ci, _ci, _ci, _ci, _ci, _vp]),
    "sbnet_gather_backward_workspace_bytes": (_sz, [_ci, _gp]),
    "sbnet_sparse_gather_backward": (_ci, [_vp, _ci, _vp, _vp, _ci, _gp, _vp, _ci, _ci, _ci, _ci, _vp, _sz, _vp]),
    "sbnet_bn_stats_workspace_bytes": (_sz, [_ci, _ci]),
    "sbnet_sparse_bn_stats": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _vp, _vp, _vp, _sz, _vp]),
    "sbnet_sparse_bn_apply": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _vp, _vp, _vp, _vp, ctypes.c_float,
                                    _ci, _vp, _vp]),
    "sbnet_bn_backward_workspace_bytes": (_sz, [_ci, _ci]),
    "sbnet_sparse_bn_backward": (_ci, [_vp, _vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _vp, _vp, _vp, _vp,
                                       ctypes.c_float, _ci, _vp, _vp, _vp, _vp, _sz, _vp]),
    "sbnet_relu_backward_on_tiles": (_ci, [_vp, _vp, _ci, _vp, _ci, _sz, _vp, _vp]),
    "sbnet_bias_backward_workspace_bytes": (_sz, [_ci, _ci]),
    "sbnet_bias_backward_on_tiles": (_ci, [_vp, _ci, _vp, _ci, _ci, _ci, _vp, _vp, _sz, _vp]),
    "sbnet_relu_bias_backward_on_tiles": (_ci, [_vp, _vp, _ci, _vp, _ci, _ci, _ci, _vp, _vp, _vp, _sz, _vp]),
    "sbnet_quantize_f8": (_ci, [_vp, _ci, _sz, ctypes.c_float, _vp, _vp]),
    "sbnet_pack_weights_f8": (_ci, [_vp, _ci, _ci, _ci, _ci, _vp, ctypes.POINTER(_sz), _vp]),
    "sbnet_conv_on_tiles_f8": (_ci, [_vp, _vp, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _ci, _ci, _ci, _ci, _ci,
                                     ctypes.c_float, _vp, _vp]),
    "sbnet_bottleneck_forward_keep_on_tiles": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _vp, _vp, _vp, _vp,
                                                     _vp, _vp, _vp, _vp, _vp, _vp]),
    "sbnet_bottleneck_backward_workspace_bytes": (_sz, [_ci, _ci, _ci, _ci, _ci, _ci]),
    "sbnet_bottleneck_backward_on_tiles": (_ci, [_vp, _vp, _vp, _vp, _ci, _vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _vp,
                                                 _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]),
    "sbnet_pack_weights": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _vp, ctypes.POINTER(_sz), _vp]),
    "sbnet_pack_weights_transposed": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _vp, ctypes.POINTER(_sz), _vp]),
    "sbnet_conv_backward_data_workspace_bytes": (_sz, [_ci, _ci, _ci, _ci, _ci, _ci, _ci, _ci, _ci]),
    "sbnet_conv_on_tiles_backward_data": (_ci, [_vp, _ci, _vp, _ci, _ci, _ci, _ci, _vp, _ci, _ci, _ci, _ci, _ci, _vp,
                                                _vp, _sz, _vp]),
    "sbnet_conv_backward_weights_workspace_bytes": (_sz, [_ci, _ci, _ci, _ci, _ci, _ci, _ci, _ci, _ci, _ci]),
    "sbnet_conv_on_tiles_backward_weights": (_ci, [_vp, _vp, _ci, _vp, _ci, _ci, _ci, _ci, _ci, _ci, _ci, _ci, _ci, _vp,
                                                   _vp, _sz, _vp]),
    "sbnet_conv_on_tiles": (_ci, [_vp, _ci, _vp, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _ci, _ci, _ci, _ci, _ci, _vp, _vp]),
    "sbnet_sparse_conv": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _gp, _vp, _vp,
                                _ci, _ci, _ci, _ci, _ci, _ci, _vp, _ci, _ci, _ci, _vp]),
    "sbnet_block_flags_bytes": (_sz, [_ci, _gp]),
    "sbnet_block_flags": (_ci, [_vp, _ci, _ci, _ci, _ci, _gp, _ci, ctypes.c_float, _vp, _sz, _vp]),
    "sbnet_sparse_conv_from_flags": (_ci, [_vp, _vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _gp, _vp, _vp,
                                           _ci, _ci, _ci, _ci, _ci, _ci, _vp, _ci, _ci, _ci, _vp]),
    "sbnet_sparse_conv_from_mask": (_ci, [_vp, _ci, _ci, _ci, _gp, _ci, ctypes.c_float, _vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci,
                                          _gp, _gp, _vp, _vp, _ci, _ci, _ci, _ci, _ci, _ci, _vp, _ci, _ci, _ci, _vp, _sz, _vp]),
    "sbnet_sparse_unit_workspace_bytes": (_sz, [_ci, _ci, _gp, _gp, _ci, _ci, _ci]),
    "sbnet_sparse_unit": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _gp, _vp, _vp, _vp, _vp, _vp,
                                _vp, _vp, _vp, _vp, _ci, _ci, _vp, _sz, _vp]),
    "sbnet_zero_outside": (_ci, [_vp, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _vp]),
    "sbnet_bottleneck_on_tiles": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _gp,
                                        _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp]),
    "sbnet_sparse_bottleneck": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _gp,
                                      _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp]),
    "sbnet_bottleneck_on_tiles_preact": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _gp,
                                               _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp]),
    "sbnet_sparse_bottleneck_preact": (_ci, [_vp, _ci, _ci, _ci, _ci, _ci, _ci, _vp, _vp, _ci, _gp, _gp,
                                             _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp]),
}


def exported_symbols():
    """Names include/sbnet.h declares; the loader resolves each of them."""
    return sorted(_SIGNATURES)


def lib():
    """Load libsbnet_hip.so (built by build.py / __graft_entry__.build()); raises if absent."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError("%s not found: run `python -m paper_1801_02108_amd.build` first" % LIB_PATH)
        l = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in _SIGNATURES.items():
            fn = getattr(l, name)
            fn.restype, fn.argtypes = res, args
        _lib = l
    return _lib


class _Calls:
    """Stands for the native module until its first use, so that the package imports before anything is built."""

    def __getattr__(self, name):
        global _calls
        lib()
        try:
            native = importlib.import_module("._torch_calls", __name__)
        except ImportError as e:
            raise ImportError("%s: run `python -m paper_1801_02108_amd.build` first" % e) from e
        native.set_types(SbnetError, Geom)
        _calls = native
        return getattr(native, name)


_calls = _Calls()


def get_tuning():
    """The compute-tile choices in force, as a dict."""
    t = Tuning()
    _check(lib().sbnet_get_tuning(ctypes.byref(t)))
    return t.asdict()


def set_tuning(**kw):
    """Change some of the compute-tile choices (keyword = field of sbnet_tuning); no keyword restores the defaults.
    Returns what is in force afterwards."""
    if not kw:
        _check(lib().sbnet_set_tuning(None))
        return get_tuning()
    t = Tuning()
    _check(lib().sbnet_get_tuning(ctypes.byref(t)))
    for k, v in kw.items():
        if k not in dict(Tuning._fields_):
            raise KeyError(k)
        setattr(t, k, int(v))
    _check(lib().sbnet_set_tuning(ctypes.byref(t)))
    return get_tuning()


def _check(code):
    if code != OK:
        raise SbnetError(code, lib().sbnet_last_error().decode())


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr()) if t is not None else ctypes.c_void_p(0)


def _dev(t, name, dtype=None):
    if not (isinstance(t, torch.Tensor) and t.is_cuda and t.is_contiguous()):
        raise TypeError("%s must be a contiguous device tensor" % name)
    if dtype is not None and t.dtype != dtype:
        raise TypeError("%s must be %s" % (name, dtype))
    return t


def _dt(t):
    try:
        return _DTYPES[t.dtype]
    except KeyError:
        raise TypeError("unsupported dtype %s" % t.dtype)


# ---------------------------------------------------------------------------------------------
def geometry(H, W, k, s, bo):
    """(g_in, g_out, H_out, W_out) for a k x k, stride-s SAME convolution with bo x bo output blocks."""
    g_in, g_out, ho, wo = Geom(), Geom(), _ci(), _ci()
    _check(lib().sbnet_geometry(H, W, k, k, s, s, bo, bo, g_in, g_out, ho, wo))
    return g_in, g_out, ho.value, wo.value


def coarse_geometry(g, factor):
    """Geometry of the same block windows on a map `factor` times coarser (sbnet_coarse_geometry)."""
    c = Geom()
    _check(lib().sbnet_coarse_geometry(g, factor, c))
    return c


def workspace_bytes(N, g):
    return int(lib().sbnet_workspace_bytes(N, g))


def reduce_mask(mask, g, pool=POOL_AVG, threshold=0.0, indices=None, count=None, workspace=None):
    """mask [N,H,W] u8/f32 -> (indices int32 [cap,3], count int32 [1]) on the device."""
    return _calls.reduce_mask(mask, g, pool, threshold, indices, count, workspace)


def reduce_mask_static(mask, g, indices, count, pool=POOL_AVG, threshold=0.0):
    """reduce_mask without a workspace argument (the library's built-in scratch): the caller passes every
    buffer, nothing is allocated on the way.  Returns (indices, count) as passed."""
    return _calls.reduce_mask_static(mask, g, indices, count, pool, threshold)


def read_count(count, cap):
    out = _ci()
    _check(lib().sbnet_read_count(_ptr(count), cap, out, _stream()))
    return out.value


def sparse_gather(x, indices, count, g, tiles=None):
    """x [N,H,W,C] -> tiles [cap, bsize_h, bsize_w, C]; rows beyond the active count are untouched."""
    return _calls.sparse_gather(x, indices, count, g, tiles)


def sparse_scatter(tiles, indices, count, g, y, add=False):
    """tiles [cap, bsize_h, bsize_w, C] -> written or added into y [N,H,W,C] in place; returns y."""
    return _calls.sparse_scatter(tiles, indices, count, g, y, add)


def sparse_gather_chw(x, indices, count, g, tiles=None):
    """Gather with the transpose fused in: x [N,H,W,C] -> channel-major tiles [cap,C,h,w]."""
    return _calls.sparse_gather_chw(x, indices, count, g, tiles)


def sparse_scatter_chw(tiles, indices, count, g, y, add=False):
    """Scatter (or scatter-add) of channel-major tiles [cap,C,h,w] into y [N,H,W,C] in place; returns y."""
    return _calls.sparse_scatter_chw(tiles, indices, count, g, y, add)


def sparse_gather_backward(dtiles, indices, count, g, dx, workspace=None):
    """Gradient of sparse_gather: adds the tile gradients [cap,h,w,C] (overlapping halos included) into dx [N,H,W,C]."""
    return _calls.sparse_gather_backward(dtiles, indices, count, g, dx, workspace)


def sparse_bn_stats(x, indices, count, g, workspace=None):
    """Per-channel mean and biased variance of x [N,H,W,C] over the pixels of the active blocks; returns (mean, var)."""
    return _calls.sparse_bn_stats(x, indices, count, g, workspace)


def sparse_bn_apply(x, indices, count, g, mean, var, gamma=None, beta=None, eps=1e-5, relu=False, y=None):
    """y = act(gamma (x - mean) / sqrt(var + eps) + beta) on the pixels of the active blocks, y untouched elsewhere
    (y defaults to x: in place); returns y."""
    return _calls.sparse_bn_apply(x, indices, count, g, mean, var, gamma, beta, eps, relu, y)


def sparse_bn_backward(x, dy, indices, count, g, mean, var, gamma=None, beta=None, eps=1e-5, relu=False, dx=None,
                       workspace=None):
    """Gradients through sparse_bn_apply in training mode (mean, var = sparse_bn_stats of x over the same blocks);
    returns (dx, dgamma, dbeta); dx defaults to a new zero tensor and is written on the active blocks only."""
    return _calls.sparse_bn_backward(x, dy, indices, count, g, mean, var, gamma, beta, eps, relu, dx, workspace)


def relu_backward_on_tiles(y_tiles, dy_tiles, count, out=None):
    """dy where the forward activation y is positive, else 0, on the active tiles of two stacks of one shape."""
    return _calls.relu_backward_on_tiles(y_tiles, dy_tiles, count, out)


def bias_backward_on_tiles(dy_tiles, count, workspace=None):
    """Sum of dy [cap,h,w,C] over the active tiles and their pixels: float32 [C]."""
    return _calls.bias_backward_on_tiles(dy_tiles, count, workspace)


def relu_bias_backward_on_tiles(y_tiles, dy_tiles, count, out=None, workspace=None):
    """(dout, db): dy [cap,h,w,C] masked by y > 0 on the active tiles, and its per-channel sum (float32 [C]), in one pass."""
    return _calls.relu_bias_backward_on_tiles(y_tiles, dy_tiles, count, out, workspace)


def quantize_f8(x, scale=1.0, out=None):
    """x (f32 / bf16 / f16 device tensor) -> uint8 tensor of FP8 E4M3 (e4m3fn) codes of clamp(x * scale, +-448)."""
    return _calls.quantize_f8(x, scale, out)


def pack_weights_f8(w_f8):
    """FP8 codes [kh,kw,Cin,Cout] (uint8 device tensor) -> packed buffer for conv_on_tiles_f8."""
    _dev(w_f8, "w_f8", torch.uint8)
    kh, kw, Cin, Cout = w_f8.shape
    nbytes = _sz()
    _check(lib().sbnet_pack_weights_f8(None, kh, kw, Cin, Cout, None, nbytes, None))
    buf = torch.empty((nbytes.value,), dtype=torch.uint8, device=w_f8.device)
    _check(lib().sbnet_pack_weights_f8(_ptr(w_f8), kh, kw, Cin, Cout, _ptr(buf), nbytes, _stream()))
    return PackedWeights(buf, (kh, kw, Cin, Cout), torch.uint8)


def conv_on_tiles_f8(tiles_f8, count, w_packed, bias=None, stride=1, relu=False, out_scale=1.0, out=None):
    """Valid convolution of FP8 tiles [cap,th,tw,Cin] (uint8 codes) with FP8 weights -> bf16 [cap,th',tw',Cout]."""
    return _calls.conv_on_tiles_f8(tiles_f8, count, w_packed, bias, stride, relu, out_scale, out)


def bottleneck_forward_keep_on_tiles(tiles, indices, count, g_in, H, W, weights):
    """Residual branch on tiles with its activations kept for the backward pass: returns (t1, t2, t3).
    weights = (w1, b1, w2, b2, w3, b3) as sparse_bottleneck takes them."""
    return _calls.bottleneck_forward_keep_on_tiles(tiles, indices, count, g_in, H, W, weights)


def bottleneck_backward_on_tiles(tiles, t1, t2, dt3, count, weights_t, workspace=None):
    """Backward of the residual branch on tiles from kept activations: returns (dtiles, dw1, db1, dw2, db2, dw3, db3).
    weights_t = (w1_t, w2_t, w3_t) from pack_weights_transposed of the three forward weight arrays."""
    return _calls.bottleneck_backward_on_tiles(tiles, t1, t2, dt3, count, weights_t, workspace)


class PackedWeights:
    """Device buffer in the library's private weight layout plus the shape it was packed for."""

    def __init__(self, buf, shape, dtype):
        self.buf, self.shape, self.dtype = buf, tuple(shape), dtype


def pack_weights(w_hwio):
    """w [kh,kw,Cin,Cout] device tensor -> opaque packed device buffer for the conv calls."""
    _dev(w_hwio, "w_hwio")
    kh, kw, Cin, Cout = w_hwio.shape
    nbytes = _sz()
    _check(lib().sbnet_pack_weights(None, _dt(w_hwio), kh, kw, Cin, Cout, None, nbytes, None))
    buf = torch.empty((nbytes.value,), dtype=torch.uint8, device=w_hwio.device)
    _check(lib().sbnet_pack_weights(_ptr(w_hwio), _dt(w_hwio), kh, kw, Cin, Cout, _ptr(buf), nbytes, _stream()))
    return PackedWeights(buf, (kh, kw, Cin, Cout), w_hwio.dtype)


def conv_on_tiles(tiles, count, w_packed, bias=None, stride=1, relu=False, out=None):
    """Valid convolution on a tile stack [cap,th,tw,Cin] -> [cap,th',tw',Cout]."""
    return _calls.conv_on_tiles(tiles, count, w_packed, bias, stride, relu, out)


def pack_weights_transposed(w_hwio):
    """Forward weights [kh,kw,Cin,Cout] -> packed buffer for conv_on_tiles_backward_data (taps mirrored, channel
    roles exchanged); .shape keeps the forward convolution's (kh, kw, Cin, Cout)."""
    _dev(w_hwio, "w_hwio")
    kh, kw, Cin, Cout = w_hwio.shape
    nbytes = _sz()
    _check(lib().sbnet_pack_weights_transposed(None, _dt(w_hwio), kh, kw, Cin, Cout, None, nbytes, None))
    buf = torch.empty((nbytes.value,), dtype=torch.uint8, device=w_hwio.device)
    _check(lib().sbnet_pack_weights_transposed(_ptr(w_hwio), _dt(w_hwio), kh, kw, Cin, Cout, _ptr(buf), nbytes,
                                               _stream()))
    return PackedWeights(buf, (kh, kw, Cin, Cout), w_hwio.dtype)


def conv_backward_data_workspace_bytes(dtype, cap, th, tw, kh, kw, stride, Cout):
    return int(lib().sbnet_conv_backward_data_workspace_bytes(_DTYPES[dtype], cap, th, tw, kh, kw, stride, stride, Cout))


def conv_on_tiles_backward_data(dout_tiles, count, w_packed_t, th, tw, stride=1, out=None, workspace=None):
    """dL/d(tiles_in) [cap,th,tw,Cin] of conv_on_tiles (no bias, no activation) from dL/d(tiles_out)
    [cap,oh,ow,Cout]; w_packed_t from pack_weights_transposed of the forward weights."""
    return _calls.conv_on_tiles_backward_data(dout_tiles, count, w_packed_t, th, tw, stride, out, workspace)


def conv_backward_weights_workspace_bytes(dtype, cap, th, tw, Cin, k, stride, Cout):
    return int(lib().sbnet_conv_backward_weights_workspace_bytes(_DTYPES[dtype], cap, th, tw, Cin, k, k, stride, stride, Cout))


def conv_on_tiles_backward_weights(tiles, dout_tiles, count, k, stride=1, out=None, workspace=None):
    """dL/dw [k,k,Cin,Cout] (float32) of conv_on_tiles from its input tiles [cap,th,tw,Cin] and dL/d(tiles_out)
    [cap,oh,ow,Cout], summed over the active tiles."""
    return _calls.conv_on_tiles_backward_weights(tiles, dout_tiles, count, k, stride, out, workspace)


def sparse_conv(x, indices, count, g_in, g_out, w_packed, bias, y, stride=1, relu=False, add=False):
    """Fused gather -> valid conv -> scatter(-add) into y [N,H_out,W_out,Cout] in place; returns y."""
    return _calls.sparse_conv(x, indices, count, g_in, g_out, w_packed, bias, y, stride, relu, add)


def block_flags(mask, g, pool=POOL_AVG, threshold=0.0, flags=None):
    """mask [N,H,W] u8/f32 -> one flag byte per block (lexicographic), padded to a multiple of 16 bytes."""
    return _calls.block_flags(mask, g, pool, threshold, flags)


def sparse_conv_from_flags(flags, x, g_in, g_out, w_packed, bias, y, indices, count, stride=1, relu=False, add=False):
    """Fused sparse conv fed by block flags; fills y in place and writes the index list and count.  Returns y."""
    return _calls.sparse_conv_from_flags(flags, x, g_in, g_out, w_packed, bias, y, indices, count, stride, relu, add)


def sparse_conv_from_mask(mask, g_mask, x, g_in, g_out, w_packed, bias, y, indices, count, workspace, pool=POOL_AVG,
                          threshold=0.0, stride=1, relu=False, add=False):
    """reduce_mask + fused sparse conv in one call (two launches where the convolution kernel takes block flags);
    fills y in place and leaves the index list and the count in indices / count.  Returns y."""
    return _calls.sparse_conv_from_mask(mask, g_mask, x, g_in, g_out, w_packed, bias, y, indices, count, workspace,
                                        pool, threshold, stride, relu, add)


def bottleneck_on_tiles(tiles, indices, count, g_in, g_out, H, W, weights, out=None, pre=None):
    """Residual branch (1x1+ReLU, 3x3+ReLU, 1x1) on gathered tiles [cap,h,w,C] -> t3 [cap,bo,bo,C];
    pre = (scale, shift): pre-activation ReLU(scale * x + shift) in front of the first convolution."""
    return _calls.bottleneck_on_tiles(tiles, indices, count, g_in, g_out, H, W, weights, out, pre)


def sparse_bottleneck(x, indices, count, g_in, g_out, weights, y, pre=None):
    """Fused sparse residual unit: y[active] = x[active] + branch(x); y is a second buffer. Returns y.
    pre = (scale, shift): pre-activation form."""
    return _calls.sparse_bottleneck(x, indices, count, g_in, g_out, weights, y, pre)


def zero_outside(tiles, indices, count, g, H, W):
    """Zero, in place, the positions of tiles [cap,h,w,C] that lie outside the H x W image."""
    return _calls.zero_outside(tiles, indices, count, g, H, W)


def sparse_unit(x, indices, count, g_in, g_out, weights, y, stride=1, shortcut=None, workspace=None):
    """Residual unit of any width: weights = (w1p, b1, w2p, b2, w3p, b3) packed, shortcut = (wsp, bs) packed 1x1 with the
    unit's stride or None for the identity.  Writes the active blocks of y [N,H_out,W_out,Cout] in place; returns y."""
    return _calls.sparse_unit(x, indices, count, g_in, g_out, weights, y, stride, shortcut, workspace)
