"""GPU parity of the tile convolution's gradients against the fp64 oracle (training support for the
convolution of Sec. 3.2): element by element on seeded inputs, for every kernel the forward dispatch can
pick for the gradient's own shape (1x1 and 3x3 matrix-core kernels, the LDS-tiled one, the direct fp32 one)."""
import numpy as np
import pytest
import torch

import oracle as orc
import paper_1801_02108_amd as sb
from paper_1801_02108_amd import inputs as gen
from util import CONV_TOL, TORCH_DT, assert_close, kernels, template_args, to_dev, to_host

pytestmark = pytest.mark.gpu


def step(msg):
    print("[case] " + msg, flush=True)


DGRAD_CASES = [
    # B, th, tw, Cin, Cout, k, s, dtype
    (5, 18, 18, 64, 64, 3, 1, "bf16"),       # the headline layer's tiles
    (3, 18, 18, 64, 64, 3, 1, "f16"),
    (4, 33, 33, 64, 96, 3, 2, "bf16"),       # downsampling layer: the output gradient is spread by the stride
    (2, 18, 18, 96, 192, 3, 1, "bf16"),
    (3, 10, 10, 32, 40, 3, 1, "bf16"),
    (2, 17, 17, 256, 384, 3, 2, "bf16"),
    (3, 16, 16, 64, 256, 1, 1, "bf16"),      # 1x1: no frame, no mirror
    (3, 18, 18, 96, 24, 1, 1, "bf16"),       # 1x1 with channel counts of the 96-channel stage
    (2, 9, 9, 24, 40, 1, 2, "f16"),          # 1x1 at stride 2: the gradient is spread, every other pixel stays zero
    (2, 12, 20, 24, 16, 3, 1, "f32"),        # direct fp32 kernel
    (2, 12, 13, 8, 8, 3, 2, "f32"),          # the last input column is not reached by any window
    (2, 14, 12, 16, 8, 3, 2, "bf16"),        # the last input row is not reached by any window
    (2, 11, 9, 6, 5, 3, 1, "bf16"),          # channel counts the matrix-core kernels do not take
    (1, 9, 9, 3, 7, 5, 1, "f16"),
    (2, 9, 11, 16, 16, 3, 3, "bf16"),        # stride 3
    (3, 10, 10, 96, 48, 3, 1, "bf16"),       # groups of 96 with the weights in LDS
    (3, 10, 10, 80, 40, 3, 1, "f16"),
    (4, 18, 18, 200, 40, 3, 1, "f16"),       # weights that do not stay there
    (2, 10, 10, 200, 40, 3, 1, "f16"),
]


@pytest.mark.parametrize("B,th,tw,Cin,Cout,k,s,dtype", DGRAD_CASES)
def test_conv_on_tiles_backward_data(B, th, tw, Cin, Cout, k, s, dtype):
    step("conv_on_tiles_backward_data %s" % ((B, th, tw, Cin, Cout, k, s, dtype),))
    r = gen.rng_for(21, th * 1000 + tw * 10 + Cin + Cout + s)
    oh, ow = (th - k) // s + 1, (tw - k) // s + 1
    g = gen.activations(r, (B + 1, oh, ow, Cout), dtype)
    w = gen.conv_weights(r, k, k, Cin, Cout, dtype, unit_variance=(dtype == "f32"))
    cnt = torch.tensor([B], dtype=torch.int32).cuda()
    wt = sb.pack_weights_transposed(to_dev(w, dtype))
    out = torch.full((B + 1, th, tw, Cin), 5.0, dtype=TORCH_DT[dtype]).cuda()
    sb.conv_on_tiles_backward_data(to_dev(g, dtype), cnt, wt, th, tw, stride=s, out=out)
    got = to_host(out)
    ref = orc.conv_valid_backward_data(g[:B], w, th, tw, stride=s)
    assert_close(got[:B], ref, CONV_TOL[dtype], "conv_on_tiles_backward_data")
    assert (got[B] == 5.0).all()                        # tiles beyond the count are not touched
    # input rows and columns that no window reaches get an exact zero
    rh, rw = (oh - 1) * s + k, (ow - 1) * s + k
    assert (got[:B, rh:] == 0).all() and (got[:B, :, rw:] == 0).all()


WGRAD_CASES = [
    # B, th, tw, Cin, Cout, k, s, dtype
    (5, 18, 18, 64, 64, 3, 1, "bf16"),       # the headline layer's tiles: one tile per split
    (300, 18, 18, 64, 64, 3, 1, "bf16"),     # more tiles than splits: several tiles per workgroup, ragged
    (7, 18, 18, 64, 64, 3, 1, "f16"),
    (20, 33, 33, 64, 96, 3, 2, "bf16"),      # downsampling layer; the second block of output channels is half empty
    (9, 34, 34, 32, 64, 3, 2, "bf16"),       # even tile at stride 2: the last row and column are never read
    (6, 18, 18, 96, 192, 3, 1, "bf16"),      # several channel blocks
    (11, 10, 10, 40, 24, 3, 1, "bf16"),      # 8x8 blocks: half-filled matrix rows, ragged channel counts
    (4, 12, 15, 8, 16, 3, 1, "f16"),         # ragged tile: 10 x 13 outputs
    (3, 34, 34, 16, 16, 3, 1, "bf16"),       # 32 x 32 outputs
    (3, 37, 41, 16, 8, 3, 2, "bf16"),        # stride 2 with two segments per row (18 x 20 outputs)
    (2, 21, 16, 8, 8, 3, 1, "bf16"),         # 19 output rows: the last stage is partly empty
    (3, 12, 20, 24, 16, 3, 1, "f32"),        # plain kernel
    (3, 11, 9, 6, 5, 3, 1, "bf16"),
    (4, 16, 16, 64, 32, 1, 1, "bf16"),       # 1x1: one accumulator per wave
    (40, 18, 18, 256, 64, 1, 1, "bf16"),     # first convolution of the residual unit on its input tile (two segments)
    (5, 16, 16, 64, 256, 1, 1, "f16"),       # its last convolution
    (300, 16, 16, 64, 64, 1, 1, "bf16"),     # 1x1 with more tiles than splits: two or three tiles per workgroup
    (3, 17, 17, 32, 48, 1, 2, "bf16"),       # 1x1 at stride 2: 9 x 9 outputs, odd phase never read
    (4, 10, 10, 40, 24, 1, 1, "bf16"),
    (6, 17, 17, 64, 64, 1, 1, "bf16"),       # 289 pixels: one pixel in the last row of 16
    (9, 7, 5, 8, 16, 1, 1, "f16"),           # 35 pixels: not a whole item of four at the end
    (2, 9, 9, 3, 7, 5, 2, "f16"),
    (2, 13, 11, 16, 16, 3, 3, "bf16"),
]


@pytest.mark.parametrize("B,th,tw,Cin,Cout,k,s,dtype", WGRAD_CASES)
def test_conv_on_tiles_backward_weights(B, th, tw, Cin, Cout, k, s, dtype):
    step("conv_on_tiles_backward_weights %s" % ((B, th, tw, Cin, Cout, k, s, dtype),))
    r = gen.rng_for(23, th * 1000 + tw * 10 + Cin + Cout + s)
    oh, ow = (th - k) // s + 1, (tw - k) // s + 1
    x = gen.activations(r, (B + 2, th, tw, Cin), dtype)
    g = gen.activations(r, (B + 2, oh, ow, Cout), dtype)
    xd, gd = to_dev(x, dtype), to_dev(g, dtype)
    ref = orc.conv_valid_backward_weights(x[:B], g[:B], k, k, stride=s)
    # fp32 accumulation of exact products over B * oh * ow terms in a tree of partial sums
    tol = 1e-4 if dtype == "f32" else 2e-5
    for n in (B, 1, 0):
        cnt = torch.tensor([n], dtype=torch.int32).cuda()
        dw = torch.full((k, k, Cin, Cout), 7.0, dtype=torch.float32).cuda()
        sb.conv_on_tiles_backward_weights(xd, gd, cnt, k, stride=s, out=dw)
        want = ref if n == B else orc.conv_valid_backward_weights(x[:n], g[:n], k, k, stride=s)
        if n == 0:
            assert (dw == 0).all()
        else:
            assert_close(to_host(dw), want, tol, "conv_on_tiles_backward_weights n=%d" % n)
        if n == B:
            dw2 = torch.empty_like(dw)
            sb.conv_on_tiles_backward_weights(xd, gd, cnt, k, stride=s, out=dw2)
            assert torch.equal(dw, dw2)                  # fixed summation order: the same bits again


@pytest.mark.parametrize("B,cap,oh,ow,Cin,Cout,k,dtype", [
    (7, 7, 8, 8, 64, 64, 3, "bf16"),       # four tiles to a stage, the last stage holds three
    (9, 12, 5, 7, 40, 24, 3, "f16"),       # one segment a row and an odd number of rows: a row of zeros
    (5, 5, 1, 1, 8, 8, 3, "bf16"),
    (3, 3, 3, 40, 32, 72, 3, "bf16"),      # five segments a row
    (2, 2, 41, 37, 64, 32, 3, "f16"),      # tiles in slices, the last one short
    (2, 2, 3, 170, 8, 40, 3, "bf16"),      # a row or two to a slice
    (70, 70, 12, 12, 96, 96, 3, "bf16"),   # more tiles than splits of nine channel blocks
    (30, 1100, 16, 16, 64, 64, 3, "bf16"), # list bounds that take the kernel for long lists
    (30, 1100, 16, 16, 64, 64, 3, "f16"),
    (5, 260, 32, 32, 64, 64, 3, "bf16"),   # ... two segments a row
    (4, 330, 30, 27, 40, 64, 3, "f16"),    # ... the second one partly empty, the last stage too
    (300, 300, 4, 4, 16, 16, 3, "f16"),    # fewer stages than splits
    (5, 9, 9, 15, 72, 64, 1, "f16"),       # runs of pixels that end inside a stage
    (64, 64, 16, 16, 64, 136, 1, "bf16"),
    (3, 3, 2, 3, 256, 8, 1, "bf16"),       # less than a stage
])
def test_weight_gradient_stages(B, cap, oh, ow, Cin, Cout, k, dtype):
    step("weight gradient, stages %s" % ((B, cap, oh, ow, Cin, Cout, k, dtype),))
    r = gen.rng_for(6, oh * 1000 + ow * 10 + Cin + Cout)
    x = gen.activations(r, (cap, oh + k - 1, ow + k - 1, Cin), dtype)
    g = gen.activations(r, (cap, oh, ow, Cout), dtype)
    xd, gd = to_dev(x, dtype), to_dev(g, dtype)
    # what lies beyond the count is not read
    xd[B:] = float("nan")
    gd[B:] = float("nan")
    for n in (B, B - 1, 1):
        cnt = torch.tensor([n], dtype=torch.int32).cuda()
        dw = sb.conv_on_tiles_backward_weights(xd, gd, cnt, k)
        want = orc.conv_valid_backward_weights(x[:n], g[:n], k, k)
        # products are exact in fp32, sums of n oh ow of them in any order
        assert_close(to_host(dw), want, 1e-4, "weight gradient, %d tiles" % n)
        assert torch.equal(dw, sb.conv_on_tiles_backward_weights(xd, gd, cnt, k))
    name = kernels(lambda: sb.conv_on_tiles_backward_weights(xd, gd, cnt, k))[0]
    assert ("wgrad_run" if k == 1 else "wgrad_mfma" if cap > 200 and oh > 4 else "wgrad_tile") in name


def test_sparse_conv_gradients_end_to_end():
    """dL/dx and dL/dw of the whole sparse convolution from library calls only: gather of dL/dy with the output
    geometry, data gradient on tiles, gather_backward into the image; gather of x, weight gradient on the two tile
    stacks; against the oracle's composition of the same steps."""
    N, H, W, Cin, Cout, bo, dtype = 2, 70, 66, 64, 96, 16, "bf16"
    for s in (1, 2):
        step("sparse conv input gradient stride %d" % s)
        r = gen.rng_for(22, s)
        g_in, g_out, Ho, Wo = sb.geometry(H, W, 3, s, bo)
        mask = (r.random((N, H, W)) < 0.002).astype(np.float64)
        og_in, og_out = orc.Geom(*g_in.astuple()), orc.Geom(*g_out.astuple())
        idx_np = orc.reduce_mask(mask, og_in)
        n, total = len(idx_np), N * g_in.bcount_h * g_in.bcount_w
        assert 0 < n < total
        buf = np.zeros((n + 2, 3), dtype=np.int32)
        buf[:n] = idx_np
        idx, cnt = torch.from_numpy(buf).cuda(), torch.tensor([n], dtype=torch.int32).cuda()
        dy = gen.activations(r, (N, Ho, Wo, Cout), dtype)
        w = gen.conv_weights(r, 3, 3, Cin, Cout, dtype)
        dy_tiles = sb.sparse_gather(to_dev(dy, dtype), idx, cnt, g_out)
        din_tiles = sb.conv_on_tiles_backward_data(dy_tiles, cnt, sb.pack_weights_transposed(to_dev(w, dtype)),
                                                   g_in.bsize_h, g_in.bsize_w, stride=s)
        dx = torch.zeros((N, H, W, Cin), dtype=TORCH_DT[dtype]).cuda()
        sb.sparse_gather_backward(din_tiles, idx, cnt, g_in, dx)
        ref_tiles = orc.conv_valid_backward_data(orc.gather(dy, idx_np, og_out), w, g_in.bsize_h, g_in.bsize_w, stride=s)
        # the library rounds the tile gradient to bf16 before the overlap sum; so does the reference
        ref_tiles_r = torch.from_numpy(ref_tiles).to(TORCH_DT[dtype]).to(torch.float64).numpy()
        ref = orc.gather_backward(ref_tiles_r, idx_np, og_in, np.zeros((N, H, W, Cin)))
        assert_close(to_host(dx), ref, CONV_TOL[dtype], "sparse conv dL/dx")
        # dL/dw of the same layer: the forward input gathered with the input geometry against the gathered dL/dy
        x = gen.activations(r, (N, H, W, Cin), dtype)
        x_tiles = sb.sparse_gather(to_dev(x, dtype), idx, cnt, g_in)
        dw = sb.conv_on_tiles_backward_weights(x_tiles, dy_tiles, cnt, 3, stride=s)
        ref_dw = orc.conv_valid_backward_weights(orc.gather(x, idx_np, og_in), orc.gather(dy, idx_np, og_out), 3, 3, stride=s)
        assert_close(to_host(dw), ref_dw, 2e-5, "sparse conv dL/dw")


@pytest.mark.parametrize("oh,ow,Cin,Cout,k,dtype,most,kernel", [
    # the longest list that the kernel takes which is faster on short ones
    (16, 16, 64, 72, 1, "bf16", 4000, "wgrad_run"),
    (31, 33, 136, 64, 1, "f16", 1000, "wgrad_run"),         # 1023 pixels: one short of a row of 16
    (16, 16, 160, 160, 1, "bf16", 3000, "wgrad_run"),       # nine blocks of 64 x 64 channels
    (16, 16, 264, 264, 1, "bf16", 700, "wgrad_run"),        # 25
    (16, 16, 64, 64, 1, "bf16", None, "wgrad_run"),         # one block
    (18, 18, 64, 72, 1, "bf16", None, "wgrad_run"),         # stages of 128 pixels would be a sixth padding
    (16, 16, 224, 224, 3, "bf16", 250, "wgrad_tile"),
    (16, 16, 64, 64, 3, "f16", 1000, "wgrad_tile"),
    (24, 24, 64, 64, 3, "bf16", None, "wgrad_tile"),
])
def test_weight_gradient_kernel_by_list_bound(oh, ow, Cin, Cout, k, dtype, most, kernel):
    step("weight gradient, list bound %s" % ((oh, ow, Cin, Cout, k, dtype, most),))
    r = gen.rng_for(8, oh * 1000 + Cin + Cout + k)
    B, rows = 5, most or 6000
    x = gen.activations(r, (B, oh + k - 1, ow + k - 1, Cin), dtype)
    g = gen.activations(r, (B, oh, ow, Cout), dtype)
    xd = torch.zeros((rows + 1,) + x.shape[1:], dtype=TORCH_DT[dtype], device="cuda")
    gd = torch.zeros((rows + 1,) + g.shape[1:], dtype=TORCH_DT[dtype], device="cuda")
    xd[:B], gd[:B] = to_dev(x, dtype), to_dev(g, dtype)
    cnt = torch.tensor([B], dtype=torch.int32).cuda()
    dw = torch.empty((k, k, Cin, Cout), dtype=torch.float32).cuda()
    want = orc.conv_valid_backward_weights(x, g, k, k)
    for cap in (rows, rows + 1):
        names = kernels(lambda: sb.conv_on_tiles_backward_weights(xd[:cap], gd[:cap], cnt, k, out=dw))
        assert (kernel if most is None or cap == rows else "wgrad_mfma") in names[0], (cap, names)
        # fp32 accumulation of exact products over B * oh * ow terms in a tree of partial sums
        assert_close(to_host(dw), want, 2e-5, "list bound %d" % cap)


@pytest.mark.parametrize("n,th,Cin,Cout,s", [(2200, 18, 64, 64, 1), (220, 18, 64, 64, 1), (550, 33, 64, 96, 2)])
def test_gradients_at_full_size_sampled(n, th, Cin, Cout, s):
    """The tile counts and shapes bench.py times (all 2200 blocks and 10 % of them for the headline layer, the dense
    downsampling layer), in its launch configuration.  The oracle computes what it can one by one: the data gradient
    of a seeded sample of tiles (the first and the last among them), and a seeded sample of weights, each of which is
    a sum over every pixel of every tile."""
    step("gradients at full size %s" % ((n, th, Cin, Cout, s),))
    dtype = "bf16"
    r = gen.rng_for(24, n + th + Cout)
    oh = (th - 3) // s + 1
    x = gen.activations(r, (n, th, th, Cin), dtype)
    g = gen.activations(r, (n, oh, oh, Cout), dtype)
    w = gen.conv_weights(r, 3, 3, Cin, Cout, dtype)
    xd, gd = to_dev(x, dtype), to_dev(g, dtype)
    cnt = torch.tensor([n], dtype=torch.int32).cuda()
    din = sb.conv_on_tiles_backward_data(gd, cnt, sb.pack_weights_transposed(to_dev(w, dtype)), th, th, stride=s)
    dw = sb.conv_on_tiles_backward_weights(xd, gd, cnt, 3, stride=s)
    pick = np.unique(np.concatenate([[0, n - 1], r.choice(n, 10, replace=False)]))
    ref = orc.conv_valid_backward_data(g[pick], w, th, th, stride=s)
    assert_close(to_host(din[torch.from_numpy(pick).cuda()]), ref, CONV_TOL[dtype], "data gradient, sampled tiles")
    got = to_host(dw)
    samples = [(int(r.integers(0, 3)), int(r.integers(0, 3)), int(r.integers(0, Cin)), int(r.integers(0, Cout))) for _ in range(48)]
    samples += [(0, 0, 0, 0), (2, 2, Cin - 1, Cout - 1), (1, 2, Cin - 1, 0), (2, 0, 0, Cout - 1)]
    want = np.array([float((x[:, kr:kr + s * (oh - 1) + 1:s, kt:kt + s * (oh - 1) + 1:s, c] * g[:, :, :, o]).sum())
                     for kr, kt, c, o in samples])
    have = np.array([got[kr, kt, c, o] for kr, kt, c, o in samples])
    # every weight's gradient is a sum of n * oh * oh products of independent unit-scale factors: scale sqrt(terms)
    scale = np.sqrt(n * oh * oh)
    assert np.abs(have - want).max() <= 2e-5 * scale + 2e-5 * np.abs(want).max()
    assert np.isfinite(got).all() and 0.3 < np.sqrt((got ** 2).mean()) / scale < 3.0


RELU_BIAS_CASES = [(7, 18, 18, 64, "bf16"), (3, 5, 7, 6, "f32"), (4, 3, 3, 10, "f16"), (2, 1, 3, 2, "bf16"), (5, 16, 16, 256, "bf16")]


@pytest.mark.parametrize("B,h,w,C,dtype", RELU_BIAS_CASES)
def test_relu_and_bias_backward_on_tiles(B, h, w, C, dtype):
    step("relu / bias backward %s" % ((B, h, w, C, dtype),))
    r = gen.rng_for(25, B * 100 + h * w + C)
    y = gen.activations(r, (B + 1, h, w, C), dtype)
    y[r.random(y.shape) < 0.3] = 0.0
    y = np.abs(y) * (r.random(y.shape) < 0.7)                       # a ReLU output: zeros and positive values
    y = gen.round_to(y.astype(np.float32), dtype)
    dy = gen.activations(r, (B + 1, h, w, C), dtype)
    cnt = torch.tensor([B], dtype=torch.int32).cuda()
    out = torch.full((B + 1, h, w, C), 3.0, dtype=TORCH_DT[dtype]).cuda()
    sb.relu_backward_on_tiles(to_dev(y, dtype), to_dev(dy, dtype), cnt, out=out)
    got = to_host(out)
    assert np.array_equal(got[:B], orc.relu_backward(y[:B], dy[:B])) and (got[B] == 3.0).all()
    inplace = to_dev(dy, dtype)
    sb.relu_backward_on_tiles(to_dev(y, dtype), inplace, cnt, out=inplace)
    assert torch.equal(inplace[:B], out[:B])
    db = sb.bias_backward_on_tiles(to_dev(dy, dtype), cnt)
    ref = orc.bias_backward(dy[:B])
    assert np.abs(db.cpu().numpy() - ref).max() <= 1e-5 * np.sqrt(B * h * w) + 1e-6
    db2 = sb.bias_backward_on_tiles(to_dev(dy, dtype), cnt)
    assert torch.equal(db, db2)
    assert (sb.bias_backward_on_tiles(to_dev(dy, dtype), torch.tensor([0], dtype=torch.int32).cuda()) == 0).all()
    # both in one pass: the masked gradient bit for bit, its sum against the oracle and, bit for bit, against the sum
    # the separate call makes of the masked stack
    out2 = torch.full((B + 1, h, w, C), 3.0, dtype=TORCH_DT[dtype]).cuda()
    _, dbm = sb.relu_bias_backward_on_tiles(to_dev(y, dtype), to_dev(dy, dtype), cnt, out=out2)
    assert torch.equal(out2, out)
    refm = orc.bias_backward(orc.relu_backward(y[:B], dy[:B]))
    assert np.abs(dbm.cpu().numpy() - refm).max() <= 1e-5 * np.sqrt(B * h * w) + 1e-6
    assert torch.equal(dbm, sb.bias_backward_on_tiles(out, cnt))
    inplace = to_dev(dy, dtype)
    _, dbi = sb.relu_bias_backward_on_tiles(to_dev(y, dtype), inplace, cnt, out=inplace)
    assert torch.equal(inplace[:B], out[:B]) and torch.equal(inplace[B], to_dev(dy, dtype)[B]) and torch.equal(dbi, dbm)
    _, db0 = sb.relu_bias_backward_on_tiles(to_dev(y, dtype), to_dev(dy, dtype), torch.tensor([0], dtype=torch.int32).cuda(), out=out2)
    assert (db0 == 0).all() and torch.equal(out2, out)             # no active tile: nothing written, zero sums


@pytest.mark.parametrize("B,h,w,C,dtype", [
    (300, 3, 5, 16, "bf16"),       # more tiles than workgroups: runs that end inside a tile
    (260, 1, 1, 8, "f16"),         # one thread column, most runs of two pixels and the last ones empty
    (2, 40, 40, 2048, "bf16"),     # the most channels a pixel may have: no slices in the last sum
    (2, 9, 9, 1024, "f32"),
    (3, 7, 7, 48, "f16"),          # six thread columns: threads of the last group stay idle
    (8, 16, 16, 64, "bf16"),       # the longest run on four waves
    (8, 17, 16, 64, "bf16"),       # ... and the next one, on sixteen
    (40, 30, 30, 6, "bf16"),       # words instead of vectors, 341 pixel groups
    (20, 64, 64, 2, "f16"),        # 1024 pixel groups for two channels
])
def test_relu_and_bias_backward_on_runs_of_pixels(B, h, w, C, dtype):
    test_relu_and_bias_backward_on_tiles(B, h, w, C, dtype)


@pytest.mark.parametrize("C,Cm,dens", [(64, 64, 0.02), (256, 64, 0.004), (96, 24, 0.01)])
def test_residual_unit_backward_composed_from_single_calls(C, Cm, dens):
    """The residual branch of a unit (Sec. 3.3) forward with its activations kept, then every gradient from library
    calls alone: weight, bias and data gradients of the three convolutions, the two ReLU masks, and the gather's
    gradient into the image.  The oracle's chain rule runs on the same kept activations (the ReLU masks are
    decisions, taken on the stored bf16 values by both sides)."""
    step("residual unit backward C=%d Cm=%d" % (C, Cm))
    dtype, bo, N, H, W = "bf16", 16, 1, 70, 66
    r = gen.rng_for(26, C)
    g_in, g_out, _, _ = sb.geometry(H, W, 3, 1, bo)
    og_in = orc.Geom(*g_in.astuple())
    mask = (r.random((N, H, W)) < dens).astype(np.float64)
    mask[0, 0, 0] = mask[0, H - 1, W - 1] = 1.0                      # corner tiles: t1 is zeroed outside the image
    idx_np = orc.reduce_mask(mask, og_in)
    n = len(idx_np)
    buf = np.zeros((n + 1, 3), dtype=np.int32)
    buf[:n] = idx_np
    idx, cnt = torch.from_numpy(buf).cuda(), torch.tensor([n], dtype=torch.int32).cuda()
    x = gen.activations(r, (N, H, W, C), dtype)
    w1, b1, w2, b2, w3, b3 = gen.bottleneck_weights(r, C, Cm, dtype)
    dt3 = gen.activations(r, (n + 1, bo, bo, C), dtype)
    dev = lambda a: to_dev(a, dtype)
    fb = lambda b: torch.from_numpy(b).cuda()
    # forward, activations kept
    tiles = sb.sparse_gather(dev(x), idx, cnt, g_in)
    t1 = sb.conv_on_tiles(tiles, cnt, sb.pack_weights(dev(w1)), fb(b1), relu=True)
    sb.zero_outside(t1, idx, cnt, g_in, H, W)
    t2 = sb.conv_on_tiles(t1, cnt, sb.pack_weights(dev(w2)), fb(b2), relu=True)
    # backward
    d3 = dev(dt3)
    th = g_in.bsize_h
    dw3 = sb.conv_on_tiles_backward_weights(t2, d3, cnt, 1)
    db3 = sb.bias_backward_on_tiles(d3, cnt)
    d2 = sb.relu_backward_on_tiles(t2, sb.conv_on_tiles_backward_data(d3, cnt, sb.pack_weights_transposed(dev(w3)), bo, bo), cnt)
    dw2 = sb.conv_on_tiles_backward_weights(t1, d2, cnt, 3)
    db2 = sb.bias_backward_on_tiles(d2, cnt)
    d1 = sb.relu_backward_on_tiles(t1, sb.conv_on_tiles_backward_data(d2, cnt, sb.pack_weights_transposed(dev(w2)), th, th), cnt)
    dw1 = sb.conv_on_tiles_backward_weights(tiles, d1, cnt, 1)
    db1 = sb.bias_backward_on_tiles(d1, cnt)
    dtiles = sb.conv_on_tiles_backward_data(d1, cnt, sb.pack_weights_transposed(dev(w1)), th, th)
    dx = torch.zeros((N, H, W, C), dtype=TORCH_DT[dtype]).cuda()
    sb.sparse_gather_backward(dtiles, idx, cnt, g_in, dx)
    # oracle on the kept activations
    ref = orc.bottleneck_backward_on_tiles(orc.gather(x, idx_np, og_in), idx_np, og_in, H, W, w1, b1, w2, b2, w3, b3, dt3[:n],
                                           saved=(to_host(t1)[:n], to_host(t2)[:n]))
    tol = 3e-2                                                       # a chain of up to three bf16 roundings of the gradient
    assert_close(to_host(dtiles)[:n], ref[0], tol, "d tiles")
    for name, got, want in (("dw1", dw1, ref[1]), ("dw2", dw2, ref[3]), ("dw3", dw3, ref[5])):
        assert_close(to_host(got), want, tol, name)
    for name, got, want in (("db1", db1, ref[2]), ("db2", db2, ref[4]), ("db3", db3, ref[6])):
        assert_close(to_host(got), want, tol, name)
    ref_tiles_r = torch.from_numpy(ref[0]).to(TORCH_DT[dtype]).to(torch.float64).numpy()
    assert_close(to_host(dx), orc.gather_backward(ref_tiles_r, idx_np, og_in, np.zeros((N, H, W, C))), tol, "dx")
    # the forward pass that keeps its activations, as one call: the same t1 and t2, and t3 against the oracle's branch
    k1, k2, k3 = sb.bottleneck_forward_keep_on_tiles(tiles, idx, cnt, g_in, H, W, (sb.pack_weights(dev(w1)), fb(b1), sb.pack_weights(dev(w2)),
                                                                                     fb(b2), sb.pack_weights(dev(w3)), fb(b3)))
    assert torch.equal(k1[:n], t1[:n]) and torch.equal(k2[:n], t2[:n])
    assert_close(to_host(k3)[:n], orc.bottleneck_on_tiles(orc.gather(x, idx_np, og_in), idx_np, og_in, H, W, w1, b1, w2, b2, w3, b3),
                 tol, "t3 of the keeping forward pass")
    # the one-call form runs the same sequence: the same bits
    one = sb.bottleneck_backward_on_tiles(tiles, t1, t2, d3, cnt, (sb.pack_weights_transposed(dev(w1)),
                                                                    sb.pack_weights_transposed(dev(w2)),
                                                                    sb.pack_weights_transposed(dev(w3))))
    for got, want in zip(one, (dtiles, dw1, db1, dw2, db2, dw3, db3)):
        assert torch.equal(got[:n] if got.dim() == 4 and got.shape[0] == n + 1 else got, want[:n] if want.dim() == 4 and want.shape[0] == n + 1 else want)


@pytest.mark.parametrize("n,cap,bo,C,Cm,dtype", [
    (5, 7, 8, 64, 16, "bf16"),         # 10x10 input tiles: one pass of 128 pixels
    (2, 2, 4, 96, 24, "bf16"),         # ... of 64
    (300, 301, 16, 64, 32, "f16"),     # 18x18 tiles, the 384-pixel items
    (40, 301, 16, 64, 32, "bf16"),     # ... and the 256-pixel ones beside them
    (90, 100, 24, 48, 40, "bf16"),     # 26x26: 256 pixels beside 128, channels that end inside a group
    (60, 70, 14, 64, 32, "bf16"),      # 16x16 tiles: the 3x3 data gradient is conv16.hip's, with a pass for the mask
    (20, 24, 30, 48, 64, "f16"),       # 32x32
    (150, 160, 12, 96, 80, "bf16"),    # groups of 96 channels for the single call, likewise
    (3, 4, 8, 24, 8, "f32"),           # no matrix kernel: passes of their own
    (3, 4, 8, 12, 6, "bf16"),
    (0, 3, 8, 64, 16, "bf16"),
])
def test_residual_unit_in_one_call_equals_single_calls(n, cap, bo, C, Cm, dtype):
    """Masks and zeroing in the epilogues of the convolutions, bias sums in one launch: the bits of the single calls."""
    _unit_in_one_call(n, cap, bo, C, Cm, dtype)


@pytest.mark.parametrize("n,cap,bo,C,Cm,dtype,kernel,args", [
    # 3x3 layers of more channel groups than weights stay in LDS for: every item shape of the LDS-tiled kernel
    (5, 7, 8, 64, 200, "bf16", "conv3", (32, 4, 2, 1, 3)),
    (5, 7, 8, 64, 200, "f16", "conv3", (32, 4, 2, 1, 3)),
    (2, 2, 4, 96, 200, "bf16", "conv3", (32, 2, 1, 1, 3)),
    (2, 2, 4, 96, 200, "f16", "conv3", (32, 2, 1, 1, 3)),
    (18, 20, 16, 64, 200, "bf16", "conv3", (32, 4, 2, 1, 6)),
    (18, 20, 16, 64, 200, "f16", "conv3", (32, 4, 2, 1, 6)),
    (36, 40, 16, 64, 200, "bf16", "conv3_pair", (32, 7, 32, 6, 3, 2, 2)),      # one round of 384-pixel items
    (20, 40, 16, 64, 200, "bf16", "conv3_pair", (32, 7, 32, 6, 3, 2, 2)),      # one of 256-pixel ones
    (36, 40, 16, 64, 200, "f16", "conv3_pair", (32, 7, 32, 6, 3, 2, 2)),
    (12, 14, 24, 48, 200, "bf16", "conv3_pair", (32, 6, 32, 6, 2, 1, 2)),      # 256 pixels
    (10, 14, 24, 48, 200, "f16", "conv3_pair", (32, 6, 32, 6, 2, 1, 2)),       # 128
    # lists too long for the kernel that keeps the weights in LDS
    (36, 1000, 16, 64, 64, "bf16", "conv3_pair", (32, 7, 32, 6, 3, 2, 2)),
    (20, 24, 12, 64, 64, "f16", "conv_wave", (2, 2, 1)),                       # ... and that kernel, with groups of 64
])
def test_residual_unit_in_one_call_masks_in_every_kernel(n, cap, bo, C, Cm, dtype, kernel, args):
    """The ReLU mask in the epilogue of the 3x3 data gradient, for every kernel and item shape that has one."""
    backward = _unit_in_one_call(n, cap, bo, C, Cm, dtype)
    of_3x3 = [k for k in kernels(backward) if kernel + "_kernel" in k]
    dt = {"bf16": 1, "f16": 2}[dtype]
    assert [template_args(k) for k in of_3x3] == [(dt, 1, 0, *args) if kernel == "conv_wave" else (dt, 1, 0, *args, 2)]


def _unit_in_one_call(n, cap, bo, C, Cm, dtype):
    step("residual unit, one call %s" % ((n, cap, bo, C, Cm, dtype),))
    r = gen.rng_for(29, n * 100 + bo + C + Cm)
    per = 20 if cap <= 400 else 32
    side = per * bo - 3                             # blocks at the right and bottom edge reach outside the image
    g_in, g_out, _, _ = sb.geometry(side, side, 3, 1, bo)
    th = bo + 2
    cells = np.sort(r.permutation(per * per)[:cap])[::-1].copy()      # the last cells first: the edge is among the active
    idx = torch.from_numpy(np.stack([np.zeros(cap), cells // per, cells % per], 1).astype(np.int32)).cuda()
    cnt = torch.tensor([n], dtype=torch.int32).cuda()
    dev = lambda a: to_dev(gen.round_to(a.astype(np.float32), dtype), dtype)   # noqa: E731
    w1, w2, w3 = (gen.conv_weights(r, k, k, a, b, dtype) for k, a, b in ((1, C, Cm), (3, Cm, Cm), (1, Cm, C)))
    b1, b2, b3 = (torch.from_numpy(gen.bias_vector(r, c, 0.5)).cuda() for c in (Cm, Cm, C))
    p1, p2, p3 = (sb.pack_weights(to_dev(w, dtype)) for w in (w1, w2, w3))
    tiles = dev(gen.activations(r, (cap, th, th, C), dtype))
    t1 = sb.conv_on_tiles(tiles, cnt, p1, b1, relu=True)
    sb.zero_outside(t1, idx, cnt, g_in, side, side)
    t2 = sb.conv_on_tiles(t1, cnt, p2, b2, relu=True)
    t3 = sb.conv_on_tiles(t2, cnt, p3, b3)
    keep = sb.bottleneck_forward_keep_on_tiles(tiles, idx, cnt, g_in, side, side, (p1, b1, p2, b2, p3, b3))
    for got, want in zip(keep, (t1, t2, t3)):
        assert torch.equal(got[:n], want[:n])
    q1, q2, q3 = (sb.pack_weights_transposed(to_dev(w, dtype)) for w in (w1, w2, w3))
    d3 = dev(gen.activations(r, (cap, bo, bo, C), dtype))
    dt2 = sb.conv_on_tiles_backward_data(d3, cnt, q3, bo, bo)
    dt2, db2 = sb.relu_bias_backward_on_tiles(t2, dt2, cnt)
    dt1 = sb.conv_on_tiles_backward_data(dt2, cnt, q2, th, th)
    dt1, db1 = sb.relu_bias_backward_on_tiles(t1, dt1, cnt)
    want = (sb.conv_on_tiles_backward_data(dt1, cnt, q1, th, th), sb.conv_on_tiles_backward_weights(tiles, dt1, cnt, 1), db1,
            sb.conv_on_tiles_backward_weights(t1, dt2, cnt, 3), db2, sb.conv_on_tiles_backward_weights(t2, d3, cnt, 1),
            sb.bias_backward_on_tiles(d3, cnt))
    one = sb.bottleneck_backward_on_tiles(tiles, t1, t2, d3, cnt, (q1, q2, q3))
    assert torch.equal(one[0][:n], want[0][:n])
    for k in range(1, 7):
        assert torch.equal(one[k], want[k]), k
    return lambda: sb.bottleneck_backward_on_tiles(tiles, t1, t2, d3, cnt, (q1, q2, q3))


def test_residual_unit_backward_writes_over_its_incoming_gradient():
    """dL/dx on the input tiles in the memory that dL/dt3 lay in: every step that reads the one runs before the step that
    writes the other."""
    step("residual unit backward, dx over dt3")
    import ctypes
    r = gen.rng_for(34)
    cap, bo, C, Cm = 40, 8, 64, 32
    th = bo + 2
    dev = lambda *shape: to_dev(gen.activations(r, shape, "bf16"), "bf16")   # noqa: E731
    x, t1, t2, dt3 = dev(cap, th, th, C), dev(cap, th, th, Cm), dev(cap, bo, bo, Cm), dev(cap, bo, bo, C)
    q = [sb.pack_weights_transposed(to_dev(gen.conv_weights(r, k, k, a, b, "bf16"), "bf16")) for k, a, b in ((1, C, Cm), (3, Cm, Cm), (1, Cm, C))]
    cnt = torch.tensor([cap], dtype=torch.int32).cuda()
    want = sb.bottleneck_backward_on_tiles(x, t1, t2, dt3, cnt, q)
    got = [torch.empty_like(w) for w in want]
    got[0].view(-1)[:dt3.numel()] = dt3.view(-1)
    need = sb.lib().sbnet_bottleneck_backward_workspace_bytes(sb.BF16, cap, th, th, C, Cm)
    ws = torch.empty((need,), dtype=torch.uint8, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())   # noqa: E731
    assert sb.lib().sbnet_bottleneck_backward_on_tiles(
        p(x), p(t1), p(t2), p(got[0]), sb.BF16, p(cnt), cap, th, th, C, Cm, *[p(w.buf) for w in q], *[p(g) for g in got], p(ws), need,
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == sb.OK
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_weight_gradient_of_a_stack_beyond_two_gib():
    """13 500 tiles of 18 x 18 x 256 (the residual unit's first convolution at the batched configurations' scale) are
    2.24 GB: byte offsets into the stack do not fit 31 bits, and the kernel addresses every tile through a descriptor
    of its own.  Inputs come from a seeded device generator (a host copy serves the oracle: sampled single weights, each a sum
    over every pixel of every tile, and the last tiles' whole contribution)."""
    step("weight gradient, stack beyond 2 GiB")
    n, th, C, K = 13500, 18, 256, 64
    gen_t = torch.Generator(device="cuda")
    gen_t.manual_seed(gen.BASE_SEED + 27)
    x = torch.randn((n, th, th, C), generator=gen_t, device="cuda", dtype=torch.float32).to(torch.bfloat16)
    g = torch.randn((n, th, th, K), generator=gen_t, device="cuda", dtype=torch.float32).to(torch.bfloat16)
    assert x.numel() * 2 > 2 ** 31
    cnt = torch.tensor([n], dtype=torch.int32).cuda()
    dw = sb.conv_on_tiles_backward_weights(x, g, cnt, 1)
    xc, gc = x.cpu(), g.cpu()
    got = dw.cpu().numpy()
    r = gen.rng_for(27)
    samples = [(int(r.integers(0, C)), int(r.integers(0, K))) for _ in range(10)] + [(0, 0), (C - 1, K - 1), (C - 1, 0), (0, K - 1)]
    scale = np.sqrt(n * th * th)
    # one weight of a 1x1 kernel depends on one input and one output channel only: the oracle's weight gradient on
    # those two channel planes of the WHOLE stack is that weight
    def plane(t, c):
        return t[..., c:c + 1].to(torch.float64).numpy()
    for c, o in samples:
        want = float(orc.conv_valid_backward_weights(plane(xc, c), plane(gc, o), 1, 1)[0, 0, 0, 0])
        assert abs(got[0, 0, c, o] - want) <= 2e-5 * scale + 2e-5 * abs(want), (c, o, got[0, 0, c, o], want)
    # the last tiles reach the sums: with three left out, every weight moves by the oracle's gradient of those three
    cnt2 = torch.tensor([n - 3], dtype=torch.int32).cuda()
    dw2 = sb.conv_on_tiles_backward_weights(x, g, cnt2, 1).cpu().numpy()
    tail = orc.conv_valid_backward_weights(xc[n - 3:].to(torch.float64).numpy(), gc[n - 3:].to(torch.float64).numpy(), 1, 1)
    assert np.abs(tail).max() > 10.0
    assert np.abs((got - dw2) - tail).max() <= 4e-5 * scale


def test_pointwise_forward_and_data_gradient_of_a_stack_beyond_two_gib():
    """The same 2.24 GB stack through the pointwise kernel, once as the input of the residual unit's first convolution
    (256 -> 64) and once as the result of that convolution's data gradient (64 -> 256): every tile is addressed from a
    64-bit base through a descriptor of its own.  Sampled tiles, the first and the last among them, against the oracle."""
    step("pointwise forward / data gradient, stack beyond 2 GiB")
    n, th, C, K = 13500, 18, 256, 64
    gen_t = torch.Generator(device="cuda")
    gen_t.manual_seed(gen.BASE_SEED + 29)
    x = torch.randn((n, th, th, C), generator=gen_t, device="cuda", dtype=torch.float32).to(torch.bfloat16)
    assert x.numel() * 2 > 2 ** 31
    r = gen.rng_for(29)
    w = gen.conv_weights(r, 1, 1, C, K, "bf16")
    wd = to_dev(w, "bf16")
    cnt = torch.tensor([n], dtype=torch.int32).cuda()
    y = sb.conv_on_tiles(x, cnt, sb.pack_weights(wd), None, relu=False)
    # whole sampled tiles, the first and the last of the stack among them, against the oracle's tile convolution
    pick = np.unique(np.concatenate([[0, n - 1, n // 2, 6472, 6473], r.integers(0, n, 8)]))   # 6473 * 165888 B > 2^30
    sel = torch.from_numpy(pick).cuda()
    assert_close(to_host(y[sel]), orc.conv_valid(to_host(x[sel]), w), CONV_TOL["bf16"], "pointwise forward, sampled tiles")
    # data gradient: dL/dx = dL/dy W^T, a stack of the size of x
    del x
    dx = sb.conv_on_tiles_backward_data(y, cnt, sb.pack_weights_transposed(wd), th, th)
    assert dx.numel() * 2 > 2 ** 31
    assert_close(to_host(dx[sel]), orc.conv_valid_backward_data(to_host(y[sel]), w, th, th), CONV_TOL["bf16"],
                 "pointwise data gradient, sampled tiles")


def _random_gradient_shapes(n, seed):
    """Seeded draws over what the matrix-core gradient kernels take: 1x1 and 3x3, stride 1 or 2, channels in multiples of 8."""
    r = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        k = (1, 3)[int(r.integers(0, 2))]
        s = int(r.integers(1, 3))
        th, tw = int(r.integers(k, 36)), int(r.integers(k, 36))
        out.append((int(r.integers(1, 7)), th, tw, 8 * int(r.integers(1, 25)), 8 * int(r.integers(1, 25)), k, s,
                    ("bf16", "f16")[int(r.integers(0, 2))]))
    return out


@pytest.mark.parametrize("B,th,tw,Cin,Cout,k,s,dtype", _random_gradient_shapes(24, 18010210))
def test_gradients_on_random_shapes(B, th, tw, Cin, Cout, k, s, dtype):
    """Both gradients on seeded random tiles: rows per stage, segments, stride phases, channel blocks and the choice
    between the pointwise, the 3x3 and the plain kernels all vary with the shape."""
    step("gradients random %s" % ((B, th, tw, Cin, Cout, k, s, dtype),))
    r = gen.rng_for(31, th * 1000 + tw * 10 + Cin + Cout + s + k)
    oh, ow = (th - k) // s + 1, (tw - k) // s + 1
    x = gen.activations(r, (B + 1, th, tw, Cin), dtype)
    g = gen.activations(r, (B + 1, oh, ow, Cout), dtype)
    w = gen.conv_weights(r, k, k, Cin, Cout, dtype)
    cnt = torch.tensor([B], dtype=torch.int32).cuda()
    dw = sb.conv_on_tiles_backward_weights(to_dev(x, dtype), to_dev(g, dtype), cnt, k, stride=s)
    assert_close(to_host(dw), orc.conv_valid_backward_weights(x[:B], g[:B], k, k, stride=s), 2e-5, "weights")
    dx = torch.full((B + 1, th, tw, Cin), 5.0, dtype=TORCH_DT[dtype]).cuda()
    sb.conv_on_tiles_backward_data(to_dev(g, dtype), cnt, sb.pack_weights_transposed(to_dev(w, dtype)), th, tw, stride=s, out=dx)
    got = to_host(dx)
    assert_close(got[:B], orc.conv_valid_backward_data(g[:B], w, th, tw, stride=s), CONV_TOL[dtype], "data")
    assert (got[B] == 5.0).all()
