"""Warm-start network kernels (BF16 MFMA convolutions and the layers around
them) against the FP64 reference of oracle/nn_reference.py.

Inputs are BF16 values, so products are exact in FP32 and the kernels differ
from the FP64 reference only by FP32 accumulation: 1e-5 relative.  The whole
network's gradients are compared with a CPU twin that rounds to BF16 at the
same points (activations, upstream gradients): 2e-3 relative.
"""
import numpy as np
import pytest

from oracle import nn_reference as R
from paper_1508_02960_amd import warmstart as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return W._Ctx("cuda")


def rel(a, b):
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-30))


def _bf_dev(ctx, a):
    t = ctx.torch
    return t.from_numpy(np.ascontiguousarray(a, np.float32)).to(ctx.dev).to(t.bfloat16)


def _f_dev(ctx, a):
    t = ctx.torch
    return t.from_numpy(np.ascontiguousarray(a, np.float32)).to(ctx.dev)


def _host(t):
    return t.float().cpu().numpy().astype(np.float64)


SHAPES = [((2, 6, 4, 8), 8, 8), ((1, 4, 6, 4), 16, 24), ((1, 4, 4, 4), 32, 80),
          ((1, 8, 8, 8), 8, 16),
          # spatially tiled forward path (4 x 8 x 8 tiles, 32-channel chunks):
          # two batch entries, 64 output channels, a ragged channel tile, and 8
          # outputs (16-column tile, as in the head)
          ((2, 16, 32, 32), 32, 32), ((1, 16, 32, 64), 64, 64), ((1, 8, 32, 64), 96, 96),
          ((2, 16, 32, 32), 32, 8),
          # spatially tiled weight gradient (at least 256 tiles): two input
          # channel chunks, two output channel tiles, and 16-channel tiles with
          # zero padding (8 inputs as in the first layer, 8 outputs as in the
          # head, 24 outputs)
          ((2, 16, 32, 64), 64, 32), ((1, 32, 32, 64), 32, 64), ((2, 16, 32, 64), 8, 32),
          ((2, 16, 32, 64), 32, 8), ((1, 32, 32, 64), 16, 24)]


@pytest.mark.parametrize("shape,ci,co", SHAPES)
def test_conv_forward_backward_match_reference(ctx, shape, ci, co):
    rng = np.random.default_rng(ci * 7 + co)
    x = R.bf16(rng.standard_normal(shape + (ci,)))
    w = R.bf16(rng.standard_normal((co, 27, ci)) * 0.2)
    b = rng.standard_normal(co).astype(np.float32).astype(np.float64)
    dy = R.bf16(rng.standard_normal(shape + (co,)))
    lib = W._nn()
    n, d, h, wd = shape
    xd, wb, bd = _bf_dev(ctx, x), _bf_dev(ctx, w), _f_dev(ctx, b)
    y = ctx.f32(n, d, h, wd, co)
    assert lib.nn_conv3d_forward(W._p(xd), W._p(wb), W._p(bd), W._p(y), n, d, h, wd, ci, co,
                                 ctx.stream) == 0
    assert rel(_host(y), R.conv3d(x, w, b)) < 1e-5
    # the fused activation equals the two-step form bit for bit
    for relu in (1, 0):
        a_ref = ctx.bf(n, d, h, wd, co)
        assert lib.nn_activation_forward(W._p(y), W._p(a_ref), y.numel(), relu, ctx.stream) == 0
        a = ctx.bf(n, d, h, wd, co)
        assert lib.nn_conv3d_forward_act(W._p(xd), W._p(wb), W._p(bd), W._p(a), n, d, h, wd, ci,
                                         co, relu, ctx.stream) == 0
        assert ctx.torch.equal(a.view(ctx.torch.int16), a_ref.view(ctx.torch.int16)), relu
    dx_ref, dw_ref, db_ref = R.conv3d_backward(x, w, dy)
    if co % 8 == 0:
        wt = ctx.bf(ci, 27, co)
        assert lib.nn_conv3d_flip_weights(W._p(wb), W._p(wt), ci, co, ctx.stream) == 0
        dx = ctx.f32(n, d, h, wd, ci)
        assert lib.nn_conv3d_backward_data(W._p(_bf_dev(ctx, dy)), W._p(wt), W._p(dx), n, d, h,
                                           wd, ci, co, ctx.stream) == 0
        assert rel(_host(dx), dx_ref) < 1e-5
        import ctypes as C
        nb = C.c_size_t()
        sp = C.c_int()
        assert lib.nn_conv3d_backward_weight_workspace(n, d, h, wd, ci, co, C.byref(nb),
                                                       C.byref(sp)) == 0
        ws = ctx.torch.empty(nb.value, dtype=ctx.torch.uint8, device=ctx.dev)
        dw = ctx.f32(co, 27, ci)
        assert lib.nn_conv3d_backward_weight(W._p(xd), W._p(_bf_dev(ctx, dy)), W._p(dw), W._p(ws),
                                             nb.value, n, d, h, wd, ci, co, ctx.stream) == 0
        assert rel(_host(dw), dw_ref) < 1e-5
        db = ctx.f32(co)
        bb = C.c_size_t()
        assert lib.nn_bias_grad_workspace(n * d * h * wd, co, C.byref(bb)) == 0
        bws = ctx.torch.empty(bb.value, dtype=ctx.torch.uint8, device=ctx.dev)
        assert lib.nn_bias_grad(W._p(_f_dev(ctx, dy)), W._p(db), W._p(bws), bb.value,
                                n * d * h * wd, co, ctx.stream) == 0
        assert rel(_host(db), db_ref) < 1e-5


# one shape per launch of the forward convolution: spatial tiles (8, 4 and 2 rows
# of 16 voxels, rows of 8; one and two groups of 32 channels, 33 outputs: element
# stores), halo tiles (1, 2 and 4 row pairs; partial tiles in every axis; channel
# counts that are no multiple of 32 or 4; four channel groups), gathered tiles
# (many partial tiles; more channels than fit in LDS)
FORWARD_TILES = [((2, 32, 64, 64), 32, 32), ((1, 32, 32, 32), 64, 64), ((1, 16, 32, 64), 32, 32),
                 ((1, 32, 40, 40), 32, 33), ((1, 16, 32, 32), 32, 32), ((1, 32, 32, 24), 8, 32),
                 ((2, 40, 40, 40), 8, 32), ((2, 9, 7, 5), 16, 24), ((1, 3, 2, 1), 8, 8),
                 ((1, 11, 13, 10), 40, 13), ((1, 4, 6, 8), 64, 136), ((1, 4, 4, 8), 704, 16),
                 ((2, 36, 36, 30), 32, 32), ((2, 32, 32, 64), 32, 96),
                 # from packed weights: half-empty tiles, and many blocks
                 ((4, 11, 13, 9), 128, 384), ((3, 20, 20, 20), 128, 160)]


@pytest.mark.parametrize("shape,ci,co", FORWARD_TILES)
def test_conv_forward_tiles_match_reference(ctx, shape, ci, co):
    """BF16 products are exact in FP32, so only the FP32 sum of 27 ci terms
    rounds: 1e-5 of the largest output, as above."""
    rng = np.random.default_rng(ci * 11 + co)
    x = R.bf16(rng.standard_normal(shape + (ci,)))
    w = R.bf16(rng.standard_normal((co, 27, ci)) * 0.2)
    b = rng.standard_normal(co).astype(np.float32).astype(np.float64)
    lib = W._nn()
    n, d, h, wd = shape
    xd, wb, bd = _bf_dev(ctx, x), _bf_dev(ctx, w), _f_dev(ctx, b)
    y = ctx.f32(n, d, h, wd, co)
    assert lib.nn_conv3d_forward(W._p(xd), W._p(wb), W._p(bd), W._p(y), n, d, h, wd, ci, co,
                                 ctx.stream) == 0
    assert rel(_host(y), R.conv3d(x, w, b)) < 1e-5
    a, a_ref = ctx.bf(n, d, h, wd, co), ctx.bf(n, d, h, wd, co)
    assert lib.nn_activation_forward(W._p(y), W._p(a_ref), y.numel(), 1, ctx.stream) == 0
    assert lib.nn_conv3d_forward_act(W._p(xd), W._p(wb), W._p(bd), W._p(a), n, d, h, wd, ci, co, 1,
                                     ctx.stream) == 0
    assert ctx.torch.equal(a.view(ctx.torch.int16), a_ref.view(ctx.torch.int16))


@pytest.mark.parametrize("shape,ci,co", FORWARD_TILES)
def test_packed_weights_give_the_same_bits(ctx, shape, ci, co):
    """nn_conv3d_forward_packed against the unpacked calls, and the packed
    backward-data weights against the flipped ones, bit for bit (the same
    products in the same order)."""
    import ctypes as C

    t, lib = ctx.torch, W._nn()
    n, d, h, wd = shape
    g = t.Generator(device=ctx.dev).manual_seed(ci + co)

    def bf(*s):
        return t.randn(s, generator=g, device=ctx.dev).to(t.bfloat16)

    def packed(ki, ko, flip):
        nb = C.c_size_t()
        assert lib.nn_conv3d_packed_bytes(ki, ko, C.byref(nb)) == 0
        buf = ctx.bf(nb.value // 2)
        assert lib.nn_conv3d_pack_weights(W._p(wb), W._p(buf), ci, co, flip, ctx.stream) == 0
        return buf

    x, wb, b = bf(n, d, h, wd, ci), bf(co, 27, ci), t.randn(co, generator=g, device=ctx.dev)
    wp = packed(ci, co, 0)
    for kind, y in ((0, ctx.f32(n, d, h, wd, co)), (1, ctx.bf(n, d, h, wd, co)),
                    (2, ctx.bf(n, d, h, wd, co))):
        ref = t.empty_like(y)
        if kind == 0:
            assert lib.nn_conv3d_forward(W._p(x), W._p(wb), W._p(b), W._p(ref), n, d, h, wd, ci,
                                         co, ctx.stream) == 0
        else:
            assert lib.nn_conv3d_forward_act(W._p(x), W._p(wb), W._p(b), W._p(ref), n, d, h, wd,
                                             ci, co, kind - 1, ctx.stream) == 0
        assert lib.nn_conv3d_forward_packed(W._p(x), W._p(wp), W._p(b), W._p(y), kind, n, d, h,
                                            wd, ci, co, ctx.stream) == 0
        assert t.equal(y, ref), kind
    assert lib.nn_conv3d_forward_packed(W._p(x), W._p(wp), W._p(b), W._p(y), 3, n, d, h, wd, ci,
                                        co, ctx.stream) != 0
    if co % 8 == 0:
        dy, wt = bf(n, d, h, wd, co), ctx.bf(ci, 27, co)
        wtp = packed(co, ci, 1)
        dx, ref = ctx.f32(n, d, h, wd, ci), ctx.f32(n, d, h, wd, ci)
        assert lib.nn_conv3d_flip_weights(W._p(wb), W._p(wt), ci, co, ctx.stream) == 0
        assert lib.nn_conv3d_backward_data(W._p(dy), W._p(wt), W._p(ref), n, d, h, wd, ci, co,
                                           ctx.stream) == 0
        assert lib.nn_conv3d_forward_packed(W._p(dy), W._p(wtp), None, W._p(dx), 0, n, d, h, wd,
                                            co, ci, ctx.stream) == 0
        assert t.equal(dx, ref)


# weight gradient tiles: 4 x 8 x 8 with more tiles than splits and an uneven count
# (300 over 85), whole planes (four of 8 x 8; one of 16 x 16), rows of a plane
# (8 of 24, 8 of 32, 2 of 64), splits that begin inside a tile (16^3, 43 chunks
# each), partial channel tiles, and edges that leave the general kernel
@pytest.mark.parametrize("shape,ci,co", [((1, 4, 8, 8), 32, 32), ((1, 20, 40, 96), 32, 32),
                                         ((1, 12, 16, 8), 24, 40), ((1, 16, 16, 16), 96, 64),
                                         ((2, 2, 8, 24), 32, 8), ((1, 6, 16, 32), 8, 32),
                                         ((1, 3, 6, 64), 16, 24), ((1, 5, 4, 12), 32, 32)])
def test_conv_weight_gradient_tiles_match_reference(ctx, shape, ci, co):
    """Exact products, FP32 sums over the voxels: 1e-5 of the largest weight's
    gradient, as above."""
    import ctypes as C

    rng = np.random.default_rng(ci * 13 + co)
    x = R.bf16(rng.standard_normal(shape + (ci,)))
    dy = R.bf16(rng.standard_normal(shape + (co,)))
    lib = W._nn()
    n, d, h, wd = shape
    nb, sp = C.c_size_t(), C.c_int()
    assert lib.nn_conv3d_backward_weight_workspace(n, d, h, wd, ci, co, C.byref(nb),
                                                   C.byref(sp)) == 0
    ws = ctx.torch.empty(nb.value, dtype=ctx.torch.uint8, device=ctx.dev)
    dw = ctx.f32(co, 27, ci)
    assert lib.nn_conv3d_backward_weight(W._p(_bf_dev(ctx, x)), W._p(_bf_dev(ctx, dy)), W._p(dw),
                                         W._p(ws), nb.value, n, d, h, wd, ci, co, ctx.stream) == 0
    ref = R.conv3d_backward(x, np.zeros((co, 27, ci)), dy)[1]
    assert rel(_host(dw), ref) < 1e-5


@pytest.mark.parametrize("c", [8, 6])
def test_pool_up_concat_split_relu(ctx, c):
    """c = 8: the 16-byte granule kernels; c = 6: the element kernels."""
    rng = np.random.default_rng(3)
    lib = W._nn()
    s = ctx.stream
    x = R.bf16(rng.standard_normal((2, 4, 6, 8, c)))
    y = ctx.bf(2, 2, 3, 4, c)
    assert lib.nn_pool2_forward(W._p(_bf_dev(ctx, x)), W._p(y), 2, 4, 6, 8, c, s) == 0
    assert rel(_host(y), R.bf16(R.pool2(x))) < 1e-6
    dy = rng.standard_normal((2, 2, 3, 4, c))
    dx = ctx.f32(2, 4, 6, 8, c)
    assert lib.nn_pool2_backward(W._p(_f_dev(ctx, dy)), W._p(dx), 2, 4, 6, 8, c, s) == 0
    assert rel(_host(dx), R.pool2_backward(dy)) < 1e-6
    xc = R.bf16(rng.standard_normal((1, 2, 3, 2, c)))
    yf = ctx.bf(1, 4, 6, 4, c)
    assert lib.nn_upsample2_forward(W._p(_bf_dev(ctx, xc)), W._p(yf), 1, 2, 3, 2, c, s) == 0
    assert np.array_equal(_host(yf), R.up2(xc))
    dyf = rng.standard_normal((1, 4, 6, 4, c))
    dxc = ctx.f32(1, 2, 3, 2, c)
    assert lib.nn_upsample2_backward(W._p(_f_dev(ctx, dyf)), W._p(dxc), 1, 2, 3, 2, c, s) == 0
    assert rel(_host(dxc), R.up2_backward(dyf)) < 1e-6
    a = R.bf16(rng.standard_normal((5, c)))
    b = R.bf16(rng.standard_normal((5, 2 * c)))
    cat = ctx.bf(5, 3 * c)
    assert lib.nn_concat_channels(W._p(_bf_dev(ctx, a)), W._p(_bf_dev(ctx, b)), W._p(cat), 5, c,
                                  2 * c, s) == 0
    assert np.array_equal(_host(cat), np.concatenate([a, b], axis=1))
    g = rng.standard_normal((5, 3 * c))
    ga, gb = ctx.f32(5, c), ctx.f32(5, 2 * c)
    assert lib.nn_split_channels(W._p(_f_dev(ctx, g)), W._p(ga), W._p(gb), 5, c, 2 * c, s) == 0
    assert rel(_host(ga), g[:, :c]) < 1e-7 and rel(_host(gb), g[:, c:]) < 1e-7
    ne = 1000 if c == 8 else 1001  # four-element and element kernels
    z = rng.standard_normal(ne)
    act = ctx.bf(ne)
    assert lib.nn_activation_forward(W._p(_f_dev(ctx, z)), W._p(act), ne, 1, s) == 0
    assert np.array_equal(_host(act), R.bf16(np.maximum(z, 0)))
    cst = ctx.bf(ne)
    assert lib.nn_cast_bf16(W._p(_f_dev(ctx, z)), W._p(cst), ne, s) == 0
    assert np.array_equal(_host(cst), R.bf16(z.astype(np.float32).astype(np.float64)))
    da = rng.standard_normal(ne)
    dz = ctx.f32(ne)
    assert lib.nn_relu_backward(W._p(_f_dev(ctx, da)), W._p(act), W._p(dz), ne, s) == 0
    assert np.allclose(_host(dz), np.where(R.bf16(np.maximum(z, 0)) > 0,
                                           da.astype(np.float32), 0))


@pytest.mark.parametrize("m,c", [(3000, 32), (777, 6), (513, 300)])
def test_relu_backward_bias_fused(ctx, m, c):
    """nn_relu_backward_bias equals nn_relu_backward, nn_cast_bf16 and
    nn_bias_grad bit for bit (c = 300: the wide-channel branch), with and
    without the ReLU; db also against the FP64 sum."""
    import ctypes as C

    t = ctx.torch
    rng = np.random.default_rng(m + c)
    lib = W._nn()
    s = ctx.stream
    da = _f_dev(ctx, rng.standard_normal((m, c)))
    act = _bf_dev(ctx, np.maximum(rng.standard_normal((m, c)), 0))
    bb = C.c_size_t()
    assert lib.nn_bias_grad_workspace(m, c, C.byref(bb)) == 0
    ws = t.empty(bb.value, dtype=t.uint8, device=ctx.dev)
    for relu in (1, 0):
        dz32 = ctx.f32(m, c)
        if relu:
            assert lib.nn_relu_backward(W._p(da), W._p(act), W._p(dz32), m * c, s) == 0
        else:
            dz32.copy_(da)
        dz_ref, db_ref = ctx.bf(m, c), ctx.f32(c)
        assert lib.nn_cast_bf16(W._p(dz32), W._p(dz_ref), m * c, s) == 0
        assert lib.nn_bias_grad(W._p(dz32), W._p(db_ref), W._p(ws), bb.value, m, c, s) == 0
        dz, db = ctx.bf(m, c), ctx.f32(c)
        assert lib.nn_relu_backward_bias(W._p(da), W._p(act) if relu else None, W._p(dz),
                                         W._p(db), W._p(ws), bb.value, m, c, relu, s) == 0
        assert t.equal(dz.view(t.int16), dz_ref.view(t.int16)), relu
        assert t.equal(db, db_ref), relu
        assert rel(_host(db), _host(dz32).sum(axis=0)) < 1e-5
    assert lib.nn_relu_backward_bias(W._p(da), None, W._p(dz), W._p(db), W._p(ws), bb.value,
                                     m, c, 1, s) == 1  # ReLU without the activation


def test_bias_grad_vector_and_scalar_accesses_agree(ctx):
    """Four channels per thread: 16-byte FP32 and 8-byte BF16 accesses when
    the pointers allow them, element accesses in the same order when they do
    not (here: every pointer one element off alignment).  dz and db of the
    fused and plain bias gradients are bit for bit the same either way."""
    import ctypes as C

    t = ctx.torch
    m, c = 2000, 32
    rng = np.random.default_rng(9)
    lib = W._nn()
    s = ctx.stream
    da_h = rng.standard_normal((m, c)).astype(np.float32)
    act_bits = _bf_dev(ctx, np.maximum(rng.standard_normal((m, c)), 0)).reshape(-1)
    bb = C.c_size_t()
    assert lib.nn_bias_grad_workspace(m, c, C.byref(bb)) == 0
    ws = t.empty(bb.value, dtype=t.uint8, device=ctx.dev)
    outs = []
    for off in (0, 1):
        da = t.zeros(m * c + 4, dtype=t.float32, device=ctx.dev)
        da[off:off + m * c] = t.from_numpy(da_h.reshape(-1)).to(ctx.dev)
        act = t.zeros(m * c + 4, dtype=act_bits.dtype, device=ctx.dev)
        act[off:off + m * c] = act_bits
        dz = t.zeros(m * c + 4, dtype=act_bits.dtype, device=ctx.dev)
        db, db_plain = ctx.f32(c), ctx.f32(c)
        pa, pact, pdz = (W._p(x[off:]) for x in (da, act, dz))
        assert lib.nn_relu_backward_bias(pa, pact, pdz, W._p(db), W._p(ws), bb.value, m, c, 1,
                                         s) == 0
        assert lib.nn_bias_grad(pa, W._p(db_plain), W._p(ws), bb.value, m, c, s) == 0
        t.cuda.synchronize()
        outs.append((dz[off:off + m * c].clone(), db.clone(), db_plain.clone()))
    (dz0, db0, dp0), (dz1, db1, dp1) = outs
    assert t.equal(dz0.view(t.int16), dz1.view(t.int16))
    assert t.equal(db0, db1) and t.equal(dp0, dp1)
    assert rel(_host(dp0), da_h.astype(np.float64).sum(axis=0)) < 1e-5


def test_mse_and_adam(ctx):
    rng = np.random.default_rng(4)
    lib = W._nn()
    m = 300
    pred = rng.standard_normal((m, 8)).astype(np.float32)
    tgt = rng.standard_normal((m, 3)).astype(np.float32)
    wgt = (rng.uniform(size=m) > 0.3).astype(np.float32)
    norm = 3.0 * wgt.sum()
    grad = ctx.f32(m, 8)
    part = ctx.torch.empty(64, dtype=ctx.torch.float64, device=ctx.dev)
    assert lib.nn_masked_mse(W._p(_f_dev(ctx, pred)), W._p(_f_dev(ctx, tgt)),
                             W._p(_f_dev(ctx, wgt)), W._p(grad), W._p(part), 64, m, 8, 3, norm,
                             ctx.stream) == 0
    d = pred[:, :3].astype(np.float64) - tgt
    loss = float(np.sum(d ** 2 * wgt[:, None]) / norm)
    assert abs(float(part.sum().item()) - loss) < 1e-6 * loss
    g_ref = np.zeros((m, 8))
    g_ref[:, :3] = 2 * d * wgt[:, None] / norm
    assert rel(_host(grad), g_ref) < 1e-6
    # Adam, two steps against the textbook update
    w = rng.standard_normal(50)
    gs = [rng.standard_normal(50), rng.standard_normal(50)]
    wd, m1, m2 = _f_dev(ctx, w), ctx.zeros(50), ctx.zeros(50)
    ref, a, b = w.copy(), np.zeros(50), np.zeros(50)
    for t, g in enumerate(gs, start=1):
        assert lib.nn_adam(W._p(wd), W._p(_f_dev(ctx, g)), W._p(m1), W._p(m2), None, 50, 1e-2,
                           0.9, 0.999, 1e-8, t, ctx.stream) == 0
        a = 0.9 * a + 0.1 * g
        b = 0.999 * b + 0.001 * g * g
        ref = ref - 1e-2 * (a / (1 - 0.9 ** t)) / (np.sqrt(b / (1 - 0.999 ** t)) + 1e-8)
    assert rel(_host(wd), ref) < 1e-5


def _cpu_unet(net, x, target, weight, norm):
    """CPU twin of UNet forward/backward in FP64 with BF16 rounding where the
    GPU stores BF16 (weights, activations, concatenations, gradients fed to
    the convolution backward)."""
    def wts(conv):
        return (R.bf16(conv.w.cpu().numpy().astype(np.float64)),
                conv.b.cpu().numpy().astype(np.float64))

    e, ins = [], []
    inp = x
    for lvl, conv in enumerate(net.enc):
        if lvl > 0:
            inp = R.bf16(R.pool2(inp))
        ins.append(inp)
        w, b = wts(conv)
        e.append(R.bf16(np.maximum(R.conv3d(inp, w, b), 0)))
        inp = e[-1]
    cur, cats, ds = e[3], {}, {}
    for j, conv in enumerate(net.dec):
        lvl = 2 - j
        cat = np.concatenate([R.up2(cur), e[lvl]], axis=-1)
        cats[lvl] = cat
        w, b = wts(conv)
        cur = R.bf16(np.maximum(R.conv3d(cat, w, b), 0))
        ds[lvl] = cur
    wh, bh = wts(net.head)
    out = R.conv3d(ds[0], wh, bh)
    d = out[..., :3] - target
    loss = np.sum(d ** 2 * weight[..., None]) / norm
    dout = np.zeros_like(out)
    dout[..., :3] = 2 * d * weight[..., None] / norm
    grads = {}
    g, grads["head"], _ = R.conv3d_backward(ds[0], wh, R.bf16(dout))
    skip = {}
    for lvl in (0, 1, 2):
        conv = net.dec[2 - lvl]
        dz = np.where(ds[lvl] > 0, g, 0)
        w, _ = wts(conv)
        dcat, grads[f"dec{lvl}"], _ = R.conv3d_backward(cats[lvl], w, R.bf16(dz))
        cc = net.widths[lvl + 1]
        skip[lvl] = dcat[..., cc:]
        g = R.up2_backward(dcat[..., :cc])
    for lvl in (3, 2, 1, 0):
        if lvl < 3:
            g = g + skip[lvl]
        dz = np.where(e[lvl] > 0, g, 0)
        w, _ = wts(net.enc[lvl])
        dinp, grads[f"enc{lvl}"], _ = R.conv3d_backward(ins[lvl], w, R.bf16(dz))
        if lvl > 0:
            g = R.pool2_backward(dinp)
    return out, loss, grads


def test_unet_gradients_match_cpu_twin(ctx):
    net = W.UNet(widths=(8, 8, 16, 16), seed=7, device="cuda")
    rng = np.random.default_rng(8)
    shape = (1, 16, 16, 16)
    fluid = (rng.uniform(size=shape) > 0.3).astype(np.float32)
    x_np = np.zeros(shape + (8,))
    x_np[..., 0] = fluid
    target = rng.standard_normal(shape + (3,)).astype(np.float32)
    norm = 3.0 * fluid.sum()
    out = net.forward(W.network_input(net.ctx, fluid))
    loss, dout = net.loss(out, _f_dev(ctx, target), _f_dev(ctx, fluid), norm)
    net.backward(dout)
    out_ref, loss_ref, g_ref = _cpu_unet(net, x_np, target.astype(np.float64),
                                         fluid.astype(np.float64), norm)
    assert rel(_host(out), out_ref) < 2e-3
    assert abs(loss / loss_ref - 1) < 2e-3
    assert rel(_host(net.head.gw), g_ref["head"]) < 2e-3
    for lvl in range(3):
        assert rel(_host(net.dec[2 - lvl].gw), g_ref[f"dec{lvl}"]) < 2e-3, lvl
    for lvl in range(4):
        assert rel(_host(net.enc[lvl].gw), g_ref[f"enc{lvl}"]) < 2e-3, lvl


def test_unet_training_reduces_loss(ctx):
    """Adam steps on a learnable target lower the loss.  The network is
    translation-equivariant, so the target is a local function of the mask:
    the fluid fraction of each voxel's 3x3x3 neighbourhood, on fluid voxels."""
    from scipy import ndimage

    net = W.UNet(widths=(8, 16, 16, 32), seed=9, device="cuda")
    rng = np.random.default_rng(10)
    shape = (2, 16, 16, 16)
    fluid = (rng.uniform(size=shape) > 0.3).astype(np.float32)
    local = np.stack([ndimage.uniform_filter(f, size=3, mode="wrap") for f in fluid])
    target = (local * fluid)[..., None] * np.array([1.0, -0.5, 0.25])
    target = target.astype(np.float32)
    x = W.network_input(net.ctx, fluid)
    t, wgt = _f_dev(ctx, target), _f_dev(ctx, fluid)
    losses = []
    for _ in range(40):
        out = net.forward(x)
        loss, g = net.loss(out, t, wgt, 3.0 * fluid.sum())
        net.backward(g)
        net.adam_step(1e-2)
        losses.append(loss)
    assert losses[-1] < 0.3 * losses[0], losses


@pytest.mark.parametrize("shape,ca,cb", [((1, 2, 2, 2), 8, 8), ((2, 3, 5, 7), 16, 8),
                                         ((1, 4, 6, 10), 24, 48), ((3, 8, 8, 8), 64, 32)])
def test_fused_sampling_steps_give_the_same_bits(ctx, shape, ca, cb):
    """Upsampling with concatenation, its gradient, and the bias gradient that
    forms its input from the pooled and the concatenated gradients: bit for bit
    the single steps (shape: the coarse box; the fine one has odd halves)."""
    import ctypes as C

    t = ctx.torch
    rng = np.random.default_rng(ca + cb)
    lib = W._nn()
    s = ctx.stream
    n, d, h, w = shape
    fine = (n, 2 * d, 2 * h, 2 * w)
    m = int(np.prod(fine))
    a, b = _bf_dev(ctx, rng.standard_normal(shape + (ca,))), _bf_dev(
        ctx, rng.standard_normal(fine + (cb,)))
    up, want, got = ctx.bf(*fine, ca), ctx.bf(*fine, ca + cb), ctx.bf(*fine, ca + cb)
    assert lib.nn_upsample2_forward(W._p(a), W._p(up), n, d, h, w, ca, s) == 0
    assert lib.nn_concat_channels(W._p(up), W._p(b), W._p(want), m, ca, cb, s) == 0
    assert lib.nn_upsample_concat(W._p(a), W._p(b), W._p(got), n, d, h, w, ca, cb, s) == 0
    assert t.equal(got.view(t.int16), want.view(t.int16))

    dcat = _f_dev(ctx, rng.standard_normal(fine + (ca + cb,)))
    dup, dskip = ctx.f32(*fine, ca), ctx.f32(*fine, cb)
    da, da_want = ctx.f32(*shape, ca), ctx.f32(*shape, ca)
    assert lib.nn_split_channels(W._p(dcat), W._p(dup), W._p(dskip), m, ca, cb, s) == 0
    assert lib.nn_upsample2_backward(W._p(dup), W._p(da_want), n, d, h, w, ca, s) == 0
    assert lib.nn_concat_upsample_backward(W._p(dcat), W._p(da), n, d, h, w, ca, cb, s) == 0
    assert t.equal(da, da_want)

    pooled, act = _f_dev(ctx, rng.standard_normal(shape + (cb,))), _bf_dev(
        ctx, np.maximum(rng.standard_normal(fine + (cb,)), 0))
    g = ctx.f32(*fine, cb)
    assert lib.nn_pool2_backward(W._p(pooled), W._p(g), *fine, cb, s) == 0
    assert lib.nn_add(W._p(g), W._p(dskip), g.numel(), s) == 0
    bb = C.c_size_t()
    assert lib.nn_bias_grad_workspace(m, cb, C.byref(bb)) == 0
    ws = t.empty(bb.value, dtype=t.uint8, device=ctx.dev)
    for relu in (1, 0):
        out = []
        for dz, db in ((ctx.bf(*fine, cb), ctx.f32(cb)), (ctx.bf(*fine, cb), ctx.f32(cb))):
            if not out:
                st = lib.nn_relu_backward_bias(W._p(g), W._p(act), W._p(dz), W._p(db), W._p(ws),
                                               bb.value, m, cb, relu, s)
            else:
                st = lib.nn_pooled_backward_bias(W._p(pooled), W._p(dcat), ca, W._p(act),
                                                 W._p(dz), W._p(db), W._p(ws), bb.value, *fine,
                                                 cb, relu, s)
            assert st == 0
            out.append((dz, db))
        assert t.equal(out[0][0].view(t.int16), out[1][0].view(t.int16)) and t.equal(
            out[0][1], out[1][1])
    assert lib.nn_pooled_backward_bias(W._p(pooled), W._p(dcat), ca, W._p(act), W._p(dz), W._p(db),
                                       W._p(ws), bb.value, n, 2 * d, 2 * h, 2 * w - 1, cb, 1,
                                       s) == 1  # odd edges cannot have been pooled


@pytest.mark.parametrize("sizes", [[5], [1024, 1, 0, 1025, 300], [257] * 60])
def test_updates_and_packings_of_many_tensors_give_the_same_bits(ctx, sizes):
    """nn_adam_many and nn_conv3d_pack_weights_many (one block's span, its edges,
    an empty tensor, more tensors than one launch takes) against the calls per
    tensor."""
    import ctypes as C

    t = ctx.torch
    rng = np.random.default_rng(len(sizes))
    lib = W._nn()
    s = ctx.stream

    def tensors(seed):
        r = np.random.default_rng(seed)
        return [[_f_dev(ctx, np.abs(r.standard_normal(n + 1))) for _ in range(4)]
                + [ctx.bf(n + 1).zero_()] for n in sizes]

    one, many = tensors(3), tensors(3)
    for n, q in zip(sizes, one):
        assert not n or lib.nn_adam(*map(W._p, q), n, 1e-2, 0.9, 0.999, 1e-8, 3, s) == 0
    rows = [tuple(v.data_ptr() for v in q) + (n,) for n, q in zip(sizes, many)]
    assert lib.nn_adam_many(*W._items(W._AdamTensor, rows), 1e-2, 0.9, 0.999, 1e-8, 3, s) == 0
    for a, b in zip(one, many):
        assert all(t.equal(x.view(t.int16), y.view(t.int16)) for x, y in zip(a, b))

    shapes = [(8, 5), (32, 16), (16, 48), (64, 24)][:len(sizes)] * (1 if len(sizes) < 30 else 8)
    items, pairs = [], []
    for ci, co in shapes:
        w = _bf_dev(ctx, rng.standard_normal((co, 27, ci)))
        for flip in (0, 1) if co % 8 == 0 else (0,):
            nb = C.c_size_t()
            assert lib.nn_conv3d_packed_bytes(*((co, ci) if flip else (ci, co)), C.byref(nb)) == 0
            a, b = ctx.bf(nb.value // 2), ctx.bf(nb.value // 2)
            assert lib.nn_conv3d_pack_weights(W._p(w), W._p(a), ci, co, flip, s) == 0
            items.append((w.data_ptr(), b.data_ptr(), ci, co, flip))
            pairs.append((a, b, w))
    assert lib.nn_conv3d_pack_weights_many(*W._items(W._PackItem, items), s) == 0
    assert all(t.equal(a.view(t.int16), b.view(t.int16)) for a, b, _ in pairs)


@pytest.mark.parametrize("m", [1, 300, 4097, 131072])
@pytest.mark.parametrize("c", [4, 33, 64])
def test_bias_gradient_folds_every_split(ctx, m, c):
    """One split to 512, channel counts around a block's 32.  Positive terms, so
    a chain of at most 64 + 64 + 512 additions rounds by less than 640 2^-24 of
    the sum."""
    import ctypes as C

    rng = np.random.default_rng(m + c)
    dy = _f_dev(ctx, rng.uniform(0.5, 1.0, (m, c)))
    lib = W._nn()
    bb = C.c_size_t()
    assert lib.nn_bias_grad_workspace(m, c, C.byref(bb)) == 0
    ws = ctx.torch.full((bb.value,), 255, dtype=ctx.torch.uint8, device=ctx.dev)
    db = ctx.f32(c)
    assert lib.nn_bias_grad(W._p(dy), W._p(db), W._p(ws), bb.value, m, c, ctx.stream) == 0
    want = _host(dy).sum(axis=0)
    assert np.max(np.abs(_host(db) - want) / want) < 640 * 2.0**-24


def test_weights_written_by_the_caller_reach_the_convolutions(ctx):
    """Conv.wb and Conv.wt are the operands of the forward and the backward-data
    convolution also after a caller has written or replaced them; refresh and
    the optimizer step renew both, also through tensors handed out before; and
    a layer that handed them out computes the bits of one that did not."""
    t = ctx.torch
    shape, ci, co = (1, 4, 8, 8), 32, 48
    rng = np.random.default_rng(23)
    x = _bf_dev(ctx, rng.standard_normal(shape + (ci,)))
    dy = _f_dev(ctx, rng.standard_normal(shape + (co,)))

    def layer(seed):
        return W.Conv(ctx, ci, co, np.random.default_rng(seed))

    def results(c):
        dx = c.backward(x, dy, shape)
        return [v.clone() for v in (c.forward(x, shape), c.forward_act(x, shape), dx)]

    def same(a, b):
        return [t.equal(p, q) for p, q in zip(a, b)]

    c, other, twin = layer(1), layer(2), layer(1)
    ra, rb = results(twin), results(other)
    assert same(ra, rb) == [False] * 3
    wb, wt = c.wb, c.wt
    assert same(results(c), ra) == [True] * 3
    wb.copy_(other.wb)  # forward follows at once, backward-data reads wt
    assert same(results(c), [rb[0], rb[1], ra[2]]) == [True] * 3
    wt.copy_(other.wt)
    assert same(results(c), rb) == [True] * 3
    c.refresh()  # both from the master weights again
    assert same(results(c), ra) == [True] * 3
    assert t.equal(wb, c.wb) and t.equal(wt, c.wt)
    for step in (1, 2):  # the gradients of both are those of the last results()
        c.adam(1e-2, step)
        twin.adam(1e-2, step)
        r = results(twin)
        assert same(results(c), r) == [True] * 3
        assert same(r, ra) == [False] * 3
    assert t.equal(wb, twin.wb) and t.equal(wt, twin.wt)
    c.wb, c.wt, c.b = other.wb, other.wt, other.b
    assert same(results(c), rb) == [True] * 3


@pytest.mark.parametrize("widths,shape", [((16, 24, 32, 40), (2, 8, 16, 24)),
                                          ((32, 64, 128, 256), (1, 184, 184, 184))])
def test_unet_with_single_calls_gives_the_same_bits(ctx, monkeypatch, widths, shape):
    """UNet forward and backward through the fused up- and downsampling calls
    and through the single ones that boxes beyond their limits take: the same
    output and gradients bit for bit (a small box of odd levels, and one whose
    voxels times the widest concatenation exceed 2^31)."""
    t = ctx.torch
    g = t.Generator(device="cuda").manual_seed(17)
    net = W.UNet(widths=widths, seed=3, device="cuda")
    x = W.network_input(net.ctx, (t.rand(shape, generator=g, device="cuda") > 0.3).to(t.uint8))
    dout = t.randn(shape + (8,), generator=g, device="cuda")
    runs = []
    for fused in (True, False):
        if not fused:
            monkeypatch.setattr(W.UNet, "_fused", lambda self, s: False)
        assert net._fused(shape) is fused
        out = net.forward(x)
        net.backward(dout)
        runs.append([out] + [v.clone() for l in net.layers() for v in (l.gw, l.gb)])
    assert all(t.equal(a, b) for a, b in zip(*runs))
    assert all(bool(t.isfinite(a).all()) and float(a.abs().max()) > 0 for a in runs[0])


# boxes whose edges leave halo tiles mostly empty (gathered tiles of 64 and 32
# channels, the last ones partial; a K of 3.4 stages; from packed weights halo
# tiles for the last), channels that do not fit in LDS (gathered tiles of 16 and
# 32 channels, 300.4 stages), and odd numbers of channel octets in halo tiles
@pytest.mark.parametrize("shape,ci,co", [((30, 30, 8, 1), 8, 200), ((12, 30, 17, 1), 120, 100),
                                         ((40, 30, 20, 1), 8, 24), ((1, 4, 4, 8), 712, 16),
                                         ((1, 4, 4, 8), 712, 24), ((1, 9, 8, 10), 56, 40),
                                         ((24, 48, 4, 2), 16, 72)])
def test_conv_forward_of_thin_boxes_and_odd_octets(ctx, shape, ci, co):
    test_conv_forward_tiles_match_reference(ctx, shape, ci, co)
    test_packed_weights_give_the_same_bits(ctx, shape, ci, co)


# splits of two and three chunks of 64 voxels over tiles of three and four 8 x 8
# planes, two of 16 x 8, 16 x 16, 8 and 3 rows of a plane, with partial channel
# tiles on either side and on both, in one LDS buffer and in two
@pytest.mark.parametrize("shape,ci,co", [((1, 52, 8, 8), 96, 96), ((1, 12, 16, 8), 104, 136),
                                         ((2, 10, 8, 24), 96, 72), ((1, 6, 16, 32), 72, 168),
                                         ((1, 3, 18, 64), 88, 96), ((3, 7, 16, 16), 160, 24),
                                         ((5, 6, 8, 8), 128, 96)])
def test_conv_weight_gradient_in_tiles_of_rows(ctx, shape, ci, co):
    test_conv_weight_gradient_tiles_match_reference(ctx, shape, ci, co)
