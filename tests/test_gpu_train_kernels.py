"""Training kernels against float64 sums, at the sizes where a tile, a channel block or a row
ends: every element within the bound of its own FP32 sum,
(K + 2) 2^-24 times the sum of its terms' magnitudes."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, say
from oracle import encoder as E

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _within(got, want, S, K):
    err = (got.detach().to("cpu", torch.float64) - want).abs()
    bound = (K + 2) * U * S
    return bool((err <= bound).all()), float((err / bound.clamp_min(1e-300)).max())


def _adjoint_terms(fine, coarse):
    """The weight gradient sum_{b,o} coarse[b,co,o] fine[b,ci,2o+k-1] in float64."""
    w = torch.zeros((coarse.shape[1], fine.shape[1], 3, 3, 3), dtype=torch.float64).requires_grad_()
    return torch.autograd.grad((E.conv(fine, w, None, False) * coarse).sum(), w)[0]


# (B, Ci, Co, D, H, W): rows that divide a wave and rows that do not, chunks of 4,096 positions
# with a rest and with many samples, channel blocks of 4 with a rest, one voxel per sample.
WGRAD = [(2, 2, 8, 10, 12, 32), (1, 1, 17, 18, 6, 64), (3, 8, 16, 6, 10, 32), (2, 9, 33, 4, 6, 32),
         (2, 2, 16, 10, 14, 16), (2, 16, 32, 6, 10, 48), (3, 20, 8, 10, 6, 8), (5, 32, 64, 8, 8, 8),
         (4, 3, 5, 10, 12, 6), (2, 1, 64, 6, 4, 2), (7, 40, 48, 2, 2, 10), (2, 2, 8, 2, 10, 14), (5000, 1, 3, 2, 2, 2),
         (1, 2, 5, 4, 6, 128), (1, 1, 2, 6, 8, 136)]


@pytest.mark.parametrize("shape", WGRAD)
def test_conv_weight_gradient(shape):
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    say(f"weight gradient {shape}")
    g = torch.Generator().manual_seed(sum(shape))
    fine = torch.randn(B, Ci, D, H, W, generator=g, dtype=torch.float64).float()
    coarse = torch.randn(B, Co, D // 2, H // 2, W // 2, generator=g, dtype=torch.float64).float()
    w = torch.randn(Co, Ci, 3, 3, 3, generator=g)
    f64, c64 = fine.double(), coarse.double()
    want, S = _adjoint_terms(f64, c64), _adjoint_terms(f64.abs(), c64.abs())
    K = B * (D // 2) * (H // 2) * (W // 2)
    ws = w.cuda().requires_grad_()
    bs = torch.zeros(Co, device="cuda").requires_grad_()
    y = nn.Conv3dS2.apply(fine.cuda(), ws, bs, ws.detach(), False)
    gw, gb = torch.autograd.grad(y, (ws, bs), coarse.cuda())
    ok, worst = _within(gw, want, S, K)
    assert ok, (shape, "dw", worst)
    ok, worst = _within(gb, c64.sum((0, 2, 3, 4)), c64.abs().sum((0, 2, 3, 4)), K)
    assert ok, (shape, "db", worst)
    # The transposed convolution: roles exchanged, its bias gradient from the fine side.
    bt = torch.zeros(Ci, device="cuda").requires_grad_()
    y = nn.ConvT3dS2.apply(coarse.cuda(), ws, bt, ws.detach(), False)
    gw, gb = torch.autograd.grad(y, (ws, bt), fine.cuda())
    ok, worst = _within(gw, want, S, K)
    assert ok, (shape, "dw of the transpose", worst)
    ok, worst = _within(gb, f64.sum((0, 2, 3, 4)), f64.abs().sum((0, 2, 3, 4)), 8 * K)
    assert ok, (shape, "db of the transpose", worst)


# (B, Ci, Co, D, H, W): the tile of one and two fine channels and the four parity tiles, each
# register size (8, 16, 32, 64 coarse channels, exact and with a rest), channel blocks of eight
# with a rest, groups of 16 voxels across rows and samples and past the last one; odd channel
# counts take the direct loop.
ADJOINT = [(2, 2, 8, 10, 12, 32), (3, 1, 4, 6, 10, 6), (1, 2, 16, 4, 4, 34), (2, 2, 40, 4, 6, 8),
           (2, 8, 16, 6, 8, 32), (3, 3, 10, 6, 10, 14), (2, 16, 32, 10, 6, 18), (5, 9, 18, 2, 6, 2),
           (3, 32, 64, 8, 8, 8), (4, 20, 34, 4, 2, 6), (7, 1, 8, 2, 2, 2), (2, 4, 7, 6, 4, 8)]


@pytest.mark.parametrize("shape", ADJOINT)
def test_conv_adjoint(shape):
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    g = torch.Generator().manual_seed(sum(shape) + 1)
    coarse = torch.randn(B, Co, D // 2, H // 2, W // 2, generator=g)
    w = torch.randn(Co, Ci, 3, 3, 3, generator=g) * 0.2
    b = torch.randn(Ci, generator=g)
    for wc in (w.to(torch.bfloat16), w):
        for bias in (b, None):
            for relu in (False, True):
                say(f"adjoint {shape} {wc.dtype} bias={bias is not None} relu={relu}")
                bd = None if bias is None else bias.cuda()
                y = nn.ConvT3dS2.apply(coarse.cuda(), w.cuda(), bd, wc.cuda(), relu)
                b64 = None if bias is None else bias.double()
                yr = E.conv_t(coarse.double(), wc.double(), b64, relu)
                S = E.conv_t(coarse.double().abs(), wc.double().abs(),
                             None if b64 is None else b64.abs(), False)
                ok, worst = _within(y, yr, S, 8 * Co)
                assert ok, (shape, wc.dtype, relu, worst)


@pytest.mark.parametrize("shape", [(2, 2, 8, 8, 8, 32), (2, 12, 16, 6, 8, 10), (2, 16, 64, 4, 4, 4)])
def test_conv_adjoint_keeps_infinities_and_nans_local(shape):
    """An infinity or a NaN reaches only the outputs whose taps hold it, with the direct loop's
    result (the float64 kernel's)."""
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    g = torch.Generator().manual_seed(5)
    coarse = torch.randn(B, Co, D // 2, H // 2, W // 2, generator=g)
    w = torch.randn(Co, Ci, 3, 3, 3, generator=g) * 0.2
    for c, z, y, x, val in ((0, 0, 0, 0, float("inf")), (Co - 1, D // 2 - 1, H // 2 - 1, W // 2 - 1, float("-inf")),
                            (1, 1, 0, 1, float("nan"))):
        coarse[0, c, z, y, x] = val
    got = nn.ConvT3dS2.apply(coarse.cuda(), w.cuda(), None, w.cuda(), False).cpu()
    want = nn.ConvT3dS2.apply(coarse.cuda().double(), w.cuda().double(), None, w.cuda().double(), False).cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(torch.isposinf(got), torch.isposinf(want))
    assert torch.equal(torch.isneginf(got), torch.isneginf(want))
    assert torch.isfinite(got).any() and not torch.isfinite(got).all()


# (B, Ci, Co, D, H, W): the first layer's kernel (one and two fine channels, rows of fours that
# start a wave and that do not, coarse channels past eight); by chunk (channels in fours, rows of
# fours) and by channel (the rest) with one and two groups of voxels per wave, terms that do not
# fill a product or a batch, 16-channel tiles with a rest, up to 32 fine channels and past them.
FORWARD = [(2, 2, 8, 8, 6, 64), (3, 1, 11, 6, 10, 24), (2, 2, 5, 4, 4, 8), (1, 1, 8, 10, 6, 256),
           (2, 2, 8, 4, 6, 12), (3, 4, 16, 6, 4, 8), (2, 32, 64, 8, 8, 8), (5, 12, 20, 4, 6, 12),
           (2, 3, 9, 6, 8, 10), (3, 32, 33, 4, 4, 6), (2, 5, 16, 8, 6, 32), (2, 36, 16, 4, 4, 8),
           (9, 8, 16, 32, 32, 24), (17, 6, 16, 32, 32, 18)]


@pytest.mark.parametrize("shape", FORWARD)
def test_conv_forward(shape):
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    g = torch.Generator().manual_seed(sum(shape) + 2)
    fine = torch.randn(B, Ci, D, H, W, generator=g)
    w = torch.randn(Co, Ci, 3, 3, 3, generator=g) * 0.2
    b = torch.randn(Co, generator=g)
    S = E.conv(fine.double().abs(), w.double().abs() * 1.01, b.double().abs(), False)
    for wc in (w.to(torch.bfloat16), w):
        for bias in (b, None):
            for relu in (False, True):
                say(f"forward {shape} {wc.dtype} bias={bias is not None} relu={relu}")
                y = nn.Conv3dS2.apply(fine.cuda(), w.cuda(), None if bias is None else bias.cuda(),
                                      wc.cuda(), relu)
                yr = E.conv(fine.double(), wc.double(), None if bias is None else bias.double(), relu)
                ok, worst = _within(y, yr, S, 27 * Ci)
                assert ok, (shape, wc.dtype, relu, worst)


@pytest.mark.parametrize("shape", [(3, 3, 9, 6, 8, 10), (3, 5, 16, 4, 6, 12), (2, 6, 20, 8, 4, 6), (3, 7, 8, 4, 4, 10),
                                   (2, 9, 16, 6, 6, 6), (3, 13, 5, 2, 4, 6), (3, 8, 16, 8, 8, 8), (3, 2, 8, 8, 8, 16)])
def test_conv_forward_keeps_infinities_and_nans_in_their_sample(shape):
    """Fine channels that do not fill a product or a batch: an infinity or a NaN of one sample
    reaches only the outputs whose taps hold it (the float64 kernel's), and the other samples'
    bits are those of a batch without it."""
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    say(f"forward, special values in sample 1 {shape}")
    g = torch.Generator().manual_seed(7)
    fine = torch.randn(B, Ci, D, H, W, generator=g)
    w = torch.randn(Co, Ci, 3, 3, 3, generator=g) * 0.2
    clean = nn.Conv3dS2.apply(fine.cuda(), w.cuda(), None, w.cuda(), False).cpu()
    fine[1, :, ::3, ::2, ::4] = float("inf")
    fine[1, :, 1::3, 1::2, ::5] = float("nan")
    got = nn.Conv3dS2.apply(fine.cuda(), w.cuda(), None, w.cuda(), False).cpu()
    want = nn.Conv3dS2.apply(fine.cuda().double(), w.cuda().double(), None, w.cuda().double(), False).cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(torch.isposinf(got), torch.isposinf(want))
    assert torch.equal(torch.isneginf(got), torch.isneginf(want))
    for b in range(B):
        assert b == 1 or torch.equal(got[b], clean[b]), b
    assert not torch.isfinite(got[1]).all()


# (B, In, Out): tiles of 16 rows and 16 or 64 columns with a rest, terms that end inside a chunk of
# 64, one chunk, several chunks in flight and past them; In not a multiple of 4 (the direct loop).
LINEAR = [(32, 512, 640), (7, 68, 36), (17, 1028, 20), (1, 4, 4), (33, 64, 2116), (5, 4096, 16), (3, 30, 8)]


@pytest.mark.parametrize("shape", LINEAR)
def test_linear_small_batch(shape):
    """Forward and all gradients; the split head with one slice gives the same bits."""
    need_gpu()
    from paper_2205_04550_amd import nn
    B, In, Out = shape
    g = torch.Generator().manual_seed(B + In + Out + 3)
    x, w = torch.randn(B, In, generator=g), torch.randn(Out, In, generator=g) * 0.1
    b, gy = torch.randn(Out, generator=g), torch.randn(B, Out, generator=g)
    for wc in (w.to(torch.bfloat16), w):
        say(f"linear {shape} {wc.dtype}")
        xd, wd, bd = x.cuda().requires_grad_(), w.cuda().requires_grad_(), b.cuda().requires_grad_()
        y = nn.Linear.apply(xd, wd, bd, wc.cuda(), False)
        if wc.dtype == torch.bfloat16 and In % 4 == 0:
            assert torch.equal(y, nn.linear_split(x.cuda(), wc.cuda(), b.cuda(), False, splits=1))
        gx, gw, gb = torch.autograd.grad(y, (xd, wd, bd), gy.cuda())
        x64, w64, g64 = x.double(), wc.double(), gy.double()
        for name, got, want, S, K in (
                ("y", y, x64 @ w64.T + b.double(), x64.abs() @ w64.abs().T + b.double().abs(), In),
                ("dx", gx, g64 @ w64, g64.abs() @ w64.abs(), Out),
                ("dw", gw, g64.T @ x64, g64.abs().T @ x64.abs(), B),
                ("db", gb, g64.sum(0), g64.abs().sum(0), B)):
            ok, worst = _within(got, want, S, K)
            assert ok, (shape, name, worst)


@pytest.mark.parametrize("shape", [(16, 68, 4096), (16, 68, 4112), (31, 64, 64), (32, 64, 64), (32, 256, 4096),
                                   (32, 260, 4096), (32, 260, 4112), (4, 256, 128), (4, 256, 132), (31, 64, 68),
                                   (32, 64, 128), (32, 4032, 68), (32, 4096, 68), (64, 4096, 256), (64, 4160, 256),
                                   (32, 16384, 260), (48, 16384, 260)])
def test_linear_either_side_of_the_small_batch_rule(shape):
    """Rows, columns and terms where the kernels of a small batch give way to the 64 x 64 tiles."""
    test_linear_small_batch(shape)


def test_adam_of_several_tensors_equals_one_by_one():
    """One launch for 37 tensors (more than a table holds, sizes around a block of 1,024 and
    pointers off 16 bytes) leaves the bits of a launch per tensor."""
    need_gpu()
    import ctypes
    from paper_2205_04550_amd.binding import LIB, _check
    g = torch.Generator().manual_seed(3)
    sizes = [1, 3, 4, 1023, 1024, 1025, 5000] + [17 + 64 * i for i in range(30)]
    st = torch.cuda.current_stream().cuda_stream

    def tensors():
        g.manual_seed(3)
        out = []
        for i, n in enumerate(sizes):
            t = [torch.randn(n + 1, generator=g).cuda()[i % 2:][:n] for _ in range(4)]
            t[2].abs_()
            out.append(t + [torch.zeros(n, dtype=torch.bfloat16, device="cuda") if i % 3 else None])
        return out

    one, many = tensors(), tensors()
    p = lambda t: None if t is None else t.data_ptr()
    for w, m, v, gr, wb in one:
        _check(LIB.nn_adam_step(w.numel(), p(w), p(m), p(v), p(gr), p(wb), 1e-3, 0.9, 0.999, 1e-8, 2, st))
    k = len(sizes)
    col = lambda i: (ctypes.c_void_p * k)(*(p(t[i]) for t in many))
    _check(LIB.nn_adam_step_multi(k, (ctypes.c_int64 * k)(*sizes), col(0), col(1), col(2), col(3), col(4),
                                  1e-3, 0.9, 0.999, 1e-8, 2, st))
    for a, b in zip(one, many):
        for x, y in zip(a, b):
            assert (x is None) == (y is None) and (x is None or torch.equal(x, y))


@pytest.mark.parametrize("shape", [(2, 2, 8, 8, 8, 64), (3, 1, 6, 6, 10, 12)])
def test_first_layer_gradient_masked_as_it_is_read(shape):
    """A layer whose input needs no gradient masks dY by its ReLU inside the weight gradient:
    the same bits as with the input gradient (the masked gradient written first)."""
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    g = torch.Generator().manual_seed(8)
    x = torch.randn(B, Ci, D, H, W, generator=g).cuda()
    w = (torch.randn(Co, Ci, 3, 3, 3, generator=g) * 0.2).cuda().requires_grad_()
    b = torch.randn(Co, generator=g).cuda().requires_grad_()
    gy = torch.randn(B, Co, D // 2, H // 2, W // 2, generator=g).cuda()
    a = torch.autograd.grad(nn.Conv3dS2.apply(x, w, b, w.detach(), True), (w, b), gy)
    xr = x.clone().requires_grad_()
    c = torch.autograd.grad(nn.Conv3dS2.apply(xr, w, b, w.detach(), True), (w, b, xr), gy)
    assert torch.equal(a[0], c[0]) and torch.equal(a[1], c[1])


def test_adam_moments_bits():
    """The moments after each of four steps, bit for bit: m = fma(1 - b1, g, b1 m) and
    v = fma(g, (1 - b2) g, b2 v) in float32 (products exact in float64, one rounding of the sum)."""
    need_gpu()
    from paper_2205_04550_amd.binding import LIB
    f = np.float32
    n, b1, b2 = 1027, f(0.9), f(0.999)
    rng = np.random.default_rng(5)
    w = torch.randn(n, device="cuda")
    m, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    mh, vh = np.zeros(n, f), np.zeros(n, f)
    for t in range(1, 5):
        g = rng.standard_normal(n).astype(f)
        gd = torch.from_numpy(g).cuda()
        say(f"adam step {t}")
        rc = LIB.nn_adam_step(n, w.data_ptr(), m.data_ptr(), v.data_ptr(), gd.data_ptr(), None, 1e-3, 0.9,
                              0.999, 1e-8, t, torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        torch.cuda.synchronize()
        mh = ((f(1) - b1).astype(np.float64) * g + (b1 * mh).astype(np.float64)).astype(f)
        vh = (g.astype(np.float64) * ((f(1) - b2) * g).astype(np.float64) + (b2 * vh)).astype(f)
        assert np.array_equal(m.cpu().numpy().view(np.uint32), mh.view(np.uint32)), t
        assert np.array_equal(v.cpu().numpy().view(np.uint32), vh.view(np.uint32)), t


@pytest.mark.parametrize("B,C,S", [(70000, 3, 1), (20000, 2, 3), (5000, 4, 27), (3, 2, 255), (40, 3, 256), (9, 2, 4097)])
def test_channel_sum(B, C, S):
    """Sums over samples and positions, in float and (with its input's ReLU, as a transposed
    convolution's backward) from rows shorter and longer than the 256 positions of a step."""
    need_gpu()
    from paper_2205_04550_amd.nn import LIB, _check
    say(f"channel sum {B} x {C} x {S}")
    g = torch.Generator().manual_seed(B + C + S)
    x = torch.randn(B, C, S, generator=g, dtype=torch.float64)
    st = torch.cuda.current_stream().cuda_stream
    for dtype, xd in ((0, x.float().cuda()), (1, x.cuda())):
        out = torch.empty(C, dtype=xd.dtype, device="cuda")
        nb = LIB.nn_channel_sum_ws_bytes(dtype, B, C, S)
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
        _check(LIB.nn_channel_sum(dtype, B, C, S, xd.data_ptr(), out.data_ptr(), ws.data_ptr(), nb, st))
        h = xd.double().cpu()
        err = (out.double().cpu() - h.sum((0, 2))).abs()
        assert bool((err <= (B * S + 2) * (U if dtype == 0 else 2.0 ** -53) * h.abs().sum((0, 2))).all())


def test_channel_sum_of_single_positions_takes_no_longer():
    """65,536 samples of one position take about as long as 256 samples of 256 (the same values)."""
    need_gpu()
    from paper_2205_04550_amd.nn import LIB, _check
    x = torch.randn(65536 * 64, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    best = {}
    for B, S in ((65536, 1), (256, 256)):
        out = torch.empty(64, device="cuda")
        nb = LIB.nn_channel_sum_ws_bytes(0, B, 64, S)
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                _check(LIB.nn_channel_sum(0, B, 64, S, x.data_ptr(), out.data_ptr(), ws.data_ptr(), nb, st))
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        best[S] = min(times[1:])
    assert best[1] < 6 * best[256], best


# (B, Ci, Co, D, H, W) either side of the estimates' lines: short and long sums, few and many samples,
# full and empty boxes, one to four tiles of coarse channels; by chunk, then by channel.
FORWARD_RULE = [(16, 12, 16, 4, 4, 4), (100, 12, 16, 8, 8, 8), (2, 12, 33, 20, 20, 20), (100, 28, 8, 16, 16, 16),
                (2, 28, 8, 16, 16, 16), (3, 32, 64, 6, 14, 8), (1, 4, 24, 40, 40, 40), (64, 4, 17, 24, 24, 24),
                (200, 32, 64, 8, 8, 8), (7, 16, 32, 12, 12, 12), (100, 3, 24, 20, 20, 22), (2, 3, 24, 20, 20, 22),
                (16, 5, 100, 20, 20, 22), (1, 9, 100, 6, 6, 6)]


@pytest.mark.parametrize("shape", FORWARD_RULE)
def test_conv_forward_either_side_of_the_rule(shape):
    test_conv_forward(shape)


@pytest.mark.parametrize("shape", [(2, 3, 2, 8, 6, 10), (2, 2, 2, 8, 6, 10), (2, 16, 4, 6, 8, 4), (2, 17, 4, 6, 8, 4),
                                   (3, 20, 6, 4, 4, 6), (1, 64, 2, 12, 4, 4)])
def test_conv_adjoint_of_few_coarse_channels(shape):
    """Few coarse channels: two take the general kernel from 32 coarse voxels on."""
    test_conv_adjoint(shape)


# The training kernels' sums run in the order of the general kernels, bit for bit. Each is compared with
# the general kernel on a call that holds the same sums among others: a wider volume, more channels or
# columns, a channel of zeros.

def _cases(w):
    return (w.cuda(), w.cuda()), (w.to(torch.bfloat16).float().cuda(), w.to(torch.bfloat16).cuda())


@pytest.mark.parametrize("shape", [(2, 8, 16, 10, 12, 24), (3, 16, 33, 6, 6, 8), (2, 32, 64, 8, 8, 4), (1, 20, 40, 4, 6, 20)])
def test_conv_forward_by_chunk_has_the_staged_kernels_bits(shape):
    """Rows of 16 voxels and more go to the staged kernel: the same columns of a volume of 64."""
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    g = torch.Generator().manual_seed(sum(shape) + 11)
    wide = torch.randn(B, Ci, D, H, 64, generator=g)
    w, b = torch.randn(Co, Ci, 3, 3, 3, generator=g), torch.randn(Co, generator=g).cuda()
    for wf, wc in _cases(w):
        say(f"bits forward by chunk {shape} {wc.dtype}")
        y = nn.Conv3dS2.apply(wide[..., :W].contiguous().cuda(), wf, b, wc, True)
        ref = nn.Conv3dS2.apply(wide.cuda(), wf, b, wc, True)
        assert torch.equal(y, ref[..., :W // 2])


@pytest.mark.parametrize("shape", [(2, 3, 9, 6, 8, 10), (2, 8, 16, 6, 6, 6), (1, 9, 20, 10, 6, 14), (3, 31, 33, 4, 4, 6),
                                   (2, 32, 64, 6, 6, 6)])
def test_conv_forward_by_channel_has_the_vector_kernels_bits(shape):
    """More than 1,024 coarse channels go to the vector kernel: the first of them."""
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    g = torch.Generator().manual_seed(sum(shape) + 12)
    x = torch.randn(B, Ci, D, H, W, generator=g).cuda()
    w, b = torch.randn(1032, Ci, 3, 3, 3, generator=g), torch.randn(1032, generator=g).cuda()
    for wf, wc in _cases(w):
        say(f"bits forward by channel {shape} {wc.dtype}")
        y = nn.Conv3dS2.apply(x, wf[:Co].contiguous(), b[:Co].contiguous(), wc[:Co].contiguous(), False)
        ref = nn.Conv3dS2.apply(x, wf, b, wc, False)
        assert torch.equal(y, ref[:, :Co])


@pytest.mark.parametrize("shape", [(2, 2, 8, 8, 6, 64), (3, 1, 11, 6, 10, 24), (40, 2, 5, 4, 4, 8)])
def test_first_layer_forward_has_the_vector_kernels_bits(shape):
    """Rows that are not whole fours of outputs go to the vector kernel: a volume one pair wider."""
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    g = torch.Generator().manual_seed(sum(shape) + 13)
    wide = torch.randn(B, Ci, D, H, W + 2, generator=g)
    w, b = torch.randn(Co, Ci, 3, 3, 3, generator=g), torch.randn(Co, generator=g).cuda()
    for wf, wc in _cases(w):
        say(f"bits first layer {shape} {wc.dtype}")
        y = nn.Conv3dS2.apply(wide[..., :W].contiguous().cuda(), wf, b, wc, False)
        ref = nn.Conv3dS2.apply(wide.cuda(), wf, b, wc, False)
        assert torch.equal(y, ref[..., :W // 2])


@pytest.mark.parametrize("shape", [(2, 2, 8, 10, 12, 32), (3, 1, 4, 6, 10, 6), (2, 2, 40, 4, 6, 8), (2, 8, 16, 6, 8, 32),
                                   (3, 3, 10, 6, 10, 14), (2, 16, 32, 10, 6, 18), (3, 32, 64, 8, 8, 8)])
def test_conv_adjoint_has_the_general_kernels_bits(shape):
    """An odd count of coarse channels goes to the general kernel: one of zero weights more."""
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    g = torch.Generator().manual_seed(sum(shape) + 14)
    x = torch.randn(B, Co + 1, D // 2, H // 2, W // 2, generator=g).cuda()
    w, b = torch.randn(Co + 1, Ci, 3, 3, 3, generator=g), torch.randn(Ci, generator=g).cuda()
    w[Co] = 0.0
    for wf, wc in _cases(w):
        say(f"bits adjoint {shape} {wc.dtype}")
        y = nn.ConvT3dS2.apply(x[:, :Co].contiguous(), wf[:Co].contiguous(), b, wc[:Co].contiguous(), False)
        assert torch.equal(y, nn.ConvT3dS2.apply(x, wf, b, wc, False))


@pytest.mark.parametrize("shape", [(32, 512, 64), (7, 132, 36), (17, 1028, 16), (33, 320, 200), (5, 4096, 16)])
def test_linear_of_a_small_batch_has_the_tiles_bits(shape):
    """The outputs (and input gradients) of a layer with thousands of columns, which goes to the
    64 x 64 tiles, and the weight gradient of one more input, which goes to the general kernel."""
    need_gpu()
    from paper_2205_04550_amd import nn
    from paper_2205_04550_amd.nn import LIB, _check
    B, K, N = shape
    g = torch.Generator().manual_seed(sum(shape) + 15)
    a, w, b = torch.randn(B, K, generator=g).cuda(), torch.randn(16640, K, generator=g), torch.randn(16640, generator=g).cuda()
    st = torch.cuda.current_stream().cuda_stream
    for wf, wc in _cases(w):
        say(f"bits linear {shape} {wc.dtype}")
        assert torch.equal(nn.Linear.apply(a, wf[:N].contiguous(), b[:N].contiguous(), wc[:N].contiguous(), True),
                           nn.Linear.apply(a, wf, b, wc, True)[:, :N])
        out = []
        for n in (N, 16640):                                   # dX [B][n] from dY [B][K], W [K][n]
            wt, dx = wc[:n].t().contiguous(), torch.empty(B, n, device="cuda")
            _check(LIB.nn_linear_bwd_data(0, B, n, K, a.data_ptr(), wt.data_ptr(), nn._wdt(wt), dx.data_ptr(), st))
            out.append(dx)
        assert torch.equal(out[0], out[1][:, :N])
    x, grads = torch.randn(B, K + 1, generator=g).cuda(), []
    dy = torch.randn(B, N, generator=g).cuda()
    for i in (K, K + 1):
        xi, dw, db = x[:, :i].contiguous(), torch.empty(N, i, device="cuda"), torch.empty(N, device="cuda")
        _check(LIB.nn_linear_bwd_weight(0, B, i, N, xi.data_ptr(), dy.data_ptr(), dw.data_ptr(), db.data_ptr(), st))
        grads.append((dw, db))
    assert torch.equal(grads[0][0], grads[1][0][:, :K]) and torch.equal(grads[0][1], grads[1][1])


@pytest.mark.parametrize("shape", [(2, 2, 8, 8, 6, 64), (3, 3, 5, 6, 10, 6), (5, 4, 9, 24, 24, 24)])
def test_conv_weight_gradient_bits(shape):
    """The order of conv_bwd_weight_partial and _final: a thread every 256th position of a chunk of
    4,096 as fused multiply-adds, lanes by halves, four waves, chunks. Inputs of 12 bits near one, so
    that float64 holds every sum before its rounding exactly."""
    need_gpu()
    from paper_2205_04550_amd import nn
    B, Ci, Co, D, H, W = shape
    rng = np.random.default_rng(sum(shape))
    f = np.float32
    draw = lambda *s: (rng.integers(512, 2048, s) * rng.choice((-1, 1), s) / 1024).astype(f)
    x, gy = draw(B, Ci, D, H, W), draw(B, Co, D // 2, H // 2, W // 2)
    say(f"bits weight gradient {shape}")
    P = gy[:, 0].size
    pad = np.pad(x, ((0, 0), (0, 0), (1, 0), (1, 0), (1, 0)))
    taps = np.stack([pad[:, :, kd:kd + D:2, kh:kh + H:2, kw:kw + W:2] for kd in range(3) for kh in range(3)
                     for kw in range(3)], 2).transpose(1, 2, 0, 3, 4, 5).reshape(Ci * 27, P)
    taps = np.concatenate([taps.reshape(Ci, 27, P), np.ones((Ci, 1, P), f)], 1).reshape(Ci * 28, P)
    g = gy.transpose(1, 0, 2, 3, 4).reshape(Co, P)
    total = np.zeros((Co, Ci * 28), f)
    for p0 in range(0, P, 4096):
        n = min(4096, P - p0)
        acc = np.zeros((Co, Ci * 28, 256), f)
        for i in range(0, n, 256):
            m = min(256, n - i)
            at = slice(p0 + i, p0 + i + m)
            acc[..., :m] = (acc[..., :m].astype(np.float64) + g[:, None, at].astype(np.float64) * taps[None, :, at]).astype(f)
        v = acc.reshape(Co, Ci * 28, 4, 64)
        while v.shape[-1] > 1:
            h = v.shape[-1] // 2
            v = v[..., :h] + v[..., h:]
        v = v[..., 0]
        total = total + (((v[..., 0] + v[..., 1]) + v[..., 2]) + v[..., 3])
    total = total.reshape(Co, Ci, 28)
    w = torch.zeros(Co, Ci, 3, 3, 3, device="cuda").requires_grad_()
    b = torch.zeros(Co, device="cuda").requires_grad_()
    y = nn.Conv3dS2.apply(torch.from_numpy(x).cuda(), w, b, w.detach(), False)
    gw, gb = torch.autograd.grad(y, (w, b), torch.from_numpy(gy).cuda())
    assert np.array_equal(gw.cpu().numpy().reshape(Co, Ci, 27), total[:, :, :27])
    assert np.array_equal(gb.cpu().numpy(), total[:, 0, 27])


def test_conv_adjoint_of_nans_takes_little_longer():
    """Infinities and NaNs all over the coarse side: the outputs that hold one are formed a second
    time by the direct loop, in at most thirty times the time of a call without them."""
    need_gpu()
    from paper_2205_04550_amd.nn import LIB, _check
    B, Ci, Co, D = 16, 16, 32, 16
    g = torch.Generator(device="cuda").manual_seed(9)
    clean = torch.randn(B, Co, D // 2, D // 2, D // 2, generator=g, device="cuda")
    w = torch.randn(Co, Ci, 3, 3, 3, generator=g, device="cuda")
    dx = torch.empty(B, Ci, D, D, D, device="cuda")
    marked = clean.clone()
    marked.view(-1)[::53] = float("inf")
    marked.view(-1)[1::71] = float("nan")
    st = torch.cuda.current_stream().cuda_stream
    best = []
    for x in (clean, marked):
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                _check(LIB.nn_conv3d_s2_bwd_data(0, B, Ci, Co, D, D, D, x.data_ptr(), w.data_ptr(), 0, None, 0,
                                                 dx.data_ptr(), st))
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        best.append(min(times[1:]))
    assert best[1] < 30 * best[0], best


@pytest.mark.parametrize("shape", [(100, 16, 24), (32, 16, 32)])
def test_conv_adjoint_of_32_channels_takes_half_of_64(shape):
    """Half the products and half the bytes read: at most 64 % of the time of 64 coarse channels (with
    few of its loads issued ahead, 67 to 74 %)."""
    need_gpu()
    from paper_2205_04550_amd.nn import LIB, _check, _wdt
    B, Ci, D = shape
    dx = torch.empty(B, Ci, D, D, D, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    best = []
    for Co in (32, 64):
        g = torch.Generator(device="cuda").manual_seed(Co)
        x = torch.randn(B, Co, D // 2, D // 2, D // 2, generator=g, device="cuda")
        w = torch.randn(Co, Ci, 3, 3, 3, generator=g, device="cuda").to(torch.bfloat16)
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                _check(LIB.nn_conv3d_s2_bwd_data(0, B, Ci, Co, D, D, D, x.data_ptr(), w.data_ptr(), _wdt(w), None, 0,
                                                 dx.data_ptr(), st))
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        best.append(min(times[2:]))
    assert best[0] < 0.64 * best[1], best
