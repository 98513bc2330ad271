"""Training kernels against float64 sums, at the sizes where a tile, a channel block or a row
ends: every element within the bound of its own FP32 sum,
(K + 2) 2^-24 times the sum of its terms' magnitudes."""
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
