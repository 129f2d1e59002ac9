"""The one-launch bf16 3x3 / stride-1 kernel of small layers (csrc/conv_small_bf16.hip) against the oracle: the same bits from DIRECT,
AUTO without workspace, the call that allocates nothing and the one that leaves statistics."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_04380_amd as sn
from paper_1801_04380_amd import workloads as wl
from _parity import rel_l2

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, pad): one pixel; a patch exactly; one row and column over both tiles' patches; channels that end inside a step of
# 16 and of 32 and output channels inside a tile; no padding and padding 2; more steps than waves; both tiles' own sizes
SHAPES = [(1, 8, 1, 1, 8, 1), (1, 32, 4, 8, 32, 1), (2, 24, 5, 9, 33, 1), (3, 40, 9, 13, 70, 0), (1, 56, 6, 5, 8, 2), (1, 8, 3, 40, 17, 1),
          (1, 512, 7, 7, 512, 1), (2, 256, 14, 14, 256, 1), (2, 64, 56, 56, 64, 1), (4, 72, 17, 31, 104, 1), (1, 1024, 4, 4, 64, 1)]
# the filter loaded together (nine steps and more, forward): a last step of fewer channels, output channels that fill no tile, of 16 and of 32
SHAPES += [(1, 264, 7, 7, 40, 1), (1, 392, 7, 7, 300, 1), (1, 264, 12, 20, 300, 1)]


@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_small_bf16(shape, out):
    N, C, H, W, K, p = shape
    P, Q = H + 2 * p - 2, W + 2 * p - 2
    ot = torch.bfloat16 if out == "bf16" else torch.float32
    x = wl.activation((N, C, H, W), "bf16", 3)
    w = wl.activation((K, C, 3, 3), "bf16", 4, scale=(2.0 / (9 * C)) ** 0.5)
    dy = wl.activation((N, K, P, Q), "bf16", 5)
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (p, p), sn.SN_BF16, sn.SN_BF16 if out == "bf16" else sn.SN_F32)
    xd, wd, dyd = x.cuda(), w.cuda(), dy.cuda()
    new = lambda like: torch.full(like.shape, float("nan"), dtype=ot, device="cuda")
    y, dx = new(dy), new(x)
    sn.sn_conv2d_fwd(xd, wd, y, sh, sn.SN_ALGO_DIRECT)
    sn.sn_conv2d_bwd_data(dyd, wd, dx, sh, sn.SN_ALGO_DIRECT)
    xo, wo, dyo = (t.double().numpy() for t in (x, w, dy))
    assert rel_l2(y.double().cpu().numpy(), oracle.conv2d_fwd(xo, wo, (1, 1), (p, p))) <= 5e-3
    assert rel_l2(dx.double().cpu().numpy(), oracle.conv2d_bwd_data(dyo, wo, x.shape, (1, 1), (p, p))) <= 5e-3
    for direction, call, a, res in ((sn.SN_CONV_FWD, sn.sn_conv2d_fwd, xd, y), (sn.SN_CONV_BWD_DATA, sn.sn_conv2d_bwd_data, dyd, dx)):
        assert sn.sn_conv_plan(sh, direction, 0)[0] == sn.SN_ALGO_DIRECT
        again = new(res)
        call(a, wd, again, sh, sn.SN_ALGO_AUTO)
        assert torch.equal(again, res)
    if C * K * 18 <= 4 << 20 and W > 1:   # (STAGED takes no rows of one pixel)
        again = new(y)
        sn.sn_conv2d_fwd_noalloc(xd, wd, again, sh)
        if C % 64:   # (on whole channel blocks STAGED may keep the product)
            assert torch.equal(again, y)
        assert rel_l2(again.double().cpu().numpy(), y.double().cpu().numpy()) <= 5e-3
    mean, invstd = torch.empty(K, device="cuda"), torch.empty(K, device="cuda")
    scratch = torch.empty(sn.sn_conv_bn_stats_scratch_bytes(sh), dtype=torch.uint8, device="cuda")
    again = new(y)
    sn.sn_conv2d_fwd_bn_stats(xd, wd, again, sh, mean, invstd, scratch, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    assert torch.equal(again, y)
    assert rel_l2(mean.double().cpu().numpy(), y.double().mean((0, 2, 3)).cpu().numpy()) <= 1e-4


@pytest.mark.parametrize("shape", [(2, 24, 9, 9, 40, 1), (2, 256, 14, 14, 256, 1)], ids=["16", "32"])
def test_infinities_stay_with_their_outputs(shape):
    N, C, H, W, K, p = shape
    x = wl.activation((N, C, H, W), "bf16", 3)
    w = wl.activation((K, C, 3, 3), "bf16", 4, scale=(2.0 / (9 * C)) ** 0.5)
    w[w == 0] = 1e-3
    x[1, C - 1, 4, 5] = float("inf")
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (p, p), sn.SN_BF16, sn.SN_BF16)
    y = torch.empty((N, K, H, W), dtype=torch.bfloat16, device="cuda")
    sn.sn_conv2d_fwd(x.cuda(), w.cuda(), y, sh, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    hit = torch.zeros((N, K, H, W), dtype=torch.bool)
    hit[1, :, 3:6, 4:7] = True
    got = y.cpu()
    assert bool(torch.isfinite(got[~hit]).all()) and bool(torch.isinf(got[hit]).all())
    sign = torch.stack([torch.stack([w[:, C - 1, 4 - h + 1, 5 - v + 1] for v in range(4, 7)], 1) for h in range(3, 6)], 1)
    assert np.array_equal((got[1, :, 3:6, 4:7] > 0).numpy(), (sign > 0).numpy())


@pytest.mark.parametrize("shape", [(2, 24, 9, 9, 40, 1), (2, 256, 14, 14, 256, 1)], ids=["16", "32"])
def test_infinite_gradients_stay_with_their_inputs(shape):
    N, C, H, W, K, p = shape
    dy = wl.activation((N, K, H, W), "bf16", 3)
    w = wl.activation((K, C, 3, 3), "bf16", 4, scale=(2.0 / (9 * C)) ** 0.5)
    w[w == 0] = 1e-3
    dy[1, K - 1, 4, 5] = float("inf")
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (p, p), sn.SN_BF16, sn.SN_BF16)
    dx = torch.empty((N, C, H, W), dtype=torch.bfloat16, device="cuda")
    sn.sn_conv2d_bwd_data(dy.cuda(), w.cuda(), dx, sh, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    hit = torch.zeros((N, C, H, W), dtype=torch.bool)
    hit[1, :, 3:6, 4:7] = True
    got = dx.cpu()
    assert bool(torch.isfinite(got[~hit]).all()) and bool(torch.isinf(got[hit]).all())
    sign = torch.stack([torch.stack([w[K - 1, :, h - 4 + 1, v - 5 + 1] for v in range(4, 7)], 1) for h in range(3, 6)], 1)
    assert np.array_equal((got[1, :, 3:6, 4:7] > 0).numpy(), (sign > 0).numpy())


@pytest.mark.parametrize("shape", [(1, 264, 7, 7, 40, 1), (1, 264, 12, 20, 300, 1)], ids=["16", "32"])
def test_an_infinite_filter_stays_with_its_output_channel(shape):
    """The last step's pieces of the filter past an output channel's last input channel are the next one's first taps."""
    N, C, H, W, K, p = shape
    x = wl.activation((N, C, H, W), "bf16", 3).abs() + 0.5
    w = wl.activation((K, C, 3, 3), "bf16", 4, scale=(2.0 / (9 * C)) ** 0.5)
    for k in (1, 17, K - 1):
        w[k, 0, 1, 1] = float("inf")
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (p, p), sn.SN_BF16, sn.SN_BF16)
    y = torch.empty((N, K, H, W), dtype=torch.bfloat16, device="cuda")
    sn.sn_conv2d_fwd(x.to(torch.bfloat16).cuda(), w.cuda(), y, sh, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    hit = torch.zeros((N, K, H, W), dtype=torch.bool)
    for k in (1, 17, K - 1):
        hit[:, k] = True
    got = y.cpu()
    assert bool(torch.isfinite(got[~hit]).all()) and bool(torch.isposinf(got[hit]).all())
