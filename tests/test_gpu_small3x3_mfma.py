"""The fp32 3x3 / stride-1 kernel of small layers of 16 reduction channels and more (csrc/conv_small.hip) against the oracle."""
import pytest
import torch

import oracle
import paper_1801_04380_amd as sn
from paper_1801_04380_amd import workloads as wl
from _parity import rel_l2

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, pad): 16 and one beside it on either side of the two kernels' line; a patch exactly, and one row and column over; channels that end
# inside a step and a tile; no padding and padding 2; more steps than waves
SHAPES = [(1, 16, 1, 1, 16, 1), (2, 15, 5, 7, 17, 1), (1, 17, 4, 4, 15, 1), (2, 33, 5, 9, 18, 0), (1, 40, 3, 6, 50, 2), (3, 16, 13, 8, 31, 1),
          (1, 300, 5, 5, 140, 1), (2, 64, 14, 14, 32, 1)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_small3x3_mfma(shape):
    N, C, H, W, K, p = shape
    x = wl.activation((N, C, H, W), "f32", 3)
    w = wl.activation((K, C, 3, 3), "f32", 4, scale=(2.0 / (9 * C)) ** 0.5)
    dy = wl.activation((N, K, H + 2 * p - 2, W + 2 * p - 2), "f32", 5)
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (p, p), sn.SN_F32, sn.SN_F32)
    y, dx = (torch.full(t.shape, float("nan"), device="cuda") for t in (dy, x))
    sn.sn_conv2d_fwd(x.cuda(), w.cuda(), y, sh, sn.SN_ALGO_DIRECT)
    sn.sn_conv2d_bwd_data(dy.cuda(), w.cuda(), dx, sh, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    xo, wo, dyo = (t.double().numpy() for t in (x, w, dy))
    assert rel_l2(y.double().cpu().numpy(), oracle.conv2d_fwd(xo, wo, (1, 1), (p, p))) <= 1e-5
    assert rel_l2(dx.double().cpu().numpy(), oracle.conv2d_bwd_data(dyo, wo, x.shape, (1, 1), (p, p))) <= 1e-5


@pytest.mark.parametrize("backward", [False, True], ids=["fwd", "bwd_data"])
def test_infinities_stay_with_their_results(backward):
    """One pixel of the last channel (inside a step and a tile); the padding beside the image's corner reads nothing."""
    N, C, H, W, K, p = 2, 33, 5, 9, 18, 1
    a = wl.activation((N, K if backward else C, H, W), "f32", 3)
    w = wl.activation((K, C, 3, 3), "f32", 4, scale=(2.0 / (9 * C)) ** 0.5)
    w[w == 0] = 1e-3
    a[1, -1, 0, W - 1] = float("inf")
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (p, p), sn.SN_F32, sn.SN_F32)
    out = torch.full((N, C if backward else K, H, W), float("nan"), device="cuda")
    (sn.sn_conv2d_bwd_data if backward else sn.sn_conv2d_fwd)(a.cuda(), w.cuda(), out, sh, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    hit = torch.zeros(out.shape, dtype=torch.bool)
    hit[1, :, 0:2, W - 2:] = True
    got = out.cpu()
    assert bool(torch.isfinite(got[~hit]).all()) and bool(torch.isinf(got[hit]).all())
    for h in range(2):
        for v in range(W - 2, W):
            r, s = (h + 1, v - (W - 1) + 1) if backward else (1 - h, W - 1 - v + 1)
            taps = w[K - 1, :, r, s] if backward else w[:, C - 1, r, s]
            assert torch.equal(got[1, :, h, v] > 0, taps > 0)
