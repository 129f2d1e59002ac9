"""The one-launch 3x3 / stride-1 backward-filter of small layers (csrc/conv_small_wgrad.hip) against the oracle, under every name that
runs it."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_04380_amd as sn
from paper_1801_04380_amd import workloads as wl
from _parity import rel_l2

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-5, "bf16": 5e-3}
CODE = {"f32": sn.SN_F32, "bf16": sn.SN_BF16}

# (N, C, H, W, K, pad_h, pad_w): one pixel; rows of 1 to 17 pixels (units of 4 and 8 with a remainder, and whole); channels in and
# over one tile; padding 0, 2 and unequal (rows read from before and behind the tensor); fewer steps than waves, and several each
SHAPES = [(1, 5, 1, 1, 3, 1, 1), (2, 16, 16, 16, 16, 1, 1), (1, 17, 4, 3, 33, 1, 1), (3, 8, 5, 9, 16, 1, 1), (2, 40, 9, 11, 24, 0, 0),
          (1, 24, 5, 6, 70, 2, 2), (2, 6, 7, 17, 20, 2, 0), (1, 7, 3, 8, 5, 0, 2), (3, 64, 8, 8, 64, 1, 1), (2, 80, 24, 24, 77, 1, 1)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_small_wgrad(shape, dtype):
    N, C, H, W, K, ph, pw = shape
    x = wl.activation((N, C, H, W), dtype, 3)
    dy = wl.activation((N, K, H + 2 * ph - 2, W + 2 * pw - 2), dtype, 5)
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (ph, pw), CODE[dtype], CODE[dtype])
    ref = oracle.conv2d_bwd_filter(x.double().numpy(), dy.double().numpy(), (K, C, 3, 3), (1, 1), (ph, pw))
    ws = torch.empty(32 << 20, dtype=torch.uint8, device="cuda")
    first = None
    for algo, w in ((sn.SN_ALGO_DIRECT, None), (sn.SN_ALGO_AUTO, None), (sn.SN_ALGO_AUTO, ws)):
        dw = torch.full((K, C, 3, 3), float("nan"), device="cuda")
        sn.sn_conv2d_bwd_filter(x.cuda(), dy.cuda(), dw, sh, algo, w)
        torch.cuda.synchronize()
        assert rel_l2(dw.double().cpu().numpy(), ref) <= TOL[dtype]
        first = dw if first is None else first
        assert torch.equal(dw, first)
    assert sn.sn_conv_plan(sh, sn.SN_CONV_BWD_FILTER, 32 << 20)[:2] == (sn.SN_ALGO_DIRECT, 0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_infinities_stay_with_their_taps(dtype):
    """x's last column is read by the taps of the first two filter columns alone, also where a unit ends past the row."""
    N, C, H, W, K = 2, 9, 6, 11, 18
    x = wl.activation((N, C, H, W), dtype, 3)
    dy = wl.activation((N, K, H, W), dtype, 5).abs() + 0.5
    x[1, 4, 0, W - 1] = float("inf")
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (1, 1), CODE[dtype], CODE[dtype])
    dw = torch.empty((K, C, 3, 3), device="cuda")
    sn.sn_conv2d_bwd_filter(x.cuda(), dy.to(x.dtype).cuda(), dw, sh, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    # output row p meets it under filter row 1 - p (p = 0, 1), output column W - 1, W - 2 under filter columns 1, 2
    hit = np.zeros((K, C, 3, 3), dtype=bool)
    hit[:, 4, 0:2, 1:3] = True
    got = dw.cpu().numpy()
    assert np.isposinf(got[hit]).all() and np.isfinite(got[~hit]).all()
