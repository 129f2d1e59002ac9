"""The fp32 3x3 / stride-1 kernel of small problems (csrc/conv_small.hip), forward and backward-data, against the oracle; the
bf16 halves run the zero-workspace kernels that take the same layers in bf16."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_04380_amd as sn
from paper_1801_04380_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-5, "bf16": 5e-3}
CODE = {"f32": sn.SN_F32, "bf16": sn.SN_BF16}

# one pixel; fewer channels than waves, and a remainder; outputs that are no multiple of four; pixels one over a wave; the largest
SHAPES = [(1, 1, 1, 1, 1, 1), (2, 3, 5, 7, 5, 1), (1, 6, 13, 5, 9, 1), (2, 16, 16, 16, 16, 1), (3, 7, 6, 9, 6, 0),
          (1, 4, 4, 6, 3, 2), (5, 64, 7, 7, 33, 1), (2, 64, 16, 16, 56, 1)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_small3x3(shape, dtype):
    N, C, H, W, K, p = shape
    P, Q = H + 2 * p - 2, W + 2 * p - 2
    x = wl.activation((N, C, H, W), dtype, 3)
    w = wl.activation((K, C, 3, 3), dtype, 4, scale=(2.0 / (9 * C)) ** 0.5)
    dy = wl.activation((N, K, P, Q), dtype, 5)
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (p, p), CODE[dtype], CODE[dtype])
    y, dx = (torch.full(s, float("nan"), dtype=x.dtype, device="cuda") for s in (dy.shape, x.shape))
    sn.sn_conv2d_fwd(x.cuda(), w.cuda(), y, sh, sn.SN_ALGO_DIRECT)
    sn.sn_conv2d_bwd_data(dy.cuda(), w.cuda(), dx, sh, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    xo, wo, dyo = (t.double().numpy() for t in (x, w, dy))
    for got, ref in ((y, oracle.conv2d_fwd(xo, wo, (1, 1), (p, p))), (dx, oracle.conv2d_bwd_data(dyo, wo, x.shape, (1, 1), (p, p)))):
        err = np.linalg.norm(got.double().cpu().numpy() - ref) / np.linalg.norm(ref)
        assert err <= TOL[dtype], err


@pytest.mark.parametrize("backward", [False, True], ids=["fwd", "bwd_data"])
def test_more_output_channels_than_a_grid_has_rows(backward):
    """Four output channels per row of the grid, of which there are 65535: beyond, the general kernel answers."""
    M, red = 300000, 2
    K, C = (red, M) if backward else (M, red)
    a = wl.activation((1, red, 1, 1), "f32", 3)
    w = wl.activation((K, C, 3, 3), "f32", 4)
    sh = sn.conv_shape(1, C, 1, 1, K, 3, 3, (1, 1), (1, 1), sn.SN_F32, sn.SN_F32)
    out = torch.full((1, M, 1, 1), float("nan"), device="cuda")
    (sn.sn_conv2d_bwd_data if backward else sn.sn_conv2d_fwd)(a.cuda(), w.cuda(), out, sh, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    taps = w[:, :, 1, 1].double().numpy()   # one pixel: the centre tap alone
    ref = a.double().numpy().reshape(red) @ (taps if backward else taps.T)
    assert np.linalg.norm(out.double().cpu().numpy().reshape(M) - ref) / np.linalg.norm(ref) <= TOL["f32"]
