"""Backward-filter of image layers (csrc/conv_image.hip) against the oracle: every column stride and tile count, strips of one
pixel and one over 64, one output row and workgroups whose rows cross strips and images, rows of padding alone; by atomics,
with the least and with all the partial sums it can use."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_04380_amd as sn
from paper_1801_04380_amd import workloads as wl

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, S, stride, pad
SHAPES = [(2, 3, 227, 227, 96, 11, 11, (4, 4), (0, 0)), (3, 3, 60, 131, 64, 7, 7, (2, 2), (3, 3)),
          (2, 3, 30, 90, 40, 7, 7, (2, 2), (3, 3)), (1, 4, 9, 9, 5, 9, 9, (1, 1), (0, 0)), (5, 1, 40, 67, 33, 6, 9, (3, 3), (2, 4)),
          (2, 2, 21, 300, 130, 5, 7, (1, 4), (4, 0)), (7, 3, 16, 64, 16, 5, 5, (1, 1), (2, 2)),
          (1, 4, 70, 30, 97, 8, 12, (4, 1), (3, 11)), (2, 3, 13, 259, 200, 4, 3, (2, 4), (5, 7))]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(str(v) for v in s[:7]))
def test_image_bwd_filter(shape):
    N, C, H, W, K, R, S, stride, pad = shape
    P, Q = (H + 2 * pad[0] - R) // stride[0] + 1, (W + 2 * pad[1] - S) // stride[1] + 1
    x, dy = wl.activation((N, C, H, W), "bf16", 3), wl.activation((N, K, P, Q), "bf16", 5)
    sh = sn.conv_shape(N, C, H, W, K, R, S, stride, pad, sn.SN_BF16, sn.SN_BF16)
    ref = oracle.conv2d_bwd_filter(x.double().numpy(), dy.double().numpy(), (K, C, R, S), stride, pad)
    least, most = sn.sn_conv_workspace_query(sh, sn.SN_CONV_BWD_FILTER, sn.SN_ALGO_STAGED)
    assert 0 < least <= most and (N * P < 8 or least < most)
    xd, dyd = x.cuda(), dy.cuda()
    for algo, b in ((sn.SN_ALGO_DIRECT, 0), (sn.SN_ALGO_STAGED, least), (sn.SN_ALGO_STAGED, most), (sn.SN_ALGO_STAGED, most + 4096)):
        dw = [torch.full((K, C, R, S), float("nan"), device="cuda") for _ in range(2)]
        ws = torch.full((b,), 255, dtype=torch.uint8, device="cuda") if b else None
        for d in dw:
            sn.sn_conv2d_bwd_filter(xd, dyd, d, sh, algo, ws)
        torch.cuda.synchronize()
        assert algo == sn.SN_ALGO_DIRECT or torch.equal(dw[0], dw[1])
        # products of bf16 values are exact in fp32, so only the sums round, in fp32
        assert np.linalg.norm(dw[0].double().cpu().numpy() - ref) / np.linalg.norm(ref) <= 1e-5


@pytest.mark.parametrize("H,W,stride,pad", [(23, 30, 2, 0), (22, 29, 2, 2), (41, 131, 4, 3), (24, 25, 3, 1)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_an_infinity_stays_with_the_products_it_belongs_to(H, W, stride, pad, value):
    """Steps of two output rows of which the second is past the end, columns of the last block past the row's end, rows and columns
    of x that no output reaches: an Inf or NaN there touches the products that read it and no others."""
    N, C, K, R = 2, 3, 40, 7
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    sh = sn.conv_shape(N, C, H, W, K, R, R, (stride, stride), (pad, pad), sn.SN_BF16, sn.SN_BF16)
    dy = wl.activation((N, K, P, Q), "bf16", 5)
    last = (P - 1) * stride - pad + R   # the first row that no output reaches, if the image has it
    for h, w in {(min(P * stride - pad, H - 1), W // 2), (H - 1, W - 1), (min(last, H - 1), 0), (0, 0)}:
        x = wl.activation((N, C, H, W), "bf16", 3)
        x[1, 1, h, w] = value
        ref = oracle.conv2d_bwd_filter(x.double().numpy(), dy.double().numpy(), (K, C, R, R), (stride, stride), (pad, pad))
        for algo in (sn.SN_ALGO_DIRECT, sn.SN_ALGO_STAGED):
            b = sn.sn_conv_workspace_query(sh, sn.SN_CONV_BWD_FILTER, algo)[1]
            dw = torch.full((K, C, R, R), 7.0, device="cuda")
            sn.sn_conv2d_bwd_filter(x.cuda(), dy.cuda(), dw, sh, algo, torch.empty(b, dtype=torch.uint8, device="cuda") if b else None)
            torch.cuda.synchronize()
            got, fine = dw.double().cpu().numpy(), np.isfinite(ref)
            assert np.array_equal(np.isfinite(got), fine), (algo, h, w)
            assert np.linalg.norm(got[fine] - ref[fine]) <= 1e-5 * np.linalg.norm(ref[fine])
