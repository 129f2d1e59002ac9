"""The image layer's forward kernel (csrc/conv_image_fwd.hip) against the oracle."""
import pytest
import torch

import oracle
import paper_1801_04380_amd as sn
from paper_1801_04380_amd import workloads as wl
from _parity import rel_l2

pytestmark = pytest.mark.gpu

# (N, C, H, W, K, R, S, stride_h, stride_w, pad_h, pad_w): one output pixel; one row of the smallest image; odd rows of an output as wide as a
# block and narrower; two blocks across with a remainder; an odd number of octets, one or two a filter row; output channels in one to three
# tiles and over; padding on every side, more than the filter reaches; several blocks a workgroup
SHAPES = [(1, 3, 11, 11, 8, 11, 11, 4, 4, 0, 0), (1, 1, 7, 9, 33, 7, 7, 2, 2, 0, 0), (2, 3, 59, 67, 96, 11, 11, 4, 4, 0, 0),
          (2, 3, 40, 150, 64, 7, 7, 2, 2, 3, 3), (3, 4, 33, 131, 65, 5, 5, 2, 2, 2, 2), (1, 2, 50, 260, 31, 9, 16, 3, 4, 1, 7),
          (2, 3, 21, 23, 40, 4, 8, 1, 2, 6, 5), (5, 3, 35, 64, 95, 11, 11, 4, 4, 2, 2), (70, 3, 63, 127, 48, 7, 7, 2, 2, 3, 3),
          (2, 1, 7, 16, 50, 7, 12, 4, 8, 0, 0), (1, 3, 16, 9, 8, 4, 4, 2, 2, 0, 0)]
# blocks 32 columns wide, one to three channel tiles and either alignment of an operand: where they take fewer rounds, and where the
# input rows of a wider one are too many
SHAPES += [(40, 1, 62, 18, 32, 9, 9, 1, 2, 0, 0), (1, 4, 62, 291, 8, 11, 11, 3, 4, 0, 0), (40, 4, 48, 13, 50, 6, 8, 1, 2, 3, 2),
           (1, 4, 40, 253, 33, 11, 11, 3, 4, 2, 0), (40, 2, 109, 13, 65, 3, 12, 2, 2, 1, 0), (1, 4, 86, 267, 65, 11, 8, 3, 4, 3, 2)]


def _case(shape, out="bf16"):
    N, C, H, W, K, R, S, sh, sw, ph, pw = shape
    x = wl.activation((N, C, H, W), "bf16", 3)
    w = wl.activation((K, C, R, S), "bf16", 4, scale=(2.0 / (C * R * S)) ** 0.5)
    code = sn.conv_shape(N, C, H, W, K, R, S, (sh, sw), (ph, pw), sn.SN_BF16, sn.SN_BF16 if out == "bf16" else sn.SN_F32)
    P, Q = (H + 2 * ph - R) // sh + 1, (W + 2 * pw - S) // sw + 1
    y = torch.full((N, K, P, Q), float("nan"), dtype=torch.bfloat16 if out == "bf16" else torch.float32, device="cuda")
    return x, w, y, code


@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_image_fwd(shape, out):
    x, w, y, code = _case(shape, out)
    assert sn.sn_conv_plan(code, sn.SN_CONV_FWD, 0)[0] == sn.SN_ALGO_DIRECT
    sn.sn_conv2d_fwd(x.cuda(), w.cuda(), y, code, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    want = oracle.conv2d_fwd(x.double().numpy(), w.double().numpy(), shape[7:9], shape[9:])
    assert rel_l2(y.double().cpu().numpy(), want) <= 5e-3


@pytest.mark.parametrize("shape", [(2, 3, 40, 67, 40, 11, 11, 4, 4, 0, 0), (2, 3, 30, 40, 20, 7, 7, 2, 2, 3, 3)], ids=["11x11", "7x7"])
def test_infinities_stay_with_their_outputs(shape):
    """The operands' columns past the filter meet real elements of x."""
    x, w, y, code = _case(shape)
    w = w.abs() + 0.01
    w = w.to(torch.bfloat16)
    N, C, H, W, K, R, S, sh, sw, ph, pw = shape
    at = [(0, 0, 0, 0), (0, 2, 17, 21), (1, 1, H - 1, W - 1)]
    for i in at:
        x[i] = float("inf")
    sn.sn_conv2d_fwd(x.cuda(), w.cuda(), y, code, sn.SN_ALGO_DIRECT)
    torch.cuda.synchronize()
    hit = torch.zeros(y.shape, dtype=torch.bool)
    for n, _, h, v in at:
        for p in range(y.shape[2]):
            for q in range(y.shape[3]):
                if 0 <= h - p * sh + ph < R and 0 <= v - q * sw + pw < S:
                    hit[n, :, p, q] = True
    got = y.cpu()
    assert bool(torch.isfinite(got[~hit]).all()) and bool(torch.isposinf(got[hit]).all())
