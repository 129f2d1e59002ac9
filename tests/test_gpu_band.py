"""The 3x3 / stride-1 kernel over at most 64 reduction channels (csrc/conv_band.hip), forward and backward-data, against the
oracle: channel counts of every size class, remainders of output channels and of a band's columns,
one output row, more bands than a workgroup has, several rounds of bands, every padding of the rows."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_1801_04380_amd as sn
from paper_1801_04380_amd import _lib
from paper_1801_04380_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _band(a, w, out, shape, backward, stats=()):
    """The kernel itself, whatever the estimates would run."""
    ptr = [t.data_ptr() for t in stats] or [None] * 3
    assert all(t.data_ptr() % 16 == 0 for t in (a, w, out))
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    status = _lib.load().sn_band_conv(*(ctypes.c_void_p(p) for p in (a.data_ptr(), w.data_ptr(), out.data_ptr())), ctypes.byref(shape),
                                      int(backward), *(ctypes.c_void_p(p) for p in ptr), ctypes.c_float(1e-5), stream)
    assert status == 0, status


# N, C, H, W, K, (pad_h, pad_w)
SHAPES = [(1, 8, 3, 8, 8, (0, 1)), (2, 64, 9, 32, 64, (1, 1)), (3, 40, 17, 40, 72, (1, 1)), (1, 48, 12, 72, 33, (1, 1)),
          (2, 32, 5, 64, 130, (2, 1)), (5, 24, 11, 24, 64, (1, 1)), (1, 56, 40, 232, 16, (0, 1)), (70, 64, 62, 40, 64, (1, 1)),
          (2, 64, 1, 64, 8, (1, 1)), (40, 16, 57, 96, 520, (2, 1)), (9, 64, 37, 48, 72, (1, 1))]


@pytest.mark.parametrize("backward", [False, True], ids=["fwd", "bwd_data"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(str(v) for v in s[:5]))
def test_band(shape, backward):
    N, red, H, W, out, (ph, pw) = shape
    # `red` channels are summed over; H x W and the padding are those of the side that is read
    ip, jp = (2 - ph, 2 - pw) if backward else (ph, pw)
    P, Q = H + 2 * ph - 2, W + 2 * pw - 2
    K, C = (red, out) if backward else (out, red)
    IH, IW = (P, Q) if backward else (H, W)
    a = wl.activation((N, red, H, W), "bf16", 3)
    w = wl.activation((K, C, 3, 3), "bf16", 4, scale=(2.0 / (9 * red)) ** 0.5)
    sh = sn.conv_shape(N, C, IH, IW, K, 3, 3, (1, 1), (ip, jp), sn.SN_BF16, sn.SN_BF16)
    print("case", shape, "backward" if backward else "forward", flush=True)
    got = torch.full((N, out, P, Q), float("nan"), dtype=torch.bfloat16, device="cuda")
    ad, wd = a.cuda(), w.cuda()
    _band(ad, wd, got, sh, backward)
    torch.cuda.synchronize()
    got = got.double().cpu().numpy()
    assert np.isfinite(got).all()
    # the whole batch was written; the images compared one by one are the first, a middle one and the last
    n = sorted({0, N // 2, N - 1})
    ao, wo = a[n].double().numpy(), w.double().numpy()
    ref = oracle.conv2d_bwd_data(ao, wo, (len(n), C, P, Q), (1, 1), (ip, jp)) if backward else oracle.conv2d_fwd(ao, wo, (1, 1), (ip, jp))
    err = np.linalg.norm(got[n] - ref) / np.linalg.norm(ref)
    assert err <= 5e-3, err   # one rounding to bf16


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("backward", [False, True], ids=["fwd", "bwd_data"])
def test_an_infinity_reaches_its_own_outputs(backward, value):
    """Without padding around it: the nine outputs over an Inf or NaN, in their own image and every output channel, and no others --
    beside a band's edge, in the last row and column, in the last channel of a class."""
    N, red, H, W, out = 3, 40, 23, 72, 72
    pad = (1, 1)
    K, C = (red, out) if backward else (out, red)
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), pad, sn.SN_BF16, sn.SN_BF16)
    w = wl.activation((K, C, 3, 3), "bf16", 4, scale=0.06)
    w[w == 0] = 0.01
    for n, c, h, x in ((1, 39, 11, 31), (1, 0, 22, 71), (0, 17, 0, 32), (2, 8, 1, 64)):
        a = wl.activation((N, red, H, W), "bf16", 3)
        a[n, c, h, x] = value
        got = torch.full((N, out, H, W), 7.0, dtype=torch.bfloat16, device="cuda")
        _band(a.cuda(), w.cuda(), got, sh, backward)
        torch.cuda.synchronize()
        reached = torch.zeros((N, out, H, W), dtype=torch.bool)
        reached[n, :, max(0, h - 1):h + 2, max(0, x - 1):x + 2] = True
        assert torch.equal(~torch.isfinite(got.cpu().float()), reached), (n, c, h, x)


def test_band_stats():
    """(count, mean, M2) over bands whose last columns and rows are not there, the mean far from 0."""
    N, C, H, W, K = 9, 64, 37, 48, 72
    x = wl.activation((N, C, H, W), "bf16", 3)
    w = (wl.activation((K, C, 3, 3), "bf16", 4, scale=0.06).float() + 0.03).bfloat16()
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (1, 1), sn.SN_BF16, sn.SN_BF16)
    y = torch.empty((N, K, H, W), dtype=torch.bfloat16, device="cuda")
    mean, invstd = (torch.empty(K, device="cuda") for _ in range(2))
    part = torch.full((K, 256, 3), float("nan"), device="cuda")
    xd, wd = x.cuda(), w.cuda()
    _band(xd, wd, y, sh, False, (part, mean, invstd))
    torch.cuda.synchronize()
    v = y.double().cpu().numpy()
    m, s = v.mean((0, 2, 3)), 1 / np.sqrt(v.var((0, 2, 3)) + 1e-5)
    assert np.linalg.norm(mean.cpu().numpy() - m) / np.linalg.norm(m) <= 1e-5
    assert np.linalg.norm(invstd.cpu().numpy() - s) / np.linalg.norm(s) <= 1e-5


@pytest.mark.parametrize("shape", [(9, 32, 37, 48, 72), (3, 48, 29, 40, 33), (2, 40, 62, 72, 130), (70, 16, 40, 32, 64)],
                         ids=lambda s: "x".join(map(str, s)))
def test_band_stats_of_fewer_channels(shape):
    """The kernels for up to 32 and up to 48 channels, remainders of output channels and columns, many bands a workgroup."""
    N, C, H, W, K = shape
    x = wl.activation((N, C, H, W), "bf16", 3)
    w = (wl.activation((K, C, 3, 3), "bf16", 4, scale=0.06).float() + 0.03).bfloat16()
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (1, 1), sn.SN_BF16, sn.SN_BF16)
    y = torch.full((N, K, H, W), float("nan"), dtype=torch.bfloat16, device="cuda")
    mean, invstd = (torch.empty(K, device="cuda") for _ in range(2))
    part = torch.full((K, 256, 3), float("nan"), device="cuda")
    _band(x.cuda(), w.cuda(), y, sh, False, (part, mean, invstd))
    torch.cuda.synchronize()
    v = y.double()
    m, s = v.mean((0, 2, 3)), (v.var((0, 2, 3), correction=0) + 1e-5).rsqrt()
    assert (mean - m).norm() / m.norm() <= 1e-5 and (invstd - s).norm() / s.norm() <= 1e-5


@pytest.mark.parametrize("algo", [sn.SN_ALGO_DIRECT, sn.SN_ALGO_STAGED], ids=["direct", "staged"])
def test_calls_take_it_where_it_is_faster(algo):
    """From some size on: the same bits as the kernel itself, with and without statistics."""
    N, C, H, W, K = 64, 64, 56, 56, 64
    x = wl.activation((N, C, H, W), "bf16", 3).cuda()
    w = wl.activation((K, C, 3, 3), "bf16", 4, scale=0.06).cuda()
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (1, 1), sn.SN_BF16, sn.SN_BF16)
    y = [torch.full((N, K, H, W), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    mean, invstd = (torch.empty(K, device="cuda") for _ in range(2))
    scratch = torch.full((sn.sn_conv_bn_stats_scratch_bytes(sh),), 255, dtype=torch.uint8, device="cuda")
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda") if algo == sn.SN_ALGO_STAGED else None
    _band(x, w, y[0], sh, False)
    sn.sn_conv2d_fwd(x, w, y[1], sh, algo, ws)
    sn.sn_conv2d_fwd_bn_stats(x, w, y[2], sh, mean, invstd, scratch, algo, ws)
    torch.cuda.synchronize()
    assert torch.equal(y[0], y[1]) and torch.equal(y[0], y[2])
    v = y[0].double()
    m, s = v.mean((0, 2, 3)), (v.var((0, 2, 3), correction=0) + 1e-5).rsqrt()
    assert (mean - m).norm() / m.norm() <= 1e-5 and (invstd - s).norm() / s.norm() <= 1e-5
