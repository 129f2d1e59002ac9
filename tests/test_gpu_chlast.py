"""The channels-last product (conv_chlast): every geometry through IM2COL_GEMM with a workspace that holds the copies, at
the sizes where it can go wrong -- filter runs that end inside a stage, output tiles with one row or pixel over, reduction
slices, residue classes without taps, passes over parts of the batch -- against the fp64 oracle."""
import pytest
import torch

import oracle
import paper_1801_04380_amd as sn
from paper_1801_04380_amd import workloads as wl
from _parity import TOL, elementwise_excess, f64, rel_l2, shape_of

pytestmark = pytest.mark.gpu

KiB, BIG = 1 << 10, 64 << 20
# N, C, H, W, K, R, S, stride, pad, workspace
CASES = {
    "tile_64x64_one_over": (3, 24, 9, 7, 65, 3, 3, (1, 1), (1, 1), BIG),
    "reduction_slices": (2, 256, 14, 14, 96, 3, 3, (1, 1), (1, 1), BIG),
    "tile_128x128": (4, 64, 64, 64, 256, 3, 3, (1, 1), (1, 1), BIG),
    "tile_256x256_row_over": (5, 16, 112, 113, 257, 3, 3, (1, 1), (1, 1), BIG),
    "runs_across_taps": (2, 40, 13, 11, 48, 5, 5, (1, 1), (2, 2), BIG),
    "few_channels_overlapping_rows": (2, 3, 47, 45, 33, 11, 11, (4, 4), (0, 0), BIG),
    "few_channels_padded": (2, 3, 30, 29, 24, 7, 7, (2, 2), (3, 3), BIG),
    "long_column": (3, 37, 17, 17, 70, 7, 1, (1, 1), (3, 0), BIG),
    "long_row": (3, 21, 6, 9, 30, 1, 7, (1, 1), (0, 3), BIG),
    "mixed_strides": (2, 20, 12, 13, 26, 4, 3, (3, 2), (2, 1), BIG),
    "classes_without_taps": (2, 16, 11, 10, 24, 1, 1, (3, 2), (0, 0), BIG),
    "padding_beyond_the_filter": (1, 8, 5, 6, 9, 2, 2, (1, 1), (3, 2), BIG),
    "passes": (7, 24, 20, 21, 40, 3, 3, (2, 2), (1, 1), 300 * KiB),
    "one_pixel": (1, 9, 3, 3, 8, 3, 3, (1, 1), (0, 0), BIG),
}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("name", list(CASES))
def test_matches_oracle(name, dtype):
    N, C, H, W, K, R, S, stride, pad, budget = CASES[name]
    if dtype == "f32" and N * C * H * W * K > 1 << 28:
        pytest.skip("the larger tiles are bf16 only")
    layer = wl.Layer(name, C, H, W, K, R, S, stride, pad, False, None, 1, False, None)
    x, w, dy = wl.conv_inputs(layer, N, dtype, 4711)
    xo, wo, dyo = f64(x), f64(w), f64(dy)
    shape = shape_of(layer, N, dtype, dtype)
    out_t = torch.bfloat16 if dtype == "bf16" else torch.float32
    P, Q = wl.out_hw(layer)
    xd, wd, dyd = x.cuda(), w.cuda(), dy.cuda()
    runs = [(sn.SN_CONV_FWD, sn.sn_conv2d_fwd, xd, wd, (N, K, P, Q), out_t, lambda: oracle.conv2d_fwd(xo, wo, stride, pad)),
            (sn.SN_CONV_BWD_DATA, sn.sn_conv2d_bwd_data, dyd, wd, (N, C, H, W), out_t,
             lambda: oracle.conv2d_bwd_data(dyo, wo, xo.shape, stride, pad)),
            (sn.SN_CONV_BWD_FILTER, sn.sn_conv2d_bwd_filter, xd, dyd, (K, C, R, S), torch.float32,
             lambda: oracle.conv2d_bwd_filter(xo, dyo, wo.shape, stride, pad))]
    for d, fn, a, b, dims, t, ref in runs:
        ws_bytes = max(budget, sn.sn_conv_workspace_query(shape, d, sn.SN_ALGO_IM2COL_GEMM)[0])
        got = torch.full(dims, float("nan"), dtype=t, device="cuda")
        ws = torch.full((ws_bytes,), 255, dtype=torch.uint8, device="cuda")   # NaNs: nothing unwritten may be used
        print(name, dtype, "dir", d, flush=True)
        fn(a, b, got, shape, sn.SN_ALGO_IM2COL_GEMM, ws)
        torch.cuda.synchronize()
        want = ref()
        assert rel_l2(f64(got), want) <= TOL[dtype], (name, d)
        assert elementwise_excess(f64(got), want, TOL[dtype], t == torch.bfloat16) <= 0, (name, d)


@pytest.mark.parametrize("C", [33, 64], ids=["past_2GiB", "4GiB"])
def test_image_beyond_32_bit_offsets(C):
    """A stride larger than the filter leaves most of an image out of the copy: the copy is small where the image itself is
    beyond what 32-bit byte offsets address, and the call still answers (by unfolding)."""
    K, H, stride = 8, 4096, 8
    shape = sn.conv_shape(1, C, H, H, K, 1, 1, (stride, stride), (0, 0), sn.SN_F32, sn.SN_F32)
    gen = torch.Generator(device="cuda").manual_seed(C)
    x = torch.randn((1, C, H, H), generator=gen, device="cuda")
    w = torch.randn((K, C, 1, 1), generator=gen, device="cuda")
    dy = torch.randn((1, K, H // stride, H // stride), generator=gen, device="cuda")
    y, dw = torch.full_like(dy, float("nan")), torch.full_like(w, float("nan"))
    for d, fn, a, b, out in ((sn.SN_CONV_FWD, sn.sn_conv2d_fwd, x, w, y), (sn.SN_CONV_BWD_FILTER, sn.sn_conv2d_bwd_filter, x, dy, dw)):
        ws = torch.empty(sn.sn_conv_workspace_query(shape, d, sn.SN_ALGO_IM2COL_GEMM)[0], dtype=torch.uint8, device="cuda")
        print("C", C, "dir", d, flush=True)
        fn(a, b, out, shape, sn.SN_ALGO_IM2COL_GEMM, ws)
        torch.cuda.synchronize()
    xs = f64(x[0, :, ::stride, ::stride].contiguous()).reshape(C, -1)
    assert rel_l2(f64(y).reshape(K, -1), f64(w).reshape(K, C) @ xs) <= TOL["f32"]
    assert rel_l2(f64(dw).reshape(K, C), f64(dy).reshape(K, -1) @ xs.T) <= TOL["f32"]
