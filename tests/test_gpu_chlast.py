"""The channels-last product (conv_chlast): every geometry through IM2COL_GEMM with a workspace that holds the copies, at
the sizes where it can go wrong -- filter runs that end inside a stage, output tiles with one row or pixel over, reduction
slices, residue classes without taps, passes over parts of the batch -- against the fp64 oracle; and every tile by name, with
a row, a pixel or a column over, where the library's own plan says that it runs."""
import ctypes

import pytest
import torch

import oracle
import paper_1801_04380_amd as sn
from paper_1801_04380_amd import _lib
from paper_1801_04380_amd import workloads as wl
from _parity import CODE, TOL, elementwise_excess, f64, rel_l2, shape_of

pytestmark = pytest.mark.gpu

KiB, BIG = 1 << 10, 64 << 20
# N, C, H, W, K, R, S, stride, pad, workspace (shapes; which tile takes them is the plan's: TILES below holds it to one)
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


def _inspect(shape, d, ws_bytes, algo=sn.SN_ALGO_IM2COL_GEMM):
    """What the library would run under this name with this workspace: ((tile m, tile n, threads), slices, passes, bytes),
    or None if not the product."""
    info, used, us = (ctypes.c_int * 5)(), ctypes.c_size_t(), ctypes.c_double()
    if not _lib.load().sn_chlast_inspect(ctypes.byref(shape), d, algo, ctypes.c_size_t(ws_bytes), info,
                                         ctypes.byref(used), ctypes.byref(us)):
        return None
    return tuple(info[:3]), info[3], info[4], used.value


def _check(name, case, dtype, d, ws_bytes):
    N, C, H, W, K, R, S, stride, pad = case
    layer = wl.Layer(name, C, H, W, K, R, S, stride, pad, False, None, 1, False, None)
    x, w, dy = wl.conv_inputs(layer, N, dtype, 4711)
    shape = shape_of(layer, N, dtype, dtype)
    t = torch.float32 if d == sn.SN_CONV_BWD_FILTER or dtype == "f32" else torch.bfloat16
    P, Q = wl.out_hw(layer)
    fn, a, b, dims, ref = {
        sn.SN_CONV_FWD: (sn.sn_conv2d_fwd, x, w, (N, K, P, Q), lambda: oracle.conv2d_fwd(f64(x), f64(w), stride, pad)),
        sn.SN_CONV_BWD_DATA: (sn.sn_conv2d_bwd_data, dy, w, (N, C, H, W),
                              lambda: oracle.conv2d_bwd_data(f64(dy), f64(w), x.shape, stride, pad)),
        sn.SN_CONV_BWD_FILTER: (sn.sn_conv2d_bwd_filter, x, dy, (K, C, R, S),
                                lambda: oracle.conv2d_bwd_filter(f64(x), f64(dy), w.shape, stride, pad))}[d]
    got = torch.full(dims, float("nan"), dtype=t, device="cuda")
    ws = torch.full((ws_bytes,), 255, dtype=torch.uint8, device="cuda")   # NaNs: nothing unwritten may be used
    print(name, dtype, "dir", d, "ws", ws_bytes, flush=True)
    fn(a.cuda(), b.cuda(), got, shape, sn.SN_ALGO_IM2COL_GEMM, ws)
    torch.cuda.synchronize()
    want = ref()
    assert rel_l2(f64(got), want) <= TOL[dtype], (name, d)
    assert elementwise_excess(f64(got), want, TOL[dtype], t == torch.bfloat16) <= 0, (name, d)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("name", list(CASES))
def test_matches_oracle(name, dtype):
    *case, budget = CASES[name]
    N, C, H, W, K, R, S, stride, pad = case
    shape = sn.conv_shape(N, C, H, W, K, R, S, stride, pad, CODE[dtype], CODE[dtype])
    for d in (sn.SN_CONV_FWD, sn.SN_CONV_BWD_DATA, sn.SN_CONV_BWD_FILTER):
        ws_bytes = max(budget, sn.sn_conv_workspace_query(shape, d, sn.SN_ALGO_IM2COL_GEMM)[0])
        assert _inspect(shape, d, ws_bytes), (name, d)
        _check(name, case, dtype, d, ws_bytes)


F, D, B = sn.SN_CONV_FWD, sn.SN_CONV_BWD_DATA, sn.SN_CONV_BWD_FILTER
# (dtype, direction, (tile m, tile n, threads), sliced), N, C, H, W, K, R, S, stride, pad: output channels, pixels and columns that
# are no whole number of tiles, planes of odd and even size, reductions longer than the ring of stages
TILES = [
    ("f32", F, (128, 128, 256), False, 7, 9, 99, 37, 65, 3, 3, (1, 1), (1, 1)),
    ("f32", F, (128, 128, 256), True, 7, 17, 17, 69, 65, 5, 5, (1, 1), (2, 2)),
    ("f32", F, (64, 64, 256), True, 2, 33, 11, 5, 65, 3, 3, (1, 1), (1, 1)),
    ("f32", D, (128, 128, 256), True, 3, 65, 59, 47, 129, 3, 1, (1, 1), (1, 0)),
    ("f32", D, (128, 128, 256), False, 7, 65, 75, 49, 193, 1, 1, (2, 2), (0, 0)),
    ("f32", D, (64, 64, 256), False, 2, 65, 17, 5, 257, 1, 1, (2, 2), (0, 0)),
    ("bf16", F, (128, 128, 256), False, 5, 17, 91, 93, 65, 3, 3, (1, 1), (1, 1)),
    ("bf16", F, (128, 128, 256), False, 16, 17, 83, 81, 129, 3, 3, (2, 2), (1, 1)),
    ("bf16", F, (128, 128, 512), False, 15, 17, 69, 25, 65, 3, 3, (1, 1), (1, 1)),
    ("bf16", F, (128, 128, 512), True, 15, 257, 43, 49, 65, 3, 3, (2, 2), (1, 1)),
    ("bf16", F, (256, 256, 512), False, 16, 17, 85, 37, 193, 3, 3, (1, 1), (1, 1)),
    ("bf16", F, (64, 256, 256), False, 5, 17, 91, 79, 129, 3, 3, (1, 1), (1, 1)),
    ("bf16", F, (64, 256, 256), True, 7, 257, 32, 55, 9, 3, 3, (1, 1), (1, 1)),
    ("bf16", F, (64, 64, 256), True, 1, 65, 22, 6, 65, 5, 5, (2, 2), (2, 2)),
    ("bf16", D, (128, 128, 256), False, 5, 65, 83, 99, 65, 3, 1, (1, 1), (1, 0)),
    ("bf16", D, (128, 128, 512), False, 16, 65, 93, 85, 321, 1, 1, (2, 2), (0, 0)),
    ("bf16", D, (128, 128, 512), True, 7, 65, 17, 69, 257, 3, 3, (1, 1), (1, 1)),
    ("bf16", D, (256, 256, 512), False, 128, 256, 48, 52, 9, 1, 1, (2, 2), (0, 0)),
    ("bf16", D, (64, 256, 256), False, 9, 129, 53, 71, 72, 3, 1, (1, 1), (1, 0)),
    ("bf16", D, (64, 64, 256), False, 3, 65, 5, 5, 9, 5, 5, (1, 1), (2, 2)),
    ("f32", B, (64, 64, 256), True, 1, 17, 57, 64, 129, 5, 5, (2, 2), (2, 2)),
    ("bf16", B, (128, 128, 256), True, 7, 9, 61, 54, 129, 3, 3, (1, 1), (1, 1)),
    ("bf16", B, (64, 128, 256), True, 16, 9, 46, 63, 9, 3, 3, (2, 2), (1, 1)),
    ("bf16", B, (64, 64, 256), False, 1, 513, 24, 14, 129, 3, 3, (2, 2), (1, 1)),
    ("bf16", B, (256, 256, 512), True, 33, 513, 13, 9, 129, 5, 5, (1, 1), (2, 2)),
]


@pytest.mark.parametrize("case", TILES, ids=lambda c: "%s-%s-%dx%dx%d%s-%d" % (c[0], "fdb"[c[1]], *c[2], "-sliced" * c[3], c[5]))
def test_each_tile(case):
    dtype, d, tile, sliced, *rest = case
    N, C, H, W, K, R, S, stride, pad = rest
    shape = sn.conv_shape(N, C, H, W, K, R, S, stride, pad, CODE[dtype], CODE[dtype])
    ran = _inspect(shape, d, BIG)
    assert ran and ran[0] == tile and (ran[1] > 1) == sliced and ran[2] == 1, ran
    _check("tile", rest, dtype, d, BIG)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [F, D, B], ids=["fwd", "bwd_data", "bwd_filter"])
def test_passes_over_the_batch(d, dtype):
    """A byte less than one pass takes: two passes, the second of fewer images."""
    case = (7, 24, 20, 21, 40, 3, 3, (2, 2), (1, 1))
    shape = sn.conv_shape(*case, CODE[dtype], CODE[dtype])
    whole = _inspect(shape, d, BIG)
    ws_bytes = whole[3]
    while _inspect(shape, d, ws_bytes)[2] == 1:
        ws_bytes = _inspect(shape, d, ws_bytes)[3] - 256
    assert whole[2] == 1 and _inspect(shape, d, ws_bytes)[2] == 2
    assert ws_bytes >= sn.sn_conv_workspace_query(shape, d, sn.SN_ALGO_IM2COL_GEMM)[0]
    _check("passes", case, dtype, d, ws_bytes)


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


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("case", [(2, 24, 13, 13, 40, 3, 3, (1, 1), (1, 1)), (2, 24, 14, 15, 40, 3, 3, (2, 2), (1, 1)),
                                  (3, 9, 5, 6, 33, 5, 5, (1, 1), (2, 2)), (2, 3, 47, 45, 16, 11, 11, (4, 4), (0, 0)),
                                  (2, 3, 30, 29, 24, 7, 7, (2, 2), (3, 3)), (2, 40, 17, 17, 32, 7, 1, (1, 1), (3, 0)),
                                  (4, 128, 56, 56, 128, 3, 3, (1, 1), (1, 1))], ids=lambda c: "x".join(map(str, c[:7])))
def test_infinite_inputs_stay_with_their_taps(case, dtype):
    """An Inf in x reaches the outputs whose windows hold it (forward) and the taps that meet it (backward-filter), nothing
    else: neither through the padding between the copies' rows nor through a piece shared with the next pixel."""
    N, C, H, W, K, R, S, stride, pad = case
    layer = wl.Layer("inf", *case[1:5], R, S, stride, pad, False, None, 1, False, None)
    x, w, dy = wl.conv_inputs(layer, N, dtype, 815)
    at = torch.zeros(x.shape, dtype=torch.bool)
    for spot in ((0, 0, 0, 0), (N - 1, C - 1, H - 1, W - 1), (N // 2, C // 2, H // 2, W // 2), (0, C - 1, H - 1, 0)):
        at[spot] = True
    x0, hit = f64(x.masked_fill(at, 0)), f64(at)
    xd = x.masked_fill(at, float("inf")).cuda()
    shape = shape_of(layer, N, dtype, dtype)
    for d, fn, b, t, touched, want in (
            (F, sn.sn_conv2d_fwd, w, w.dtype, oracle.conv2d_fwd(hit, f64(torch.ones_like(w)), stride, pad),
             oracle.conv2d_fwd(x0, f64(w), stride, pad)),
            (B, sn.sn_conv2d_bwd_filter, dy, torch.float32, oracle.conv2d_bwd_filter(hit, f64(torch.ones_like(dy)), w.shape, stride, pad),
             oracle.conv2d_bwd_filter(x0, f64(dy), w.shape, stride, pad))):
        ws_bytes = max(BIG, sn.sn_conv_workspace_query(shape, d, sn.SN_ALGO_IM2COL_GEMM)[0])
        assert _inspect(shape, d, ws_bytes)
        out = torch.zeros(want.shape, dtype=t, device="cuda")
        print("case", case, dtype, "dir", d, flush=True)
        fn(xd, b.cuda(), out, shape, sn.SN_ALGO_IM2COL_GEMM, torch.empty(ws_bytes, dtype=torch.uint8, device="cuda"))
        clean = touched < 0.5
        got = f64(out)
        assert (abs(got[clean]) < float("inf")).all(), (d, "reached outputs it does not belong to")
        assert not (abs(got[~clean]) < float("inf")).any(), (d, "lost")
        assert rel_l2(got[clean], want[clean]) <= TOL[dtype]


def test_measurements_choose_between_staged_kernels():
    """Where STAGED with enough workspace is the product, autotuning also times STAGED's own kernel (with the workspace that
    runs it), and AUTO runs what was measured, with the workspace it was measured with."""
    layer, N = wl.Layer("w14", 64, 14, 14, 128, 3, 3, (1, 1), (1, 1), True, None, 1, False, None), 4
    x, w, _ = (t.cuda() for t in wl.conv_inputs(layer, N, "bf16", 16))
    shape = shape_of(layer, N, "bf16", "bf16")
    mn, pf = sn.sn_conv_workspace_query(shape, F, sn.SN_ALGO_STAGED)
    assert _inspect(shape, F, pf, sn.SN_ALGO_STAGED) and not _inspect(shape, F, mn, sn.SN_ALGO_STAGED)
    ws = torch.empty(4 << 20, dtype=torch.uint8, device="cuda")

    def run(algo, ws):
        y = torch.full((N, 128, 14, 14), float("nan"), dtype=torch.bfloat16, device="cuda")
        sn.sn_conv2d_fwd(x, w, y, shape, algo, ws)
        return y

    own, product = run(sn.SN_ALGO_STAGED, ws[:mn]), run(sn.SN_ALGO_STAGED, ws[:pf])
    assert not torch.equal(own, product)   # (another order of the sums: what tells them apart below)
    sn.sn_planner_clear()
    sn.sn_conv_autotune(F, x, w, torch.empty_like(own), shape, ws, iters=2)
    sn.sn_planner_record(shape, F, sn.SN_ALGO_DIRECT, 0, 1e6)
    algo, used, ms = sn.sn_conv_plan(shape, F, mn)
    assert (algo, used) == (sn.SN_ALGO_STAGED, mn) and 0 < ms < 1e6
    sn.sn_planner_record(shape, F, sn.SN_ALGO_STAGED, mn, 1e-6)
    assert torch.equal(run(sn.SN_ALGO_AUTO, ws), own)
    sn.sn_planner_record(shape, F, sn.SN_ALGO_STAGED, mn, 1e6)
    sn.sn_planner_record(shape, F, sn.SN_ALGO_STAGED, pf, 1e-6)
    assert torch.equal(run(sn.SN_ALGO_AUTO, ws), product)
    sn.sn_planner_clear()


def test_measurements_reach_the_backward_filter_kernel():
    """The same for backward-filter, whose own kernel takes more workspace than the product: its time is recorded under the bytes
    that name it, and AUTO runs it where that is the fastest record."""
    layer, N = wl.Layer("w14", 64, 14, 14, 64, 3, 3, (1, 1), (1, 1), True, None, 1, False, None), 16
    x, _, dy = (t.cuda() for t in wl.conv_inputs(layer, N, "bf16", 17))
    shape = shape_of(layer, N, "bf16", "bf16")
    assert _inspect(shape, B, 64 << 20, sn.SN_ALGO_STAGED)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    sn.sn_planner_clear()
    sn.sn_conv_autotune(B, x, dy, torch.empty((64, 64, 3, 3), device="cuda"), shape, ws, iters=2)
    slow = [(sn.SN_ALGO_DIRECT, 0)]
    algo, used, _ = sn.sn_conv_plan(shape, B, 64 << 20)
    while _inspect(shape, B, used, algo) or algo == sn.SN_ALGO_DIRECT:   # put what is not STAGED's own kernel out of the way
        sn.sn_planner_record(shape, B, algo, used, 1e6 + len(slow))
        slow.append((algo, used))
        algo, used, ms = sn.sn_conv_plan(shape, B, 64 << 20)
        assert len(slow) < 8 and ms < 1e6, slow
    assert algo == sn.SN_ALGO_STAGED
    out = [torch.full((64, 64, 3, 3), float("nan"), device="cuda") for _ in range(2)]
    sn.sn_conv2d_bwd_filter(x, dy, out[0], shape, sn.SN_ALGO_STAGED, ws[:used])
    sn.sn_conv2d_bwd_filter(x, dy, out[1], shape, sn.SN_ALGO_AUTO, ws)
    assert torch.equal(out[0], out[1])
    assert rel_l2(f64(out[0]), oracle.conv2d_bwd_filter(f64(x), f64(dy), (64, 64, 3, 3), (1, 1), (1, 1))) <= TOL["bf16"]
    sn.sn_planner_clear()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [F, D, B], ids=["fwd", "bwd_data", "bwd_filter"])
def test_more_output_channels_than_a_grid_has_rows(d, dtype):
    case = (1, 8, 5, 5, 70000, 1, 1, (1, 1), (0, 0)) if d != D else (1, 70000, 5, 5, 8, 1, 1, (1, 1), (0, 0))
    shape = sn.conv_shape(*case, CODE[dtype], CODE[dtype])
    try:
        least = sn.sn_conv_workspace_query(shape, d, sn.SN_ALGO_IM2COL_GEMM)[0]
    except sn.SnError:   # (unfolding 70000 input channels is refused; the name with it)
        return
    _check("channels", case, dtype, d, max(BIG, least))
