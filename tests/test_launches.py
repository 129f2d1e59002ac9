"""What the library's host code launches, recorded without a GPU (tests/launches/recorder.cpp): the sums over slices stay inside the
workspace that the query and the plan asked for."""
import os
import random
import re
import subprocess

import pytest

import paper_1801_04380_amd as sn
import test_gpu_image
import test_gpu_image_fwd
import test_gpu_small3x3_mfma
import test_gpu_small_bf16
import test_gpu_small_wgrad
from paper_1801_04380_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "launches")
FIELDS = [n for n, _ in _lib.ConvShape._fields_]


@pytest.fixture(scope="session")
def recorded():
    """calls -> [(status, [(kernel, grid, threads, lds, limit, reach)])], a call being (direction, algorithm, workspace bytes, shape)."""
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    exe = os.path.join(HERE, "_build", "recorder")
    _lib.load()
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-o", exe, os.path.join(HERE, "recorder.cpp"),
                    _lib.LIB_PATH, "-ldl", "-Wl,-rpath," + os.path.dirname(_lib.LIB_PATH), "-Wl,--allow-shlib-undefined"], check=True)

    def run(calls, plans=None):
        lines = "\n".join(" ".join(map(str, (d, a, b) + tuple(getattr(s, f) for f in FIELDS))) for d, a, b, s in calls)
        env = dict(os.environ, LD_LIBRARY_PATH="/opt/rocm/lib:" + os.environ.get("LD_LIBRARY_PATH", ""))
        out = subprocess.run([exe], input=lines, stdout=subprocess.PIPE, text=True, check=True, env=env).stdout
        res, launches = [], []
        for line in out.splitlines():
            w = line.split()
            if w[0] == "call":
                res.append((int(w[1]), launches))
                if plans is not None:
                    plans.append(int(w[2]))
                launches = []
            else:
                v = list(map(int, w[2:]))
                launches.append((re.sub(r"^_ZN2sn(12_GLOBAL__N_1)?", "", w[1]), tuple(v[:3])) + tuple(v[3:]))
        assert len(res) == len(calls)
        return res

    return run


def test_partial_sums_stay_in_the_workspace(recorded):
    """STAGED backward-filter under the least, the preferred and the planned bytes.  Most shapes have few channels and a stride on
    one axis or both: over their phase planes they run as a stride-1 shape that as a layer of its own would run another kernel."""
    sn.sn_planner_clear()
    rnd, calls = random.Random(7), []
    for i in range(6000):
        few = i % 4 != 0
        R, S = rnd.choice([(3, 3), (3, 3), (1, 1), (2, 2), (5, 5), (3, 1), (1, 7), (4, 3)])
        stride = rnd.choice([(1, 2), (2, 1), (2, 2)] if few else [(1, 1), (2, 2), (3, 2), (4, 4)])
        C = rnd.randint(1, 4) if few else rnd.choice([8, 16, 24, 64, 100])
        H, W = (rnd.randint(max(R, S), 256 if few else 64) for _ in range(2))
        pad = rnd.choice([(0, 0), (R // 2, S // 2)])
        s = sn.conv_shape(rnd.choice([1, 2, 8, 32]), C, H, W, rnd.choice([8, 16, 33, 64, 128]), R, S, stride, pad, sn.SN_BF16, sn.SN_BF16)
        mn, pf = sn.sn_conv_workspace_query(s, sn.SN_CONV_BWD_FILTER, sn.SN_ALGO_STAGED)
        algo, used, _ = sn.sn_conv_plan(s, sn.SN_CONV_BWD_FILTER, 256 << 20)
        calls += [(sn.SN_CONV_BWD_FILTER, a, b, s) for a, b in ((sn.SN_ALGO_STAGED, mn), (sn.SN_ALGO_STAGED, pf), (algo, used))]
    sums = over = 0
    worst = None
    for (d, a, b, s), (status, launches) in zip(calls, recorded(calls)):
        assert status == 0
        for k, *_, reach in launches:
            sums += reach >= 0
            if reach > b:
                over += 1
                worst = worst or ([getattr(s, f) for f in FIELDS], a, b, reach)
    assert sums > 5000 and over == 0, (sums, over, worst)


def test_image_layers_take_the_faster_kernel(recorded):
    """Backward-filter of few input channels under a large filter: its own kernel where there is work for it, the general one where its
    start would be most of the time, and without partial sums fewer slices than compute units where the
    atomics of more would cost more than their rows."""
    sn.sn_planner_clear()
    D, S = sn.SN_ALGO_DIRECT, sn.SN_ALGO_STAGED
    want = [((128, 3, 227, 227, 96, 11, 4, 0), True, True), ((64, 3, 224, 224, 64, 7, 2, 3), True, True), ((32, 3, 32, 32, 64, 5, 1, 2), True, True),
            ((2, 3, 20, 20, 512, 11, 4, 5), False, False), ((6, 3, 44, 44, 256, 11, 1, 0), False, False), ((5, 1, 18, 18, 8, 7, 4, 0), False, True)]
    calls = []
    for (N, C, H, W, K, R, st, pad), _, _ in want:
        s = sn.conv_shape(N, C, H, W, K, R, R, (st, st), (pad, pad), sn.SN_BF16, sn.SN_BF16)
        calls += [(sn.SN_CONV_BWD_FILTER, D, 0, s), (sn.SN_CONV_BWD_FILTER, S, sn.sn_conv_workspace_query(s, sn.SN_CONV_BWD_FILTER, S)[1] + 256, s)]
    res = recorded(calls)
    for i, (shape, direct, staged) in enumerate(want):
        for image, (status, launches) in zip((direct, staged), res[2 * i:2 * i + 2]):
            assert status == 0 and any("image_wgrad" in k[0] for k in launches) == image, (shape, launches)
    grid = [next(k[1] for k in launches if "image_wgrad" in k[0]) for _, launches in res[4:6]]
    assert grid[0][0] < grid[1][0] <= 256


def test_the_image_tests_run_every_kernel(recorded):
    sn.sn_planner_clear()
    calls = []
    for N, C, H, W, K, R, S, stride, pad in test_gpu_image.EVERY:
        s = sn.conv_shape(N, C, H, W, K, R, S, stride, pad, sn.SN_BF16, sn.SN_BF16)
        calls += [(sn.SN_CONV_BWD_FILTER, a, b, s) for a, b in
                  ((sn.SN_ALGO_DIRECT, 0), (sn.SN_ALGO_STAGED, sn.sn_conv_workspace_query(s, sn.SN_CONV_BWD_FILTER, sn.SN_ALGO_STAGED)[1]))]
    res = recorded(calls)
    for one in (res[0::2], res[1::2]):
        assert len({k[0] for _, launches in one for k in launches if "image_wgrad_kernel" in k[0]}) == 48


def test_every_kernel_is_given_the_lds_that_it_is_launched_with(recorded):
    """Beyond 64 KB dynamic LDS is enabled kernel by kernel, not for the first one of a family that a process runs."""
    sn.sn_planner_clear()
    rnd, calls = random.Random(3), []
    for _ in range(4000):
        few = rnd.random() < 0.7
        R, S = rnd.choice([(11, 11), (7, 7), (5, 5), (3, 3), (9, 12), (7, 3), (4, 8)] if few else [(3, 3), (1, 1), (5, 5), (1, 7), (7, 1)])
        st = rnd.choice([1, 2, 4])
        s = sn.conv_shape(rnd.choice([1, 8, 64]), rnd.randint(1, 4) if few else rnd.choice([16, 64, 128]), rnd.randint(R, 200), rnd.randint(S, 200),
                          rnd.choice([8, 64, 96, 200]), R, S, (st, st), rnd.choice([(0, 0), (R // 2, S // 2)]), sn.SN_BF16, sn.SN_BF16)
        for d in (sn.SN_CONV_FWD, sn.SN_CONV_BWD_DATA, sn.SN_CONV_BWD_FILTER):
            algo, used, _ = sn.sn_conv_plan(s, d, rnd.choice([0, 64 << 20]))
            calls.append((d, algo, used, s))
    large = {}
    for status, launches in recorded(calls):
        assert status == 0
        for kernel, _, _, lds, limit, _ in launches:
            if lds > 64 << 10:
                large[kernel] = min(limit - lds, large.get(kernel, 0))
    assert len(large) > 40 and all(room >= 0 for room in large.values()), [k for k, room in large.items() if room < 0]


def test_the_streaming_kernel_is_given_no_workspace(recorded):
    """Few reduction channels: where the kernel that writes no packed filter runs, none is asked for under either name."""
    sn.sn_planner_clear()
    calls = []
    for N, C, H, W, K in ((64, 64, 56, 56, 64), (32, 64, 224, 224, 64), (32, 32, 112, 112, 64)):
        s = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (1, 1), sn.SN_BF16, sn.SN_BF16)
        assert sn.sn_conv_workspace_query(s, sn.SN_CONV_FWD, sn.SN_ALGO_STAGED) == (0, 0)
        assert sn.sn_conv_plan(s, sn.SN_CONV_FWD, 256 << 20)[:2] == (sn.SN_ALGO_DIRECT, 0)
        calls += [(sn.SN_CONV_FWD, a, b, s) for a, b in ((sn.SN_ALGO_DIRECT, 0), (sn.SN_ALGO_STAGED, 0), (sn.SN_ALGO_STAGED, 1 << 20),
                                                         (sn.SN_ALGO_AUTO, 0), (sn.SN_ALGO_AUTO, 256 << 20))]
    for status, launches in recorded(calls):
        assert status == 0 and [re.sub(r"^\d+", "", k[0])[:15] for k in launches] == ["band3x3_kernelI"], launches


def test_small_fp32_layers_keep_their_kernel_with_workspace(recorded):
    """3x3 layers that one launch takes without workspace: no amount of it makes AUTO run WINOGRAD's four instead."""
    sn.sn_planner_clear()
    calls = []
    for N, C, H, W, K in ((1, 128, 7, 7, 128), (2, 96, 8, 8, 96), (1, 256, 7, 7, 128), (1, 512, 4, 4, 200), (1, 1024, 5, 5, 8)):
        s = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (1, 1), sn.SN_F32, sn.SN_F32)
        calls += [(d, sn.SN_ALGO_AUTO, b, s) for d in (sn.SN_CONV_FWD, sn.SN_CONV_BWD_DATA) for b in (0, 32 << 20, 512 << 20)]
    for (d, _, b, s), (status, launches) in zip(calls, recorded(calls)):
        kernel = "small3x3_mfma_kernel" if (s.C if d == sn.SN_CONV_FWD else s.K) >= 16 else "small3x3_kernel"
        assert status == 0 and [kernel in k[0] for k in launches] == [True], (d, b, [getattr(s, f) for f in FIELDS], launches)


def test_small_layers_backward_filter_takes_the_faster_kernel(recorded):
    """With workspace: the one launch where the layer is small, the product over copies where it is the faster one (by 1.4 times on the
    shapes here: long sums on few compute units, or many workgroups on each)."""
    sn.sn_planner_clear()
    small = [(2, 16, 16, 16, 16, "f32"), (2, 16, 16, 16, 16, "bf16"), (1, 64, 8, 8, 64, "bf16"), (2, 80, 24, 24, 77, "bf16"), (4, 112, 5, 5, 240, "f32")]
    product = [(10, 16, 11, 26, 16, "bf16"), (3, 51, 26, 26, 384, "bf16"), (13, 40, 10, 10, 464, "bf16"), (1, 16, 38, 38, 64, "f32")]
    calls = []
    for N, C, H, W, K, dtype in small + product:
        t = sn.SN_BF16 if dtype == "bf16" else sn.SN_F32
        calls.append((sn.SN_CONV_BWD_FILTER, sn.SN_ALGO_AUTO, 64 << 20, sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (1, 1), t, t)))
    for i, (status, launches) in enumerate(recorded(calls)):
        one = [k[0] for k in launches if "small3x3_wgrad" in k[0]]
        assert status == 0 and (len(launches) == len(one) == 1 if i < len(small) else not one), ((small + product)[i], launches)


def test_small_bf16_layers_take_the_faster_kernel(recorded):
    """Forward and backward-data: the one launch on small layers; the tiles where there are few reduction channels and many outputs, the product
    over copies where it has the workspace and is the faster one (each side timed on these shapes: 1.2 to 1.4 times)."""
    sn.sn_planner_clear()
    F, D, AUTO = sn.SN_CONV_FWD, sn.SN_CONV_BWD_DATA, sn.SN_ALGO_AUTO
    STATS, NOALLOC = 3, 4
    want = [(F, AUTO, 0, (9, 16, 55, 26, 320, 1), "conv_tile_kernel"), (F, AUTO, 0, (12, 16, 33, 33, 304, 1), "conv_tile_kernel"),
            (D, AUTO, 0, (8, 360, 40, 40, 16, 1), "conv_tile_kernel"), (D, AUTO, 64 << 20, (2, 320, 53, 53, 48, 0), "cl_gemm_kernel"),
            (D, AUTO, 64 << 20, (3, 480, 37, 37, 23, 1), "cl_gemm_kernel"), (F, AUTO, 64 << 20, (4, 128, 13, 54, 288, 1), "cl_gemm_kernel"),
            (F, sn.SN_ALGO_STAGED, 8 << 20, (15, 32, 28, 28, 240, 1), "conv_tile2_kernel"), (NOALLOC, AUTO, 0, (15, 32, 28, 28, 240, 1), "conv_tile2_kernel"),
            (STATS, AUTO, 0, (4, 32, 57, 57, 256, 1), "conv_tile_kernel")]
    for d in (F, D, STATS):
        for b in (0, 64 << 20):
            want += [(d, AUTO, b, s, "small3x3_bf16_kernel") for s in ((2, 256, 14, 14, 256, 1), (8, 16, 16, 16, 16, 1), (1, 512, 7, 7, 512, 1))]
    calls = [(d, a, b, sn.conv_shape(s[0], s[1], s[2], s[3], s[4], 3, 3, (1, 1), (s[5], s[5]), sn.SN_BF16, sn.SN_BF16)) for d, a, b, s, _ in want]
    for w, (status, launches) in zip(want, recorded(calls)):
        assert status == 0 and any(w[4] in k[0] for k in launches), (w, launches)
        assert w[4] == "small3x3_bf16_kernel" or not any("small3x3" in k[0] for k in launches), (w, launches)


def test_small_calls_make_few_plans(recorded):
    """A plan of the channels-last product is 1 to 2 us of the host, as much as the rest of a call: none where the small layers' kernel is
    estimated below the least that the product is, one where both are weighed, and a named algorithm's least workspace asks for none."""
    sn.sn_planner_clear()
    F, D, B, AUTO, NOALLOC = sn.SN_CONV_FWD, sn.SN_CONV_BWD_DATA, sn.SN_CONV_BWD_FILTER, sn.SN_ALGO_AUTO, 4
    tiny, small, large = (8, 16, 16, 16, 16), (1, 512, 7, 7, 512), (32, 256, 56, 56, 256)
    most = [(F, AUTO, 64 << 20, tiny, 0), (D, AUTO, 64 << 20, tiny, 0), (B, AUTO, 64 << 20, (2, 64, 14, 14, 64), 0), (F, AUTO, 64 << 20, small, 1),
            (NOALLOC, 0, 0, small, 1), (NOALLOC, 0, 0, large, 1), (F, sn.SN_ALGO_STAGED, 64 << 20, large, 1), (D, sn.SN_ALGO_STAGED, 64 << 20, large, 1)]
    plans = []
    recorded([(d, a, b, sn.conv_shape(*s, 3, 3, (1, 1), (1, 1), sn.SN_BF16, sn.SN_BF16)) for d, a, b, s, _ in most], plans)
    assert all(n <= m[4] for n, m in zip(plans, most)), list(zip(plans, most))


def test_the_call_that_allocates_nothing_takes_the_faster_kernel(recorded):
    """No measurement chooses for it: small layers run as one launch also on whole blocks of 64 channels, where STAGED by its name keeps the
    channels-last product with the same workspace."""
    sn.sn_planner_clear()
    shapes = [(4, 64, 14, 14, 128), (1, 64, 28, 28, 64), (16, 64, 9, 9, 40)]
    calls = [(d, sn.SN_ALGO_STAGED, sn.SN_NOALLOC_SCRATCH_BYTES, sn.conv_shape(*s, 3, 3, (1, 1), (1, 1), sn.SN_BF16, sn.SN_BF16))
             for s in shapes for d in (sn.SN_CONV_FWD, 4)]
    res = recorded(calls)
    for i, s in enumerate(shapes):
        (status, named), (status4, noalloc) = res[2 * i:2 * i + 2]
        assert status == status4 == 0 and "cl_gemm_kernel" in named[1][0], (s, named)
        assert len(noalloc) == 1 and "small3x3_bf16_kernel" in noalloc[0][0], (s, noalloc)


def _kernels(res):
    assert all(status == 0 for status, _ in res)
    return [re.sub(r"^\d+", "", launches[0][0]).split("EvP")[0] for _, launches in res]


def test_the_image_forward_tests_run_every_kernel(recorded):
    """One to three channel tiles, blocks 64 and 32 columns wide, operands on 4 and 8 bytes."""
    sn.sn_planner_clear()
    shapes = [sn.conv_shape(N, C, H, W, K, R, S, (sh, sw), (ph, pw), sn.SN_BF16, sn.SN_BF16)
              for N, C, H, W, K, R, S, sh, sw, ph, pw in test_gpu_image_fwd.SHAPES]
    names = _kernels(recorded([(sn.SN_CONV_FWD, sn.SN_ALGO_DIRECT, 0, s) for s in shapes]))
    assert all(n.startswith("image_fwd_kernel") for n in names) and len(set(names)) == 12, sorted(set(names))


def test_the_small_layers_tests_run_the_kernels_that_they_name(recorded):
    """As DIRECT, bf16 forward and backward-data on either tile, forward with the filter loaded by lane and together; the fp32 kernels on either
    side of 16 reduction channels; backward-filter in both types."""
    sn.sn_planner_clear()
    F, D, B, direct = sn.SN_CONV_FWD, sn.SN_CONV_BWD_DATA, sn.SN_CONV_BWD_FILTER, sn.SN_ALGO_DIRECT
    call = lambda d, s, t: (d, direct, 0, sn.conv_shape(*s[:5], 3, 3, (1, 1), (s[5], s[-1]), t, t))
    names = _kernels(recorded([call(d, s, sn.SN_BF16) for s in test_gpu_small_bf16.SHAPES for d in (F, D)]))
    assert all(n.startswith("small3x3_bf16_kernel") for n in names) and len(set(names)) == 6, sorted(set(names))
    shapes = test_gpu_small3x3_mfma.SHAPES
    names = _kernels(recorded([call(d, s, sn.SN_F32) for s in shapes for d in (F, D)]))
    for n, red in zip(names, [c for s in shapes for c in (s[1], s[4])]):
        assert n.startswith("small3x3_mfma_kernel" if red >= 16 else "small3x3_kernel"), (n, red)
    names = _kernels(recorded([call(B, s, t) for s in test_gpu_small_wgrad.SHAPES for t in (sn.SN_BF16, sn.SN_F32)]))
    assert all(n.startswith("small3x3_wgrad_kernel") for n in names) and len(set(names)) == 2, sorted(set(names))
