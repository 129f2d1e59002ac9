"""CPU-only property tests of the planner against brute force on made-up timing
tables (Sec. 3.5: skip the algorithms that need more memory than is free, take
the fastest of the rest; more workspace never makes the plan slower)."""
import ctypes
import itertools
import random
import time

import paper_1801_04380_amd as sn
from paper_1801_04380_amd import _lib

DIRS = (sn.SN_CONV_FWD, sn.SN_CONV_BWD_DATA, sn.SN_CONV_BWD_FILTER)
ALGOS = (sn.SN_ALGO_DIRECT, sn.SN_ALGO_IM2COL_GEMM, sn.SN_ALGO_STAGED, sn.SN_ALGO_WINOGRAD)


def _needs(shape, d):
    out = {}
    for a in ALGOS:
        try:
            out[a] = sn.sn_conv_workspace_query(shape, d, a)
        except sn.SnError as e:
            assert e.status == 2
    return out


def test_cold_start_ranking_is_always_feasible():
    sn.sn_planner_clear()
    shape = sn.conv_shape(8, 64, 28, 28, 64, 3, 3, (1, 1), (1, 1), sn.SN_BF16, sn.SN_BF16)
    for d in DIRS:
        needs = _needs(shape, d)
        for budget in (0, 255, 256, 1 << 16, 1 << 22, 1 << 34):
            algo, used, ms = sn.sn_conv_plan(shape, d, budget)
            assert ms is None
            assert algo in needs and needs[algo][0] <= budget and used <= budget
        assert sn.sn_conv_plan(shape, d, 0)[0] == sn.SN_ALGO_DIRECT


def test_fastest_feasible_matches_brute_force():
    rnd = random.Random(5)
    shape = sn.conv_shape(4, 32, 20, 20, 48, 3, 3, (1, 1), (1, 1), sn.SN_BF16, sn.SN_F32)
    other = sn.conv_shape(4, 32, 20, 20, 48, 3, 3, (2, 2), (1, 1), sn.SN_BF16, sn.SN_F32)
    for trial in range(20):
        sn.sn_planner_clear()
        table = []
        for d in DIRS:
            needs = _needs(shape, d)
            for a, (mn, pf) in needs.items():
                for ws in sorted({mn, pf, (mn + pf) // 2}):
                    if rnd.random() < 0.8:
                        ms = round(rnd.uniform(0.1, 5.0), 3)
                        sn.sn_planner_record(shape, d, a, ws, ms)
                        table.append((d, a, ws, ms))
        # records of another shape must not leak in
        sn.sn_planner_record(other, sn.SN_CONV_FWD, sn.SN_ALGO_DIRECT, 0, 0.001)
        for d in DIRS:
            rows = [r for r in table if r[0] == d]
            budgets = sorted({0, 1 << 40} | {r[2] for r in rows} | {max(r[2] - 1, 0) for r in rows})
            last = None
            for budget in budgets:
                feasible = [r for r in rows if r[2] <= budget]
                algo, used, ms = sn.sn_conv_plan(shape, d, budget)
                if feasible:
                    # the fastest; among the records within 3 % of it the smallest workspace, then the faster
                    fastest = min(r[3] for r in feasible)
                    near = [r for r in feasible if r[3] <= fastest * 1.03 + 1e-9]
                    best = min(near, key=lambda r: (r[2], r[3]))
                    assert abs(ms - best[3]) < 1e-6 and used == best[2] and algo == best[1], (trial, d, budget)
                    assert ms <= fastest * 1.03 + 1e-6
                    if last is not None:
                        assert fastest <= last + 1e-6   # a bigger budget never makes the fastest feasible step slower
                    last = fastest
                else:
                    assert ms is None and used <= budget
    sn.sn_planner_clear()


def test_record_rejects_infeasible_measurements():
    shape = sn.conv_shape(2, 16, 16, 16, 16, 3, 3, (1, 1), (1, 1))
    mn, _ = sn.sn_conv_workspace_query(shape, sn.SN_CONV_FWD, sn.SN_ALGO_IM2COL_GEMM)
    try:
        sn.sn_planner_record(shape, sn.SN_CONV_FWD, sn.SN_ALGO_IM2COL_GEMM, mn - 1, 1.0)
        assert False
    except sn.SnError as e:
        assert e.status == 3
    try:
        sn.sn_planner_record(shape, sn.SN_CONV_FWD, sn.SN_ALGO_STAGED, 1 << 20, 1.0)
        assert False
    except sn.SnError as e:
        assert e.status == 2
    # overwriting a record keeps one entry
    sn.sn_planner_clear()
    sn.sn_planner_record(shape, sn.SN_CONV_FWD, sn.SN_ALGO_DIRECT, 0, 2.0)
    sn.sn_planner_record(shape, sn.SN_CONV_FWD, sn.SN_ALGO_DIRECT, 0, 1.5)
    assert abs(sn.sn_conv_plan(shape, sn.SN_CONV_FWD, 0)[2] - 1.5) < 1e-6
    sn.sn_planner_clear()


def test_cold_start_on_strided_shapes_counts_the_passes():
    """Without measurements the phase planes are guessed only where they pay (Sec. 3.5 leaves the
    ranking to measurement; this is the stand-in before any exists): backward-data in at most
    two passes, forward only with the whole batch; the zero-workspace kernel otherwise (never the
    explicit algorithm, which is picked on measurement only)."""
    sn.sn_planner_clear()
    shape = sn.conv_shape(64, 128, 56, 56, 128, 3, 3, (2, 2), (1, 1), sn.SN_BF16, sn.SN_BF16)
    mn, pf = sn.sn_conv_workspace_query(shape, sn.SN_CONV_BWD_DATA, sn.SN_ALGO_STAGED)
    assert mn < pf                                     # one image's planes up to the whole batch
    per_image = (pf - mn) // 63
    assert sn.sn_conv_plan(shape, sn.SN_CONV_BWD_DATA, pf)[0] == sn.SN_ALGO_STAGED
    assert sn.sn_conv_plan(shape, sn.SN_CONV_BWD_DATA, mn + 31 * per_image)[0] == sn.SN_ALGO_STAGED     # 32 images: 2 passes
    algo, used, _ = sn.sn_conv_plan(shape, sn.SN_CONV_BWD_DATA, mn + 30 * per_image)                   # 31 images: 3 passes
    assert algo == sn.SN_ALGO_DIRECT and used == 0
    assert sn.sn_conv_plan(shape, sn.SN_CONV_BWD_DATA, 4096)[0] == sn.SN_ALGO_DIRECT
    fmn, fpf = sn.sn_conv_workspace_query(shape, sn.SN_CONV_FWD, sn.SN_ALGO_STAGED)
    assert sn.sn_conv_plan(shape, sn.SN_CONV_FWD, fpf)[0] == sn.SN_ALGO_STAGED
    assert sn.sn_conv_plan(shape, sn.SN_CONV_FWD, fpf - 256)[0] == sn.SN_ALGO_DIRECT


def test_backward_filter_workspace_is_a_range():
    """STAGED backward-filter on the row-stationary kernel runs with a quarter of its slices upward
    (Sec. 3.5: the more workspace, the faster); without measurements the planner guesses it down to
    half of them and the zero-workspace form below that."""
    sn.sn_planner_clear()
    shape = sn.conv_shape(64, 96, 35, 35, 96, 3, 3, (1, 1), (1, 1), sn.SN_BF16, sn.SN_BF16)
    mn, pf = sn.sn_conv_workspace_query(shape, sn.SN_CONV_BWD_FILTER, sn.SN_ALGO_STAGED)
    per = 96 * 96 * 9 * 4
    assert 0 < mn < pf and pf % per < 256 and mn <= pf // 4 + per + 256
    algo, used, _ = sn.sn_conv_plan(shape, sn.SN_CONV_BWD_FILTER, pf)
    assert algo == sn.SN_ALGO_STAGED and used == pf
    half = mn + (pf - mn) // 3
    algo, used, _ = sn.sn_conv_plan(shape, sn.SN_CONV_BWD_FILTER, half + per)
    assert algo == sn.SN_ALGO_STAGED and used == half + per
    assert sn.sn_conv_plan(shape, sn.SN_CONV_BWD_FILTER, half - per)[0] == sn.SN_ALGO_DIRECT
    assert sn.sn_conv_plan(shape, sn.SN_CONV_BWD_FILTER, mn - 256)[0] == sn.SN_ALGO_DIRECT


def _random_shape(rnd):
    dt = rnd.choice((sn.SN_F32, sn.SN_BF16))
    R, S = rnd.choice(((1, 1), (3, 3), (3, 3), (5, 5), (7, 7), (1, 7), (7, 1), (4, 3), (11, 11)))
    stride = rnd.choice(((1, 1), (1, 1), (2, 2), (2, 2), (3, 2), (4, 4)))
    pad = rnd.choice(((0, 0), ((R - 1) // 2, (S - 1) // 2)))
    H, W = (rnd.randint(max(R, S), 64) for _ in range(2))
    C, K = (rnd.choice((3, 8, 24, 64, 160, 288, rnd.randint(1, 400))) for _ in range(2))
    return sn.conv_shape(rnd.choice((1, 2, 9, 32, 61)), C, H, W, K, R, S, stride, pad, dt, dt)


def test_planned_calls_are_accepted_with_the_bytes_planned():
    """What sn_conv_plan hands out can be called: bytes_used is at least the named algorithm's least workspace and at most
    the budget, and planning again with it as the budget names the same algorithm with the same bytes."""
    sn.sn_planner_clear()
    rnd = random.Random(11)
    named = {a: 0 for a in ALGOS}
    for _ in range(4000):
        shape, d = _random_shape(rnd), rnd.choice(DIRS)
        budget = rnd.choice((1 << 18, 1 << 22, 32 << 20, 64 << 20, 512 << 20))
        algo, used, _ = sn.sn_conv_plan(shape, d, budget)
        mn, pf = sn.sn_conv_workspace_query(shape, d, algo)
        case = ([getattr(shape, f) for f, _ in shape._fields_], d, budget, algo, used, mn, pf)
        assert mn <= used <= budget and mn <= pf, case
        again = sn.sn_conv_plan(shape, d, used)
        assert again[:2] == (algo, used), case + again
        named[algo] += 1
    assert all(named.values()), named


def test_strided_backward_data_is_given_its_planes():
    """Where the phase planes run (the channels-last product is not estimated to be faster), the workspace reported and
    planned holds the planes of the whole batch -- dx once over -- so that they run in one pass."""
    sn.sn_planner_clear()
    for N, C, H, K in ((52, 240, 16, 64), (9, 96, 32, 64)):
        shape = sn.conv_shape(N, C, H, H, K, 3, 3, (2, 2), (1, 1), sn.SN_BF16, sn.SN_BF16)
        _, pf = sn.sn_conv_workspace_query(shape, sn.SN_CONV_BWD_DATA, sn.SN_ALGO_STAGED)
        algo, used, _ = sn.sn_conv_plan(shape, sn.SN_CONV_BWD_DATA, 512 << 20)
        assert algo == sn.SN_ALGO_STAGED and used == pf >= N * C * H * H * 2


def test_cold_start_weighs_winograd_against_the_product():
    """fp32 3x3: WINOGRAD's fewer products win on many channels and tiles (8 x 256 x 56x56, 512 MiB: 230 us against 275), the
    product over channels-last copies, whose copies are cheaper than the transforms, on fewer (16 x 144 x 32x17 -> 312, 64 MiB:
    80 us against 108)."""
    sn.sn_planner_clear()
    for N, C, H, W, K, mib, algo in ((8, 256, 56, 56, 256, 512, sn.SN_ALGO_WINOGRAD), (4, 512, 61, 61, 512, 256, sn.SN_ALGO_WINOGRAD),
                                     (16, 144, 32, 17, 312, 64, sn.SN_ALGO_IM2COL_GEMM), (8, 64, 69, 69, 64, 512, sn.SN_ALGO_IM2COL_GEMM)):
        shape = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (1, 1), sn.SN_F32, sn.SN_F32)
        for d in (sn.SN_CONV_FWD, sn.SN_CONV_BWD_DATA):
            assert sn.sn_conv_plan(shape, d, mib << 20)[0] == algo, (N, C, H, d)


def test_backward_filters_own_kernels_have_a_workspace_that_names_them():
    """STAGED backward-filter's own kernels can take more workspace than the channels-last product; one unit beyond what they can
    use runs them, whatever the estimates say, so that they can be measured against it."""
    lib = _lib.load()
    info, used, us = (ctypes.c_int * 5)(), ctypes.c_size_t(), ctypes.c_double()
    rnd = random.Random(23)
    beyond = 0
    for _ in range(1000):
        shape = _random_shape(rnd)
        _, pf = sn.sn_conv_workspace_query(shape, sn.SN_CONV_BWD_FILTER, sn.SN_ALGO_STAGED)
        runs = [lib.sn_chlast_inspect(ctypes.byref(shape), sn.SN_CONV_BWD_FILTER, sn.SN_ALGO_STAGED, ctypes.c_size_t(b), info,
                                      ctypes.byref(used), ctypes.byref(us)) for b in (pf + 256, 1 << 32)]
        assert not runs[0]
        beyond += runs[1]
    assert beyond > 100   # (shapes whose STAGED is the product with more)


def test_more_output_channels_than_a_grid_has_rows():
    """The product's slice sums give every output channel a row of the grid, of which there are 65535: with more channels there
    are no slices, and no product for backward-filter."""
    lib = _lib.load()
    info, used, us = (ctypes.c_int * 5)(), ctypes.c_size_t(), ctypes.c_double()
    for K, R, dt in ((65535, 1, sn.SN_BF16), (65536, 1, sn.SN_BF16), (70000, 3, sn.SN_BF16), (70000, 3, sn.SN_F32)):
        shape = sn.conv_shape(1, 512, 5, 5, K, R, R, (1, 1), (R // 2, R // 2), dt, dt)
        for d in (sn.SN_CONV_FWD, sn.SN_CONV_BWD_FILTER):
            runs = lib.sn_chlast_inspect(ctypes.byref(shape), d, sn.SN_ALGO_IM2COL_GEMM, ctypes.c_size_t(1 << 34), info, ctypes.byref(used),
                                         ctypes.byref(us))
            assert runs == (d == sn.SN_CONV_FWD or K <= 65535), (K, d)
            assert not runs or K <= 65535 or info[3] == 1, (K, d, list(info))


def test_planning_a_tall_layer_takes_no_longer():
    """3x3 layers of few reduction channels: the rows are split into bands without trying every number of them."""
    sn.sn_planner_clear()
    us = {}
    for H, W in ((224, 224), (65536, 8)):
        shape = sn.conv_shape(1, 64, H, W, 64, 3, 3, (1, 1), (1, 1), sn.SN_BF16, sn.SN_BF16)
        runs = []
        for _ in range(9):
            t = time.perf_counter()
            for _ in range(50):
                sn.sn_conv_plan(shape, sn.SN_CONV_FWD, 64 << 20)
            runs.append(time.perf_counter() - t)
        us[H] = min(runs)
    assert us[65536] < 8 * us[224], us
