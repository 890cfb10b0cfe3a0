"""Which kernel a GEMM takes and with what grid: the launchers' host code over a recording stand-in for the HIP runtime."""
import os
import random
import re
import subprocess

import pytest

from paper_2508_07329_amd import build as hip_build
from tests.tile_sizes import DENSE_TILES, STREAM_ROWS, TALL_GROUPS

LINEAR, SWIGLU, LINEAR_ASYM, SWIGLU_ASYM = range(4)
F16_ROWS, COLUMN_MAXIMA = -1, -2
HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
         "-I", os.path.join(hip_build.ROOT, "include"), "-I", hip_build.CSRC]


def _host_program(out, tag, sources, defines=()):
    """An executable of the sources' host code; the device code and the HIP runtime that it refers to do not exist."""
    objs = []
    for src in sources:
        objs.append(str(out / (os.path.basename(src) + tag + ".o")))
        subprocess.run([*HIPCC, *defines, "-c", "-x", "hip", src, "-o", objs[-1]], check=True)
    exe = str(out / ("prog" + tag))
    subprocess.run(["g++", *objs, "-o", exe, "-pthread", "-no-pie", "-Wl,--unresolved-symbols=ignore-all"], check=True)
    return exe


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    """plan(problems, *defines) -> [(kernel, its integer template arguments, work-groups)]; a problem is
    (epi, M, N, K, n_sel, max_rows, which, acc_dbg)."""
    out = tmp_path_factory.mktemp("plan")
    sources = [os.path.join(hip_build.CSRC, "gemm.hip"), os.path.join(hip_build.CSRC, "skinny.hip"), os.path.join(hip_build.CSRC, "quant.hip"),
               os.path.join(HERE, "launch_recorder.cpp")]
    built = {}

    def run(problems, *defines):
        if defines not in built:
            built[defines] = _host_program(out, str(len(built)), sources, defines)
        text = "".join(" ".join(map(str, p)) + "\n" for p in problems)
        lines = subprocess.run([built[defines]], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.splitlines()
        assert len(lines) == len(problems)
        res = []
        for line in lines:
            name, grid = line.split()
            m = re.search(r"(gemm_i8|skinny_linear|stream_linear|stream_grouped|fused_linear|weight_col_absmax|none)_kernel", name)
            res.append((m.group(1), [int(v) for v in re.findall(r"L[ib](\d+)E", name)], int(grid)))
        return res

    return run


WIDE_MAIN_TILE = ("-DHAQ_BM=256", "-DHAQ_BN=256", "-DHAQ_MINB=1", "-DHAQ_STAGES=3", "-DHAQ_WAVES_M=4")


@pytest.mark.parametrize("defines", [(), WIDE_MAIN_TILE], ids=["default", "256-row main tile"])
def test_every_tile_has_a_work_group(plan, defines):
    """Single matrices and expert groups of random sizes, also when the main tile is overridden at compile time."""
    rng = random.Random(7)
    problems, groups = [], []
    for _ in range(600):
        K = rng.choice((64, 512, 2048, 4096, 14336))
        if rng.random() < 0.5:
            M, N = int(2 ** rng.uniform(0, 12.5)), 16 * int(2 ** rng.uniform(0, 12))
            problems.append((rng.choice((LINEAR, LINEAR_ASYM)), M, N, K, 0, 0, 0, int(rng.random() < 0.1)))
            groups.append([M])
        else:
            which, N = rng.randrange(2), 64 * int(2 ** rng.uniform(0, 8))
            m = [int(2 ** rng.uniform(0, 9.5)) - 1 for _ in range(rng.randrange(1, 17))]
            epi = rng.choice((LINEAR, LINEAR_ASYM) if which else (SWIGLU, SWIGLU_ASYM))
            problems.append((epi, 0, N, K, len(m), sum(m) + rng.randrange(3), which, 0))
            groups.append(m)
    for p, m, (kernel, t, grid) in zip(problems, groups, plan(problems, *defines)):
        N, cd = p[2], lambda a, b: -(-a // b)
        if kernel == "gemm_i8":
            bm, bn, few = t[0], t[1], t[8]
            need = sum(cd(x, bm) for x in m) * (cd(cd(N, bn), 8) * 8 if few else cd(N, bn))
        elif kernel == "stream_grouped":
            need = sum(cd(x, 128) for x in m) * cd(N // 64, 8) * 8
        elif kernel == "stream_linear":
            need = cd(m[0], 16 * t[0]) * cd(N, 64)
        else:
            assert m[0] <= 16 * t[1]
            need = cd(N, 16 * t[0])
        assert grid >= need, (p, m, kernel, t, grid, need)
        assert kernel in ("skinny_linear", "stream_grouped") or grid % 8 == 0


def test_short_batches_leave_the_streaming_kernel_where_it_was_slower(plan):
    """Layers whose 64-channel units need several rounds of work-groups with too few K-steps, or too many rows, to carry
    them: up to 2.2 times slower there than the tiled kernel.  And the sizes next to them, where it is faster."""
    tiled = [(16, 768, 65536), (17, 768, 24576), (32, 1536, 65536), (33, 1536, 24576), (64, 1024, 50272), (64, 4096, 50272),
             (65, 512, 16384), (128, 768, 16384), (96, 4096, 24576), (96, 8192, 24576), (128, 512, 16384), (128, 1024, 65536), (100, 768, 50272),
             (16, 1024, 50272), (15, 848, 37168), (32, 2048, 24576), (23, 1536, 37840), (32, 2048, 65536), (33, 4096, 50272), (64, 2048, 32768), (96, 768, 16384), (128, 1024, 16384)]
    skinny = [(1, 512, 16384), (16, 1024, 32768), (16, 1472, 50272), (3, 1456, 33872), (9, 896, 40960), (32, 2176, 24576), (19, 5008, 41616), (29, 2560, 41072), (33, 4096, 16384), (64, 512, 16384), (96, 1104, 16384),
              (128, 1168, 16384), (128, 16384, 4096), (128, 4096, 4096), (1, 768, 3072), (128, 512, 512)]
    rows64 = [(65, 512, 6144), (128, 1024, 8176), (96, 4096, 8192), (128, 8192, 8192)]  # two row tiles of 64 rows, one round
    for epi in (LINEAR, LINEAR_ASYM):
        of = lambda sizes: plan([(epi, M, N, K, 0, 0, 0, 0) for M, K, N in sizes])
        for p, (kernel, t, _) in zip(tiled, of(tiled)):
            assert kernel == "gemm_i8" and t[0] == 128, (p, kernel, t)  # 256-row tiles would be half empty
        assert all(kernel == "skinny_linear" for kernel, _, _ in of(skinny)), of(skinny)
        assert all(kernel == "stream_linear" and t[0] == 4 for kernel, t, _ in of(rows64)), of(rows64)


def test_one_launch_linears_only_where_a_second_work_group_on_a_cu_pays(plan):
    """(rows, K, channels): up to 26 % slower than the two launches where it did not."""
    one = [(16, 768, 3072), (16, 1024, 16384), (1, 8192, 4096), (16, 16, 4096), (2, 8192, 8192),  # a work-group for each CU
           (16, 288, 8176), (8, 2048, 8176), (2, 8192, 8176), (16, 288, 32768), (16, 1024, 32768)]
    two = [(16, 16, 4112), (1, 16, 8176), (8, 272, 8176), (8, 1040, 16400), (8, 2048, 32768), (2, 8192, 32768), (16, 272, 16400),
           (17, 768, 3072), (9, 1040, 512), (3, 4112, 512), (1, 8208, 512), (16, 1024, 32784)]
    of = lambda sizes: [k for k, _, _ in plan([(F16_ROWS, M, N, K, 0, 0, 0, 0) for M, K, N in sizes])]
    assert set(of(one)) == {"fused_linear"} and set(of(two)) == {"none"}, (of(one), of(two))


def test_column_maxima_of_small_weights_in_short_stretches(plan):
    """(K, channels, work-groups): eight rows to each where there are few, 64 where there are two for each CU."""
    sizes = [(64, 16, 8), (63, 16, 8), (8, 16, 1), (1, 16, 1), (256, 256, 32), (768, 768, 3 * 96), (4096, 4096, 16 * 64), (64, 65536, 256 * 2), (65535, 16, 1024)]
    assert [g for _, _, g in plan([(COLUMN_MAXIMA, 0, N, K, 0, 0, 0, 0) for K, N, _ in sizes])] == [g for _, _, g in sizes]


def test_streaming_row_tiles_only_where_k_steps_carry_their_start_and_end(plan):
    tiled = [(333, 512, 4096), (512, 512, 4096), (512, 768, 3072), (640, 768, 3072), (777, 4096, 4096), (333, 2048, 8192),
             (400, 768, 3072), (512, 1024, 4096), (300, 8192, 8192), (170, 4352, 10304), (185, 5872, 8800), (700, 16384, 4096)]
    stream = [(256, 512, 4096), (333, 16384, 4096), (512, 16384, 4096), (1024, 3072, 768)]
    for epi in (LINEAR, LINEAR_ASYM):
        of = lambda sizes: [k for k, _, _ in plan([(epi, M, N, K, 0, 0, 0, 0) for M, K, N in sizes])]
        assert set(of(tiled)) == {"gemm_i8"} and set(of(stream)) == {"stream_linear"}, (of(tiled), of(stream))


def test_dense_tile_shapes_by_rows_channels_and_k(plan):
    """Each shape at sizes where it measured the fastest or within 3 % of it, and 64-bit addresses from 4 GB on."""
    best = {(128, 128): [(512, 8192, 8192), (1024, 16384, 4096), (333, 2048, 8192), (200, 4096, 11008), (1024, 768, 3072)],
            (192, 128): [(333, 4096, 16384), (600, 8192, 8192), (1300, 16384, 4096), (1536, 4096, 4096)],
            (192, 256): [(1300, 2048, 8192), (600, 4096, 16384), (3000, 16384, 4096), (777, 4096, 11008)],
            (256, 256): [(2048, 4096, 16384), (1024, 5120, 13824), (4096, 8192, 8192), (4096, 4096, 4096)],
            (128, 256): [(1306, 6672, 11472), (529, 1024, 23264), (2671, 14560, 5920)],
            (256, 128): [(2048, 16384, 4096), (418, 864, 10352), (708, 1328, 9312), (2559, 816, 2160), (1130, 3456, 5424), (3887, 7808, 1552)]}
    thrice = [(617, 608, 13936), (879, 544, 12704), (1366, 576, 8112)]  # 128 x 128, three work-groups to a CU
    for epi in (LINEAR, LINEAR_ASYM):
        for shape, sizes in best.items():
            for p, (kernel, t, _) in zip(sizes, plan([(epi, M, N, K, 0, 0, 0, 0) for M, K, N in sizes])):
                assert (kernel, tuple(t[:2]), t[9]) == ("gemm_i8", shape, 0), (p, kernel, t)
        assert [t[:2] + [t[5]] for _, t, _ in plan([(epi, M, N, K, 0, 0, 0, 0) for M, K, N in thrice])] == [[128, 128, 3]] * 3
        assert [t[9] for _, t, _ in plan([(epi, M, N, K, 0, 0, 0, 0) for M, N, K in [(128, 16384, 512), (192, 24576, 4096), (193, 24576, 4096)]])] == [2, 2, 0]
        edge = [(300, 2 ** 22 - 256, 1024), (300, 2 ** 22, 1024), (2 ** 22, 300, 1024), (2 ** 22 - 1024, 300, 1024), (300, 2 ** 22, 1025)]
        assert [t[9] for _, t, _ in plan([(epi, M, N, K, 0, 0, 0, 0) for M, N, K in edge])] == [0, 1, 1, 0, 1]
        assert [t[9] for _, t, _ in plan([(epi, M, N, K, 0, 0, 0, 1) for M, N, K in edge])] == [0, 1, 1, 0, 1]  # with the accumulators


def test_sizes_of_the_gpu_tests_take_the_tiles_that_they_are_for(plan):
    for epi in (LINEAR, LINEAR_ASYM):
        for shape, sizes in DENSE_TILES.items():
            for p, (kernel, t, _) in zip(sizes, plan([(epi, M, N, K, 0, 0, 0, 0) for M, K, N in sizes])):
                assert kernel == "gemm_i8" and (t[0], t[1], t[5]) == shape, (p, kernel, t)
        for rb, sizes in STREAM_ROWS.items():
            for p, (kernel, t, _) in zip(sizes, plan([(epi, M, N, K, 0, 0, 0, 0) for M, K, N in sizes])):
                assert kernel == "stream_linear" and t[0] == rb, (p, kernel, t)
        groups = [(epi, 0, H, I, len(first) + len(second), sum(first) + sum(second), 1, 0) for H, I, first, second in TALL_GROUPS]
        for p, (kernel, t, _) in zip(groups, plan(groups)):
            assert kernel == "gemm_i8" and t[:2] == [192, 256], (p, kernel, t)


def test_projections_of_expert_groups_on_either_side_of_their_lines(plan):
    """(experts, channels, K, rows for each): 192 x 256 tiles of down projections, 128 x 128 tiles of gate/up projections and
    weights that pass the caches by."""
    tall = [(8, 4096, 14336, 256), (8, 4096, 14336, 512), (8, 4096, 14336, 1024), (16, 2048, 5632, 512)]
    flat = [(8, 4096, 14336, 128), (8, 4096, 14336, 194), (16, 2048, 5632, 300), (8, 1024, 3584, 600),
            # few K-steps in several rounds
            (16, 6016, 704, 177), (8, 5952, 3712, 437), (8, 3648, 832, 930), (16, 5184, 512, 316), (16, 5888, 1728, 428)]
    for epi in (LINEAR, LINEAR_ASYM):
        of = lambda sizes: [(k, t[:2], t[8:10]) for k, t, _ in plan([(epi, 0, N, K, n, n * rows, 1, 0) for n, N, K, rows in sizes])]
        assert all(r == ("gemm_i8", [192, 256], [0, 0]) for r in of(tall)), of(tall)
        assert all(r == ("gemm_i8", [128, 256], [0, 0]) for r in of(flat)), of(flat)
        assert of([(8, 4096, 14336, 75)]) == [("gemm_i8", [128, 128], [0, 2])]
        assert of([(4, 2048, 8192, 300), (4, 4096, 14336, 128)]) == [("gemm_i8", [128, 128], [0, 0])] * 2  # several row tiles to a group
    for epi in (SWIGLU, SWIGLU_ASYM):
        of = lambda rows: [(k, t[:2], t[8:10]) for k, t, _ in plan([(epi, 0, 28672, 4096, 8, 8 * r, 0, 0) for r in rows])]
        assert of([9, 32]) == [("gemm_i8", [128, 128], [1, 0])] * 2 and of([33, 112]) == [("gemm_i8", [128, 256], [1, 0])] * 2
        assert of([113, 1024]) == [("gemm_i8", [128, 256], [0, 0])] * 2
        # (experts, hidden and intermediate channels, rows for each): few K-steps carry 128 x 128 tiles where they are few
        few_k = [(32, 128, 12672, 4), (32, 512, 9984, 7), (32, 384, 4032, 14), (32, 1472, 11648, 1), (16, 1728, 11648, 8), (16, 128, 2624, 8)]
        short = [(8, 2048, 10944, 16), (16, 768, 1216, 10), (4, 64, 576, 32), (16, 128, 2560, 8), (12, 1408, 6464, 26), (32, 1856, 4096, 1), (6, 1152, 11584, 11), (32, 2112, 5696, 4)]
        of = lambda sizes: [t[:2] + t[8:9] for _, t, _ in plan([(epi, 0, 2 * I, H, n, n * r, 0, 0) for n, H, I, r in sizes])]
        assert of(few_k) == [[128, 256, 1]] * len(few_k) and of(short) == [[128, 128, 1]] * len(short)


def test_group_tiles_are_dealt_once_and_evenly(tmp_path):
    """Every tile of every group once, all row tiles of a channel tile on one XCD; with one row tile for each group the
    XCDs differ by one tile at most, whatever the number of channel tiles is."""
    exe = _host_program(tmp_path, "deal", [os.path.join(HERE, "group_tiles_check.cpp")])
    rng = random.Random(11)
    even = [(128, ntn, [rng.randrange(1, 129) for _ in range(n)]) for ntn in (1, 5, 7, 8, 9, 12, 14, 44, 64) for n in (1, 4, 8, 17, 32)]
    mixed = [(rng.choice((128, 256)), rng.randrange(1, 113), [rng.choice((0, 1, rng.randrange(700))) for _ in range(rng.randrange(1, 33))])
             for _ in range(300)]
    text = "".join(f"{bm} {ntn} {len(rows)} {' '.join(map(str, rows))}\n" for bm, ntn, rows in even + mixed)
    lines = subprocess.run([exe], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.splitlines()
    assert len(lines) == len(even + mixed)
    for p, line in zip(even + mixed, lines):
        assert line.startswith("covered"), (p, line)
    for p, line in zip(even, lines):
        lo, hi = map(int, line.split()[1:])
        assert hi - lo <= 1, (p, lo, hi)


def test_down_projections_of_expert_groups_by_units_and_rows(plan):
    """(experts, channels, K, rows for each) on both sides of the lines between the streaming kernel, 128 x 128 tiles and the
    tiled form for few rows; each projection's epilogue in both codes."""
    stream = [(8, 4096, 14336, 64), (16, 2048, 5632, 64), (4, 4096, 14336, 104), (8, 3072, 14336, 112), (8, 1024, 3584, 112),
              (8, 4096, 14336, 24), (8, 4096, 14336, 49), (16, 2048, 5632, 25), (16, 1344, 4416, 29), (8, 3072, 14336, 77), (8, 2048, 8192, 104),
              (16, 3072, 8192, 24), (16, 4096, 7168, 48), (1, 4096, 14336, 100)]
    small = [(8, 4096, 14336, 65), (8, 4096, 14336, 104), (8, 3584, 8192, 112), (16, 2048, 5632, 80), (4, 4096, 14336, 128),
             (4, 4096, 14336, 112), (8, 2048, 8192, 112), (8, 4096, 14336, 25), (8, 4096, 14336, 48), (8, 3072, 14336, 76), (8, 3584, 8192, 36)]
    few = [(8, 4096, 14336, 105), (16, 3072, 8192, 25), (16, 2560, 5632, 112), (16, 4096, 7168, 49), (16, 2112, 3008, 56)]
    many = [(8, 3584, 8192, 128), (8, 3072, 14336, 113), (16, 1536, 6144, 128), (8, 4096, 14336, 113)]
    for epi in (LINEAR, LINEAR_ASYM):
        of = lambda sizes: plan([(epi, 0, N, K, n, n * rows, 1, 0) for n, N, K, rows in sizes])
        assert {k for k, _, _ in of(stream)} == {"stream_grouped"}, of(stream)
        for sizes, bn, is_few in ((small, 128, 0), (few, 256, 1), (many, 256, 0)):
            for p, (kernel, t, _) in zip(sizes, of(sizes)):
                assert (kernel, t[:2], t[8]) == ("gemm_i8", [128, bn], is_few), (p, kernel, t)
